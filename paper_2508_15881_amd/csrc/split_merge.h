// Merge of the partial results of one (slice, sequence, head), shared by the stand-alone merge
// (decode_generic.hip) and the merge fused with the combine (absorb_combine_mfma.hip).
#pragma once
#include "tpla_internal.h"

namespace tpla {

// The partial-result slots of (slice, sequence) vb = slice * B + b: consecutive in both plans.
struct SlotRange {
  int first, cnt;
};
__device__ __forceinline__ SlotRange merge_slots(const DecodeArgs& a, int vb, int b) {
  if (a.balanced) return {a.plan[vb] + vb, a.plan[a.n_shards * a.B + vb]};   // left there by the split kernel
  const int n_pages = (seq_len_clipped(a, b) + a.page_tokens - 1) / a.page_tokens;
  return {vb * a.n_splits, min((n_pages + a.pages_per_split - 1) / a.pages_per_split, a.n_splits)};
}

// (reference, sum) of slot `first + s` for the lanes with s < s1; empty otherwise.
__device__ __forceinline__ float2 merge_load_ml(const DecodeArgs& a, int h, int first, int s, int s1) {
  float2 v = make_float2(-INFINITY, 0.f);
  if (s < s1) v = *reinterpret_cast<const float2*>(a.part_ml + ((size_t)(first + s) * a.H + h) * 2);
  return v;
}

// One wave merges `SW` = 256 / SUBS consecutive latent columns over the slots [s0, s1): 64 / SUBS lanes hold
// four columns each, lane group `sub` takes every SUBS-th slot.  A slot's row piece is then one contiguous
// read (1 KB for SUBS = 1) and its weight is the same for the whole group, 16 rows are in flight per
// wave, and the references of 64 slots are agreed on at once.  Result: sum of rows x weights relative to the
// reference M, and the sum of weights l (not normalised), the same in every lane group.
struct MergedPiece {
  f32x4 x;
  float M, l;
};

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) v = fmaxf(v, __shfl_xor(v, m));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m);
  return v;
}

template <int SUBS>
__device__ __forceinline__ float slot_weight(float w, int s, int sub) {
  if constexpr (SUBS == 1) return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), s));
  return __shfl(w, s + sub);
}

// N loads of this lane group's slots i, i + SUBS, ... of a block of n; slots past the end read the last one
// and count as zero rows (not as rows of weight zero: a row may hold infinities).
template <int SUBS, int N>
__device__ __forceinline__ void merge_rows(f32x4& x, const float* src, size_t stride, float w, int i, int n, int sub) {
  f32x4 p[N];
#pragma unroll
  for (int u = 0; u < N; ++u) p[u] = *reinterpret_cast<const f32x4*>(src + (size_t)min(i + u * SUBS + sub, n - 1) * stride);
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const bool live = i + u * SUBS + sub < n;
    const float ws = slot_weight<SUBS>(w, i + u * SUBS, sub);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = fmaf(live ? p[u][e] : 0.f, ws, x[e]);
  }
}

// ml0: merge_load_ml() of the first 64 slots (lane l: slot s0 + l), requested early by the caller.
template <int SUBS>
__device__ __forceinline__ MergedPiece merge_piece(const DecodeArgs& a, int h, int first, int s0, int s1, int col,
                                                   float2 ml0) {
  constexpr int LPR = 64 / SUBS, AHEAD = 16;
  const int lane = threadIdx.x & 63, sub = lane / LPR;
  const size_t stride = (size_t)a.H * a.dl;
  const float* src = a.part_acc + ((size_t)(first + s0) * a.H + h) * a.dl + col + 4 * (lane % LPR);
  MergedPiece r;
  r.x = f32x4{0.f, 0.f, 0.f, 0.f};
  r.M = -INFINITY;
  r.l = 0.f;
  for (int base = s0; base < s1; base += 64, src += 64 * stride) {
    const float2 ml = base == s0 ? ml0 : merge_load_ml(a, h, first, base + lane, s1);
    const float Mb = wave_max(ml.x);
    if (Mb == -INFINITY) continue;
    const float M_new = fmaxf(r.M, Mb);
    const float alpha = exp2f(r.M - M_new);            // 0 the first time
    const float w = exp2f(ml.x - M_new);               // 0 in the lanes past the last slot
    r.l = fmaf(r.l, alpha, wave_sum(ml.y * w));
    r.M = M_new;
    if (alpha != 1.0f) r.x *= alpha;
    const int n = min(64, s1 - base);
    int i = 0;
    for (; n - i > AHEAD * SUBS / 2; i += AHEAD * SUBS) merge_rows<SUBS, AHEAD>(r.x, src, stride, w, i, n, sub);
    if (n - i > AHEAD * SUBS / 4)
      merge_rows<SUBS, AHEAD / 2>(r.x, src, stride, w, i, n, sub);
    else if (n - i > 0)
      merge_rows<SUBS, AHEAD / 4>(r.x, src, stride, w, i, n, sub);
  }
#pragma unroll
  for (int m = LPR; m < 64; m <<= 1)
#pragma unroll
    for (int e = 0; e < 4; ++e) r.x[e] += __shfl_xor(r.x[e], m);
  return r;
}

// Adds what another wave merged from later slots of the same piece (in slot order, so the bits are fixed).
__device__ __forceinline__ void merge_join(MergedPiece& r, const f32x4& x, float M, float l) {
  if (M == -INFINITY) return;
  const float M_new = fmaxf(r.M, M);
  const float ra = exp2f(r.M - M_new), xa = exp2f(M - M_new);   // ra = 0 when nothing has been merged yet
  r.x = r.x * ra + x * xa;
  r.l = r.l * ra + l * xa;
  r.M = M_new;
}
__device__ __forceinline__ void merge_normalise(MergedPiece& r) {
  if (r.l > 0.f) r.x *= 1.0f / r.l;
}
__device__ __forceinline__ float merged_lse(const MergedPiece& r) {
  return r.l > 0.f ? (r.M + log2f(r.l)) * 0.6931471805599453f : -INFINITY;
}

// Columns that one wave merges at a time: the largest piece that divides a slice (0: this code does not apply).
__host__ __device__ __forceinline__ int merge_piece_width(int dl) {
  return dl % 256 == 0 ? 256 : dl % 128 == 0 ? 128 : dl % 64 == 0 ? 64 : 0;
}

}  // namespace tpla
