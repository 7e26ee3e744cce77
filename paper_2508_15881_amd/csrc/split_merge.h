// Merge of the partial results of one (slice, sequence, head), shared by the stand-alone merge
// (decode_generic.hip) and the merge fused with the combine (absorb_combine_mfma.hip).
#pragma once
#include "tpla_internal.h"

namespace tpla {

// The partial-result slots of (slice, sequence) vb[g] = slice * B + b[g]: consecutive in both plans.  All of a wave's
// at once, without a branch or a wait between the loads: each is a round trip to memory.
template <int G>
__device__ __forceinline__ void merge_slots(const DecodeArgs& a, const int (&vb)[G], const int (&b)[G], int (&first)[G], int (&cnt)[G]) {
  if (a.balanced) {                                    // left in the plan table by the split kernel
    const int n_v = a.n_shards * a.B;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      first[g] = a.plan[vb[g]];
      cnt[g] = a.plan[n_v + vb[g]];
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      first[g] = __builtin_amdgcn_readfirstlane(first[g]) + vb[g];
      cnt[g] = __builtin_amdgcn_readfirstlane(cnt[g]);
    }
  } else {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int n_pages = (seq_len_clipped(a, b[g]) + a.page_tokens - 1) / a.page_tokens;
      first[g] = vb[g] * a.n_splits;
      cnt[g] = __builtin_amdgcn_readfirstlane(min((n_pages + a.pages_per_split - 1) / a.pages_per_split, a.n_splits));
    }
  }
}

// (reference, sum) of slot `first + s` for the lanes with s < s1; empty otherwise.  (The address is clamped, not the load
// predicated: no branch.  Slot `first` of an empty sequence exists and is not looked at.)
__device__ __forceinline__ float2 merge_load_ml(const DecodeArgs& a, int h, int first, int s, int s1) {
  const float2 v = *reinterpret_cast<const float2*>(a.part_ml + ((size_t)(first + max(min(s, s1 - 1), 0)) * a.H + h) * 2);
  return s < s1 ? v : make_float2(-INFINITY, 0.f);
}

// A piece: SW = 256 / SUBS consecutive latent columns of one (slice, sequence, head), merged by one wave: 64 / SUBS
// lanes hold four columns each, lane group `sub` takes every SUBS-th slot.  A slot's row is then one contiguous
// read (1 KB for SUBS = 1) and its weight is the same for the whole group.  merge_piece() takes any number of
// slots, merge_short_pieces() several pieces of at most MERGE_SHORT slots at a time.
struct MergedPiece {
  f32x4 x;                 // sum of rows x weights relative to the reference M, the same in every lane group
  float M, l;              // reference and sum of the weights
};
// -inf says "empty": the sum is 0 there and nowhere else.  A sum that is NaN stays one.
__device__ __forceinline__ float merge_lse(float M, float l) { return l != 0.f ? (M + log2f(l)) * 0.6931471805599453f : -INFINITY; }

__device__ __forceinline__ float wave_max(float v) {
  const int lane = threadIdx.x & 63;
  v = fmaxf(v, lane_xor<1>(v, lane));
  v = fmaxf(v, lane_xor<2>(v, lane));
  v = fmaxf(v, lane_xor<4>(v, lane));
  v = fmaxf(v, lane_xor<8>(v, lane));
  v = fmaxf(v, lane_xor<16>(v, lane));
  return fmaxf(v, lane_xor<32>(v, lane));
}
__device__ __forceinline__ float wave_sum(float v) {
  const int lane = threadIdx.x & 63;
  v += lane_xor<1>(v, lane);
  v += lane_xor<2>(v, lane);
  v += lane_xor<4>(v, lane);
  v += lane_xor<8>(v, lane);
  v += lane_xor<16>(v, lane);
  return v + lane_xor<32>(v, lane);
}

template <int SUBS>
__device__ __forceinline__ float slot_weight(float w, int s, int sub) {
  if constexpr (SUBS == 1) return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), s));
  return __shfl(w, s + sub);
}

// N rows of this lane group, slots i, i + SUBS, ... of a block of n > 0; slots past the end read the last one and
// are added as zero rows (not as rows of weight zero: a row may hold infinities).  `base` is the same in all
// lanes and the rest of the address 32 bits wide (merge_piece_width): one register per row in flight.
template <int SUBS, int N>
__device__ __forceinline__ void merge_load_rows(f32x4 (&p)[N], const float* base, unsigned row_bytes, int i, int n, int sub) {
  const unsigned lane_bytes = 16u * ((threadIdx.x & 63) % (64 / SUBS));
#pragma unroll
  for (int u = 0; u < N; ++u)
    p[u] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(base) + ((unsigned)min(i + u * SUBS + sub, n - 1) * row_bytes + lane_bytes));
}
template <int SUBS, int N>
__device__ __forceinline__ void merge_add_rows(f32x4& x, const f32x4 (&p)[N], float w, int i, int n, int sub) {
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const bool live = i + u * SUBS + sub < n;
    const float ws = slot_weight<SUBS>(w, i + u * SUBS, sub);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = fmaf(live ? p[u][e] : 0.f, ws, x[e]);
  }
}
// Takes a block of 64 slots into the reference and the sum; returns the weight of this lane's slot.  A slot whose reference is
// -inf holds no finite score and a sum that is NaN (no slot: 0): the sum is kept, so that the result is NaN and not that of
// an empty sequence.
__device__ __forceinline__ float merge_weights(MergedPiece& r, float2 ml) {
  const float M_new = fmaxf(r.M, wave_max(ml.x));
  if (M_new == -INFINITY) {
    r.l += wave_sum(ml.y);
    return 0.f;
  }
  const float alpha = exp2f(r.M - M_new);              // 0 the first time
  const float w = exp2f(ml.x - M_new);                 // 0 in the lanes past the last slot
  r.l = fmaf(r.l, alpha, wave_sum(ml.y * w));
  r.M = M_new;
  if (alpha != 1.0f) r.x *= alpha;
  return w;
}

// Slots [s0, s1) of a piece; the references of 64 slots are agreed on at once, N rows per lane group are in flight.
template <int SUBS, int N = SUBS == 1 ? 8 : 4>
__device__ __forceinline__ MergedPiece merge_piece(const DecodeArgs& a, int h, int first, int s0, int s1, int col) {
  constexpr int LPR = 64 / SUBS;
  const int lane = threadIdx.x & 63, sub = lane / LPR;
  const unsigned stride = (unsigned)a.H * (unsigned)a.dl * 4u;
  MergedPiece r;
  r.x = f32x4{0.f, 0.f, 0.f, 0.f};
  r.M = -INFINITY;
  r.l = 0.f;
  for (int base = s0; base < s1; base += 64) {
    const int n = min(64, s1 - base);
    const float* src = a.part_acc + ((size_t)(first + base) * a.H + h) * a.dl + col;
    const float2 ml = merge_load_ml(a, h, first, base + lane, s1);
    f32x4 p[N];
    merge_load_rows<SUBS>(p, src, stride, 0, n, sub);
    const float w = merge_weights(r, ml);
    merge_add_rows<SUBS>(r.x, p, w, 0, n, sub);
    for (int i = N * SUBS; i < n; i += N * SUBS) {
      merge_load_rows<SUBS>(p, src, stride, i, n, sub);
      merge_add_rows<SUBS>(r.x, p, w, i, n, sub);
    }
  }
#pragma unroll
  for (int m = LPR; m < 64; m <<= 1)
#pragma unroll
    for (int e = 0; e < 4; ++e) r.x[e] += __shfl_xor(r.x[e], m);
  return r;
}

// G <= 4 pieces of at most 16 slots each (cnt 0: empty): the (reference, sum) pairs of all of them are one load --
// lane 16 g + s has slot s of piece g -- and one pass of arithmetic over 16-lane rows, so that what is left per
// piece are its rows.  The first A rows per lane of all pieces are in flight together.  x: normalised columns;
// lse: log-sum-exp of piece lane / 16.
constexpr int MERGE_SHORT = 16;
// The head whose (reference, sum) pair a lane reads.  Lanes past the last piece and pieces past the last head (their
// cnt is 0) repeat an existing one: part_ml may end there.
__host__ __device__ __forceinline__ int merge_short_head(int lane, int h, int hstep, int n_pieces, int H) {
  const int g = (lane >> 4) < n_pieces ? lane >> 4 : n_pieces - 1;
  return h + g * hstep < H ? h + g * hstep : H - 1;
}
template <int SUBS, int G, int A>
__device__ __forceinline__ void merge_short_pieces(const DecodeArgs& a, int h, int hstep, const int (&first)[G], const int (&cnt)[G],
                                                   const int (&col)[G], f32x4 (&x)[G], float& lse) {
  static_assert(G <= 4, "one row of 16 lanes per piece");
  constexpr int LPR = 64 / SUBS;
  const int lane = threadIdx.x & 63, sub = lane / LPR;
  const unsigned stride = (unsigned)a.H * (unsigned)a.dl * 4u;
  int first_l = first[0], cnt_l = cnt[0];
#pragma unroll
  for (int g = 1; g < G; ++g) {
    first_l = lane >= 16 * g ? first[g] : first_l;
    cnt_l = lane >= 16 * g ? cnt[g] : cnt_l;
  }
  if (lane >= 16 * G) cnt_l = 0;
  const float2 ml = merge_load_ml(a, merge_short_head(lane, h, hstep, G, a.H), first_l, lane & 15, cnt_l);
  f32x4 p[G][A];
  auto source = [&](int g) -> const float* {
    return a.part_acc + ((size_t)first[g] * a.H + h + g * hstep) * a.dl + col[g];
  };
#pragma unroll
  for (int g = 0; g < G; ++g)
    if (cnt[g] > 0) merge_load_rows<SUBS>(p[g], source(g), stride, 0, cnt[g], sub);
  float M = ml.x;
  M = fmaxf(M, lane_xor<1>(M, lane));
  M = fmaxf(M, lane_xor<2>(M, lane));
  M = fmaxf(M, lane_xor<4>(M, lane));
  M = fmaxf(M, lane_xor<8>(M, lane));
  float w = M == -INFINITY ? 0.f : exp2f(ml.x - M);        // 0 in the lanes past the last slot; M = -inf: see merge_weights
  float l = ml.y * w;
  l += lane_xor<1>(l, lane);
  l += lane_xor<2>(l, lane);
  l += lane_xor<4>(l, lane);
  l += lane_xor<8>(l, lane);
  lse = merge_lse(M, l);
  if (l != 0.f) w *= 1.0f / l;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    x[g] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (cnt[g] == 0) continue;
    const float wg = __int_as_float(__builtin_amdgcn_ds_bpermute((16 * g + (lane & 15)) * 4, __float_as_int(w)));
    merge_add_rows<SUBS>(x[g], p[g], wg, 0, cnt[g], sub);
    for (int i = A * SUBS; i < cnt[g]; i += 4 * SUBS) {
      f32x4 q[4];
      merge_load_rows<SUBS>(q, source(g), stride, i, cnt[g], sub);
      merge_add_rows<SUBS>(x[g], q, wg, i, cnt[g], sub);
    }
#pragma unroll
    for (int m = LPR; m < 64; m <<= 1)
#pragma unroll
      for (int e = 0; e < 4; ++e) x[g][e] += __shfl_xor(x[g][e], m);
  }
}

// Adds what another wave merged from later slots of the same piece (in slot order, so the bits are fixed).
__device__ __forceinline__ void merge_join(MergedPiece& r, const f32x4& x, float M, float l) {
  if (M == -INFINITY) {
    r.l += l;
    return;
  }
  const float M_new = fmaxf(r.M, M);
  const float ra = exp2f(r.M - M_new), xa = exp2f(M - M_new);   // ra = 0 when nothing has been merged yet
  r.x = r.x * ra + x * xa;
  r.l = r.l * ra + l * xa;
  r.M = M_new;
}
__device__ __forceinline__ void merge_normalise(MergedPiece& r) {
  if (r.l != 0.f) r.x *= 1.0f / r.l;
}

// Columns that one wave merges at a time: the largest piece that divides a slice.  0: this code does not apply (also
// where 64 rows of a slot are more than 32 bits of address: H dl from 2^24 on).
__host__ __device__ __forceinline__ int merge_piece_width(int dl, int H) {
  if ((long long)H * dl >= 1 << 24) return 0;
  return dl % 256 == 0 ? 256 : dl % 128 == 0 ? 128 : dl % 64 == 0 ? 64 : 0;
}

}  // namespace tpla
