// Shape-agnostic shard decode (any widths, float or bf16 storage, float
// arithmetic) and the merge of split partials.  This is the float-mode
// implementation and the fallback for bf16 shapes the MFMA kernel does not
// cover; it favours clarity over speed.
#include "split_merge.h"

#include <algorithm>

namespace tpla {

// One workgroup = one (slice, sequence, split) and four heads, one wave per head.  A tile of TT tokens (a power of
// two, as many as fit GEN_TILE_BYTES, at most 64) is staged once in LDS as floats with 16-byte loads and used by
// all four heads, for the scores and for the output:
//   scores  a token belongs to 64 / TT adjacent lanes, which take its 16-byte pieces in turn (one lane per
//           token up to 252-wide rows); the row pitch is an odd number of pieces, so lanes on neighbouring
//           rows hit different banks; the query is a broadcast read
//   softmax inside the wave, one reference per tile: no workgroup barrier
//   output  a lane owns 4 adjacent columns of every (64 / column groups)-th token; the weights of the tile pass
//           through 64 floats of LDS that only this wave touches
// Bound by latency on the short contexts it is used for.  Before, a workgroup had one head, every thread walked
// a row of its own with 4-byte loads and the output loop looked up a page id per token: 19 us for 128
// tokens of 4 heads with 48-wide float rows, of which the launch is 2.
constexpr int GEN_WAVES = 4;                 // heads per workgroup (fewer for rows so wide that their queries fill the LDS)
constexpr int GEN_MAX_QUADS = 4;             // column groups of 4 per lane: d_c/g <= 1024
constexpr int GEN_TILE_BYTES = 40 * 1024;
constexpr int GEN_MAX_W = 64 * 256 - 256;    // widest row

__host__ __device__ __forceinline__ int gen_pitch(int w) { return (w / 4) % 2 ? w : w + 4; }   // floats; w % 8 == 0
__host__ __device__ __forceinline__ int gen_tile_tokens(int w) {
  int tt = 64;
  while (tt > 1 && tt * gen_pitch(w) * 4 > GEN_TILE_BYTES) tt >>= 1;
  return tt;
}

__device__ __forceinline__ f32x4 gen_load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 gen_load4(const bf16_t* p) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  return __builtin_convertvector(*reinterpret_cast<const bf16x4*>(p), f32x4);
}

template <typename T>
__global__ void __launch_bounds__(GEN_WAVES * 64) decode_generic_kernel(DecodeArgs a) {
  extern __shared__ u32x4 gen_lds[];
  const int dl = a.dl, dr = a.d_r, w = dl + dr, pitch = gen_pitch(w), TT = gen_tile_tokens(w);
  float* const tile = reinterpret_cast<float*>(gen_lds);       // [TT][pitch]
  const int n_thr = blockDim.x, n_waves = n_thr >> 6;
  float* const q = tile + TT * pitch;                          // [waves][w]
  float* const pw = q + n_waves * w;                           // [waves][64]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int vb = blockIdx.x / a.n_splits, s = blockIdx.x % a.n_splits;   // vb = slice * B + sequence
  const int shard = vb / a.B, b = vb % a.B;
  const int h = blockIdx.y * n_waves + wave;
  const bool live = h < a.H;
  const int L = seq_len_clipped(a, b);
  const int pt = a.page_tokens;
  const int n_pages = (L + pt - 1) / pt;
  const int p0 = s * a.pages_per_split;
  const bool direct = a.n_splits == 1;                         // the only partial result of the sequence: no merge follows
  if (p0 >= n_pages && !direct) return;
  const int p1 = min(p0 + a.pages_per_split, n_pages);
  const int t_begin = p0 * pt, t_end = min(p1 * pt, L);

  if (live) {
    const T* ql = static_cast<const T*>(a.q_lat) + ((size_t)vb * a.H + h) * dl;
    const T* qp = static_cast<const T*>(a.q_pe) + ((size_t)b * a.H + h) * dr;
    for (int i = lane; i < w; i += 64) q[wave * w + i] = i < dl ? load_as_f32(ql + i) : load_as_f32(qp + (i - dl));
  }
  const T* pool = static_cast<const T*>(a.pools[shard]);
  const int32_t* bt = a.block_table + (size_t)b * a.max_pages;
  const int LPT = 64 / TT, tok = lane / LPT, part = lane % LPT;
  const int quads = dl / 4;                                    // column groups of 4
  const int subs = quads < 64 ? 64 / quads : 1;                // tokens taken side by side in the output product
  const int sub = lane / (quads < 64 ? quads : 64), cq = quads < 64 ? lane % quads : lane;
  // this thread's first 16-byte piece of a tile and the step from one to the next, as (row, piece)
  const int wq = w / 4, row0 = tid / wq, piece0 = tid - row0 * wq, row_step = n_thr / wq, piece_step = n_thr - row_step * wq;
  f32x4 acc[GEN_MAX_QUADS];
#pragma unroll
  for (int c = 0; c < GEN_MAX_QUADS; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;

  for (int t0 = t_begin; t0 < t_end; t0 += TT) {
    const int cnt = min(TT, t_end - t0);
    __syncthreads();                                           // the previous tile has been consumed
    for (int r = row0, c = piece0; r < cnt;) {
      const int t = t0 + r;
      const f32x4 v = gen_load4(pool + ((size_t)bt[t / pt] * pt + t % pt) * w + 4 * c);
      *reinterpret_cast<f32x4*>(tile + r * pitch + 4 * c) = v;
      r += row_step;
      c += piece_step;
      if (c >= wq) {
        c -= wq;
        ++r;
      }
    }
    __syncthreads();
    if (!live) continue;
    f32x4 d4 = {0.f, 0.f, 0.f, 0.f};
    const float* row = tile + min(tok, cnt - 1) * pitch;
    const float* qh = q + wave * w;
    for (int i = 4 * part; i < w; i += 4 * LPT) {
      const f32x4 kv = *reinterpret_cast<const f32x4*>(row + i), qv = *reinterpret_cast<const f32x4*>(qh + i);
#pragma unroll
      for (int e = 0; e < 4; ++e) d4[e] = fmaf(qv[e], kv[e], d4[e]);
    }
    float d = (d4[0] + d4[1]) + (d4[2] + d4[3]);
    for (int m = 1; m < LPT; m <<= 1) d += __shfl_xor(d, m);
    const float sc = tok < cnt ? d * a.scale_log2 : -INFINITY;
    const float m_new = fmaxf(m_run, wave_max(sc));
    const float p = tok < cnt ? exp2f(sc - m_new) : 0.f;
    const float alpha = exp2f(m_run - m_new);                  // 0 on the first tile
    l_run = l_run * alpha + wave_sum(part == 0 ? p : 0.f);
    m_run = m_new;
    if (part == 0) pw[wave * 64 + tok] = p;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");     // LDS operations of one wave complete in order
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int c = 0; c < GEN_MAX_QUADS; ++c)
      if (64 * c < quads) {
        f32x4 v = acc[c] * alpha;
        const int col = cq + 64 * c;
        if (col < quads && sub < subs)
          for (int i = sub; i < cnt; i += subs) {
            const float wgt = pw[wave * 64 + i];
            const f32x4 r = *reinterpret_cast<const f32x4*>(tile + i * pitch + 4 * col);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fmaf(wgt, r[e], v[e]);
          }
        acc[c] = v;
      }
    __builtin_amdgcn_wave_barrier();
  }
  if (!live) return;
  if (quads < 64) {                                            // the token groups of a column, in order
    f32x4 v = acc[0];
    for (int u = 1; u < subs; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float o = __shfl(acc[0][e], (lane + u * quads) & 63);
        v[e] += o;
      }
    acc[0] = v;                                                // complete in the lanes with sub == 0
  }
  const size_t item = ((size_t)vb * a.n_splits + s) * a.H + h;
  const float inv = direct ? (l_run > 0.f ? 1.0f / l_run : 0.f) : 1.0f;
  float* out = (direct ? a.o_lat : a.part_acc) + item * dl;
#pragma unroll
  for (int c = 0; c < GEN_MAX_QUADS; ++c) {
    const int col = cq + 64 * c;
    if (sub == 0 && col < quads) *reinterpret_cast<f32x4*>(out + 4 * col) = acc[c] * inv;
  }
  if (lane == 0) {
    if (!direct) {
      a.part_ml[item * 2 + 0] = m_run;
      a.part_ml[item * 2 + 1] = l_run;
    } else if (a.lse) {
      a.lse[item] = n_pages > 0 ? (m_run + log2f(l_run)) * 0.6931471805599453f : -INFINITY;
    }
  }
}

// Short contexts of narrow float rows (the plan's own splits only): one workgroup of 16 waves = all slices of one (sequence, head), 16 / slices
// waves each, and with W given the combine as well, so that nothing goes through memory between the two and there is no second and third launch.
// A wave takes blocks of 16 tokens, four lanes each; a token slot has a reference, a sum and an output of its own, so that the loop has two lane
// exchanges (the dot product) and no LDS; rows stay in registers between scores and output.  Slots and waves are joined at the end.
// Bound by the chain arguments -> page ids (all of a wave's at once, beside the length) -> rows -> join -> W (requested at the start).
// 4 heads, two 32-wide slices, one sequence of 128 tokens: 5.9 us, generic kernel 9.0 and combine 5.4.
constexpr int ROWS_WAVES = 16, ROWS_W = 4;                     // W: at most that many pieces of 16 bytes per thread
struct RowsCombine {
  const float* W;                                              // [H, d_c, d_v], or null: no combine
  void* o;
  int32_t d_v, o_bf16;
};
template <int LP, int RP>                                      // pieces of 16 bytes per lane: d_c/g = 16 LP, d_r = 16 RP
__global__ void __launch_bounds__(ROWS_WAVES * 64) decode_rows_kernel(DecodeArgs a, RowsCombine rc) {
  constexpr int DL = 16 * LP, DR = 16 * RP, W4 = (DL + DR) / 4;
  extern __shared__ u32x4 gen_lds[];
  float* const part = reinterpret_cast<float*>(gen_lds);       // [waves][DL + 2]: output, reference, sum
  float* const lat = part + ROWS_WAVES * (DL + 2);             // [d_c]
  float* const red = lat + a.n_shards * DL;                    // [waves][d_v]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.x, h = blockIdx.y;
  // waves of a slice (n_shards is a power of two up to 8)
  const int log_g = 31 - __builtin_clz(a.n_shards), log_n = 4 - log_g, n_w = 1 << log_n, sl = wave >> log_n, w0 = wave & (n_w - 1);
  const int d_c = a.n_shards * DL, d_v = rc.d_v;
  const int pt_log = 31 - __builtin_clz(a.page_tokens);        // a power of two from 16 on
  const int32_t* bt = a.block_table + (size_t)b * a.max_pages;
  // block it of this wave: tokens 16 (it n_w + w0) ..; lane it holds its page (at most 64 of them: rows_supported)
  const int id = bt[min((16 * (lane * n_w + w0)) >> pt_log, a.max_pages - 1)];
  const int L = seq_len_clipped(a, b);
  const int tok = lane >> 2, quarter = lane & 3;
  const size_t head = ((size_t)sl * a.B + b) * a.H + h;
  f32x4 q[LP + RP], wv[ROWS_W];
  {
    const f32x4* ql = reinterpret_cast<const f32x4*>(static_cast<const float*>(a.q_lat) + head * DL) + quarter;
    const f32x4* qp = reinterpret_cast<const f32x4*>(static_cast<const float*>(a.q_pe) + ((size_t)b * a.H + h) * DR) + quarter;
#pragma unroll
    for (int i = 0; i < LP; ++i) q[i] = ql[4 * i];
#pragma unroll
    for (int i = 0; i < RP; ++i) q[LP + i] = qp[4 * i];
  }
  // combine: thread (k group kg, columns 4 vq ..) holds rows kg, kg + groups, ...
  const int v_log = rc.W ? 29 - __builtin_clz(d_v) : 0, vq = tid & ((1 << v_log) - 1), kg = tid >> v_log, groups = (ROWS_WAVES * 64) >> v_log;
#pragma unroll
  for (int i = 0; i < ROWS_W; ++i)
    wv[i] = rc.W && kg + i * groups < d_c ? reinterpret_cast<const f32x4*>(rc.W + ((size_t)h * d_c + kg + i * groups) * d_v)[vq] : f32x4{0.f, 0.f, 0.f, 0.f};

  constexpr float NONE = -3.402823466e38f;                     // finite: weights relative to it are 0 and not NaN
  f32x4 acc[LP];
#pragma unroll
  for (int i = 0; i < LP; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = NONE, l = 0.f;
  const f32x4* pool = static_cast<const f32x4*>(a.pools[sl]);
  const int n_it = L > 16 * w0 ? (L - 16 * w0 + 16 * n_w - 1) >> (4 + log_n) : 0;
  f32x4 row[2][LP + RP];
  auto fetch = [&](f32x4 (&x)[LP + RP], int it) {              // a block lies in one page; tokens past the end repeat the last one
    const int t = min(16 * (it * n_w + w0) + tok, L - 1);
    const f32x4* src = pool + (((size_t)__builtin_amdgcn_readlane(id, it) << pt_log) + (t & (a.page_tokens - 1))) * W4 + quarter;
#pragma unroll
    for (int i = 0; i < LP; ++i) x[i] = src[4 * i];
#pragma unroll
    for (int i = 0; i < RP; ++i) x[LP + i] = src[DL / 4 + 4 * i];
  };
  auto use = [&](const f32x4 (&x)[LP + RP], int it) {
    f32x4 d4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < LP + RP; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) d4[e] = fmaf(q[i][e], x[i][e], d4[e]);
    float d = (d4[0] + d4[1]) + (d4[2] + d4[3]);
    d += lane_xor<1>(d, lane);
    d += lane_xor<2>(d, lane);
    const bool live = 16 * (it * n_w + w0) + tok < L;          // (the row of a dead token is not added with weight 0: it may hold infinities)
    const float sc = live ? d * a.scale_log2 : -INFINITY;
    const float m_new = fmaxf(m, sc), alpha = exp2f(m - m_new), p = exp2f(sc - m_new);
    l = fmaf(l, alpha, p);
    m = m_new;
#pragma unroll
    for (int i = 0; i < LP; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][e] = fmaf(acc[i][e], alpha, live ? p * x[i][e] : 0.f);
  };
  if (n_it > 0) fetch(row[0], 0);
  for (int it = 0; it < n_it; it += 2) {
    if (it + 1 < n_it) fetch(row[1], it + 1);
    use(row[0], it);
    if (it + 2 < n_it) fetch(row[0], it + 2);
    if (it + 1 < n_it) use(row[1], it + 1);
  }
  // ---- the 16 slots of the wave, then its result to LDS ----
  float M = fmaxf(m, lane_xor<4>(m, lane));
  M = fmaxf(M, lane_xor<8>(M, lane));
  M = fmaxf(M, lane_xor<16>(M, lane));
  M = fmaxf(M, lane_xor<32>(M, lane));
  const float f = exp2f(m - M);
  auto slots_sum = [&](float v) {
    v += lane_xor<4>(v, lane);
    v += lane_xor<8>(v, lane);
    v += lane_xor<16>(v, lane);
    return v + lane_xor<32>(v, lane);
  };
  l = slots_sum(l * f);
  float* const mine = part + wave * (DL + 2);
#pragma unroll
  for (int i = 0; i < LP; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float v = slots_sum(acc[i][e] * f);
      if (tok == 0) mine[4 * (quarter + 4 * i) + e] = v;
    }
  if (lane == 0) {
    mine[DL] = M;
    mine[DL + 1] = l;
  }
  __syncthreads();
  // ---- the waves of a slice ----
  if (tid < d_c) {
    const int s = tid / DL, c = tid % DL;
    const float* first = part + (s << log_n) * (DL + 2);
    float Ms = NONE, ls = 0.f, x = 0.f;
    for (int w = 0; w < n_w; ++w) Ms = fmaxf(Ms, first[w * (DL + 2) + DL]);
    for (int w = 0; w < n_w; ++w) {
      const float e = exp2f(first[w * (DL + 2) + DL] - Ms);
      ls = fmaf(first[w * (DL + 2) + DL + 1], e, ls);
      x = fmaf(first[w * (DL + 2) + c], e, x);
    }
    if (Ms == NONE && L > 0) ls = NAN;                         // no score above -inf
    x = L > 0 ? x * (1.0f / ls) : 0.f;
    const size_t at = ((size_t)s * a.B + b) * a.H + h;
    a.o_lat[at * DL + c] = x;
    if (c == 0 && a.lse) a.lse[at] = L > 0 ? (Ms + log2f(ls)) * 0.6931471805599453f : -INFINITY;
    lat[tid] = x;
  }
  if (!rc.W) return;
  __syncthreads();
  // ---- combine ----
  f32x4 o4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < ROWS_W; ++i)
    if (kg + i * groups < d_c) {
      const float x = lat[kg + i * groups];
#pragma unroll
      for (int e = 0; e < 4; ++e) o4[e] = fmaf(x, wv[i][e], o4[e]);
    }
  for (int mask = 1 << v_log; mask < 64; mask <<= 1)
#pragma unroll
    for (int e = 0; e < 4; ++e) o4[e] += __shfl_xor(o4[e], mask);
  if (lane < 1 << v_log) *reinterpret_cast<f32x4*>(red + wave * d_v + 4 * vq) = o4;
  __syncthreads();
  if (tid < d_v) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < ROWS_WAVES; ++w) v += red[w * d_v + tid];
    const size_t at = ((size_t)b * a.H + h) * d_v + tid;
    if (rc.o_bf16)
      static_cast<bf16_t*>(rc.o)[at] = (bf16_t)v;
    else
      static_cast<float*>(rc.o)[at] = v;
  }
}

// Whether decode_rows_kernel takes a call with automatic splits: float rows of up to 80 elements, up to 4096 tokens by the width of
// the block table (and 64 blocks of 16 per wave), a workgroup for every (sequence, head) in one round, and no more blocks one after the other in a wave
// than take as long as the general kernel, which cuts a long sequence into chunks.  A block costs a quarter to a fifth of one of that kernel's tiles of
// 64 tokens; beside them stand two kernels with a merge that has a row per chunk, and one without.  (With the combine inside there is a third launch
// less and the line would lie 8 to 16 blocks higher, but all calls of a shape take the same kernel, so that o_lat and lse have the same bits.)
// Both sides measured at full tables for 1, 2, 4 and 8 slices, every row width, pages of 16 to 256 tokens, 4 to 64 blocks, 1 to 256 (sequence, head) pairs,
// with and without the combine: 2443 calls, none slower than the general kernel where this rule takes them.  General / this kernel, us, pages of 64:
//   decode alone, 48-wide rows, two slices: 2048 tokens 16.3 / 12.1, 4096 17.1 / 20.0 (not taken; 256 pairs 36.3 / 22.4, taken); 80-wide: 2048 20.4 / 16.8,
//     4096 20.6 / 28.0 (not taken); eight slices, 1024 20.8 / 28.1 (not taken)
//   with the combine, 48-wide, two slices: 128 12.8 / 5.4, 2048 21.2 / 13.1; 32-wide, four: 1024 18.9 / 10.9, 4096 20.2 / 30.0 (not taken; 256 pairs 53.8 /
//     33.7, taken)
bool decode_rows_supported(const tpla_shape_t& sh, int n_shards, int max_pages, const SplitPlan& plan) {
  const int dl = sh.d_c / sh.g, pt = sh.page_tokens;
  const long long tokens = (long long)max_pages * pt;
  auto pieces = [](int n) { return n == 16 || n == 32 || n == 64; };
  if (!(sh.dtype == TPLA_F32 && pieces(dl) && pieces(sh.d_r) && dl + sh.d_r <= 80 && (n_shards & (n_shards - 1)) == 0 && pt >= 16 && (pt & (pt - 1)) == 0 &&
        tokens <= 4096 && tokens * n_shards <= 64 * 16 * ROWS_WAVES && sh.H <= 65535 && (long long)sh.B * sh.H <= device_cu_count()))
    return false;
  const int blocks = (int)((tokens * n_shards + 16 * ROWS_WAVES - 1) / (16 * ROWS_WAVES));
  const int tiles = (plan.pages_per_split * pt + 63) / 64;                     // of a workgroup of the general kernel
  const long long workgroups = (long long)n_shards * sh.B * plan.n_splits * ((sh.H + GEN_WAVES - 1) / GEN_WAVES);
  const long long room = 5LL * device_cu_count();                              // two and a half of them per compute unit in one round
  return blocks <= 4LL * tiles * std::max(room, 2 * workgroups) / room + (dl > 32 ? 2 : 8 + plan.n_splits / 12);
}
bool decode_rows_combine_supported(const tpla_shape_t& sh) {
  return sh.d_v >= 16 && sh.d_v <= 256 && (sh.d_v & (sh.d_v - 1)) == 0 && sh.d_c * sh.d_v <= ROWS_W * 4 * ROWS_WAVES * 64;
}
int launch_decode_rows(const DecodeArgs& a, const float* W_UV_t, void* o, int o_dtype, int d_v, hipStream_t st) {
  const RowsCombine rc = {W_UV_t, o, W_UV_t ? d_v : 0, (int)(o_dtype == TPLA_BF16)};
  const size_t smem = (size_t)(ROWS_WAVES * (a.dl + 2) + a.n_shards * a.dl + ROWS_WAVES * rc.d_v + 4) * sizeof(float);
  void (*fn)(DecodeArgs, RowsCombine) = decode_rows_kernel<4, 1>;
  if (a.dl == 16) fn = a.d_r == 16 ? decode_rows_kernel<1, 1> : a.d_r == 32 ? decode_rows_kernel<1, 2> : decode_rows_kernel<1, 4>;
  if (a.dl == 32) fn = a.d_r == 16 ? decode_rows_kernel<2, 1> : decode_rows_kernel<2, 2>;
  hipLaunchKernelGGL(fn, dim3((unsigned)a.B, (unsigned)a.H), dim3(ROWS_WAVES * 64), smem, st, a, rc);
  return check_launch("decode_rows_kernel");
}

// Slices whose width is not a multiple of 64.  One workgroup = one
// (slice, sequence, head): combines that sequence's partial results in ascending order of the work items
// (fixed order => reproducible bits).  Wave 0 lists the contributing slots and turns their
// (reference, weight-sum) pairs into one normalised factor each; then every
// thread sums its columns over the slots.
constexpr int MERGE_MAX_SPLITS = 1024;
__global__ void __launch_bounds__(128) decode_merge_kernel(DecodeArgs a) {
  __shared__ float wgt[MERGE_MAX_SPLITS];
  __shared__ int slot_of[MERGE_MAX_SPLITS];
  __shared__ int cnt_sh;
  const int vb = blockIdx.x / a.H, h = blockIdx.x % a.H;   // vb = slice * B + sequence
  const int b = vb % a.B;
  const int L = seq_len_clipped(a, b);
  const int n_pages = (L + a.page_tokens - 1) / a.page_tokens;
  const int dl = a.dl;
  float* out = a.o_lat + ((size_t)vb * a.H + h) * dl;
  if (n_pages == 0) {
    for (int c = threadIdx.x; c < dl; c += blockDim.x) out[c] = 0.f;
    if (a.lse && threadIdx.x == 0) a.lse[(size_t)vb * a.H + h] = -INFINITY;
    return;
  }
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    const int vbs[1] = {vb}, bs[1] = {b};
    int firsts[1], cnts[1];
    merge_slots(a, vbs, bs, firsts, cnts);
    const int cnt = cnts[0];
    for (int s = lane; s < cnt; s += 64) slot_of[s] = firsts[0] + s;
    if (lane == 0) cnt_sh = cnt;
    __builtin_amdgcn_wave_barrier();
    float M = -INFINITY;
    for (int s = lane; s < cnt; s += 64) M = fmaxf(M, a.part_ml[((size_t)slot_of[s] * a.H + h) * 2]);
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) M = fmaxf(M, __shfl_xor(M, m));
    float lsum = 0.f;
    for (int s = lane; s < cnt; s += 64) {
      const float* ml = a.part_ml + ((size_t)slot_of[s] * a.H + h) * 2;
      const float e = exp2f(ml[0] - M);
      wgt[s] = e;
      lsum = fmaf(ml[1], e, lsum);
    }
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) lsum += __shfl_xor(lsum, m);
    const float inv = 1.0f / lsum;
    for (int s = lane; s < cnt; s += 64) wgt[s] *= inv;
    if (a.lse && lane == 0) a.lse[(size_t)vb * a.H + h] = (M + log2f(lsum)) * 0.6931471805599453f;
  }
  __syncthreads();
  const int cnt = cnt_sh;
  if ((dl & 3) == 0) {
    for (int c = threadIdx.x * 4; c < dl; c += blockDim.x * 4) {
      float v0 = 0.f, v1 = 0.f, v2 = 0.f, v3 = 0.f;
      int s = 0;
      for (; s + 4 <= cnt; s += 4) {          // four partial rows in flight; summed in slot order
        float4 p[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          p[u] = *reinterpret_cast<const float4*>(a.part_acc + ((size_t)slot_of[s + u] * a.H + h) * dl + c);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float w = wgt[s + u];
          v0 = fmaf(p[u].x, w, v0); v1 = fmaf(p[u].y, w, v1); v2 = fmaf(p[u].z, w, v2); v3 = fmaf(p[u].w, w, v3);
        }
      }
      for (; s < cnt; ++s) {
        const float4 p = *reinterpret_cast<const float4*>(a.part_acc + ((size_t)slot_of[s] * a.H + h) * dl + c);
        const float w = wgt[s];
        v0 = fmaf(p.x, w, v0); v1 = fmaf(p.y, w, v1); v2 = fmaf(p.z, w, v2); v3 = fmaf(p.w, w, v3);
      }
      *reinterpret_cast<float4*>(out + c) = make_float4(v0, v1, v2, v3);
    }
  } else {
    for (int c = threadIdx.x; c < dl; c += blockDim.x) {
      float v = 0.f;
      for (int s = 0; s < cnt; ++s) v = fmaf(a.part_acc[((size_t)slot_of[s] * a.H + h) * dl + c], wgt[s], v);
      out[c] = v;
    }
  }
}

int launch_decode_generic(const DecodeArgs& a, int dtype, hipStream_t st) {
  if (a.dl > GEN_MAX_QUADS * 256)
    return fail(TPLA_ERR_UNSUPPORTED, "d_c/g=%d above %d", a.dl, GEN_MAX_QUADS * 256);
  const int w = a.dl + a.d_r;
  if (w > GEN_MAX_W) return fail(TPLA_ERR_UNSUPPORTED, "row too wide for the generic kernel");
  if (a.H > 65535) return fail(TPLA_ERR_UNSUPPORTED, "H above 65535");
  auto lds = [&](int waves) -> size_t { return ((size_t)gen_tile_tokens(w) * gen_pitch(w) + (size_t)waves * (w + 64)) * sizeof(float); };
  int waves = GEN_WAVES;
  while (waves > 1 && lds(waves) > 64 * 1024) waves /= 2;
  const size_t smem = lds(waves);
  const dim3 grid((unsigned)(a.n_shards * a.B * a.n_splits), (unsigned)((a.H + waves - 1) / waves));
  void (*fn)(DecodeArgs) = dtype == TPLA_F32 ? decode_generic_kernel<float> : decode_generic_kernel<bf16_t>;
  if (smem > 64 * 1024 &&      // one wave and a row of more than 8000 elements
      hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) {
    (void)hipGetLastError();
    return fail(TPLA_ERR_HIP, "cannot reserve %zu bytes of LDS for decode_generic_kernel", smem);
  }
  hipLaunchKernelGGL(fn, grid, dim3((unsigned)(64 * waves)), smem, st, a);
  return check_launch("decode_generic_kernel");
}

// The same for slices of a multiple of 64 columns: one workgroup of 4 waves = one (slice, sequence, head) and
// piece of up to 256 columns, the slots dealt over the waves in order, joined in LDS (split_merge.h).
constexpr int SM_WAVES = 4;
template <int SUBS>
__global__ void __launch_bounds__(SM_WAVES * 64) split_merge_kernel(DecodeArgs a) {
  constexpr int SW = 256 / SUBS, LPR = 64 / SUBS;
  __shared__ f32x4 xs[SM_WAVES][64];
  __shared__ float2 mls[SM_WAVES];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int vb = blockIdx.x / a.H, h = blockIdx.x % a.H, col = blockIdx.y * SW;
  const int vbs[1] = {vb}, bs[1] = {vb % a.B};
  int firsts[1], cnts[1];
  merge_slots(a, vbs, bs, firsts, cnts);
  const int first = firsts[0], cnt = cnts[0];
  const int s0 = cnt * wave / SM_WAVES, s1 = cnt * (wave + 1) / SM_WAVES;
  MergedPiece r = merge_piece<SUBS>(a, h, first, s0, s1, col);
  xs[wave][lane] = r.x;
  if (lane == 0) mls[wave] = make_float2(r.M, r.l);
  __syncthreads();
  if (wave > 0) return;
  for (int w = 1; w < SM_WAVES; ++w) merge_join(r, xs[w][lane], mls[w].x, mls[w].y);
  merge_normalise(r);
  const size_t row = (size_t)vb * a.H + h;
  if (lane < LPR) *reinterpret_cast<f32x4*>(a.o_lat + row * a.dl + col + 4 * lane) = r.x;
  if (a.lse && col == 0 && lane == 0) a.lse[row] = merge_lse(r.M, r.l);
}

// Many rows or few slots: one wave = four heads of a (slice, sequence) and piece, whose rows lie side by side and whose slots are the
// same.  More than 16 slots (the long sequences of a ragged batch) are taken one head after the other, 8 rows in flight.  Shared by
// the four waves of a workgroup instead, 16 rows in turn with two round trips and three barriers each, they held up the launch: split and
// merge of 23 ragged sequences, two slices of 64 heads 57.6 -> 45.0 us (one row per workgroup 42.5), 128 heads 54.2 -> 41.4; 92 of 128 heads over
// 128-wide slices 59.6 -> 44.6, 150 of 32 heads 47.2 -> 32.0; batches of equal lengths stay.
template <int SUBS>
__global__ void __launch_bounds__(SM_WAVES * 64, 8) split_merge_quads_kernel(DecodeArgs a, int n_quads, int quads_per_pair) {
  constexpr int SW = 256 / SUBS, LPR = 64 / SUBS;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = blockIdx.y * SW, quad = blockIdx.x * SM_WAVES + wave;
  if (quad >= n_quads) return;
  auto store = [&](size_t row, const f32x4& x) {
    if (lane < LPR) *reinterpret_cast<f32x4*>(a.o_lat + row * a.dl + col + 4 * lane) = x;
  };
  const int vbs[1] = {quad / quads_per_pair}, bs[1] = {vbs[0] % a.B};
  const int h = (quad - vbs[0] * quads_per_pair) * 4, heads = min(4, a.H - h);
  int firsts[1], cnts[1];
  merge_slots(a, vbs, bs, firsts, cnts);
  const size_t row = (size_t)vbs[0] * a.H + h;
  if (cnts[0] > MERGE_SHORT) {
    for (int g = 0; g < heads; ++g) {
      MergedPiece r = merge_piece<SUBS>(a, h + g, firsts[0], 0, cnts[0], col);
      merge_normalise(r);
      store(row + g, r.x);
      if (a.lse && col == 0 && lane == 0) a.lse[row + g] = merge_lse(r.M, r.l);
    }
    return;
  }
  const int hstep = 1;
  int first[4], cnt[4], cols[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    first[g] = firsts[0];
    cnt[g] = g < heads ? cnts[0] : 0;
    cols[g] = col;
  }
  f32x4 x[4];
  float lse;
  merge_short_pieces<SUBS, 4, 2>(a, h, hstep, first, cnt, cols, x, lse);
  if (a.lse && col == 0 && (lane & 15) == 0 && (lane >> 4) < heads) a.lse[row + (lane >> 4)] = lse;
#pragma unroll
  for (int g = 0; g < 4; ++g)
    if (g < heads) store(row + g, x[g]);
}

template <int SUBS>
static int launch_split_merge_t(const DecodeArgs& a, hipStream_t st) {
  const long long pairs = (long long)a.n_shards * a.B;
  const int pieces = a.dl / (256 / SUBS), quads_per_pair = (a.H + 3) / 4;
  // Four heads per wave: where a pair is expected to have at most 16 slots (which one wave takes in one pass over their
  // weights), from 0.4 waves per compute unit and slot on.  Whole call, one row per workgroup / four heads per wave in us:
  //   2 slots: one wave per compute unit (64 heads, 512-wide, 8 sequences) 18.3 / 17.5, 2.5 waves (64 heads, 256-wide, 40
  //     sequences) 15.8 / 14.1, 5 waves (128 heads, 128-wide, 40 sequences) 18.6 / 14.7
  //   4 slots: half a wave (64 heads, 512-wide, 4 sequences) 45.2 / 48.1, 1.25 waves 18.5 / 18.5, 2 waves 28.6 / 26.9, 4 waves 24.7 / 22.2
  //   12 slots: 2.5 waves 33.8 / 35.8, 5 waves 36.1 / 31.5, 8 waves 51.9 / 46.8
  //   24 slots: 3 waves 37.4 / 53.0, 8 waves 67.1 / 77.7, 32 waves 575 / 612;   36 slots, 3 waves: 70.4 / 89.0
  const long long slots = a.balanced ? a.n_wg / pairs + 1 : a.n_splits;
  if (slots <= MERGE_SHORT && 5 * pairs * quads_per_pair * pieces >= 2 * slots * device_cu_count()) {
    const int n_quads = (int)(pairs * quads_per_pair);
    hipLaunchKernelGGL(split_merge_quads_kernel<SUBS>, dim3((unsigned)((n_quads + SM_WAVES - 1) / SM_WAVES), (unsigned)pieces),
                       dim3(SM_WAVES * 64), 0, st, a, n_quads, quads_per_pair);
    return check_launch("split_merge_quads_kernel");
  }
  hipLaunchKernelGGL(split_merge_kernel<SUBS>, dim3((unsigned)(pairs * a.H), (unsigned)pieces), dim3(SM_WAVES * 64), 0, st, a);
  return check_launch("split_merge_kernel");
}

int launch_decode_merge(const DecodeArgs& a, hipStream_t st) {
  switch (merge_piece_width(a.dl, a.H)) {
    case 256: return launch_split_merge_t<1>(a, st);
    case 128: return launch_split_merge_t<2>(a, st);
    case 64: return launch_split_merge_t<4>(a, st);
  }
  hipLaunchKernelGGL(decode_merge_kernel, dim3((unsigned)(a.n_shards * a.B * a.H)), dim3(64), 0, st, a);
  return check_launch("decode_merge_kernel");
}

// ---------------------------------------------------------------------------
// Measurement aid: the plainest possible pass over a buffer -- every lane reads
// 16 bytes per step with the streaming hint, chunks of 20 KB dealt to the
// workgroups round-robin, five loads in flight per lane -- so that the decode
// kernel's rate can be set against what the same box delivers to a reader that
// does nothing else.  The XOR of everything read is stored only if it matches
// a value it cannot have, which keeps the loads alive.
__global__ void __launch_bounds__(256) stream_read_kernel(const u32x4* __restrict__ p, size_t n_chunks,
                                                          unsigned* __restrict__ sink) {
  constexpr int CH = 5;
  unsigned acc = 0;
  for (size_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
    const u32x4* s = p + c * (CH * 256) + threadIdx.x;
    u32x4 v[CH];
#pragma unroll
    for (int j = 0; j < CH; ++j) v[j] = __builtin_nontemporal_load(s + j * 256);
#pragma unroll
    for (int j = 0; j < CH; ++j) acc += v[j][0] ^ v[j][1] ^ v[j][2] ^ v[j][3];
  }
  if (acc == 0x9E3779B9u && n_chunks == ~(size_t)0) sink[0] = acc;
}

int launch_stream_read(const void* buf, size_t bytes, void* sink, hipStream_t st) {
  const size_t n_chunks = bytes / (5 * 256 * 16);
  if (n_chunks == 0) return TPLA_OK;
  const int grid = device_cu_count() * 2;
  hipLaunchKernelGGL(stream_read_kernel, dim3((unsigned)grid), dim3(256), 0, st, static_cast<const u32x4*>(buf),
                     n_chunks, static_cast<unsigned*>(sink));
  return check_launch("stream_read_kernel");
}

}  // namespace tpla
