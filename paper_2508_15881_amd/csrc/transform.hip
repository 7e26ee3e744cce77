// Orthogonal reparameterisation kernels (Sec. 4.1 / 4.3 of the paper) and the
// MLA-style cache write.
//   * transform_axis_kernel: shape-agnostic, one workgroup per vector, LDS (float storage, identity, in place,
//     widths and few vectors, which the matrix-core kernel of transform_weights.hip does not take).
//   * transform_paged_fwht_kernel: streaming cache pass on the vector ALU -- one
//     row per group of d_c/8 lanes, 8 elements per lane, Walsh-Hadamard
//     butterflies in registers (strides 1,2,4) and across lanes (strides
//     8..d_c/2).  Runs the identity (slicing-only) pass, float storage and the
//     widths the matrix-core pass (transform_mfma.hip) does not take.
//   * transform_paged_generic_kernel: identity / dense U / wide rows.
#include "tpla_internal.h"

namespace tpla {

// ---------------------------------------------------------------------------
// In-LDS transform of one vector x[0..d) (float), result left in x.
// mode identity: nothing.  Hadamard: natural-order butterflies, 1/sqrt(d),
// sign diagonal before (forward) or after (inverse).  Dense: y = x U or x U^T.
// `tmp` is a second d-float buffer.  All threads of the block must call.
__device__ void transform_vector_lds(float* x, float* tmp, int d, const TransformArgs& t) {
  const int tid = threadIdx.x, nt = blockDim.x;
  if (t.mode == TPLA_U_IDENTITY) return;
  if (t.mode == TPLA_U_HADAMARD) {
    if (t.signs && !t.inverse) {
      for (int i = tid; i < d; i += nt) x[i] *= t.signs[i];
      __syncthreads();
    }
    for (int h = 1; h < d; h <<= 1) {
      for (int i = tid; i < d / 2; i += nt) {
        const int lo = ((i / h) * 2 * h) + (i % h), hi = lo + h;
        const float u = x[lo], v = x[hi];
        x[lo] = u + v;
        x[hi] = u - v;
      }
      __syncthreads();
    }
    const float sc = 1.0f / sqrtf((float)d);
    for (int i = tid; i < d; i += nt) {
      float v = x[i] * sc;
      if (t.signs && t.inverse) v *= t.signs[i];
      x[i] = v;
    }
    __syncthreads();
    return;
  }
  // dense
  for (int j = tid; j < d; j += nt) {
    float s = 0.f;
    if (!t.inverse)
      for (int k = 0; k < d; ++k) s = fmaf(x[k], t.U[(size_t)k * d + j], s);
    else
      for (int k = 0; k < d; ++k) s = fmaf(x[k], t.U[(size_t)j * d + k], s);
    tmp[j] = s;
  }
  __syncthreads();
  for (int j = tid; j < d; j += nt) x[j] = tmp[j];
  __syncthreads();
}

template <typename T>
__global__ void __launch_bounds__(256) transform_axis_kernel(TransformArgs t, const T* __restrict__ src,
                                                             T* __restrict__ dst, int64_t n_inner) {
  extern __shared__ float smem[];
  const int d = t.d_c;
  float* x = smem;
  float* tmp = smem + d;
  const int64_t o = blockIdx.x / n_inner, i = blockIdx.x % n_inner;
  const T* s = src + (size_t)o * d * n_inner + i;
  T* q = dst + (size_t)o * d * n_inner + i;
  for (int k = threadIdx.x; k < d; k += blockDim.x) x[k] = load_as_f32(s + (size_t)k * n_inner);
  __syncthreads();
  transform_vector_lds(x, tmp, d, t);
  for (int k = threadIdx.x; k < d; k += blockDim.x) store_from_f32(q + (size_t)k * n_inner, x[k]);
}

int launch_transform_axis(const TransformArgs& t, const void* src, void* dst, int64_t n_outer,
                          int64_t n_inner, hipStream_t st) {
  if (transform_weights_mfma_supported(t, src, dst, n_outer, n_inner))
    return launch_transform_weights_mfma(t, src, dst, n_outer, n_inner, st);
  const size_t smem = 2u * (size_t)t.d_c * sizeof(float);
  const dim3 grid((unsigned)(n_outer * n_inner));
  if (t.dtype == TPLA_F32)
    hipLaunchKernelGGL(transform_axis_kernel<float>, grid, dim3(256), smem, st, t,
                       static_cast<const float*>(src), static_cast<float*>(dst), n_inner);
  else
    hipLaunchKernelGGL(transform_axis_kernel<bf16_t>, grid, dim3(256), smem, st, t,
                       static_cast<const bf16_t*>(src), static_cast<bf16_t*>(dst), n_inner);
  return check_launch("transform_axis_kernel");
}

// ---------------------------------------------------------------------------
// Streaming pass over MLA pages: row = [latent d_c | k_pe d_r].  LPR = d_c/8
// lanes cooperate on one row (LPR a power of two <= 64).  After the transform
// lane l holds elements 8l..8l+7 of c U, which belong to slice (8l)/dl.
constexpr int FWHT_ROWS_MAX = 4;
template <int M>
__device__ __forceinline__ void fwht_lane_stage(Vec8* x, int n_rows_here, int l, int lane, int lpr) {
  if (M >= lpr) return;
  const float sg = (l & M) ? -1.0f : 1.0f;
#pragma unroll
  for (int r = 0; r < FWHT_ROWS_MAX; ++r)
    if (r < n_rows_here)
#pragma unroll
    for (int i = 0; i < 8; ++i) x[r].v[i] = fmaf(x[r].v[i], sg, lane_xor<M>(x[r].v[i], lane));
}

constexpr int FWHT_ROWS = FWHT_ROWS_MAX;   // rows per lane group: their loads and butterflies are independent
template <typename T, bool HADAMARD>
__global__ void __launch_bounds__(256) transform_paged_fwht_kernel(
    TransformArgs t, const T* __restrict__ mla_pool, ShardPools pools, const int32_t* __restrict__ page_ids,
    int64_t n_rows, int page_tokens, int d_r, int g) {
  const int d_c = t.d_c, dl = d_c / g;
  const int lpr = d_c / 8;
  const int rows_per_block = (256 / lpr) * FWHT_ROWS;
  const int sub = threadIdx.x / lpr, l = threadIdx.x % lpr;
  // 32-bit row arithmetic (n_rows < 2^31 is checked by the caller); one
  // division per lane group, the following rows step through the page
  const unsigned row0 = blockIdx.x * (unsigned)rows_per_block + (unsigned)sub * FWHT_ROWS;
  const unsigned last = (unsigned)(n_rows - 1);
  const unsigned base_row = min(row0, last);
  const unsigned pg0 = base_row / (unsigned)page_tokens;
  const unsigned slot0 = base_row - pg0 * (unsigned)page_tokens;
  // rows past the end redo the last row (same values to the same place), so
  // every lane takes part in the lane exchanges
  size_t in_row[FWHT_ROWS], out_row[FWHT_ROWS];
  Vec8 x[FWHT_ROWS], kpe[FWHT_ROWS];
  const bool has_kpe = 8 * l < d_r;          // d_r <= d_c for this kernel: one piece per lane at most
#pragma unroll
  for (int r = 0; r < FWHT_ROWS; ++r) {
    unsigned pg = pg0, slot = slot0;
    if (row0 + r <= last) {
      slot += r;
      if (slot >= (unsigned)page_tokens) { slot -= page_tokens; pg += 1; }   // FWHT_ROWS <= page_tokens
    }
    const size_t page = page_ids ? (size_t)page_ids[pg] : (size_t)pg;
    const size_t tok = page * page_tokens + slot;
    in_row[r] = tok * (size_t)(d_c + d_r);
    out_row[r] = tok * (size_t)(dl + d_r);
    x[r] = load8(mla_pool + in_row[r] + 8 * l);
    if (has_kpe) kpe[r] = load8(mla_pool + in_row[r] + d_c + 8 * l);
  }
  if (HADAMARD) {
    if (t.signs) {
      float sg[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) sg[i] = t.signs[8 * l + i];
#pragma unroll
      for (int r = 0; r < FWHT_ROWS; ++r)
#pragma unroll
        for (int i = 0; i < 8; ++i) x[r].v[i] *= sg[i];
    }
    // strides 1, 2, 4 inside the lane
#pragma unroll
    for (int r = 0; r < FWHT_ROWS; ++r)
#pragma unroll
      for (int h = 1; h < 8; h <<= 1)
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (!(i & h)) {
            const float u = x[r].v[i], v = x[r].v[i | h];
            x[r].v[i] = u + v;
            x[r].v[i | h] = u - v;
          }
    // strides 8 .. d_c/2 across lanes: partner lane l ^ m, new = partner + (upper ? -own : own)
    const int lane = threadIdx.x & 63;
    fwht_lane_stage<1>(x, FWHT_ROWS, l, lane, lpr);
    fwht_lane_stage<2>(x, FWHT_ROWS, l, lane, lpr);
    fwht_lane_stage<4>(x, FWHT_ROWS, l, lane, lpr);
    fwht_lane_stage<8>(x, FWHT_ROWS, l, lane, lpr);
    fwht_lane_stage<16>(x, FWHT_ROWS, l, lane, lpr);
    fwht_lane_stage<32>(x, FWHT_ROWS, l, lane, lpr);
    const float sc = 1.0f / sqrtf((float)d_c);
#pragma unroll
    for (int r = 0; r < FWHT_ROWS; ++r)
#pragma unroll
      for (int i = 0; i < 8; ++i) x[r].v[i] *= sc;
  }
  const int col = 8 * l;
  const int shard = col / dl;
#pragma unroll
  for (int r = 0; r < FWHT_ROWS; ++r) {
    if (row0 + r > last) break;
    store8(static_cast<T*>(pools.p[shard]) + out_row[r] + (col - shard * dl), x[r]);
    // replicate the RoPE key on every slice
    if (has_kpe)
      for (int i = 0; i < g; ++i) store8(static_cast<T*>(pools.p[i]) + out_row[r] + dl + 8 * l, kpe[r]);
  }
}

// Any mode / width: one workgroup per row through LDS.
template <typename T>
__global__ void __launch_bounds__(256) transform_paged_generic_kernel(
    TransformArgs t, const T* __restrict__ mla_pool, ShardPools pools, const int32_t* __restrict__ page_ids,
    int page_tokens, int d_r, int g) {
  extern __shared__ float smem[];
  const int d_c = t.d_c, dl = d_c / g;
  float* x = smem;
  float* tmp = smem + d_c;
  const int64_t row = blockIdx.x;
  const int64_t pg = row / page_tokens;
  const int slot = (int)(row % page_tokens);
  const int64_t page = page_ids ? (int64_t)page_ids[pg] : pg;
  const T* in = mla_pool + ((size_t)page * page_tokens + slot) * (size_t)(d_c + d_r);
  const size_t out_row = ((size_t)page * page_tokens + slot) * (size_t)(dl + d_r);
  for (int k = threadIdx.x; k < d_c; k += blockDim.x) x[k] = load_as_f32(in + k);
  __syncthreads();
  transform_vector_lds(x, tmp, d_c, t);
  for (int k = threadIdx.x; k < d_c; k += blockDim.x) {
    const int shard = k / dl;
    store_from_f32(static_cast<T*>(pools.p[shard]) + out_row + (k - shard * dl), x[k]);
  }
  for (int k = threadIdx.x; k < d_r; k += blockDim.x) {
    const T v = in[d_c + k];
    for (int i = 0; i < g; ++i) static_cast<T*>(pools.p[i])[out_row + dl + k] = v;
  }
}

template <typename T>
static int launch_paged_t(const TransformArgs& t, const tpla_shape_t& sh, const void* mla_pool,
                          const ShardPools& pools, const int32_t* page_ids, int64_t n_pages,
                          hipStream_t st) {
  const int64_t n_rows = n_pages * sh.page_tokens;
  const int lpr = sh.d_c / 8;
  const bool pow2 = (sh.d_c & (sh.d_c - 1)) == 0;
  const bool fast = pow2 && lpr >= 1 && lpr <= 64 && sh.d_r <= sh.d_c && sh.page_tokens >= FWHT_ROWS &&
                    (t.mode == TPLA_U_HADAMARD || t.mode == TPLA_U_IDENTITY);
  const T* in = static_cast<const T*>(mla_pool);
  if (fast) {
    const int rows_per_block = (256 / lpr) * FWHT_ROWS;
    const dim3 grid((unsigned)((n_rows + rows_per_block - 1) / rows_per_block));
    if (t.mode == TPLA_U_HADAMARD)
      hipLaunchKernelGGL((transform_paged_fwht_kernel<T, true>), grid, dim3(256), 0, st, t, in, pools,
                         page_ids, n_rows, sh.page_tokens, sh.d_r, sh.g);
    else
      hipLaunchKernelGGL((transform_paged_fwht_kernel<T, false>), grid, dim3(256), 0, st, t, in, pools,
                         page_ids, n_rows, sh.page_tokens, sh.d_r, sh.g);
    return check_launch("transform_paged_fwht_kernel");
  }
  const size_t smem = 2u * (size_t)sh.d_c * sizeof(float);
  hipLaunchKernelGGL(transform_paged_generic_kernel<T>, dim3((unsigned)n_rows), dim3(256), smem, st, t,
                     in, pools, page_ids, sh.page_tokens, sh.d_r, sh.g);
  return check_launch("transform_paged_generic_kernel");
}

int launch_transform_paged(const TransformArgs& t, const tpla_shape_t& sh, const void* mla_pool,
                           const ShardPools& pools, const int32_t* page_ids, int64_t n_pages,
                           hipStream_t st) {
  if (transform_paged_mfma_supported(t, sh, n_pages))
    return launch_transform_paged_mfma(t, sh, mla_pool, pools, page_ids, n_pages, st);
  if (transform_paged_dense_mfma_supported(t, sh, n_pages))
    return launch_transform_paged_dense_mfma(t, sh, mla_pool, pools, page_ids, n_pages, st);
  if (sh.dtype == TPLA_F32) return launch_paged_t<float>(t, sh, mla_pool, pools, page_ids, n_pages, st);
  return launch_paged_t<bf16_t>(t, sh, mla_pool, pools, page_ids, n_pages, st);
}

// ---------------------------------------------------------------------------
// MLA-style cache write (HBM, streaming).  A wave takes WC_TOK tokens; their slots, 16-byte pieces (8 elements
// per lane: a 512-wide latent is one piece per lane) and RoPE keys are all requested before the first is
// needed, stay in registers between the sum of squares and the scaling, and leave as 128-bit stores.
// Rows are 16-byte aligned: every width is a multiple of 8 elements.  Latents above 64 WC_PIECES pieces are
// read a second time for the scaling.  127485 tokens of 512 + 64 bf16 (294 MB read and written): 140 us with one
// 2-byte access per lane, 71 us now = 4.1 TB/s (a large copy: 4.9).  One, two, four, eight tokens per wave: 70, 71, 74,
// 106 us, and the pass that slices the pages into the shard pools, which usually follows and finds part of them in the
// last-level cache, 70, 60, 69, 66.  (Plain stores for the same reason: with streaming ones 78 us.)
__device__ __forceinline__ void store8_cached(bf16_t* p, const Vec8& r) {
  u32x4 raw;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    raw[i] = (unsigned)f32_to_bf16_bits(r.v[2 * i]) | ((unsigned)f32_to_bf16_bits(r.v[2 * i + 1]) << 16);
  *reinterpret_cast<u32x4*>(p) = raw;
}
__device__ __forceinline__ void store8_cached(float* p, const Vec8& r) {
#pragma unroll
  for (int i = 0; i < 8; i += 4) *reinterpret_cast<f32x4*>(p + i) = f32x4{r.v[i], r.v[i + 1], r.v[i + 2], r.v[i + 3]};
}
constexpr int WC_TOK = 2;
constexpr int WC_PIECES = 2;     // pieces per lane held in registers: d_c <= 1024

template <typename T>
__global__ void __launch_bounds__(256) write_mla_cache_kernel(const T* __restrict__ c_raw,
                                                              const T* __restrict__ k_pe,
                                                              const int32_t* __restrict__ slot_mapping,
                                                              int64_t n_tok, float rms_eps, T* __restrict__ pool,
                                                              int d_c, int d_r) {
  const int lane = threadIdx.x & 63;
  const int64_t t0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * WC_TOK;
  if (t0 >= n_tok) return;
  const int np = d_c >> 3;                         // pieces of a latent
  const bool in_regs = np <= 64 * WC_PIECES;
  const size_t pitch = (size_t)(d_c + d_r);
  int slot[WC_TOK];
  Vec8 x[WC_TOK][WC_PIECES];
#pragma unroll
  for (int i = 0; i < WC_TOK; ++i) slot[i] = t0 + i < n_tok ? slot_mapping[t0 + i] : -1;
#pragma unroll
  for (int i = 0; i < WC_TOK; ++i) {
    const T* c = c_raw + (size_t)min(t0 + i, n_tok - 1) * d_c;
#pragma unroll
    for (int u = 0; u < WC_PIECES; ++u)
      if (lane + 64 * u < np) x[i][u] = load8(c + 8 * (lane + 64 * u));
  }
  // RoPE keys of the wave's tokens: consecutive in memory, dealt to the lanes 16 bytes at a time, copied as bits
  constexpr int EP = 16 / (int)sizeof(T);
  const int npe = d_r / EP;
  const T* kp = k_pe + (size_t)t0 * d_r;
  const int n_kpe = (int)min((int64_t)WC_TOK, n_tok - t0) * npe;
  for (int p = lane; p < n_kpe; p += 64) {
    const u32x4 v = *reinterpret_cast<const u32x4*>(kp + EP * p);
    const int i = p / npe, s = slot_mapping[t0 + i];
    if (s >= 0) *reinterpret_cast<u32x4*>(pool + (size_t)s * pitch + d_c + EP * (p - i * npe)) = v;
  }
#pragma unroll
  for (int i = 0; i < WC_TOK; ++i) {
    if (slot[i] < 0) continue;
    const T* c = c_raw + (size_t)(t0 + i) * d_c;
    T* out = pool + (size_t)slot[i] * pitch;
    float scale = 1.0f;
    if (rms_eps >= 0.f) {
      float ss = 0.f;
#pragma unroll
      for (int u = 0; u < WC_PIECES; ++u)
        if (lane + 64 * u < np)
#pragma unroll
          for (int e = 0; e < 8; ++e) ss = fmaf(x[i][u].v[e], x[i][u].v[e], ss);
      if (!in_regs)
        for (int p = lane + 64 * WC_PIECES; p < np; p += 64) {
          const Vec8 v = load8_cached(c + 8 * p);
#pragma unroll
          for (int e = 0; e < 8; ++e) ss = fmaf(v.v[e], v.v[e], ss);
        }
#pragma unroll
      for (int m = 32; m > 0; m >>= 1) ss += __shfl_xor(ss, m);
      scale = 1.0f / sqrtf(ss / (float)d_c + rms_eps);
    }
#pragma unroll
    for (int u = 0; u < WC_PIECES; ++u)
      if (lane + 64 * u < np) {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[i][u].v[e] *= scale;
        store8_cached(out + 8 * (lane + 64 * u), x[i][u]);
      }
    if (!in_regs)
      for (int p = lane + 64 * WC_PIECES; p < np; p += 64) {
        Vec8 v = load8_cached(c + 8 * p);
#pragma unroll
        for (int e = 0; e < 8; ++e) v.v[e] *= scale;
        store8(out + 8 * p, v);
      }
  }
}

// Latents of fewer than 64 pieces: 1 << lg lanes per token, one piece each, so that a wave's lanes are not left idle.  One
// 2-byte access per lane and token / the kernel above / this one, bf16, in us: 100 tokens of 64 + 16 2.5 / 3.5 / 2.3, 40000
// of them 11.1 / 12.3 / 3.6; 40000 tokens of 256 + 64 20.8 / 16.3 / 10.6, of 384 + 64 25.6 / 18.3 / 15.8.
constexpr int WC_NARROW = 63;    // pieces
template <typename T>
__global__ void __launch_bounds__(256) write_mla_cache_narrow_kernel(const T* __restrict__ c_raw, const T* __restrict__ k_pe,
                                                                     const int32_t* __restrict__ slot_mapping, int64_t n_tok,
                                                                     float rms_eps, T* __restrict__ pool, int d_c, int d_r, int lg) {
  constexpr int EP = 16 / (int)sizeof(T);
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, tkn = i >> lg;
  const int lanes = 1 << lg, l = (int)(i & (lanes - 1)), np = d_c >> 3, npe = d_r / EP;
  const int slot = tkn < n_tok ? slot_mapping[tkn] : -1;
  T* out = pool + (size_t)max(slot, 0) * (size_t)(d_c + d_r);
  const bool mine = slot >= 0 && l < np;
  Vec8 x;
#pragma unroll
  for (int e = 0; e < 8; ++e) x.v[e] = 0.f;
  if (mine) x = load8_cached(c_raw + (size_t)tkn * d_c + 8 * l);
  if (slot >= 0)
    for (int p = l; p < npe; p += lanes)
      *reinterpret_cast<u32x4*>(out + d_c + EP * p) = *reinterpret_cast<const u32x4*>(k_pe + (size_t)tkn * d_r + EP * p);
  if (rms_eps >= 0.f) {
    float ss = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) ss = fmaf(x.v[e], x.v[e], ss);
    for (int m = 1; m < lanes; m <<= 1) ss += __shfl_xor(ss, m);
    const float scale = 1.0f / sqrtf(ss / (float)d_c + rms_eps);
#pragma unroll
    for (int e = 0; e < 8; ++e) x.v[e] *= scale;
  }
  if (mine) store8_cached(out + 8 * l, x);
}

template <typename T>
static int launch_write_mla_cache_t(const tpla_shape_t& sh, const T* c_raw, const T* k_pe, const int32_t* slot_mapping, int64_t n_tok,
                                    float rms_eps, T* pool, hipStream_t st) {
  const int np = sh.d_c / 8;
  if (np <= WC_NARROW) {
    int lg = 0;
    while ((1 << lg) < np) ++lg;
    hipLaunchKernelGGL(write_mla_cache_narrow_kernel<T>, dim3((unsigned)(((n_tok << lg) + 255) / 256)), dim3(256), 0, st, c_raw, k_pe,
                       slot_mapping, n_tok, rms_eps, pool, sh.d_c, sh.d_r, lg);
    return check_launch("write_mla_cache_narrow_kernel");
  }
  hipLaunchKernelGGL(write_mla_cache_kernel<T>, dim3((unsigned)((n_tok + 4 * WC_TOK - 1) / (4 * WC_TOK))), dim3(256), 0, st, c_raw, k_pe,
                     slot_mapping, n_tok, rms_eps, pool, sh.d_c, sh.d_r);
  return check_launch("write_mla_cache_kernel");
}

int launch_write_mla_cache(const tpla_shape_t& sh, const void* c_raw, const void* k_pe,
                           const int32_t* slot_mapping, int64_t T, float rms_eps, void* mla_pool,
                           hipStream_t st) {
  if (sh.dtype == TPLA_F32)
    return launch_write_mla_cache_t(sh, static_cast<const float*>(c_raw), static_cast<const float*>(k_pe), slot_mapping, T, rms_eps,
                                    static_cast<float*>(mla_pool), st);
  return launch_write_mla_cache_t(sh, static_cast<const bf16_t*>(c_raw), static_cast<const bf16_t*>(k_pe), slot_mapping, T, rms_eps,
                                  static_cast<bf16_t*>(mla_pool), st);
}

// ---------------------------------------------------------------------------
// Decode-token append with per-slice RMSNorm: one wave per (sequence, slice).  A chain of round trips is all there is to it, so the slot, the slice
// (8 elements per lane, kept in registers up to 1024 of them) and the RoPE key are requested together.  One element per lane and load, the slot waited for
// first and the slice read twice: 3.8 us for one token of two slices, now 2.1.  (23 tokens behind a kernel that leaves dirty lines: 4.8 either way.)
template <typename T>
__global__ void __launch_bounds__(64) append_token_sliced_kernel(const T* __restrict__ c_t,
                                                                 const T* __restrict__ k_pe,
                                                                 MuFactors alpha, float rms_eps,
                                                                 const int32_t* __restrict__ slots,
                                                                 ShardPools pools, int d_c, int d_r, int dl) {
  constexpr int KEPT = 2, KP = sizeof(T) / 2;                // chunks of 512 in registers; 16-byte pieces of 8 elements
  const int b = blockIdx.x, i = blockIdx.y, lane = threadIdx.x;
  const int slot = slots[b];
  const T* x = c_t + (size_t)b * d_c + (size_t)i * dl;       // dl and d_r are multiples of 8, rows 16-byte aligned
  const u32x4* kp = reinterpret_cast<const u32x4*>(k_pe + (size_t)b * d_r);
  const int n_kp = d_r / 8 * KP;
  Vec8 v[KEPT];
#pragma unroll
  for (int j = 0; j < KEPT; ++j) {
    const int c = 512 * j + 8 * lane;
    if (c < dl)
      v[j] = load8_cached(x + c);
    else
#pragma unroll
      for (int e = 0; e < 8; ++e) v[j].v[e] = 0.f;
  }
  u32x4 key = {0u, 0u, 0u, 0u};
  if (lane < n_kp) key = kp[lane];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < KEPT; ++j)
#pragma unroll
    for (int e = 0; e < 8; ++e) ss = fmaf(v[j].v[e], v[j].v[e], ss);
  for (int c = 512 * KEPT + 8 * lane; c < dl; c += 512) {
    const Vec8 r = load8_cached(x + c);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss = fmaf(r.v[e], r.v[e], ss);
  }
  ss += lane_xor<1>(ss, lane);
  ss += lane_xor<2>(ss, lane);
  ss += lane_xor<4>(ss, lane);
  ss += lane_xor<8>(ss, lane);
  ss += lane_xor<16>(ss, lane);
  ss += lane_xor<32>(ss, lane);
  if (slot < 0) return;
  const float scale = 1.0f / sqrtf(alpha.v[i] * ss / (float)d_c + rms_eps);
  T* out = static_cast<T*>(pools.p[i]) + (size_t)slot * (size_t)(dl + d_r);
  auto put = [&](int c, Vec8 r) {
#pragma unroll
    for (int e = 0; e < 8; ++e) r.v[e] *= scale;
    store8_cached(out + c, r);
  };
#pragma unroll
  for (int j = 0; j < KEPT; ++j)
    if (512 * j + 8 * lane < dl) put(512 * j + 8 * lane, v[j]);
  for (int c = 512 * KEPT + 8 * lane; c < dl; c += 512) put(c, load8_cached(x + c));
  u32x4* key_out = reinterpret_cast<u32x4*>(out + dl);
  if (lane < n_kp) key_out[lane] = key;
  for (int p = 64 + lane; p < n_kp; p += 64) key_out[p] = kp[p];
}

int launch_append_token_sliced(const tpla_shape_t& sh, const void* c_t, const void* k_pe,
                               const MuFactors& alpha, float rms_eps, const int32_t* slots,
                               const ShardPools& pools, hipStream_t st) {
  const dim3 grid((unsigned)sh.B, (unsigned)sh.g);
  if (sh.dtype == TPLA_F32)
    hipLaunchKernelGGL(append_token_sliced_kernel<float>, grid, dim3(64), 0, st, static_cast<const float*>(c_t),
                       static_cast<const float*>(k_pe), alpha, rms_eps, slots, pools, sh.d_c, sh.d_r, sh.d_c / sh.g);
  else
    hipLaunchKernelGGL(append_token_sliced_kernel<bf16_t>, grid, dim3(64), 0, st, static_cast<const bf16_t*>(c_t),
                       static_cast<const bf16_t*>(k_pe), alpha, rms_eps, slots, pools, sh.d_c, sh.d_r, sh.d_c / sh.g);
  return check_launch("append_token_sliced_kernel");
}

}  // namespace tpla
