// PCA calibration (Sec. 4.3.2 of the paper): the second moments of cached
// latents on the GPU, the eigen-decomposition of their covariance on the host.
//   * latent_gram_mfma_kernel: G = sum_r x_r^T x_r and s = sum_r x_r over paged
//     bf16 rows, 128 x 128 blocks of the upper triangle on the matrix cores.
//     The contraction runs over rows, so both MFMA operands are columns of the
//     staged tile, fetched with transposing LDS reads.
//   * latent_gram_generic_kernel: any storage type / width (plain FMA).
//   * latent_moments_reduce_kernel, latent_moments_reduce_blocked_kernel: sum the
//     per-split partials in double, in a fixed order, and mirror the triangle.
//   * pca_basis_host: covariance = G/n - m m^T, Householder tridiagonalisation
//     and implicit QR steps in double, eigenvalues sorted descending; the variance fractions of the g
//     slices (the alpha, beta of Sec. 4.3.2).
#include "lds_tile.h"

#include <algorithm>
#include <cmath>
#include <numeric>
#include <vector>

namespace tpla {

constexpr int GB = 128;                  // block edge of the Gram matrix

__host__ __device__ inline int gram_blocks(int nbk) { return nbk * (nbk + 1) / 2; }

// Workgroup = (block of the upper triangle, split); split sp takes pages [sp * pages_per_split, ...).
// part_gram[sp][blk][128][128], part_sum[sp][d_c] (column sums written by the diagonal blocks).
//
// Bound by how fast the tiles come in: 4 waves multiply a staged tile in about the time its LDS reads take.  So
//   * tiles of 32 rows go straight from global memory into a ring of 3 LDS buffers, two in flight and one barrier per
//     tile; three workgroups per compute unit (144 KB of LDS) cover each other's barriers: 146 us in the case below,
//     two workgroups with a ring of 4 172 us;
//   * the LDS reads are written in assembly, because the compiler makes every LDS read of its own wait for all loads
//     to LDS;
//   * the blocks of one split, which read the same rows, run on one XCD (workgroup ids congruent mod 8), so
//     that a row comes from memory once and from that XCD's L2 for the other blocks;
//   * a diagonal block stages its one slab once and uses it for both operands; its column sums are one more
//     product, with ones.
// The tile is read back transposed (both operands are columns of it; pieces swizzled as in lds_tile.h).  Rows past a
// page's fill repeat its first row and are cleared in LDS before they are used.
// 368311 rows of d_c = 512 in 5773 pages: 268 us with registers as the only stage, 148 us with this ring (0.82 PFLOP/s; 143 with the quadrants below; what is
// left is the LDS reads, 8 KB per wave and tile, which take as long as its matrix products).
constexpr int GT = 32;                   // rows per tile: one MFMA k-step
constexpr int GST = 3;                   // ring of tiles
constexpr int G_PER_CU = 3;              // workgroups per compute unit that the LDS and 170 registers allow
constexpr int G_SLAB = GT * GB * 2;      // bytes of a slab of the tile
constexpr size_t G_LDS = (size_t)GST * 2 * G_SLAB;

// Page ids and fills of 64 consecutive listed pages, one per lane, read back with v_readlane: fetched page by page they
// are a round trip to memory each, in front of the page's rows (208 us instead of 172 with a ring of 4).
struct PageWindow {
  int base, ids, fills;
  __device__ __forceinline__ void load(const int32_t* page_ids, const int32_t* page_fill, int first, int pg_end, int page_tokens) {
    base = first;
    const int p = max(min(first + (int)(threadIdx.x & 63), pg_end - 1), 0);
    ids = page_ids ? page_ids[p] : p;
    fills = page_fill ? min(page_fill[p], page_tokens) : page_tokens;
    asm volatile("" : "+v"(ids), "+v"(fills));           // the wait stays here
  }
  __device__ __forceinline__ int id(int p) const { return __builtin_amdgcn_readlane(ids, p - base); }
  __device__ __forceinline__ int fill(int p) const { return __builtin_amdgcn_readlane(fills, p - base); }
};

// What a wave computes of its quadrant: all of it; of a block on the diagonal the quadrants on it from the diagonal on (their rows and columns are the same
// fragments) and nothing below it: the reduction mirrors the triangle.  A copy of the loop for each: the waves of a workgroup meet at its barriers.
// 36 products of 64 per 32 rows of such a block (44 of 72 with those of the column sums), 4 of the 10 of d_c = 512: 368311 rows 151 -> 143 us.  (With a branch in one loop the
// accumulators were copied and spilled: 1030 us.)
enum GramQuadrant { GRAM_FULL, GRAM_ABOVE, GRAM_ON, GRAM_BELOW };
template <GramQuadrant QUADRANT>
__device__ __forceinline__ void gram_block(const bf16_t* __restrict__ mla_pool, const int32_t* __restrict__ page_ids,
                                           const int32_t* __restrict__ page_fill, int pg, int pg_end, int page_tokens,
                                           int in_pitch, int bi, int bj, char* lds, f32x4 (&acc)[4][4], f32x4 (&csum)[4]) {
  constexpr bool DIAGONAL = QUADRANT != GRAM_FULL;
  constexpr int CPT = DIAGONAL ? 2 : 4;                  // loads per wave and tile
  const int tid = threadIdx.x, lane = tid & 63, j16 = lane & 15, q4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wi = wave >> 1, wj = wave & 1;
  const unsigned lds_base = (unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)lds);

  // instruction k of a slab fills its pieces [64k, 64k + 64): rows 4k .. 4k + 3; this wave issues k = wave and wave + 4
  int ld_row[2];
  unsigned ld_col[2];                                    // elements into the 128 columns of the slab
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    ld_row[u] = 4 * (wave + 4 * u) + q4;
    ld_col[u] = 8u * (unsigned)(j16 ^ wswz(ld_row[u]));
  }
  int row0 = 0, fill = 0;                                // the next tile to request: rows row0 .. of page pg
  PageWindow win;
  win.load(page_ids, page_fill, pg, pg_end, page_tokens);
  auto seek = [&]() {                                    // to the first page from pg on that holds a row
    for (; pg < pg_end; ++pg) {
      if (pg - win.base >= 64) win.load(page_ids, page_fill, pg, pg_end, page_tokens);
      fill = win.fill(pg);
      if (fill > 0) break;
    }
  };
  auto request = [&](int buf) -> int {                   // returns the tile's valid rows and steps past it
    const size_t page = (size_t)win.id(pg);
    const bf16_t* base = mla_pool + page * (size_t)page_tokens * in_pitch;
    const int valid = min(GT, fill - row0);
#pragma unroll
    for (int sl = 0; sl < (DIAGONAL ? 1 : 2); ++sl)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int r = ld_row[u] < valid ? row0 + ld_row[u] : 0;
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void*)(base + (size_t)r * in_pitch + GB * (sl ? bj : bi) + ld_col[u]),
            (__attribute__((address_space(3))) void*)(lds + (buf * 2 + sl) * G_SLAB + (wave + 4 * u) * 1024), 16, 0, 0);
      }
    row0 += GT;
    if (row0 >= fill) {
      row0 = 0;
      ++pg;
      seek();
    }
    return valid;
  };
  // rows 8 q4 + j16/4 (+ 4: 1024 bytes on, same swizzle), columns 16 cb + 4 (j16 % 4) ..
  const int r0 = 8 * q4 + (j16 >> 2);
  unsigned a_off[4], b_off[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    auto off = [&](int cb) -> unsigned { return (unsigned)((r0 * 16 + ((2 * cb + ((j16 & 3) >> 1)) ^ wswz(r0))) * 16 + (j16 & 1) * 8); };
    a_off[m] = off(4 * wi + m);
    b_off[m] = off(4 * wj + m) + (DIAGONAL ? 0 : G_SLAB);
  }

  // of the columns of this wave, by the waves of the upper half: a product with ones
  auto column_sums = [&](const bf16x8 (&f)[4]) {
    if (wi > 0) return;
    const u32x4 one4 = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
#pragma unroll
    for (int b = 0; b < 4; ++b) csum[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, one4), f[b], csum[b], 0, 0, 0);
  };

  seek();
  static_assert(GST == 3, "two tiles in flight");
  int in_flight = 0;
  int valid = 0, next_valid = 0;                         // rows of the oldest tile requested and of the one after it
  if (pg < pg_end) {
    valid = request(0);
    in_flight = 1;
  }
  if (pg < pg_end) {
    next_valid = request(1);
    in_flight = 2;
  }
  for (int cur = 0; in_flight > 0; cur = cur + 1 == GST ? 0 : cur + 1) {
    // the oldest tile has landed once only the loads of the younger one are outstanding
    if (in_flight == 2)
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(CPT));
    else
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __builtin_amdgcn_s_barrier();                        // it is visible to all waves, the one before it no longer read
    const int v = valid;
    valid = next_valid;
    --in_flight;
    if (pg < pg_end) {                                   // two are in flight whenever there is more to come
      next_valid = request(cur == 0 ? GST - 1 : cur - 1);
      ++in_flight;
    }
    const unsigned tile = lds_base + (unsigned)(cur * 2 * G_SLAB);
    if (v < GT) {
      const u32x4 zero = {0u, 0u, 0u, 0u};
      for (int x = tid; x < (DIAGONAL ? 1 : 2) * GT * 16; x += 256)
        if (((x >> 4) & (GT - 1)) >= v) asm volatile("ds_write_b128 %0, %1" ::"v"(tile + (unsigned)x * 16u), "v"(zero) : "memory");
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
    }
    if constexpr (QUADRANT == GRAM_ON) {
      u32x2 fl[4], fh[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        lds_read_tr_b64<0>(fl[m], tile + a_off[m]);
        lds_read_tr_b64<1024>(fh[m], tile + a_off[m]);
      }
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(fl[0]), "+v"(fh[0]), "+v"(fl[1]), "+v"(fh[1]), "+v"(fl[2]), "+v"(fh[2]), "+v"(fl[3]), "+v"(fh[3])
                   :
                   : "memory");
      bf16x8 f[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) f[m] = __builtin_bit_cast(bf16x8, u32x4{fl[m][0], fl[m][1], fh[m][0], fh[m][1]});
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = a; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[a], f[b], acc[a][b], 0, 0, 0);
      column_sums(f);
    } else if constexpr (QUADRANT != GRAM_BELOW) {
      u32x2 al[4], ah[4], bl[4], bh[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        lds_read_tr_b64<0>(al[m], tile + a_off[m]);
        lds_read_tr_b64<1024>(ah[m], tile + a_off[m]);
        lds_read_tr_b64<0>(bl[m], tile + b_off[m]);
        lds_read_tr_b64<1024>(bh[m], tile + b_off[m]);
      }
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(al[0]), "+v"(ah[0]), "+v"(bl[0]), "+v"(bh[0]), "+v"(al[1]), "+v"(ah[1]), "+v"(bl[1]), "+v"(bh[1]),
                     "+v"(al[2]), "+v"(ah[2]), "+v"(bl[2]), "+v"(bh[2]), "+v"(al[3]), "+v"(ah[3]), "+v"(bl[3]), "+v"(bh[3])
                   :
                   : "memory");
      bf16x8 fa[4], fb[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        fa[m] = __builtin_bit_cast(bf16x8, u32x4{al[m][0], al[m][1], ah[m][0], ah[m][1]});
        fb[m] = __builtin_bit_cast(bf16x8, u32x4{bl[m][0], bl[m][1], bh[m][0], bh[m][1]});
      }
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
      if constexpr (DIAGONAL) column_sums(fb);
    }
  }
}

__global__ void __launch_bounds__(256, G_PER_CU) latent_gram_mfma_kernel(
    const bf16_t* __restrict__ mla_pool, const int32_t* __restrict__ page_ids, const int32_t* __restrict__ page_fill,
    int n_pages, int n_splits, int pages_per_split, int page_tokens, int d_c, int d_r, float* __restrict__ part_gram,
    float* __restrict__ part_sum) {
  extern __shared__ u32x4 gram_lds[];
  char* const lds = reinterpret_cast<char*>(gram_lds);
  const int nbk = d_c / GB, n_blk = gram_blocks(nbk);
  const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
  const int sp = xcd + 8 * (seq / n_blk), block = seq % n_blk;
  if (sp >= n_splits) return;
  int blk = block, bi = 0;
  while (blk >= nbk - bi) { blk -= nbk - bi; ++bi; }     // row bi of the triangle holds nbk - bi blocks
  const int bj = bi + blk;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lo = lane & 15, hi = lane >> 4;
  const int wi = wave >> 1, wj = wave & 1;
  f32x4 acc[4][4], csum[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    csum[a] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int pg = sp * pages_per_split, pg_end = min(n_pages, pg + pages_per_split);
  auto quadrant = [&](auto kind) {
    gram_block<decltype(kind)::value>(mla_pool, page_ids, page_fill, pg, pg_end, page_tokens, d_c + d_r, bi, bj, lds, acc, csum);
  };
  if (bi != bj)
    quadrant(std::integral_constant<GramQuadrant, GRAM_FULL>{});
  else if (wi < wj)
    quadrant(std::integral_constant<GramQuadrant, GRAM_ABOVE>{});
  else if (wi == wj)
    quadrant(std::integral_constant<GramQuadrant, GRAM_ON>{});
  else
    quadrant(std::integral_constant<GramQuadrant, GRAM_BELOW>{});

  // partial block: lane holds column 64 wj + 16 b + lo, rows 64 wi + 16 a + 4 hi + e
  float* out = part_gram + ((size_t)sp * n_blk + block) * (GB * GB);
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        out[(64 * wi + 16 * a + 4 * hi + e) * GB + 64 * wj + 16 * b + lo] = acc[a][b][e];
  // column sums of the diagonal blocks: every row of the product with ones is the same
  if (bi == bj && wi == 0 && hi == 0)
#pragma unroll
    for (int b = 0; b < 4; ++b) part_sum[(size_t)sp * d_c + GB * bi + 64 * wj + 16 * b + lo] = csum[b][0];
}

// Any storage / width: thread (i, j >= i) of a 16 x 16 patch, rows of split sp.
// part_gram[sp][d_c][d_c] (upper triangle), part_sum[sp][d_c].
template <typename T>
__global__ void __launch_bounds__(256) latent_gram_generic_kernel(
    const T* __restrict__ mla_pool, const int32_t* __restrict__ page_ids, const int32_t* __restrict__ page_fill,
    int n_pages, int pages_per_split, int page_tokens, int d_c, int d_r, float* __restrict__ part_gram,
    float* __restrict__ part_sum) {
  const int i = blockIdx.x * 16 + threadIdx.x / 16, j = blockIdx.y * 16 + threadIdx.x % 16;
  const int sp = blockIdx.z;
  if (blockIdx.y < blockIdx.x) return;                  // below the diagonal: mirrored by the reduction
  const bool live = i < d_c && j < d_c;
  const int in_pitch = d_c + d_r;
  float g = 0.f, s = 0.f;
  const int pg_end = min(n_pages, (sp + 1) * pages_per_split);
  for (int pg = sp * pages_per_split; pg < pg_end; ++pg) {
    const size_t page = page_ids ? (size_t)page_ids[pg] : (size_t)pg;
    const int fill = page_fill ? min(page_fill[pg], page_tokens) : page_tokens;
    const T* base = mla_pool + page * (size_t)page_tokens * in_pitch;
    if (live)
      for (int r = 0; r < fill; ++r) {
        const float xi = load_as_f32(base + (size_t)r * in_pitch + i), xj = load_as_f32(base + (size_t)r * in_pitch + j);
        g = fmaf(xi, xj, g);
        s += xj;
      }
  }
  if (!live) return;
  part_gram[((size_t)sp * d_c + i) * d_c + j] = g;
  if (i == j) part_sum[(size_t)sp * d_c + j] = s;
}

// Partials as full matrices (latent_gram_generic_kernel).
__global__ void __launch_bounds__(256) latent_moments_reduce_kernel(
    const float* __restrict__ part_gram, const float* __restrict__ part_sum, int n_splits, int d_c,
    double* __restrict__ sum, double* __restrict__ gram) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= d_c * d_c) return;
  const int i = idx / d_c, j = idx % d_c;
  if (j < i) return;
  double g = 0.0;
  const float* p = part_gram + (size_t)i * d_c + j;
  for (int sp = 0; sp < n_splits; ++sp) g += (double)p[(size_t)sp * d_c * d_c];
  gram[(size_t)i * d_c + j] = g;
  gram[(size_t)j * d_c + i] = g;
  if (i == j) {
    double s = 0.0;
    for (int sp = 0; sp < n_splits; ++sp) s += (double)part_sum[(size_t)sp * d_c + j];
    sum[j] = s;
  }
}

// Partials as 128 x 128 blocks of the upper triangle: workgroup = one 16 x 16 tile of one block, wave w adds the splits
// w, w + 4, ..., and the tile is written in both orders, 128 bytes a row.  The tiles on the diagonal add the column sums
// of their 16 columns.  Bound by reading the partials (38 MB of tiles on and above the diagonal for 72 splits of d_c = 512); one thread per
// element walking all splits, the column sums in one chain of loads per column, took 27 us, this kernel 11.3.  The tiles of one row of tiles run
// on one XCD (workgroup ids congruent mod 8): a row of a tile is half a 128-byte line, and the neighbour on another XCD fetched it again: 15.7.
__global__ void __launch_bounds__(256) latent_moments_reduce_blocked_kernel(
    const float* __restrict__ part_gram, const float* __restrict__ part_sum, int n_splits, int d_c,
    double* __restrict__ sum, double* __restrict__ gram) {
  __shared__ double red[4][16 * 17];
  const int ti = blockIdx.x & 7, tj = blockIdx.x >> 3, n_blk = gridDim.y, nbk = d_c / GB;
  int blk = blockIdx.y, bi = 0;
  while (blk >= nbk - bi) { blk -= nbk - bi; ++bi; }
  const int bj = bi + blk;
  if (bi == bj && tj < ti) return;                         // written by its mirror image
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r4 = lane >> 2, c4 = 4 * (lane & 3);
  const float* p = part_gram + (size_t)blockIdx.y * (GB * GB) + (16 * ti + r4) * GB + 16 * tj + c4;
  const size_t stride = (size_t)n_blk * (GB * GB);
  double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
  for (int sp = wave; sp < n_splits; sp += 4) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(p + sp * stride);
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] += (double)v[e];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) red[wave][r4 * 17 + c4 + e] = s[e];
  __syncthreads();
  const int r = tid >> 4, c = tid & 15;
  auto total = [&](int row, int col) -> double {
    const int x = row * 17 + col;
    return (red[0][x] + red[1][x]) + (red[2][x] + red[3][x]);
  };
  const int i0 = GB * bi + 16 * ti, j0 = GB * bj + 16 * tj;
  if (i0 == j0) {
    gram[(size_t)(i0 + r) * d_c + j0 + c] = total(min(r, c), max(r, c));
    double cs = 0.0;
    for (int sp = r; sp < n_splits; sp += 16) cs += (double)part_sum[(size_t)sp * d_c + j0 + c];
    __syncthreads();
    red[0][r * 17 + c] = cs;
    __syncthreads();
    if (tid < 16) {
      double t = 0.0;
#pragma unroll
      for (int k = 0; k < 16; ++k) t += red[0][k * 17 + tid];
      sum[j0 + tid] = t;
    }
  } else {
    gram[(size_t)(i0 + r) * d_c + j0 + c] = total(r, c);
    gram[(size_t)(j0 + r) * d_c + i0 + c] = total(c, r);
  }
}

static bool gram_mfma_supported(const tpla_shape_t& sh) {
  return sh.dtype == TPLA_BF16 && sh.d_c % GB == 0 && sh.d_c <= 1024 && sh.d_r % 8 == 0;
}

int latent_moments_splits(const tpla_shape_t& sh, int64_t n_pages) {
  // enough workgroups for every place on the chip, rows per split bounded so float partials stay accurate
  const int per_cu = gram_mfma_supported(sh) ? G_PER_CU : 2;
  const int blocks = gram_mfma_supported(sh) ? gram_blocks(sh.d_c / GB) : ((sh.d_c + 15) / 16) * ((sh.d_c + 15) / 16);
  int64_t s = (per_cu * (int64_t)device_cu_count() + blocks - 1) / blocks;
  const int64_t by_rows = (n_pages * sh.page_tokens + 16383) / 16384;
  s = std::max<int64_t>(s, by_rows);
  s = std::min<int64_t>(s, std::min<int64_t>(n_pages, 1024));
  return (int)std::max<int64_t>(s, 1);
}

size_t latent_moments_workspace(const tpla_shape_t& sh, int64_t n_pages) {
  const size_t S = (size_t)latent_moments_splits(sh, n_pages);
  const size_t per = gram_mfma_supported(sh) ? (size_t)gram_blocks(sh.d_c / GB) * GB * GB : (size_t)sh.d_c * sh.d_c;
  return S * (per + sh.d_c) * sizeof(float);
}

int launch_latent_moments(const tpla_shape_t& sh, const void* mla_pool, const int32_t* page_ids,
                          const int32_t* page_fill, int64_t n_pages, float* workspace, double* sum, double* gram,
                          hipStream_t st) {
  const bool mfma = gram_mfma_supported(sh);
  const int n_blk = mfma ? gram_blocks(sh.d_c / GB) : 1;
  int S = latent_moments_splits(sh, n_pages);            // what the workspace holds
  if (mfma) {
    // whole rounds of G_PER_CU workgroups per compute unit, the blocks of a split on one XCD: at d_c = 512 (10 blocks)
    // that is 72 splits, where 77 would leave a second round of 4 of 96 places per XCD
    const int round = 8 * std::max(1, G_PER_CU * device_cu_count() / 8 / n_blk);
    const int by_rows = (int)((n_pages * sh.page_tokens + 16383) / 16384);
    if (S > round && S / round * round >= by_rows) S = S / round * round;
  }
  const int pps = (int)((n_pages + S - 1) / S);
  const size_t per = mfma ? (size_t)n_blk * GB * GB : (size_t)sh.d_c * sh.d_c;
  float* part_gram = workspace;
  float* part_sum = workspace + (size_t)S * per;
  if (mfma) {
    const dim3 grid((unsigned)(8 * n_blk * ((S + 7) / 8)));
    hipLaunchKernelGGL(latent_gram_mfma_kernel, grid, dim3(256), G_LDS, st, static_cast<const bf16_t*>(mla_pool), page_ids,
                       page_fill, (int)n_pages, S, pps, sh.page_tokens, sh.d_c, sh.d_r, part_gram, part_sum);
  } else {
    const dim3 grid((sh.d_c + 15) / 16, (sh.d_c + 15) / 16, S);
    if (sh.dtype == TPLA_F32)
      hipLaunchKernelGGL(latent_gram_generic_kernel<float>, grid, dim3(256), 0, st, static_cast<const float*>(mla_pool),
                         page_ids, page_fill, (int)n_pages, pps, sh.page_tokens, sh.d_c, sh.d_r, part_gram, part_sum);
    else
      hipLaunchKernelGGL(latent_gram_generic_kernel<bf16_t>, grid, dim3(256), 0, st,
                         static_cast<const bf16_t*>(mla_pool), page_ids, page_fill, (int)n_pages, pps, sh.page_tokens,
                         sh.d_c, sh.d_r, part_gram, part_sum);
  }
  int rc = check_launch("latent_gram kernel");
  if (rc) return rc;
  if (mfma)
    hipLaunchKernelGGL(latent_moments_reduce_blocked_kernel, dim3((GB / 16) * (GB / 16), n_blk), dim3(256), 0, st,
                       part_gram, part_sum, S, sh.d_c, sum, gram);
  else
    hipLaunchKernelGGL(latent_moments_reduce_kernel, dim3((sh.d_c * sh.d_c + 255) / 256), dim3(256), 0, st, part_gram,
                       part_sum, S, sh.d_c, sum, gram);
  return check_launch("latent_moments_reduce_kernel");
}

// ---------------------------------------------------------------------------
// Host: eigen-decomposition of the symmetric covariance in two textbook steps:
// Householder reflections bring A to tridiagonal form T = Q^T A Q, then
// implicit QR steps with Wilkinson's shift diagonalise T.  A is d x d row-major
// (overwritten); V gets the eigenvectors as ROWS (every rotation and reflection
// then works on contiguous rows); lam gets the eigenvalues, unsorted.  Returns
// false if the QR iteration does not converge.
static bool symmetric_eigen(std::vector<double>& A, std::vector<double>& V, std::vector<double>& lam, int d) {
  std::vector<double> off((size_t)std::max(d, 1), 0.0), v((size_t)d), p((size_t)d), u((size_t)d);
  std::fill(V.begin(), V.end(), 0.0);
  for (int i = 0; i < d; ++i) V[(size_t)i * d + i] = 1.0;
  // ---- tridiagonal form: step k clears row/column k beyond its first off-diagonal entry ----
  for (int k = 0; k + 2 < d; ++k) {
    const int m = d - k - 1;                       // size of the trailing block, indices k+1 .. d-1
    const double* x = &A[(size_t)k * d + k + 1];   // row k right of the diagonal (= column k below it)
    double norm2 = 0.0;
    for (int i = 0; i < m; ++i) norm2 += x[i] * x[i];
    double tail2 = norm2 - x[0] * x[0];
    if (tail2 <= 0.0) {                            // already tridiagonal here
      off[k] = x[0];
      continue;
    }
    const double sigma = std::sqrt(norm2);
    const double alpha = x[0] > 0.0 ? -sigma : sigma;          // the entry that replaces x
    for (int i = 0; i < m; ++i) v[i] = x[i];
    v[0] -= alpha;
    const double vnorm2 = tail2 + v[0] * v[0];
    const double beta = 2.0 / vnorm2;                          // H = I - beta v v^T
    // trailing block B <- H B H = B - v w^T - w v^T with p = beta B v, w = p - (beta/2)(v.p) v
    double vp = 0.0;
    for (int i = 0; i < m; ++i) {
      const double* Bi = &A[(size_t)(k + 1 + i) * d + k + 1];
      double acc = 0.0;
      for (int j = 0; j < m; ++j) acc += Bi[j] * v[j];
      p[i] = beta * acc;
      vp += v[i] * p[i];
    }
    const double half = 0.5 * beta * vp;
    for (int i = 0; i < m; ++i) p[i] -= half * v[i];           // p is w from here on
    for (int i = 0; i < m; ++i) {
      double* Bi = &A[(size_t)(k + 1 + i) * d + k + 1];
      const double vi = v[i], wi = p[i];
      for (int j = 0; j < m; ++j) Bi[j] -= vi * p[j] + wi * v[j];
    }
    off[k] = alpha;
    // V = Q^T: rows k+1.. of V <- H (rows k+1.. of V)
    std::fill(u.begin(), u.end(), 0.0);
    for (int i = 0; i < m; ++i) {
      const double* Vi = &V[(size_t)(k + 1 + i) * d];
      const double vi = v[i];
      for (int j = 0; j < d; ++j) u[j] += vi * Vi[j];
    }
    for (int i = 0; i < m; ++i) {
      double* Vi = &V[(size_t)(k + 1 + i) * d];
      const double bv = beta * v[i];
      for (int j = 0; j < d; ++j) Vi[j] -= bv * u[j];
    }
  }
  for (int i = 0; i < d; ++i) lam[i] = A[(size_t)i * d + i];
  if (d >= 2) off[d - 2] = A[(size_t)(d - 2) * d + d - 1];
  // ---- QR steps on the unreduced block [lo, hi] at the bottom, deflating as off-diagonals vanish ----
  const double eps = 2.220446049250313e-16;
  int hi = d - 1;
  long budget = 60L * d;
  while (hi > 0) {
    if (std::fabs(off[hi - 1]) <= eps * (std::fabs(lam[hi - 1]) + std::fabs(lam[hi]))) {
      off[hi - 1] = 0.0;
      --hi;
      continue;
    }
    if (--budget < 0) return false;
    int lo = hi - 1;
    while (lo > 0 && std::fabs(off[lo - 1]) > eps * (std::fabs(lam[lo - 1]) + std::fabs(lam[lo]))) --lo;
    if (lo > 0) off[lo - 1] = 0.0;
    // Wilkinson's shift: the eigenvalue of the last 2 x 2 block closer to its last entry
    const double delta = 0.5 * (lam[hi - 1] - lam[hi]), b = off[hi - 1];
    const double mu = lam[hi] - b * b / (delta + (delta >= 0.0 ? 1.0 : -1.0) * std::hypot(delta, b));
    double x = lam[lo] - mu, z = off[lo];
    for (int k = lo; k < hi; ++k) {
      // rotation in the (k, k+1) plane that sends (x, z) to (r, 0); T <- G^T T G chases the bulge down
      const double r = std::hypot(x, z);
      const double c = r != 0.0 ? x / r : 1.0, sn = r != 0.0 ? -z / r : 0.0;
      if (k > lo) off[k - 1] = r;
      const double a = lam[k], e = off[k], cc = lam[k + 1];
      lam[k] = a * c * c - 2.0 * e * c * sn + cc * sn * sn;
      lam[k + 1] = a * sn * sn + 2.0 * e * c * sn + cc * c * c;
      off[k] = (a - cc) * c * sn + e * (c * c - sn * sn);
      x = off[k];
      if (k + 1 < hi) {
        z = -sn * off[k + 1];
        off[k + 1] *= c;
      }
      double* Vk = &V[(size_t)k * d];
      double* Vk1 = &V[(size_t)(k + 1) * d];
      for (int j = 0; j < d; ++j) {
        const double p0 = Vk[j], p1 = Vk1[j];
        Vk[j] = c * p0 - sn * p1;
        Vk1[j] = sn * p0 + c * p1;
      }
    }
  }
  return true;
}

int pca_basis_host(int d, int g, double n_rows, const double* sum, const double* gram, float* U, double* eig,
                   double* frac) {
  std::vector<double> A((size_t)d * d), V((size_t)d * d);
  for (int i = 0; i < d; ++i)
    for (int j = 0; j < d; ++j)
      A[(size_t)i * d + j] = gram[(size_t)i * d + j] / n_rows - (sum[i] / n_rows) * (sum[j] / n_rows);
  for (int i = 0; i < d; ++i)                            // exact symmetry whatever the caller passed
    for (int j = i + 1; j < d; ++j) A[(size_t)j * d + i] = A[(size_t)i * d + j] = 0.5 * (A[(size_t)i * d + j] + A[(size_t)j * d + i]);
  std::vector<double> lam((size_t)d);
  if (!symmetric_eigen(A, V, lam, d)) return fail(TPLA_ERR_UNSUPPORTED, "the QR iteration did not converge");
  std::vector<int> order(d);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return lam[a] > lam[b]; });
  double total = 0.0;
  for (int k = 0; k < d; ++k) {
    const int src = order[k];
    eig[k] = lam[src];
    total += eig[k];
    // sign convention: the largest-magnitude component of every eigenvector is positive
    int big = 0;
    for (int i = 1; i < d; ++i)
      if (std::fabs(V[(size_t)src * d + i]) > std::fabs(V[(size_t)src * d + big])) big = i;
    const double sg = V[(size_t)src * d + big] < 0.0 ? -1.0 : 1.0;
    for (int i = 0; i < d; ++i) U[(size_t)i * d + k] = (float)(sg * V[(size_t)src * d + i]);   // column k
  }
  const int dl = d / g;
  for (int i = 0; i < g; ++i) {
    double part = 0.0;
    for (int k = i * dl; k < (i + 1) * dl; ++k) part += eig[k];
    frac[i] = total != 0.0 ? part / total : 1.0 / g;
  }
  return TPLA_OK;
}

}  // namespace tpla
