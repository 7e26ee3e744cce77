// Matrix-core versions of the two per-head contractions around the decode
// (bf16 weights): absorb  q_lat = mu * (q_nope @ W_UK')   (Sec. 3.3 / 4 / 4.2)
//                 combine o = sum_i o_lat_i @ W_UV'[slice i]   (Sec. 4)
// Both are X[b, k] @ W[k, j] per head with W row-major (j contiguous), while
// the MFMA B operand wants 8 consecutive k per lane: the weight slab goes
// through LDS and comes back through the transposing read, which hands lane j
// the 4 rows of column j.  The float o_lat is split into two or three bf16 terms
// (an MFMA each), 16 or all 24 of its bits.
#include "lds_tile.h"
#include "split_merge.h"

#include <algorithm>

namespace tpla {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

#define TPLA_LDS4(p) ((__attribute__((address_space(3))) s16x4*)(p))

// B fragment (32 k-rows x 16 columns) of MFMA 16x16x32 from the slab.
// rows k0..k0+31, 16-byte piece pair (2*cb, 2*cb+1) of a PPR-piece row.
template <int PPR>
__device__ __forceinline__ bf16x8 read_b_frag(const char* slab, int k0, int cb, int j16, int q4) {
  const int r0 = k0 + 8 * q4 + (j16 >> 2);
  const int p = 2 * cb + ((j16 & 3) >> 1);
  const int byte = (j16 & 1) * 8;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      TPLA_LDS4(slab + (r0 * PPR + (p ^ wswz(r0))) * 16 + byte));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      TPLA_LDS4(slab + ((r0 + 4) * PPR + (p ^ wswz(r0 + 4))) * 16 + byte));
  const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

// ---------------------------------------------------------------------------
// absorb: grid (H, d_c / 128, Z); 4 waves, wave w owns columns 32w..32w+31 of the
// slab; LDS slab = W_UK'[h][0..d_n)[c0..c0+128).  A wave reads its columns back once, transposed, and keeps them in registers
// over its blocks of 16 sequences; batches of more than 32 sequences are
// dealt over Z workgroups per (head, column block), each staging the slab for itself
// (32 KB from L2): block mb goes to z = mb mod Z.  The weights are the M operand, so that a lane holds 8 adjacent
// columns of one sequence and stores them at once; with 2-byte stores of a column per lane 16 sequences took 4.8 us, 128
// sequences 11.3, with four slices 14.7.
// Latency bounds it (for one sequence 1.4 us from the start to the slab, which memory takes): whatever does not need the slab is done under its
// loads, the factor mu among it (indexed per lane it is a load from the arguments, which lie in host memory), and there is no division.
constexpr int AQ_COLS = 128;
template <int KS>                              // d_n = 32 KS
__global__ void __launch_bounds__(256) absorb_query_mfma_kernel(const bf16_t* __restrict__ q_nope,
                                                                const bf16_t* __restrict__ W, MuFactors mu,
                                                                bf16_t* __restrict__ q_lat, int B, int H, int d_c, int g) {
  extern __shared__ u32x4 slab4[];
  char* slab = reinterpret_cast<char*>(slab4);
  constexpr int PPR = AQ_COLS / 8, d_n = 32 * KS;   // 16 pieces per row
  const int h = blockIdx.x, c0 = blockIdx.y * AQ_COLS;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), j16 = lane & 15, q4 = lane >> 4;
  // the slab goes straight into LDS: instruction k fills pieces [64k, 64k + 64), rows 4k .. 4k + 3, the swizzle (the same for rows 16 apart) is
  // applied to the address each lane fetches from
  {
    const int r = 4 * wave + q4;
    const bf16_t* src = W + ((size_t)h * d_n + r) * d_c + c0 + 8 * (j16 ^ wswz(r));
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + (size_t)(16 * i) * d_c),
                                       (__attribute__((address_space(3))) void*)(slab + (wave + 4 * i) * 1024), 16, 0, 0);
  }
  const int n_mb = (B + 15) / 16, mb_step = gridDim.z;
  auto load_rows = [&](bf16x8 (&x)[KS], int mb) {
    const bf16_t* qrow = q_nope + ((size_t)min(16 * mb + j16, B - 1) * H + h) * d_n + 8 * q4;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) x[ks] = *reinterpret_cast<const bf16x8*>(qrow + 32 * ks);
  };
  // the first block's query rows are on their way while the slab lands
  bf16x8 x[KS];
  load_rows(x, blockIdx.z);                    // blockIdx.z < n_mb by the launch
  // lane i of a tile is column 8 (i >> 2) + 4 cb + (i & 3) of the wave's 32: a 4-column piece of the transposing read
  // is half of 16 bytes, and a lane ends up with 8 adjacent columns
  const int r0 = 8 * q4 + (j16 >> 2), piece = 4 * wave + (j16 & 3);
  const unsigned w_at = lds_at(slab) + (unsigned)((r0 * PPR + (piece ^ wswz(r0))) * 16);     // rows + 4: the same swizzle
  const int dl = d_c / g;
  int col = c0 + 32 * wave + 8 * q4, sl = 0;   // dl is a multiple of 16: the 8 are in one slice
  float m = mu.v[0];
#pragma unroll
  for (int i = 1; i < TPLA_MAX_G; ++i)
    if (col >= dl) {
      col -= dl;
      ++sl;
      m = mu.v[i];
    }
  bf16_t* const out = q_lat + ((size_t)sl * B * H + h) * dl + col;
  asm volatile("" : : "v"(m), "v"(out));
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  bf16x8 w[KS][2];
  static_for<KS>([&](auto ic) {
    constexpr int ks = decltype(ic)::value, W_STEP = 32 * PPR * 16;
    u32x2 v[2][2];
    static_for<2>([&](auto cc) {
      constexpr int cb = decltype(cc)::value;
      lds_read_tr_b64<ks * W_STEP + 8 * cb>(v[cb][0], w_at);
      lds_read_tr_b64<ks * W_STEP + 4 * PPR * 16 + 8 * cb>(v[cb][1], w_at);
    });
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      lds_wait<0>(v[cb][0], v[cb][1]);
      const u32x4 w4 = {v[cb][0][0], v[cb][0][1], v[cb][1][0], v[cb][1][1]};
      w[ks][cb] = __builtin_bit_cast(bf16x8, w4);
    }
  });
  for (int mb = blockIdx.z; mb < n_mb; mb += mb_step) {
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][cb], x[ks], acc[cb], 0, 0, 0);
    if (mb + mb_step < n_mb) load_rows(x, mb + mb_step);     // under this block's stores
    // acc[cb][i]: column col + 4 cb + i, sequence 16 mb + j16
    const int bb = 16 * mb + j16;
    if (bb < B) {
      bf16x8 y;
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = (bf16_t)(acc[e >> 2][e & 3] * m);
      *reinterpret_cast<bf16x8*>(out + (size_t)bb * H * dl) = y;
    }
  }
}

bool absorb_mfma_supported(const tpla_shape_t& sh) {
  return sh.dtype == TPLA_BF16 && sh.d_n % 32 == 0 && sh.d_n <= 256 && sh.d_c % AQ_COLS == 0 &&
         (sh.d_c / sh.g) % 16 == 0 && sh.d_c / AQ_COLS <= 65535;
}

int launch_absorb_query_mfma(const tpla_shape_t& sh, const void* q_nope, const void* W_UK_t,
                             const MuFactors& mu, void* q_lat, hipStream_t st) {
  const size_t smem = (size_t)sh.d_n * AQ_COLS * 2;
  const int n_mb = (sh.B + 15) / 16;
  // two blocks per workgroup, at most 8 deep; one block each while that is no more than two workgroups per compute
  // unit (64 heads, d_c = 512: 32 sequences 9.4 -> 7.6 us; 32 heads, 64 sequences: 8.0 -> 6.4; 64 heads, 128 sequences, where
  // it would be eight per compute unit: 14.4 with two blocks, 17.5 with one; all with 2-byte stores)
  int Z = n_mb <= 2 ? 1 : (n_mb + 1) / 2 < 8 ? (n_mb + 1) / 2 : 8;
  const long long per_block = (long long)sh.H * (sh.d_c / AQ_COLS);
  const int fit = (int)std::min<long long>(n_mb, std::max<long long>(1, 2LL * device_cu_count() / per_block));
  if (Z < fit) Z = fit < 8 ? fit : 8;
  typedef void (*Kernel)(const bf16_t*, const bf16_t*, MuFactors, bf16_t*, int, int, int, int);
  static const Kernel kernels[8] = {absorb_query_mfma_kernel<1>, absorb_query_mfma_kernel<2>, absorb_query_mfma_kernel<3>, absorb_query_mfma_kernel<4>,
                                    absorb_query_mfma_kernel<5>, absorb_query_mfma_kernel<6>, absorb_query_mfma_kernel<7>, absorb_query_mfma_kernel<8>};
  hipLaunchKernelGGL(kernels[sh.d_n / 32 - 1], dim3((unsigned)sh.H, (unsigned)(sh.d_c / AQ_COLS), (unsigned)Z), dim3(256), smem, st,
                     static_cast<const bf16_t*>(q_nope), static_cast<const bf16_t*>(W_UK_t), mu, static_cast<bf16_t*>(q_lat), sh.B, sh.H,
                     sh.d_c, sh.g);
  return check_launch("absorb_query_mfma_kernel");
}

// ---------------------------------------------------------------------------
// Combine  o = sum_i o_lat_i @ W_UV'[slice i], with the merge of the decode's partial results in front of
// it (MERGE: the partial results go straight into the product, o_lat and lse are written on the way) or
// without (o_lat is read).  Grid (H, ceil(B / spw), ceil(d_v / 128)): a workgroup owns one head, spw
// sequences and 128 output columns, and walks the latent axis in chunks.  Bound by latency and by
// what one compute unit can pull in (128 KB of weights and up to 128 KB of partial results each), so the
// two streams run side by side in waves of their own:
//   * waves 8..11 bring the chunk of W_UV'[h] into LDS with direct loads and wait for it;
//   * waves 0..7 merge.  A unit of work is (sequence, up to 256 consecutive latent columns of one
//     slice): one wave, its 64 lanes side by side along the row (split_merge.h).  Units of up to 16
//     slots are taken two or four at a time, with one load and one pass of arithmetic for the weights of
//     all: done unit by unit over 64 lanes, that arithmetic took most of the kernel on batches of many
//     sequences with two or three slots each.  With fewer than 8 units in a launch of fewer than 8 sequences per
//     workgroup the slots of a unit are dealt over 8 / units waves, which meet in LDS in slot order
//     (mc_waves_per_unit; the last sequences of a larger launch are merged a unit per wave).
// The merged rows go to LDS as three bf16 terms (A operands; widths of two terms, mc_terms, have kernels of their own below); wave w then owns output columns
// 16 w .. 16 w + 15 over the whole chunk: nothing is summed across waves.  The first terms have accumulators of their
// own: a product that is NaN only because of the low terms (an infinity leaves inf - inf behind it, or meets a low
// term of zero) takes the sum of the first terms, in which the finite products no longer matter.
// Three terms against the float FMAs before them, one slice of d_c = 256, 64 heads, 32 sequences: 14.7 -> 6.1 us (two terms:
// 4.8), 2-norm error against 64 bits 9.3e-8 -> 6.2e-8 (two terms: 2.5e-6), largest 5.6e-7 of the root mean square in both;
// with two instead of four partial sums of the first term 7.0e-8 and 7.0e-7.
// Before, one kernel did the same with the weights requested ahead of the merge by the same waves: loads
// complete in order, so the slot list and every (reference, sum) pair waited for 128 KB of weights, and
// a sequence was merged by four lanes with 16 scattered columns each.
constexpr int MC_LOAD_WAVES = 4;
constexpr int MC_THREADS = (MC_MERGE_WAVES + MC_LOAD_WAVES) * 64;

template <int SUBS, bool MERGE, typename OT>
__global__ void __launch_bounds__(MC_THREADS, MERGE ? 3 : 6) merge_combine_mfma_kernel(DecodeArgs a, const bf16_t* __restrict__ W,
                                                                        OT* __restrict__ o, int d_c, int d_v, int spw) {
  extern __shared__ u32x4 slab4[];            // weights [rows][16 pieces], A operands [term][spw][columns], join buffers
  char* slab = reinterpret_cast<char*>(slab4);
  constexpr int TERMS = 3, PPR = MC_COLS / 8, MC_ROWS = mc_rows(MERGE, TERMS);
  constexpr int SW = 256 / SUBS, LPR = 64 / SUBS;
  const int h = blockIdx.x, mb = blockIdx.y, col0 = blockIdx.z * MC_COLS;
  const int lane = threadIdx.x & 63, j16 = lane & 15, q4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int B = a.B, H = a.H, dl = a.dl;
  const int n_seq = min(spw, B - spw * mb);
  const McLds lds = mc_lds(MERGE, TERMS, spw, d_c);
  char* const xop = slab + lds.operands;
  char* const join = slab + lds.join;

  constexpr int CHAINS = 4;                   // partial sums over the k-steps
  f32x4 first[CHAINS], low[TERMS - 1][2];     // of the first term and of the others
#pragma unroll
  for (int i = 0; i < CHAINS; ++i) first[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 2 * (TERMS - 1); ++i) low[i >> 1][i & 1] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int kc = 0; kc < d_c; kc += MC_ROWS) {
    const int cols = min(MC_ROWS, d_c - kc);
    const int plane = spw * cols * 2;                        // bytes of one term
    const int xmask = cols % 128 ? 7 : 15;                   // piece swizzle: row & xmask
    if (kc > 0) __syncthreads();                             // everybody is done with the previous chunk
    // unit u: sequence u / n_pieces, piece u % n_pieces of the chunk (u < 128: a multiplication and a shift; an
    // integer division costs a wave a hundred cycles and there are several per unit)
    const int n_pieces = cols / SW;                          // at most 8
    const unsigned inv_pieces = (65536u + n_pieces - 1) / n_pieces;
    auto seq_of = [&](int u) -> int { return (int)(((unsigned)u * inv_pieces) >> 16); };
    const int n_units = n_seq * n_pieces;
    const int per_unit = mc_waves_per_unit(MERGE, TERMS, spw, n_units);
    const int sl_kc = kc / dl;
    auto locate = [&](int u, int& sl, int& col) {            // slice and first column in it of the piece of unit u
      sl = sl_kc;
      col = kc - sl_kc * dl + (u - seq_of(u) * n_pieces) * SW;
#pragma unroll
      for (int i = 1; i < MC_ROWS / SW; ++i)                 // a chunk reaches into that many further slices at most
        if (col >= dl) {
          col -= dl;
          ++sl;
        }
    };
    auto store_operand = [&](int u, const f32x4& x) {
      const int seq = seq_of(u), c = (u - seq * n_pieces) * SW + 4 * (lane % LPR);
      typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
      char* dst = xop + seq * cols * 2 + ((c >> 3) ^ (seq & xmask)) * 16 + (c & 4) * 2;
      f32x4 rest = x;
#pragma unroll
      for (int t = 0; t < TERMS; ++t) {
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = (bf16_t)rest[e];
          rest[e] -= (float)v[e];
        }
        if (!MERGE || lane < LPR) *reinterpret_cast<bf16x4*>(dst + t * plane) = v;
      }
    };
    auto finish = [&](int u, const f32x4& x) {               // merged values out, and into the A operands
      if (blockIdx.z == 0 && lane < LPR) {
        int sl, col;
        locate(u, sl, col);
        *reinterpret_cast<f32x4*>(a.o_lat + (((size_t)sl * B + spw * mb + seq_of(u)) * H + h) * dl + col + 4 * lane) = x;
      }
      store_operand(u, x);
    };
    auto finish_lse = [&](int u, float lse) {                // called by one lane per unit
      int sl, col;
      locate(u, sl, col);
      if (a.lse && blockIdx.z == 0 && col == 0) a.lse[((size_t)sl * B + spw * mb + seq_of(u)) * H + h] = lse;
    };
    if (wave >= MC_MERGE_WAVES) {
      // instruction k fills pieces [64k, 64k + 64): rows 4k .. 4k + 3; columns past d_v repeat the last ones
      const bf16_t* Wh = W + ((size_t)h * d_c + kc) * d_v;
#pragma unroll 8
      for (int k = wave - MC_MERGE_WAVES; k < cols * PPR / 64; k += MC_LOAD_WAVES) {
        const int r = 4 * k + q4, p = j16 ^ wswz(r);
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void*)(Wh + (size_t)r * d_v + min(col0 + 8 * p, d_v - 8)),
            (__attribute__((address_space(3))) void*)(slab + k * 1024), 16, 0, 0);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    } else if constexpr (!MERGE) {
      // lane group `sub` of the wave takes its own unit: SUBS units per wave and load
      for (int u0 = wave * SUBS; u0 < n_units; u0 += 4 * MC_MERGE_WAVES * SUBS) {
        f32x4 x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int u = min(u0 + i * MC_MERGE_WAVES * SUBS + lane / LPR, n_units - 1);
          int sl, col;
          locate(u, sl, col);
          x[i] = *reinterpret_cast<const f32x4*>(a.o_lat + (((size_t)sl * B + spw * mb + seq_of(u)) * H + h) * dl + col + 4 * (lane % LPR));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int u = u0 + i * MC_MERGE_WAVES * SUBS + lane / LPR;
          if (u < n_units) store_operand(u, x[i]);
        }
      }
    } else {
      // slots of the units u0, u0 + 8, ... (none for those past n_units)
      auto find = [&](int u0, auto& first, auto& cnt, auto& col) {
        constexpr int G = sizeof(first) / sizeof(int);
        int vb[G], bs[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const int u = min(u0 + g * MC_MERGE_WAVES, n_units - 1);
          int sl;
          locate(u, sl, col[g]);
          bs[g] = spw * mb + seq_of(u);
          vb[g] = sl * B + bs[g];
        }
        merge_slots(a, vb, bs, first, cnt);
#pragma unroll
        for (int g = 0; g < G; ++g)
          if (u0 + g * MC_MERGE_WAVES >= n_units) cnt[g] = 0;
      };
      auto merge_group = [&](auto groups, auto ahead, int u0) {
        constexpr int G = decltype(groups)::value, A = decltype(ahead)::value;
        int first[G], cnt[G], col[G], most = 0;
        find(u0, first, cnt, col);
#pragma unroll
        for (int g = 0; g < G; ++g) most = max(most, cnt[g]);
        if (most <= MERGE_SHORT) {
          f32x4 x[G];
          float lse;
          merge_short_pieces<SUBS, G, A>(a, h, 0, first, cnt, col, x, lse);
          const int ul = u0 + (lane >> 4) * MC_MERGE_WAVES;
          if ((lane & 15) == 0 && lane < 16 * G && ul < n_units) finish_lse(ul, lse);
#pragma unroll
          for (int g = 0; g < G; ++g)
            if (u0 + g * MC_MERGE_WAVES < n_units) finish(u0 + g * MC_MERGE_WAVES, x[g]);
        } else {
          for (int u = u0; u < min(n_units, u0 + G * MC_MERGE_WAVES); u += MC_MERGE_WAVES) {
            int f1[1], c1[1], k1[1];
            find(u, f1, c1, k1);
            MergedPiece r = merge_piece<SUBS>(a, h, f1[0], 0, c1[0], k1[0]);
            merge_normalise(r);
            if (lane == 0) finish_lse(u, merge_lse(r.M, r.l));
            finish(u, r.x);
          }
        }
      };
      if (per_unit > 1) {
        const int u = wave / per_unit, part = wave % per_unit;
        if (u < n_units) {
          int f1[1], c1[1], k1[1];
          find(u, f1, c1, k1);
          const MergedPiece r = merge_piece<SUBS>(a, h, f1[0], c1[0] * part / per_unit, c1[0] * (part + 1) / per_unit, k1[0]);
          *reinterpret_cast<f32x4*>(join + wave * 1024 + lane * 16) = r.x;
          if (lane == 0) *reinterpret_cast<float2*>(join + MC_MERGE_WAVES * 1024 + wave * 16) = make_float2(r.M, r.l);
        }
      } else if (n_units <= 2 * MC_MERGE_WAVES) {
        merge_group(std::integral_constant<int, 2>{}, std::integral_constant<int, 8 / SUBS>{}, wave);
      } else {
        for (int u0 = wave; u0 < n_units; u0 += 4 * MC_MERGE_WAVES)
          merge_group(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{}, u0);
      }
    }
    if (per_unit > 1) {
      __syncthreads();
      if (wave < n_units * per_unit && wave % per_unit == 0) {
        MergedPiece r;
        r.x = f32x4{0.f, 0.f, 0.f, 0.f};
        r.M = -INFINITY;
        r.l = 0.f;
        for (int w = wave; w < wave + per_unit; ++w) {
          const float2 ml = *reinterpret_cast<const float2*>(join + MC_MERGE_WAVES * 1024 + w * 16);
          merge_join(r, *reinterpret_cast<const f32x4*>(join + w * 1024 + lane * 16), ml.x, ml.y);
        }
        merge_normalise(r);
        if (lane == 0) finish_lse(wave / per_unit, merge_lse(r.M, r.l));
        finish(wave / per_unit, r.x);
      }
    }
    __syncthreads();                                         // weights and A operands are in place
    if (wave < MC_MERGE_WAVES) {
      // rows of the A tile past spw repeat the last one: an output row depends on its own row only, and these are not stored
      const int row = min(j16, spw - 1);
      const char* xrow = xop + row * cols * 2;
      for (int ks0 = 0; ks0 < cols / 32; ks0 += CHAINS) {
#pragma unroll
        for (int e = 0; e < CHAINS; ++e) {
          const int ks = ks0 + e;
          if (e >= 2 && ks >= cols / 32) break;              // cols is a multiple of 64
          const char* src = xrow + ((4 * ks + q4) ^ (row & xmask)) * 16;
          bf16x8 xt[TERMS];
#pragma unroll
          for (int t = 0; t < TERMS; ++t) xt[t] = *reinterpret_cast<const bf16x8*>(src + t * plane);
          const bf16x8 bf = read_b_frag<PPR>(slab, 32 * ks, wave, j16, q4);
          first[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[0], bf, first[e], 0, 0, 0);
#pragma unroll
          for (int t = 1; t < TERMS; ++t)
            low[t - 1][e & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[t], bf, low[t - 1][e & 1], 0, 0, 0);
        }
      }
    }
  }
  if (wave < MC_MERGE_WAVES) {
    f32x4 s1 = first[0] + first[1], s2 = low[1][0] + low[1][1];
    s1 += first[2] + first[3];
    s2 += low[0][0] + low[0][1];
    f32x4 t = s1 + s2;
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = t[i] == t[i] ? t[i] : s1[i];
    // t[i]: sequence spw mb + 4 q4 + i, column col0 + 16 wave + j16
    const int col = col0 + 16 * wave + j16;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * q4 + i < n_seq && col < d_v) store_from_f32(o + ((size_t)(spw * mb + 4 * q4 + i) * H + h) * d_v + col, t[i]);
  }
}

// One wave's 16 columns of the sum of the first terms' products (s1) and the others' (s2): sequences b0 + 4 q4 + i, column col.
__device__ __forceinline__ void store_combined(const f32x4& s1, const f32x4& s2, void* o, int o_bf16, int b0, int n_seq, int h, int H, int col,
                                               int d_v, int q4) {
  const f32x4 t = s1 + s2;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (4 * q4 + i < n_seq && col < d_v) {
      const float v = t[i] == t[i] ? t[i] : s1[i];
      const size_t at = ((size_t)(b0 + 4 * q4 + i) * H + h) * d_v + col;
      if (o_bf16)
        static_cast<bf16_t*>(o)[at] = (bf16_t)v;
      else
        static_cast<float*>(o)[at] = v;
    }
}

// The same with the merge for two terms (latent widths that are a multiple of 512, so that chunks are whole), without what the general kernel
// above finds out at run time: SUBS fixes the pieces of a chunk, the launch chooses how the units of work are dealt and the columns of a
// workgroup.  What bounds it is the chain slot list -> (reference, sum) pairs and rows -> LDS -> product, so everything a wave
// executes once counts: the general kernel's loop-invariant arithmetic alone (seven integer divisions, spilled scalars) held up the first
// request by 1.4 us, the weights by 2.0.  (The instances of PARTS > 1 spill 0 to 11 scalars, those with whole units per wave
// still 14 to 88, the general kernel 70 to 76.)
//   PARTS > 1: fewer than five units; the columns of a unit are dealt over PARTS waves (its slots, joined in LDS, before: 1.4 us more)
//   PARTS == 1: G units per wave at a time
//   COLS < 128: launches that would leave compute units idle: the weights of a head over several of them, each of which merges
// Kernel time in us, general kernel / COLS 128 / the column width chosen: 64 heads, one sequence of 1237 tokens 8.0 / 6.2 / 5.2 (32), two 8.0 / 6.4 / 5.7
// (64), three 8.4 / 6.5 / -, four 8.7 / 7.2 / -, one of 131072 10.8 / 9.4 / 8.8 (32); 16 heads, one of 5000 8.6 / 8.1 / 6.9 (32), four of 30000
// 7.4 / 6.3 / 5.5 (32).  23 ragged sequences of 64 heads 11.1 / 10.4 / -.  Where every compute unit has a workgroup (16 x 4096 tokens: 200 KB each)
// the streams take 3.8 of 6.4 us, some 7 TB/s of partial results and first reads of the weights, and little is gained.
template <int SUBS, int PARTS, int G, int COLS>
__global__ void __launch_bounds__(MC_THREADS, 3) merge_combine_pair_kernel(DecodeArgs a, const bf16_t* __restrict__ W, void* __restrict__ o,
                                                                           int d_c, int d_v, int spw, int o_bf16) {
  extern __shared__ u32x4 slab4[];            // weights [512][COLS / 8 pieces], A operands [2][spw][512]
  constexpr int ROWS = mc_rows(true, 2), PPR = COLS / 8, SW = 256 / SUBS, NP = ROWS / SW;
  asm volatile("" : : "s"(a.part_ml), "s"(a.o_lat), "s"(a.plan), "s"(a.n_shards), "s"(a.balanced), "s"(W), "s"(d_c));   // one wait for all arguments
  char* const slab = reinterpret_cast<char*>(slab4);
  char* const xop = slab + mc_lds(true, 2, 0, ROWS).operands;
  const int lane = threadIdx.x & 63, j16 = lane & 15, q4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = blockIdx.x, b0 = spw * blockIdx.y, col0 = blockIdx.z * COLS;
  const int plane = spw * ROWS * 2;                           // bytes of one term
  const int n_seq = min(spw, a.B - b0);
  f32x4 first[2], low[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) first[i] = low[i] = f32x4{0.f, 0.f, 0.f, 0.f};

  int sl_kc = 0, col_kc = 0;                                  // slice and column in it of the chunk's first
  for (int kc = 0; kc < d_c; kc += ROWS) {
    if (kc > 0) {
      lds_barrier();                                          // everybody is done with the previous chunk
      for (col_kc += ROWS; col_kc >= a.dl; col_kc -= a.dl) ++sl_kc;
    }
    if (wave >= MC_MERGE_WAVES) {
      // instruction k fills 64 pieces, 64 / PPR rows, and the wave every fourth: the rows of a lane are a multiple of 16 apart, so that
      // its swizzle is the same in all of them; columns past d_v repeat the last ones
      const int k = wave - MC_MERGE_WAVES, r = k * (64 / PPR) + lane / PPR, p = (lane % PPR) ^ (wswz(r) & (PPR - 1));
      const bf16_t* src = W + ((size_t)h * d_c + kc + r) * d_v + min(col0 + 8 * p, d_v - 8);
      const size_t step = (size_t)(MC_LOAD_WAVES * 64 / PPR) * d_v;
#pragma unroll 4
      for (int i = 0; i < ROWS * PPR / 64 / MC_LOAD_WAVES; ++i, src += step)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                         (__attribute__((address_space(3))) void*)(slab + (k + i * MC_LOAD_WAVES) * 1024), 16, 0, 0);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    } else {
      // unit u: sequence u / NP, piece u % NP of the chunk
      const int n_units = n_seq * NP;
      auto locate = [&](int u, int& sl, int& col) {
        sl = sl_kc;
        col = col_kc + u % NP * SW;
#pragma unroll
        for (int i = 1; i < NP; ++i)
          if (col >= a.dl) {
            col -= a.dl;
            ++sl;
          }
      };
      // columns [at, at + 4 lpr) of unit u, four per lane: merged values out, and into the A operands as two terms
      auto finish = [&](int u, int at, int lpr, const f32x4& x, bool has_lse, float lse) {
        if (lane < lpr) {
          const int c = u % NP * SW + at + 4 * lane, seq = u / NP;
          char* dst = xop + seq * (ROWS * 2) + ((c >> 3) ^ (seq & 15)) * 16 + (c & 4) * 2;
          bf16x4 v[2];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[0][e] = (bf16_t)x[e];
            v[1][e] = (bf16_t)(x[e] - (float)v[0][e]);
          }
          *reinterpret_cast<bf16x4*>(dst) = v[0];
          *reinterpret_cast<bf16x4*>(dst + plane) = v[1];
        }
        if (blockIdx.z == 0) {
          int sl, col;
          locate(u, sl, col);
          const size_t row = ((size_t)sl * a.B + b0 + u / NP) * a.H + h;
          if (lane < lpr) *reinterpret_cast<f32x4*>(a.o_lat + row * a.dl + col + at + 4 * lane) = x;
          if (has_lse && col + at == 0 && a.lse) a.lse[row] = lse;
        }
      };
      if constexpr (PARTS > 1) {
        constexpr int S = SUBS * PARTS;
        const int u = wave / PARTS, at = wave % PARTS * (SW / PARTS);
        if (u < n_units) {
          int sl, col, f1[1], c1[1];
          locate(u, sl, col);
          const int b1[1] = {b0 + u / NP}, v1[1] = {sl * a.B + b1[0]};
          merge_slots(a, v1, b1, f1, c1);
          MergedPiece r = merge_piece<S, 8>(a, h, f1[0], 0, c1[0], col + at);
          merge_normalise(r);
          finish(u, at, 64 / S, r.x, lane == 0, merge_lse(r.M, r.l));
        }
      } else {
        for (int u0 = wave; u0 < n_units; u0 += G * MC_MERGE_WAVES) {
          // units u0, u0 + 8, ...: no slots for those past n_units
          int vb[G], bs[G], col[G], first_slot[G], cnt[G], most = 0;
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const int u = min(u0 + g * MC_MERGE_WAVES, n_units - 1);
            int sl;
            locate(u, sl, col[g]);
            bs[g] = b0 + u / NP;
            vb[g] = sl * a.B + bs[g];
          }
          merge_slots(a, vb, bs, first_slot, cnt);
#pragma unroll
          for (int g = 0; g < G; ++g) {
            if (u0 + g * MC_MERGE_WAVES >= n_units) cnt[g] = 0;
            most = max(most, cnt[g]);
          }
          if (most <= MERGE_SHORT) {
            f32x4 x[G];
            float lse;
            merge_short_pieces<SUBS, G, G == 1 ? 16 / SUBS : G == 2 ? 8 / SUBS : 4>(a, h, 0, first_slot, cnt, col, x, lse);
#pragma unroll
            for (int g = 0; g < G; ++g)
              if (u0 + g * MC_MERGE_WAVES < n_units)
                finish(u0 + g * MC_MERGE_WAVES, 0, 64 / SUBS, x[g], lane == 16 * g, lse);
          } else {
#pragma unroll
            for (int g = 0; g < G; ++g)
              if (u0 + g * MC_MERGE_WAVES < n_units) {
                MergedPiece r = merge_piece<SUBS>(a, h, first_slot[g], 0, cnt[g], col[g]);
                merge_normalise(r);
                finish(u0 + g * MC_MERGE_WAVES, 0, 64 / SUBS, r.x, lane == 0, merge_lse(r.M, r.l));
              }
          }
        }
      }
    }
    lds_barrier();                                            // weights and A operands are in place
    if (wave < COLS / 16) {
      // rows of the A tile past spw repeat the last one: an output row depends on its own row only, and these are not stored
      const int row = min(j16, spw - 1), r0 = 8 * q4 + (j16 >> 2);
      const unsigned x_at = lds_at(xop) + (unsigned)(row * (ROWS * 2) + (q4 ^ (row & 15)) * 16);       // k-step ks: ^ 64 (ks & 3), + 256 (ks >> 2)
      const unsigned w_at = lds_at(slab) + (unsigned)((r0 * PPR + ((2 * wave + ((j16 & 3) >> 1)) ^ (wswz(r0) & (PPR - 1)))) * 16 + (j16 & 1) * 8);
      // three k-steps on their way: read one after the other they were most of this phase
      constexpr int NK = ROWS / 32, R = 3;
      bf16x8 xt[R][2];
      u32x2 wlo[R], whi[R];
      auto read = [&](auto ic) {
        constexpr int i = decltype(ic)::value, at = i % R, W_STEP = 32 * PPR * 16;
        const unsigned x0 = (x_at ^ (64u * (i & 3)));
        lds_read_b128<256 * (i >> 2)>(xt[at][0], x0);
        lds_read_b128<256 * (i >> 2)>(xt[at][1], x0 + plane);
        const unsigned w0 = w_at + (unsigned)((i >> 1) * (2 * W_STEP));
        lds_read_tr_b64<(i & 1) * W_STEP>(wlo[at], w0);
        lds_read_tr_b64<(i & 1) * W_STEP + 4 * PPR * 16>(whi[at], w0);
      };
      static_for<R>(read);
      static_for<NK>([&](auto ic) {
        constexpr int i = decltype(ic)::value, at = i % R;
        constexpr int ahead = (NK - 1 - i) < R - 1 ? (NK - 1 - i) : R - 1;
        lds_wait<4 * ahead>(wlo[at], whi[at]);
        lds_wait<4 * ahead>(xt[at][0]);
        lds_wait<4 * ahead>(xt[at][1]);
        const u32x4 w4 = {wlo[at][0], wlo[at][1], whi[at][0], whi[at][1]};
        first[i & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[at][0], __builtin_bit_cast(bf16x8, w4), first[i & 1], 0, 0, 0);
        low[i & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[at][1], __builtin_bit_cast(bf16x8, w4), low[i & 1], 0, 0, 0);
        if constexpr (i + R < NK) read(std::integral_constant<int, i + R>{});
      });
    }
  }
  if (wave < COLS / 16) {
    store_combined(first[0] + first[1], low[0] + low[1], o, o_bf16, b0, n_seq, h, a.H, col0 + 16 * wave + j16, d_v, q4);
  }
}

// Combine alone for latent widths that are a multiple of 256, as merge_combine_pair_kernel without the merge: a wave brings whole rows of a
// chunk, four columns per lane, whatever slices they lie in.  General kernel / this one, us: 32 sequences of one
// 256-wide slice, 64 heads 6.0 / 5.2 (weights and rows 2.5, the rest start, product and end), 128 of four 128-wide slices 15.7 / 11.3 (82 MB through
// L2: two workgroups per compute unit).
template <int TERMS>
__global__ void __launch_bounds__(MC_THREADS, 6) combine_rows_kernel(DecodeArgs a, const bf16_t* __restrict__ W, void* __restrict__ o, int d_c,
                                                                     int d_v, int spw, int o_bf16) {
  extern __shared__ u32x4 slab4[];            // weights [256][16 pieces], A operands [TERMS][spw][256]
  constexpr int ROWS = mc_rows(false, TERMS), PPR = MC_COLS / 8;
  static_assert(ROWS == 4 * 64, "a row of a chunk is four columns per lane");
  asm volatile("" : : "s"(a.o_lat), "s"(a.B), "s"(W), "s"(d_c));       // one wait for all arguments
  char* const slab = reinterpret_cast<char*>(slab4);
  char* const xop = slab + mc_lds(false, TERMS, 0, ROWS).operands;
  const int lane = threadIdx.x & 63, j16 = lane & 15, q4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = blockIdx.x, b0 = spw * blockIdx.y, col0 = blockIdx.z * MC_COLS;
  const int plane = spw * ROWS * 2;                           // bytes of one term
  const int n_seq = min(spw, a.B - b0);
  constexpr int CHAINS = TERMS == 3 ? 4 : 2, LOWS = TERMS == 3 ? 1 : 2;        // partial sums of the first term and of each other one
  f32x4 first[CHAINS], low[TERMS - 1][LOWS];
#pragma unroll
  for (int i = 0; i < CHAINS; ++i) first[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < LOWS * (TERMS - 1); ++i) low[i / LOWS][i % LOWS] = f32x4{0.f, 0.f, 0.f, 0.f};

  int sl = 0, col = 4 * lane;                                 // slice and column in it of this lane's four
  for (int kc = 0; kc < d_c; kc += ROWS) {
    if (kc > 0) {
      lds_barrier();                                          // everybody is done with the previous chunk
      col += ROWS;
    }
    if (wave >= MC_MERGE_WAVES) {
      // as in merge_combine_pair_kernel
      const int k = wave - MC_MERGE_WAVES, r = k * 4 + q4, p = j16 ^ wswz(r);
      const bf16_t* src = W + ((size_t)h * d_c + kc + r) * d_v + min(col0 + 8 * p, d_v - 8);
      const size_t step = (size_t)(MC_LOAD_WAVES * 4) * d_v;
#pragma unroll 4
      for (int i = 0; i < ROWS / 4 / MC_LOAD_WAVES; ++i, src += step)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                         (__attribute__((address_space(3))) void*)(slab + (k + i * MC_LOAD_WAVES) * 1024), 16, 0, 0);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    } else {
      while (__any(col >= a.dl))
        if (col >= a.dl) {
          col -= a.dl;
          ++sl;
        }
      const float* src = a.o_lat + (((size_t)sl * a.B + b0) * a.H + h) * a.dl + col;
      const size_t next = (size_t)a.H * a.dl;                 // to the next sequence
      f32x4 x[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) x[i] = *reinterpret_cast<const f32x4*>(src + min(wave + i * MC_MERGE_WAVES, n_seq - 1) * next);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int seq = wave + i * MC_MERGE_WAVES;
        if (seq < n_seq) {
          char* dst = xop + seq * (ROWS * 2) + ((lane >> 1) ^ (seq & 15)) * 16 + (lane & 1) * 8;
#pragma unroll
          for (int t = 0; t < TERMS; ++t) {
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              v[e] = (bf16_t)x[i][e];
              x[i][e] -= (float)v[e];
            }
            *reinterpret_cast<bf16x4*>(dst + t * plane) = v;
          }
        }
      }
    }
    lds_barrier();                                            // weights and A operands are in place
    if (wave < MC_MERGE_WAVES) {
      const int row = min(j16, spw - 1), r0 = 8 * q4 + (j16 >> 2);
      const unsigned x_at = lds_at(xop) + (unsigned)(row * (ROWS * 2) + (q4 ^ (row & 15)) * 16);       // k-step ks: ^ 64 (ks & 3), + 256 (ks >> 2)
      const unsigned w_at = lds_at(slab) + (unsigned)((r0 * PPR + ((2 * wave + ((j16 & 3) >> 1)) ^ wswz(r0))) * 16 + (j16 & 1) * 8);
      constexpr int NK = ROWS / 32, R = 5 - TERMS, OPS = TERMS + 2;       // (with three terms two registers are kept in scratch over a chunk's product)
      bf16x8 xt[R][TERMS];
      u32x2 wlo[R], whi[R];
      auto read = [&](auto ic) {
        constexpr int i = decltype(ic)::value, at = i % R, W_STEP = 32 * PPR * 16;
        const unsigned x0 = x_at ^ (64u * (i & 3));
#pragma unroll
        for (int t = 0; t < TERMS; ++t) lds_read_b128<256 * (i >> 2)>(xt[at][t], x0 + t * plane);
        const unsigned w0 = w_at + (unsigned)((i >> 2) * (4 * W_STEP));
        lds_read_tr_b64<(i & 3) * W_STEP>(wlo[at], w0);
        lds_read_tr_b64<(i & 3) * W_STEP + 4 * PPR * 16>(whi[at], w0);
      };
      static_for<R>(read);
      static_for<NK>([&](auto ic) {
        constexpr int i = decltype(ic)::value, at = i % R;
        constexpr int ahead = (NK - 1 - i) < R - 1 ? (NK - 1 - i) : R - 1;
        lds_wait<OPS * ahead>(wlo[at], whi[at]);
#pragma unroll
        for (int t = 0; t < TERMS; ++t) lds_wait<OPS * ahead>(xt[at][t]);
        const u32x4 w4 = {wlo[at][0], wlo[at][1], whi[at][0], whi[at][1]};
        const bf16x8 bf = __builtin_bit_cast(bf16x8, w4);
        first[i % CHAINS] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[at][0], bf, first[i % CHAINS], 0, 0, 0);
#pragma unroll
        for (int t = 1; t < TERMS; ++t)
          low[t - 1][i % LOWS] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[at][t], bf, low[t - 1][i % LOWS], 0, 0, 0);
        if constexpr (i + R < NK) read(std::integral_constant<int, i + R>{});
      });
    }
  }
  if (wave < MC_MERGE_WAVES) {
    f32x4 s1 = first[0] + first[1], s2;
    if constexpr (TERMS == 3) {
      s1 += first[2] + first[3];
      s2 = low[1][0] + low[0][0];
    } else {
      s2 = low[0][0] + low[0][1];
    }
    store_combined(s1, s2, o, o_bf16, b0, n_seq, h, a.H, col0 + 16 * wave + j16, d_v, q4);
  }
}

bool merge_combine_mfma_supported(const tpla_shape_t& sh) {
  return sh.dtype == TPLA_BF16 && sh.d_v % 8 == 0 && merge_piece_width(sh.d_c / sh.g, sh.H) > 0 &&
         (sh.d_v + MC_COLS - 1) / MC_COLS <= 65535 && sh.B <= 65535;
}

// Merge and combine as one kernel, or the stand-alone merge and then the combine.  The fused kernel's workgroups fill
// a compute unit's LDS, so it pays while they run in one round (of up to 16 sequences each, as the launch then takes
// them); a second round starts its chain of round trips (slot list, weights, rows) over with nothing beside it, which
// merge_combine_pair_kernel makes up for where its pieces are 256 wide and its workgroups are not nearly full.  Layer-step behind other caches,
// separate kernels / two rounds, us: 64 heads, two slices, 80 sequences of 400 tokens 46.1 / 42.3, of 500 to 6000 81.3 / 77.8, 112 (14 per workgroup) 104.1 / 99.6, 120
// 105.9 / 106.8, 128 of 400 48.9 / 50.5; 128 heads, 40 71.9 / 68.3, 48 (12 per workgroup) 79.9 / 76.2, one slice 93.2 / 91.2, 52 98.9 / 100.5, 64 112.0 / 113.8; 32 heads, one slice,
// 240 (15) 165.8 / 161.7, 256 of 400 56.9 / 58.5; four 128-wide slices, 128 sequences of 1024 to 131072 909 / 915, 128 heads (four rounds) 214 / 226.
static bool merge_combine_rounds(const tpla_shape_t& sh, int n) {
  return (long long)sh.H * ((sh.d_v + MC_COLS - 1) / MC_COLS) * ((sh.B + 15) / 16) <= (long long)n * device_cu_count();
}
bool merge_combine_in_one_round(const tpla_shape_t& sh) { return merge_combine_rounds(sh, 1); }
// Sequences per workgroup with the merge: as few as still make one round of workgroups, or two (merge_combine_pays).
// Layer-step, two slices, contexts of 800 to 2500 tokens, against the largest power of two up to 8 that gives every compute
// unit a workgroup: 16 heads, 33 sequences 43.1 -> 36.7 us; 32 heads, 24 sequences 42.2 -> 36.2; 64 heads, four slices,
// 64 sequences of 170 to 500 tokens 50.6 -> 47.9.
static int merge_combine_sequences(const tpla_shape_t& sh) {
  const long long per_block = (long long)sh.H * ((sh.d_v + MC_COLS - 1) / MC_COLS);
  const long long most = (merge_combine_in_one_round(sh) ? 1LL : 2LL) * device_cu_count();
  int spw = 1;
  while (spw < 16 && per_block * ((sh.B + spw - 1) / spw) > most) ++spw;
  return spw;
}

bool merge_combine_pays(const tpla_shape_t& sh) {
  if (merge_combine_in_one_round(sh)) return true;
  const long long per_block = (long long)sh.H * ((sh.d_v + MC_COLS - 1) / MC_COLS);
  return mc_terms(sh.d_c, sh.d_v) == 2 && merge_piece_width(sh.d_c / sh.g, sh.H) == 256 && merge_combine_rounds(sh, 2) &&
         merge_combine_sequences(sh) <= 16 - (per_block + 31) / 32;
}

template <int SUBS, int PARTS, int G, int COLS = MC_COLS>
static int launch_merge_combine_pair(const DecodeArgs& a, const tpla_shape_t& sh, const void* W_UV_t, void* o, int o_dtype, int spw, hipStream_t st) {
  constexpr int most = mc_lds(true, 2, 16, mc_rows(true, 2)).bytes;
  static_assert(most <= 160 * 1024, "one workgroup's LDS");
  const int rc = allow_lds(reinterpret_cast<const void*>(merge_combine_pair_kernel<SUBS, PARTS, G, COLS>), most, "merge_combine_pair_kernel");
  if (rc) return rc;
  const dim3 grid((unsigned)sh.H, (unsigned)((sh.B + spw - 1) / spw), (unsigned)((sh.d_v + COLS - 1) / COLS));
  hipLaunchKernelGGL((merge_combine_pair_kernel<SUBS, PARTS, G, COLS>), grid, dim3(MC_THREADS), (size_t)mc_lds(true, 2, spw, sh.d_c).bytes, st, a,
                     static_cast<const bf16_t*>(W_UV_t), o, sh.d_c, sh.d_v, spw, (int)(o_dtype == TPLA_BF16));
  return check_launch("merge_combine_pair_kernel");
}
template <int SUBS>
static int launch_merge_combine_pairs(const DecodeArgs& a, const tpla_shape_t& sh, const void* W_UV_t, void* o, int o_dtype, int spw, hipStream_t st) {
  constexpr int PARTS = SUBS < 4 ? 4 / SUBS : 1;             // of one sequence's units
  if (spw == 1) {
    const long long rows = (long long)sh.H * sh.B;
    if (rows * ((sh.d_v + 31) / 32) <= device_cu_count()) return launch_merge_combine_pair<SUBS, PARTS, 1, 32>(a, sh, W_UV_t, o, o_dtype, spw, st);
    if (rows * ((sh.d_v + 63) / 64) <= device_cu_count()) return launch_merge_combine_pair<SUBS, PARTS, 1, 64>(a, sh, W_UV_t, o, o_dtype, spw, st);
    return launch_merge_combine_pair<SUBS, PARTS, 1>(a, sh, W_UV_t, o, o_dtype, spw, st);
  }
  const int units = spw * 2 * SUBS;
  if constexpr (SUBS == 1)
    if (spw == 2) return launch_merge_combine_pair<1, 2, 1>(a, sh, W_UV_t, o, o_dtype, spw, st);
  if (units <= MC_MERGE_WAVES) return launch_merge_combine_pair<SUBS, 1, 1>(a, sh, W_UV_t, o, o_dtype, spw, st);
  if (units <= 2 * MC_MERGE_WAVES) return launch_merge_combine_pair<SUBS, 1, 2>(a, sh, W_UV_t, o, o_dtype, spw, st);
  return launch_merge_combine_pair<SUBS, 1, 4>(a, sh, W_UV_t, o, o_dtype, spw, st);
}

// Without: as many as still give every compute unit a workgroup (two, for 16: the weights of a head are fetched once per workgroup).
static int combine_sequences(const tpla_shape_t& sh) {
  const long long per_block = (long long)sh.H * ((sh.d_v + MC_COLS - 1) / MC_COLS);
  int spw = per_block * ((sh.B + 15) / 16) >= 2LL * device_cu_count() ? 16 : 8;
  while (spw > 1 && spw < 16 && (spw / 2 >= sh.B || per_block * ((sh.B + spw - 1) / spw) < device_cu_count())) spw /= 2;
  return spw;
}

template <int TERMS>
static int launch_combine_rows(const DecodeArgs& a, const tpla_shape_t& sh, const void* W_UV_t, void* o, int o_dtype, hipStream_t st) {
  const int spw = combine_sequences(sh);
  constexpr int most = mc_lds(false, TERMS, 16, mc_rows(false, TERMS)).bytes;
  static_assert((TERMS == 2 ? 2 : 1) * most <= 160 * 1024, "LDS of two workgroups, of one with three terms");
  const int rc = allow_lds(reinterpret_cast<const void*>(combine_rows_kernel<TERMS>), most, "combine_rows_kernel");
  if (rc) return rc;
  const dim3 grid((unsigned)sh.H, (unsigned)((sh.B + spw - 1) / spw), (unsigned)((sh.d_v + MC_COLS - 1) / MC_COLS));
  hipLaunchKernelGGL(combine_rows_kernel<TERMS>, grid, dim3(MC_THREADS), (size_t)mc_lds(false, TERMS, spw, sh.d_c).bytes, st, a,
                     static_cast<const bf16_t*>(W_UV_t), o, sh.d_c, sh.d_v, spw, (int)(o_dtype == TPLA_BF16));
  return check_launch("combine_rows_kernel");
}

template <int SUBS, bool MERGE, typename OT>
static int launch_merge_combine_t(const DecodeArgs& a, const tpla_shape_t& sh, const void* W_UV_t, OT* o, hipStream_t st) {
  constexpr int TERMS = 3;
  const int spw = MERGE ? merge_combine_sequences(sh) : combine_sequences(sh);
  const size_t smem = (size_t)mc_lds(MERGE, TERMS, spw, sh.d_c).bytes;
  constexpr int most = mc_lds(MERGE, TERMS, 16, mc_rows(MERGE, TERMS)).bytes;
  static_assert(most <= 160 * 1024 && mc_lds(MERGE, TERMS, MC_MERGE_WAVES - 1, mc_rows(MERGE, TERMS)).bytes <= most, "one workgroup's LDS");
  const int rc = allow_lds(reinterpret_cast<const void*>(merge_combine_mfma_kernel<SUBS, MERGE, OT>), most, "merge_combine_mfma_kernel");
  if (rc) return rc;
  const dim3 grid((unsigned)sh.H, (unsigned)((sh.B + spw - 1) / spw), (unsigned)((sh.d_v + MC_COLS - 1) / MC_COLS));
  hipLaunchKernelGGL((merge_combine_mfma_kernel<SUBS, MERGE, OT>), grid, dim3(MC_THREADS), smem, st, a,
                     static_cast<const bf16_t*>(W_UV_t), o, sh.d_c, sh.d_v, spw);
  return check_launch("merge_combine_mfma_kernel");
}

template <bool MERGE, typename OT>
static int launch_merge_combine_to(const DecodeArgs& a, const tpla_shape_t& sh, const void* W_UV_t, OT* o, hipStream_t st) {
  const int width = merge_piece_width(sh.d_c / sh.g, sh.H);
  if constexpr (MERGE)                       // (without the merge all widths of 256-wide pieces are combine_rows_kernel's)
    if (width == 256) return launch_merge_combine_t<1, MERGE>(a, sh, W_UV_t, o, st);
  return width == 128 ? launch_merge_combine_t<2, MERGE>(a, sh, W_UV_t, o, st) : launch_merge_combine_t<4, MERGE>(a, sh, W_UV_t, o, st);
}

int launch_merge_combine_mfma(const DecodeArgs& a, const tpla_shape_t& sh, const void* W_UV_t, void* o, int o_dtype,
                              hipStream_t st) {
  if (mc_terms(sh.d_c, sh.d_v) == 2) {
    const int spw = merge_combine_sequences(sh);
    switch (merge_piece_width(sh.d_c / sh.g, sh.H)) {
      case 256: return launch_merge_combine_pairs<1>(a, sh, W_UV_t, o, o_dtype, spw, st);
      case 128: return launch_merge_combine_pairs<2>(a, sh, W_UV_t, o, o_dtype, spw, st);
      default: return launch_merge_combine_pairs<4>(a, sh, W_UV_t, o, o_dtype, spw, st);
    }
  }
  if (o_dtype == TPLA_BF16) return launch_merge_combine_to<true>(a, sh, W_UV_t, static_cast<bf16_t*>(o), st);
  return launch_merge_combine_to<true>(a, sh, W_UV_t, static_cast<float*>(o), st);
}

bool combine_mfma_supported(const tpla_shape_t& sh) { return merge_combine_mfma_supported(sh); }

int launch_combine_shards_mfma(const tpla_shape_t& sh, const float* o_lat, const void* W_UV_t, void* o, int o_dtype,
                               hipStream_t st) {
  DecodeArgs a = {};
  a.o_lat = const_cast<float*>(o_lat);      // only read
  a.B = sh.B;
  a.H = sh.H;
  a.dl = sh.d_c / sh.g;
  if (sh.d_c % 256 == 0)
    return mc_terms(sh.d_c, sh.d_v) == 2 ? launch_combine_rows<2>(a, sh, W_UV_t, o, o_dtype, st) : launch_combine_rows<3>(a, sh, W_UV_t, o, o_dtype, st);
  if (o_dtype == TPLA_BF16) return launch_merge_combine_to<false>(a, sh, W_UV_t, static_cast<bf16_t*>(o), st);
  return launch_merge_combine_to<false>(a, sh, W_UV_t, static_cast<float*>(o), st);
}

// ---------------------------------------------------------------------------
// Output projection  out[b, n] = sum_k x[b, k] W[k, n]  (x = the combined
// per-head outputs flattened to [B, H d_v], W = W_O [H d_v, D]; Sec. 3.3: the
// value up-projection is not merged into W_O, so this runs after the combine).
// A weight-streaming skinny GEMM: grid (D / 128, KSPLIT); a workgroup owns 128
// output columns and one contiguous k-range and walks it in chunks of OP_ROWS
// rows.  A chunk = the weight rows (16 KB) and the matching columns of 16 MB rows
// of x (4 MB KB, float), both brought in by direct-to-LDS loads into a ring of
// buffers by four waves of their own, so that two or three chunks per workgroup are in
// flight whatever the others are doing, and every vector-memory operation of those four is
// one of these loads (the wait counts below rely on that).  Each of the other four owns 64 columns and half of
// the rows over a whole chunk: no sum across waves, and x, which is split into bf16
// hi + lo (two MFMAs, so that the product keeps float accuracy), is read and split
// twice per workgroup instead of four times.  The float partial tiles of
// the KSPLIT ranges are summed in order by a second kernel.
// What bounds it is the stream of weights, so a pass takes as many rows as the LDS has room for (MB = 2, 4 or 8 blocks of
// 16): passes of 32 rows at any B read W_O again for each.  The loads have waves of their own because the others
// would stand at 6 to 12 of them per chunk (128 sequences: this kernel 65 -> 46 us, two load waves the same; 23: 24.0 -> 23.1).
// Whole attention blocks before / now, short contexts, D = 7168 and 64 heads: 33 sequences 86 / 63 us, 64 98 / 73, 128 177 / 111;
// 70 of 32 heads 84 / 59; D = 2048: 48 of 32 heads 52 / 42, 128 of 16 heads 62 / 53.
constexpr int OP_COLS = 128;
constexpr int OP_ROWS = 64;
constexpr int OP_W_BYTES = OP_ROWS * OP_COLS * 2;     // 16 rows of 16 pieces per KB: 16 instructions
constexpr int OP_WAVES = 4, OP_LOAD_WAVES = 4, OP_THREADS = (OP_WAVES + OP_LOAD_WAVES) * 64;
constexpr int op_stage(int mb) { return OP_W_BYTES + mb * 16 * OP_ROWS * 4; }     // rows of x: 16 pieces each
constexpr int op_stages(int mb) { return mb > 4 ? 3 : 4; }

template <int OFF>
__device__ __forceinline__ void lds_read_f4(f32x4& dst, unsigned addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
}

// Registers that an earlier wait covers: their consumers cannot be scheduled before it.
template <typename V>
__device__ __forceinline__ void lds_landed(V& a, V& b) {
  asm volatile("" : "+v"(a), "+v"(b));
}

template <int MB>
__global__ void __launch_bounds__(OP_THREADS) output_projection_mfma_kernel(const float* __restrict__ x,
                                                                        const bf16_t* __restrict__ W,
                                                                        float* __restrict__ part, int B, int K,
                                                                        int N, int k_per_split) {
  extern __shared__ u32x4 ring4[];                 // NST stages of [W chunk | x chunk]
  constexpr int NST = op_stages(MB), STAGE = op_stage(MB), MW = MB / 2;
  constexpr int W_LOADS = OP_W_BYTES / 1024 / OP_LOAD_WAVES, X_LOADS = 4 * MB / OP_LOAD_WAVES;   // per load wave and chunk
  constexpr int LOADS = W_LOADS + X_LOADS;
  static_assert(NST == 3 || NST == 4, "the wait counts cover one or two younger chunks");
  static_assert((NST - 2) * LOADS < 64, "the counter's range");
  char* ring = reinterpret_cast<char*>(ring4);
  const unsigned lds_base = (unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)ring4);
  const int c0 = blockIdx.x * OP_COLS, kz = blockIdx.y;
  const int k_begin = kz * k_per_split;
  const int n_chunks = k_per_split / OP_ROWS;
  const int tid = threadIdx.x, lane = tid & 63, j16 = lane & 15, q4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row_half = (wave >> 1) & 1, col_half = wave & 1;
  const int n_mb = (B + 15) / 16;

  // LDS read offsets.  Weights: rows 32 ks + 8 q4 + (j16 >> 2) (+4), piece pair of column block
  // 4 col_half + cb.  x: row 16 m + j16, pieces 8 ks + 2 q4 + {0, 1}, stored at piece ^ (row & 15).
  const int r0 = 8 * q4 + (j16 >> 2);
  unsigned b_off[4], a_off[2][2];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
    b_off[cb] = (unsigned)((r0 * 16 + ((2 * (4 * col_half + cb) + ((j16 & 3) >> 1)) ^ wswz(r0))) * 16 + (j16 & 1) * 8);
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      a_off[ks][h] = (unsigned)(OP_W_BYTES + row_half * MW * 4096 + (j16 * 16 + ((8 * ks + 2 * q4 + h) ^ j16)) * 16);

  if (wave >= OP_WAVES) {
    // Instruction k of a region fills its pieces [64k, 64k + 64): row 4k + q4, position j16.  This wave issues
    // k = lw + 4 j, i.e. rows 4 lw + q4 + 16 j; the piece that belongs at position j16 of such a row is
    // j16 ^ swizzle(row), the same for every j.
    static_assert(OP_LOAD_WAVES == 4, "rows 16 apart from j to j");
    const int lw = wave - OP_WAVES, wr = 4 * lw + q4;
    const char* w_src = reinterpret_cast<const char*>(W + (size_t)(k_begin + wr) * N + c0 + 8 * (j16 ^ wswz(wr)));
    const size_t w_rows16 = (size_t)16 * N * 2, w_chunk = (size_t)OP_ROWS * N * 2;
    for (int mb0 = 0; mb0 < n_mb; mb0 += MB) {
      const char* x_src[X_LOADS];
#pragma unroll
      for (int j = 0; j < X_LOADS; ++j) {
        const int bl = wr + 16 * j;                  // row of the x chunk
        const int b = min(16 * mb0 + bl, B - 1);     // rows past the batch repeat the last one, never stored
        x_src[j] = reinterpret_cast<const char*>(x + (size_t)b * K + k_begin + 4 * (j16 ^ (bl & 15)));
      }
      auto issue = [&](int t) {
        char* dst = ring + (t % NST) * STAGE + lw * 1024;
#pragma unroll
        for (int j = 0; j < W_LOADS; ++j)
          __builtin_amdgcn_global_load_lds(
              (const __attribute__((address_space(1))) void*)(w_src + (size_t)t * w_chunk + j * w_rows16),
              (__attribute__((address_space(3))) void*)(dst + j * 4096), 16, 0, 2 /* streaming: the weights are read once */);
#pragma unroll
        for (int j = 0; j < X_LOADS; ++j)
          __builtin_amdgcn_global_load_lds(
              (const __attribute__((address_space(1))) void*)(x_src[j] + (size_t)t * (OP_ROWS * 4)),
              (__attribute__((address_space(3))) void*)(dst + OP_W_BYTES + j * 4096), 16, 0, 0);
      };
      __builtin_amdgcn_s_barrier();            // the previous pass is done with LDS
#pragma unroll
      for (int t = 0; t < NST - 1; ++t)
        if (t < n_chunks) issue(t);
      for (int t = 0; t < n_chunks; ++t) {
        // chunk t has landed once only the loads of the chunks requested after it are outstanding
        switch (min(n_chunks - 1 - t, NST - 2)) {
          case 0: __builtin_amdgcn_s_waitcnt(vmcnt_imm(0)); break;
          case 1: __builtin_amdgcn_s_waitcnt(vmcnt_imm(LOADS)); break;
          default: __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * LOADS)); break;
        }
        __builtin_amdgcn_s_barrier();          // chunk t visible to all waves, chunk t-1 no longer read
        if (t + NST - 1 < n_chunks) issue(t + NST - 1);
      }
    }
    return;
  }

  for (int mb0 = 0; mb0 < n_mb; mb0 += MB) {
    f32x4 acc[MW][4];
#pragma unroll
    for (int m = 0; m < MW; ++m)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) acc[m][cb] = f32x4{0.f, 0.f, 0.f, 0.f};

    __builtin_amdgcn_s_barrier();              // every read of the previous pass has been waited for
    for (int t = 0; t < n_chunks; ++t) {
      __builtin_amdgcn_s_barrier();            // chunk t is in place
      asm volatile("" ::: "memory");
      const unsigned st = lds_base + (unsigned)((t % NST) * STAGE);
      f32x4 xf[2][MW][2];                    // [ks][m][half]
      u32x2 wlo[2][4], whi[2][4];            // [ks][cb]
      static_for<2>([&](auto kc) {
        constexpr int ks = decltype(kc)::value;
        static_for<4>([&](auto cc) {
          constexpr int cb = decltype(cc)::value;
          lds_read_tr_b64<ks * 8192>(wlo[ks][cb], st + b_off[cb]);
          lds_read_tr_b64<ks * 8192 + 1024>(whi[ks][cb], st + b_off[cb]);
        });
        static_for<MW>([&](auto mc) {
          constexpr int m = decltype(mc)::value;
          lds_read_f4<m * 4096>(xf[ks][m][0], st + a_off[ks][0]);
          lds_read_f4<m * 4096>(xf[ks][m][1], st + a_off[ks][1]);
        });
      });
      static_for<2>([&](auto kc) {
        constexpr int ks = decltype(kc)::value;
        // the reads of the first step are done while those of the second may be outstanding (the counter reaches 15)
        constexpr int younger = ks ? 0 : (8 + 2 * MW < 15 ? 8 + 2 * MW : 15);
        lds_wait<younger>(wlo[ks][0], whi[ks][0]);
        static_for<4>([&](auto cc) { lds_landed(wlo[ks][decltype(cc)::value], whi[ks][decltype(cc)::value]); });
        static_for<MW>([&](auto mc) { lds_landed(xf[ks][decltype(mc)::value][0], xf[ks][decltype(mc)::value][1]); });
        bf16x8 bf[4];
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) bf[cb] = __builtin_bit_cast(bf16x8, u32x4{wlo[ks][cb][0], wlo[ks][cb][1], whi[ks][cb][0], whi[ks][cb][1]});
#pragma unroll
        for (int m = 0; m < MW; ++m) {
          bf16x8 ah, al;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float v = xf[ks][m][e >> 2][e & 3];
            ah[e] = (bf16_t)v;
            al[e] = (bf16_t)(v - (float)ah[e]);
          }
#pragma unroll
          for (int cb = 0; cb < 4; ++cb) acc[m][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bf[cb], acc[m][cb], 0, 0, 0);
#pragma unroll
          for (int cb = 0; cb < 4; ++cb) acc[m][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bf[cb], acc[m][cb], 0, 0, 0);
        }
      });
    }
    // acc[m][cb][i]: row 16 (mb0 + MW row_half + m) + 4 q4 + i, column c0 + 64 col_half + 16 cb + j16
#pragma unroll
    for (int m = 0; m < MW; ++m)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int bb = 16 * (mb0 + MW * row_half + m) + 4 * q4 + i;
          if (bb < B) part[((size_t)kz * B + bb) * N + c0 + 64 * col_half + 16 * cb + j16] = acc[m][cb][i];
        }
  }
}

template <typename OT>
__global__ void __launch_bounds__(256) output_projection_reduce_kernel(const float* __restrict__ part,
                                                                       OT* __restrict__ out, size_t n,
                                                                       int ksplit) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  float v = part[i];
  for (int z = 1; z < ksplit; ++z) v += part[(size_t)z * n + i];
  store_from_f32(out + i, v);
}

// Any storage type and width: one thread per output element.
template <typename T, typename OT>
__global__ void __launch_bounds__(256) output_projection_simple_kernel(const float* __restrict__ x,
                                                                       const T* __restrict__ W,
                                                                       OT* __restrict__ out, int K, int N) {
  const int n = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
  if (n >= N) return;
  float v = 0.f;
  for (int k = 0; k < K; ++k) v = fmaf(x[(size_t)b * K + k], load_as_f32(W + (size_t)k * N + n), v);
  store_from_f32(out + (size_t)b * N + n, v);
}

// k-range split of the matrix-core path (0 = that path does not apply).
int output_projection_ksplit(const tpla_shape_t& sh, int D) {
  const long long K = (long long)sh.H * sh.d_v;
  if (sh.dtype != TPLA_BF16 || D % OP_COLS != 0 || K % OP_ROWS != 0 || K > 2147483647LL) return 0;
  const int slabs = D / OP_COLS;
  // about one workgroup per compute unit (its ring takes 96 to 144 KB of LDS): for D = 7168, K = 8192 at B = 32 that is
  // 224 workgroups of 32 chunks, 27 us for both kernels; 448 of 16 chunks on a ring of 3 took 29.5 us
  int ks = (device_cu_count() + slabs - 1) / slabs;
  const int chunks = (int)(K / OP_ROWS);
  if (ks > chunks) ks = chunks;
  if (ks < 1) ks = 1;
  while (chunks % ks) --ks;                                   // equal k-ranges, whole chunks
  return ks;
}

template <typename OT>
static int launch_output_projection_to(const tpla_shape_t& sh, const float* x, const void* W_O, int D, float* part,
                                       OT* out, hipStream_t st) {
  const int K = sh.H * sh.d_v;
  const int ks = output_projection_ksplit(sh, D);
  constexpr bool direct_ok = sizeof(OT) == sizeof(float);     // the matrix-core kernel writes float tiles
  if (ks == 0) {
    const dim3 grid((unsigned)((D + 255) / 256), (unsigned)sh.B);
    if (sh.dtype == TPLA_F32)
      hipLaunchKernelGGL((output_projection_simple_kernel<float, OT>), grid, dim3(256), 0, st, x,
                         static_cast<const float*>(W_O), out, K, D);
    else
      hipLaunchKernelGGL((output_projection_simple_kernel<bf16_t, OT>), grid, dim3(256), 0, st, x,
                         static_cast<const bf16_t*>(W_O), out, K, D);
    return check_launch("output_projection_simple_kernel");
  }
  // as few passes over the weights as the rows allow.  With one or two chunks per k-range nothing of a pass is in flight beside it, but the
  // loads of the next pass are beside its stores: passes of 64 rows where that is two or three well-filled ones and
  // every compute unit has a workgroup.  16 heads, D = 2048 (two chunks), both kernels, passes of 64 / 128 rows in us: 96 sequences 19.2 / 18.6, 112 19.4 / 20.3 (8 heads 18.4 / 18.1),
  // 128 19.3 / 21.7, 136 20.7 / 23.0, 192 22.9 / 25.1, 256 27.5 / 26.6; 32 heads (four chunks) 128 23.4 / 23.2, 256 36.0 / 32.5; D = 512 (half of
  // the compute units) 128 18.3 / 17.8.
  const bool short_ranges = K / ks <= 2 * OP_ROWS && D / OP_COLS * ks >= device_cu_count() && sh.B > 112 && sh.B <= 192;
  const int mb = sh.B <= 32 ? 2 : sh.B <= 64 || short_ranges ? 4 : 8;
  auto* const kernel = mb == 2 ? output_projection_mfma_kernel<2> : mb == 4 ? output_projection_mfma_kernel<4> : output_projection_mfma_kernel<8>;
  const size_t smem = (size_t)op_stages(mb) * op_stage(mb);
  int rc = allow_lds(reinterpret_cast<const void*>(kernel), smem, "output_projection_mfma_kernel");
  if (rc) return rc;
  const bool direct = ks == 1 && direct_ok;
  float* dst = direct ? reinterpret_cast<float*>(out) : part;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(D / OP_COLS), (unsigned)ks), dim3(OP_THREADS), smem,
                     st, x, static_cast<const bf16_t*>(W_O), dst, sh.B, K, D, K / ks);
  rc = check_launch("output_projection_mfma_kernel");
  if (rc || direct) return rc;
  const size_t n = (size_t)sh.B * D;
  hipLaunchKernelGGL(output_projection_reduce_kernel<OT>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, part,
                     out, n, ks);
  return check_launch("output_projection_reduce_kernel");
}

// Scratch floats of the matrix-core path for an output of the given type (a bf16 output always goes
// through the float partial tiles, also with a single k-range).
size_t output_projection_scratch_floats(const tpla_shape_t& sh, int D, int out_dtype) {
  const int ks = output_projection_ksplit(sh, D);
  if (ks == 0 || (ks == 1 && out_dtype == TPLA_F32)) return 0;
  return (size_t)ks * sh.B * D;
}

int launch_output_projection(const tpla_shape_t& sh, const float* x, const void* W_O, int D, float* part, void* out,
                             int out_dtype, hipStream_t st) {
  if (out_dtype == TPLA_BF16)
    return launch_output_projection_to(sh, x, W_O, D, part, static_cast<bf16_t*>(out), st);
  return launch_output_projection_to(sh, x, W_O, D, part, static_cast<float*>(out), st);
}

}  // namespace tpla
