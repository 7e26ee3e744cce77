// Weights brought into another basis on the matrix cores (Sec. 4.1: W_new = U^T W; Sec. 4.3 for U):
//   rows    (n_inner = 1)  Y[r, j] = sum_k X[r, k] V[k, j]        W_UK: rows of d_c
//   columns (n_inner > 1)  Y[j, i] = sum_k V[k, j] X[k, i]        W_UV: [d_c, d_v] per head
// with V = U, or U^T for the inverse.  X is bf16, an exact MFMA operand.  V is float and is split into three
// bf16 terms (8 significant bits each, 24 in all: exact), every product of a term is exact in float, so
// the result carries the float sums that a float FMA loop would and is rounded to bf16 once.  The
// entries of the Hadamard matrix are +-1 times a common factor: one term, scaled at the end.
//
// A few MB of weights and 2 n_vec d_c^2 x terms flop: what bounds it is latency, of the conversion of V and of
// the vectors coming in.  A workgroup (8 waves) owns 32 columns j:
// it converts its d_c x 32 slab of V once into LDS in B-operand order and walks over its share of the
// vectors.  Rows come straight from global memory (16 bytes a lane are its share of the A operand);
// columns are staged 64 k x 128 i at a time and read back through the transposing LDS read, so that i is
// the M dimension in both forms and a lane ends up with adjacent outputs.  64 heads of [128, 512] and [512, 128] with
// a dense basis: 30 and 29 us (columns 34.5 while they were staged 32 k at a time, with a barrier that also waited for the chunks on their way);
// one workgroup per vector (transform_axis_kernel) took 316 and 337.  Rows: the 16 workgroups that read the same ones take 134 MB through L2,
// without which the kernel takes 17 us; eight k-steps in flight instead of four: 2 us more.
#include "lds_tile.h"

#include <algorithm>

namespace tpla {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int TW_COLS = 32;                 // output columns per workgroup: two MFMA column tiles
constexpr int TW_WAVES = 8;
constexpr int TW_ROWS = 32 * TW_WAVES;      // rows per workgroup pass: 32 per wave, both column tiles
constexpr int TW_VEC = 128;                 // columns per workgroup pass: 32 per wave, one column tile per half of the waves
constexpr int TW_PITCH = TW_VEC * 2 + 32;   // bytes per staged row: rows of a 4-row group 8 banks apart
constexpr int TW_MAX_D = 512;               // the slab of V must fit the LDS
constexpr int TW_CHUNK = 64;                // k per staged chunk: two k-steps
constexpr int TW_STAGE = TW_CHUNK * TW_PITCH;

// V[k0 .. k0 + 7][j] of the transform, without the Hadamard matrix's common factor.  The basis is TERMS' own (launch_transform_weights_mfma)
// and direction and signs are decided once per 8 entries: a branch around every single load made each of a thread's 32 a
// round trip of its own (Hadamard basis, 64 heads of [128, 512] and [512, 128]: 25.2 and 23.7 -> 23.0 and 21.0 us, dense 30.9 and 34.2 ->
// 29.2 and 33.4).
template <int TERMS>
__device__ __forceinline__ void tw_entries(const TransformArgs& t, int k0, int j, float (&v)[8]) {
  if constexpr (TERMS > 1) {                 // dense
    const float* p = t.inverse ? t.U + (size_t)j * t.d_c + k0 : t.U + (size_t)k0 * t.d_c + j;
    const int step = t.inverse ? 1 : t.d_c;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = p[e * step];
  } else {
    float sg[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sg[e] = 1.f;
    if (t.signs) {
      const float* p = t.inverse ? t.signs + j : t.signs + k0;
      const int step = t.inverse ? 0 : 1;
#pragma unroll
      for (int e = 0; e < 8; ++e) sg[e] = p[e * step];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (__popc((k0 + e) & j) & 1) ? -sg[e] : sg[e];
  }
}

template <int TERMS, bool COLUMNS>
__global__ void __launch_bounds__(TW_WAVES * 64) transform_weights_mfma_kernel(TransformArgs t, const bf16_t* __restrict__ src,
                                                                        bf16_t* __restrict__ dst, int n_outer, int n_inner,
                                                                        float scale) {
  __shared__ int nan_of[TW_WAVES];           // COLUMNS: waves that hold a NaN
  extern __shared__ u32x4 panel[];           // [TERMS][KS][2][64] operands of 8 bf16, then the staged rows
  const int d = t.d_c, KS = d >> 5;
  char* const stage = reinterpret_cast<char*>(panel + TERMS * KS * 128);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lo = lane & 15, hi = lane >> 4;
  const int j0 = blockIdx.x * TW_COLS;

  // operand of k-step s, column tile nt: lane (column j0 + 2 lo + nt, k group hi) holds k = 32 s + 8 hi + e
#pragma unroll 2
  for (int idx = tid; idx < KS * 128; idx += TW_WAVES * 64) {
    const int ln = idx & 63, nt = (idx >> 6) & 1, s = idx >> 7;
    const int j = j0 + 2 * (ln & 15) + nt, k0 = 32 * s + 8 * (ln >> 4);
    float v[8];
    tw_entries<TERMS>(t, k0, j, v);
#pragma unroll
    for (int term = 0; term < TERMS; ++term) {
      bf16x8 b;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        b[e] = (bf16_t)v[e];
        v[e] -= (float)b[e];
      }
      panel[(term * KS + s) * 128 + nt * 64 + ln] = __builtin_bit_cast(u32x4, b);
    }
  }
  __syncthreads();
  const unsigned panel_at = lds_at(reinterpret_cast<const char*>(panel)) + 16 * lane;

  // blocks of TW_ROWS rows, or of TW_VEC columns of one outer index
  const int per_outer = COLUMNS ? (n_inner + TW_VEC - 1) / TW_VEC : 1;
  const int n_blocks = COLUMNS ? n_outer * per_outer : (n_outer + TW_ROWS - 1) / TW_ROWS;
  for (int blk = blockIdx.y; blk < n_blocks; blk += gridDim.y) {
    f32x4 acc[2][2];
    constexpr int NT = COLUMNS ? 1 : 2;                      // column tiles of this wave, from nt0 on
    const int nt0 = COLUMNS ? wave >> 2 : 0, group = COLUMNS ? wave & 3 : wave;
    auto multiply = [&](auto n_terms, int s, const bf16x8 (&av)[2]) {
#pragma unroll
      for (int term = decltype(n_terms)::value - 1; term >= 0; --term)   // small terms first
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const bf16x8 bv = __builtin_bit_cast(bf16x8, panel[(term * KS + s) * 128 + (nt0 + nt) * 64 + lane]);
#pragma unroll
          for (int mt = 0; mt < 2; ++mt) acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[mt], bv, acc[mt][nt], 0, 0, 0);
        }
    };
    const int r0 = blk * TW_ROWS + 32 * group;                          // rows
    const int o = blk / per_outer, i0 = (blk - o * per_outer) * TW_VEC;  // columns
    auto has_nan = [&]() -> bool {
      bool nan = false;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) nan |= acc[i >> 1][i & 1][e] != acc[i >> 1][i & 1][e];
      return __any(nan) != 0;
    };
    auto pass = [&](auto n_terms) {
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i >> 1][i & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (!COLUMNS) {
        const bf16_t* ap[2];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) ap[mt] = src + (size_t)min(r0 + 16 * mt + lo, n_outer - 1) * d + 8 * hi;
        constexpr int AHEAD = 4;                               // k-steps of rows in flight (KS is a multiple of 2)
        u32x4 a[AHEAD][2];
#pragma unroll
        for (int f = 0; f < AHEAD; ++f)
#pragma unroll
          for (int mt = 0; mt < 2; ++mt) a[f][mt] = *reinterpret_cast<const u32x4*>(ap[mt] + 32 * min(f, KS - 1));
        for (int s0 = 0; s0 < KS; s0 += AHEAD) {
#pragma unroll
          for (int f = 0; f < AHEAD; ++f) {
            const int s = s0 + f;
            if (s >= KS) break;
            bf16x8 av[2];
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) {
              av[mt] = __builtin_bit_cast(bf16x8, a[f][mt]);
              a[f][mt] = *reinterpret_cast<const u32x4*>(ap[mt] + 32 * min(s + AHEAD, KS - 1));
            }
            multiply(n_terms, s, av);
          }
        }
      } else {
        constexpr int NTERMS = decltype(n_terms)::value;
        const bf16_t* X = src + (size_t)o * d * n_inner;
        // staging: thread t fetches 8 columns at 8 (t % 16) of rows t / 16 and 32 + t / 16 of a chunk, two chunks ahead of the one
        // in use; columns past n_inner (a multiple of 8) repeat the last ones
        static_assert(TW_WAVES * 64 == 32 * (TW_VEC / 8), "two 16-byte pieces per thread and chunk");
        const int st_row = tid >> 4, st_col = (tid & 15) * 8;
        const bf16_t* sp = X + (size_t)st_row * n_inner + min(i0 + st_col, n_inner - 8);
        const unsigned st_at = lds_at(stage) + (unsigned)(st_row * TW_PITCH + st_col * 2);
        // lane (column 32 group + 16 mt + lo) gets k = 8 hi + 0..7
        const unsigned x_at = lds_at(stage) + (unsigned)((8 * hi + (lo >> 2)) * TW_PITCH + (32 * group + 4 * (lo & 3)) * 2);
        u32x4 v[2][2];
        auto request = [&](u32x4 (&x)[2], int s) {
#pragma unroll
          for (int e = 0; e < 2; ++e) x[e] = *reinterpret_cast<const u32x4*>(sp + (size_t)(32 * (min(s, KS - 2) + e)) * n_inner);
        };
        auto chunk = [&](u32x4 (&x)[2], int s) {
          const unsigned buf = (unsigned)((s >> 1) & 1) * TW_STAGE;
#pragma unroll
          for (int e = 0; e < 2; ++e) *reinterpret_cast<u32x4*>(stage + (st_at - lds_at(stage)) + buf + e * (32 * TW_PITCH)) = x[e];
          request(x, s + 4);
          lds_barrier();             // the chunk is in place; the other buffer was read before the previous barrier
          // of each k-step four pieces of the vectors, then a fragment per term from the smallest: all of the chunk's on their way (left to the
          // compiler each waited for its own 130 and more clocks in front of two MFMAs of 16)
          constexpr int OPS = 4 + NTERMS;
          u32x2 xv[2][2][2];
          bf16x8 bv[2][NTERMS];
          const unsigned xa = x_at + buf;
          unsigned at[NTERMS];
#pragma unroll
          for (int term = 0; term < NTERMS; ++term) at[term] = panel_at + (unsigned)((term * KS + s) * 2048 + nt0 * 1024);
          static_for<2>([&](auto ec) {
            constexpr int e = decltype(ec)::value;
            static_for<2>([&](auto mc) {
              constexpr int mt = decltype(mc)::value;
              lds_read_tr_b64<e * 32 * TW_PITCH + mt * 32>(xv[e][mt][0], xa);
              lds_read_tr_b64<e * 32 * TW_PITCH + mt * 32 + 4 * TW_PITCH>(xv[e][mt][1], xa);
            });
            static_for<NTERMS>([&](auto tc) { lds_read_b128<e * 2048>(bv[e][decltype(tc)::value], at[NTERMS - 1 - decltype(tc)::value]); });
          });
          static_for<2>([&](auto ec) {
            constexpr int e = decltype(ec)::value, after = (1 - e) * OPS;         // requested after this k-step's
            bf16x8 av[2];
            static_for<NTERMS>([&](auto tc) {
              constexpr int i = decltype(tc)::value;
              lds_wait<after + NTERMS - 1 - i>(bv[e][i]);
              if constexpr (i == 0) {
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                  lds_wait<after + NTERMS - 1>(xv[e][mt][0], xv[e][mt][1]);
                  const u32x4 x4 = {xv[e][mt][0][0], xv[e][mt][0][1], xv[e][mt][1][0], xv[e][mt][1][1]};
                  av[mt] = __builtin_bit_cast(bf16x8, x4);
                }
              }
#pragma unroll
              for (int mt = 0; mt < 2; ++mt) acc[mt][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[mt], bv[e][i], acc[mt][0], 0, 0, 0);
            });
          });
        };
        request(v[0], 0);
        request(v[1], 2);
        for (int s = 0; s < KS; s += 4) {
          chunk(v[0], s);
          if (s + 2 < KS) chunk(v[1], s + 2);
        }
        if constexpr (decltype(n_terms)::value > 1) {
          const bool nan = has_nan();
          if (lane == 0) nan_of[wave] = nan;
        }
        __syncthreads();             // the staging buffers are free for the next block
      }
    };
    pass(std::integral_constant<int, TERMS>{});
    if constexpr (TERMS > 1) {
      // An infinity times a low term that is zero is a NaN beside the first term's correct infinity: what is NaN takes the
      // sum of the first terms alone, in which the finite products no longer matter.
      bool again = has_nan();
      if constexpr (COLUMNS) {                               // the waves of a workgroup stage together
        again = false;
#pragma unroll
        for (int w = 0; w < TW_WAVES; ++w) again |= nan_of[w] != 0;
      }
      if (again) {
        f32x4 all[2][2];
#pragma unroll
        for (int i = 0; i < 4; ++i) all[i >> 1][i & 1] = acc[i >> 1][i & 1];
        pass(std::integral_constant<int, 1>{});
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float v = all[i >> 1][i & 1][e];
            if (v == v) acc[i >> 1][i & 1][e] = v;
          }
      }
    }
    if constexpr (!COLUMNS) {
      // rows r0 + 16 mt + 4 hi + e, columns j0 + 2 lo + nt
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = r0 + 16 * mt + 4 * hi + e;
          if (r < n_outer) {
            const bf16x2 v = __builtin_convertvector(f32x2{acc[mt][0][e] * scale, acc[mt][1][e] * scale}, bf16x2);
            *reinterpret_cast<bf16x2*>(dst + (size_t)r * d + j0 + 2 * lo) = v;
          }
        }
    } else {
      // columns i0 + 32 group + 16 mt + 4 hi + e, output row j0 + 2 lo + nt0
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        const int i = i0 + 32 * group + 16 * mt + 4 * hi;
        if (i < n_inner) {
          const bf16x4 y = __builtin_convertvector(acc[mt][0] * scale, bf16x4);
          *reinterpret_cast<bf16x4*>(dst + ((size_t)o * d + j0 + 2 * lo + nt0) * n_inner + i) = y;
        }
      }
    }
  }
}

bool transform_weights_mfma_supported(const TransformArgs& t, const void* src, const void* dst, int64_t n_outer,
                                      int64_t n_inner) {
  if (t.dtype != TPLA_BF16 || t.mode == TPLA_U_IDENTITY || t.d_c % 64 != 0 || t.d_c > TW_MAX_D) return false;
  if (n_inner != 1 && n_inner % 8 != 0) return false;
  // Few vectors are faster in the general kernel, whose butterflies cost d log d where this one multiplies by a matrix it has
  // to write into LDS first.  Hadamard basis, general / this kernel in us:
  //   rows of 512: 300 5.1 / 14.8, 4000 14.0 / 16.1, 8192 25.4 / 25.5, 16384 46.5 / 43.9; of 256: 2000 6.4 / 10.0, 4000
  //     10.2 / 9.9, 8192 17.4 / 10.9; of 128: 2000 4.8 / 6.8, 3000 6.7 / 6.8, 4000 7.8 / 6.8; of 64: 2000 4.4 / 5.5, 3000 6.1 / 5.5
  //   columns of 512: 128 5.7 / 9.3, 768 8.5 / 9.3, 1024 9.8 / 9.4, 2048 15.9 / 9.5; of 256: 512 5.5 / 6.0, 768 6.1 / 6.0; of 128:
  //     256 4.2 / 4.4, 512 4.6 / 4.4; of 64: 4.1 / 4.0
  // A dense basis: rows of 64 1000 4.6 / 5.1, 4000 7.7 / 5.1; everything wider and all columns here (rows of 512: 300 38 / 14).
  const int64_t n_vec = n_outer * n_inner;
  const bool hadamard = t.mode == TPLA_U_HADAMARD;
  if (n_inner == 1 ? (hadamard || t.d_c == 64) && n_vec < (t.d_c < 192 ? 3000 : 16 * t.d_c) : hadamard && n_vec < 3 * t.d_c) return false;
  // a workgroup reads whole vectors and writes 32 of their columns: not in place, not over an overlap
  const size_t bytes = (size_t)n_outer * n_inner * t.d_c * 2;
  const uintptr_t s = (uintptr_t)src, q = (uintptr_t)dst;
  return s + bytes <= q || q + bytes <= s;
}

template <int TERMS, bool COLUMNS>
static int launch_weights_t(const TransformArgs& t, const bf16_t* src, bf16_t* dst, int64_t n_outer, int64_t n_inner,
                            hipStream_t st) {
  constexpr int most = TERMS * (TW_MAX_D / 32) * 128 * 16 + (COLUMNS ? 2 * TW_STAGE : 0);
  const int rc = allow_lds(reinterpret_cast<const void*>(transform_weights_mfma_kernel<TERMS, COLUMNS>), most, "transform_weights_mfma_kernel");
  if (rc) return rc;
  const size_t smem = (size_t)TERMS * (t.d_c / 32) * 128 * 16 + (COLUMNS ? 2 * TW_STAGE : 0);
  const int64_t n_blocks = COLUMNS ? n_outer * ((n_inner + TW_VEC - 1) / TW_VEC) : (n_outer + TW_ROWS - 1) / TW_ROWS;
  const int slabs = t.d_c / TW_COLS;
  // one workgroup per compute unit: each converts its slab of V for itself.  Where two do not fit a compute unit, no more of them than there are
  // compute units: the few left over of 260 started when the others had ended.  Dense basis, columns, 64 x 128 and 64 x 512 vectors, us: d_c = 320 19.6 -> 15.3 and
  // 62.8 -> 41.1 (with chunks of 32 k, of which two workgroups fit, 18.2 and 54.5), 384 24.4 -> 19.6 and 83 -> 52, 448 31.3 -> 21.5 and 106 -> 65; 16384 rows of 448 56 -> 38.
  const int cus = device_cu_count(), round_up = 2 * smem <= 160 * 1024 ? slabs - 1 : 0;
  int64_t workers = std::max(1, (cus + round_up) / slabs);
  if (workers > n_blocks) workers = n_blocks;
  const float scale = t.mode == TPLA_U_HADAMARD ? 1.0f / sqrtf((float)t.d_c) : 1.0f;
  hipLaunchKernelGGL((transform_weights_mfma_kernel<TERMS, COLUMNS>), dim3((unsigned)slabs, (unsigned)workers), dim3(TW_WAVES * 64),
                     smem, st, t, src, dst, (int)n_outer, (int)n_inner, scale);
  return check_launch("transform_weights_mfma_kernel");
}

int launch_transform_weights_mfma(const TransformArgs& t, const void* src, void* dst, int64_t n_outer, int64_t n_inner,
                                  hipStream_t st) {
  const bf16_t* s = static_cast<const bf16_t*>(src);
  bf16_t* q = static_cast<bf16_t*>(dst);
  if (t.mode == TPLA_U_HADAMARD)
    return n_inner == 1 ? launch_weights_t<1, false>(t, s, q, n_outer, n_inner, st) : launch_weights_t<1, true>(t, s, q, n_outer, n_inner, st);
  return n_inner == 1 ? launch_weights_t<3, false>(t, s, q, n_outer, n_inner, st) : launch_weights_t<3, true>(t, s, q, n_outer, n_inner, st);
}

}  // namespace tpla
