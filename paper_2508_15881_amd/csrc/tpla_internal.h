// Internal declarations shared by the translation units of libtpla.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "tpla.h"

namespace tpla {

// Records the message returned by tpla_last_error() and hands back `code`.
int fail(int code, const char* fmt, ...);
// Checks hipGetLastError() after a launch.
int check_launch(const char* what);
// Number of compute units of the current device (cached per device).
int device_cu_count();
// Dynamic LDS above the 64 KiB default has to be asked for, once per kernel and DEVICE.  `bytes`: the most any launch of this
// kernel takes (always the same for a kernel).
int allow_lds(const void* kernel, size_t bytes, const char* what);

typedef __bf16 bf16_t;

// Split plan of the decode: the sequence axis of every sequence is cut into
// chunks of pages_per_split pages; chunk s of sequence b is non-empty when
// s * pages_per_split < ceil(seq_lens[b] / page_tokens).
// Balanced mode instead lays all pages end to end and gives each of n_wg
// workgroups an equal range (see decode_mfma_balanced_kernel).
struct SplitPlan {
  int32_t balanced;
  int32_t n_wg;              // balanced: workgroups; partial slots = n_wg + n_shards * B
  int32_t n_splits;          // static
  int32_t pages_per_split;   // static
  int32_t round_wt[4];       // balanced: weight of the ranges of each placement round
  int32_t xcc_wt[2];         // balanced: weight of the ranges of even / odd workgroups
  int32_t second_pages, all_pages;   // balanced: see BalancedPlan
  int32_t n_cus;             // balanced: compute units per row of heads
};
SplitPlan plan_splits(const tpla_shape_t& sh, int32_t n_shards, int32_t max_pages_per_seq, int32_t n_splits_req);

// Balanced plan.  The T pages of all (slice, sequence) pairs are laid end to end and cut into W
// ranges, one per workgroup; range w is [plan_start(w), plan_start(w + 1)).  Ranges are weighted by
// the placement round of their workgroup (round = w / n_cus; the hardware fills every compute unit
// once before it places a second workgroup on any) and by the parity of its position in the round
// (workgroups go to the eight XCCs in turn and n_cus is a multiple of 8 on the hardware, so this is the
// parity of the XCC): the weight of range w is wt[w / n_cus] * wx[(w % n_cus) & 1].
// All weights equal = ranges [w T / W, (w + 1) T / W).
struct BalancedPlan {
  int32_t W;        // ranges = workgroups
  int32_t n_cus;    // workgroups per placement round (compute units, over the rows of workgroups that share a range)
  int32_t wt[4];    // weight of a range of round min(r, 3); positive
  int32_t wx[2];    // weight of a range at an even / odd position of its round; positive
  int32_t second_pages, all_pages;   // pages from which a second range per compute unit, and all W ranges, are used (plan_fit)
};
// Sum of the weights of ranges 0 .. w-1.
__host__ __device__ __forceinline__ long long plan_cum(const BalancedPlan& p, int w) {
  long long c = 0;
  int r = 0, left = w;
  const long long pair = (long long)p.wx[0] + p.wx[1];
  while (r < 3 && left > p.n_cus) {
    c += ((long long)(p.n_cus / 2) * pair + (long long)(p.n_cus & 1) * p.wx[0]) * p.wt[r];
    left -= p.n_cus;
    ++r;
  }
  return c + ((long long)(left / 2) * pair + (long long)(left & 1) * p.wx[0]) * p.wt[r];
}
// First page of range w, 0 <= w <= W (T pages in all; T * total weight stays below 2^62).
// total = plan_cum(p, p.W), for callers that need several ranges.
__host__ __device__ __forceinline__ int plan_start(const BalancedPlan& p, long long T, int w, long long total) {
  return (int)(T * plan_cum(p, w) / total);
}
__host__ __device__ __forceinline__ int plan_start(const BalancedPlan& p, long long T, int w) {
  return plan_start(p, T, w, plan_cum(p, p.W));
}
__host__ __device__ __forceinline__ bool plan_equal_weights(const BalancedPlan& p) {
  return p.wt[0] == p.wt[1] && p.wt[1] == p.wt[2] && p.wt[2] == p.wt[3] && p.wx[0] == p.wx[1];
}
// Range w of n equal ranges of T pages, and the range that holds page c: 32-bit arithmetic, n T < 2^31.
__host__ __device__ __forceinline__ void equal_range(int n, int T, int w, int* start, int* end) {
  *start = w < n ? (int)((unsigned)w * (unsigned)T / (unsigned)n) : T;
  *end = w < n ? (int)(((unsigned)w + 1u) * (unsigned)T / (unsigned)n) : T;
}
__host__ __device__ __forceinline__ int equal_owner(int n, int c, int T) {
  return (int)((((unsigned)c + 1u) * (unsigned)n + (unsigned)T - 1u) / (unsigned)T - 1u);
}
// Range w as [*start, *end) = [plan_start(w), plan_start(w + 1)), 0 <= w < W: equal ranges of not too many
// pages in 32-bit arithmetic (every workgroup of the split kernel begins with this).
__host__ __device__ __forceinline__ void plan_range(const BalancedPlan& p, int T, int w, int* start, int* end) {
  if (plan_equal_weights(p) && (long long)T * p.W < 2147483647LL) {
    equal_range(p.W, T, w, start, end);
    return;
  }
  const long long total = plan_cum(p, p.W);
  *start = plan_start(p, T, w, total);
  *end = plan_start(p, T, w + 1, total);
}
// The range that holds page c, 0 <= c < T.
__host__ __device__ __forceinline__ int balanced_owner(const BalancedPlan& p, int c, int T) {
  if (plan_equal_weights(p) && (long long)T * p.W < 2147483647LL) {
    return equal_owner(p.W, c, T);   // the last w with w T / W <= c, in 32-bit arithmetic
  }
  // First guess from the inverse of the piecewise linear cumulative weight (with the mean of the two
  // parity weights) in floating point, then steps to the exact range with the test
  //   plan_start(w) <= c   <=>   T cum(w) < (c + 1) total
  // which needs no division (a 64-bit integer division costs the GPU a hundred instructions; the
  // guess only decides how many steps follow, the result is exact either way).
  const long long total = plan_cum(p, p.W);
  const double pair = (double)p.wx[0] + (double)p.wx[1];
  double x = (double)c * (double)total / (double)T;
  int r = 0, base = 0;
  while (r < 3 && base + p.n_cus < p.W) {
    const double round_weight = (double)(plan_cum(p, base + p.n_cus) - plan_cum(p, base));
    if (x < round_weight) break;
    x -= round_weight;
    base += p.n_cus;
    ++r;
  }
  int w = base + (int)(2.0 * x / ((double)p.wt[r] * pair));
  if (w > p.W - 1) w = p.W - 1;
  if (w < 0) w = 0;
  const long long bound = ((long long)c + 1) * total;
  while (w + 1 < p.W && (long long)T * plan_cum(p, w + 1) < bound) ++w;
  while (w > 0 && !((long long)T * plan_cum(p, w) < bound)) --w;
  return w;
}
// The plan as a launch uses it once the lengths are known: T pages in all.  The host sizes W (and the
// partial-result slots) for block-table rows that are full; how long the sequences are is only known on
// the device, and a serving engine's rows are usually far from full.
//   * Long ranges (32 pages or more each): the plan as it is, weights included.
//   * Shorter ones: equal ranges, one per compute unit, two from second_pages pages on, all W from all_pages on.  A
//     range costs its queries and a partial result of H d_c/g floats, written here and read by the merge, so the
//     wider that is the more pages a further workgroup on a compute unit wants (decode_mfma_range_pages).  Numbers
//     in between leave some compute units with two ranges and others with one of the same length.  (Where a compute unit holds
//     one workgroup, as for all 256-wide slices: one range each.)
//   * Fewer pages than that: one page per range.  No range between two non-empty ones is then ever
//     empty, and the partial results of a sequence are consecutive slots: the merge no longer tests range
//     by range with 64-bit divisions which of them exist (one sequence of 1237 tokens in a table for 4096,
//     64 heads: merge-and-combine 63 us with the tests).
// Returns the number of equal ranges to use instead, or 0 for the plan as it is.  (A number and not a
// plan of its own: a plan chosen at run time has its weights indexed in scratch memory, which cost every
// launch of the split kernel 0.6 us and more.)
__host__ __device__ __forceinline__ int plan_fit(const BalancedPlan& p, int T) {
  if (T / 32 >= p.W) return 0;
  int w = T >= p.all_pages ? p.W : T >= p.second_pages ? 2 * p.n_cus : p.n_cus;
  if (w > p.W) w = p.W;
  return w < T ? w : (T > 0 ? T : 1);
}
// Range that workgroup w takes of n equal ranges (plan_fit) of T pages.  Workgroups are dealt to the eight XCCs in turn: in that order the ranges of a
// sequence lie on all of them, and every L2 fetches the queries of every sequence (40 KB each at 64 heads over 256-wide slices, a fifth of what
// an 8-page range reads).  Side by side on one XCC they are fetched once.  What that costs is how the launch ends: in turn some XCCs often hold the
// shorter ranges and write their partial results back while the others still work; side by side all XCCs end together.  So it is done for eight
// (slice, sequence) pairs or more, where there are two slices (twice the queries), where ranges are long (longer where two rows of workgroups share one)
// or where partial results are small.  Split and merge behind absorb, caches not resident, in turn / side by side, us:
//   two slices, 64 heads: 16 x 4096 tokens 36.1 / 34.7, 16 x 1000 26.9 / 25.1, 48 x 3000 61.0 / 56.7; four, 128 heads: 128 of 100 to 6000 160 / 149
//   one slice, 64 heads, 256-wide: 32 of 5003 to 16384 55.1 / 52.0 (19 pages a range); 32 x 700 23.7 / 25.0, 4 x 8000 23.5 / 24.2, 20 of 600 to 9000 28.6 / 29.2 (in
//     turn); 512-wide, 32 heads: 32 x 700 28.8 / 29.8, 16 heads, 8 x 1000 19.7 / 21.2 (in turn)
//   one slice, 16 heads, 256-wide (16 KB a range): 16 x 2000 16.5 / 15.7; 64 heads, 128-wide: 16 x 4096 23.2 / 22.1
// 740 pairs of measurements over 16 to 128 heads, 1 to 4 slices of every width and 27 batches: by this rule 1.3 % faster where it acts, 7 of 465 slower by more
// than 2.5 %; side by side everywhere 48 of 740.  Groups of 2, 4 or 8 ranges per XCC in turn: no better.
__host__ __device__ __forceinline__ int range_of_workgroup(int n, int T, int w, int n_shards, int B, int H, int dl) {
  const bool side_by_side = n_shards * B >= 8 && (n_shards > 1 || T >= (H > 64 ? 9 : 6) * n || (dl <= 256 && H * dl <= 8192));
  return side_by_side && (n & 7) == 0 && w < n ? (w & 7) * (n >> 3) + (w >> 3) : w;
}
// The work item of a workgroup that owns the pages [start, end) in a sequence whose n pages begin at
// page e of the laid-out order: its pages [*p0, *p1) counted inside the sequence.  False when the two
// ranges share no page (also for an empty workgroup range that lies inside the sequence).
__host__ __device__ __forceinline__ bool balanced_item(int start, int end, int e, int n, int* p0, int* p1) {
  const int lo = start > e ? start : e, hi = end < e + n ? end : e + n;
  *p0 = lo - e;
  *p1 = hi - e;
  return lo < hi;
}

// Partial results of one (slice, sequence, split): acc [n_shards, B, S, H, dl]
// floats, then ml [n_shards, B, S, H, 2] floats (running max in log2 units, sum of weights).
// Several latent slices can share one launch: slice i uses q_lat[i], pools[i],
// the common q_pe / page table / lengths, and row i of every output.
// Bytes of the plan table (see DecodeArgs::plan) of n_v (slice, sequence) pairs.  Two ints per pair are written; the size is the
// one that callers' workspaces have always been asked for (three per pair and two more).
inline size_t plan_table_bytes(size_t n_v) { return ((3 * n_v + 2) * sizeof(int32_t) + 15) / 16 * 16; }

struct DecodeArgs {
  const void* q_lat;     // [n_shards, B, H, dl]
  const void* q_pe;      // [B, H, d_r]
  const void* pools[TPLA_MAX_G];   // each [P, page_tokens, dl + d_r]
  const int32_t* block_table;
  const int32_t* seq_lens;
  float* part_acc;
  float* part_ml;
  float* o_lat;          // [n_shards, B, H, dl]
  float* lse;            // [n_shards, B, H] or nullptr
  int32_t n_shards;
  int32_t B, H, dl, d_r, page_tokens, max_pages;
  int32_t n_splits, pages_per_split;
  int32_t balanced, n_wg;
  BalancedPlan geom;     // balanced: ranges and their weights (geom.W == n_wg)
  // balanced, written by the split kernel for the merge, n_v = n_shards * B entries each: [0, n_v) the range
  // that owns the first page of a (slice, sequence); [n_v, 2 n_v) how many ranges from there to the owner
  // of its last page (0 for an empty sequence).  Every one of them holds pages of it (plan_fit).
  int32_t* plan;         // plan_table_bytes()
  float scale_log2;      // sm_scale * log2(e)
};

// True when the MFMA kernel covers this shape (bf16 only).
bool decode_mfma_supported(const tpla_shape_t& sh);
// Workgroups of the matrix-core kernel for this shape that fit on one compute
// unit (0 = unknown).
int decode_mfma_blocks_per_cu(const tpla_shape_t& sh);
// Rows of workgroups per range: heads beyond what one workgroup takes.
int decode_mfma_head_rows(const tpla_shape_t& sh);
// Range weights by placement round (wt) and by even / odd position in the round (wx) for a launch that
// puts per_cu workgroups of the matrix-core kernel on every compute unit.
void decode_mfma_round_weights(const tpla_shape_t& sh, int per_cu, int32_t wt[4], int32_t wx[2]);
// Pages from which a launch uses two workgroups per compute unit, and as many as fit, and not one.
void decode_mfma_range_pages(const tpla_shape_t& sh, int32_t* second, int32_t* all);
// ev_start / ev_stop (both or neither): events that receive the kernel's begin and end times.
int launch_decode_mfma(const DecodeArgs& a, hipStream_t st, hipEvent_t ev_start = nullptr,
                       hipEvent_t ev_stop = nullptr);
// Length of sequence b as every decode kernel uses it: clipped to what its block-table row can
// address, so a length that disagrees with max_pages_per_seq gives wrong numbers, never a read
// past the table.
__device__ __forceinline__ int clip_length(const DecodeArgs& a, int length) {
  const long long cap = (long long)a.max_pages * a.page_tokens;
  const long long L = length;
  return (int)(L < 0 ? 0 : (L > cap ? cap : L));
}
__device__ __forceinline__ int seq_len_clipped(const DecodeArgs& a, int b) { return clip_length(a, a.seq_lens[b]); }

int launch_decode_generic(const DecodeArgs& a, int dtype, hipStream_t st);
// Short contexts of narrow float rows, all slices of a (sequence, head) per workgroup; W_UV_t given: with the combine, where it is supported.  (plan: what
// the general kernel would take.)
bool decode_rows_supported(const tpla_shape_t& sh, int n_shards, int max_pages, const SplitPlan& plan);
bool decode_rows_combine_supported(const tpla_shape_t& sh);
int launch_decode_rows(const DecodeArgs& a, const float* W_UV_t, void* o, int o_dtype, int d_v, hipStream_t st);
int launch_decode_merge(const DecodeArgs& a, hipStream_t st);

struct TransformArgs {
  int32_t d_c, dtype, mode, inverse;
  const float* signs;
  const float* U;
};
int launch_transform_axis(const TransformArgs& t, const void* src, void* dst, int64_t n_outer,
                          int64_t n_inner, hipStream_t st);
// Matrix-core weights transform (bf16, d_c a multiple of 64 up to 512, not in place): see transform_weights.hip.
bool transform_weights_mfma_supported(const TransformArgs& t, const void* src, const void* dst, int64_t n_outer,
                                      int64_t n_inner);
int launch_transform_weights_mfma(const TransformArgs& t, const void* src, void* dst, int64_t n_outer, int64_t n_inner,
                                  hipStream_t st);
struct ShardPools {
  void* p[TPLA_MAX_G];
};
int launch_transform_paged(const TransformArgs& t, const tpla_shape_t& sh, const void* mla_pool,
                           const ShardPools& pools, const int32_t* page_ids, int64_t n_pages,
                           hipStream_t st);
// Matrix-core Hadamard pass (bf16, d_c 256 / 512): see transform_mfma.hip.
bool transform_paged_mfma_supported(const TransformArgs& t, const tpla_shape_t& sh, int64_t n_pages);
int launch_transform_paged_mfma(const TransformArgs& t, const tpla_shape_t& sh, const void* mla_pool,
                                const ShardPools& pools, const int32_t* page_ids, int64_t n_pages,
                                hipStream_t st);
bool transform_paged_dense_mfma_supported(const TransformArgs& t, const tpla_shape_t& sh, int64_t n_pages);
int launch_transform_paged_dense_mfma(const TransformArgs& t, const tpla_shape_t& sh, const void* mla_pool,
                                      const ShardPools& pools, const int32_t* page_ids, int64_t n_pages,
                                      hipStream_t st);
int launch_write_mla_cache(const tpla_shape_t& sh, const void* c_raw, const void* k_pe,
                           const int32_t* slot_mapping, int64_t T, float rms_eps, void* mla_pool,
                           hipStream_t st);

int launch_append_token_sliced(const tpla_shape_t& sh, const void* c_t, const void* k_pe,
                               const struct MuFactors& alpha, float rms_eps, const int32_t* slots,
                               const ShardPools& pools, hipStream_t st);

// Output projection (after the combine): out = x @ W_O.
int output_projection_ksplit(const tpla_shape_t& sh, int D);
size_t output_projection_scratch_floats(const tpla_shape_t& sh, int D, int out_dtype);
int launch_output_projection(const tpla_shape_t& sh, const float* x, const void* W_O, int D, float* part,
                             void* out, int out_dtype, hipStream_t st);

// Prefill (un-absorbed MLA, causal, packed sequences): see prefill_mfma.hip.
bool prefill_mfma_supported(const tpla_shape_t& sh);
int launch_prefill_attention(const tpla_shape_t& sh, const void* q_nope, const void* q_pe, const void* c,
                             const void* k_pe, const void* W_UK, const void* W_UV, const int32_t* cu_seqlens,
                             int T, int max_seq_len, void* kv_workspace, float* o, hipStream_t st);

int launch_stream_read(const void* buf, size_t bytes, void* sink, hipStream_t st);

// PCA calibration: see pca.hip.
int latent_moments_splits(const tpla_shape_t& sh, int64_t n_pages);
size_t latent_moments_workspace(const tpla_shape_t& sh, int64_t n_pages);
int launch_latent_moments(const tpla_shape_t& sh, const void* mla_pool, const int32_t* page_ids,
                          const int32_t* page_fill, int64_t n_pages, float* workspace, double* sum, double* gram,
                          hipStream_t st);
int pca_basis_host(int d, int g, double n_rows, const double* sum, const double* gram, float* U, double* eig,
                   double* frac);

struct MuFactors {
  float v[TPLA_MAX_G];
};
int launch_absorb_query(const tpla_shape_t& sh, const void* q_nope, const void* W_UK_t,
                        const MuFactors& mu, void* q_lat, hipStream_t st);
int launch_combine_shards(const tpla_shape_t& sh, const float* o_lat, const void* W_UV_t, void* o, int o_dtype,
                          hipStream_t st);
// Matrix-core variants (bf16 weights, widths that tile): see absorb_combine_mfma.hip.
bool absorb_mfma_supported(const tpla_shape_t& sh);
int launch_absorb_query_mfma(const tpla_shape_t& sh, const void* q_nope, const void* W_UK_t,
                             const MuFactors& mu, void* q_lat, hipStream_t st);
bool combine_mfma_supported(const tpla_shape_t& sh);
int launch_combine_shards_mfma(const tpla_shape_t& sh, const float* o_lat, const void* W_UV_t, void* o, int o_dtype,
                               hipStream_t st);
// LDS of the merge-and-combine kernel, for the kernel, its launcher and the host checks.
constexpr int MC_COLS = 128;                  // output columns per workgroup
constexpr int MC_MERGE_WAVES = 8;
constexpr int MC_JOIN_BYTES = MC_MERGE_WAVES * (1024 + 16);   // a piece, its reference and sum per wave
// bf16 terms that carry a float of o_lat into the product.  Two (16 bits) for the widths that always had a matrix-core
// kernel; three (24 bits, exact) for the others, which plain float FMAs used to serve.
__host__ __device__ constexpr int mc_terms(int d_c, int d_v) { return d_c % 512 == 0 && d_v % 64 == 0 ? 2 : 3; }
// Latent columns per chunk.  Without a merge half as many, so that two workgroups share a compute unit and one's weights
// arrive under the other's product; with a merge and three terms 512 and 16 sequences would not fit.
__host__ __device__ constexpr int mc_rows(bool merge, int terms) { return merge && terms == 2 ? 512 : 256; }
// Whether the slots of a unit may be dealt over several waves: the launches that reserve the join buffers.  (With two terms a unit's columns are.)
__host__ __device__ constexpr bool mc_joins(bool merge, int terms, int spw) { return merge && terms == 3 && spw < MC_MERGE_WAVES; }
struct McLds {
  int operands, join, bytes;                  // offsets of the A operands (weights before them) and of the join buffers; size
};
__host__ __device__ constexpr McLds mc_lds(bool merge, int terms, int spw, int d_c) {
  const int rows = d_c < mc_rows(merge, terms) ? d_c : mc_rows(merge, terms);
  const int operands = rows * MC_COLS * 2, join = operands + terms * spw * rows * 2;
  return McLds{operands, join, join + (mc_joins(merge, terms, spw) ? MC_JOIN_BYTES : 0)};
}
// Waves per unit of work of a workgroup with n_units of them.  spw and not the units decides first: the last group of
// a batch can be left with few units in a launch that has no join buffers.
__host__ __device__ constexpr int mc_waves_per_unit(bool merge, int terms, int spw, int n_units) {
  return mc_joins(merge, terms, spw) && n_units < MC_MERGE_WAVES ? MC_MERGE_WAVES / n_units : 1;
}
// Split merge fused with the combine: reads the decode's partial results, writes o_lat, lse and o.
bool merge_combine_mfma_supported(const tpla_shape_t& sh);
bool merge_combine_in_one_round(const tpla_shape_t& sh);
// Whether the fused kernel is the faster one: in one round, and for some shapes in two.
bool merge_combine_pays(const tpla_shape_t& sh);
int launch_merge_combine_mfma(const DecodeArgs& a, const tpla_shape_t& sh, const void* W_UV_t, void* o, int o_dtype,
                              hipStream_t st);

// ---- small device helpers -------------------------------------------------
// Value of lane (l ^ M) without going through LDS: DPP for M < 16, the
// row / half swaps of gfx950 above that.
template <int M>
__device__ __forceinline__ float lane_xor(float v, int lane) {
  const int x = __float_as_int(v);
  if constexpr (M == 1) return __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
  if constexpr (M == 2) return __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
  if constexpr (M == 4) {
    // rotations by 4 and 12 inside a row of 16: one of them is lane l + 4, the other l - 4
    const int a = __builtin_amdgcn_update_dpp(x, x, 0x124, 0xF, 0xF, false);   // row_ror:4  -> lane (l - 4) & 15
    const int b = __builtin_amdgcn_update_dpp(x, x, 0x12C, 0xF, 0xF, false);   // row_ror:12 -> lane (l + 4) & 15
    return __int_as_float((lane & 4) ? a : b);
  }
  if constexpr (M == 8) return __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0x128, 0xF, 0xF, false));  // row_ror:8
  if constexpr (M == 16) {
    // swaps rows 1,3 of the first operand with rows 0,2 of the second
    const auto r = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false);
    return __int_as_float((int)((lane & 16) ? r[0] : r[1]));
  }
  if constexpr (M == 32) {
    // swaps the upper half of the first operand with the lower half of the second
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
    return __int_as_float((int)((lane & 32) ? r[0] : r[1]));
  }
  return v;
}

__device__ __forceinline__ float bf16_to_f32(bf16_t x) { return (float)x; }
__device__ __forceinline__ float load_as_f32(const float* p) { return *p; }
__device__ __forceinline__ float load_as_f32(const bf16_t* p) { return (float)*p; }
__device__ __forceinline__ void store_from_f32(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_from_f32(bf16_t* p, float v) { *p = (bf16_t)v; }

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// 8 consecutive elements of a row, as floats.
struct Vec8 {
  float v[8];
};
__device__ __forceinline__ Vec8 load8(const bf16_t* p) {
  const u32x4 raw = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  Vec8 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    r.v[2 * i] = __uint_as_float(raw[i] << 16);
    r.v[2 * i + 1] = __uint_as_float(raw[i] & 0xffff0000u);
  }
  return r;
}
__device__ __forceinline__ Vec8 load8(const float* p) {
  const u32x4 a = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  const u32x4 b = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p) + 1);
  Vec8 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    r.v[i] = __uint_as_float(a[i]);
    r.v[4 + i] = __uint_as_float(b[i]);
  }
  return r;
}
__device__ __forceinline__ unsigned short f32_to_bf16_bits(float f) {
  return __builtin_bit_cast(unsigned short, (bf16_t)f);
}
__device__ __forceinline__ void store8(bf16_t* p, const Vec8& r) {
  u32x4 raw;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    raw[i] = (unsigned)f32_to_bf16_bits(r.v[2 * i]) | ((unsigned)f32_to_bf16_bits(r.v[2 * i + 1]) << 16);
  __builtin_nontemporal_store(raw, reinterpret_cast<u32x4*>(p));
}
__device__ __forceinline__ void store8(float* p, const Vec8& r) {
  u32x4 a, b;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a[i] = __float_as_uint(r.v[i]);
    b[i] = __float_as_uint(r.v[4 + i]);
  }
  __builtin_nontemporal_store(a, reinterpret_cast<u32x4*>(p));
  __builtin_nontemporal_store(b, reinterpret_cast<u32x4*>(p) + 1);
}

// Plain (cached) variant of load8 for operands that are re-read.
__device__ __forceinline__ Vec8 load8_cached(const bf16_t* p) {
  const u32x4 raw = *reinterpret_cast<const u32x4*>(p);
  Vec8 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    r.v[2 * i] = __uint_as_float(raw[i] << 16);
    r.v[2 * i + 1] = __uint_as_float(raw[i] & 0xffff0000u);
  }
  return r;
}
__device__ __forceinline__ Vec8 load8_cached(const float* p) {
  const u32x4 a = *reinterpret_cast<const u32x4*>(p);
  const u32x4 b = *(reinterpret_cast<const u32x4*>(p) + 1);
  Vec8 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    r.v[i] = __uint_as_float(a[i]);
    r.v[4 + i] = __uint_as_float(b[i]);
  }
  return r;
}

}  // namespace tpla
