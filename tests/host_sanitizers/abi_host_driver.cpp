// Host-side exerciser of libtpla's C ABI for a build with AddressSanitizer and
// UndefinedBehaviorSanitizer on the host code (no GPU work: a call fails
// validation, runs on the host, or has its launches recorded by
// recorded_launches.h).  It walks the argument checks of every entry point with
// fake, aligned device addresses, the page-table validator on in-range and
// out-of-range tables, the host eigen-solver of the PCA basis on matrices whose
// decomposition is known, the page-range plan, and what the launchers ask for.  Exit status 0 = every
// expectation held and no sanitizer report was raised (reports abort).
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <vector>

#include "tpla.h"
#include "tpla_internal.h"   // the plan arithmetic shared by the split kernel and the merge kernels
#include "split_merge.h"
#include "recorded_launches.h"

static int g_failures = 0;
#define EXPECT(cond)                                                        \
  do {                                                                      \
    if (!(cond)) {                                                          \
      fprintf(stderr, "%s:%d: expectation failed: %s (last error: %s)\n", __FILE__, __LINE__, #cond, \
              tpla_last_error());                                           \
      ++g_failures;                                                         \
    }                                                                       \
  } while (0)

static tpla_shape_t shape(int B = 2, int H = 64, int d_c = 512, int g = 2) {
  tpla_shape_t s;
  s.B = B; s.H = H; s.d_c = d_c; s.g = g; s.d_r = 64; s.d_n = 128; s.d_v = 128;
  s.page_tokens = 64; s.dtype = TPLA_BF16; s.sm_scale = 0.07f;
  return s;
}

// x_{n+1} = x_n * 6364136223846793005 + 1442695040888963407, top bits -> (-1, 1)
static double lcg(uint64_t& st) {
  st = st * 6364136223846793005ULL + 1442695040888963407ULL;
  return (double)(st >> 11) / 4503599627370496.0 - 1.0;
}

static void* const A = (void*)(uintptr_t)4096;        // aligned, never dereferenced
static void* const A2 = (void*)(uintptr_t)(4096 + 2); // misaligned

static void argument_checks() {
  tpla_shape_t s = shape();
  float* Af = (float*)A;
  const int32_t* Ai = (const int32_t*)A;
  // decode: one slice, all slices, with the combine, without a workspace
  EXPECT(tpla_decode_shard(&s, NULL, A, A, Ai, 4, Ai, 0, A, (size_t)1 << 30, Af, NULL, NULL) == TPLA_ERR_NULL);
  EXPECT(tpla_decode_shard(&s, A, A, A, Ai, 0, Ai, 0, A, (size_t)1 << 30, Af, NULL, NULL) == TPLA_ERR_SHAPE);
  EXPECT(tpla_decode_shard(&s, A2, A, A, Ai, 4, Ai, 0, A, (size_t)1 << 30, Af, NULL, NULL) == TPLA_ERR_ALIGN);
  EXPECT(tpla_decode_shard(&s, A, A, A, Ai, 4, Ai, 2, A, 16, Af, NULL, NULL) == TPLA_ERR_WORKSPACE);
  EXPECT(tpla_decode_shard(NULL, A, A, A, Ai, 4, Ai, 2, A, 16, Af, NULL, NULL) == TPLA_ERR_NULL);
  tpla_shape_t bad = shape(); bad.dtype = 7;
  EXPECT(tpla_decode_shard(&bad, A, A, A, Ai, 4, Ai, 0, A, (size_t)1 << 30, Af, NULL, NULL) == TPLA_ERR_DTYPE);
  bad = shape(2, 64, 512, 3);
  EXPECT(tpla_decode_shard(&bad, A, A, A, Ai, 4, Ai, 0, A, (size_t)1 << 30, Af, NULL, NULL) == TPLA_ERR_SHAPE);
  bad = shape(2, 64, 1024, 16);
  EXPECT(tpla_decode_shard(&bad, A, A, A, Ai, 4, Ai, 0, A, (size_t)1 << 30, Af, NULL, NULL) == TPLA_ERR_SHAPE);
  bad = shape(); bad.sm_scale = NAN;
  EXPECT(tpla_decode_shard(&bad, A, A, A, Ai, 4, Ai, 0, A, (size_t)1 << 30, Af, NULL, NULL) == TPLA_ERR_SHAPE);
  const void* pools[TPLA_MAX_G] = {A, A};
  const void* pools_hole[TPLA_MAX_G] = {A, NULL};
  EXPECT(tpla_decode_shards(&s, A, A, pools_hole, Ai, 4, Ai, 0, A, (size_t)1 << 30, Af, NULL, NULL) == TPLA_ERR_NULL);
  EXPECT(tpla_decode_shards(&s, A, A, pools, Ai, 4, Ai, 3, A, 16, Af, NULL, NULL) == TPLA_ERR_WORKSPACE);
  EXPECT(tpla_decode_shards(&s, A, A, pools, Ai, 2147483647, Ai, 3, A, 16, Af, NULL, NULL) == TPLA_ERR_SHAPE);
  EXPECT(tpla_decode_shards_combine(&s, A, A, pools, Ai, 4, Ai, 0, A, (size_t)1 << 30, NULL, Af, Af, NULL, NULL) == TPLA_ERR_NULL);
  EXPECT(tpla_decode_shards_combine(&s, A, A, pools, Ai, 4, Ai, 0, A, (size_t)1 << 30, A2, Af, Af, NULL, NULL) == TPLA_ERR_ALIGN);
  EXPECT(tpla_decode_shards_combine(&s, A, A, pools, Ai, 4, Ai, 2, A, 16, A, Af, Af, NULL, NULL) == TPLA_ERR_WORKSPACE);
  tpla_shape_t big = shape(32);
  EXPECT(tpla_decode_shards_combine_static(&big, A, A, pools, Ai, 2048, Ai, 1024, A, Af, Af, NULL, NULL) == TPLA_ERR_WORKSPACE);
  EXPECT(tpla_decode_shards_combine_static(&s, A, A, pools, Ai, 0, Ai, 0, A, Af, Af, NULL, NULL) == TPLA_ERR_SHAPE);
  EXPECT(tpla_decode_shards_combine_static(&s, A, A, pools, Ai, 4, Ai, 0, NULL, Af, Af, NULL, NULL) == TPLA_ERR_NULL);
  // workspace sizes: plain arithmetic on the plan
  EXPECT(tpla_workspace_bytes(&s, 512, 1) == (size_t)2 * 64 * (256 + 2) * 4);
  EXPECT(tpla_workspace_bytes(&s, 512, 8) == (size_t)8 * 2 * 64 * (256 + 2) * 4);
  EXPECT(tpla_workspace_bytes(&s, 4, 100) == (size_t)4 * 2 * 64 * (256 + 2) * 4);
  EXPECT(tpla_workspace_bytes(&s, 512, 0) > 0 && tpla_workspace_bytes_all(&s, 512, 0) >= tpla_workspace_bytes(&s, 512, 0));
  EXPECT(tpla_workspace_bytes(&s, 0, 0) == 0 && tpla_workspace_bytes_all(&s, 4, -1) == 0);
  // absorb, combine, transforms, cache writes
  const float mu_bad[TPLA_MAX_G] = {1.0f, INFINITY};
  EXPECT(tpla_absorb_query(&s, NULL, A, NULL, A, NULL) == TPLA_ERR_NULL);
  EXPECT(tpla_absorb_query(&s, A, A2, NULL, A, NULL) == TPLA_ERR_ALIGN);
  EXPECT(tpla_absorb_query(&s, A, A, mu_bad, A, NULL) == TPLA_ERR_SHAPE);
  EXPECT(tpla_combine_shards(&s, Af, NULL, Af, NULL) == TPLA_ERR_NULL);
  EXPECT(tpla_transform_latent(&s, 9, 0, NULL, NULL, A, A, 4, 1, NULL) == TPLA_ERR_SHAPE);
  bad = shape(2, 64, 96, 2);
  EXPECT(tpla_transform_latent(&bad, TPLA_U_HADAMARD, 0, NULL, NULL, A, A, 4, 1, NULL) == TPLA_ERR_SHAPE);
  EXPECT(tpla_transform_latent(&s, TPLA_U_DENSE, 0, NULL, NULL, A, A, 4, 1, NULL) == TPLA_ERR_NULL);
  EXPECT(tpla_transform_latent(&s, TPLA_U_IDENTITY, 0, NULL, NULL, A, A, 0, 1, NULL) == TPLA_OK);
  void* wpools[TPLA_MAX_G] = {A, A};
  void* wpools_mis[TPLA_MAX_G] = {A, A2};
  EXPECT(tpla_transform_latent_paged(&s, TPLA_U_IDENTITY, NULL, NULL, A, wpools_mis, NULL, 3, NULL) == TPLA_ERR_ALIGN);
  EXPECT(tpla_transform_latent_paged(&s, TPLA_U_IDENTITY, NULL, NULL, A, wpools, NULL, -1, NULL) == TPLA_ERR_SHAPE);
  EXPECT(tpla_transform_latent_paged(&s, TPLA_U_IDENTITY, NULL, NULL, A, wpools, NULL, 0, NULL) == TPLA_OK);
  EXPECT(tpla_write_mla_cache(&s, A, A, NULL, 5, 1e-6f, A, NULL) == TPLA_ERR_NULL);
  EXPECT(tpla_write_mla_cache(&s, A, A, Ai, -5, 1e-6f, A, NULL) == TPLA_ERR_SHAPE);
  EXPECT(tpla_write_mla_cache(&s, A, A, Ai, 0, 1e-6f, A, NULL) == TPLA_OK);
  const float alpha_bad[TPLA_MAX_G] = {2.0f, -1.0f};
  EXPECT(tpla_append_token_sliced(&s, A, A, alpha_bad, 1e-6f, Ai, wpools, NULL) == TPLA_ERR_SHAPE);
  EXPECT(tpla_append_token_sliced(&s, A, A, NULL, -1.0f, Ai, wpools, NULL) == TPLA_ERR_SHAPE);
  EXPECT(tpla_append_token_sliced(&s, A, A, NULL, 1e-6f, Ai, wpools_mis, NULL) == TPLA_ERR_ALIGN);
  // output projection, PCA moments, prefill
  EXPECT(tpla_output_projection(&s, Af, NULL, 64, A, (size_t)1 << 20, Af, NULL) == TPLA_ERR_NULL);
  EXPECT(tpla_output_projection(&s, Af, A, 0, A, (size_t)1 << 20, Af, NULL) == TPLA_ERR_SHAPE);
  EXPECT(tpla_latent_moments_workspace_bytes(&s, 0) == 0 && tpla_latent_moments_workspace_bytes(&s, 40) > 0);
  EXPECT(tpla_latent_moments(&s, A, NULL, NULL, 4, A, 16, (double*)A, (double*)A, NULL) == TPLA_ERR_WORKSPACE);
  EXPECT(tpla_latent_moments(&s, A, NULL, NULL, 0, A, (size_t)1 << 30, (double*)A, (double*)A, NULL) == TPLA_ERR_SHAPE);
  EXPECT(tpla_prefill_workspace_bytes(&s, 100) == (size_t)100 * 64 * 256 * 2);
  EXPECT(tpla_prefill_attention(&s, A, A, A, A, A, A, NULL, 8, 8, A, (size_t)1 << 30, Af, NULL) == TPLA_ERR_NULL);
  EXPECT(tpla_prefill_attention(&s, A, A, A, A, A, A, Ai, 8, 8, A, 64, Af, NULL) == TPLA_ERR_WORKSPACE);
  bad = shape(); bad.d_n = 64;
  EXPECT(tpla_prefill_attention(&bad, A, A, A, A, A, A, Ai, 8, 8, A, (size_t)1 << 30, Af, NULL) == TPLA_ERR_UNSUPPORTED);
  // measurement aids
  float ms[4]; int32_t n = -1;
  EXPECT(tpla_profile_enable(-1) == TPLA_ERR_SHAPE);
  EXPECT(tpla_profile_collect(ms, -3, &n) == TPLA_ERR_SHAPE);
  EXPECT(tpla_profile_collect(ms, 4, &n) == TPLA_OK && n == 0);
  EXPECT(tpla_stream_read(NULL, 100, A, NULL) == TPLA_ERR_NULL);
  EXPECT(strlen(tpla_last_error()) > 0 && tpla_version() >= 100);
}

static void block_table_checks() {
  tpla_shape_t s = shape(3);
  // exactly-sized heap arrays: a read past a row or past the lengths is a sanitizer report
  std::vector<int32_t> bt = {0, 1, 2, 3, 4, 5, 0, 0, 6, 0, 0, 0};
  std::vector<int32_t> ln = {200, 65, 1};
  EXPECT(tpla_validate_block_table(&s, bt.data(), 4, ln.data(), 7, 0) == TPLA_OK);
  EXPECT(tpla_validate_block_table(&s, bt.data(), 4, ln.data(), 7, 1) == TPLA_OK);
  EXPECT(tpla_validate_block_table(&s, bt.data(), 4, ln.data(), 6, 0) == TPLA_ERR_SHAPE);
  EXPECT(strstr(tpla_last_error(), "block_table[2][0]=6") != NULL);
  std::vector<int32_t> full = {256, 256, 256};             // every row used to its last entry
  EXPECT(tpla_validate_block_table(&s, bt.data(), 4, full.data(), 7, 0) == TPLA_OK);
  EXPECT(tpla_validate_block_table(&s, bt.data(), 4, full.data(), 7, 1) == TPLA_ERR_SHAPE);   // page 0 repeats
  std::vector<int32_t> over = {257, 65, 1};
  EXPECT(tpla_validate_block_table(&s, bt.data(), 4, over.data(), 7, 0) == TPLA_ERR_SHAPE);
  std::vector<int32_t> neg = {200, -1, 1};
  EXPECT(tpla_validate_block_table(&s, bt.data(), 4, neg.data(), 7, 0) == TPLA_ERR_SHAPE);
  std::vector<int32_t> huge_id = bt; huge_id[0] = 2147483647;
  EXPECT(tpla_validate_block_table(&s, huge_id.data(), 4, ln.data(), 7, 1) == TPLA_ERR_SHAPE);
  std::vector<int32_t> neg_id = bt; neg_id[5] = -2147483647 - 1;
  EXPECT(tpla_validate_block_table(&s, neg_id.data(), 4, ln.data(), 7, 1) == TPLA_ERR_SHAPE);
  EXPECT(tpla_validate_block_table(&s, NULL, 4, ln.data(), 7, 0) == TPLA_ERR_NULL);
  EXPECT(tpla_validate_block_table(&s, bt.data(), 4, ln.data(), 0, 0) == TPLA_ERR_SHAPE);
}


// The decomposition of C: U orthonormal, U^T C U = diag(eig) descending, fractions sum to 1.
static void check_basis(int d, int g, const std::vector<double>& C, double n_rows_scale, const char* what) {
  std::vector<double> sum((size_t)d, 0.0), gram((size_t)d * d), eig((size_t)d), frac((size_t)g);
  std::vector<float> U((size_t)d * d);
  for (size_t i = 0; i < gram.size(); ++i) gram[i] = C[i] * n_rows_scale;
  const int rc = tpla_pca_basis(d, g, (int64_t)n_rows_scale, sum.data(), gram.data(), U.data(), eig.data(), frac.data());
  EXPECT(rc == TPLA_OK);
  if (rc != TPLA_OK) return;
  double worst_orth = 0.0, worst_diag = 0.0, cmax = 0.0, fs = 0.0;
  for (double c : C) cmax = fmax(cmax, fabs(c));
  for (int i = 0; i + 1 < d; ++i) EXPECT(eig[i] >= eig[i + 1]);
  std::vector<double> CU((size_t)d * d, 0.0);
  for (int i = 0; i < d; ++i)
    for (int k = 0; k < d; ++k) {
      const double c = C[(size_t)i * d + k];
      for (int j = 0; j < d; ++j) CU[(size_t)i * d + j] += c * U[(size_t)k * d + j];
    }
  for (int a = 0; a < d; ++a)
    for (int b = 0; b < d; ++b) {
      double dot = 0.0, q = 0.0;
      for (int i = 0; i < d; ++i) {
        dot += (double)U[(size_t)i * d + a] * U[(size_t)i * d + b];
        q += (double)U[(size_t)i * d + a] * CU[(size_t)i * d + b];
      }
      worst_orth = fmax(worst_orth, fabs(dot - (a == b ? 1.0 : 0.0)));
      worst_diag = fmax(worst_diag, fabs(q - (a == b ? eig[a] : 0.0)));
    }
  for (double f : frac) fs += f;
  if (!(worst_orth <= 1e-5 && worst_diag <= 1e-5 * cmax && fabs(fs - 1.0) <= 1e-12)) {
    fprintf(stderr, "%s: orthogonality %.3g, off-diagonal %.3g (scale %.3g), fractions %.17g\n", what, worst_orth,
            worst_diag, cmax, fs);
    ++g_failures;
  }
}

static void pca_checks() {
  uint64_t st = 12345;
  for (int d : {1, 2, 7, 64, 160}) {
    // C = X^T X / m from a random m x d matrix with column scales 1 .. 1/d
    const int m = 3 * d + 1;
    std::vector<double> X((size_t)m * d), C((size_t)d * d, 0.0);
    for (int r = 0; r < m; ++r)
      for (int j = 0; j < d; ++j) X[(size_t)r * d + j] = lcg(st) / (1.0 + j);
    for (int r = 0; r < m; ++r)
      for (int i = 0; i < d; ++i)
        for (int j = 0; j < d; ++j) C[(size_t)i * d + j] += X[(size_t)r * d + i] * X[(size_t)r * d + j] / m;
    check_basis(d, (d % 2 == 0) ? 2 : 1, C, 1000.0, "random covariance");
  }
  {  // repeated eigenvalues and an exactly diagonal input
    const int d = 12;
    std::vector<double> C((size_t)d * d, 0.0);
    for (int i = 0; i < d; ++i) C[(size_t)i * d + i] = (i % 3 == 0) ? 5.0 : 2.0;
    check_basis(d, 4, C, 10.0, "diagonal with repeated values");
    std::vector<double> Z((size_t)d * d, 0.0);
    check_basis(d, 3, Z, 10.0, "zero matrix");
  }
  std::vector<double> z(16, 0.0);
  std::vector<float> zf(16, 0.f);
  EXPECT(tpla_pca_basis(4, 3, 10, z.data(), z.data(), zf.data(), z.data(), z.data()) == TPLA_ERR_SHAPE);
  EXPECT(tpla_pca_basis(4, 2, 0, z.data(), z.data(), zf.data(), z.data(), z.data()) == TPLA_ERR_SHAPE);
  EXPECT(tpla_pca_basis(4, 2, 10, NULL, z.data(), zf.data(), z.data(), z.data()) == TPLA_ERR_NULL);
}

// Balanced plan: range w of W is [plan_start(w), plan_start(w + 1)) of the T pages of all sequences laid
// end to end, with equal or round-weighted shares.  The split kernel derives its work items with
// balanced_item, and leaves the merge kernels the owners of a sequence's first and last page (balanced_owner): for
// every (T, W, weights, lengths) both must name the same (workgroup, sequence) pairs, every page exactly once.  These are
// the plan's own ranges; what short launches make of them is fitted_plan_checks().
static void plan_checks() {
  uint64_t st = 99;
  const int Ws[] = {1, 2, 3, 7, 16, 40, 256, 512, 768};
  const int wts[][4] = {{1, 1, 1, 1}, {135, 121, 128, 128}, {149, 131, 106, 128}, {128, 128, 128, 128}, {3, 1, 1, 7}};
  const int cus[] = {256, 8, 5};
  const int wxs[][2] = {{1, 1}, {128, 118}, {100, 131}};
  for (const auto& wx : wxs)
  for (const auto& wt : wts)
    for (int n_cus : cus)
      for (int W : Ws)
        for (int trial = 0; trial < 12; ++trial) {
          tpla::BalancedPlan p;
          p.W = W;
          p.n_cus = n_cus;
          for (int r = 0; r < 4; ++r) p.wt[r] = wt[r];
          p.wx[0] = wx[0];
          p.wx[1] = wx[1];
          const int n_seq = 1 + (int)((lcg(st) + 1.0) * 6.0);
          std::vector<int> pages((size_t)n_seq), excl((size_t)n_seq);
          int T = 0;
          for (int v = 0; v < n_seq; ++v) {
            // short batches (T < W: empty ranges), empty sequences, and long ones
            const double u = lcg(st);
            pages[v] = u < -0.6 ? 0 : (trial % 3 == 0 ? (int)((u + 1.0) * 3.0) : (int)((u + 1.0) * 0.8 * W));
            excl[v] = T;
            T += pages[v];
          }
          if (T == 0) continue;
          EXPECT(tpla::plan_start(p, T, 0) == 0 && tpla::plan_start(p, T, W) == T);
          for (int w = 0; w < W; ++w) {
            EXPECT(tpla::plan_start(p, T, w) <= tpla::plan_start(p, T, w + 1));
            EXPECT(tpla::plan_start(p, T, w) == (int)((long long)T * tpla::plan_cum(p, w) / tpla::plan_cum(p, W)));
            int r0 = -1, r1 = -1;
            tpla::plan_range(p, T, w, &r0, &r1);                         // what a workgroup computes for itself
            EXPECT(r0 == tpla::plan_start(p, T, w) && r1 == tpla::plan_start(p, T, w + 1));
          }
          if (wt[0] == wt[1] && wt[1] == wt[2] && wt[2] == wt[3] && wx[0] == wx[1])      // equal weights: the plain equal shares
            for (int w = 0; w <= W; ++w) EXPECT(tpla::plan_start(p, T, w) == (int)((long long)w * T / W));
          for (int c = 0; c < T; ++c) {
            const int w = tpla::balanced_owner(p, c, T);
            EXPECT(w >= 0 && w < W && tpla::plan_start(p, T, w) <= c && c < tpla::plan_start(p, T, w + 1));
          }
          std::vector<int> covered((size_t)T, 0);
          for (int v = 0; v < n_seq; ++v) {
            int n_items = 0, w_first = -1, w_last = -1;
            for (int w = 0; w < W; ++w) {
              const int start = tpla::plan_start(p, T, w), end = tpla::plan_start(p, T, w + 1);
              int p0 = -1, p1 = -1;
              const bool item = pages[v] > 0 && tpla::balanced_item(start, end, excl[v], pages[v], &p0, &p1);
              if (!item) continue;
              EXPECT(0 <= p0 && p0 < p1 && p1 <= pages[v]);
              for (int q = p0; q < p1; ++q) ++covered[(size_t)(excl[v] + q)];
              if (w_first < 0) w_first = w;
              w_last = w;
              ++n_items;
            }
            if (pages[v] > 0) {
              // what the merge computes: first and last owner of the sequence's pages
              EXPECT(w_first == tpla::balanced_owner(p, excl[v], T));
              EXPECT(w_last == tpla::balanced_owner(p, excl[v] + pages[v] - 1, T));
              EXPECT(n_items >= 1 && n_items <= w_last - w_first + 1);   // (a range in between may be empty: fewer pages than ranges)
            } else {
              EXPECT(n_items == 0);
            }
          }
          for (int c = 0; c < T; ++c) EXPECT(covered[(size_t)c] == 1);
        }
  // the weighted plans of the library's own launches, used from 32 pages per range on, leave no range empty (the merge
  // relies on it)
  const int full[][8] = {{512, 256, 135, 121, 128, 128, 128, 128}, {768, 256, 140, 129, 115, 128, 128, 128},
                         {768, 256, 149, 131, 106, 128, 128, 113}, {512, 256, 128, 128, 128, 128, 128, 123},
                         {512, 256, 128, 128, 128, 128, 128, 115}, {256, 256, 128, 128, 128, 128, 128, 123}};
  for (const auto& f : full) {
    tpla::BalancedPlan p;
    p.W = f[0];
    p.n_cus = f[1];
    for (int r = 0; r < 4; ++r) p.wt[r] = f[2 + r];
    p.wx[0] = f[6];
    p.wx[1] = f[7];
    for (int T : {32 * f[0], 32 * f[0] + 17, 100000, 2000000})
      for (int w = 0; w < p.W; ++w) EXPECT(tpla::plan_start(p, T, w) < tpla::plan_start(p, T, w + 1));
    // owners at the edges of every range for page counts on both sides of the 32-bit path's limit
    // (T W < 2^31) and far beyond it
    for (int T : {4194303, 4194304, 4194305, 2796202, 2796203, 123456789, 2000000000})
      for (int w = 0; w < p.W; ++w) {
        const int lo = tpla::plan_start(p, T, w), hi = tpla::plan_start(p, T, w + 1);
        EXPECT(lo < hi);
        EXPECT(lo == (int)((long long)T * tpla::plan_cum(p, w) / tpla::plan_cum(p, p.W)));
        EXPECT(tpla::balanced_owner(p, lo, T) == w && tpla::balanced_owner(p, hi - 1, T) == w);
        EXPECT(tpla::balanced_owner(p, lo + (hi - lo) / 2, T) == w);
      }
  }
  // the same with equal weights (the 32-bit path and its fallback)
  for (int W : {1, 3, 256, 512, 768}) {
    tpla::BalancedPlan p;
    p.W = W;
    p.n_cus = 256;
    for (int r = 0; r < 4; ++r) p.wt[r] = 128;
    p.wx[0] = p.wx[1] = 128;
    for (long long T64 : {2147483647LL / W - 1, 2147483647LL / W, 2147483647LL / W + 1, 2147483647LL / W + 2, 2000000000LL}) {
      if (T64 > 2147483647LL) continue;
      const int T = (int)T64;
      for (int w = 0; w < W; ++w) {
        const int lo = tpla::plan_start(p, T, w), hi = tpla::plan_start(p, T, w + 1);
        EXPECT(lo == (int)((long long)w * T / W) && lo < hi);
        int r0 = -1, r1 = -1;
        tpla::plan_range(p, T, w, &r0, &r1);
        EXPECT(r0 == lo && r1 == hi);
        EXPECT(tpla::balanced_owner(p, lo, T) == w && tpla::balanced_owner(p, hi - 1, T) == w);
      }
    }
  }
}

// The plan as a launch uses it (plan_fit, then equal_range / equal_owner or the plan's own ranges), as the split kernel computes
// it, for page totals around every line of the rule: each page in one range, no empty range between the owners of a
// sequence's first and last page -- the merge walks the slots from one to the other --, and all slots different and
// inside the workspace.
static void fitted_plan_checks() {
  uint64_t st = 7;
  const int plans[][5] = {// W, compute units, round weights 149 : 131 : 106 or equal, second_pages, all_pages (per compute unit)
                          {1, 8, 0, 18, 18}, {5, 8, 0, 1, 1}, {8, 8, 0, 18, 18}, {16, 8, 0, 18, 18}, {24, 8, 0, 5, 13}, {24, 8, 1, 5, 13}, {16, 8, 0, 1, 1},
                          {256, 256, 0, 18, 18}, {512, 256, 0, 18, 18}, {768, 256, 1, 5, 13}, {300, 256, 0, 5, 13}};
  for (const auto& q : plans) {
    tpla::BalancedPlan p;
    p.W = q[0];
    p.n_cus = q[1];
    const int wt[4] = {149, 131, 106, 128};
    for (int r = 0; r < 4; ++r) p.wt[r] = q[2] ? wt[r] : 128;
    p.wx[0] = 128;
    p.wx[1] = q[2] ? 113 : 128;
    p.second_pages = q[3] * p.n_cus;
    p.all_pages = q[4] * p.n_cus;
    std::vector<int> totals;
    for (int c : {0, p.n_cus, 2 * p.n_cus, p.W, p.second_pages, p.all_pages, 32 * p.W, 40 * p.W})
      for (int d : {-1, 0, 1}) totals.push_back(c + d);
    for (int t = 2; t < 3 * p.n_cus && t < 60; ++t) totals.push_back(t);
    for (int T : totals)
      for (int trial = 0; T >= 0 && trial < 3; ++trial) {
        const int n_v = 1 + (int)((lcg(st) + 1.0) * 10.0);
        std::vector<int> pages((size_t)n_v), excl((size_t)n_v);
        int left = T;
        for (int v = 0; v < n_v; ++v) {
          pages[v] = v == n_v - 1 ? left : trial == 0 ? left / (n_v - v) : (int)((lcg(st) + 1.0) * 0.5 * (left + 0.999));
          if (trial == 2 && v != n_v - 1 && lcg(st) < 0.0) pages[v] = 0;
          excl[v] = T - left;
          left -= pages[v];
        }
        const int n = tpla::plan_fit(p, T);
        EXPECT(n >= 0 && n <= p.W && (T > 0 ? n <= T : n == 1) && (n == 0) == (T / 32 >= p.W));
        std::vector<int> start((size_t)p.W), end((size_t)p.W), covered((size_t)T, 0);
        for (int w = 0; w < p.W; ++w) {
          if (n > 0)
            tpla::equal_range(n, T, w, &start[w], &end[w]);
          else
            tpla::plan_range(p, T, w, &start[w], &end[w]);
          EXPECT(0 <= start[w] && start[w] <= end[w] && end[w] <= T);
          if (n == 0 || w < n) EXPECT(T == 0 || start[w] < end[w]);
          for (int c = start[w]; c < end[w]; ++c) ++covered[(size_t)c];
        }
        for (int c = 0; c < T; ++c) EXPECT(covered[(size_t)c] == 1);
        std::vector<int> used((size_t)(p.W + n_v), 0);
        for (int v = 0; v < n_v; ++v) {
          if (pages[v] == 0) continue;
          const int last = excl[v] + pages[v] - 1;
          const int w0 = n > 0 ? tpla::equal_owner(n, excl[v], T) : tpla::balanced_owner(p, excl[v], T);
          const int w1 = n > 0 ? tpla::equal_owner(n, last, T) : tpla::balanced_owner(p, last, T);
          EXPECT(0 <= w0 && w0 <= w1 && w1 < p.W);
          if (!(0 <= w0 && w0 <= w1 && w1 < p.W)) return;
          for (int w = 0; w < p.W; ++w) {
            int p0, p1;
            EXPECT(tpla::balanced_item(start[w], end[w], excl[v], pages[v], &p0, &p1) == (w >= w0 && w <= w1));
          }
          for (int w = w0; w <= w1; ++w) EXPECT(++used[(size_t)(w + v)] == 1);
        }
      }
  }
}

// LDS of the merge-and-combine launches, over the batches that leave the last workgroups any number of sequences: what a
// workgroup uses (mc_lds and, where slots are joined, mc_waves_per_unit: the kernels call the same; the operands of the kernels of whole
// chunks begin where mc_lds has them, term by term) against what the launch reserves.
static void merge_combine_launch_checks() {
  g_device = 0;
  g_record_ints = {5};                                                // spw
  for (bool merge : {true, false})
    for (int d_c : {128, 192, 256, 320, 512, 576, 768, 1024})
      for (int g : {1, 2, 4})
        for (int H : {4, 16, 32, 64, 128})
          for (int d_v : {64, 128, 200, 256})
            for (int B = 1; B <= 300; ++B) {
              tpla_shape_t s = shape(B, H, d_c, g);
              s.d_v = d_v;
              if (!tpla::merge_combine_mfma_supported(s)) continue;
              tpla::DecodeArgs a = {};
              a.B = B;
              a.H = H;
              a.dl = d_c / g;
              g_launches.clear();
              const int rc = merge ? tpla::launch_merge_combine_mfma(a, s, A, A, TPLA_F32, NULL)
                                   : tpla::launch_combine_shards_mfma(s, (const float*)A, A, A, TPLA_F32, NULL);
              EXPECT(rc == TPLA_OK && g_launches.size() == 1);
              if (g_launches.size() != 1) return;
              const RecordedLaunch& l = g_launches[0];
              const int spw = l.ints[0], sw = tpla::merge_piece_width(a.dl, H);
              const int terms = tpla::mc_terms(d_c, d_v), rows = tpla::mc_rows(merge, terms);
              const tpla::McLds lds = tpla::mc_lds(merge, terms, spw, d_c);
              EXPECT(spw >= 1 && spw <= 16 && (int)l.grid.y * spw >= B && ((int)l.grid.y - 1) * spw < B);
              EXPECT(l.lds <= 160 * 1024 && (int)l.lds <= l.lds_allowed);
              // what the dispatch takes for one round of workgroups is one
              if (merge && tpla::merge_combine_in_one_round(s)) {
                EXPECT(l.grid.x * l.grid.y * l.grid.z <= 256);
                if (l.grid.x * l.grid.y * l.grid.z > 256) {
                  fprintf(stderr, "B=%d H=%d d_c=%d g=%d d_v=%d: %d workgroups for one round of 256\n", B, H, d_c, g, d_v, (int)(l.grid.x * l.grid.y * l.grid.z));
                  return;
                }
              }
              for (int mb = 0; mb < (int)l.grid.y; ++mb)
                for (int kc = 0; kc < d_c; kc += rows) {
                  const int n_seq = spw < B - spw * mb ? spw : B - spw * mb;
                  const int cols = d_c - kc < rows ? d_c - kc : rows;
                  const int n_units = n_seq * (cols / sw), per_unit = tpla::mc_waves_per_unit(merge, terms, spw, n_units);
                  EXPECT(cols * tpla::MC_COLS * 2 <= lds.operands && lds.operands + terms * spw * cols * 2 <= lds.join);
                  EXPECT(n_units >= 1 && n_units <= 128 && per_unit >= 1);
                  EXPECT(per_unit == 1 || n_units * per_unit <= tpla::MC_MERGE_WAVES);
                  const int used = per_unit > 1 ? lds.join + tpla::MC_JOIN_BYTES : lds.join;
                  EXPECT(used <= (int)l.lds);
                  if (used > (int)l.lds) {
                    fprintf(stderr, "B=%d H=%d d_c=%d g=%d d_v=%d merge=%d: group %d of %d uses %d bytes of LDS, %zu reserved\n", B, H, d_c, g,
                            d_v, merge, mb, (int)l.grid.y, used, l.lds);
                    return;
                  }
                }
            }
}

// The pairs that the merge of four heads per wave reads for the last (slice, sequence) lie inside the array, for head counts
// that leave the last wave fewer than four.
static void merge_pair_index_checks() {
  for (int H = 1; H <= 9; ++H)
    for (int n_splits = 2; n_splits <= 5; ++n_splits) {
      const int n_v = 3, first = (n_v - 1) * n_splits;
      for (int h = 0; h < H; h += 4)
        for (int lane = 0; lane < 64; ++lane) {
          const int cnt = h + (lane >> 4) < H ? n_splits : 0, s = (lane & 15) < cnt ? lane & 15 : (cnt > 0 ? cnt - 1 : 0);
          const int head = tpla::merge_short_head(lane, h, 1, 4, H);
          EXPECT(head >= 0 && head < H && (cnt == 0 || head == h + (lane >> 4)));
          EXPECT((first + s) * H + head < n_v * n_splits * H);
        }
    }
}

// Every launch of a kernel with more than 64 KiB of dynamic LDS has been allowed that much on the device it goes to, also on
// a device that is used after another.
static void lds_opt_in_checks() {
  const void* pools[TPLA_MAX_G] = {A, A, A, A, A, A, A, A};
  float* Af = (float*)A;
  const int32_t* Ai = (const int32_t*)A;
  const size_t big = (size_t)1 << 40;
  g_record_ints.clear();
  g_launches.clear();
  for (int dev : {0, 1, 63, 200}) {
    g_device = dev;
    for (int d_c : {256, 512, 1024})
      for (int g : {1, 2})
        for (int H : {16, 32, 64, 128, 5})
          for (int d_v : {72, 128}) {
            tpla_shape_t s = shape(9, H, d_c, g);
            s.d_v = d_v;
            for (int n_splits : {0, 3}) {
              EXPECT(tpla_decode_shards_project(&s, A, A, pools, Ai, 40, Ai, n_splits, A, big, A, A, 256, A, TPLA_BF16, Af, Af, Af, NULL) == TPLA_OK);
              EXPECT(tpla_decode_shards_combine_to(&s, A, A, pools, Ai, 40, Ai, n_splits, A, big, A, A, TPLA_BF16, Af, Af, NULL) == TPLA_OK);
            }
            EXPECT(tpla_combine_shards(&s, Af, A, Af, NULL) == TPLA_OK);
            EXPECT(tpla_combine_shards_to(&s, Af, A, A, TPLA_BF16, NULL) == TPLA_OK);
          }
    tpla_shape_t s = shape();
    for (int mode : {TPLA_U_HADAMARD, TPLA_U_DENSE})
      for (int n_inner : {1, 128})
        EXPECT(tpla_transform_latent(&s, mode, 0, NULL, Af, A, (void*)((uintptr_t)1 << 40), 64, n_inner, NULL) == TPLA_OK);
  }
  size_t wide = 0;
  for (const RecordedLaunch& l : g_launches) {
    wide += l.lds > 64 * 1024 && l.device == 63;
    EXPECT((int)l.lds <= l.lds_allowed);
    if ((int)l.lds > l.lds_allowed) {
      fprintf(stderr, "a launch with %zu bytes of LDS on device %d, %d allowed\n", l.lds, l.device, l.lds_allowed);
      return;
    }
  }
  EXPECT(wide > 100);
  g_device = 0;
}

// Which grid a launch takes, by the rules whose two sides were measured.
static const RecordedLaunch& last_launch() { return g_launches.back(); }
static void dispatch_checks() {
  g_device = 0;
  g_record_ints.clear();
  float* Af = (float*)A;
  // prefill: tiles end to end (one row of workgroups) only where those are fewer than tiles of the longest x sequences
  const int batches[][4] = {{64, 3200, 50, 0}, {64, 3300, 150, 1}, {12, 12 * 129, 129, 0}, {2, 600, 300, 0}, {11, 10088, 3001, 1}, {65, 6500, 200, 0}, {1, 5000, 5000, 0}};
  for (const auto& b : batches) {
    tpla_shape_t s = shape(b[0]);
    EXPECT(tpla_prefill_attention(&s, A, A, A, A, A, A, (const int32_t*)A, b[1], b[2], A, (size_t)1 << 40, Af, NULL) == TPLA_OK);
    const RecordedLaunch& l = last_launch();
    const int tiles = (b[2] + 127) / 128;
    EXPECT((int)l.grid.y == (b[3] ? 1 : b[0]) && (int)(l.grid.x * l.grid.y) <= tiles * s.H * b[0]);
  }
  // stand-alone merge: four heads per wave (4 waves a workgroup: ceil(quads / 4) in x) or a workgroup per row, by waves per
  // compute unit against slots per pair
  const int merges[][6] = {{64, 256, 40, 2, 2, 1}, {64, 512, 4, 47, 4, 0}, {128, 128, 24, 11, 11, 0}, {128, 128, 40, 11, 11, 1}, {128, 128, 24, 256, 40, 0},
                           {128, 128, 64, 256, 40, 0}, {64, 256, 40, 2, 0, 1}, {64, 256, 16, 512, 0, 0}};
  for (const auto& m : merges) {
    tpla_shape_t s = shape(m[2], m[0], m[1], 1);
    EXPECT(tpla_decode_shard(&s, A, A, A, (const int32_t*)A, m[3], (const int32_t*)A, m[4], A, (size_t)1 << 40, Af, Af, NULL) == TPLA_OK);
    const int quads = m[2] * m[0] / 4;
    EXPECT((int)last_launch().grid.x == (m[5] ? (quads + 3) / 4 : m[2] * m[0]));
  }
  // cache write: 2^k lanes per token for latents of fewer than 64 pieces, two tokens per wave from there on
  const int writes[][3] = {{8, 1000, 4}, {64, 1000, 32}, {72, 1000, 63}, {256, 1000, 125}, {504, 1000, 250}, {512, 1000, 125}, {1536, 1000, 125}};
  for (const auto& w : writes) {
    tpla_shape_t s = shape(1, 64, w[0], 1);
    EXPECT(tpla_write_mla_cache(&s, A, A, (const int32_t*)A, w[1], 1e-6f, A, NULL) == TPLA_OK);
    EXPECT((int)last_launch().grid.x == w[2]);
  }
  // weights into another basis: a workgroup of 256 per vector for few vectors of a Hadamard basis, the matrix-core kernel
  // (512 threads) from its break-even on and for dense bases
  const int counts[][5] = {{512, 8191, 1, 0, 256}, {512, 8192, 1, 0, 512}, {512, 300, 1, 1, 512}, {64, 2999, 1, 0, 256}, {64, 2999, 1, 1, 256},
                           {64, 3000, 1, 1, 512}, {128, 3000, 1, 0, 512}, {256, 4095, 1, 0, 256}, {512, 11, 136, 0, 256}, {512, 12, 136, 0, 512},
                           {64, 1, 184, 0, 256}, {64, 1, 192, 0, 512}, {512, 1, 8, 1, 512}};
  for (const auto& c : counts) {
    tpla_shape_t s = shape(1, 64, c[0], 1);
    EXPECT(tpla_transform_latent(&s, c[3] ? TPLA_U_DENSE : TPLA_U_HADAMARD, 0, NULL, Af, A, (void*)((uintptr_t)1 << 40), c[1], c[2], NULL) == TPLA_OK);
    EXPECT((int)last_launch().block.x == c[4]);
  }
}

// Narrow float rows: the kernel of all slices of a (sequence, head) per workgroup (1024 threads) where a wave's blocks of 16 tokens take no longer
// than the general kernel's chunks (256 threads), with both sides measured; either side of the line for slice widths, numbers of slices and
// heads and page sizes; the same with and without the combine (the same bits).
static void decode_rows_dispatch_checks() {
  g_device = 0;
  g_record_ints.clear();
  const void* pools[TPLA_MAX_G] = {A, A, A, A, A, A, A, A};
  float* Af = (float*)A;
  const int32_t* Ai = (const int32_t*)A;
  // heads, sequences, d_c/g, slices, d_r, page tokens, table tokens, with the combine, expected
  const int cases[][9] = {{4, 1, 32, 2, 16, 64, 128, 1, 1},   {1, 1, 32, 2, 16, 64, 4096, 1, 0},  {1, 1, 32, 2, 16, 64, 4096, 0, 0}, {4, 1, 32, 2, 16, 64, 2048, 0, 1},
                          {1, 1, 64, 2, 16, 64, 4096, 1, 0},  {64, 1, 64, 2, 16, 64, 2048, 1, 1}, {1, 1, 16, 4, 16, 64, 4096, 1, 0}, {16, 16, 16, 4, 16, 64, 4096, 1, 1},
                          {16, 4, 16, 4, 16, 64, 4096, 1, 0}, {1, 1, 64, 8, 16, 64, 2048, 1, 0},  {1, 1, 64, 8, 16, 64, 2048, 0, 0}, {16, 16, 64, 8, 16, 64, 2048, 0, 1},
                          {1, 1, 64, 1, 16, 64, 4096, 0, 1},  {1, 1, 64, 1, 16, 32, 4096, 0, 0},  {1, 1, 64, 1, 16, 16, 2048, 0, 0}, {1, 1, 64, 1, 16, 16, 1024, 0, 1},
                          {1, 1, 32, 2, 16, 128, 4096, 0, 1}, {1, 1, 64, 2, 16, 256, 4096, 0, 1}, {1, 1, 32, 4, 32, 64, 4096, 0, 0}, {8, 1, 16, 2, 64, 64, 2048, 0, 1}};
  for (const auto& c : cases) {
    tpla_shape_t s = shape(c[1], c[0], c[2] * c[3], c[3]);
    s.dtype = TPLA_F32;
    s.d_r = c[4];
    s.d_v = 32;
    s.page_tokens = c[5];
    const int pages = c[6] / c[5];
    g_launches.clear();
    const int rc = c[7] ? tpla_decode_shards_combine(&s, A, A, pools, Ai, pages, Ai, 0, A, (size_t)1 << 40, A, Af, Af, Af, NULL)
                        : tpla_decode_shards(&s, A, A, pools, Ai, pages, Ai, 0, A, (size_t)1 << 40, Af, Af, NULL);
    EXPECT(rc == TPLA_OK && !g_launches.empty());
    const bool rows = !g_launches.empty() && g_launches[0].block.x == 1024;
    EXPECT(rows == (c[8] != 0) && (!rows || g_launches.size() == 1));
    if (rows != (c[8] != 0)) fprintf(stderr, "H=%d B=%d d_c/g=%d g=%d d_r=%d pages of %d, %d tokens, combine %d\n", c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7]);
  }
}

// Weights transform: where two workgroups do not fit the 160 KB of a compute unit, there are no more than compute units, and they cover all slabs.
static void weights_grid_checks() {
  g_device = 0;
  g_record_ints.clear();
  int full = 0;
  for (int d = 64; d <= 512; d += 64)
    for (int inner : {1, 128, 512})
      for (int outer : {64, 512, 16384}) {
        tpla_shape_t s = shape(1, 64, d, 1);
        g_launches.clear();
        EXPECT(tpla_transform_latent(&s, TPLA_U_DENSE, 0, NULL, (const float*)A, A, (void*)((uintptr_t)1 << 40), outer, inner, NULL) == TPLA_OK);
        const RecordedLaunch& l = last_launch();
        if (l.block.x != 512) continue;
        EXPECT((int)l.grid.x == d / 32 && l.grid.y >= 1);
        EXPECT(2 * l.lds <= 160 * 1024 || l.grid.x * l.grid.y <= 256);
        full += 2 * l.lds > 160 * 1024 && l.grid.x * l.grid.y > 240;
      }
  EXPECT(full > 10);
}

// Which range a workgroup takes: every range by one workgroup, workgroups beyond the ranges their own number, and ranges side by side on an XCC
// only where both sides were measured.
static void range_order_checks() {
  for (int n = 0; n <= 1024; ++n)
    for (int per : {1, 5, 6, 31})
      for (int g : {1, 2}) {
        std::vector<int> taken((size_t)n, 0);
        for (int w = 0; w < 1024; ++w) {
          const int r = tpla::range_of_workgroup(n, n * per, w, g, 8, 64, 256);
          EXPECT(w < n ? r >= 0 && r < n : r == w);
          if (w < n && r >= 0 && r < n) ++taken[(size_t)r];
        }
        for (int c : taken) EXPECT(c == 1);
      }
  // slices, sequences, heads, d_c/g, pages per range of 256, expected
  const int cases[][6] = {{1, 32, 64, 256, 1, 0}, {1, 32, 64, 256, 5, 0}, {1, 32, 64, 256, 6, 1},  {2, 16, 64, 256, 1, 1},  {2, 3, 64, 256, 1, 0},  {1, 8, 16, 512, 1, 0},  {1, 4, 32, 512, 9, 0},
                          {1, 8, 16, 256, 1, 1},  {1, 16, 32, 256, 2, 1}, {1, 16, 64, 128, 2, 1}, {1, 32, 128, 128, 8, 0}, {1, 32, 128, 256, 9, 1}, {4, 128, 128, 128, 2, 1}, {1, 32, 16, 512, 8, 1}};
  for (const auto& c : cases) EXPECT((tpla::range_of_workgroup(256, 256 * c[4], 1, c[0], c[1], c[2], c[3]) == 32) == (c[5] != 0));
}

// Merge and combine in one kernel (split and this one) or separate (split, merge, combine): in one round of workgroups, and in two where both
// sides were measured; never in more.
static void merge_combine_dispatch_checks() {
  g_device = 0;
  g_record_ints.clear();
  const void* pools[TPLA_MAX_G] = {A, A, A, A, A, A, A, A};
  float* Af = (float*)A;
  const int32_t* Ai = (const int32_t*)A;
  auto launches = [&](int H, int g, int B) {
    tpla_shape_t s = shape(B, H, 512, g);
    g_launches.clear();
    EXPECT(tpla_decode_shards_combine(&s, A, A, pools, Ai, 40, Ai, 0, A, (size_t)1 << 40, A, Af, Af, Af, NULL) == TPLA_OK);
    const RecordedLaunch& l = last_launch();
    EXPECT(g_launches.size() == 3 || (g_launches.size() == 2 && l.grid.x * l.grid.y * l.grid.z <= 2 * 256));
    return (int)g_launches.size();
  };
  const int cases[][4] = {{64, 2, 64, 2},  {64, 2, 65, 2},  {64, 2, 112, 2}, {64, 2, 113, 3}, {64, 1, 128, 3}, {128, 1, 32, 2}, {128, 1, 48, 2}, {128, 1, 49, 3},
                          {128, 2, 64, 3}, {32, 1, 128, 2}, {32, 1, 240, 2}, {32, 1, 256, 3}, {64, 4, 64, 2},  {64, 4, 65, 3},  {16, 2, 256, 2}};
  for (const auto& c : cases) {
    const int n = launches(c[0], c[1], c[2]);
    EXPECT(n == c[3]);
    if (n != c[3]) fprintf(stderr, "H=%d g=%d B=%d: %d launches\n", c[0], c[1], c[2], n);
  }
  for (int H : {16, 32, 64, 128})
    for (int B = 1; B <= 600; ++B) launches(H, 2, B);
}

// Which kernel absorbs: by its grid, the matrix cores (128 columns), few rows (64 columns of one sequence) up to a workgroup per compute unit, and the
// general one (256 columns of 8 sequences).
static void absorb_dispatch_checks() {
  g_device = 0;
  g_record_ints.clear();
  // float, heads, sequences, d_n, d_c, columns, sequences per workgroup (0: not looked at)
  const int cases[][7] = {{0, 64, 1, 128, 512, 128, 0}, {0, 2, 270, 32, 128, 128, 0}, {0, 1, 1, 256, 128, 128, 0}, {0, 1, 1, 40, 128, 64, 1}, {0, 1, 1, 128, 72, 64, 1}, {1, 4, 1, 32, 64, 64, 1},
                          {1, 64, 4, 256, 64, 64, 1},   {1, 64, 5, 32, 64, 256, 8},   {1, 32, 1, 128, 520, 256, 8}, {1, 4, 1, 264, 64, 256, 8}, {0, 21, 5, 40, 192, 256, 8}};
  for (const auto& c : cases) {
    tpla_shape_t s = shape(c[2], c[1], c[4], 1);
    s.dtype = c[0] ? TPLA_F32 : TPLA_BF16;
    s.d_n = c[3];
    EXPECT(tpla_absorb_query(&s, A, A, NULL, A, NULL) == TPLA_OK);
    const RecordedLaunch& l = last_launch();
    EXPECT((int)l.grid.x == s.H && (int)l.grid.y == (s.d_c + c[5] - 1) / c[5] && (c[6] == 0 || (int)l.grid.z == (s.B + c[6] - 1) / c[6]));
  }
}

int main() {
  plan_checks();
  fitted_plan_checks();
  range_order_checks();
  dispatch_checks();
  decode_rows_dispatch_checks();
  weights_grid_checks();
  absorb_dispatch_checks();
  merge_combine_dispatch_checks();
  lds_opt_in_checks();
  merge_pair_index_checks();
  merge_combine_launch_checks();
  argument_checks();
  block_table_checks();
  pca_checks();
  if (g_failures) {
    fprintf(stderr, "%d expectation(s) failed\n", g_failures);
    return 1;
  }
  printf("abi_host_driver: all expectations held\n");
  return 0;
}
