// bf16 shard decode on the matrix cores (gfx950).
//
// A workgroup processes work items: page ranges of one sequence of one latent
// slice, either a static chunk or whatever falls into its equal share of all
// pages (the balanced kernels).  Cache rows go straight from global memory into a ring of
// LDS buffers with 128-bit direct-to-LDS loads, ahead of the ones being consumed, and
// are shared there by all heads:
//   S^T[tok, head] = K[tok, :] . Q[head, :]      MFMA 16x16x32, M = tokens, N = heads
//   online softmax per head (a lane only ever sees one head of a block)
//   O^T[dim, head] += V^T[dim, tok] . P^T[tok, head]   M = latent dims, N = heads
// The latent prefix of a row is both key and value, so the same LDS rows are
// read row-wise for the scores and through the transposing LDS read for the
// output.  The S^T accumulator layout is already the B-operand layout of the
// second product once the token order inside a 32-token step is permuted
// identically for V^T.
//
// LDS reads of the rows are issued from inline assembly with hand-placed
// lgkmcnt waits: the compiler would otherwise make every LDS read wait for
// all outstanding direct-to-LDS loads, which would serialise the prefetch.
// The compiler takes the destination of such a read for valid from the moment
// it is issued: read, wait and first use must stay in straight-line code, or a
// register copy may land between the read and its wait.
//
// Three bodies: decode_pages (256-wide slices: a page per step, waves of their own for the loads, 32 heads per LDS
// fragment), decode_item (128-wide slices, 16 heads over 512-wide ones, and many static chunks of the others, see static_launch: a tile of
// 32 tokens per step, 16 heads per wave) and decode_item_shared (512-wide slices: two waves per 16 heads, scores handed over through LDS).
#include <hip/hip_ext.h>
#include <algorithm>
#include "lds_tile.h"

namespace tpla {

constexpr int PAGE_TOKENS = 64;

// The reference of the exponentials before a head's first score and after pages on which all of them are -inf: finite, so that their
// weights are 0 (and not NaN, as relative to -inf) and any score moves it.  Which pages or tokens of a sequence come first in a range depends
// on the plan.  A range without any score above -inf has no weights: NaN, which split_merge.h expects beside a reference of -inf.
constexpr float NO_SCORE = -3.402823466e38f;
__device__ __forceinline__ float item_reference(float m) { return m == NO_SCORE ? -INFINITY : m; }
__device__ __forceinline__ float item_sum(float m, float l) { return m == NO_SCORE ? NAN : l; }

// Measurement build only (-DTPLA_WG_TIMELINE, see bench.py --wg-timeline): every workgroup of the
// balanced kernel leaves four readings of the 100 MHz wall clock (start, first tile landed, tile loop
// done, end) and where it ran (XCC id and hardware id registers).  Nothing of this is compiled otherwise.
#ifdef TPLA_WG_TIMELINE
__device__ unsigned long long g_wg_times[4096 * 4];
__device__ unsigned g_wg_where[4096 * 2];
#define TPLA_TL_MARK(k) do { if (threadIdx.x == 0 && blockIdx.y == 0 && blockIdx.x < 4096) g_wg_times[blockIdx.x * 4 + (k)] = wall_clock64(); } while (0)
#define TPLA_TL_MARK_ONCE(k) do { if (threadIdx.x == 0 && blockIdx.y == 0 && blockIdx.x < 4096 && g_wg_times[blockIdx.x * 4 + (k)] == 0) g_wg_times[blockIdx.x * 4 + (k)] = wall_clock64(); } while (0)
#else
#define TPLA_TL_MARK(k) do { } while (0)
#define TPLA_TL_MARK_ONCE(k) do { } while (0)
#endif

// One work item: pages [p0, p1) of sequence b of slice `shard` (L tokens in
// the sequence, p1 <= its page count); the partial result goes to slot
// `slot` of the workspace.  Called by every thread of the workgroup.
template <int DL, int DR, int NW, int TOK, int NSTAGE, int KR>
__device__ __forceinline__ void decode_item(const DecodeArgs& a, u32x4* smem, int shard, int b, int L,
                                            int p0, int p1, size_t slot) {
  constexpr int RC = (DL + DR) / 8;      // 16-byte pieces per row
  constexpr int KS = (DL + DR) / 32;     // k-steps of the score product
  constexpr int DB = DL / 16;            // 16-wide blocks of latent dims
  constexpr int TB = TOK / 16;           // 16-token blocks per tile
  constexpr int S2 = TOK / 32;           // 32-token k-steps of the output product
  constexpr int TC = TOK * RC;           // pieces per tile
  constexpr int NI = TC / 64;            // direct-to-LDS instructions per tile
  constexpr int CPT = (NI + NW - 1) / NW;   // of which each wave issues this many
  constexpr int TPP = PAGE_TOKENS / TOK; // tiles per page
  constexpr int TILE_BYTES = TC * 16;
  static_assert(RC % 8 == 0, "row must be a multiple of 64 elements");
  static_assert(TOK % 32 == 0 && PAGE_TOKENS % TOK == 0 && TC % 64 == 0, "tile size");
  static_assert(NSTAGE >= 2 && NSTAGE <= 4, "the wait counts below cover one to three tiles in flight");
  constexpr int FL = NSTAGE - 1;         // tiles in flight
  static_assert(KR >= 4 && (KR & (KR - 1)) == 0 && KR <= 16, "fragment ring depth");

  const unsigned lds_base = (unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j16 = lane & 15, q4 = lane >> 4;
  const int vb = shard * a.B + b;
  // Page ids of this chunk live in a register, 64 pages at a time (lane i
  // holds page p0 + pg_base + i), and are read back with v_readlane: a memory
  // load per tile would have to wait for every direct-to-LDS load before it.
  int pg_reg = a.block_table[(size_t)b * a.max_pages + min(p0 + lane, p1 - 1)];
  asm volatile("" : "+v"(pg_reg));
  const int t_begin = p0 * PAGE_TOKENS;
  const int t_end = min(p1 * PAGE_TOKENS, L);
  const int ntiles = (t_end - t_begin + TOK - 1) / TOK;
  const int32_t* bt = a.block_table + (size_t)b * a.max_pages;
  const char* pool = static_cast<const char*>(a.pools[shard]);
  // the ring restarts at buffer 0: nobody may still be reading the previous item's tiles
  __syncthreads();

  // ---- direct-to-LDS bookkeeping ---------------------------------------------
  // Instruction k of a tile fills LDS pieces [64k, 64k+64).  This wave issues
  // k = wave + j*NW; when NI is not a multiple of NW the surplus instruction
  // repeats the wave's previous one (same data to the same place).
  int ld_tok[CPT];          // token row of the piece this lane fetches
  unsigned ld_goff[CPT];    // its byte offset inside the tile in global memory
  int ld_k[CPT];
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    int k = wave + j * NW;
    if (k >= NI) k -= NW;
    const int x = k * 64 + lane;                 // LDS piece index
    const int tok = x / RC, cs = x % RC;         // swizzled position -> source piece
    ld_k[j] = k;
    ld_tok[j] = tok;
    ld_goff[j] = (unsigned)((tok * RC + (cs ^ swz(tok))) * 16);
  }
  int pg_base = 0;
  auto issue = [&](int t) {
    const int T = p0 * TPP + t;
    const int pg = t / TPP;                 // page of this chunk, uniform
    if (pg - pg_base >= 64) {
      pg_base += 64;
      pg_reg = bt[min(p0 + pg_base + lane, p1 - 1)];
      asm volatile("" : "+v"(pg_reg));      // the load's wait stays inside this branch
    }
    const int page = __builtin_amdgcn_readlane(pg_reg, pg - pg_base);
    const char* src = pool + (size_t)page * (PAGE_TOKENS * RC * 16) + (size_t)(T % TPP) * TILE_BYTES;
    const int valid = t_end - (t_begin + t * TOK);   // rows >= valid are not read
    char* dst = reinterpret_cast<char*>(smem) + (t % NSTAGE) * TILE_BYTES;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      // every lane issues (the wait counts rely on it); rows past the end of
      // the sequence fetch row 0 of the tile instead and are zeroed afterwards
      const unsigned off = (ld_tok[j] < valid) ? ld_goff[j] : (ld_goff[j] % (RC * 16));
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + off),
                                       (__attribute__((address_space(3))) void*)(dst + ld_k[j] * 1024),
                                       16, 0, 2 /* streaming: do not keep in L2 */);
    }
  };

  // ---- per-lane LDS byte offsets -------------------------------------------
  // score product: token 16*tb + j16, piece 4*ks + q4
  const int xk = swz(j16);
  unsigned k_off[2];
  k_off[0] = (unsigned)((j16 * RC + ((q4) ^ xk)) * 16);
  k_off[1] = (unsigned)((j16 * RC + ((4 | q4) ^ xk)) * 16);
  // output product: token 4*q4 + (j16>>2) (+16), dims 16*db + 4*(j16&3) .. +4
  const int v_tok = 4 * q4 + (j16 >> 2);
  const int xv = swz(v_tok);
  const int cb = (j16 & 3) >> 1;
  unsigned v_off[4];
#pragma unroll
  for (int d = 0; d < 4; ++d)
    v_off[d] = (unsigned)((v_tok * RC + (((d << 1) | cb) ^ xv)) * 16 + (j16 & 1) * 8);

  f32x4 acc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = NO_SCORE, l_run = 0.f;

  issue(0);
  if (FL >= 2 && ntiles > 1) issue(1);
  if (FL >= 3 && ntiles > 2) issue(2);

  // ---- this wave's 16 heads of the query, as B operands --------------------
  const int head = (blockIdx.y * NW + wave) * 16 + j16;
  bf16x8 qreg[KS];
  {
    const bf16_t* ql = static_cast<const bf16_t*>(a.q_lat) + ((size_t)vb * a.H + head) * DL;
    const bf16_t* qp = static_cast<const bf16_t*>(a.q_pe) + ((size_t)b * a.H + head) * DR;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int k0 = ks * 32 + q4 * 8;
      qreg[ks] = (k0 < DL) ? *reinterpret_cast<const bf16x8*>(ql + k0)
                           : *reinterpret_cast<const bf16x8*>(qp + (k0 - DL));
    }
    // complete these loads here: a wait left for their first use would sit
    // inside the tile loop and drain the prefetched tiles on every iteration
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[ks]));
  }


  for (int t = 0; t < ntiles; ++t) {
    // tile t has landed once only the loads of the tiles requested after it are outstanding
    {
      const int later = ntiles - 1 - t;      // tiles after t that exist (FL - 1 of them are in flight at most)
      if (FL >= 3 && later >= 2)
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * CPT));
      else if (FL >= 2 && later >= 1)
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(CPT));
      else
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    }
    // all waves: tile t visible, tile t-1 no longer read.  A bare barrier:
    // __syncthreads() would add a fence that waits for the loads in flight.
    __builtin_amdgcn_s_barrier();
    if (t == 0) TPLA_TL_MARK_ONCE(1);
    if (t + FL < ntiles) issue(t + FL);
    const unsigned tile = lds_base + (unsigned)((t % NSTAGE) * TILE_BYTES);
    const int valid = t_end - (t_begin + t * TOK);
    if (valid < TOK) {
      // last, partial tile: clear the rows past the end of the sequence so
      // that whatever the pool holds there can never reach the accumulators
      u32x4* tl = smem + (t % NSTAGE) * TC;
      for (int x = tid; x < TC; x += NW * 64)
        if (x / RC >= valid) tl[x] = u32x4{0u, 0u, 0u, 0u};
      __syncthreads();
    }

    // ---- scores: a ring of 4 K fragments ahead of the MFMAs -------------------
    f32x4 sacc[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) sacc[tb] = f32x4{0.f, 0.f, 0.f, 0.f};
    {
      constexpr int NQ = KS * TB;          // MFMAs, in order (ks, tb)
      bf16x8 kf[KR];
      const unsigned ka[2] = {tile + k_off[0], tile + k_off[1]};
      static_for<KR>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        constexpr int ks = i / TB, tb = i % TB;
        lds_read_b128<(ks >> 1) * 128 + tb * (16 * RC * 16)>(kf[i], ka[ks & 1]);
      });
      static_for<NQ>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        constexpr int ks = i / TB, tb = i % TB;
        constexpr int ahead = (NQ - 1 - i) < KR - 1 ? (NQ - 1 - i) : KR - 1;
        lds_wait<ahead>(kf[i & (KR - 1)]);
        sacc[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[i & (KR - 1)], qreg[ks], sacc[tb], 0, 0, 0);
        if constexpr (i + KR < NQ) {
          constexpr int ks2 = (i + KR) / TB, tb2 = (i + KR) % TB;
          lds_read_b128<(ks2 >> 1) * 128 + tb2 * (16 * RC * 16)>(kf[i & (KR - 1)], ka[ks2 & 1]);
        }
      });
    }

    // ---- online softmax (lane = one head; tokens 16*tb + 4*q4 + i) ----------
    // The reference m_run of the exponentials is only moved when some score
    // exceeds it by more than LAZY (weights stay <= 2^LAZY, harmless in
    // float), so the accumulator rescale is off the common path.
    if (valid < TOK) {
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (16 * tb + 4 * q4 + i >= valid) sacc[tb][i] = -INFINITY;
    }
    float mx = sacc[0][0];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
#pragma unroll
      for (int i = 0; i < 4; ++i) mx = fmaxf(mx, sacc[tb][i]);
    mx *= a.scale_log2;
    if (__any(mx > m_run + LAZY)) {
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m_run, mx);
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);   // 0 on the first tile
      l_run *= alpha;
      m_run = m_new;
#pragma unroll
      for (int d = 0; d < DB; ++d) acc[d] *= alpha;
    }
    float psum = 0.f;
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sacc[tb][i], a.scale_log2, -m_run));
        sacc[tb][i] = p;
        psum += p;
      }
    l_run += psum;

    // ---- output: O^T += V^T P^T, a ring of 4 V fragments ---------------------
#pragma unroll
    for (int s2 = 0; s2 < S2; ++s2) {
      bf16x8 pb;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        pb[i] = (bf16_t)sacc[2 * s2][i];
        pb[4 + i] = (bf16_t)sacc[2 * s2 + 1][i];
      }
      constexpr int VR = KR <= 8 ? KR : 8;     // two reads per fragment: the wait counter allows 15 outstanding
      u32x2 vlo[VR], vhi[VR];
      unsigned va[4];
#pragma unroll
      for (int d = 0; d < 4; ++d) va[d] = tile + v_off[d] + (unsigned)(s2 * (32 * RC * 16));
      static_for<VR>([&](auto ic) {
        constexpr int d = decltype(ic)::value;
        lds_read_tr_b64<(d >> 2) * 128>(vlo[d], va[d & 3]);
        lds_read_tr_b64<(d >> 2) * 128 + 16 * RC * 16>(vhi[d], va[d & 3]);
      });
      static_for<DB>([&](auto ic) {
        constexpr int d = decltype(ic)::value;
        constexpr int ahead = (DB - 1 - d) < VR - 1 ? (DB - 1 - d) : VR - 1;
        lds_wait<2 * ahead>(vlo[d & (VR - 1)], vhi[d & (VR - 1)]);
        const u32x4 v4 = {vlo[d & (VR - 1)][0], vlo[d & (VR - 1)][1], vhi[d & (VR - 1)][0], vhi[d & (VR - 1)][1]};
        acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v4), pb, acc[d], 0, 0, 0);
        if constexpr (d + VR < DB) {
          constexpr int d2 = d + VR;
          lds_read_tr_b64<(d2 >> 2) * 128>(vlo[d & (VR - 1)], va[d2 & 3]);
          lds_read_tr_b64<(d2 >> 2) * 128 + 16 * RC * 16>(vhi[d & (VR - 1)], va[d2 & 3]);
        }
      });
    }
    }

  TPLA_TL_MARK(2);
  float l_tot = l_run + __shfl_xor(l_run, 16);
  l_tot += __shfl_xor(l_tot, 32);
  const size_t item = slot * a.H + head;
  float* pacc = a.part_acc + item * DL + 4 * q4;
#pragma unroll
  for (int d = 0; d < DB; ++d) *reinterpret_cast<f32x4*>(pacc + 16 * d) = acc[d];
  if (q4 == 0) {
    a.part_ml[item * 2 + 0] = item_reference(m_run);
    a.part_ml[item * 2 + 1] = item_sum(m_run, l_tot);
  }
}

// The same work item for rows too wide for two workgroups per compute unit (576-wide rows: one tile is
// 36 KB), where decode_item would leave every SIMD with a single wave and nothing to run under its MFMAs.
// Two waves share 16 heads.  Of a 32-token tile each computes the scores of 16 tokens (half the score
// MFMAs) and hands them to its partner through LDS; both then run the same softmax on all 32 tokens --
// same inputs, same operations, so their running reference and sum stay equal bit for bit -- and each
// multiplies the weights into its own half of the latent dims (half the output MFMAs, 64 accumulator
// registers instead of 128, which is what lets two waves share a SIMD).  The hand-over would cost a
// second barrier per tile; instead the loop is skewed by one tile: round r computes the scores of tile r
// and the softmax and output product of tile r - 1, and the round's one barrier publishes the tile and
// the partner's scores together.  Ring: tiles r - 1 and r in use, r + 1 and r + 2 in flight.
// LDS: NSTAGE tiles, then two buffers of one f32x4 per lane of every wave for the scores.
template <int DL, int DR, int NW, int TOK, int NSTAGE, int KR>
__device__ __forceinline__ void decode_item_shared(const DecodeArgs& a, u32x4* smem, int shard, int b, int L,
                                                   int p0, int p1, size_t slot) {
  constexpr int RC = (DL + DR) / 8;      // 16-byte pieces per row
  constexpr int KS = (DL + DR) / 32;     // k-steps of the score product
  constexpr int DBH = DL / 32;           // 16-wide blocks of this wave's half of the latent dims
  constexpr int TC = TOK * RC;           // pieces per tile
  constexpr int NI = TC / 64;            // direct-to-LDS instructions per tile
  constexpr int NWT = 2 * NW;            // waves in the workgroup
  constexpr int CPT = (NI + NWT - 1) / NWT;
  constexpr int TPP = PAGE_TOKENS / TOK;
  constexpr int TILE_BYTES = TC * 16;
  constexpr int VR = 4;                  // V fragments in flight
  static_assert(TOK == 32 && NSTAGE == 4, "two tiles in use, two in flight");
  static_assert(RC % 8 == 0 && TC % 64 == 0 && DBH % VR == 0, "tile shape");
  static_assert(KR >= 4 && (KR & (KR - 1)) == 0 && KR <= 16, "fragment ring depth");

  const unsigned lds_base = (unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)smem);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int half = wv / NW, wave = wv % NW;      // half 0: tokens 0-15 and the first DL/2 dims; wave: heads 16 wave ..
  const int partner = (1 - half) * NW + wave;
  const int j16 = lane & 15, q4 = lane >> 4;
  const int vb = shard * a.B + b;
  int pg_reg = a.block_table[(size_t)b * a.max_pages + min(p0 + lane, p1 - 1)];
  asm volatile("" : "+v"(pg_reg));
  const int t_begin = p0 * PAGE_TOKENS;
  const int t_end = min(p1 * PAGE_TOKENS, L);
  // scalar: the rounds below branch on it, and a branch the compiler takes for divergent would put
  // register copies between an LDS read in assembly and the wait that makes its result valid
  const int ntiles = __builtin_amdgcn_readfirstlane((t_end - t_begin + TOK - 1) / TOK);
  const int32_t* bt = a.block_table + (size_t)b * a.max_pages;
  const char* pool = static_cast<const char*>(a.pools[shard]);
  // the ring and the score buffers restart: nobody may still be reading the previous item's
  __syncthreads();

  // ---- direct-to-LDS bookkeeping (as in decode_item, over all waves of the workgroup) ----
  int ld_tok[CPT];
  unsigned ld_goff[CPT];
  int ld_k[CPT];
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    int k = wv + j * NWT;
    if (k >= NI) k -= NWT;                       // surplus instruction: repeats the wave's previous one
    const int x = k * 64 + lane;
    const int tok = x / RC, cs = x % RC;
    ld_k[j] = k;
    ld_tok[j] = tok;
    ld_goff[j] = (unsigned)((tok * RC + (cs ^ swz(tok))) * 16);
  }
  int pg_base = 0;
  auto issue = [&](int t) {
    const int T = p0 * TPP + t;
    const int pg = t / TPP;
    if (pg - pg_base >= 64) {
      pg_base += 64;
      pg_reg = bt[min(p0 + pg_base + lane, p1 - 1)];
      asm volatile("" : "+v"(pg_reg));
    }
    const int page = __builtin_amdgcn_readlane(pg_reg, pg - pg_base);
    const char* src = pool + (size_t)page * (PAGE_TOKENS * RC * 16) + (size_t)(T % TPP) * TILE_BYTES;
    const int valid = t_end - (t_begin + t * TOK);
    char* dst = reinterpret_cast<char*>(smem) + (t % NSTAGE) * TILE_BYTES;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      const unsigned off = (ld_tok[j] < valid) ? ld_goff[j] : (ld_goff[j] % (RC * 16));
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + off),
                                       (__attribute__((address_space(3))) void*)(dst + ld_k[j] * 1024),
                                       16, 0, 2 /* streaming: do not keep in L2 */);
    }
  };
  // rows of a tile past the end of the sequence are cleared once it has landed (the last tile only)
  auto clear_tail = [&](int t) {
    const int valid = t_end - (t_begin + t * TOK);
    if (valid < TOK) {
      u32x4* tl = smem + (t % NSTAGE) * TC;
      for (int x = tid; x < TC; x += NWT * 64)
        if (x / RC >= valid) tl[x] = u32x4{0u, 0u, 0u, 0u};
      __syncthreads();
    }
  };

  // ---- per-lane LDS byte offsets ----
  // score product: token 16 half + j16, piece 4 ks + q4
  const int k_tok = 16 * half + j16;
  const int xk = swz(k_tok);
  unsigned k_off[2];
  k_off[0] = (unsigned)((k_tok * RC + ((q4) ^ xk)) * 16);
  k_off[1] = (unsigned)((k_tok * RC + ((4 | q4) ^ xk)) * 16);
  // output product: token 4 q4 + (j16 >> 2) (+16), dims (DL / 2) half + 16 d + 4 (j16 & 3) .. +4
  const int v_tok = 4 * q4 + (j16 >> 2);
  const int xv = swz(v_tok);
  const int cb = (j16 & 3) >> 1;
  unsigned v_off[4];
#pragma unroll
  for (int d = 0; d < 4; ++d)
    v_off[d] = (unsigned)((v_tok * RC + (((d << 1) | cb) ^ xv)) * 16 + (j16 & 1) * 8 + half * DL);   // DL bytes = DL / 2 dims

  f32x4 acc[DBH];
#pragma unroll
  for (int d = 0; d < DBH; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = NO_SCORE, l_run = 0.f;

  issue(0);
  if (ntiles > 1) issue(1);

  // ---- the 16 heads of this wave pair, as B operands ----
  const int head = (blockIdx.y * NW + wave) * 16 + j16;
  bf16x8 qreg[KS];
  {
    const bf16_t* ql = static_cast<const bf16_t*>(a.q_lat) + ((size_t)vb * a.H + head) * DL;
    const bf16_t* qp = static_cast<const bf16_t*>(a.q_pe) + ((size_t)b * a.H + head) * DR;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int k0 = ks * 32 + q4 * 8;
      qreg[ks] = (k0 < DL) ? *reinterpret_cast<const bf16x8*>(ql + k0)
                           : *reinterpret_cast<const bf16x8*>(qp + (k0 - DL));
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[ks]));   // complete before the loop
  }

  // scores of this wave's 16 tokens of the tile at LDS address `tile`
  auto scores = [&](unsigned tile) {
    f32x4 sc = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 kf[KR];
    const unsigned ka[2] = {tile + k_off[0], tile + k_off[1]};
    static_for<KR>([&](auto ic) {
      constexpr int ks = decltype(ic)::value;
      lds_read_b128<(ks >> 1) * 128>(kf[ks], ka[ks & 1]);
    });
    static_for<KS>([&](auto ic) {
      constexpr int ks = decltype(ic)::value;
      constexpr int ahead = (KS - 1 - ks) < KR - 1 ? (KS - 1 - ks) : KR - 1;
      lds_wait<ahead>(kf[ks & (KR - 1)]);
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks & (KR - 1)], qreg[ks], sc, 0, 0, 0);
      if constexpr (ks + KR < KS) lds_read_b128<((ks + KR) >> 1) * 128>(kf[ks & (KR - 1)], ka[(ks + KR) & 1]);
    });
    return sc;
  };

  // ---- round 0: the scores of tile 0 ----
  if (ntiles > 1)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(CPT));
  else
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  __builtin_amdgcn_s_barrier();
  TPLA_TL_MARK_ONCE(1);
  if (ntiles > 2) issue(2);
  clear_tail(0);
  // The hand-over is written with a plain store (the compiler then keeps the wait states an MFMA result
  // needs before an LDS instruction may read it) and read with inline assembly like the tiles (a plain
  // LDS load after a direct-to-LDS load would make the compiler wait for every load in flight).
  f32x4* x_own = reinterpret_cast<f32x4*>(smem + NSTAGE * TC) + wv * 64 + lane;
  const unsigned x_partner = lds_base + (unsigned)(NSTAGE * TILE_BYTES + (partner * 64 + lane) * 16);
  constexpr unsigned XBUF = NWT * 64 * 16;       // bytes per hand-over buffer
  f32x4 s_own = scores(lds_base);
  x_own[0] = s_own;

  // ---- round r: scores of tile r (while there is one), softmax and output product of tile r - 1 ----
  for (int r = 1; r <= ntiles; ++r) {
    const bool more = r < ntiles;
    // tile r has landed once only tile r + 1 (requested in the round before) is outstanding
    if (r + 1 < ntiles)
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(CPT));
    else
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    // the hand-over written in round r - 1 must have left this wave before the barrier publishes it
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();        // tile r and the partners' scores of tile r - 1 visible; tile r - 2 no longer read
    if (r + 2 < ntiles) issue(r + 2);
    if (more) clear_tail(r);
    const f32x4 s_prev = s_own;
    f32x4 s_partner;
    asm volatile("ds_read_b128 %0, %1" : "=v"(s_partner) : "v"(x_partner + ((r - 1) & 1) * XBUF) : "memory");
    if (more) {
      s_own = scores(lds_base + (unsigned)((r % NSTAGE) * TILE_BYTES));
      x_own[(r & 1) * (XBUF / 16)] = s_own;
    }
    // one wait on one path for both cases, straight after the branch (which does not touch s_partner)
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(s_partner) : : "memory");
    const unsigned tile = lds_base + (unsigned)(((r - 1) % NSTAGE) * TILE_BYTES);
    const int valid = t_end - (t_begin + (r - 1) * TOK);

    // the first V fragments start now, under the softmax arithmetic
    u32x2 vlo[VR], vhi[VR];
    unsigned va[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) va[d] = tile + v_off[d];
    static_for<VR>([&](auto ic) {
      constexpr int d = decltype(ic)::value;
      lds_read_tr_b64<(d >> 2) * 128>(vlo[d], va[d & 3]);
      lds_read_tr_b64<(d >> 2) * 128 + 16 * RC * 16>(vhi[d], va[d & 3]);
    });

    // ---- online softmax on all 32 tokens (lane = one head; tokens 16 tb + 4 q4 + i) ----
    f32x4 sacc[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sacc[0][i] = half ? s_partner[i] : s_prev[i];
      sacc[1][i] = half ? s_prev[i] : s_partner[i];
    }
    if (valid < TOK) {
#pragma unroll
      for (int tb = 0; tb < 2; ++tb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (16 * tb + 4 * q4 + i >= valid) sacc[tb][i] = -INFINITY;
    }
    float mx = sacc[0][0];
#pragma unroll
    for (int tb = 0; tb < 2; ++tb)
#pragma unroll
      for (int i = 0; i < 4; ++i) mx = fmaxf(mx, sacc[tb][i]);
    mx *= a.scale_log2;
    if (__any(mx > m_run + LAZY)) {
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m_run, mx);
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);   // 0 on the first tile
      l_run *= alpha;
      m_run = m_new;
#pragma unroll
      for (int d = 0; d < DBH; ++d) acc[d] *= alpha;
    }
    float psum = 0.f;
    bf16x8 pb;
#pragma unroll
    for (int tb = 0; tb < 2; ++tb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sacc[tb][i], a.scale_log2, -m_run));
        psum += p;
        pb[4 * tb + i] = (bf16_t)p;
      }
    l_run += psum;

    // ---- output: O^T += V^T P^T over this wave's half of the dims ----
    static_for<DBH>([&](auto ic) {
      constexpr int d = decltype(ic)::value;
      constexpr int ahead = (DBH - 1 - d) < VR - 1 ? (DBH - 1 - d) : VR - 1;
      lds_wait<2 * ahead>(vlo[d & (VR - 1)], vhi[d & (VR - 1)]);
      const u32x4 v4 = {vlo[d & (VR - 1)][0], vlo[d & (VR - 1)][1], vhi[d & (VR - 1)][0], vhi[d & (VR - 1)][1]};
      acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v4), pb, acc[d], 0, 0, 0);
      if constexpr (d + VR < DBH) {
        constexpr int d2 = d + VR;
        lds_read_tr_b64<(d2 >> 2) * 128>(vlo[d & (VR - 1)], va[d2 & 3]);
        lds_read_tr_b64<(d2 >> 2) * 128 + 16 * RC * 16>(vhi[d & (VR - 1)], va[d2 & 3]);
      }
    });
  }

  TPLA_TL_MARK(2);
  float l_tot = l_run + __shfl_xor(l_run, 16);
  l_tot += __shfl_xor(l_tot, 32);
  const size_t item = slot * a.H + head;
  float* pacc = a.part_acc + item * DL + (DL / 2) * half + 4 * q4;
#pragma unroll
  for (int d = 0; d < DBH; ++d) *reinterpret_cast<f32x4*>(pacc + 16 * d) = acc[d];
  if (q4 == 0 && half == 0) {
    a.part_ml[item * 2 + 0] = item_reference(m_run);
    a.part_ml[item * 2 + 1] = item_sum(m_run, l_tot);
  }
}

// Rows of up to 320 elements: one workgroup per compute unit, one page (64 tokens) per step, all pages of the
// workgroup through one ring of LDS buffers.
//
// What bounds the step per 16 heads and wave that decode_item takes (whole tile read from LDS by every wave, tiles requested by
// the waves that compute) at 64 heads: LDS, 144 KB of reads and the 20 KB themselves per tile, 1300 of its 1700 clocks at 128 bytes per clock, and in short
// launches the requests: with the memory system busy a wave stands for 100 clocks and more at each of its five direct-to-LDS loads, 600 of
// the 1900 clocks of a tile.  Here
//   * NP waves of their own request the pages (and never compute), NSTAGE - 1 pages ahead, across the ends of sequences;
//   * (a compute unit holds one such workgroup; half as many partial results for the merge to read)
//   * a wave computes for 16 HB heads (32; 16 where there are no more), so that an LDS fragment serves two blocks of heads:
//     of a page, the scores of 16 tokens (part of 4), and of the output product a quarter of the latent dims.  The four waves of a
//     head group swap their exponentiated weights through LDS in bf16 between the two, as the B operands they are read as.
// LDS reads per 64 tokens, 64 heads and 256-wide slices: 80 KB keys, 64 KB values, 32 KB weights (decode_item: 288 KB); with what is
// written some 1800 of 3200 clocks per page, matrix cores 36 % busy, waves waiting half of their time.  An
// item's queries come through the ring too, as a step of their own laid out like a page: read from global memory by every wave they
// are 160 KB per workgroup in 64-byte pieces, which held up its first page by 2 us.
// Split kernel, 64 heads over 256-wide slices, against decode_item with two workgroups per compute unit (us): one sequence of
// 1300 tokens 11.0 -> 9.8, 16 x 4096 27.5 -> 22.4, 23 ragged sequences (145 MB) 42.5 -> 34.4, 32 x 32768 (1342 MB) 216 -> 203 = 6.6 TB/s; 32
// heads, 64 x 32768: 399 -> 392; 16 heads, 164 MB: 36.6 -> 30.4; 128 heads, 164 MB: 59.0 -> 50.0 (3.3 TB/s: two rows of workgroups fetch
// every page, and each computes as much for it as 64 heads do).  A page takes 1.4 to 1.6 us in the launches of up to 64 heads, near what
// memory allows; what is left is 5 us to the first page and the flush of the results.
//
// Barriers of a step, met by every wave of the workgroup: the page has landed (and nobody reads the page, the weights and
// the sums before it any more); on an item's first page, the highest scores are in LDS; the weights are written.  When later a score exceeds the running reference of its head by more
// than LAZY (the rule of the other bodies), the wave that sees it writes the step's number to a flag next to the weights; every wave reads it after the
// second barrier, and all of them then agree on the new reference through LDS (two more barriers) and write the weights again.
//
// LDS: NSTAGE pages; weights [head group][head block][32-token step][lane][8]; candidates for the reference and sums
// [wave][32] floats each; references [head group][32] floats; the flag.
constexpr int PARTS = 4;
template <int DL, int DR, int HG, int HB, int NSTAGE>
struct PageLds {
  static constexpr int RC = (DL + DR) / 8, PAGE_BYTES = PAGE_TOKENS * RC * 16;
  static constexpr int weights = NSTAGE * PAGE_BYTES;
  static constexpr int cand = weights + HG * HB * 2 * 1024;
  static constexpr int sums = cand + HG * PARTS * 32 * 4;
  static constexpr int refs = sums + HG * PARTS * 32 * 4;
  static constexpr int flag = refs + HG * 32 * 4;
  static constexpr int bytes = flag + 16;
};

// The order of an item's pages: from one in the middle to the end, then from the first.  With pools whose pages lie in sequence
// order the workgroups would otherwise begin at equal distances from each other and stay there, on few memory
// channels at a time.  Where an item begins is a fraction of it, from one workgroup to the next in steps of `STEP` / 2^16.  What the
// steps do depends on how the ranges lie to the channels; this one is the best of 60 over 19 shapes (16 to 64 heads, 8 to 96 sequences of
// 8192 to 131072 tokens) and within 6 % of the best for each of them.  Split and merge, pools in sequence order, us:
//                                          from the first page   617 / 1024   a hash   this
//   64 heads, 32 x 32768, one slice              116.6             132.4       115.2    113.6   (pages in random order 110)
//   8 x 131072, one slice                        116.5             134.2       113.6    112.3
//   32 x 32832, one slice                        113.2             130.8       116.8    114.6
//   32 heads, 64 x 32768, both                   433.9             394.2       401.2    394.6
//   64 heads, 32 x 32768, both                   217.6             214.2       215.0    210.7
// (Longer ranges than 2^16 pages begin within their first 2^16.)
struct PageOrder {
  static constexpr unsigned STEP = 12337;
  int p, p0, p1;
  __device__ __forceinline__ PageOrder(int turn, int first, int end)
      : p(first + (int)((((unsigned)turn * STEP) & 65535u) * (unsigned)(end - first) >> 16)), p0(first), p1(end) {}
  __device__ __forceinline__ int next() const { return p + 1 == p1 ? p0 : p + 1; }
};

// Work of one workgroup (for the heads of its blockIdx.y): for_items(f) calls f(slice, sequence, tokens of the sequence, first page,
// end page, slot, turn) for its items in order; turn decides where in an item it begins.  Called by every thread of the workgroup.
// KEEP: pages stay in L2.  For long ranges of two rows of workgroups, where the other row finds them (both run on the same XCD); shorter ones
// lose more to the partial results that have to make room.  128 heads, split and merge, streaming / kept: 512 pages in the
// workgroup's range 758 / 731 us, 256 381 / 374, 128 194.7 / 195.0, 13 (ragged) 38.5 / 39.4; one row 210 / 230.  A copy of the body
// for each: with a branch around the loads instead, launches of either kind took 8 to 12 % longer.
constexpr int KEEP_PAGES = 128;      // of a range
template <int DL, int DR, int HG, int HB, int NP, int NSTAGE, bool KEEP, typename ForItems>
__device__ __forceinline__ void decode_pages(const DecodeArgs& a, u32x4* smem, ForItems&& for_items) {
  using Lds = PageLds<DL, DR, HG, HB, NSTAGE>;
  constexpr int RC = Lds::RC;            // 16-byte pieces per row
  constexpr int KS = (DL + DR) / 32;     // k-steps of the score product
  constexpr int DB = DL / 16 / PARTS;    // 16-wide blocks of a wave's quarter of the latent dims
  constexpr int TC = PAGE_TOKENS * RC;   // pieces per page
  constexpr int NI = TC / 64;            // direct-to-LDS instructions per page
  constexpr int CPT = NI / NP;           // of which each loading wave issues this many
  constexpr int GROUP_BYTES = 16 * RC * 16, CPG = CPT / 4;      // 16 rows; instructions per group and loading wave
  constexpr int FL = NSTAGE - 1;         // pages in flight
  constexpr int NC = HG * PARTS;         // waves that compute
  constexpr int HEADS = HG * HB * 16;    // of this workgroup
  static_assert(RC % 8 == 0 && TC % 64 == 0 && NI % (4 * NP) == 0, "page shape");
  static_assert(NSTAGE >= 2 && NSTAGE <= 5 && (FL - 1) * CPT < 64, "the waits below");
  static_assert(KS >= 4 && (HB == 1 || HB == 2), "fragment ring, head blocks");

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int lane = threadIdx.x & 63;
  const unsigned lds_base = (unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)smem);
  const unsigned flag_at = lds_base + Lds::flag;
  // one step's flag, the same in all waves (and lanes): the step's number + 1 if a reference has to move
  auto flag_raised = [&](int step) {
    int f;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(f) : "v"(flag_at) : "memory");
    return __builtin_amdgcn_readfirstlane(f) == step + 1;
  };
  if (threadIdx.x == 0) *reinterpret_cast<int*>(reinterpret_cast<char*>(smem) + Lds::flag) = 0;
  __syncthreads();

  if (wave >= NC) {
    // ======== the waves that request the pages ========
    // Groups of 16 rows, all fetched alike: instruction k of a group fills its LDS pieces [64k, 64k+64); this wave issues
    // k = pw + j*NP.  (Little code and in one place: what runs once per launch costs its instruction fetches.)
    const int pw = wave - NC;
    unsigned goff[CPG];                  // byte offset inside the group of the piece this lane fetches
#pragma unroll
    for (int j = 0; j < CPG; ++j) {
      const int x = (pw + j * NP) * 64 + lane;     // LDS piece index
      const int tok = x / RC, cs = x % RC;         // swizzled position -> source piece
      goff[j] = (unsigned)((tok * RC + (cs ^ swz(tok))) * 16);
    }
    int n = 0;                           // steps requested
    unsigned queries = 0;                // bit k: step n - 1 - k brings queries
    // groups [g0, g1) of page n.  Rows past the end of the sequence fetch its row 0 of the page instead: their scores are
    // masked and their weights 0, and every lane issues (the wait counts rely on it).
    auto request = [&](const char* src, int valid, int g0, int g1) {
      char* dst = reinterpret_cast<char*>(smem) + (n % NSTAGE) * Lds::PAGE_BYTES + pw * 1024;
#pragma clang loop unroll(disable)
      for (int g = g0; g < g1; ++g) {
        unsigned off[CPG];
#pragma unroll
        for (int j = 0; j < CPG; ++j) off[j] = goff[j] + g * GROUP_BYTES;
        if (valid < 16 * (g + 1)) {
#pragma unroll
          for (int j = 0; j < CPG; ++j)
            if (off[j] >= (unsigned)(valid * RC * 16)) off[j] %= RC * 16;
        }
#pragma unroll
        for (int j = 0; j < CPG; ++j)
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + off[j]),
                                           (__attribute__((address_space(3))) void*)(dst + g * GROUP_BYTES + j * NP * 1024),
                                           16, 0, KEEP ? 0 : 2 /* streaming: do not keep in L2 */);
      }
    };
    // the barriers of step m, after the first of which step m + FL may be requested into the buffer of step m - 1: half
    // of it between the barriers
    auto step = [&](int m, const char* src, int valid) {
      // what was requested after step m may be outstanding: its pages (that of queries, which has fewer instructions, is waited for)
      const int later = n - 1 - m - __builtin_popcount(queries & ((1u << (n - 1 - m)) - 1));
      if (later >= 3 && FL >= 4)
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(3 * CPT < 64 ? 3 * CPT : 63));
      else if (later >= 2 && FL >= 3)
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * CPT < 64 ? 2 * CPT : 63));
      else if (later >= 1 && FL >= 2)
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(CPT));
      else
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      __builtin_amdgcn_s_barrier();
      if (src) request(src, valid, 0, 2);
      const unsigned kind = queries >> (n - 1 - m);
      if (kind & 1) return;
      if (kind & 2) __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_s_barrier();
      if (flag_raised(m)) {
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_s_barrier();
      }
    };
    for_items([&](int shard, int b, int L, int p0, int p1, size_t, int turn) {
      // page ids come through scalar loads: a vector load would have to wait for every direct-to-LDS load before it
      const __attribute__((address_space(4))) int32_t* bt =
          (const __attribute__((address_space(4))) int32_t*)(uintptr_t)(a.block_table + (size_t)b * a.max_pages);
      const char* pool = static_cast<const char*>(a.pools[shard]);
      if (n >= FL) step(n - FL, nullptr, 0);
      // the queries, laid out like a page: row h is head h of this workgroup, latent part then RoPE part
      const char* ql = static_cast<const char*>(a.q_lat) + ((size_t)(shard * a.B + b) * a.H + blockIdx.y * HEADS) * (DL * 2);
      const char* qp = static_cast<const char*>(a.q_pe) + ((size_t)b * a.H + blockIdx.y * HEADS) * (DR * 2);
      // scalar loads return in any order, so a wait is for all of them: the arguments first, then the page id under the
      // requests of the queries
      asm volatile("" : "+s"(ql), "+s"(qp), "+s"(pool), "+s"(bt));
      PageOrder at(turn, p0, p1);
      int id = bt[at.p];
      {
        char* dst = reinterpret_cast<char*>(smem) + (n % NSTAGE) * Lds::PAGE_BYTES + pw * 1024;
        const char* src[CPG];
        unsigned next[CPG];              // from a group of 16 heads to the next
#pragma unroll
        for (int j = 0; j < CPG; ++j) {
          const unsigned row = goff[j] / (RC * 16), in_row = goff[j] % (RC * 16);
          const bool latent = in_row < DL * 2;
          src[j] = latent ? ql + row * (DL * 2) + in_row : qp + row * (DR * 2) + (in_row - DL * 2);
          next[j] = 16 * 2 * (latent ? DL : DR);
        }
#pragma clang loop unroll(disable)
        for (int g = 0; g < HEADS / 16; ++g)
#pragma unroll
          for (int j = 0; j < CPG; ++j) {
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src[j],
                                             (__attribute__((address_space(3))) void*)(dst + g * GROUP_BYTES + j * NP * 1024), 16, 0, 0);
            src[j] += next[j];
          }
        queries = queries << 1 | 1;
        ++n;
      }
      for (int i = p0; i < p1; ++i) {
        const char* src = pool + (size_t)id * Lds::PAGE_BYTES;
        const int valid = min(L - at.p * PAGE_TOKENS, PAGE_TOKENS);
        at.p = at.next();
        id = bt[at.p];
        if (n >= FL) step(n - FL, src, valid);
        request(src, valid, n >= FL ? 2 : 0, 4);
        queries <<= 1;
        ++n;
      }
    });
    for (int m = n < FL ? 0 : n - FL; m < n; ++m) step(m, nullptr, 0);      // what is still in flight
    __builtin_amdgcn_s_barrier();        // the sums of the last item
    return;
  }

  // ======== the waves that compute ========
  const int part = wave % PARTS, hg = wave / PARTS;
  float* const cand = reinterpret_cast<float*>(reinterpret_cast<char*>(smem) + Lds::cand);
  float* const sums = reinterpret_cast<float*>(reinterpret_cast<char*>(smem) + Lds::sums);
  float* const refs = reinterpret_cast<float*>(reinterpret_cast<char*>(smem) + Lds::refs);
  const int j16 = lane & 15, q4 = lane >> 4;
  // ---- per-lane LDS byte offsets ----
  // score product: token 16 part + j16, piece 4 ks + q4
  const int k_tok = 16 * part + j16;
  const int xk = swz(k_tok);
  const unsigned k_off = (unsigned)((k_tok * RC + (q4 ^ xk)) * 16);          // odd k-steps: ^ 64
  // output product: token 4 q4 + (j16 >> 2) (+ 16, + 32, + 48), dims (DL / 4) part + 16 d + 4 (j16 & 3) .. + 4
  const int v_tok = 4 * q4 + (j16 >> 2);
  const int v_pc = part * (DL / 8 / PARTS) + ((j16 & 3) >> 1);
  const unsigned v_off = (unsigned)((v_tok * RC + (v_pc ^ swz(v_tok))) * 16 + (j16 & 1) * 8);      // block d: ^ 32 d
  // weights of the tokens of part p: k-step p / 2, elements 4 (p % 2) .. + 4 of every lane
  const unsigned w_read = lds_base + (unsigned)(Lds::weights + hg * (HB * 2048) + lane * 16);
  const unsigned w_write = w_read + (unsigned)((part >> 1) * 1024 + (part & 1) * 8);

  int n = 0;                             // pages done
  // (reference, sum) of the item before, still to be written: its address, or null
  float* ml_pending = nullptr;
  auto write_pending = [&]() {           // between two barriers; dealt over the parts by head block
    if (ml_pending && part < HB) {
      int ln = lane;                     // computed anew: the addresses would hold registers for good
      asm volatile("" : "+v"(ln));
      if (ln < 16) {
      const int h = part * 16 + ln;
      float l = 0.f;
#pragma unroll
      for (int i = 0; i < PARTS; ++i) l += sums[(hg * PARTS + i) * 32 + h];
      ml_pending[2 * h] = refs[hg * 32 + h];
      ml_pending[2 * h + 1] = l;
      }
    }
    ml_pending = nullptr;
  };

  for_items([&](int shard, int b, int L, int p0, int p1, size_t slot, int turn) {
    const int vb = shard * a.B + b;
    const int head0 = (blockIdx.y * HG + hg) * (HB * 16);
    // ---- the heads of this group, as B operands: read from the step that brought the queries ----
    __builtin_amdgcn_s_barrier();
    write_pending();
    bf16x8 qreg[HB][KS];
    {
      const unsigned q_off = lds_base + (unsigned)((n % NSTAGE) * Lds::PAGE_BYTES + ((hg * (HB * 16) + j16) * RC + (q4 ^ xk)) * 16);
      const unsigned qa[2] = {q_off, q_off ^ 64u};
      static_for<HB>([&](auto hc) {                // (the wait counter holds 15)
        constexpr int hb = decltype(hc)::value;
        static_for<KS>([&](auto ic) {
          constexpr int ks = decltype(ic)::value;
          lds_read_b128<(ks >> 1) * 128 + hb * (16 * RC * 16)>(qreg[hb][ks], qa[ks & 1]);
        });
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) lds_wait<0>(qreg[hb][ks]);
      });
      ++n;
    }
    f32x4 acc[HB][DB];
    float m_run[HB], l_run[HB];
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) {
      m_run[hb] = -INFINITY;
      l_run[hb] = 0.f;
#pragma unroll
      for (int d = 0; d < DB; ++d) acc[hb][d] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    PageOrder at(turn, p0, p1);
#pragma clang loop unroll(disable)
    for (int i = p0; i < p1; ++i, ++n, at.p = at.next()) {
      __builtin_amdgcn_s_barrier();
      if (n == 1) TPLA_TL_MARK_ONCE(1);          // step 0 brought the queries
      const unsigned page = lds_base + (unsigned)((n % NSTAGE) * Lds::PAGE_BYTES);
      const int valid = L - at.p * PAGE_TOKENS;

      // ---- scores of this wave's 16 tokens: a ring of 4 K fragments ahead of the MFMAs ----
      // (lane = head j16 of every block; tokens 16 part + 4 q4 + i)
      f32x4 sacc[HB];
      auto scores = [&]() {
        bf16x8 kf[4];
        const unsigned ka[2] = {page + k_off, (page + k_off) ^ 64u};
        static_for<4>([&](auto ic) {
          constexpr int ks = decltype(ic)::value;
          lds_read_b128<(ks >> 1) * 128>(kf[ks], ka[ks & 1]);
        });
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) sacc[hb] = f32x4{0.f, 0.f, 0.f, 0.f};
        static_for<KS>([&](auto ic) {
          constexpr int ks = decltype(ic)::value;
          constexpr int ahead = (KS - 1 - ks) < 3 ? (KS - 1 - ks) : 3;
          lds_wait<ahead>(kf[ks & 3]);
#pragma unroll
          for (int hb = 0; hb < HB; ++hb)
            sacc[hb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks & 3], qreg[hb][ks], sacc[hb], 0, 0, 0);
          if constexpr (ks + 4 < KS) lds_read_b128<((ks + 4) >> 1) * 128>(kf[ks & 3], ka[(ks + 4) & 1]);
        });
        // The wait states between an MFMA and the first VALU instruction that reads its result, by hand: with the branch
        // below in between, the compiler left them out where the last MFMA is the one that matters (one block of heads).
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) asm volatile("" : "+v"(sacc[hb]));
        asm volatile("s_nop 7\n\ts_nop 3" : "+v"(sacc[HB - 1]));
        if (valid < PAGE_TOKENS) {
          int ln = lane;
          asm volatile("" : "+v"(ln));
#pragma unroll
          for (int hb = 0; hb < HB; ++hb)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (16 * part + 4 * (ln >> 4) + i >= valid) sacc[hb][i] = -INFINITY;
        }
      };
      scores();

      // ---- online softmax ----
      // The first page of an item sets the reference m_run of the exponentials: its highest score.  It is moved only when a score
      // exceeds it by more than LAZY, since agreeing on a new one costs two barriers.  (A reference 24 above the highest score, to be
      // exceeded by as much, moves less often and is no faster: 64 x 32768 tokens of 32 heads with heavy channels 401 us either way.  The
      // exponents are then rounded at 24 instead of near 0, and the weights of 2^24 overflow sums of large latents.)
      auto agree = [&]() {
        int ln = lane;                             // as above
        asm volatile("" : "+v"(ln));
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) {
          float x = a.scale_log2 * fmaxf(fmaxf(sacc[hb][0], sacc[hb][1]), fmaxf(sacc[hb][2], sacc[hb][3]));
          x = fmaxf(x, lane_xor<16>(x, lane));
          x = fmaxf(x, lane_xor<32>(x, lane));
          if (ln < 16) cand[wave * 32 + hb * 16 + ln] = x;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) {
          float m_new = -INFINITY;
#pragma unroll
          for (int i = 0; i < PARTS; ++i) m_new = fmaxf(m_new, cand[(hg * PARTS + i) * 32 + hb * 16 + (ln & 15)]);
          m_new = fmaxf(m_run[hb], fmaxf(m_new, NO_SCORE));
          const float alpha = __builtin_amdgcn_exp2f(m_run[hb] - m_new);   // 0 on the first page
          l_run[hb] *= alpha;
          m_run[hb] = m_new;
#pragma unroll
          for (int d = 0; d < DB; ++d) acc[hb][d] *= alpha;
        }
      };
      if (i == p0) {
        agree();
      } else {
        bool move = false;
#pragma unroll
        for (int hb = 0; hb < HB; ++hb)
          move = move || a.scale_log2 * fmaxf(fmaxf(sacc[hb][0], sacc[hb][1]), fmaxf(sacc[hb][2], sacc[hb][3])) > m_run[hb] + LAZY;
        if (__any(move)) asm volatile("ds_write_b32 %0, %1" : : "v"(flag_at), "v"(n + 1) : "memory");
      }
      float psum[HB];
      auto weights = [&]() {
        static_for<HB>([&](auto ic) {
          constexpr int hb = decltype(ic)::value;
          bf16x4 p4;
          psum[hb] = 0.f;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float w = __builtin_amdgcn_exp2f(fmaf(sacc[hb][i], a.scale_log2, -m_run[hb]));
            psum[hb] += w;
            p4[i] = (bf16_t)w;
          }
          lds_write_b64<hb * 2048>(w_write, __builtin_bit_cast(u32x2, p4));
        });
      };
      weights();

      // ---- the first V fragments are requested under the barrier ----
      constexpr int NV = 2 * DB, VR = 4;           // fragments (32-token step s2, block d), in flight
      u32x2 vlo[VR], vhi[VR];
      const unsigned va = page + v_off;
      auto read_v = [&](auto ic) {
        constexpr int i = decltype(ic)::value, s2 = i / DB, d = i % DB;
        const unsigned at = va ^ (unsigned)(32 * d);
        lds_read_tr_b64<s2 * (32 * RC * 16)>(vlo[i & (VR - 1)], at);
        lds_read_tr_b64<s2 * (32 * RC * 16) + 16 * RC * 16>(vhi[i & (VR - 1)], at);
      };
      static_for<VR>(read_v);
      asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(2 * VR) : "memory");      // weights and flag are written
      __builtin_amdgcn_s_barrier();
      bf16x8 pb[HB];                               // weights of one 32-token step
      auto read_weights = [&](auto sc) {
        constexpr int s2 = decltype(sc)::value;
        static_for<HB>([&](auto ic) { lds_read_b128<decltype(ic)::value * 2048 + s2 * 1024>(pb[decltype(ic)::value], w_read); });
      };
      read_weights(std::integral_constant<int, 0>{});
      const bool raised = flag_raised(n);          // waits for everything requested before it
#pragma unroll
      for (int i = 0; i < VR; ++i) lds_wait<0>(vlo[i], vhi[i]);
#pragma unroll
      for (int hb = 0; hb < HB; ++hb) lds_wait<0>(pb[hb]);
      if (__builtin_expect(raised, 0)) {
        scores();                                  // again, like the V fragments below: kept, they would cost registers
        agree();
        weights();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        static_for<VR>(read_v);
        read_weights(std::integral_constant<int, 0>{});
#pragma unroll
        for (int i = 0; i < VR; ++i) lds_wait<0>(vlo[i], vhi[i]);
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) lds_wait<0>(pb[hb]);
      }
#pragma unroll
      for (int hb = 0; hb < HB; ++hb) l_run[hb] += psum[hb];

      // ---- output: O^T += V^T P^T over this wave's quarter of the dims ----
      static_for<NV>([&](auto ic) {
        constexpr int i = decltype(ic)::value, d = i % DB;
        // fragments requested after this one (the weights of the second step come between DB - 1 + VR and DB + VR)
        constexpr int ahead = (NV - 1 - i) < VR - 1 ? (NV - 1 - i) : VR - 1;
        if constexpr (i == DB) {
#pragma unroll
          for (int hb = 0; hb < HB; ++hb) lds_wait<(DB - 1 + VR < NV ? 2 : 0)>(pb[hb]);
        }
        lds_wait<2 * ahead>(vlo[i & (VR - 1)], vhi[i & (VR - 1)]);
        const u32x4 v4 = {vlo[i & (VR - 1)][0], vlo[i & (VR - 1)][1], vhi[i & (VR - 1)][0], vhi[i & (VR - 1)][1]};
#pragma unroll
        for (int hb = 0; hb < HB; ++hb)
          acc[hb][d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v4), pb[hb], acc[hb][d], 0, 0, 0);
        if constexpr (i == DB - 1) read_weights(std::integral_constant<int, 1>{});
        if constexpr (i + VR < NV) read_v(std::integral_constant<int, i + VR>{});
      });
    }

    // ---- the item's partial result; its sums over the parts are written after the next barrier ----
    const size_t item = slot * a.H + head0;
    int ln = lane;                       // computed anew for every item, as above
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) {
      float l = l_run[hb] + __shfl_xor(l_run[hb], 16);
      l += __shfl_xor(l, 32);
      if (ln < 16) {
        sums[wave * 32 + hb * 16 + (ln & 15)] = item_sum(m_run[hb], l);
        if (part == 0) refs[hg * 32 + hb * 16 + (ln & 15)] = item_reference(m_run[hb]);
      }
      float* pacc = a.part_acc + (item + hb * 16 + (ln & 15)) * DL + (DL / PARTS) * part + 4 * (ln >> 4);
#pragma unroll
      for (int d = 0; d < DB; ++d) *reinterpret_cast<f32x4*>(pacc + 16 * d) = acc[hb][d];
    }
    ml_pending = a.part_ml + item * 2;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  });
  TPLA_TL_MARK(2);
  __builtin_amdgcn_s_barrier();          // the sums of the last item
  write_pending();
}

// Waves per SIMD the register allocation must allow: with 128-wide slices three 4-wave workgroups (or one
// of 8 waves) share a compute unit, with 256-wide ones two; a 512-wide slice only
// fits one workgroup per compute unit in LDS, so it keeps the full budget.
constexpr int HPW_PAIR = 8;      // value of HPW that selects decode_item_shared: 16 heads per pair of waves
template <int DL, int NW, int HPW = 16>
constexpr int waves_per_simd() {
  if (HPW == HPW_PAIR) return 2 * NW >= 8 ? 2 : 1;
  return DL < 512 && NW >= 4 ? 2 : 1;
}
// Tiles in the LDS ring (one fewer in flight; two fewer in decode_item_shared) and fragment ring depth (LDS reads ahead of the
// MFMA that consumes them).  Measured: a ring of 4 tiles is no faster than 3 in decode_item (128-wide slices: 1144
// against 1122 us on the ragged batch), and fragment rings of 8 or 16 change nothing even where a wave
// has its SIMD to itself (576-wide rows: 248 / 251 / 261 us for 4 / 8 / 16).
template <int HPW>
constexpr int ring_stages() { return HPW == HPW_PAIR ? 4 : 3; }
constexpr int FRAG_RING = 4;

// Static chunks: workgroup = (slice, sequence, chunk s), pages [s*pps, (s+1)*pps).
template <int DL, int DR, int NW, int TOK, int NSTAGE, int KR, int HPW>
__global__ void __launch_bounds__(NW * 64 * (HPW == HPW_PAIR ? 2 : 1), (waves_per_simd<DL, NW, HPW>())) decode_mfma_kernel(DecodeArgs a) {
  extern __shared__ u32x4 smem[];        // NSTAGE tiles
  const int vb = blockIdx.x / a.n_splits, s = blockIdx.x % a.n_splits;   // vb = slice * B + sequence
  const int shard = vb / a.B, b = vb % a.B;
  const int L = seq_len_clipped(a, b);
  const int n_pages = (L + PAGE_TOKENS - 1) / PAGE_TOKENS;
  const int p0 = s * a.pages_per_split;
  if (p0 >= n_pages) return;
  const int p1 = min(p0 + a.pages_per_split, n_pages);
  if constexpr (HPW == HPW_PAIR)
    decode_item_shared<DL, DR, NW, TOK, NSTAGE, KR>(a, smem, shard, b, L, p0, p1, (size_t)vb * a.n_splits + s);
  else
    decode_item<DL, DR, NW, TOK, NSTAGE, KR>(a, smem, shard, b, L, p0, p1, (size_t)vb * a.n_splits + s);
}

// Inclusive prefix sum over the wave: row shifts of 1, 2, 4, 8 lanes, then the last lanes of the rows broadcast.
__device__ __forceinline__ int wave_prefix_sum(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);
  return x;
}
// One field of every cache line of the arguments, requested together at the kernel's start: they lie in host memory, and left to
// their first uses the lines are fetched one after the other.
__device__ __forceinline__ void fetch_arguments(const DecodeArgs& a) {
  asm volatile("" : : "s"(a.q_lat), "s"(a.pools[6]), "s"(a.part_ml), "s"(a.max_pages), "s"(a.scale_log2));
}
// v mod B of a pair: fewer instructions (which are fetched anew by every launch) than a division.
__device__ __forceinline__ int sequence_of(const DecodeArgs& a, int v) {
#pragma clang loop unroll(disable)
  for (int i = 1; i < a.n_shards; ++i) v -= v >= a.B ? a.B : 0;
  return v;
}
// The plan as every wave of a launch derives it from the lengths (no LDS, no barrier).  Lengths and prefix sums of the first
// 64 pairs stay in a register each; batches with more take a second pass over the rest.
struct BalancedRange {
  int w;                         // number of this workgroup's range
  int total, n_equal;            // pages of all pairs; number of equal ranges, or 0 for the plan's own (plan_fit)
  int start, end;                // this workgroup's range
  int L_first, incl_first;       // pair `lane`: its length, pages up to its end
};
__device__ __forceinline__ BalancedRange balanced_range(const DecodeArgs& a, int w, int lane) {
  BalancedRange r;
  const int n_v = a.n_shards * a.B;
  r.L_first = lane < n_v ? seq_len_clipped(a, sequence_of(a, lane)) : 0;
  r.incl_first = wave_prefix_sum((r.L_first + PAGE_TOKENS - 1) / PAGE_TOKENS);
  r.total = __builtin_amdgcn_readlane(r.incl_first, 63);
  for (int v0 = 64; v0 < n_v; v0 += 64) {
    const int v = v0 + lane;
    const int L = v < n_v ? seq_len_clipped(a, sequence_of(a, v)) : 0;
    r.total += __builtin_amdgcn_readlane(wave_prefix_sum((L + PAGE_TOKENS - 1) / PAGE_TOKENS), 63);
  }
  // workgroups beyond the ranges of the fitted plan have no pages (and still write their share of the plan table)
  r.n_equal = plan_fit(a.geom, r.total);
  w = range_of_workgroup(r.n_equal, r.total, w, a.n_shards, a.B, a.H, a.dl);
  r.w = w;
  if (r.n_equal > 0)
    equal_range(r.n_equal, r.total, w, &r.start, &r.end);
  else
    plan_range(a.geom, r.total, w, &r.start, &r.end);
  r.start = __builtin_amdgcn_readfirstlane(r.start);
  r.end = __builtin_amdgcn_readfirstlane(r.end);
  return r;
}
// The items of a range: f(slice, sequence, its tokens, first page, end page, slot, w), all scalar.  The wave finds the pair that
// holds the range's first page by the prefix sums; the pairs after it follow one by one with scalar loads of their lengths, so
// that nothing per lane stays alive over the items.
template <typename F>
__device__ __forceinline__ void balanced_items(const DecodeArgs& a, const BalancedRange& r, int w, int lane, F&& f) {
  if (r.start >= r.end) return;
  const int n_v = a.n_shards * a.B;
  int v = 0, e = 0, L = 0;                       // the pair, its first page in the laid-out order, its length
  int Ll = r.L_first, incl = r.incl_first;
  for (int v0 = 0;;) {
    const unsigned long long past = __ballot(incl > r.start);
    if (past) {
      const int src = __builtin_ctzll(past);
      v = v0 + src;
      L = __builtin_amdgcn_readlane(Ll, src);
      e = __builtin_amdgcn_readlane(incl, src) - (L + PAGE_TOKENS - 1) / PAGE_TOKENS;
      break;
    }
    v0 += 64;
    if (v0 >= n_v) return;                       // not reached: start < total
    const int base = __builtin_amdgcn_readlane(incl, 63);
    Ll = v0 + lane < n_v ? seq_len_clipped(a, sequence_of(a, v0 + lane)) : 0;
    incl = base + wave_prefix_sum((Ll + PAGE_TOKENS - 1) / PAGE_TOKENS);
  }
  const __attribute__((address_space(4))) int32_t* lens = (const __attribute__((address_space(4))) int32_t*)(uintptr_t)a.seq_lens;
  int shard = 0, b = v;
  for (; b >= a.B; b -= a.B) ++shard;
  for (;;) {
    const int pg = (L + PAGE_TOKENS - 1) / PAGE_TOKENS;
    int p0, p1;
    if (balanced_item(r.start, r.end, e, pg, &p0, &p1)) f(shard, b, L, p0, p1, (size_t)w + shard * a.B + b, w);
    e += pg;
    if (e >= r.end) return;
    if (++b == a.B) {
      b = 0;
      ++shard;
    }
    L = clip_length(a, lens[b]);
  }
}
// Static chunks as items, the order of a chunk's pages by its number.  A workgroup each, or, with fewer workgroups than
// chunks, the chunks that exist laid end to end and cut into equal shares, all of a workgroup's through one ring of pages (static_launch).
template <typename F>
__device__ __forceinline__ void chunk_items(const DecodeArgs& a, int lane, F&& f) {
  const int n_v = a.n_shards * a.B, S = a.n_splits, pps = a.pages_per_split;
  auto pages = [](int L) { return (L + PAGE_TOKENS - 1) / PAGE_TOKENS; };
  auto chunks = [&](int L) { return (pages(L) + pps - 1) / pps; };
  auto length = [&](int v) { return v < n_v ? seq_len_clipped(a, sequence_of(a, v)) : 0; };
  const __attribute__((address_space(4))) int32_t* lens = (const __attribute__((address_space(4))) int32_t*)(uintptr_t)a.seq_lens;
  int v, c, left;                                // the pair, the next of its chunks, chunks still to do
  if ((int)gridDim.x == n_v * S) {
    v = blockIdx.x / S;
    c = blockIdx.x - v * S;
    left = 1;
  } else {
    int total = 0;
    for (int v0 = 0; v0 < n_v; v0 += 64) total += __builtin_amdgcn_readlane(wave_prefix_sum(chunks(length(v0 + lane))), 63);
    const int start = (int)((long long)blockIdx.x * total / gridDim.x);
    left = (int)((long long)(blockIdx.x + 1) * total / gridDim.x) - start;
    if (left == 0) return;
    int base = 0;
    for (int v0 = 0;; v0 += 64) {                // ends: start < total
      const int n = chunks(length(v0 + lane)), incl = base + wave_prefix_sum(n);
      const unsigned long long past = __ballot(incl > start);
      if (past) {
        const int src = __builtin_ctzll(past);
        v = v0 + src;
        c = start - (__builtin_amdgcn_readlane(incl, src) - __builtin_amdgcn_readlane(n, src));
        break;
      }
      base = __builtin_amdgcn_readlane(incl, 63);
    }
  }
  int shard = 0, b = v;
  for (; b >= a.B; b -= a.B) ++shard;
  for (;;) {
    const int L = clip_length(a, lens[b]);
    const int pg = pages(L);
    for (; c * pps < pg && left > 0; ++c, --left) f(shard, b, L, c * pps, min((c + 1) * pps, pg), (size_t)v * S + c, b * S + c);
    if (left == 0 || (int)gridDim.x == n_v * S) return;
    c = 0;
    ++v;
    if (++b == a.B) {
      b = 0;
      ++shard;
    }
  }
}
// What the merge needs of the plan, once per launch instead of once per lane of the merge kernel: for
// every (slice, sequence) the range that owns its first page and the number of ranges up to the owner
// of its last.  Dealt over the workgroups (pair v to workgroup v mod W, one lane of its first wave) and
// done after the workgroup's own range: inside the scan above it cost the ragged batch 7 % (the owner
// search then lives in the loop that holds the items' registers).
__device__ __forceinline__ void write_plan_table(const DecodeArgs& a, const BalancedRange& r, int w, int lane) {
  const int n_v = a.n_shards * a.B;
  int base = 0;
  for (int v0 = 0; v0 < n_v; v0 += 64) {
    const int v = v0 + lane;
    const int L = v0 == 0 ? r.L_first : ((v < n_v) ? seq_len_clipped(a, sequence_of(a, v)) : 0);
    const int pg = (L + PAGE_TOKENS - 1) / PAGE_TOKENS;
    const int incl = v0 == 0 ? r.incl_first : wave_prefix_sum(pg);
    const int excl = base + incl - pg;
    if (v < n_v && v % a.n_wg == w) {
      int w0 = 0, cnt = 0;
      if (pg > 0) {
        const int last = excl + pg - 1;
        w0 = r.n_equal > 0 ? equal_owner(r.n_equal, excl, r.total) : balanced_owner(a.geom, excl, r.total);
        cnt = (r.n_equal > 0 ? equal_owner(r.n_equal, last, r.total) : balanced_owner(a.geom, last, r.total)) - w0 + 1;
      }
      a.plan[v] = w0;
      a.plan[n_v + v] = cnt;
    }
    base += __builtin_amdgcn_readlane(incl, 63);
  }
}

__device__ __forceinline__ void timeline_start() {
#ifdef TPLA_WG_TIMELINE
  if (threadIdx.x == 0 && blockIdx.y == 0 && blockIdx.x < 4096) {
    g_wg_times[blockIdx.x * 4] = wall_clock64();
    g_wg_times[blockIdx.x * 4 + 1] = 0;
    g_wg_where[blockIdx.x * 2] = __builtin_amdgcn_s_getreg((31 << 11) | 20);      // XCC_ID
    g_wg_where[blockIdx.x * 2 + 1] = __builtin_amdgcn_s_getreg((31 << 11) | 4);   // HW_ID
  }
#endif
}
// Balanced ranges: the pages of all (slice, sequence) pairs are laid end to
// end (T pages) and a workgroup takes one of the W ranges of the plan (equal shares, which of them
// by range_of_workgroup, or shares weighted by placement round, workgroup w range w: see BalancedPlan), whatever
// sequences that covers; every (workgroup, sequence) overlap is one work item
// whose partial result goes to slot w + v (w: the range; v = slice * B + sequence; strictly
// increasing along the items, hence unique).
template <int DL, int DR, int NW, int TOK, int NSTAGE, int KR, int HPW>
__global__ void __launch_bounds__(NW * 64 * (HPW == HPW_PAIR ? 2 : 1), (waves_per_simd<DL, NW, HPW>())) decode_mfma_balanced_kernel(DecodeArgs a) {
  extern __shared__ u32x4 smem[];
  timeline_start();
  const int lane = threadIdx.x & 63;
  const BalancedRange r = balanced_range(a, blockIdx.x, lane);
  const int w = r.w;
  balanced_items(a, r, w, lane, [&](int shard, int b, int L, int p0, int p1, size_t slot, int) {
    if constexpr (HPW == HPW_PAIR)
      decode_item_shared<DL, DR, NW, TOK, NSTAGE, KR>(a, smem, shard, b, L, p0, p1, slot);
    else
      decode_item<DL, DR, NW, TOK, NSTAGE, KR>(a, smem, shard, b, L, p0, p1, slot);
  });
  if (threadIdx.x < 64 && blockIdx.y == 0 && w < a.n_shards * a.B) write_plan_table(a, r, w, lane);
#ifdef TPLA_WG_TIMELINE
  __syncthreads();
  TPLA_TL_MARK(3);
#endif
}

// The same two launches for rows of up to 320 elements: decode_pages.
template <int DL, int HG, int HB, bool ONE_ROW>
struct PageKernel {
  // NP: waves that request pages (four are no faster); NSTAGE: pages in the ring
  static constexpr int NP = 2, NSTAGE = 3;
  static constexpr int waves = HG * PARTS + NP, per_simd = (waves + 3) / 4;
  using Lds = PageLds<DL, 64, HG, HB, NSTAGE>;
};
template <int DL, int HG, int HB, bool ONE_ROW>
__global__ void __launch_bounds__((PageKernel<DL, HG, HB, ONE_ROW>::waves * 64), (PageKernel<DL, HG, HB, ONE_ROW>::per_simd)) decode_mfma_pages_kernel(DecodeArgs a) {
  extern __shared__ u32x4 smem[];
  using K = PageKernel<DL, HG, HB, ONE_ROW>;
  fetch_arguments(a);
  const int lane = threadIdx.x & 63;
  const auto items = [&](auto&& f) { chunk_items(a, lane, f); };
  if (!ONE_ROW && a.pages_per_split >= KEEP_PAGES)
    decode_pages<DL, 64, HG, HB, K::NP, K::NSTAGE, !ONE_ROW>(a, smem, items);
  else
    decode_pages<DL, 64, HG, HB, K::NP, K::NSTAGE, false>(a, smem, items);
}
template <int DL, int HG, int HB, bool ONE_ROW>
__global__ void __launch_bounds__((PageKernel<DL, HG, HB, ONE_ROW>::waves * 64), (PageKernel<DL, HG, HB, ONE_ROW>::per_simd)) decode_mfma_pages_balanced_kernel(DecodeArgs a) {
  extern __shared__ u32x4 smem[];
  using K = PageKernel<DL, HG, HB, ONE_ROW>;
  fetch_arguments(a);
  timeline_start();
  const int lane = threadIdx.x & 63;
  const BalancedRange r = balanced_range(a, blockIdx.x, lane);
  const int w = r.w;
  const auto items = [&](auto&& f) { balanced_items(a, r, w, lane, f); };
  if (!ONE_ROW && r.end - r.start >= KEEP_PAGES)
    decode_pages<DL, 64, HG, HB, K::NP, K::NSTAGE, !ONE_ROW>(a, smem, items);
  else
    decode_pages<DL, 64, HG, HB, K::NP, K::NSTAGE, false>(a, smem, items);
  if (threadIdx.x < 64 && blockIdx.y == 0 && w < a.n_shards * a.B) write_plan_table(a, r, w, lane);
#ifdef TPLA_WG_TIMELINE
  __syncthreads();
  TPLA_TL_MARK(3);
#endif
}

bool decode_mfma_supported(const tpla_shape_t& sh) {
  if (sh.dtype != TPLA_BF16 || sh.page_tokens != PAGE_TOKENS || sh.d_r != 64) return false;
  const int dl = sh.d_c / sh.g;
  if (dl != 128 && dl != 256 && dl != 512) return false;
  return sh.H == 16 || sh.H == 32 || sh.H == 64 || sh.H == 128;
}

// Kernel entry, its LDS size and how many of its workgroups fit on one
// compute unit (0 when the runtime cannot tell, e.g. without a device).
struct KernelInfo {
  void (*fn)(DecodeArgs) = nullptr;
  void (*fn_balanced)(DecodeArgs) = nullptr;
  size_t smem = 0;
  int threads = 0;
  int heads = 0;           // of a workgroup: the grid has H / heads rows
  int blocks_per_cu = 0;
  bool ready = false;
};

static void finish_kernel_info(KernelInfo& info) {
  info.ready = allow_lds(reinterpret_cast<const void*>(info.fn), info.smem, "decode_mfma_kernel") == TPLA_OK &&
               (!info.fn_balanced || allow_lds(reinterpret_cast<const void*>(info.fn_balanced), info.smem, "decode_mfma_balanced_kernel") == TPLA_OK);
  if (!info.ready || !info.fn_balanced) return;
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void*>(info.fn_balanced), info.threads,
                                                   info.smem) != hipSuccess) {
    (void)hipGetLastError();
    n = 0;
  }
  info.blocks_per_cu = n;
}

// BALANCED: whether automatic plans run it too.
template <int DL, int NW, int HPW, bool BALANCED>
static KernelInfo make_kernel_info() {
  constexpr int TOK = 32, KR = FRAG_RING, NSTAGE = ring_stages<HPW>();
  KernelInfo info;
  info.fn = decode_mfma_kernel<DL, 64, NW, TOK, NSTAGE, KR, HPW>;
  if constexpr (BALANCED) info.fn_balanced = decode_mfma_balanced_kernel<DL, 64, NW, TOK, NSTAGE, KR, HPW>;
  info.smem = (size_t)NSTAGE * TOK * ((DL + 64) / 8) * 16;
  info.threads = NW * 64;
  if (HPW == HPW_PAIR) {
    info.smem += (size_t)2 * (2 * NW) * 64 * 16;     // the two hand-over buffers
    info.threads *= 2;
  }
  info.heads = NW * 16;
  finish_kernel_info(info);
  return info;
}

template <int DL, int NW, int HPW = 16, bool BALANCED = true>
static int kernel_info(KernelInfo** out) {
  static KernelInfo info = make_kernel_info<DL, NW, HPW, BALANCED>();   // initialised once, thread-safe
  if (!info.ready) return fail(TPLA_ERR_HIP, "cannot raise the dynamic LDS limit to %zu", info.smem);
  *out = &info;
  return TPLA_OK;
}

template <int DL, int HG, int HB, bool ONE_ROW>
static KernelInfo make_page_kernel_info() {
  using K = PageKernel<DL, HG, HB, ONE_ROW>;
  KernelInfo info;
  info.fn = decode_mfma_pages_kernel<DL, HG, HB, ONE_ROW>;
  info.fn_balanced = decode_mfma_pages_balanced_kernel<DL, HG, HB, ONE_ROW>;
  info.smem = K::Lds::bytes;
  info.threads = K::waves * 64;
  info.heads = HG * HB * 16;
  finish_kernel_info(info);
  return info;
}

template <int DL, int HG, int HB, bool ONE_ROW = true>
static int page_kernel_info(KernelInfo** out) {
  static KernelInfo info = make_page_kernel_info<DL, HG, HB, ONE_ROW>();
  if (!info.ready) return fail(TPLA_ERR_HIP, "cannot raise the dynamic LDS limit to %zu", info.smem);
  *out = &info;
  return TPLA_OK;
}

// 128 heads run as two rows of workgroups of 64.
template <int DL>
static int kernel_info_dl(int H, KernelInfo** out) {
  if (H != 16 && H != 32 && H != 64 && H != 128) return fail(TPLA_ERR_UNSUPPORTED, "H=%d", H);
  if constexpr (DL == 128) {
    return H == 16 ? kernel_info<DL, 1>(out) : H == 32 ? kernel_info<DL, 2>(out) : H == 64 ? kernel_info<DL, 4>(out) : kernel_info<DL, 8>(out);
  } else if constexpr (DL == 256) {
    return H == 16 ? page_kernel_info<DL, 1, 1>(out) : H == 32 ? page_kernel_info<DL, 1, 2>(out)
                   : H == 64 ? page_kernel_info<DL, 2, 2>(out) : page_kernel_info<DL, 2, 2, false>(out);
  } else {
    if (H == 16) return kernel_info<DL, 1>(out);
    return H == 32 ? kernel_info<DL, 2, HPW_PAIR>(out) : kernel_info<DL, 4, HPW_PAIR>(out);
  }
}

static int kernel_info_for(int dl, int H, KernelInfo** out) {
  switch (dl) {
    case 128: return kernel_info_dl<128>(H, out);
    case 256: return kernel_info_dl<256>(H, out);
    case 512: return kernel_info_dl<512>(H, out);
  }
  return fail(TPLA_ERR_UNSUPPORTED, "d_c/g=%d", dl);
}

// Kernel and workgroups per row of a launch of `chunks` static chunks of `pps` pages.  The kernels of 256-wide slices hold a compute unit by
// themselves: up to one chunk each they are the faster ones, beyond that the start of a workgroup (lengths, page id, queries,
// first page) has nothing beside it and the rest of the last round waits.  From four rounds on they deal the chunks over one round of workgroups (chunk_items);
// between, two or more workgroups of 16 heads per wave share a compute unit.  Kernel, one workgroup per chunk / dealt / 16 heads per wave, us:
//   64 heads: 256 chunks of 64 pages 111 / - / 131, 260 of 16 54.2 / 56.4 / 46.5, 512 of 8 43.7 / 43.5 / 40.5, 512 of 32 130 / 125 / 118,
//     1024 of 4 57.4 / 49.8 / 51.2, 4096 of one 124 / 88 / 97, 2048 of 8 151 / 149 / 144
//   32 heads: 512 of 16 62.9 / 62.9 / 58.2, 1024 of 8 71.5 / 69.0 / 68.9, 4096 of two 102 / 86 / 97, ragged 1024 of up to 20 84 / 56 / 91
//   16 heads: 512 of 16 58.9 / 58.3 / 56.1, 1024 of 8 65.4 / 64.8 / 63.6, 8192 of one 135 / 86 / 107, ragged 1024 of up to 40 139 / 85 / 175
//   128 heads (half as many at once): 256 of 16 70.9 / 56.5 / 52.3, 256 of 64 250 / 189 / 174, 4096 of one 250 / 166 / 206
// (The second kernel takes two rounds from 513 chunks on, which a third of the first beats for few heads: 600 of 16 pages, one workgroup per chunk / 16 heads
// per wave: 16 heads 74.4 / 91.2, 32 80.8 / 93.0, 64 89.1 / 90.2; of 4 pages 27.6 / 31.0, 31.0 / 33.9, 39.7 / 36.2; 800 of 16 99.7 / 96.3,
// 108.7 / 100.3, 120 / 111.)
// 512-wide slices and 128 heads, two rows of workgroups / all heads in one, whose pages are read once and whose start counts less:
//   128 chunks of 4 28.2 / 46.3, 192 of 8 66.6 / 76.1, 512 of 2 84.5 / 70.2, 512 of 4 104.9 / 99.5, 1024 of 4 204.1 / 204.2, 512 of 8 149 / 158,
//   4096 of one 502 / 371
static int static_launch(int dl, int H, int chunks, int pps, KernelInfo** k, unsigned* workgroups) {
  const int rc = kernel_info_for(dl, H, k);
  if (rc) return rc;
  *workgroups = (unsigned)chunks;
  const int at_once = std::max(1, device_cu_count() * (*k)->heads / H);
  if (chunks <= at_once) return TPLA_OK;
  if (dl == 512 && H == 128 && pps <= 4) return kernel_info<512, 8, 16, false>(k);
  if (dl != 256) return TPLA_OK;
  if (chunks / 4 >= at_once) {
    *workgroups = (unsigned)at_once;
    return TPLA_OK;
  }
  if (H <= 32 && chunks > 2 * at_once && chunks <= 3 * at_once) return TPLA_OK;
  return H == 16 ? kernel_info<256, 1, 16, false>(k) : H == 32 ? kernel_info<256, 2, 16, false>(k)
         : H == 64 ? kernel_info<256, 4, 16, false>(k) : kernel_info<256, 8, 16, false>(k);
}

int decode_mfma_head_rows(const tpla_shape_t& sh) {
  KernelInfo* k = nullptr;
  if (kernel_info_for(sh.d_c / sh.g, sh.H, &k) != TPLA_OK) return 1;
  return sh.H / k->heads;
}

int decode_mfma_blocks_per_cu(const tpla_shape_t& sh) {
  KernelInfo* k = nullptr;
  if (kernel_info_for(sh.d_c / sh.g, sh.H, &k) != TPLA_OK) return 0;
  return k->blocks_per_cu;
}

// Measured with per-workgroup timestamps on full launches of equal ranges: when two or three workgroups
// (of decode_item) share a compute unit and their waves share its SIMDs, the workgroup placed first takes 5 - 9 % less
// time than the average and the one placed last 5 % (two per compute unit) or 10 % (three) more,
// whatever the wave priorities (s_setprio changes nothing).  With two per compute unit the late
// workgroups still keep the memory system full when they are alone at the end, and sizing the ranges by
// round made the launch slower (227 against 222 us at 32 x 32768 tokens); with three (128-wide slices:
// 12 KB tiles, 24 KB in flight per workgroup) the lone last round does not, and weighted ranges take
// the ragged batch from 1122 to 1073 us with 140 : 129 : 115.  With the XCC weights below in place the
// best round weights are further apart (one box, same units: 140:129:115 1047 us, 143:130:112 1035,
// 146:130:109 1026, 149:131:106 1022, 152:131:103 1034, 155:132:100 1040, 160:132:95 1055 us; on
// another box 1072 -> 1051 us for 149:131:106 against 140:129:115).  With one wave per SIMD (32 heads
// and fewer) the rounds run alike.  Weights in units of 1/128 of the average range.
//
// The XCCs differ too, the same way on every box measured: workgroups on the odd-numbered ones take
// up to 9 % longer over equal ranges than those on the even-numbered ones (32 heads, 128-wide slices).  Workgroups are dealt
// to the XCCs in turn, so the odd positions of a round get shorter ranges.  Measured with the weight of the odd positions at 128 (equal),
// 123, 118, 115, 113 / 128, in us:
//   256-wide, 16 heads: 64 ragged sequences 225.3, 224.5, 224.5, 222.7, 221.0; 32 x 32768 in order 199.6, 200.4, 200.6, 200.7, 201.6, scattered
//     205.7, 206.6, 205.5, 204.5, 203.6;  32 heads: 233.5, 232.6, 230.1, 230.2, 228.7; 203.5, 204.1, 205.0, 204.9, 206.1; 209.4, 210.7, 208.1, 207.7, 206.2
//   256-wide, 64 heads: 203.3, 204.3, 206.5, -, 208.2 (kernel); 128 heads 182.6, 183.2, 185.2, -, 185.8
//   512-wide, 32 x 32768 scattered: 16 heads 298.7, 303.3, 308.4, 312.8, 313.1; 32 heads 193.3, 193.2, 192.9, 194.4, 194.2; 64 heads 225.6, 223.7, 223.7,
//     226.2, 225.7;  32 ragged sequences: 173.4, 174.1, 178.4, 180.9, 181.7; 120.8, 120.4, 119.6, 119.5, 119.9; 137.2, 137.6, 138.5, 139.5, 140.3
//   128-wide, ragged batch: 1072, 1061, 1051, -, 1047 (other box: 113 1043, 108 1057, 103 1069)
void decode_mfma_round_weights(const tpla_shape_t& sh, int per_cu, int32_t wt[4], int32_t wx[2]) {
  for (int r = 0; r < 4; ++r) wt[r] = 128;
  const int dl = sh.d_c / sh.g;
  wx[0] = wx[1] = 128;
#ifdef TPLA_EQUAL_RANGES      // measurement build: the plan without any weights, for the timeline comparison
  (void)dl;
  (void)per_cu;
  return;
#endif
  wx[1] = dl == 128 ? 113 : dl == 512 ? (sh.H == 16 ? 128 : sh.H == 32 ? 115 : sh.H == 64 ? 123 : 128) : sh.H <= 32 ? 115 : 128;
  const int heads_per_wave = 16;
  const int waves_per_simd_launched = (sh.H / heads_per_wave) * per_cu / 4;
  if (waves_per_simd_launched < 2) return;
  if (per_cu == 3) {
    wt[0] = 149;
    wt[1] = 131;
    wt[2] = 106;
  }
}

// Split kernel by workgroups per compute unit (one / two / three), ragged batches, by pages per compute unit:
//   64 heads, 128-wide (32 KB of partial result per range): 4.3 pages 19.2 / - / 20.9 us, 8.5 25.6 / 23.4 / 25.1, 17 37.1 / - / 33.0
//   less (16 KB): 1.6 pages 17.0 / 15.0, 2.1 18.8 / 17.8, 6.4 30.2 / 24.1 (one / as many as fit)
// Everywhere else (256- and 512-wide slices; 128 heads) one workgroup per compute unit is all that fits and the lines do not matter.
void decode_mfma_range_pages(const tpla_shape_t& sh, int32_t* second, int32_t* all) {
  const int partial = sh.H * (sh.d_c / sh.g) * 4, cus = device_cu_count();
  *second = (partial >= 32 * 1024 ? 5 : 1) * cus;
  *all = (partial >= 32 * 1024 ? 13 : 1) * cus;
}

#ifdef TPLA_WG_TIMELINE
// Device addresses of the timeline arrays ([4096][4] uint64 ticks of 10 ns, [4096][2] uint32).
extern "C" __attribute__((visibility("default"))) int tpla_debug_wg_timeline(void** times, void** where) {
  if (hipGetSymbolAddress(times, HIP_SYMBOL(g_wg_times)) != hipSuccess) return TPLA_ERR_HIP;
  if (hipGetSymbolAddress(where, HIP_SYMBOL(g_wg_where)) != hipSuccess) return TPLA_ERR_HIP;
  return TPLA_OK;
}
#endif

int launch_decode_mfma(const DecodeArgs& a, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  KernelInfo* k = nullptr;
  unsigned workgroups = (unsigned)a.n_wg;
  int rc = a.balanced ? kernel_info_for(a.dl, a.H, &k)
                      : static_launch(a.dl, a.H, a.n_shards * a.B * a.n_splits, a.pages_per_split, &k, &workgroups);
  if (rc) return rc;
  const dim3 grid(workgroups, (unsigned)(a.H / k->heads));
  void (*fn)(DecodeArgs) = a.balanced ? k->fn_balanced : k->fn;
  rc = allow_lds(reinterpret_cast<const void*>(fn), k->smem, "decode_mfma_kernel");   // kernel_info asked on its first device only
  if (rc) return rc;
  if (ev_start && ev_stop)
    // the events take the kernel's own begin and end times (no marker packets around it)
    hipExtLaunchKernelGGL(fn, grid, dim3(k->threads), (uint32_t)k->smem, st, ev_start, ev_stop, 0, a);
  else
    hipLaunchKernelGGL(fn, grid, dim3(k->threads), k->smem, st, a);
  return check_launch("decode_mfma_kernel");
}

}  // namespace tpla
