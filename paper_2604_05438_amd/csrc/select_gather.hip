// Fused Top-K select + gather of the filtered pipeline (bf16 caches, and fp32 ones of short contexts at d = 64, on the matrix cores):
// topk_select, exact_branch and residual_correct for the retrieved tokens in one launch.
// grid (split, Hq, n_problems), NTHR = 1024 or 512 threads: `split` workgroups share a query head.
//
// The score pass left, per query head, every token whose score key reaches the head's lower bound, in
// per-wavefront lists (score_tile.h): the first cand_T entries of a list in a compact array, the rest in
// the list's full-capacity region.  If at least K candidates exist, the K best mid tokens
// (Sec. "Models, tasks, and protocol": exhaustive Top-K, ties to the lower index) are all among them.
//
// Every workgroup of a head first finds the same selection threshold, on its own (the candidates of a
// head are ~100 KB and the search is a few thousand instructions: cheaper than a launch boundary):
//   * the candidates are visited in "sweeps" in which a thread owns kSweepEntries consecutive entries of
//     one list; the first sweep's addresses depend on the launch geometry only and are loaded together
//     with the problem record, so the common case is one memory round trip
//   * histogram of a fine monotone binning of the score keys -> boundary bin b* (tokens in higher bins
//     are retrieved); the candidates in b* are ranked by counting (or, beyond kBCap of them, by radix
//     passes over the sweeps) -> the K-th best composite (score key, lower index first), `thr`
//   * fewer than K candidates (the sampled bound was too high: a ~1e-6 event per head by design), or a list that was not made for
//     want of a bound (kNoList); tkphi_tuning::select_test = 1 forces both: the workgroup first rescans its head's
//     keys with no bound, which makes every mid token a candidate
// Short contexts (Geom::direct) come without a bound and without lists: the score pass stored a row of scores per head, which
// is loaded whole and packed as it is.
// Then workgroup `part` takes an equal share of the packed candidates (of the lists, where they are too many to pack): its
// winners (composite >= thr) go to the head's retrieved list, in order, behind those of the shares before
// it, and are gathered 256 or 512 at a time (16-token tiles, one or two per wavefront):
//     m_loc = max s_i,  Z_loc = sum exp(s_i - m_loc),  nu_loc = sum exp(s_i - m_loc) v_i     (eq. (exact_terms))
//     zsum = sum z_i,  zv = sum z_i v_i,  z_i = phi_q . phi_k(k_i) recomputed                (eq. (subtraction))
// into one partial per workgroup, [m, Z, zsum, count, nu[d], zv[d]], which the merge kernel combines in
// part order.  No atomics on global memory; every sum runs in a fixed order.
#include <algorithm>

#include "gather_tile.h"
#include "merge_head.h"
#include "mlp_pack.h"
#include "mlp_query.h"
#include "score_tile.h"
#include "select_utils.h"
#include "tkphi_internal.h"

namespace tkphi {

constexpr int kBCap = 1024;            // boundary-bin candidates ranked in LDS
constexpr int kSweepLoads = kSweepEntries / 2;
constexpr int kLocalTiles = 6;         // anchor tiles of a head that its only workgroup merges out of LDS
// winners gathered per round: 16-token tile t of a round goes to wavefront t mod 16.  Two tiles per wavefront at
// d = 64 (one round for most heads of a batch of short sequences); at d = 128 the second tile's rows do not fit
// the registers
template <int D, int NTHR, typename KV> constexpr int kBatchOf = (D * sizeof(KV) == 128 && NTHR == 1024) ? 512 : 256;
// winners of a workgroup kept in LDS (the rest are re-read from the retrieved list)
template <int NTHR> constexpr int kWinLdsOf = NTHR == 1024 ? 1536 : 1024;

// every mid token of query head gq becomes a candidate: list k of the rescan set takes the tokens [k cap, (k + 1) cap), cap =
// scan_chunk / 4, a multiple of 16 (what the score pass wrote stays as it is: other workgroups of the head may still be reading
// it).  The wavefronts take the tiles of 16 tokens in turn, however long the lists are: a short sequence under large bounds has few
// lists, and a wavefront to each was a chain of up to 64 round trips beside idle ones (step of a 3B layer of 1090 tokens under bounds
// of 128K, all heads rescanning: 104 -> 58 us; of 131072 tokens 1215 -> 1133, a 1B layer 687 -> 697).  One tile in flight per wavefront: the
// rare path must not cost the common one registers.
template <int D, int NTHR>
__device__ __forceinline__ void rescan_head(const Geom& g, const tkphi_problem& pr, char* blk, int gq, int n, int n_reg) {
  const int h = gq / g.G, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63, r = lane & 15, kg = lane >> 4;
  const int cap = g.scan_chunk / 4, T = g.cand_T;
  const size_t reg0 = (size_t)gq * g.n_scan_chunks * 4;
  ScoreFrag bq[kTileFrags<D>];
  load_query_frags<D>(g, pr, h, bq);
  const char* Kl = (const char*)pr.K + ((size_t)h * pr.stride_head + (size_t)g.n_sink * pr.stride_tok) * 2 + score_lane_offset<false>();
  for (int t0 = wv * 16; t0 < n; t0 += NTHR / 4) {
    const int reg = t0 / cap;
    const glb_u32x2 list = (glb_u32x2)(blk + g.off_resf) + (reg0 + reg) * (size_t)cap;
    const glb_u32x2 head = (glb_u32x2)(blk + g.off_resc) + (reg0 + reg) * (size_t)T;
    ScoreFrag a[kTileFrags<D>];
    request_tile<D, false>(a, [&](int i) { return Kl + (uint64_t)(uint32_t)min(t0 + i, n - 1) * (uint64_t)(pr.stride_tok * 2); });
    const st_floatx4 acc = score_tile<D, false>(a, bq);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int tok = t0 + 4 * kg + i, at = tok - reg * cap;
      const st_u32x2 e = (st_u32x2){__float_as_uint(fmaf(acc[i], g.score_scale, 0.0f)), (uint32_t)tok};
      if (r == gq % g.G && tok < n) {
        if (at < T) head[at] = e;
        else list[at] = e;
      }
    }
  }
  for (int reg = threadIdx.x; reg < n_reg; reg += NTHR)
    ((uint32_t*)(blk + g.off_rescount))[reg0 + reg] = (uint32_t)max(0, min(cap, n - reg * cap));
}

// The selecting and gathering work of workgroup (part, gq, p); returns early where there is nothing to retrieve
// DIRECT: Geom::direct (a row of scores per head instead of candidate lists).  LIST: Geom::list (ends with the retrieved list of the head,
// whose only workgroup this is).  KV: storage type of keys, values and Wk (fp32 only with DIRECT, d = 64)
// True: the head is merged and its output written (a head's only workgroup, see below)
template <int D, int NTHR, bool DIRECT, bool LIST, bool LOCAL, typename KV>
__device__ __forceinline__ bool select_gather_body(const Geom& g, const tkphi_problem* __restrict__ probs, char* __restrict__ ws,
                                                   int part, int gq, int p, int mode) {
  constexpr int EPL = Elem<KV>::per16, KS = D * (int)sizeof(KV) / 64;        // elements of 16 bytes; 16-byte pieces of a key row per lane
  constexpr int WROW = wk_row_bytes(D, sizeof(KV));
  // select phase: histogram (8 KB) + boundary candidates (8 KB); gather phase: reduction scratch of the value sums
  __shared__ __attribute__((aligned(16))) char lds_a[16384];
  __shared__ __attribute__((aligned(16))) char wk_lds[D * WROW];
  constexpr int kDense = packed_candidates(D, NTHR), kWinLds = kWinLdsOf<NTHR>, NWV = NTHR / 64;
  __shared__ __attribute__((aligned(16))) uint2 dense[kDense];   // the candidates of the head, packed (select phase)
  float* sh_parts = (float*)dense;                  // then [kLocalTiles + 1][2 D + 4], the partials of a head that is merged here
  __shared__ int w_tok[kWinLds];
  __shared__ float w_s[kWinLds];
  constexpr int kBatch = kBatchOf<D, NTHR, KV>;
  __shared__ float b_w[2][kBatch], b_z[2][kBatch], sh_wave[3][NWV];    // (maxima, shares of Z_loc and of zsum)
  __shared__ float sh_bk[D], sh_pq[D];              // bk[h] and phi_q of the head, staged with Wk
  __shared__ int sh_scan[NWV];
  __shared__ uint64_t sh_prefix, sh_thr;
  __shared__ int sh_want, sh_tot;
  __shared__ int sh_bstar, sh_krem, sh_chi, sh_nb, sh_nbc;
  __shared__ uint32_t sh_total, sh_ovp;
  __shared__ LocalMerge sh_lm;
  uint32_t* sh_hist = (uint32_t*)lds_a;
  uint64_t* bcand = (uint64_t*)(lds_a + 8192);
  float* red = (float*)lds_a;                       // [16 wavefronts][2][128]

  const int tid = threadIdx.x;
  const int lane = tid & 63, wv = tid >> 6;
  TKPHI_PHASE(ws, 10);
  char* blk = problem_block(g, ws, p);
  const int T = g.cand_T;
  const int n_reg_max = g.n_scan_chunks * 4;
  const uint32_t cap_w = (uint32_t)(g.scan_chunk / 4);
  // (after a rescan these three point at the rescan set)
  const uint32_t* ccount = (const uint32_t*)(blk + g.off_ccount) + (size_t)gq * n_reg_max;
  const uint2* compact = (const uint2*)(blk + g.off_candc) + (size_t)gq * n_reg_max * T;
  const uint2* sparse = (const uint2*)(blk + g.off_candf) + (size_t)gq * n_reg_max * cap_w;

  // ---- first sweep, speculatively: addresses depend on the launch geometry only --------------------------
  u32x4 e0[kSweepLoads];
  uint32_t c0 = 0;
  const uint32_t edge0 = DIRECT ? 0u : ((const uint32_t*)(blk + g.off_thr))[gq];   // the bound the score pass pruned this head with
  if constexpr (DIRECT) {                         // the head's row of scores, 4 tokens per load
    const float* row = (const float*)(blk + g.off_scores) + (size_t)gq * g.mid_stride;
#pragma unroll
    for (int k = 0; k < kSweepEntries / 4; ++k)
      if (4 * (tid + k * NTHR) < g.mid_stride) e0[k] = gload128(row + 4 * (tid + k * NTHR));
  } else {
    const int s = kSweepEntries * tid, list = s / T;
    if (list < n_reg_max) {
      c0 = ccount[list];
#pragma unroll
      for (int u = 0; u < kSweepLoads; ++u) e0[u] = gload128(compact + s + 2 * u);
    }
  }
  const tkphi_problem pr = probs[p];
  if (pr.L < 1 || pr.L > g.max_L) return false;
  const int n = mid_size(pr.L, g.n_sink, g.n_tail);
  const int Ksel = max(0, min(min(pr.topk, n), g.max_K));
  SelPlan* plan = (SelPlan*)(blk + g.off_plan) + gq;
  if (Ksel == 0) {
    if (tid == 0 && part == 0) *plan = SelPlan{-1, 0, 0, 0, 0};
    return false;
  }
  const int h = gq / g.G;
  const int n_chunks = (n + g.scan_chunk - 1) / g.scan_chunk;
  const int n_reg = n_chunks * 4;
  const int rounds = (n_reg * T + NTHR * kSweepEntries - 1) / (NTHR * kSweepEntries);
  int32_t* sel_idx = (int32_t*)(blk + g.off_selidx) + (size_t)gq * g.max_K;
  float* sel_score = (float*)(blk + g.off_selscore) + (size_t)gq * g.max_K;

  // entries [0, nvalid) at src are the share of thread t in sweep sw; they belong to list `list`
  struct Share { const uint2* src; int nvalid; int list; };
  int max_passes = 0;                               // overflow sweeps per round (set below)
  auto share_of = [&](int sw, int t, int known = -1) -> Share {   // known: the list's length if the caller has it
    const int r = sw < rounds ? sw : (sw - rounds) / max_passes;
    const int s = kSweepEntries * (t + NTHR * r), list = s / T, pos = s % T;
    if (list >= n_reg) return Share{compact, 0, list};
    const int c = (int)min(known >= 0 ? (uint32_t)known : ccount[list], cap_w);
    if (sw < rounds) return Share{compact + s, max(0, min(min(c, T) - pos, kSweepEntries)), list};
    const int k = (sw - rounds) % max_passes;
    const int start = T + (k * (T / kSweepEntries) + pos / kSweepEntries) * kSweepEntries;
    return Share{sparse + (size_t)list * cap_w + start, max(0, min(c - start, kSweepEntries)), list};
  };
  auto load_share = [&](const Share& sh, u32x4 (&e)[kSweepLoads]) {
#pragma unroll
    for (int u = 0; u < kSweepLoads; ++u)
      if (2 * u < sh.nvalid) e[u] = gload128(sh.src + 2 * u);
  };
  auto entry = [](const u32x4 (&e)[kSweepLoads], int i) { return (i & 1) ? make_uint2(e[i >> 1].z, e[i >> 1].w) : make_uint2(e[i >> 1].x, e[i >> 1].y); };

  // ---- candidate count, overflow depth (and, on a threshold miss, the rescan) ---------------------------
  bool have_e0 = true;
  int n_sweeps = 0;
  if constexpr (!DIRECT) for (int attempt = 0;; ++attempt) {
    if (tid == 0) { sh_total = 0u; sh_ovp = 0u; }
    __syncthreads();
    uint32_t tot = 0, ovp = 0;
    for (int r = 0; r < rounds; ++r) {
      const int s = kSweepEntries * (tid + NTHR * r), list = s / T;
      if (s % T == 0 && list < n_reg) {               // the thread that owns the head of a list counts it
        const uint32_t len = (r == 0 && have_e0) ? c0 : ccount[list], c = min(len, cap_w);
        tot += c;
        if (c > (uint32_t)T) ovp = max(ovp, (c - T + T - 1) / T);
        if (len == kNoList) ovp = kNoList;
      }
    }
    if (tot) atomicAdd(&sh_total, tot);
    if (ovp) atomicMax(&sh_ovp, ovp);
    __syncthreads();
    if ((sh_total >= (uint32_t)Ksel && sh_ovp != kNoList) || attempt > 0) {
      max_passes = (int)sh_ovp;
      n_sweeps = rounds + rounds * max_passes;
      break;
    }
    __syncthreads();
    // (every workgroup of the head takes this branch, the counts it depends on being the score pass's, and writes
    // the same values to the rescan set: no ordering between them is needed.  A head's only workgroup may write the first set
    // over: every thread has read its counts before the barrier above, and nothing else of that set is read again)
    rescan_head<D, NTHR>(g, pr, blk, gq, n, n_reg);
    ccount = (const uint32_t*)(blk + g.off_rescount) + (size_t)gq * n_reg_max;
    compact = (const uint2*)(blk + g.off_resc) + (size_t)gq * n_reg_max * T;
    sparse = (const uint2*)(blk + g.off_resf) + (size_t)gq * n_reg_max * cap_w;
    have_e0 = false;
    __syncthreads();
  }
  if (DIRECT) n_sweeps = 1;
  const uint32_t total = DIRECT ? (uint32_t)n : sh_total;
  TKPHI_PHASE(ws, 11);
  float* partial = (float*)(blk + g.off_part) + ((size_t)gq * (g.n_tiles + g.n_atiles) + part) * g.part_stride;
  auto empty_partial = [&]() {
    if (LIST) return;
    if (tid == 0) { store_agent(partial, -INFINITY); store_agent(partial + 1, 0.f); store_agent(partial + 2, 0.f); store_agent(partial + 3, 0.f); }
    if (tid < D) { store_agent(partial + 4 + tid, 0.f); store_agent(partial + 4 + D + tid, 0.f); }
  };
  if (total < (uint32_t)Ksel) {                     // cannot happen after a rescan (every mid token is a candidate)
    if (tid == 0 && part == 0) *plan = SelPlan{-1, 0, 0, 0, 0};
    empty_partial();
    return false;
  }
  // Wk[h] for the gather phase: requested now (the first sweep has arrived, nothing else is in flight; the barrier after the
  // histogram pass orders LDS only, so it does not wait for these loads)
  WkPieces<D, NTHR, sizeof(KV)> wkp;
  float bk_t = 0.f, pq_t = 0.f;
  if constexpr (!LIST) wkp.request(pr.Wk, h);
  if (!LIST && tid < D) { bk_t = pr.bk[(size_t)h * D + tid]; pq_t = ((const float*)(blk + g.off_phiq))[(size_t)gq * D + tid]; }

  // A head's only workgroup merges it on the spot: its partial stays in LDS, and the anchors' partials and the summary terms, which an
  // earlier launch left, are requested here, long before they are needed.  By way of memory, as from workgroup to workgroup, the
  // merge of a short context was 3 us of 12.5 (two round trips at the end of the chain): 1B layer at 4K 19.4 -> 18.0 us per step, 3B layer at
  // 2K 19.1 -> 17.8, one fp32 head of 4K 17.1 -> 15.9, 256 ragged sequences 2630 -> 2587.
  // (what the end needs of the record waits in LDS: the list kernels with a merge of their own already spill 57 to 64 scalars)
  if (LOCAL && tid == 0) {
    const int n_at = (g.n_sink + g.n_tail + min(max(pr.n_gen, 0), g.max_gen) + 63) / 64;
    const bool local = !pr.topk_idx && n_at <= kLocalTiles;
    sh_lm = LocalMerge{pr.out, pr.aux, local ? n_at : 0, has_residual(mode, n, Ksel) ? 1 : 0, mode == TKPHI_MODE_SUB ? 1 : 0};
  }
  u32x4 anc;
  float pre_n = 0.f, pre_z = 0.f;
  auto request_local = [&]() {                      // (behind at least one barrier)
    if constexpr (!LOCAL) return;
    const int n_at = sh_lm.n_at;
    if (4 * tid < n_at * (2 * D + 4))
      anc = gload128((const float*)(blk + g.off_part) + ((size_t)gq * (g.n_tiles + g.n_atiles) + g.n_tiles) * (2 * D + 4) + 4 * tid);
    if (n_at > 0 && tid < D) {
      pre_n = ((const float*)(blk + g.off_sphi))[(size_t)gq * D + tid];
      pre_z = ((const float*)(blk + g.off_uphi))[gq];
    }
  };

  // (to LDS once the threshold is found: the barriers of the winners' prefix sums publish it, and the gather begins with its loads)
  auto commit_wk = [&]() {
    if constexpr (!LIST) {
      wkp.commit(wk_lds);
      if (tid < D) { sh_bk[tid] = bk_t; sh_pq[tid] = pq_t; }
    }
  };

  // (have_e0 is false exactly after a rescan: those lists were written without a bound)
  const SelBins bin_of{edge0, have_e0 && edge0 != 0u && edge0 != 0xffffffffu};
  const int split = g.sg_split;
  int my_base = 0, my_count = 0;                    // winners ahead of this workgroup's; winners of this workgroup
  // The candidates are packed, sweep by sweep, into an LDS array (96 KB at d = 64, 80 at d = 128 that are otherwise unused: a
  // workgroup of 1024 threads has a CU to itself; 32 KB for 512 threads); histogram, threshold and winners then walk 3-4 entries per thread (about 3 K candidates per
  // head at a 1 % budget of 128K) instead of 12 list slots per sweep, and workgroup `part` takes the winners of an equal
  // share of the array.  More candidates than it holds: a first pass over the sweeps finds the boundary bin, and only
  // what lies in it or above is packed.
  auto clear_hist = [&]() {
    for (int i = tid; i < kFineBins; i += NTHR) sh_hist[i] = 0u;
    if (tid == 0) { sh_bstar = -1; sh_krem = 0; sh_chi = 0; sh_nb = 0; sh_nbc = 0; sh_thr = 0ull; }
  };
  // histogram -> boundary bin: thread t takes the BPT bins below kFineBins - BPT t, highest first: a prefix sum over the
  // threads is a suffix sum over the bins
  auto boundary_bin = [&]() {
    constexpr int BPT = kFineBins / NTHR;
    int cb[BPT], own = 0;
#pragma unroll
    for (int e = 0; e < BPT; ++e) { cb[e] = (int)sh_hist[kFineBins - 1 - BPT * tid - e]; own += cb[e]; }
    int gt = sel_scan_incl(own, sh_scan) - own;              // candidates in bins above this thread's
#pragma unroll
    for (int e = 0; e < BPT; ++e) {
      if (gt + cb[e] >= Ksel && gt < Ksel) { sh_bstar = kFineBins - 1 - BPT * tid - e; sh_krem = Ksel - gt; sh_chi = gt; sh_nb = cb[e]; }
      gt += cb[e];
    }
    lds_barrier();
  };
  auto sweep_histogram = [&]() {
    for (int sw = 0; sw < n_sweeps; ++sw) {
      const Share sh = share_of(sw, tid);
      u32x4 e[kSweepLoads];
      load_share(sh, e);
#pragma unroll
      for (int i = 0; i < kSweepEntries; ++i)
        if (i < sh.nvalid) atomicAdd(&sh_hist[bin_of(score_key(__uint_as_float(entry(e, i).x)))], 1u);
    }
    lds_barrier();                                    // (the histogram is LDS traffic; the Wk loads stay in flight)
  };
  bool packed = DIRECT || total <= (uint32_t)kDense;     // (Geom::direct: the mid-region fits the array)
  int min_bin = 0;                                  // candidates in lower bins are not packed
  if (!DIRECT && !packed) {
    clear_hist();
    __syncthreads();
    sweep_histogram();
    boundary_bin();
    min_bin = sh_bstar;
    packed = min_bin >= 0 && sh_chi + sh_nb <= kDense;       // (else all scores (nearly) equal, or a budget beyond the array)
    lds_barrier();
  }
  if (DIRECT || packed) {
    int n_cand = 0;
    clear_hist();
    if constexpr (DIRECT) {                        // entry i = token i, straight from the registers of the speculative loads
#pragma unroll
      for (int k = 0; k < kSweepEntries / 4; ++k) {
        const uint32_t sc[4] = {e0[k].x, e0[k].y, e0[k].z, e0[k].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int tok = 4 * (tid + k * NTHR) + i;
          if (tok < n) dense[tok] = make_uint2(sc[i], (uint32_t)tok);
        }
      }
      n_cand = n;
      lds_barrier();
    } else if (n_sweeps == 1 && have_e0 && min_bin == 0) {  // the usual case, straight from the registers of the speculative sweep
      const int nv = share_of(0, tid, (int)min(c0, cap_w)).nvalid;
      const int off = sel_scan_incl(nv, sh_scan) - nv;       // (its barriers also publish the cleared histogram)
#pragma unroll
      for (int i = 0; i < kSweepEntries; ++i)
        if (i < nv) dense[off + i] = entry(e0, i);
      n_cand = (int)total;
      lds_barrier();
    } else {
      for (int sw = 0; sw < n_sweeps; ++sw) {
        const Share sh = share_of(sw, tid);
        u32x4 e[kSweepLoads];
        load_share(sh, e);
        uint32_t keep = 0;
#pragma unroll
        for (int i = 0; i < kSweepEntries; ++i)
          if (i < sh.nvalid && (min_bin == 0 || bin_of(score_key(__uint_as_float(entry(e, i).x))) >= min_bin)) keep |= 1u << i;
        const int nw = __popc(keep);
        const int incl = sel_scan_incl(nw, sh_scan);
        int at = n_cand + incl - nw;
#pragma unroll
        for (int i = 0; i < kSweepEntries; ++i)
          if (keep & (1u << i)) dense[at++] = entry(e, i);
        if (tid == NTHR - 1) sh_tot = incl;
        lds_barrier();
        n_cand += sh_tot;
      }
    }
    const int r0 = (int)((uint32_t)(n_cand * part) / (uint32_t)split), r1 = (int)((uint32_t)(n_cand * (part + 1)) / (uint32_t)split);
    // ---- histogram -> boundary bin ----------------------------------------------------------------------------
    for (int idx = tid; idx < n_cand; idx += NTHR) atomicAdd(&sh_hist[bin_of(score_key(__uint_as_float(dense[idx].x)))], 1u);
    lds_barrier();
    TKPHI_PHASE(ws, 12);
    boundary_bin();
    const int bstar = sh_bstar, krem = sh_krem, c_hi = sh_chi, nb = sh_nb;
    if (bstar < 0) {                                  // cannot happen: total >= Ksel
      if (tid == 0 && part == 0) *plan = SelPlan{-1, 0, 0, 0, 0};
      empty_partial();
      return false;
    }
    TKPHI_PHASE(ws, 13);
    request_local();
    // ---- thr: the K_rem-th best composite of the boundary bin -------------------------------------------------
    if (nb <= kBCap) {
      for (int idx = tid; idx < n_cand; idx += NTHR) {
        const uint2 en = dense[idx];
        const uint32_t key = score_key(__uint_as_float(en.x));
        if (bin_of(key) == bstar) {
          const int at = atomicAdd(&sh_nbc, 1);
          if (at < kBCap) bcand[at] = composite(key, en.y);
        }
      }
      lds_barrier();
      const int sub = tid & 7, slot = tid >> 3;
      for (int k0 = 0; k0 < nb; k0 += NTHR / 8) {
        const int j = k0 + slot;
        const bool valid = j < nb;
        const uint64_t mine = valid ? bcand[j] : ~0ull;
        int rank = 0;
        for (int i = sub; i < nb; i += 8) rank += bcand[i] > mine ? 1 : 0;
        rank = lanes_sum(rank, 8);
        if (valid && sub == 0 && rank == krem - 1) sh_thr = mine;
      }
      lds_barrier();
    } else {                                          // (e.g. all scores equal) radix passes over the packed array
      auto get = [&](int j, uint64_t* v) {
        const uint2 en = dense[j];
        const uint32_t key = score_key(__uint_as_float(en.x));
        *v = composite(key, en.y);
        return bin_of(key) == bstar;
      };
      const uint64_t t = radix_select_desc(n_cand, krem, get, sh_hist, sh_scan, &sh_prefix, &sh_want);
      if (tid == 0) sh_thr = t;
      __syncthreads();
    }
    const uint64_t thr = sh_thr;
    TKPHI_PHASE(ws, 14);
    commit_wk();
    if (tid == 0 && part == 0) *plan = SelPlan{bstar, krem, c_hi, nb, Ksel};
    // ---- winners of the packed range [r0, r1) --------------------------------------------------------------------
    auto is_winner = [&](int idx, int lim, uint2* en) {
      if (idx >= lim) return false;
      *en = dense[idx];
      return composite(score_key(__uint_as_float(en->x)), en->y) >= thr;
    };
    {
      // thread t owns the `per` consecutive entries from r0 + t per: one prefix sum over the threads keeps list order
      const int per = (r1 - r0 + NTHR - 1) / NTHR, first = r0 + tid * per;
      int mine = 0;
      for (int e = 0; e < per; ++e) { uint2 en; mine += is_winner(first + e, r1, &en) ? 1 : 0; }
      const int incl = sel_scan_incl(mine, sh_scan);
      if (tid == NTHR - 1) sh_tot = incl;
      int at = incl - mine;
      for (int e = 0; e < per; ++e) {
        uint2 en;
        if (is_winner(first + e, r1, &en)) {
          if (LIST) { if (at < min(Ksel, g.max_K)) { sel_idx[at] = (int32_t)en.y; sel_score[at] = __uint_as_float(en.x); } }
          else if (at < kWinLds) { w_tok[at] = (int)en.y; w_s[at] = __uint_as_float(en.x); }
          ++at;
        }
      }
      lds_barrier();
      my_count = sh_tot;
    }
    // the retrieved list of the head, for the export of the merge and for winners beyond the LDS stage
    if (!LIST && (my_count > kWinLds || pr.topk_idx)) {
      int before = 0;
      for (int idx = tid; idx < r0; idx += NTHR) { uint2 en; before += is_winner(idx, r0, &en) ? 1 : 0; }
      const int incl_b = sel_scan_incl(before, sh_scan);
      if (tid == NTHR - 1) sh_tot = incl_b;
      lds_barrier();
      my_base = sh_tot;
      lds_barrier();
      int seen = 0;
      for (int base = r0; base < r1; base += NTHR) {
        uint2 en = make_uint2(0u, 0u);
        const int flag = is_winner(base + tid, r1, &en) ? 1 : 0;
        const int incl = sel_scan_incl(flag, sh_scan);
        if (tid == NTHR - 1) sh_tot = incl;
        const int at = my_base + seen + incl - flag;
        if (flag && at < min(Ksel, g.max_K)) { sel_idx[at] = (int32_t)en.y; sel_score[at] = __uint_as_float(en.x); }
        __syncthreads();
        seen += sh_tot;
        __syncthreads();
      }
    }
  } else {
    // (the general path: the candidates that may be winners do not fit the packed array; every phase reads its entries from the
    // lists again)
    // ---- pass A: histogram of the candidates' fine bins ----------------------------------------------------------
    // (this workgroup's share of the gather: the winners of lists [l0, l1), in list order)
    const int per_part = (n_reg + split - 1) / split;
    const int l0 = part * per_part, l1 = min(n_reg, l0 + per_part);
    clear_hist();
    __syncthreads();
    sweep_histogram();
    TKPHI_PHASE(ws, 12);
    boundary_bin();
    const int bstar = sh_bstar, krem = sh_krem, c_hi = sh_chi, nb = sh_nb;
    if (bstar < 0) {                                  // cannot happen: total >= Ksel
      if (tid == 0 && part == 0) *plan = SelPlan{-1, 0, 0, 0, 0};
      empty_partial();
      return false;
    }
    TKPHI_PHASE(ws, 13);
    request_local();

    // ---- thr: the K_rem-th best composite of the boundary bin ------------------------------------------------
    if (nb <= kBCap) {
      // stage the boundary candidates (any order: ranks do not depend on it), then rank by counting the larger
      // composites, 8 lanes per candidate; the candidate of rank K_rem - 1 is the threshold
      for (int sw = 0; sw < n_sweeps; ++sw) {
        const Share sh = share_of(sw, tid);
        u32x4 e[kSweepLoads];
        load_share(sh, e);
#pragma unroll
        for (int i = 0; i < kSweepEntries; ++i) {
          if (i < sh.nvalid) {
            const uint2 en = entry(e, i);
            const uint32_t key = score_key(__uint_as_float(en.x));
            if (bin_of(key) == bstar) {
              const int at = atomicAdd(&sh_nbc, 1);
              if (at < kBCap) bcand[at] = composite(key, en.y);
            }
          }
        }
      }
      lds_barrier();
      const int sub = tid & 7, slot = tid >> 3;
      for (int k0 = 0; k0 < nb; k0 += NTHR / 8) {
        const int j = k0 + slot;
        const bool valid = j < nb;
        const uint64_t mine = valid ? bcand[j] : ~0ull;
        int rank = 0;
        int i = sub;
        for (; i + 24 < nb; i += 32) {
          const uint64_t x0 = bcand[i], x1 = bcand[i + 8], x2 = bcand[i + 16], x3 = bcand[i + 24];
          rank += (x0 > mine ? 1 : 0) + (x1 > mine ? 1 : 0) + (x2 > mine ? 1 : 0) + (x3 > mine ? 1 : 0);
        }
        for (; i < nb; i += 8) rank += bcand[i] > mine ? 1 : 0;
        rank = lanes_sum(rank, 8);
        if (valid && sub == 0 && rank == krem - 1) sh_thr = mine;
      }
      lds_barrier();
    } else {
      // the slot (sweep, thread, entry) as one index for the radix passes (e.g. all scores equal)
      auto get = [&](int j, uint64_t* v) {
        const int sw = j / (NTHR * kSweepEntries), rem = j % (NTHR * kSweepEntries);
        const Share sh = share_of(sw, rem / kSweepEntries);
        const int i = rem % kSweepEntries;
        if (i >= sh.nvalid) return false;
        const uint2 e = sh.src[i];
        const uint32_t key = score_key(__uint_as_float(e.x));
        *v = composite(key, e.y);
        return bin_of(key) == bstar;
      };
      const uint64_t t = radix_select_desc(n_sweeps * NTHR * kSweepEntries, krem, get, sh_hist, sh_scan, &sh_prefix, &sh_want);
      if (tid == 0) sh_thr = t;
      __syncthreads();
    }
    const uint64_t thr = sh_thr;
    TKPHI_PHASE(ws, 14);
    commit_wk();
    if (tid == 0 && part == 0) *plan = SelPlan{bstar, krem, c_hi, nb, Ksel};

    // ---- this workgroup's winners: lists [l0, l1), in list order -----------------------------------------------
    for (int sw = 0; sw < n_sweeps; ++sw) {
      const Share sh = share_of(sw, tid);
      u32x4 e[kSweepLoads];
      load_share(sh, e);
      uint32_t fw = 0;                                // bit i: entry i is retrieved
#pragma unroll
      for (int i = 0; i < kSweepEntries; ++i) {
        if (i < sh.nvalid) {
          const uint2 en = entry(e, i);
          if (composite(score_key(__uint_as_float(en.x)), en.y) >= thr) fw |= 1u << i;
        }
      }
      const int nw = __popc(fw);
      const bool mine = sh.list >= l0 && sh.list < l1;
      // (winners of one sweep: <= 12288 mine, <= 12288 before: 16 bits each)
      const int packed = (mine ? nw : 0) | ((sh.list < l0 ? nw : 0) << 16);
      const int incl = sel_scan_incl(packed, sh_scan);
      if (tid == NTHR - 1) sh_tot = incl;
      int at = my_count + ((incl - packed) & 0xffff);   // rank among this workgroup's winners
      lds_barrier();
      const int tot = sh_tot;
      if (mine) {
#pragma unroll
        for (int i = 0; i < kSweepEntries; ++i) {
          if (fw & (1u << i)) {
            const uint2 en = entry(e, i);
            if (!LIST && at < kWinLds) { w_tok[at] = (int)en.y; w_s[at] = __uint_as_float(en.x); }
            // (global position: filled in below, once the winners of earlier lists in later sweeps are known)
            ++at;
          }
        }
      }
      my_count += tot & 0xffff;
      my_base += tot >> 16;
      lds_barrier();
    }
    // the retrieved list of the head, for the exports of the merge kernel and for winners beyond the LDS stage:
    // a second pass writes this workgroup's winners at my_base + rank (list positions never leave [0, Ksel))
    {
      int seen = 0;
      const bool need_global = my_count > kWinLds;
      for (int sw = 0; sw < n_sweeps; ++sw) {
        const Share sh = share_of(sw, tid);
        const bool mine = sh.list >= l0 && sh.list < l1;
        if (!LIST && n_sweeps == 1 && !need_global && !pr.topk_idx) break;     // (nothing reads the list)
        u32x4 e[kSweepLoads];
        load_share(sh, e);
        uint32_t fw = 0;
#pragma unroll
        for (int i = 0; i < kSweepEntries; ++i) {
          if (mine && i < sh.nvalid) {
            const uint2 en = entry(e, i);
            if (composite(score_key(__uint_as_float(en.x)), en.y) >= thr) fw |= 1u << i;
          }
        }
        const int nw = __popc(fw);
        const int incl = sel_scan_incl(nw, sh_scan);
        if (tid == NTHR - 1) sh_tot = incl;
        int at = my_base + seen + incl - nw;
#pragma unroll
        for (int i = 0; i < kSweepEntries; ++i) {
          if (fw & (1u << i)) {
            const uint2 en = entry(e, i);
            if (at < min(Ksel, g.max_K)) { sel_idx[at] = (int32_t)en.y; sel_score[at] = __uint_as_float(en.x); }
            ++at;
          }
        }
        __syncthreads();
        seen += sh_tot;
        __syncthreads();
      }
    }
  }
  TKPHI_PHASE(ws, 15);
  if constexpr (LIST) return false;

  // ---- gather: kBatch winners per round, one or two 16-token tiles per wavefront -----------------------------
  const int r = lane & 15, kg = lane >> 4;
  const int64_t head_off = (int64_t)h * pr.stride_head;
  constexpr int LPR = D / EPL;                      // lanes per value row (16 bytes each)
  constexpr int RPP = NTHR / LPR;            // rows per pass (64 or 128)
  constexpr int NPASS = kBatch / RPP;               // value rows per thread and round (4)
  constexpr int NTW = kBatch / (16 * NWV);    // 16-token tiles per wavefront and round
  const int seg = tid % LPR, rsub = tid / LPR;
  // mid indices of N winners of the round that starts at b0, all LDS reads together; those beyond the LDS stage (rare) from the list
  const bool staged = my_count <= kWinLds;
  auto winners = [&](auto& tok, int b0, int first, int step) {
    constexpr int N = sizeof(tok) / sizeof(int);
    const int last = min(kBatch, my_count - b0) - 1;
#pragma unroll
    for (int k = 0; k < N; ++k) tok[k] = w_tok[min(b0 + min(first + k * step, last), kWinLds - 1)];
    if (!staged) {
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const int i = b0 + min(first + k * step, last);
        if (i >= kWinLds) tok[k] = sel_idx[min(my_base + i, g.max_K - 1)];
      }
      wait_vm_loads<0>();                           // (here, or the common path would wait for its rows as well)
    }
#pragma unroll
    for (int k = 0; k < N; ++k) tok[k] = g.n_sink + min(max(tok[k], 0), n - 1);
  };
  auto score_of = [&](int i) {
    float s = w_s[min(i, kWinLds - 1)];
    if (!staged) {
      if (i >= kWinLds) s = sel_score[min(my_base + i, g.max_K - 1)];
      wait_vm_loads<0>();
    }
    return s;
  };
  // The key rows of this wavefront's tiles and the value rows of all passes only need the token indices.  The rows
  // of round b + 1 are requested inside round b, each set into the registers round b has just finished with (keys
  // after the feature dots, values after the weighted sums): a round trip to memory per workgroup, not per round.
  GatherFrag a[NTW][KS];
  u32x4 vrow[NPASS];
  auto load_keys = [&](int b0) {
    const int cnt = min(kBatch, my_count - b0);
    int tk[NTW];
    winners(tk, b0, wv * 16 + r, NWV * 16);
#pragma unroll
    for (int u = 0; u < NTW; ++u) {
      const int t16 = (wv + u * NWV) * 16;      // first token of this wavefront's u-th tile
      if (t16 < cnt) {
        const char* rp = (const char*)pr.K + (head_off + (int64_t)tk[u] * pr.stride_tok) * sizeof(KV) + kg * 16;
#pragma unroll
        for (int j = 0; j < KS; ++j) a[u][j].u = gload128(rp + j * 64);
      }
    }
  };
  auto load_values = [&](int b0) {
    const int cnt = min(kBatch, my_count - b0);
    int tk[NPASS];
    winners(tk, b0, rsub, RPP);
#pragma unroll
    for (int ps = 0; ps < NPASS; ++ps)
      if (ps * RPP < cnt) vrow[ps] = gload128((const char*)pr.V + (head_off + (int64_t)tk[ps] * pr.stride_tok + seg * EPL) * sizeof(KV));
  };
  if constexpr (LOCAL) {
    const int n_at = sh_lm.n_at;
    if (4 * tid < n_at * (2 * D + 4)) *(u32x4*)(sh_parts + 4 * tid) = anc;
    if (n_at > 0 && tid < D) { sh_parts[(kLocalTiles + 1) * (2 * D + 4) + tid] = pre_n; if (tid == 0) sh_lm.pre_z = pre_z; }
  }
  if (my_count > 0) { load_keys(0); load_values(0); }
  // The scores' maximum (known behind the first round's barrier): the weights of all rounds have one shift, and the rounds no sums to rescale
  {
    float lm = -INFINITY;
    for (int i = tid; i < my_count; i += NTHR) lm = fmaxf(lm, score_of(i));
    lm = wave_max(lm);
    if (lane == 0) sh_wave[0][wv] = lm;
  }
  float run_m = -INFINITY;
  float Zt = 0.f, zst = 0.f;                        // this thread's share of Z_loc; of zsum (a lane's four tokens, the same in all of r)
  float an[EPL], az[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) { an[e] = 0.f; az[e] = 0.f; }
  // One barrier per round: scores and z of its tokens go through the buffers that the round before last has read.  With five barriers, and the
  // sums over the wavefronts in every round, a round of 256 took 8 us at d = 128, now 5: 3B layer at 128K 4 % 91.1 -> 88.0 us per step, 16 ragged
  // ones of 10K..40K at 3 % 243 -> 230, 256 ragged ones of the 1B layer at 1 % 2600 -> 2560; with one round 1B layer at 4K 18.1 -> 17.7, 32K 27.5 -> 27.0.
#pragma unroll 1
  for (int b0 = 0, par = 0; b0 < my_count; b0 += kBatch, par ^= 1) {
    const int cnt = min(kBatch, my_count - b0);
    const bool more = b0 + kBatch < my_count;
    const float s_own = tid < cnt ? score_of(b0 + tid) : -INFINITY;
    if (tid < kBatch) b_w[par][tid] = s_own;        // (scores; every reader makes its weight of one)
    // z_i of this wavefront's tokens
#pragma unroll
    for (int u = 0; u < NTW; ++u) {
      const int t16 = (wv + u * NWV) * 16;
      if (t16 < cnt) {
        float z[4];
        if constexpr (sizeof(KV) == 4) wave_feature_dots_f32<D>(a[u], wk_lds, sh_bk, sh_pq, g.a, g.c, z);
        else wave_feature_dots<D>(a[u], wk_lds, sh_bk, sh_pq, g.a, g.c, z);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool in = t16 + 4 * kg + i < cnt;
          if (in) zst += z[i];
          if (r == 0) b_z[par][t16 + 4 * kg + i] = in ? z[i] : 0.f;
        }
      }
    }
    if (more) load_keys(b0 + kBatch);
    lds_barrier();
    if (b0 == 0) run_m = lanes_reduce(sh_wave[0][lane & (NWV - 1)], NWV, MaxOp());
    Zt += __expf(s_own - run_m);
    // weighted value sums of this thread's rows
#pragma unroll
    for (int ps = 0; ps < NPASS; ++ps) {
      const int i = ps * RPP + rsub;
      if (ps * RPP < cnt && i < cnt) {
        float x[EPL];
        Elem<KV>::unpack(make_uint4(vrow[ps].x, vrow[ps].y, vrow[ps].z, vrow[ps].w), x);
        const float wi = __expf(b_w[par][i] - run_m), zi = b_z[par][i];
#pragma unroll
        for (int e = 0; e < EPL; ++e) { an[e] = fmaf(wi, x[e], an[e]); az[e] = fmaf(zi, x[e], az[e]); }
      }
    }
    if (more) load_values(b0 + kBatch);
  }
  // rows of one wavefront that share a segment, then the wavefronts
  static_assert(LPR == 8 || LPR == 16, "lanes per row");
#pragma unroll
  for (int e = 0; e < EPL; ++e) { an[e] = strided_sum(an[e], LPR); az[e] = strided_sum(az[e], LPR); }
  if (lane < LPR) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) { red[(wv * 2 + 0) * 128 + lane * EPL + e] = an[e]; red[(wv * 2 + 1) * 128 + lane * EPL + e] = az[e]; }
  }
  Zt = wave_sum(Zt);
  zst = strided_sum(zst, 16);
  if (lane == 0) { sh_wave[1][wv] = Zt; sh_wave[2][wv] = zst; }
  lds_barrier();
  // channel tid < D; the wavefront behind those adds up Z_loc and zsum
  float* own = sh_parts;                            // (LOCAL)
  int n_at = 0;
  if constexpr (LOCAL) { n_at = sh_lm.n_at; own += n_at * (2 * D + 4); }
  auto out = [&](int k, float x) {                  // (GPU-coherent: the workgroup that merges the head may run on another XCD)
    if (LOCAL && n_at) own[k] = x;
    else store_agent(partial + k, x);
  };
  if (tid < D) {
    float nu = 0.f, zv = 0.f;
    for (int k = 0; k < NWV; ++k) { nu += red[(k * 2 + 0) * 128 + tid]; zv += red[(k * 2 + 1) * 128 + tid]; }
    out(4 + tid, nu);
    out(4 + D + tid, zv);
  } else if (wv == D / 64) {
    const float Z = lanes_reduce(sh_wave[1][lane & (NWV - 1)], NWV, AddOp()), zs = lanes_reduce(sh_wave[2][lane & (NWV - 1)], NWV, AddOp());
    if (lane == 0) { out(0, run_m); out(1, Z); out(2, zs); out(3, (float)my_count); }
  }
  if (LOCAL && n_at) {
    lds_barrier();
    if (tid < D) merge_head_local<D>(sh_lm, n_at + 1, sh_parts, sh_parts[(kLocalTiles + 1) * (2 * D + 4) + tid], (uint32_t*)(ws + g.off_status), gq);
    return true;
  }
  TKPHI_PHASE(ws, 16);
  return false;
}

// grid (sg_split, Hq, n_problems).  After its own share every workgroup of a head counts itself in (its partial made
// visible first); the one that arrives last finds all partials of the head complete and merges them (merge_head.h)
// with its first 256 threads: no separate merge launch.  The counters are cleared by a launch before this one in the
// same call: the phi jobs of whichever launch carries them.  (The other wavefronts of that workgroup end before the merge's
// barriers: a barrier waits only for the wavefronts of the workgroup that are still running.)
// LOCAL: sg_split is 1
template <int D, int NTHR, bool DIRECT, bool LIST, bool LOCAL, typename KV = uint16_t>
__global__ __launch_bounds__(NTHR) __attribute__((amdgpu_waves_per_eu(4, 4))) void select_gather_kernel(Geom g, const tkphi_problem* __restrict__ probs,
                                                                    char* __restrict__ ws, int mode) {
  __shared__ int sh_last;
  if constexpr (LIST) {
    // grid (Hq + Hq d_emb / 64 + ..): behind a workgroup per head, on the CUs that the selection leaves idle, a stage of phi_q (the
    // second, where the first rode in a score launch long enough for it) and, for a step that recomputes features, the weights of
    // the chain over the retrieved keys (a single problem: slot 0).  As a launch between select and chain the packing took 9 us of a
    // 3B layer's step; phi_q on a second stream, joined before the gather, held a step with a feature cache at 65 us up to 16K
    // tokens (now 40 at 4K, 49 at 16K).
    const int idx = blockIdx.x, n_phi = g.d_emb / 64 * g.Hq, p = 0;
    if (idx >= g.Hq) {
      const tkphi_problem& pr = probs[p];
      if (pr.L < 1 || pr.L > g.max_L) return;
      if (idx < g.Hq + n_phi) {
        __shared__ __attribute__((aligned(16))) float sh_q[kQuerySliceLds];
        mlp_phi_q_slice<DIRECT ? 0 : 1>(g, pr, problem_block(g, ws, p), (idx - g.Hq) % g.Hq, (idx - g.Hq) / g.Hq, sh_q);
        return;
      }
      const int wg = idx - g.Hq - n_phi, n_wg = ((int)gridDim.x - g.Hq - n_phi) / g.Hkv, h = wg % g.Hkv;
      const tkphi_mlp mp = pr.mlp_k[h];
      for (size_t q = (size_t)(wg / g.Hkv) * NTHR + threadIdx.x; q < packed_pieces(g); q += (size_t)n_wg * NTHR) pack_piece(g, ws, mp, 0, h, q, true);
      return;
    }
    const int gq = idx;
    select_gather_body<D, NTHR, DIRECT, LIST, LOCAL, KV>(g, probs, ws, 0, gq, p, mode);
    if (!DIRECT && g.fused && threadIdx.x == 0) ((uint64_t*)(problem_block(g, ws, p) + g.off_hand))[gq] = 0ull;     // (as below)
    return;
  } else {
  const int part = blockIdx.x, gq = blockIdx.y, p = blockIdx.z;
  if (select_gather_body<D, NTHR, DIRECT, LIST, LOCAL, KV>(g, probs, ws, part, gq, p, mode)) {
    if (!DIRECT && g.fused && threadIdx.x == 0) ((uint64_t*)(problem_block(g, ws, p) + g.off_hand))[gq] = 0ull;     // (as below)
    return;
  }
  const int L = probs[p].L;
  if (L < 1 || L > g.max_L) return;                 // (the merge writes nothing for such a problem either)
  // The partial went out with GPU-coherent stores and the merge reads the partials with GPU-coherent loads.  Every wavefront waits
  // for its own stores before the barrier behind which thread 0 counts the workgroup in: the barrier itself waits for LDS
  // only, and at d = 128 the second wavefront's half of the sums could otherwise still be on its way when another XCD merges.
  // Only the optional export of the retrieved indices reads what ordinary stores of other workgroups wrote (the retrieved list):
  // then, and only then, device-wide fences (each writes back / invalidates a whole L2) bracket the count.
  const bool exports = probs[p].topk_idx != nullptr;
  if (exports) __threadfence();
  else if (g.sg_split > 1) wait_stores();
  __syncthreads();
  // (a head's only workgroup is its last, and need not ask memory: 0.6 us)
  if (g.sg_split > 1 && threadIdx.x == 0) {
    uint32_t* arrived = (uint32_t*)(problem_block(g, ws, p) + g.off_mcount) + gq;
    sh_last = atomicAdd(arrived, 1u) == (uint32_t)g.sg_split - 1u ? 1 : 0;
  }
  if (g.sg_split > 1) __syncthreads();
  if ((g.sg_split > 1 && !sh_last) || threadIdx.x >= kThreads) return;
  if (exports) __threadfence();
  // (the handed-over bound has been read: a replay of this call from a graph, whose tag is the same, must not find it)
  if (!DIRECT && g.fused && threadIdx.x == 0) ((uint64_t*)(problem_block(g, ws, p) + g.off_hand))[gq] = 0ull;
  merge_head<false, true>(g, probs, ws, gq, p, mode);
  }
}

void launch_select_gather(const Geom& g, const tkphi_problem* probs, char* ws, int mode, hipStream_t s) {
  dim3 grid(g.sg_split, g.Hq, g.n_problems);       // (Geom::n_tiles of this pipeline: one partial per workgroup)
  if (g.list) {
    const bool pack = g.sel_feat && g.max_K > 0 && g.max_mid > 0;
    grid = dim3(g.Hq + g.d_emb / 64 * g.Hq + (pack ? g.Hkv * std::max(1, 192 / g.Hkv) : 0));
  }
  const auto launch = [&](auto fn, int threads) { TKPHI_LAUNCH(ST_SELECT, fn, grid, dim3(threads), 0, s, g, probs, ws, mode); };
  // (the kernel of a head's only workgroup is one of its own: lists with the merge in it spill 57 to 64 scalars to vector registers, without it 15 to 17)
  const bool direct = g.direct, local = g.sg_split == 1;
#define TKPHI_SELECT(D, NTHR)                                                                                              \
  do {                                                                                                                     \
    if (direct && local) launch(select_gather_kernel<D, NTHR, true, false, true>, NTHR);                                   \
    else if (direct) launch(select_gather_kernel<D, NTHR, true, false, false>, NTHR);                                      \
    else if (local) launch(select_gather_kernel<D, NTHR, false, false, true>, NTHR);                                       \
    else launch(select_gather_kernel<D, NTHR, false, false, false>, NTHR);                                                 \
  } while (0)
  if (g.list) {
    if (g.d == 128) { if (direct) launch(select_gather_kernel<128, 1024, true, true, false>, 1024); else launch(select_gather_kernel<128, 1024, false, true, false>, 1024); }
    else { if (direct) launch(select_gather_kernel<64, 1024, true, true, false>, 1024); else launch(select_gather_kernel<64, 1024, false, true, false>, 1024); }
  } else if (g.dtype == TKPHI_F32) {
    if (local) launch(select_gather_kernel<64, 1024, true, false, true, float>, 1024);
    else launch(select_gather_kernel<64, 1024, true, false, false, float>, 1024);
  } else if (g.d == 128) TKPHI_SELECT(128, 1024);
  else if (g.sg_threads == 1024) TKPHI_SELECT(64, 1024);
  else if (direct) launch(select_gather_kernel<64, 512, true, false, true>, 512);        // (512 threads: sg_split is 1)
  else launch(select_gather_kernel<64, 512, false, false, true>, 512);
#undef TKPHI_SELECT
}

}  // namespace tkphi
