// Host layer of libtkphi: argument validation, launch geometry / workspace planning and
// the extern "C" entry points declared in include/tkphi.h.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>

#include "tkphi_internal.h"

namespace tkphi {

static thread_local char g_last_error[512] = "";
thread_local KernelTimer* g_kernel_timer = nullptr;

void set_error(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_last_error, sizeof(g_last_error), fmt, ap);
  va_end(ap);
}

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Entries of the compact part of a candidate list (a quarter of a chunk of scan_chunk tokens) for a budget of K in n: the expected
// number of its tokens above the sampled bound (estimated as for the smallest sample of 512 rows, whose bound is the
// loosest) and five standard deviations, no more than one sweep of the select kernel holds for every list, at least 24.
// Whatever the sweep has room for instead: 1 us slower at 32K and 52K (the entries are read whether they are filled or not);
// 24 for lists of 256 tokens: one overflows in most calls, and the select kernel takes 28 or 35 us instead of 23.
static int list_head(int scan_chunk, int64_t K, int64_t n, int sweep, int64_t n_chunks) {
  const double share = n <= 0 ? 0.0 : (double)K / (double)n, mu = 512.0 * share;
  const double mean = std::min(1.0, (mu + 5.0 * std::sqrt(mu) + 2.0) / 512.0) * scan_chunk / 4;
  const int want = (int)std::min<double>(mean + 5.0 * std::sqrt(mean) + 4.0, scan_chunk / 4);
  const int fit = (int)(sweep / (4 * n_chunks)) / kSweepEntries * kSweepEntries;
  return std::max(kMinListHead, std::min(fit, (int)align_up((size_t)want, kSweepEntries)));
}

// The filtered pipeline runs for budgets of at most 1 / (this number) of the mid-region.  Against the spill pipeline it saves the
// write-back of the scores, and pays for a larger budget with what one workgroup of its select kernel gathers alone.  Measured
// over 1000 combinations of shape, batch, length and budget (spill / filtered, us; the filtered side before sample and scores of one
// problem or a few went into one launch and the reductions off the LDS pipe, 12 to 18 us of a single layer: the lines may lie
// higher for those now):
//   * short contexts: always faster (1.07 to 1.6x)
//   * up to 1/64: as it always was (faster wherever the score pass lasts)
//   * beyond, where the select kernel's workgroups fill the last of their rounds over the 256 CUs to 4/5: up to 1/12 (3B layer
//     at 128K and 6 % 135 / 123; 28 3B sequences of 64K and 8 % 1530 / 1403); to 3/4: up to 1/16 (18 1B sequences of 40K, 576 heads:
//     4 % 352 / 349, 8 % 443 / 475); to 3/5 and long sequences: up to 1/25 (5 1B sequences of 40K, 160 heads: 2.8 % 114 / 98,
//     8 % 150 / 158; 11 3B sequences of 16K, 264 heads, the second round nearly empty: 2 % 147 / 149, 6 % 175 / 190);
//     512-thread workgroups, of which the next takes a CU's place as soon as one ends: up to 1/12
//   * not with fewer than 16 heads, which leave CUs without a workgroup, and more than 2048 retrieved (3 / 1 heads at 128K and
//     4 % 53 / 64), nor where the winners nearly fill the packed array (3B layer at 128K and 8 % 147 / 158: beyond it every
//     phase reads the lists again)
static int filtered_min_inverse_budget(bool short_context, int64_t heads, int split, int threads, int packed, int max_mid, int max_K) {
  if (short_context) return 12;
  if (max_K > packed / 5 * 4 || (heads < 16 && max_K > 2048)) return 64;
  const int64_t wgs = heads * split, slots = (wgs + 255) / 256 * 256;
  if (threads == 512 || heads < 16 || wgs * 5 >= slots * 4) return 12;
  return wgs * 4 >= slots * 3 ? 16 : wgs * 5 >= slots * 3 && max_mid > 32768 ? 25 : 64;
}

// What a call tries in turn until one fits its scratch memory.  kFast: the fastest.  kSeparate: where that is the one-launch score pass
// (Geom::fused), sample and score pass in two, whose chunks may fit where those do not.  kCompact: its needs grow with max_L, max_K and the
// number of problems (one chunk rule for all lengths, the filtered pipeline with its two full-length lists per head for budgets
// up to 1/64 only), so a workspace sized for larger bounds serves the smaller calls (but for a budget of at most 1/64 where the
// workspace was sized for one beyond 1/12).  For summary builds see make_geom.
enum Fit { kFast, kSeparate, kCompact };
// most_build_chunks: the partials of a KV head that a summary build has room for (0: as many as it likes)
static tkphi_status make_geom_as(const tkphi_config* cfg, int n_problems, int max_L, int max_K, Fit fit, bool diag, Geom* g, int64_t most_build_chunks = 0) {
  const bool compact = fit == kCompact;
  if (!cfg) { set_error("cfg is null"); return TKPHI_EINVAL; }
  if (n_problems < 0 || max_L < 1 || max_K < 0) {
    set_error("n_problems=%d max_L=%d max_K=%d out of range", n_problems, max_L, max_K);
    return TKPHI_EINVAL;
  }
  if (cfg->kv_dtype != TKPHI_F32 && cfg->kv_dtype != TKPHI_BF16) {
    set_error("kv_dtype=%d is not a tkphi_dtype", cfg->kv_dtype);
    return TKPHI_EINVAL;
  }
  if (cfg->n_kv_heads < 1 || cfg->n_q_heads < 1 || cfg->n_q_heads % cfg->n_kv_heads != 0 ||
      cfg->n_q_heads / cfg->n_kv_heads > kMaxGroup) {
    set_error("head counts %d/%d unsupported (need Hq %% Hkv == 0, ratio <= %d)", cfg->n_q_heads,
              cfg->n_kv_heads, kMaxGroup);
    return TKPHI_ESHAPE;
  }
  if (cfg->d_head != 64 && cfg->d_head != 128) {
    set_error("d_head=%d unsupported (64 or 128)", cfg->d_head);
    return TKPHI_ESHAPE;
  }
  if (cfg->d_phi < 16 || cfg->d_phi > kMaxDim || cfg->d_phi % 16 != 0) {
    set_error("d_phi=%d unsupported (multiple of 16 in [16, %d])", cfg->d_phi, kMaxDim);
    return TKPHI_ESHAPE;
  }
  if (cfg->phi_kind != TKPHI_PHI_EXP_AFFINE && cfg->phi_kind != TKPHI_PHI_MLP) {
    set_error("phi_kind=%d is not a tkphi_phi_kind", cfg->phi_kind);
    return TKPHI_EINVAL;
  }
  if (cfg->phi_kind == TKPHI_PHI_MLP) {
    if (cfg->kv_dtype != TKPHI_BF16) {
      set_error("the MLP feature maps need bf16 storage");
      return TKPHI_EUNSUPPORTED;
    }
    if (cfg->d_emb < 64 || cfg->d_emb > 1024 || (cfg->d_emb & (cfg->d_emb - 1)) != 0) {
      set_error("d_emb=%d unsupported (a power of two in [64, 1024])", cfg->d_emb);
      return TKPHI_ESHAPE;
    }
    // decode recomputes retrieved-key features with the one-launch chain only (the widths it is built for)
    const bool chain_widths = (cfg->d_emb == 128 || cfg->d_emb == 256 || cfg->d_emb == 512) && cfg->d_phi <= 256;
    if (!cfg->cache_features && !chain_widths) {
      set_error("the MLP feature maps without cache_features need d_emb in {128, 256, 512} and d_phi <= 256 "
                "(d_emb=%d, d_phi=%d)", cfg->d_emb, cfg->d_phi);
      return TKPHI_EUNSUPPORTED;
    }
  }
  if (cfg->max_gen < 0 || cfg->max_gen > (1 << 20)) { set_error("max_gen=%d out of range [0, 2^20]", cfg->max_gen); return TKPHI_EINVAL; }
  const tkphi_tuning& tn = cfg->tuning;
  if (tn.force_generic < 0 || tn.force_generic > 1 || tn.scan_chunk < 0 || tn.scan_chunk > 32768 || tn.interleave < 0 ||
      tn.interleave > 2 || tn.build_chunk < 0 || tn.build_chunk > (1 << 20) || tn.mlp_block < 0 || tn.mlp_block > 8192 ||
      tn.mlp_mode < 0 || tn.mlp_mode > 2 || tn.select_mode < 0 || tn.select_mode > 2 || tn.select_test < 0 || tn.select_test > 2) {
    set_error("tuning field out of range (force_generic=%d scan_chunk=%d interleave=%d build_chunk=%d mlp_block=%d mlp_mode=%d "
              "select_mode=%d select_test=%d)", tn.force_generic, tn.scan_chunk, tn.interleave, tn.build_chunk, tn.mlp_block,
              tn.mlp_mode, tn.select_mode, tn.select_test);
    return TKPHI_EINVAL;
  }
  for (int i = 0; i < 4; ++i)
    if (tn.reserved[i] != 0) { set_error("tuning.reserved[%d] must be 0", i); return TKPHI_EINVAL; }
  if (n_problems > 65535) { set_error("n_problems=%d exceeds 65535", n_problems); return TKPHI_ESHAPE; }
  if (cfg->n_sink < 0 || cfg->n_tail < 0) {
    set_error("n_sink=%d n_tail=%d must be >= 0", cfg->n_sink, cfg->n_tail);
    return TKPHI_EINVAL;
  }
  memset(g, 0, sizeof(*g));
  g->Hq = cfg->n_q_heads; g->Hkv = cfg->n_kv_heads; g->G = g->Hq / g->Hkv;
  g->d = cfg->d_head; g->dphi = cfg->d_phi; g->n_sink = cfg->n_sink; g->n_tail = cfg->n_tail;
  g->dtype = cfg->kv_dtype;
  g->cache = cfg->cache_features ? 1 : 0;
  g->phi_kind = cfg->phi_kind; g->d_emb = cfg->d_emb;
  g->max_gen = cfg->max_gen;
  g->mlp_mode = tn.mlp_mode;
  g->use_mfma = (cfg->kv_dtype == TKPHI_BF16 && cfg->d_phi == cfg->d_head && !tn.force_generic) ? 1 : 0;
  g->n_problems = n_problems; g->max_L = max_L;
  const int64_t mid = (int64_t)max_L - cfg->n_sink - cfg->n_tail;
  g->max_mid = (int)std::max<int64_t>(mid, 0);
  g->max_K = max_K;
  g->mid_stride = (int)align_up((size_t)std::max(g->max_mid, 1), 64);
  g->score_scale = cfg->score_scale; g->a = cfg->phi_in_scale; g->c = cfg->phi_norm_coef;

  const int64_t units = (int64_t)g->max_mid * g->Hkv * std::max(n_problems, 1);
  // fused select + gather kernel of the filtered pipeline: the workgroups that share a query head, one partial each (about one
  // workgroup per CU for a single layer, one per head in big batches); batches of short sequences at d = 64 (one workgroup
  // per head, at least two heads per CU) take 512-thread workgroups, two per CU, so that one head's memory round trips
  // hide behind the other's arithmetic
  const int64_t heads = (int64_t)g->Hq * std::max(n_problems, 1);
  const int max_split = (int)std::clamp<int64_t>(256 / heads, 1, 16);
  g->sg_threads = cfg->kv_dtype == TKPHI_BF16 && g->d == 64 && max_split == 1 && (int64_t)g->Hq * n_problems >= 512 && max_K <= 1024 ? 512 : 1024;
  const int sweep = g->sg_threads * kSweepEntries;   // candidate slots of a head that kernel reads in one go
  const int packed = packed_candidates(g->d, g->sg_threads);
  const bool short_context = !compact && tn.scan_chunk == 0 && tn.select_test == 0 && g->max_mid <= std::min(sweep, packed);
  const int min_inverse_budget = compact ? 64 : filtered_min_inverse_budget(short_context, heads, max_split, g->sg_threads, packed, g->max_mid, max_K);
  // (a step with the diagnostics runs the spill pipeline; of one problem also on its chunks: on the few long ones that the
  // filtered pass likes a 3B layer at 128K took 107.5 us instead of 101.5, batches are as fast or faster on theirs)
  g->diag = diag ? 1 : 0;
  g->filtered = (g->use_mfma && cfg->phi_kind == TKPHI_PHI_EXP_AFFINE && !g->cache && tn.select_mode != 1 && !(diag && n_problems <= 1) &&
                 (tn.select_mode == 2 || (int64_t)max_K * min_inverse_budget <= g->max_mid)) ? 1 : 0;
  // fp32 caches at d = d_phi = 64, short contexts: the two launches of the filtered pipeline instead of six.  (At d = 128 Wk in fp32 and the
  // packed array do not fit LDS together.)
  if (cfg->kv_dtype == TKPHI_F32 && g->d == 64 && g->dphi == 64 && cfg->phi_kind == TKPHI_PHI_EXP_AFFINE && !g->cache && !diag && short_context &&
      g->max_mid > 0 && !tn.force_generic && tn.select_mode != 1 && (int64_t)max_K * 12 <= g->max_mid)
    g->filtered = 1;
  // MLP maps: one problem (Geom::fused, below, or short contexts), and budgets whose winners leave the packed array some room; one workgroup per head then selects in 15 us what plan, emit and resolve took 26 for (3B layer at 128K)
  g->list = (g->use_mfma && cfg->phi_kind == TKPHI_PHI_MLP && g->max_mid > 0 && !compact && !diag && tn.select_mode != 1 && n_problems <= 1 &&
             (tn.select_mode == 2 || ((int64_t)max_K * 12 <= g->max_mid && max_K <= packed / 5 * 4))) ? 1 : 0;
  // matrix-core score kernel: 4 wavefronts x 64 (d = 128) or 128 (d = 64) tokens per iteration;
  // a chunk is a whole number of such units
  g->scan_unit = g->use_mfma ? (g->d == 128 ? 256 : 512) : 256;
  // spill pipeline: about 1024 workgroups, 256..8192 tokens each (uint16 chunk histograms: < 65536)
  int sc = (int)align_up((size_t)std::clamp<int64_t>(ceil_div(units, 1024), 256, 8192), 256);
  // Filtered pipeline, one or a few problems: sample and score pass in one launch, whose workgroups hold the scores of their chunk in
  // LDS (two workgroups per CU: half of it, of which 2 KB are left for what else the kernel holds; with one per CU the sample, phi and
  // anchor workgroups hold CUs that as many score workgroups wait for: 1B layer at 128000 tokens 48 us instead of 45, 64 / 8 heads
  // of 64 at 100000 tokens 55 instead of 48).  One problem: the pass lasts as long as its busiest CU and wants one
  // workgroup on each.  A few (ragged: up to half of the chunks that the bounds allow for are empty): about 1024 workgroups.  At most
  // 128 chunks per KV head (one sweep of the select kernel).  Two launches / one, us per step: 3B layer at 16K 41 / 35, 50K 56 / 48,
  // 128K 84 / 77; 1B layer at 32K 37.5 / 34, 96K 52 / 43; 1B sequences of 4K to 16K, 2 of them 35 / 32, 4 of them 50 / 42; 2 3B
  // sequences of 32K to 64K 75 / 70.  Beyond 32 KV heads the sample is a small part and the workgroups that wait for it cost more:
  // 8 3B sequences of 16K to 64K 193 / 200, 16 1B ones 206 / 224.
  const int unit = keep_unit(g->d), keep_most = 79872 / (g->G * (int)sizeof(float)) / unit * unit;
  int64_t keep_chunk = ceil_div(g->max_mid, std::clamp(256 / g->Hkv, 1, 128));
  if (n_problems > 1)
    for (keep_chunk = 1024; keep_chunk * 1024 < units || ceil_div(g->max_mid, keep_chunk) > 128;) keep_chunk *= 2;
  keep_chunk = std::min<int64_t>(align_up((size_t)std::max<int64_t>(keep_chunk, 1), unit), keep_most);
  int64_t given = (int64_t)align_up((size_t)tn.scan_chunk, unit);        // (one too short for the bounds grows, below)
  while (tn.scan_chunk > 0 && ceil_div(g->max_mid, given) > kMaxScanChunks && given < 32768) given *= 2;
  const bool fusable = (g->filtered || g->list) && !compact && !diag && !short_context && (n_problems <= 1 || (int64_t)g->Hkv * n_problems <= 32) &&
                       (tn.scan_chunk > 0 ? given <= keep_most : ceil_div(g->max_mid, keep_chunk) <= 128);
  g->fused = fusable && fit == kFast ? 1 : 0;
  if (g->list && (g->fused || short_context)) g->filtered = 1;
  g->list = g->list && g->filtered;
  if (g->fused) {
    g->scan_unit = unit;
    sc = (int)keep_chunk;
  } else if (g->filtered && !compact && n_problems <= 1) {
    // One problem of more than 128 kept chunks per KV head (64 / 8 heads from 320 K tokens, 24 / 8 from 850 K), or kSeparate: the
    // pass takes as long as its busiest CU, so the chunk is chosen for full rounds of 256 workgroups (score pass of a 3B
    // layer at 50 K tokens: 232 workgroups of 1792 tokens 22.4 us, 400 of 1024 25.0, 312 of 1280 29.2); one workgroup per CU
    // streams 7 % slower at d = 128 and, with 2.7 times the score work per byte, 40 % at d = 64.  Against that stands what the
    // select kernel pays for more lists: 0.35 us per 1000 slots of their compact heads.
    const double ideal_us = (double)units * g->d * 2 / 6.2e6;
    double best = 0.0;
    for (int c = g->scan_unit; c <= 8192; c += g->scan_unit) {
      const int64_t chunks = std::max<int64_t>(1, ceil_div(g->max_mid, c)), rounds = ceil_div(chunks * g->Hkv, 256);
      if (chunks * 4 * kMinListHead > sweep && c + g->scan_unit <= 8192) continue;
      const double eff = (double)units / ((double)rounds * 256 * c) * (rounds > 1 ? 1.0 : g->d == 128 ? 0.93 : 0.7);
      const double cost = ideal_us / eff + 0.35e-3 * (double)(chunks * 4 * list_head(c, std::min<int64_t>(max_K, g->max_mid), g->max_mid, sweep, chunks));
      if (best == 0.0 || cost <= best) { best = cost; sc = c; }
    }
  } else if (g->filtered && !compact) {
    // Filtered pipeline, batches: 4096 workgroups by the bounds of the call, a power of two of tokens each.  Ragged batches have
    // far fewer, which then still even out over the CUs (8 sequences of 8K to 32K at d = 128: score pass 74 -> 58 us against a
    // target of 1024, 16 of 16K to 64K at d = 64: 168 -> 152).  At most 4096 tokens where sequences may be longer than 32K: a
    // workgroup of 8192 that starts last alone on its CU ends 30 us late (64 sequences of 16K to 64K: step 743 -> 708 us at
    // d = 64, 1364 -> 1280 at d = 128; 28 of 128K, where the last round is full: 1472 -> 1486), below that at most 8192 (200 of
    // 16K: 966 against 990 us with 4096).
    const int most = g->max_mid > 32768 ? 4096 : 8192;
    sc = 256;
    while (sc < most && (int64_t)sc * 4096 < units) sc *= 2;
    while (sc < 32768 && ceil_div(g->max_mid, std::max(sc, g->scan_unit)) * 4 * kMinListHead > sweep) sc *= 2;
  }
  if (tn.scan_chunk > 0) sc = tn.scan_chunk;
  // Short contexts, as long as every token fits one sweep and the packed array of the select kernel: one unit per chunk, all
  // scores stored, no bound and no prep launch (1B layer at 4K 34.5 -> 22.6 us, at 10K 34.9 -> 24.6; 3B layer 34.6 -> 26.0 and 37.5 -> 31.8).  Few
  // winners then, and what workgroups of a head hand each other costs more than a gather round: one per 64 of the budget, and a single
  // one, which merges its head out of LDS, up to 128 of a bf16 cache (1B layer at 4K 3 % 18.1 -> 16.7 us, at 12K 1 % 23.7 -> 23.1, 3B layer at
  // 2K 4 % 19.6 -> 18.6, at 5K 2 % 22.0 -> 21.2; 170 of the 3B layer at 8.5K would lose: 25.0 -> 25.6, and 75 fp32 rows of four
  // times the matrix instructions: 24.2 -> 24.8)
  g->sg_split = g->filtered ? g->list ? 1 : max_split : 0;
  g->direct = g->filtered && short_context ? 1 : 0;
  if (g->direct) {
    if (cfg->kv_dtype == TKPHI_F32) g->scan_unit = direct_unit_f32;
    sc = g->scan_unit;
    const int most_K = (int)std::min<int64_t>(max_K, g->max_mid), alone = cfg->kv_dtype == TKPHI_F32 ? 64 : 128;
    g->sg_split = most_K <= alone ? 1 : std::min(g->sg_split, (int)ceil_div(most_K, 64));
  }
  g->scan_chunk = std::clamp((int)align_up((size_t)std::max(sc, 1), g->scan_unit), g->scan_unit, 32768);
  while (ceil_div(g->max_mid, g->scan_chunk) > kMaxScanChunks && g->scan_chunk < 32768) g->scan_chunk *= 2;
  if (ceil_div(g->max_mid, g->scan_chunk) > kMaxScanChunks) {
    set_error("max_L=%d too long: more than %d score chunks of 32768 tokens", max_L, kMaxScanChunks);
    return TKPHI_ESHAPE;
  }
  g->n_scan_chunks = (int)std::max<int64_t>(1, ceil_div(g->max_mid, g->scan_chunk));
  // with many chunks per head (one long sequence) the workgroups read neighbouring rows at any
  // moment instead of far-apart ranges (3B layer at 128K: 47.9 against 49.5 us); with few chunks per head or
  // several problems contiguous ranges are as fast or faster (16 ragged sequences at d = 64, chunks of 1024: 137 against 153 us)
  g->interleave = tn.interleave ? (tn.interleave == 1 ? 1 : 0)
                                : (g->use_mfma && g->scan_unit < g->scan_chunk && (g->fused || (g->n_scan_chunks >= 64 && (n_problems == 1 || !g->filtered)))) ? 1 : 0;
  if (!g->use_mfma || g->scan_unit >= g->scan_chunk) g->interleave = 0;
  // The filtered score pass reads keys of more than 64 MB (by the bounds) with non-temporal loads of whole lines (score_tile.h): 256
  // ragged sequences 2857 -> 2653 us per step, 16 208 -> 188, the 3B layer at 128K 73.4 -> 69.3, at 48K 42.3 -> 41.9; less than that is
  // served from the caches to the select kernel's gather: 1B layer at 32K 28.2 -> 28.9.
  g->stream_keys = units * g->d * 2 > ((int64_t)64 << 20) ? 1 : 0;
  g->sel_test = tn.select_test;
  // gather: tiles of kPairsPerWG retrieved tokens per query head
  g->n_tiles = (int)ceil_div(std::min<int64_t>(max_K, g->max_mid), kPairsPerWG);
  g->n_atiles = (int)std::max<int64_t>(1, ceil_div(std::min<int64_t>((int64_t)cfg->n_sink + cfg->n_tail, max_L) + cfg->max_gen, 64));
  // summary_build: 512 workgroups fill the chip (2 per CU); larger jobs get about 2048 chunks of at
  // least 2048 tokens so that the last, partly filled round of workgroups stays a small share.  The fp32-arithmetic
  // kernel spends 32 times the bf16 one's time on a token: there a workgroup takes as little as one tile of 64
  const bool f32_build = !g->use_mfma && cfg->phi_kind == TKPHI_PHI_EXP_AFFINE;
  // One problem at d = 64: one workgroup per CU (the wavefronts have no barrier to hide, and half the workgroups leave half the
  // partials: 20K 17.2 -> 15.2 us, 32K 21.3 -> 20.0, 128K 51.7 -> 49.5).  Several: two per CU, whether their lengths differ or not, which the
  // bounds do not tell (3 ragged ones of 5K to 20K: two per CU 24.4, one 26.6; 2 of 32K: two 31.3, one 28.2)
  const bool one_per_cu = g->use_mfma && cfg->phi_kind == TKPHI_PHI_EXP_AFFINE && g->d == 64 && n_problems == 1;
  // Short layers at d = 128 too, as long as its tiles of four wavefronts (0.9 us each) weigh more than its partials of 66 KB: up to 384 tokens a
  // chunk for one workgroup per CU (8 KV heads: 7K tokens 23.6 -> 22.2 us, 9K 28.6 -> 24.2, 12K 30.6 -> 27.6; 16K in chunks of 384 33.1
  // against 32.7 with two per CU), but chunks of up to 192 for about 200 workgroups (of 64: 160), since the reduction adds a head's partials one behind
  // the other (8 KV heads: 3K 19.4 -> 16.8, 1.5K in chunks of 64 15.0 and of 128 14.2 against 18.1; 1 KV head: 16K in chunks of 64
  // 19.0 and of 128 15.5 against 17.9, 32K in chunks of 128 21.2 and of 192 19.7 against 20.7)
  const bool short_layer = g->use_mfma && cfg->phi_kind == TKPHI_PHI_EXP_AFFINE && g->d == 128 && !compact;
  const int64_t per_cu = ceil_div(units, 256), two_per_cu = ceil_div(units, 512);
  const int64_t bc_small = one_per_cu ? std::clamp<int64_t>(per_cu, 256, 4096)
                           : short_layer ? (per_cu <= 384 ? std::max(per_cu, std::clamp<int64_t>(ceil_div(units, 208), units <= 160 * 64 ? 64 : 128, 192)) : std::clamp<int64_t>(two_per_cu, 256, 2048))
                                         : std::clamp<int64_t>(two_per_cu, f32_build && !compact ? 64 : 256, 2048);
  int bc = (int)align_up((size_t)std::clamp<int64_t>(ceil_div(units, 2048), bc_small, 1 << 20), 64);
  if (!g->use_mfma) bc = std::min(bc, 4096);    // fp32 FMA chains stay short on the generic kernel
  // Several resident rounds of the matrix-core kernel (512 workgroup slots): among the
  // chunk counts within two of that guess, the one whose last round is fullest (28 layers of 128K: 9 chunks per head
  // = 2016 workgroups = 3.94 rounds instead of 10 = 4.375, which pays for 5)
  if (g->use_mfma && cfg->phi_kind == TKPHI_PHI_EXP_AFFINE && g->max_mid > 0) {
    const int64_t slots = one_per_cu ? 256 : 512, heads = (int64_t)g->Hkv * std::max(n_problems, 1);
    const int64_t c0 = ceil_div(g->max_mid, bc);
    if (c0 * heads > slots) {
      double best_fill = -1.0;
      int best_bc = bc;
      for (int64_t c = std::max<int64_t>(1, c0 - 2); c <= c0 + 2; ++c) {
        const int cand = (int)align_up((size_t)std::max<int64_t>(256, ceil_div(g->max_mid, c)), 64);
        const int64_t wgs = ceil_div(g->max_mid, cand) * heads;
        const double fill = (double)wgs / (double)(ceil_div(wgs, slots) * slots);
        if (fill > best_fill + 1e-9 || (std::fabs(fill - best_fill) <= 1e-9 && std::abs(cand - bc) < std::abs(best_bc - bc))) {
          best_fill = fill; best_bc = cand;
        }
      }
      bc = best_bc;
    }
  }
  if (most_build_chunks > 0) bc = std::max(bc, (int)align_up((size_t)ceil_div(g->max_mid, most_build_chunks), 64));
  if (tn.build_chunk > 0) bc = tn.build_chunk;
  g->build_chunk = std::max(64, bc / 64 * 64);
  g->n_build_chunks = (int)std::max<int64_t>(1, ceil_div(g->max_mid, g->build_chunk));
  g->part_stride = 2 * g->d + 4;

  // workspace layout
  size_t off = 0;
  g->off_status = off; off += 4096;
  g->off_problem0 = off;
  size_t p = 0;
  g->off_scores = p;
  g->off_candf = p;     // (the two pipelines never run in the same call)
  // The second set of candidate lists, which a rescan writes while other workgroups of the head may still read the first, is the
  // first one where a head has one workgroup: a batch of 256 sequences of 50K at 2 % needs 4.4 GB so, 8.2 with two sets (the
  // spill pipeline 2.1).  (The compact geometry keeps the room; short contexts have no lists, but keep it too, so that the
  // reported size stays the smallest accepted for one problem.)
  const size_t lists = g->filtered ? (size_t)g->Hq * g->n_scan_chunks : 0;
  const bool one_set = !compact && max_split == 1;
  p = align_up(p + std::max((size_t)g->Hq * g->mid_stride * sizeof(float), lists * g->scan_chunk * sizeof(uint2)), 256);
  g->cand_T = compact || !g->filtered || g->direct ? (int)align_up((size_t)std::max(kMinListHead, g->scan_chunk / 4 * 3 / 32), kSweepEntries)
                                      : list_head(g->scan_chunk, std::min(max_K, g->max_mid), g->max_mid, sweep, g->n_scan_chunks);
  g->head_strip = (size_t)4 * g->G * g->cand_T * sizeof(uint2) <= 32768 ? 1 : 0;
  g->off_candc = p;   p = align_up(p + lists * 4 * g->cand_T * sizeof(uint2), 256);
  g->off_ccount = p;  p = align_up(p + lists * 4 * sizeof(uint32_t), 256);
  if (one_set) {
    g->off_resf = g->off_candf; g->off_resc = g->off_candc; g->off_rescount = g->off_ccount;
  } else {
    g->off_resf = p;    p = align_up(p + lists * g->scan_chunk * sizeof(uint2), 256);
    g->off_resc = p;    p = align_up(p + lists * 4 * g->cand_T * sizeof(uint2), 256);
    g->off_rescount = p; p = align_up(p + lists * 4 * sizeof(uint32_t), 256);
  }
  g->off_thr = p;     p = align_up(p + (size_t)g->Hq * sizeof(uint32_t), 256);
  g->off_mcount = p;  p = align_up(p + (size_t)g->Hq * sizeof(uint32_t), 256);
  g->off_sphi = p;    p = align_up(p + (size_t)g->Hq * g->d * sizeof(float), 256);
  g->off_uphi = p;    p = align_up(p + (size_t)g->Hq * sizeof(float), 256);
  g->off_hist = g->off_hand = p;    p = align_up(p + (size_t)g->n_scan_chunks * g->Hq * kBins * sizeof(uint16_t), 256);
  g->off_plan = p;    p = align_up(p + (size_t)g->Hq * sizeof(SelPlan), 256);
  g->off_diag = p;    p = align_up(p + (size_t)g->n_scan_chunks * g->Hq * 4 * sizeof(float), 256);
  g->off_chunkoff = p; p = align_up(p + (size_t)g->Hq * g->n_scan_chunks * 2 * sizeof(int32_t), 256);
  g->off_cand = p;    p = align_up(p + (size_t)g->Hq * kCandCap * sizeof(uint2), 256);
  g->off_selidx = p;  p = align_up(p + (size_t)g->Hq * std::max(max_K, 1) * sizeof(int32_t), 256);
  g->off_selscore = p; p = align_up(p + (size_t)g->Hq * std::max(max_K, 1) * sizeof(float), 256);
  g->off_phiq = p;    p = align_up(p + (size_t)g->Hq * g->dphi * sizeof(float), 256);
  g->off_mlpq = p;    p = align_up(p + (size_t)g->Hq * 2 * g->d_emb * sizeof(float), 256);
  g->sel_feat = cfg->phi_kind == TKPHI_PHI_MLP && !g->cache;
  g->off_selphi = p;  p = align_up(p + (g->sel_feat ? (size_t)g->Hq * std::max(max_K, 1) * g->dphi * sizeof(float) : (size_t)0), 256);
  g->off_part = p;
  p = align_up(p + (size_t)g->Hq * (std::max(g->n_tiles, g->filtered ? max_split : 0) + g->n_atiles) * g->part_stride * sizeof(float), 256);
  if (p >> 40) {                       // (WsOffset; no GPU holds it)
    set_error("scratch of one problem beyond 1 TB (max_L=%d max_K=%d)", max_L, max_K);
    return TKPHI_ESHAPE;
  }
  g->per_problem = p;
  const size_t decode_total = g->off_problem0 + (size_t)std::max(n_problems, 1) * g->per_problem;
  size_t decode_all = decode_total;
  g->off_bpart = g->off_problem0;
  const size_t build_total = g->off_bpart + (size_t)std::max(n_problems, 1) * g->Hkv * g->n_build_chunks *
                                                (size_t)g->dphi * (g->d + 1) * sizeof(float);
  size_t build_all = build_total;
  if (cfg->phi_kind == TKPHI_PHI_MLP) {
    // the fp32 activations of a token block (g and h, every KV head) are written by one GEMM launch and
    // read by the next: a block of about 64 MB stays in the 256 MB last-level cache between the
    // launches, but a launch should also bring two 64-token workgroups per CU (512 in all), which
    // measured faster than the smaller block (4.6 against 6.5 ms for 8 KV heads of 131004 tokens)
    const int64_t blk = std::max<int64_t>(((int64_t)64 << 20) / ((int64_t)2 * g->Hkv * g->d_emb * sizeof(float)),
                                          (int64_t)512 * 64 / g->Hkv);
    g->mlp_block = (int)std::clamp<int64_t>((tn.mlp_block > 0 ? tn.mlp_block : (int)blk) / 64 * 64, 64, 8192);
    // (the activations, the packed weights and the feature buffer lie behind the decode blocks as well: a decode
    // without a feature cache sends the retrieved keys through the same chain)
    g->off_act = align_up(std::max(build_total, decode_total), 256);
    // (the one-launch chain keeps its activations on chip)
    const bool chain_build = tn.mlp_mode == 0 && (cfg->d_emb == 128 || cfg->d_emb == 256 || cfg->d_emb == 512) &&
                             (g->dphi == 64 || g->dphi == 128 || g->dphi == 256);
    const size_t act_bytes = chain_build ? 0 : (size_t)2 * g->Hkv * g->mlp_block * g->d_emb * sizeof(float);
    g->off_wpack = align_up(g->off_act + act_bytes, 256);
    // Problems per chain launch: their packed weights (and, without a feature cache, the features of their
    // mid-regions, fp32) are held together; up to 16 problems, the feature buffer at most 1 GiB (one problem if a
    // single one is larger).
    const size_t wpack_one = (size_t)g->Hkv * ((size_t)g->d_emb * g->d + (size_t)2 * g->d_emb * g->d_emb + (size_t)g->dphi * g->d_emb) * 2;
    const size_t feat_one = g->cache ? 0 : (size_t)g->Hkv * std::max<int64_t>(g->max_mid, 1) * g->dphi * sizeof(float);
    g->mlp_group = std::clamp(n_problems, 1, 16);
    if (feat_one > 0) g->mlp_group = (int)std::clamp<size_t>(((size_t)1 << 30) / feat_one, 1, (size_t)g->mlp_group);
    g->off_feat = align_up(g->off_wpack + (size_t)g->mlp_group * wpack_one, 256);
    build_all = g->off_feat + (size_t)g->mlp_group * feat_one;
    if (g->sel_feat) decode_all = g->off_feat;          // (up to the end of the packed weights)
  }
  g->decode_bytes = align_up(decode_all, 256);
  g->build_bytes = align_up(build_all, 256);
  g->total_bytes = align_up(std::max(decode_all, build_all), 256);
  return TKPHI_OK;
}

// have / need: the scratch bytes that the caller has and the member that says what its call takes (null: no limit).
// A summary build takes as many chunks as the scratch has room for, down to a quarter of the compact geometry's.  The number of chunks that its rules
// choose (whole rounds of workgroups) goes up and down with the length and the number of problems, by less than that, so a workspace sized for
// larger bounds serves the smaller builds too (MLP maps without a feature cache aside, whose problems per launch change as well).
tkphi_status make_geom(const tkphi_config* cfg, int n_problems, int max_L, int max_K, Geom* g, size_t have, size_t Geom::*need, bool diag) {
  int64_t least_chunks = 0;
  for (const Fit fit : {kFast, kSeparate, kCompact}) {
    tkphi_status st = make_geom_as(cfg, n_problems, max_L, max_K, fit, diag, g);
    if (st != TKPHI_OK || !need || g->*need <= have) return st;
    if (need != &Geom::build_bytes) continue;
    if (least_chunks == 0) {
      Geom compact;
      st = make_geom_as(cfg, n_problems, max_L, max_K, kCompact, diag, &compact);
      if (st != TKPHI_OK) return st;
      least_chunks = ceil_div(compact.n_build_chunks, 4);
    }
    const size_t chunk_bytes = (size_t)std::max(n_problems, 1) * g->Hkv * g->dphi * (g->d + 1) * sizeof(float);      // of every KV head
    const int64_t fit_chunks = g->n_build_chunks - (int64_t)std::min<size_t>((g->build_bytes - have + chunk_bytes - 1) / chunk_bytes, g->n_build_chunks);
    if (fit_chunks < least_chunks) continue;
    st = make_geom_as(cfg, n_problems, max_L, max_K, fit, diag, g, fit_chunks);
    if (st != TKPHI_OK || g->build_bytes <= have) return st;
  }
  return TKPHI_OK;                     // (the caller sees what the last one needs)
}

static tkphi_status check_call(const tkphi_problem* problems, int n_problems, const void* ws,
                               size_t ws_bytes, const Geom& g, size_t need = 0) {
  if (need == 0) need = g.total_bytes;
  if (n_problems > 0 && !problems) { set_error("problems is null"); return TKPHI_EINVAL; }
  if (!ws) { set_error("workspace is null"); return TKPHI_EWORKSPACE; }
  if (((uintptr_t)ws) % 256 != 0) { set_error("workspace must be 256-byte aligned"); return TKPHI_EWORKSPACE; }
  if (ws_bytes < need) {
    set_error("workspace too small: %zu < %zu bytes", ws_bytes, need);
    return TKPHI_EWORKSPACE;
  }
  if (((uintptr_t)problems) % 8 != 0) { set_error("problem table must be 8-byte aligned"); return TKPHI_EALIGN; }
  return TKPHI_OK;
}

static tkphi_status hip_ok(hipError_t e, const char* what) {
  if (e == hipSuccess) return TKPHI_OK;
  set_error("%s: %s", what, hipGetErrorString(e));
  return TKPHI_EHIP;
}

}  // namespace tkphi

using namespace tkphi;

extern "C" {

size_t tkphi_workspace_bytes(const tkphi_config* cfg, int32_t n_problems, int32_t max_L, int32_t max_K) {
  Geom g;
  if (make_geom(cfg, n_problems, max_L, max_K, &g) != TKPHI_OK) return 0;
  size_t bytes = 0;
  // enough for the compact geometry too, which a call with smaller bounds may fall back to, for a step with the diagnostics (other
  // chunks), and for the largest number of problems whose heads have two workgroups (and two sets of candidate lists): it may need
  // more than a few problems beyond it
  const int fewer = std::min(n_problems, 128 / cfg->n_q_heads);
  for (int n : {n_problems, fewer})
    for (bool diag : {false, true})
      for (Fit fit : {kFast, kCompact}) {
        if (make_geom_as(cfg, n, max_L, max_K, fit, diag, &g) != TKPHI_OK) return 0;
        bytes = std::max(bytes, g.total_bytes);
      }
  return bytes;
}

tkphi_status tkphi_build_summaries(const tkphi_config* cfg, const tkphi_problem* problems,
                                   int32_t n_problems, int32_t max_L, void* workspace,
                                   size_t workspace_bytes, void* hip_stream) {
  Geom g;
  tkphi_status st = make_geom(cfg, n_problems, max_L, 0, &g, workspace_bytes, &Geom::build_bytes);
  if (st != TKPHI_OK) return st;
  st = check_call(problems, n_problems, workspace, workspace_bytes, g, g.build_bytes);   // (the decode scratch depends on max_K)
  if (st != TKPHI_OK) return st;
  if (n_problems == 0) return TKPHI_OK;
  hipStream_t s = (hipStream_t)hip_stream;
  (void)hipGetLastError();
  launch_build(g, problems, (char*)workspace, s);
  return hip_ok(hipGetLastError(), "tkphi_build_summaries launch");
}

// The kernels of one decode call in stream order.  With the MLP feature maps the three phi_q
// launches of several problems (a chain of small cold-weight matrix-vector products, ~30 us if serialised) go to a
// second stream of the library's own that forks from `s` at the start of the call and joins
// before the gather, so that they run beside the score pass (one problem: Geom::list).  One such stream and event pair per
// device, created on first use at the default priority and kept until the process ends; MLP decode
// calls hold a mutex while they enqueue (the events are shared).
struct SideStream {
  hipStream_t stream = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
};
static std::mutex g_side_mutex;
static SideStream g_side[64];

static tkphi_status side_stream(SideStream** out) {
  int dev = 0;
  tkphi_status st = hip_ok(hipGetDevice(&dev), "hipGetDevice");
  if (st != TKPHI_OK) return st;
  if (dev < 0 || dev >= 64) { set_error("device ordinal %d out of range", dev); return TKPHI_EINVAL; }
  SideStream& ss = g_side[dev];
  if (!ss.stream) {
    hipStream_t str = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    st = hip_ok(hipStreamCreateWithFlags(&str, hipStreamNonBlocking), "hipStreamCreateWithFlags");
    if (st == TKPHI_OK) st = hip_ok(hipEventCreateWithFlags(&e0, hipEventDisableTiming), "hipEventCreateWithFlags");
    if (st == TKPHI_OK) st = hip_ok(hipEventCreateWithFlags(&e1, hipEventDisableTiming), "hipEventCreateWithFlags");
    if (st != TKPHI_OK) {
      if (e0) (void)hipEventDestroy(e0);
      if (e1) (void)hipEventDestroy(e1);
      if (str) (void)hipStreamDestroy(str);
      return st;
    }
    ss.stream = str; ss.fork = e0; ss.join = e1;
  }
  *out = &ss;
  return TKPHI_OK;
}

// Marks the bounds that one call's sample workgroups hand to its score workgroups: another one for every call, spread over 32
// bits so that what other calls leave in the same scratch memory is not taken for it, never 0 (what a finished call leaves)
static uint32_t next_tag() {
  static std::atomic<uint32_t> calls{0};
  uint32_t x = calls.fetch_add(1, std::memory_order_relaxed);
  x = (x ^ 0x5bd1e995u) * 0x9e3779b1u;               // (one to one)
  x ^= x >> 15;
  return x ? x : 0x9e3779b1u;
}

static tkphi_status enqueue_decode(const Geom& g, const tkphi_problem* problems, char* ws, int acct, hipStream_t s) {
  const bool filtered = g.filtered && !g.diag;         // (the diagnostics are by-products of the spill pipeline's emit pass)
  const auto launch_filtered = [&](Geom gf) {
    if (!gf.list) gf.n_tiles = gf.sg_split;            // one partial per workgroup of the fused select + gather kernel
    if (gf.direct) {
      launch_score_direct(gf, problems, ws, s);
    } else if (gf.fused) {
      gf.tag = next_tag();
      launch_score_fused(gf, problems, ws, s);
    } else {
      launch_prep(gf, problems, ws, s);
      launch_score_filtered(gf, problems, ws, s);
    }
    launch_select_gather(gf, problems, ws, acct, s);   // (Geom::list aside its last workgroup per head merges)
  };
  if (filtered && !g.list) {
    launch_filtered(g);
    return TKPHI_OK;
  }
  if (g.phi_kind != TKPHI_PHI_MLP) {
    launch_score_mid(g, problems, ws, s);
    launch_select(g, problems, ws, s);
    launch_gather(g, problems, ws, acct, s);
    launch_merge(g, problems, ws, acct, s);
    return TKPHI_OK;
  }
  std::lock_guard<std::mutex> lock(g_side_mutex);
  SideStream* ss = nullptr;
  tkphi_status st = side_stream(&ss);  // (also where it is not used: any MLP call outside a capture makes later ones fit for it)
  if (st != TKPHI_OK) return st;
  if (g.list) {                        // most of phi_q rides in the score and select launches
    launch_filtered(g);
    launch_mlp_phi_q(g, problems, ws, s);
    if (g.sel_feat) launch_mlp_sel_features(g, problems, ws, s);    // no feature cache: phi_k of the retrieved keys
    launch_gather(g, problems, ws, acct, s);
    launch_merge(g, problems, ws, acct, s);
    return TKPHI_OK;
  }
  st = hip_ok(hipEventRecord(ss->fork, s), "hipEventRecord");
  if (st == TKPHI_OK) st = hip_ok(hipStreamWaitEvent(ss->stream, ss->fork, 0), "hipStreamWaitEvent");
  if (st != TKPHI_OK) return st;
  launch_mlp_phi_q(g, problems, ws, ss->stream);
  st = hip_ok(hipEventRecord(ss->join, ss->stream), "hipEventRecord");
  launch_score_mid(g, problems, ws, s);
  launch_select(g, problems, ws, s);
  if (g.sel_feat) launch_mlp_sel_features(g, problems, ws, s);
  // (the join is enqueued even after an error above: the side stream must not be left forked)
  const tkphi_status st2 = hip_ok(hipStreamWaitEvent(s, ss->join, 0), "hipStreamWaitEvent");
  if (st != TKPHI_OK) return st;
  if (st2 != TKPHI_OK) return st2;
  launch_gather(g, problems, ws, acct, s);
  launch_merge(g, problems, ws, acct, s);
  return TKPHI_OK;
}

tkphi_status tkphi_decode(const tkphi_config* cfg, const tkphi_problem* problems, int32_t n_problems,
                          int32_t max_L, int32_t max_K, int32_t mode, void* workspace,
                          size_t workspace_bytes, void* hip_stream) {
  const int acct = mode & ~TKPHI_FLAG_DIAG;
  if (acct != TKPHI_MODE_SUB && acct != TKPHI_MODE_NOSUB && acct != TKPHI_MODE_TOPK_ONLY) {
    set_error("mode=%d is not a tkphi_mode (optionally | TKPHI_FLAG_DIAG)", mode);
    return TKPHI_EINVAL;
  }
  Geom g;
  tkphi_status st = make_geom(cfg, n_problems, max_L, max_K, &g, workspace_bytes, &Geom::decode_bytes, (mode & TKPHI_FLAG_DIAG) != 0);
  if (st != TKPHI_OK) return st;
  st = check_call(problems, n_problems, workspace, workspace_bytes, g, g.decode_bytes);
  if (st != TKPHI_OK) return st;
  if (n_problems == 0) return TKPHI_OK;
  hipStream_t s = (hipStream_t)hip_stream;
  char* ws = (char*)workspace;
  (void)hipGetLastError();
  st = enqueue_decode(g, problems, ws, acct, s);
  if (st != TKPHI_OK) return st;
  return hip_ok(hipGetLastError(), "tkphi_decode launch");
}

// ---- decode for callers that cannot allocate ------------------------------------------------
// The scratch memory of a decode call (everything tkphi_decode keeps in the caller's workspace)
// in a file-scope device array.  Each GPU the library runs on holds its own copy of the array,
// at its own address, until the process ends; the address is resolved once per device, with that
// device current, and kept.  Host code never uses the array's name for anything else: kernels,
// like every other consumer, get the resolved pointer.
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[TKPHI_STATIC_SCRATCH_BYTES];
static std::mutex g_scratch_mutex;
static char* g_scratch_ptr[64];

static tkphi_status static_scratch(char** out) {
  int dev = 0;
  tkphi_status st = hip_ok(hipGetDevice(&dev), "hipGetDevice");
  if (st != TKPHI_OK) return st;
  if (dev < 0 || dev >= 64) { set_error("device ordinal %d out of range", dev); return TKPHI_EINVAL; }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    st = hip_ok(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
    if (st != TKPHI_OK) return st;
    if (!ptr || ((uintptr_t)ptr) % 256 != 0) { set_error("static scratch resolved to %p", ptr); return TKPHI_EHIP; }
    g_scratch_ptr[dev] = (char*)ptr;
  }
  *out = g_scratch_ptr[dev];
  return TKPHI_OK;
}

tkphi_status tkphi_decode_static(const tkphi_config* cfg, const tkphi_problem* problems, int32_t n_problems,
                                 int32_t max_L, int32_t max_K, int32_t mode, void* hip_stream) {
  const int acct = mode & ~TKPHI_FLAG_DIAG;
  if (acct != TKPHI_MODE_SUB && acct != TKPHI_MODE_NOSUB && acct != TKPHI_MODE_TOPK_ONLY) {
    set_error("mode=%d is not a tkphi_mode (optionally | TKPHI_FLAG_DIAG)", mode);
    return TKPHI_EINVAL;
  }
  Geom g;
  tkphi_status st = make_geom(cfg, n_problems, max_L, max_K, &g, TKPHI_STATIC_SCRATCH_BYTES, &Geom::decode_bytes, (mode & TKPHI_FLAG_DIAG) != 0);
  if (st != TKPHI_OK) return st;
  if (g.phi_kind == TKPHI_PHI_MLP) {      // that path creates a stream and events on first use
    set_error("tkphi_decode_static does not run the MLP feature maps");
    return TKPHI_EUNSUPPORTED;
  }
  if (g.decode_bytes > (size_t)TKPHI_STATIC_SCRATCH_BYTES) {
    set_error("decode scratch of %zu bytes exceeds the static array of %zu bytes (n_problems=%d max_L=%d max_K=%d)",
              g.decode_bytes, (size_t)TKPHI_STATIC_SCRATCH_BYTES, n_problems, max_L, max_K);
    return TKPHI_EWORKSPACE;
  }
  char* ws = nullptr;
  st = static_scratch(&ws);
  if (st != TKPHI_OK) return st;
  st = check_call(problems, n_problems, ws, g.decode_bytes, g, g.decode_bytes);
  if (st != TKPHI_OK) return st;
  if (n_problems == 0) return TKPHI_OK;
  (void)hipGetLastError();
  st = enqueue_decode(g, problems, ws, acct, (hipStream_t)hip_stream);
  if (st != TKPHI_OK) return st;
  return hip_ok(hipGetLastError(), "tkphi_decode_static launch");
}

tkphi_status tkphi_decode_stage_times(const tkphi_config* cfg, const tkphi_problem* problems,
                                      int32_t n_problems, int32_t max_L, int32_t max_K, int32_t mode,
                                      void* workspace, size_t workspace_bytes, void* hip_stream,
                                      float* stage_ms_out) {
  if (!stage_ms_out) { set_error("stage_ms_out is null"); return TKPHI_EINVAL; }
  const int acct = mode & ~TKPHI_FLAG_DIAG;
  if (acct != TKPHI_MODE_SUB && acct != TKPHI_MODE_NOSUB && acct != TKPHI_MODE_TOPK_ONLY) {
    set_error("mode=%d is not a tkphi_mode (optionally | TKPHI_FLAG_DIAG)", mode);
    return TKPHI_EINVAL;
  }
  Geom g;
  tkphi_status st = make_geom(cfg, n_problems, max_L, max_K, &g, workspace_bytes, &Geom::decode_bytes, (mode & TKPHI_FLAG_DIAG) != 0);
  if (st != TKPHI_OK) return st;
  st = check_call(problems, n_problems, workspace, workspace_bytes, g, g.decode_bytes);
  if (st != TKPHI_OK) return st;
  for (int i = 0; i < TKPHI_N_STAGES; ++i) stage_ms_out[i] = 0.f;
  if (n_problems == 0) return TKPHI_OK;
  hipStream_t s = (hipStream_t)hip_stream;
  char* ws = (char*)workspace;
  // one (start, stop) event pair per kernel, recorded at the kernel's own begin and end
  static_assert(TKPHI_N_STAGES == ST_COUNT, "stage list out of sync with include/tkphi.h");
  hipEvent_t ev[2 * ST_COUNT];
  int made = 0;
  for (; made < 2 * ST_COUNT; ++made)
    if ((st = hip_ok(hipEventCreate(&ev[made]), "hipEventCreate")) != TKPHI_OK) break;
  if (st == TKPHI_OK) {
    KernelTimer t;
    for (int i = 0; i < ST_COUNT; ++i) { t.start[i] = ev[2 * i]; t.stop[i] = ev[2 * i + 1]; t.used[i] = false; }
    (void)hipGetLastError();
    g_kernel_timer = &t;
    st = enqueue_decode(g, problems, ws, acct, s);
    g_kernel_timer = nullptr;
    if (st == TKPHI_OK) st = hip_ok(hipGetLastError(), "tkphi_decode_stage_times launch");
    if (st == TKPHI_OK) st = hip_ok(hipStreamSynchronize(s), "hipStreamSynchronize");
    for (int i = 0; st == TKPHI_OK && i < ST_COUNT; ++i)
      if (t.used[i]) st = hip_ok(hipEventElapsedTime(&stage_ms_out[i], t.start[i], t.stop[i]), "hipEventElapsedTime");
  }
  for (int i = 0; i < made; ++i) (void)hipEventDestroy(ev[i]);
  return st;
}

tkphi_status tkphi_check_problems(const tkphi_config* cfg, const tkphi_problem* ph, int32_t n_problems,
                                  int32_t max_L, int32_t max_K, int32_t for_decode) {
  Geom g;
  tkphi_status st = make_geom(cfg, n_problems, max_L, max_K, &g);
  if (st != TKPHI_OK) return st;
  if (n_problems > 0 && !ph) { set_error("problems_host is null"); return TKPHI_EINVAL; }
  const size_t es = cfg->kv_dtype == TKPHI_BF16 ? 2 : 4;
  for (int p = 0; p < n_problems; ++p) {
    const tkphi_problem& q = ph[p];
    const bool mlp = cfg->phi_kind == TKPHI_PHI_MLP;     // then Wq, bq, Wk, bk are not read
    const void* req[] = {q.K, q.V, q.S, q.u, q.Wk, q.bk};
    const char* names[] = {"K", "V", "S", "u", "Wk", "bk"};
    for (int i = 0; i < (mlp ? 4 : 6); ++i) {
      if (!req[i]) { set_error("problem %d: %s is null", p, names[i]); return TKPHI_EINVAL; }
      if (((uintptr_t)req[i]) % 16 != 0) { set_error("problem %d: %s not 16-byte aligned", p, names[i]); return TKPHI_EALIGN; }
    }
    if (cfg->phi_kind == TKPHI_PHI_MLP) {
      if (!q.mlp_k || (for_decode && !q.mlp_q)) { set_error("problem %d: mlp_k / mlp_q is null", p); return TKPHI_EINVAL; }
      if (((uintptr_t)q.mlp_k) % 8 != 0 || ((uintptr_t)q.mlp_q) % 8 != 0) { set_error("problem %d: mlp table misaligned", p); return TKPHI_EALIGN; }
    }
    if (cfg->cache_features) {
      if (!q.phi_cache) { set_error("problem %d: phi_cache is null (cfg.cache_features is set)", p); return TKPHI_EINVAL; }
      if (((uintptr_t)q.phi_cache) % 16 != 0) { set_error("problem %d: phi_cache not 16-byte aligned", p); return TKPHI_EALIGN; }
    }
    if (q.diag && ((uintptr_t)q.diag) % 4 != 0) { set_error("problem %d: diag misaligned", p); return TKPHI_EALIGN; }
    if (for_decode) {
      const void* rq[] = {q.q, q.out, q.Wq, q.bq};
      const char* nq[] = {"q", "out", "Wq", "bq"};
      for (int i = 0; i < (mlp ? 2 : 4); ++i) {
        if (!rq[i]) { set_error("problem %d: %s is null", p, nq[i]); return TKPHI_EINVAL; }
        if (((uintptr_t)rq[i]) % 16 != 0) { set_error("problem %d: %s not 16-byte aligned", p, nq[i]); return TKPHI_EALIGN; }
      }
      if (q.n_gen < 0 || q.n_gen > cfg->max_gen) { set_error("problem %d: n_gen=%d outside [0, cfg.max_gen=%d]", p, q.n_gen, cfg->max_gen); return TKPHI_ESHAPE; }
      if (q.topk < 0 || q.topk > max_K) { set_error("problem %d: topk=%d outside [0, max_K=%d]", p, q.topk, max_K); return TKPHI_ESHAPE; }
      if (q.topk_idx && ((uintptr_t)q.topk_idx) % 4 != 0) { set_error("problem %d: topk_idx misaligned", p); return TKPHI_EALIGN; }
      if (q.aux && ((uintptr_t)q.aux) % 4 != 0) { set_error("problem %d: aux misaligned", p); return TKPHI_EALIGN; }
      if (q.scores && ((uintptr_t)q.scores) % 4 != 0) { set_error("problem %d: scores misaligned", p); return TKPHI_EALIGN; }
    }
    if (q.L < 1 || q.L > max_L) { set_error("problem %d: L=%d outside [1, max_L=%d]", p, q.L, max_L); return TKPHI_ESHAPE; }
    if (q.stride_tok < cfg->d_head || (q.stride_tok * es) % 16 != 0) {
      set_error("problem %d: stride_tok=%lld invalid (>= d_head, 16-byte multiple)", p, (long long)q.stride_tok);
      return TKPHI_EALIGN;
    }
    if (q.stride_head < 0 || (q.stride_head * es) % 16 != 0 ||
        (cfg->n_kv_heads > 1 && q.stride_head < cfg->d_head)) {
      set_error("problem %d: stride_head=%lld invalid", p, (long long)q.stride_head);
      return TKPHI_EALIGN;
    }
  }
  return TKPHI_OK;
}

tkphi_status tkphi_read_device_status(const void* workspace, void* hip_stream, uint32_t* status_out) {
  if (!workspace || !status_out) { set_error("null argument"); return TKPHI_EINVAL; }
  hipStream_t s = (hipStream_t)hip_stream;
  tkphi_status st = hip_ok(hipStreamSynchronize(s), "hipStreamSynchronize");
  if (st != TKPHI_OK) return st;
  return hip_ok(hipMemcpy(status_out, workspace, sizeof(uint32_t), hipMemcpyDeviceToHost), "hipMemcpy status");
}

int32_t tkphi_budget_paper(int64_t L, int32_t r_bp, int32_t n_sink, int32_t n_tail) {
  if (L < 0 || r_bp < 0 || n_sink < 0 || n_tail < 0) return 0;
  const int64_t anchors = std::min<int64_t>(L, (int64_t)n_sink + n_tail);
  const int64_t ceil_rL = (L * r_bp + 9999) / 10000;
  return (int32_t)std::max<int64_t>(0, ceil_rL - anchors);
}

int32_t tkphi_budget_mid(int64_t L, int32_t r_bp, int32_t n_sink, int32_t n_tail) {
  if (L < 0 || r_bp < 0 || n_sink < 0 || n_tail < 0) return 0;
  const int64_t mid = std::max<int64_t>(0, L - n_sink - n_tail);
  return (int32_t)(mid * r_bp / 10000);
}

const char* tkphi_status_string(int32_t status) {
  switch (status) {
    case TKPHI_OK: return "ok";
    case TKPHI_EINVAL: return "invalid argument";
    case TKPHI_ESHAPE: return "unsupported shape";
    case TKPHI_EALIGN: return "misaligned pointer or stride";
    case TKPHI_EWORKSPACE: return "workspace null, misaligned or too small";
    case TKPHI_EHIP: return "HIP runtime error";
    case TKPHI_EUNSUPPORTED: return "unsupported request";
    default: return "unknown status";
  }
}

const char* tkphi_last_error(void) { return g_last_error; }

}  // extern "C"
