// Decode front end of the filtered pipeline (bf16 caches on the matrix cores; fp32 ones of short contexts in vector arithmetic).
//
// The exhaustive Top-K over the mid-region (Sec. "Models, tasks, and protocol") needs every score
// s_i = q . k_i / sqrt(d_h) once, but only the scores that can still reach the top K have to
// leave the chip.  Two launches for batches and very long sequences, decode_prep and score_filtered; one otherwise:
//
//   decode_prep     one small launch of independent jobs that need no selection (of several problems the sample jobs only, the others are
//                   blocks of score_filtered):
//                   * sample: per KV head, the scores of an evenly spaced sample of mid-region rows
//                     -> per query head a lower bound of the K-th largest score (a bin edge chosen so
//                     that the sample count above it exceeds its expectation at the K-th score by five
//                     standard deviations); the bound only prunes: the select kernel verifies that at
//                     least K tokens passed and otherwise rescans the head without a bound
//                   * phi:    phi_q(q) of a query head (App. "Head-wise phi architecture": per query
//                     head, once per step) and the summary terms S_M^T phi_q, phi_q . u_M that
//                     eq. (subtraction) and eq. (hybrid_merge) start from
//                   * anchor: the exact terms of eq. (exact_terms) over a tile of 64 anchors (sink,
//                     tail, generated tokens of eq. (implemented_decode))
//   score_filtered  the streaming pass over all mid-region keys, each KV head read once for its G
//                   query heads; a score goes to memory only if its key is >= the head's bound
//                   (about 2-3 K tokens per head instead of |M|), appended to per-wavefront lists.
//   score_fused     both in one launch for one problem or a few (score_fused_few; Geom::fused): the scan keeps its scores in LDS until
//                   the sample's bound, which the sample workgroups hand over inside the launch, has come.
//   score_direct    instead of both where contexts are short (Geom::direct): every score stored, one row per head,
//                   with the phi and anchor jobs in the same launch.
#include <algorithm>

#include "decode_side.h"
#include "mlp_query.h"
#include "score_tile.h"
#include "tkphi_internal.h"

namespace tkphi {

#ifdef TKPHI_PHASE_CLOCK
#define TKPHI_WAVE_MARK(ws, base)                                                                               \
  do {                                                                                                          \
    if ((threadIdx.x & 63) == 0 && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)                       \
      ((unsigned long long*)((ws) + 16))[(base) + (threadIdx.x >> 6)] = wall_clock64();                         \
  } while (0)
#else
#define TKPHI_WAVE_MARK(ws, base) do {} while (0)
#endif

constexpr int kPrepThreads = 1024;
constexpr int kPrepWaves = kPrepThreads / 64;

// Rows of the mid-region whose scores are sampled for a problem with n mid tokens: everything up to 1024
// tokens; beyond that n / 64 rows (at least 512, at most 1024) in evenly spaced groups of 16 consecutive rows
// (one matrix-core tile, one 4 KB page of 256-byte rows: scattered single rows cost a page walk each).
__device__ __forceinline__ int sample_size(int n) {
  return n <= 1024 ? n : min(1024, max(512, n / 64)) / 16 * 16;
}
// mid row of sample si (0 <= si < m)
__device__ __forceinline__ int sample_row(int si, int n, int m) {
  return m >= n ? si : (si >> 4) * (n / (m >> 4)) + (si & 15);
}

// ---- sample job: one workgroup per (problem, KV head) ------------------------------------------------
// LDS: sc [G][1024] sampled scores, hist [G][kBins], nin [G], inb [G][kInBin] keys of the boundary bin
constexpr int kInBin = 256;
// Margin of the sampled bound in standard deviations.  A miss costs a rescan of the head (2.3 ms for a 128K head): over rows
// that are independent of each other it came up once per 40 000 heads at four - every fourth call of a batch of 8192 heads (select
// 540 -> 690 us on average) -, at five once per 800 000 for 11 % more candidates, which cost 0.5 % of a batch's step and
// nothing measurable of one problem's.
constexpr int kSigmas = 5;
// Heads gl0 .. gl0 + G - 1 of the group, by NTHR threads; FUSED: the bounds are also handed to the score workgroups of the same
// launch (await_bounds).
template <int D, int TPI, int NTHR, bool FUSED>
__device__ __forceinline__ void prep_sample(const Geom& g, const tkphi_problem& pr, char* blk, int h, int gl0, int G, float* sc,
                                            uint32_t* hist, uint32_t* inb, int* nin, char* stage_all) {
  constexpr int NWV = NTHR / 64;
  constexpr int KS = D / 32, TOK = TPI * 16;
  // The sampled key rows are loaded whole-row-wise (a load instruction covers 64 / LPRW complete rows: one
  // workgroup pulls 2.6 times the bytes per second that it gets with the 16 rows x 64 bytes of the MFMA operand
  // layout) and pass through a wavefront-private LDS strip of one 16-row tile into the operand layout.
  constexpr int LPRW = D / 8, RPI = 64 / LPRW, NLD = TOK / RPI, ROWP = D * 2 + 16;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, r = lane & 15, kg = lane >> 4;
  const int n = mid_size(pr.L, g.n_sink, g.n_tail);
  const int Ksel = max(0, min(min(pr.topk, n), g.max_K));
  auto publish = [&](int gl, uint32_t edge) {
    const int gq = h * g.G + gl0 + gl;
    ((uint32_t*)(blk + g.off_thr))[gq] = edge;
    if (FUSED) store_agent((uint64_t*)(blk + g.off_hand) + gq, ((uint64_t)g.tag << 32) | edge);
  };
  if (n == 0 || Ksel == 0 || g.sel_test == 1) {         // nothing to retrieve (or test: a bound nothing passes)
    if (tid < G) publish(tid, 0xffffffffu);
    return;
  }
  if (g.sel_test == 2) {                                // test: no pruning at all
    if (tid < G) publish(tid, 0u);
    return;
  }
  const int m = sample_size(n);
  TKPHI_PHASE((blk - g.off_problem0), 3);
  TKPHI_WAVE_MARK((blk - g.off_problem0), 64);       // sample job entered
  for (int i = tid; i < G * kBins; i += NTHR) hist[i] = 0u;
  if (tid < G) nin[tid] = 0;
  ScoreFrag bq[kTileFrags<D>];
  load_query_frags<D>(g, pr, h, bq);
  const size_t row_bytes = (size_t)pr.stride_tok * 2;
  const char* K0 = (const char*)pr.K + ((size_t)h * pr.stride_head + (size_t)g.n_sink * pr.stride_tok) * 2 + (size_t)(lane % LPRW) * 16;
  char* stage = stage_all + (size_t)wv * 16 * ROWP;
  TKPHI_WAVE_MARK((blk - g.off_problem0), 80);       // before the key loads
  for (int i0 = wv * TOK; i0 < m; i0 += NWV * TOK) {
    u32x4 raw[NLD];
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const int si = min(i0 + u * RPI + lane / LPRW, m - 1);
      raw[u] = gload128(K0 + (size_t)sample_row(si, n, m) * row_bytes);
    }
    __builtin_amdgcn_sched_barrier(0);
    TKPHI_WAVE_MARK((blk - g.off_problem0), 96);     // loads issued
#ifdef TKPHI_PHASE_CLOCK
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
    TKPHI_WAVE_MARK((blk - g.off_problem0), 112);    // loads complete
#pragma unroll
    for (int t = 0; t < TPI; ++t) {
      // tile t = rows 16 t .. 16 t + 15 of the wavefront's share = load instructions 16 t / RPI .. ; LDS operations of
      // one wavefront execute in order, so the strip needs no barrier
#pragma unroll
      for (int u = t * 16 / RPI; u < (t + 1) * 16 / RPI; ++u)
        *(u32x4*)(stage + (u * RPI + lane / LPRW - t * 16) * ROWP + (lane % LPRW) * 16) = raw[u];
      ScoreFrag a[KS];
#pragma unroll
      for (int j = 0; j < KS; ++j) a[j].u = *(const u32x4*)(stage + r * ROWP + j * 64 + kg * 16);
      const st_floatx4 acc = score_tile<D, false>(a, bq);
      // lane (r, kg) holds head r's scores of samples i0 + t 16 + 4 kg + {0..3}: to LDS, so that every lane
      // takes part in what follows (12 of 64 lanes hold all the scores here)
      if (r >= gl0 && r < gl0 + G) *(st_floatx4*)(sc + (r - gl0) * 1024 + i0 + t * 16 + 4 * kg) = acc;
    }
  }
  __syncthreads();
  TKPHI_PHASE((blk - g.off_problem0), 4);
  // thread t <-> samples t, t + NTHR, ..: first-level histogram per head
  constexpr int SPT = 1024 / NTHR, MG = FUSED ? 1 : kMaxGroup;
  uint32_t key[SPT][MG];
#pragma unroll
  for (int k = 0; k < SPT; ++k) {
#pragma unroll
    for (int gl = 0; gl < MG; ++gl) {
      if (gl < G && tid + k * NTHR < m) {
        key[k][gl] = score_key(sc[gl * 1024 + tid + k * NTHR] * g.score_scale + 0.0f);
        atomicAdd(&hist[gl * kBins + key_bin(key[k][gl])], 1u);
      }
    }
  }
  __syncthreads();
  TKPHI_PHASE((blk - g.off_problem0), 5);
  // The whole mid-region sampled: the bound is the K-th score itself.  Otherwise: the tau-th largest sampled
  // score, tau = mu + kSigmas sqrt(mu) + 2 with mu = K m / n: the number of samples above the true K-th
  // score has mean <= mu and standard deviation <= sqrt(mu), so the bound lies below the K-th score except
  // with the tail probability of kSigmas standard deviations.
  int tau = Ksel;
  if (m < n) {
    const float mu = (float)Ksel * (float)m / (float)n;
    tau = (int)ceilf(mu + (float)kSigmas * sqrtf(mu) + 2.f);
  }
  __shared__ int sh_bin[kMaxGroup], sh_rem[kMaxGroup];
  if (wv < G) {
    const uint32_t* hrow = hist + wv * kBins + lane * 8;               // lane owns bins 8 lane .. 8 lane + 7
    uint32_t sfx[8], run = 0;
#pragma unroll
    for (int e = 7; e >= 0; --e) { run += hrow[e]; sfx[e] = run; }
    const int incl = wave_scan_incl((int)run);
    const uint32_t above = (uint32_t)(__builtin_amdgcn_readlane(incl, 63) - incl);      // samples in the bins of higher lanes
    int best = -1, rem = 0;                                            // highest bin b with count(>= b) >= tau; tau - count(> b)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if ((int)(sfx[e] + above) >= tau) { best = lane * 8 + e; rem = tau - (int)(sfx[e] + above - hrow[e]); }
    }
    const int top = wave_max(best);
    if (best == top && best >= 0 && (lane * 8 <= top && top < lane * 8 + 8)) { sh_bin[wv] = top; sh_rem[wv] = rem; }
    if (top < 0 && lane == 0) { sh_bin[wv] = -1; sh_rem[wv] = 0; }
  }
  __syncthreads();
  // inside that bin: the rem-th largest sampled key is the bound (ranked by counting; the bin holds a few dozen samples)
#pragma unroll
  for (int k = 0; k < SPT; ++k) {
#pragma unroll
    for (int gl = 0; gl < MG; ++gl) {
      if (gl < G && tid + k * NTHR < m && sh_bin[gl] >= 0 && key_bin(key[k][gl]) == sh_bin[gl]) {
        const int at = atomicAdd(&nin[gl], 1);
        if (at < kInBin) inb[gl * kInBin + at] = key[k][gl];
      }
    }
  }
  __syncthreads();
  if (wv < G) {
    const int gl = wv, cnt = nin[gl], rem = sh_rem[gl], b = sh_bin[gl];
    uint32_t edge;
    if (tau > m || b < 0) edge = 0u;                                   // more than the sample holds: no pruning
    else if (cnt > kInBin) edge = bin_lower_key(b);                    // (a very full bin: its lower edge)
    else {
      edge = 0u;
      for (int j = lane; j < cnt; j += 64) {
        const uint32_t mine = inb[gl * kInBin + j];
        int ge = 0;                                                    // samples of the bin with key >= mine, ties included
        for (int i = 0; i < cnt; ++i) ge += inb[gl * kInBin + i] >= mine ? 1 : 0;
        // the largest key with at least rem keys >= it
        if (ge >= rem) edge = max(edge, mine);
      }
      edge = wave_max(edge);
    }
    if (lane == 0) publish(gl, edge);
  }
}

// ---- phi job: one workgroup per query head ----------------------------------------------------------------
// phi_q -> workspace; sphi[c] = sum_j phi_q[j] S[h][j][c]; uphi = sum_j phi_q[j] u[h][j].  Every global load
// (S, u, the rows of Wq, q, the biases) is issued before anything is consumed: one memory round trip.
// Sums run in a fixed order.
__device__ __forceinline__ void prep_phi(const Geom& g, const tkphi_problem& pr, char* blk, int gq, float* pu /*[kMaxDim]*/,
                                         float* sh_phiq /*[kMaxDim]*/, float* red /*[4096]*/) {
  const int tid = threadIdx.x, d = g.d, dphi = g.dphi, h = gq / g.G;
  const int QPR = d / 4, NG = kPrepThreads / QPR;     // float4 per row of S; feature groups (32 for d = 128, 64 for d = 64)
  const int jg = tid / QPR, c4 = tid % QPR;
  const int per = (dphi + NG - 1) / NG;               // features per group (<= 8)
  const int j0 = jg * per, j1 = min(dphi, j0 + per);
  const float* __restrict__ S = pr.S + (size_t)h * dphi * d;
  constexpr int MAXF = 8;
  u32x4 sv[MAXF];
#pragma unroll
  for (int k = 0; k < MAXF; ++k)
    if (j0 + k < j1) sv[k] = gload128(S + (size_t)(j0 + k) * d + c4 * 4);
  const float uj = tid < dphi ? pr.u[(size_t)h * dphi + tid] : 0.f;
  // rows of Wq: LPR lanes per row (16 bytes each), rows_pp rows per pass, at most 4 passes (d_phi <= 256)
  const int LPR = d / 8, seg = tid % LPR, row_in = tid / LPR, rows_pp = kPrepThreads / LPR;
  constexpr int MAXP = 4;
  u32x4 wv[MAXP];
  float bj[MAXP];
#pragma unroll
  for (int k = 0; k < MAXP; ++k) {
    if (k * rows_pp >= dphi) break;                   // (uniform)
    const int j = min(k * rows_pp + row_in, dphi - 1);
    wv[k] = gload128((const char*)pr.Wq + (((size_t)gq * dphi + j) * d + seg * 8) * 2);
    bj[k] = pr.bq[(size_t)gq * dphi + j];
  }
  const u32x4 qv = gload128((const char*)pr.q + ((size_t)gq * d + seg * 8) * 2);
  float qx[8];
  Elem<uint16_t>::unpack(make_uint4(qv.x, qv.y, qv.z, qv.w), qx);
  float nrm = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) nrm = fmaf(qx[e], qx[e], nrm);
  nrm = lanes_sum(nrm, LPR);
  float* phiq = (float*)(blk + g.off_phiq) + (size_t)gq * dphi;
#pragma unroll
  for (int k = 0; k < MAXP; ++k) {
    if (k * rows_pp >= dphi) break;
    const int jr = k * rows_pp + row_in;
    float x[8];
    Elem<uint16_t>::unpack(make_uint4(wv[k].x, wv[k].y, wv[k].z, wv[k].w), x);
    float dot = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) dot = fmaf(x[e], qx[e], dot);
    dot = lanes_sum(dot, LPR);
    if (jr < dphi && seg == 0) {
      const float f = expf(g.a * dot - g.c * nrm + bj[k]);
      phiq[jr] = f;
      sh_phiq[jr] = f;
    }
  }
  __syncthreads();
  float4 sacc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int k = 0; k < MAXF; ++k) {
    if (j0 + k < j1) {
      const float pj = sh_phiq[j0 + k];
      sacc.x = fmaf(pj, __uint_as_float(sv[k].x), sacc.x); sacc.y = fmaf(pj, __uint_as_float(sv[k].y), sacc.y);
      sacc.z = fmaf(pj, __uint_as_float(sv[k].z), sacc.z); sacc.w = fmaf(pj, __uint_as_float(sv[k].w), sacc.w);
    }
  }
  *(float4*)(red + jg * d + c4 * 4) = sacc;           // NG d = 4096 floats
  if (tid < dphi) pu[tid] = sh_phiq[tid] * uj;        // phi_q[j] u[j], summed below in feature order
  __syncthreads();
  if (tid < d) {
    float a = 0.f;
    for (int k = 0; k < NG; ++k) a += red[k * d + tid];
    ((float*)(blk + g.off_sphi))[(size_t)gq * d + tid] = a;
  } else if (tid == 64 * (kPrepWaves - 1)) {
    float a = 0.f;
    for (int j = 0; j < dphi; ++j) a += pu[j];
    ((float*)(blk + g.off_uphi))[gq] = a;
  }
}

// ---- anchor job: one workgroup per (query head, tile of 64 anchors) -------------------------------------------
// Anchors are the rows [0, n_sink) u [L - n_tail, L) (every row if the mid-region is empty) followed by the
// generated tokens [L, L + n_gen).  Writes the tile's partial in the layout of the gather kernels:
// [m_loc, Z_loc, 0, count, nu_loc[d], 0[d]].
__device__ __forceinline__ void prep_anchor(const Geom& g, const tkphi_problem& pr, char* blk, int gq, int batch, float* a_s /*[64]*/,
                                            float* a_w /*[64]*/, float* red /*[16][128]*/) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, d = g.d, h = gq / g.G;
  const int n = mid_size(pr.L, g.n_sink, g.n_tail);
  const int n_prefill = n > 0 ? g.n_sink + g.n_tail : pr.L;
  const int n_anchor = n_prefill + min(max(pr.n_gen, 0), g.max_gen);
  const int base = batch * 64;
  if (base >= n_anchor) return;
  const int cnt = min(64, n_anchor - base);
  float* part = (float*)(blk + g.off_part) + ((size_t)gq * (g.n_tiles + g.n_atiles) + g.n_tiles + batch) * g.part_stride;
  const int LPR = d / 8, seg = tid % LPR, row = tid / LPR;          // 16-byte segments per row; rows >= 64 idle (d = 64)
  const bool live = row < cnt;
  const int a = base + min(row, cnt - 1);
  const int tok = a >= n_prefill ? pr.L + (a - n_prefill) : (n > 0 && a >= g.n_sink) ? (pr.L - g.n_tail + (a - g.n_sink)) : a;
  const size_t off = ((size_t)h * pr.stride_head + (size_t)tok * pr.stride_tok + seg * 8) * 2;
  const u32x4 kv = gload128((const char*)pr.K + off), vv = gload128((const char*)pr.V + off);
  const u32x4 qv = gload128((const char*)pr.q + ((size_t)gq * d + seg * 8) * 2);
  float kx[8], vx[8], qx[8];
  Elem<uint16_t>::unpack(make_uint4(kv.x, kv.y, kv.z, kv.w), kx);
  Elem<uint16_t>::unpack(make_uint4(vv.x, vv.y, vv.z, vv.w), vx);
  Elem<uint16_t>::unpack(make_uint4(qv.x, qv.y, qv.z, qv.w), qx);
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) s = fmaf(kx[e], qx[e], s);
  s = lanes_sum(s, LPR);
  if (seg == 0 && row < 64) a_s[row] = live ? s * g.score_scale + 0.0f : -INFINITY;
  __syncthreads();
  if (wv == 0) {
    const float sl = a_s[lane];
    const float mb = wave_max(sl);
    const float w = lane < cnt ? __expf(sl - mb) : 0.f;
    a_w[lane] = w;
    const float Z = wave_sum(w);
    if (lane == 0) { part[0] = mb; part[1] = Z; part[2] = 0.f; part[3] = (float)cnt; }
  }
  __syncthreads();
  const float w = live ? a_w[row] : 0.f;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = w * vx[e];
  // rows of one wavefront that share a segment: lanes seg, seg + LPR, ...
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = strided_sum(acc[e], LPR);
  if (lane < LPR) {
#pragma unroll
    for (int e = 0; e < 8; ++e) red[wv * 128 + lane * 8 + e] = acc[e];
  }
  __syncthreads();
  if (tid < d) {
    float x = 0.f;
    for (int k = 0; k < kPrepWaves; ++k) x += red[k * 128 + tid];
    part[4 + tid] = x;
    part[4 + d + tid] = 0.f;
  }
}

// grid (jobs, Hkv, n_problems), 1024 threads.  Job 0: sample; of one problem also jobs 1 .. G: phi of the group's query heads, then
// n_atiles anchor tiles per query head.  (The sample needs ~90 KB of LDS, one workgroup per CU: the many small jobs of a batch
// would be held to that.)
template <int D, int TPI>
__global__ __launch_bounds__(kPrepThreads) void decode_prep_kernel(Geom g, const tkphi_problem* __restrict__ probs,
                                                                   char* __restrict__ ws) {
  // sample job: sc [G][1024] floats + hist [G][kBins] + inb [G][kInBin] (G (4096 + 2048 + 1024) bytes), then the
  // staging strips, 16 wavefronts x 16 rows x (2 D + 16) bytes; phi / anchor jobs: 16 KB of reduction scratch
  extern __shared__ __attribute__((aligned(16))) float sh_dyn[];
  __shared__ float sh_a[kMaxDim], sh_b[kMaxDim];
  __shared__ int sh_nin[kMaxGroup];
  const int job = blockIdx.x, h = blockIdx.y, p = blockIdx.z;
  TKPHI_PHASE(ws, 0);
  TKPHI_WAVE_MARK(ws, 32);                           // kernel entered

  if (job == 0 && h == 0 && p == 0) write_device_status(g, probs, ws, true);
  const tkphi_problem pr = probs[p];
  if (pr.L < 1 || pr.L > g.max_L) return;
  char* blk = problem_block(g, ws, p);
  TKPHI_PHASE(ws, 1);
  TKPHI_WAVE_MARK(ws, 48);                           // problem record loaded
#ifdef TKPHI_PHASE_CLOCK
  if (threadIdx.x == 0 && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0) ((unsigned long long*)(ws + 16))[26] = clock64();
#endif
  if (job == 0) {
    uint32_t* hist = (uint32_t*)(sh_dyn + g.G * 1024);
    prep_sample<D, TPI, kPrepThreads, false>(g, pr, blk, h, 0, g.G, sh_dyn, hist, hist + g.G * kBins, sh_nin, (char*)(hist + g.G * (kBins + kInBin)));
    TKPHI_PHASE(ws, 2);
#ifdef TKPHI_PHASE_CLOCK
    if (threadIdx.x == 0 && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0) ((unsigned long long*)(ws + 16))[27] = clock64();
#endif
  } else if (job <= g.G) {
    // (also: nobody has arrived yet at this head's merge, see the fused select + gather kernel)
    if (threadIdx.x == 0) ((uint32_t*)(blk + g.off_mcount))[h * g.G + job - 1] = 0u;
    prep_phi(g, pr, blk, h * g.G + job - 1, sh_a, sh_b, sh_dyn);
  } else {
    const int j = job - 1 - g.G;
    prep_anchor(g, pr, blk, h * g.G + j / g.n_atiles, j % g.n_atiles, sh_a, sh_b, sh_dyn);
  }
}

// The phi and anchor jobs of KV head h of a problem as workgroups of 256 threads: job j < G: phi of query head h G + j (and that head's
// arrival counter <- 0: nobody has arrived yet at its merge), then n_atiles anchor tiles per query head.
constexpr int kSideLds = (2 * kMaxDim + 1024) * (int)sizeof(float);
template <int D, int EARLY, typename T = uint16_t>
__device__ __forceinline__ void side_job(const Geom& g, const tkphi_problem& pr, char* blk, int h, int job, float* sh_f) {
  if (job < g.G) {
    if (threadIdx.x == 0) ((uint32_t*)(blk + g.off_mcount))[h * g.G + job] = 0u;
    side_phi<D, EARLY, T>(g, pr, blk, h * g.G + job, sh_f, sh_f + kMaxDim, sh_f + 2 * kMaxDim);
  } else {
    const int j = job - g.G;
    side_anchor<D, T>(g, pr, blk, h * g.G + j / g.n_atiles, j % g.n_atiles, sh_f, sh_f + 64, sh_f + 128);
  }
}

// The phi and anchor jobs of several problems are blocks of the score launch, behind all its chunks: the last of those leave room on
// the CUs (a launch of their own, us per step before / now: d = 64, 256 ragged sequences of 64K 2300 / 2200, 64 of 16K 276 / 259, 16
// ragged ones of 20K 79 / 69; d = 128, 64 of 16K 491 / 471, 16 ragged ones of 40K 206 / 194; on the sample launch 11 of 25K 108 / 100).  Among
// the chunks they take the places of workgroups that stream (64 ragged sequences of 17K with 8 / 8 heads of 64: 156 apart, 164 among
// them, 149 behind them; 32 of 36K with 32 / 4 160, 163, 148).  Of a single problem the prep launch has them, whose sample leaves most CUs
// idle (64 / 8 heads of 64 at 500K: 119, among the chunks 128), up to four of those workgroups per CU.
__host__ __device__ __forceinline__ int side_jobs(const Geom& g) {
  const int jobs = g.G * (1 + g.n_atiles);
  return g.n_problems == 1 && (1 + jobs) * g.Hkv <= 1024 ? 0 : jobs;
}

// Chunk of block x of the KV head with running number `head`, S blocks per head.  Workgroups go to the XCDs, there to the shader engines and to CUs
// in turn by their index, and the short sequences of a ragged batch have no late chunks: all 256 places must get early and late ones
// alike.  With an odd S the heads' blocks run through all places by themselves (rotated by the head's number a chunk would move on by S - 1
// places, 32 of them at S = 33: 12 sequences of 66K at d = 128 203 us per step, rotated 245; 16 of 33K with 4 / 4 heads of 64 52 and 59),
// with an even one the rotation makes them do so.  For few blocks it comes around: after 256 workgroups the same chunk is at the same
// place again if S is 8 or 16 (32: every fourth time), so there it moves on with every 256 (d = 128, 150 ragged sequences of 25K 1.29
// times as fast by it, 100 of 32K 1.12; d = 64, 200 of 32K 1100 -> 953 us; with S = 32 12 of 128K at d = 128 would lose 2.4 %), odd numbers
// as well (5 to 31 blocks: 0 to 5 % faster than unrotated).
__device__ __forceinline__ int chunk_at(uint32_t x, uint32_t head, uint32_t S) {
  return (int)((x + (S < 32 ? head + head * S / 256 : S % 2 ? 0 : head)) % S);
}

// 256 threads; the chunks of all KV heads, then their side jobs, numbered over a grid of one or more rows: wavefront w is slot w of the workgroup's chunk.  Bound by HBM for long
// caches, by the latency of a few round trips for short ones.  A wavefront holds two groups of TPI / 4 tiles, one on its way
// while the other is contracted: whole units at a time (16 loads, wait, 16 tiles' scores, next unit) took 49.5 us
// against 47.9 for the 3B layer at 128K, 13.2 against 8.7 us for the 1B layer at 32K; three or four groups ahead, or groups twice
// as large, gain nothing at 128K and lose 2 us at 32K (the first group is consumed later).  Groups of TPI / 2 for batches at
// d = 64: within 0.6 % either way over 66 batches of 4 to 400 sequences on the same buffers.
template <int D, int TPI, bool STREAM, bool STRIP>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 6))) void score_filtered_kernel(Geom g, const tkphi_problem* __restrict__ probs,
                                                                  char* __restrict__ ws) {
  extern __shared__ __attribute__((aligned(16))) st_u32x2 sh_heads[];      // [4 wavefronts][G][cand_T]; side jobs: kSideLds bytes
  const uint32_t S = g.n_scan_chunks, heads = (uint32_t)g.Hkv * g.n_problems, at = blockIdx.y * gridDim.x + blockIdx.x;
  const bool side = at >= S * heads;
  const uint32_t i = side ? at - S * heads : at, per = side ? side_jobs(g) : S, head = per ? i / per : heads;
  if (head >= heads) return;                       // (behind the last job of a grid of several rows)
  const int x = i - head * per, p = head / g.Hkv, h = head % g.Hkv;
  const tkphi_problem pr = probs[p];
  if (pr.L < 1 || pr.L > g.max_L) return;
  char* blk = problem_block(g, ws, p);
  if (side) {
    side_job<D, 0>(g, pr, blk, h, x, (float*)sh_heads);
    return;
  }
  const int n = mid_size(pr.L, g.n_sink, g.n_tail);
  const int n_chunks = (n + g.scan_chunk - 1) / g.scan_chunk;
  const int chunk = chunk_at(x, head, S);
  if (chunk >= n_chunks) return;
  const int r = threadIdx.x & 15;
  ScoreFrag bq[kTileFrags<D>];
  load_query_frags<D>(g, pr, h, bq);
  const uint32_t edge_r = ((const uint32_t*)(blk + g.off_thr))[h * g.G + min(r, g.G - 1)];
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  scan_wave_slot<D, TPI, TPI / 4, 2, STREAM, STRIP>(g, pr, blk, h, n, n_chunks, chunk, wv, bq, edge_r,
                                                       (lds_u32x2)sh_heads + (STRIP ? wv * g.G * g.cand_T : 0));
}

// ---- sample and score pass in one launch ------------------------------------------------------------------------------
// The bounds of KV head h (lane gl < G: head h G + gl) from the sample workgroups, which lie ahead of every score workgroup in
// the launch and wait for nothing, so the words arrive; the polls are counted all the same, and the lists of a head
// whose bound has not come by then are marked as not made (kNoList: the select kernel rescans that head).  False for such a
// lane.  A word is (tag, bound): tags differ from call to call, and the merging workgroup of the select kernel clears the
// word, for replays of a captured call.
constexpr int kBoundPolls = 1 << 14;     // of a microsecond or so
__device__ __forceinline__ bool await_bounds(const Geom& g, const char* blk, int h, uint32_t* edge) {
  const uint64_t* word = (const uint64_t*)(blk + g.off_hand) + h * g.G + min((int)(threadIdx.x & 63), g.G - 1);
  uint64_t w = 0;
  for (int k = 0; k < kBoundPolls; ++k) {
    w = load_agent(word);
    if (__all((uint32_t)(w >> 32) == g.tag)) break;
    __builtin_amdgcn_s_sleep(4);
  }
  *edge = (uint32_t)w;
  return (uint32_t)(w >> 32) == g.tag;
}

// n_problems (Hq (2 + n_atiles) + Hkv n_scan_chunks) workgroups of 512 threads: a sample job per query head, the phi and anchor jobs
// (behind the score chunks their loads are served last: they ended with the pass instead of after 10 us), the score chunks; with MLP
// maps (Geom::list) no phi and anchor jobs but the first stage of phi_q, behind the score chunks.  A score workgroup keeps its scores in
// LDS (G scan_chunk floats) and lists those that reach the bound at its end, when the sample is long since done: the launch that only
// sampled had nothing to run beside it.  The jobs of a kind of all problems come before those of the next kind: problem by problem, a
// problem's samples started behind the chunks of those before it and its own chunks held CUs waiting for them (3 3B sequences of 2K to
// 30K under bounds of 128K 75 us instead of 55, 4 of 60K to 128K 195 instead of 184, 32 single heads of 128 of 1K to 60K 79 instead of
// 66, which the two launches took 70 for; the other way round, 4 1B sequences of 16K to 64K 56 instead of 57, 20 of 3 / 1 heads of up
// to 20K 37 instead of 38).
// Bound by HBM for long contexts (3B layer at 128K: 268 MB; behind the last row the lists take 1.6 us, CUs that also sample end 3 us
// late), by the sample's round trips for short ones (1B layer at 32K: scores complete after 6.6 us, bounds there after 10).  Prep +
// score launches / this one: 11.1 + 48.7 / 47.5 us (52.5 with half-line loads) and 7.6 + 9.6 / 12.4 us.
constexpr int kFusedThreads = 512;
// job x of problem p.  LIST: with MLP maps (one problem)
template <int D, int TPI, bool STREAM, bool LIST>
__device__ __forceinline__ void score_fused_job(const Geom& g, const tkphi_problem* __restrict__ probs, char* __restrict__ ws, int x, int p) {
  extern __shared__ __attribute__((aligned(16))) float sh_dyn[];
  __shared__ int sh_n;
  constexpr int NWV = kFusedThreads / 64;
  if (blockIdx.x == 0) write_device_status(g, probs, ws, true);
  const tkphi_problem pr = probs[p];
  if (pr.L < 1 || pr.L > g.max_L) return;
  char* blk = problem_block(g, ws, p);
  if (x < g.Hq) {
    uint32_t* hist = (uint32_t*)(sh_dyn + 1024);
    prep_sample<D, TPI, kFusedThreads, true>(g, pr, blk, x / g.G, x % g.G, 1, sh_dyn, hist, hist + kBins, &sh_n, (char*)(hist + kBins + kInBin));
    return;
  }
  x -= g.Hq;
  if (!LIST || !g.list) {
    if (x < g.Hq) {
      if (threadIdx.x == 0) ((uint32_t*)(blk + g.off_mcount))[x] = 0u;
      side_phi<D, 0>(g, pr, blk, x, sh_dyn, sh_dyn + kMaxDim, sh_dyn + 2 * kMaxDim);
      return;
    }
    x -= g.Hq;
    if (x < g.Hq * g.n_atiles) {
      side_anchor<D>(g, pr, blk, x / g.n_atiles, x % g.n_atiles, sh_dyn, sh_dyn + 64, sh_dyn + 128);
      return;
    }
    x -= g.Hq * g.n_atiles;
  } else if (x >= g.Hkv * g.n_scan_chunks) {
    x -= g.Hkv * g.n_scan_chunks;
    mlp_phi_q_slice<0>(g, pr, blk, x % g.Hq, x / g.Hq, sh_dyn);
    return;
  }
  const int n = mid_size(pr.L, g.n_sink, g.n_tail);
  const int n_chunks = (n + g.scan_chunk - 1) / g.scan_chunk;
  const int h = x / g.n_scan_chunks, chunk = (x % g.n_scan_chunks + h + p * g.Hkv) % g.n_scan_chunks;
  if (chunk >= n_chunks) return;
  if (threadIdx.x == 0) sh_n = NWV;
  ScoreFrag bq[kTileFrags<D>];
  load_query_frags<D>(g, pr, h, bq);
  lds_barrier();
  scan_keep<D, TPI / 4, NWV, STREAM>(g, pr, h, n, n_chunks, chunk, bq, (lds_f32)sh_dyn, &sh_n);
  uint32_t edge;
  bool known = await_bounds(g, blk, h, &edge);
  if (g.sel_test == 1 && (chunk & 1)) known = false;      // (test: as if the wait had run out)
  lds_barrier();
  list_kept<D, NWV>(g, pr, blk, h, n, n_chunks, chunk, (lds_f32)sh_dyn, edge, known);
}

// one problem
template <int D, int TPI, bool STREAM>
__global__ __launch_bounds__(kFusedThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void score_fused_kernel(Geom g, const tkphi_problem* __restrict__ probs,
                                                                                                              char* __restrict__ ws) {
  score_fused_job<D, TPI, STREAM, true>(g, probs, ws, blockIdx.x, 0);
}

// a few: the jobs of one kind of every problem, then those of the next kind (in the kernel for one problem this sorting would cost a layer's
// step 0.4 us)
struct FusedJobs { int n_problems, per_problem[4]; };    // sample, phi, anchor, score jobs of a problem (beside probs in the arguments: the
                                                         // record's address waits for no other line of them)
template <int D, int TPI, bool STREAM>
__global__ __launch_bounds__(kFusedThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void score_fused_few_kernel(Geom g, const tkphi_problem* __restrict__ probs,
                                                                                                                  char* __restrict__ ws, FusedJobs jobs) {
  int x = blockIdx.x, ahead = 0, per = 0;  // jobs of a problem of the kinds before this one's, of this one's
  bool found = false;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (found) continue;
    per = jobs.per_problem[k];
    found = x < per * jobs.n_problems;
    if (!found) { x -= per * jobs.n_problems; ahead += per; }
  }
  const int p = x / per;
  score_fused_job<D, TPI, STREAM, false>(g, probs, ws, x - p * per + ahead, p);
}

// The phi and anchor jobs as a launch, where there is no mid-region to score: grid (G (1 + n_atiles), Hkv, n_problems), 256 threads
template <int D>
__global__ __launch_bounds__(kThreads) void decode_side_kernel(Geom g, const tkphi_problem* __restrict__ probs, char* __restrict__ ws) {
  __shared__ __attribute__((aligned(16))) float sh_f[2 * kMaxDim + 1024];
  const int h = blockIdx.y, p = blockIdx.z;
  const tkphi_problem pr = probs[p];
  if (pr.L < 1 || pr.L > g.max_L) return;
  side_job<D, 0>(g, pr, problem_block(g, ws, p), h, blockIdx.x, sh_f);
}

// The front end of short contexts (Geom::direct) in one launch: grid (G (1 + n_atiles) + n_scan_chunks, Hkv, n_problems), 256
// threads; first the phi and anchor jobs, then the score chunks, which store every score: the
// select kernel takes the exact threshold from all of them, and the sample job, a launch that nothing could overlap with
// (7-9 us), is not needed.
template <int D, int TPI, int EARLY>
__global__ __launch_bounds__(kThreads) void score_direct_kernel(Geom g, const tkphi_problem* __restrict__ probs, char* __restrict__ ws) {
  __shared__ __attribute__((aligned(16))) float sh_f[2 * kMaxDim + 1024];
  const int n_side = g.list ? 0 : g.G * (1 + g.n_atiles);
  const int x = blockIdx.x, h = blockIdx.y, p = blockIdx.z;
  if (x == 0 && h == 0 && p == 0) write_device_status(g, probs, ws, true);
  const tkphi_problem pr = probs[p];
  if (pr.L < 1 || pr.L > g.max_L) return;
  char* blk = problem_block(g, ws, p);
  if (x < n_side) {
    side_job<D, EARLY>(g, pr, blk, h, x, sh_f);
    return;
  }
  const int n = mid_size(pr.L, g.n_sink, g.n_tail);
  const int chunk = x - n_side, n_chunks = (n + g.scan_chunk - 1) / g.scan_chunk;
  if (chunk >= n_chunks) return;
  ScoreFrag bq[kTileFrags<D>];
  load_query_frags<D>(g, pr, h, bq);
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  scan_wave_slot<D, TPI, TPI / 4, 2, false, false, true>(g, pr, blk, h, n, n_chunks, chunk, wv, bq, 0u, (lds_u32x2) nullptr);
}

void launch_score_fused(const Geom& g, const tkphi_problem* probs, char* ws, hipStream_t s) {
  const FusedJobs jobs = {g.n_problems, {g.Hq, g.Hq, g.Hq * g.n_atiles, g.max_mid > 0 ? g.Hkv * g.n_scan_chunks : 0}};
  const int n_score = jobs.per_problem[3], n_jobs = g.list ? g.Hq * (1 + g.d_emb / 64) + n_score : g.Hq * (2 + g.n_atiles) + n_score;
  const size_t sample = (size_t)(1024 + kBins + kInBin) * 4 + (size_t)(kFusedThreads / 64) * 16 * (g.d * 2 + 16);
  static_assert(kQuerySliceLds <= 1024 + kBins + kInBin + 128 * (64 * 2 + 16) / 4, "the sample's share holds phi_q's as well");
  const size_t lds = std::max(sample, (size_t)g.G * g.scan_chunk * sizeof(float));       // (more than the 6 KB of the phi jobs)
  const auto launch = [&](auto fn, auto... more) {
    const hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) { set_error("hipFuncSetAttribute(%zu bytes of LDS): %s", lds, hipGetErrorString(e)); return; }
    TKPHI_LAUNCH(ST_SCORE, fn, dim3(g.n_problems * n_jobs), dim3(kFusedThreads), lds, s, g, probs, ws, more...);
  };
  if (g.n_problems == 1) {
    if (g.d == 128) { if (g.stream_keys) launch(score_fused_kernel<128, 4, true>); else launch(score_fused_kernel<128, 4, false>); }
    else { if (g.stream_keys) launch(score_fused_kernel<64, 8, true>); else launch(score_fused_kernel<64, 8, false>); }
  } else if (g.d == 128) { if (g.stream_keys) launch(score_fused_few_kernel<128, 4, true>, jobs); else launch(score_fused_few_kernel<128, 4, false>, jobs); }
  else { if (g.stream_keys) launch(score_fused_few_kernel<64, 8, true>, jobs); else launch(score_fused_few_kernel<64, 8, false>, jobs); }
}

// The same for fp32 caches (d = 64): scores in vector arithmetic, 128 rows per workgroup and all of them requested before the first
// is used (16 lanes x 16 bytes to a row).  Bound by latency: one head of 4K tokens is 32 such workgroups.
constexpr int kDirectRowsF32 = 128;
__global__ __launch_bounds__(kThreads) void score_direct_f32_kernel(Geom g, const tkphi_problem* __restrict__ probs, char* __restrict__ ws) {
  constexpr int D = 64, LPR = D / 4, RPP = kThreads / LPR, UNR = kDirectRowsF32 / RPP;
  __shared__ __attribute__((aligned(16))) float sh_f[2 * kMaxDim + 1024];
  const int n_side = g.G * (1 + g.n_atiles);
  const int x = blockIdx.x, h = blockIdx.y, p = blockIdx.z;
  if (x == 0 && h == 0 && p == 0) write_device_status(g, probs, ws, true);
  const tkphi_problem pr = probs[p];
  if (pr.L < 1 || pr.L > g.max_L) return;
  char* blk = problem_block(g, ws, p);
  if (x < n_side) {
    side_job<D, 0, float>(g, pr, blk, h, x, sh_f);
    return;
  }
  const int n = mid_size(pr.L, g.n_sink, g.n_tail), row0 = (x - n_side) * kDirectRowsF32;
  if (row0 >= n) return;
  const int tid = threadIdx.x, seg = tid % LPR, rsub = tid / LPR;
  const char* Kb = (const char*)pr.K + ((int64_t)h * pr.stride_head + (int64_t)g.n_sink * pr.stride_tok + seg * 4) * 4;
  u32x4 v[UNR];
#pragma unroll
  for (int u = 0; u < UNR; ++u) v[u] = gload128(Kb + (int64_t)min(row0 + u * RPP + rsub, n - 1) * pr.stride_tok * 4);
  const glb_f32 rows = (glb_f32)(blk + g.off_scores);
  for (int gl = 0; gl < g.G; ++gl) {
    const int gq = h * g.G + gl;
    const u32x4 qv = gload128((const char*)pr.q + ((size_t)gq * D + seg * 4) * 4);
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) s = fmaf(__uint_as_float(v[u][e]), __uint_as_float(qv[e]), s);
      s = lanes_sum(s, LPR);
      const int tok = row0 + u * RPP + rsub;
      if (seg == 0 && tok < n) {
        s = s * g.score_scale + 0.0f;              // + 0.0f: -0 -> +0, equal scores get equal keys
        rows[(size_t)gq * g.mid_stride + tok] = s;
        if (pr.scores) ((glb_f32)pr.scores)[(size_t)gq * n + tok] = s;
      }
    }
  }
}

void launch_score_direct(const Geom& g, const tkphi_problem* probs, char* ws, hipStream_t s) {
  if (g.dtype == TKPHI_F32) {
    static_assert(kDirectRowsF32 == direct_unit_f32, "chunks of the geometry");
    dim3 grid(g.G * (1 + g.n_atiles) + (g.max_mid > 0 ? g.n_scan_chunks : 0), g.Hkv, g.n_problems);
    TKPHI_LAUNCH(ST_SCORE, score_direct_f32_kernel, grid, dim3(kThreads), 0, s, g, probs, ws);
    return;
  }
  dim3 grid((g.list ? 0 : g.G * (1 + g.n_atiles)) + (g.max_mid > 0 ? g.n_scan_chunks : 0), g.Hkv, g.n_problems);
  // (the phi job's rows of S ahead of everything else: 0.3 us off one 3B layer of 4K or 9K tokens, but at twice the
  // registers the whole launch of 256 problems of 1.5K took 258 us instead of 224 at d = 128, 154 instead of 128 at d = 64, when both were
  // measured; now 215 and 116 without)
  if (g.d == 128 && g.n_problems == 1) TKPHI_LAUNCH(ST_SCORE, (score_direct_kernel<128, 4, 16>), grid, dim3(kThreads), 0, s, g, probs, ws);
  else if (g.d == 128) TKPHI_LAUNCH(ST_SCORE, (score_direct_kernel<128, 4, 0>), grid, dim3(kThreads), 0, s, g, probs, ws);
  else TKPHI_LAUNCH(ST_SCORE, (score_direct_kernel<64, 8, 0>), grid, dim3(kThreads), 0, s, g, probs, ws);
}

void launch_prep(const Geom& g, const tkphi_problem* probs, char* ws, hipStream_t s) {
  dim3 grid(side_jobs(g) ? 1 : 1 + g.G * (1 + g.n_atiles), g.Hkv, g.n_problems);
  // <= 56 KB at G = 8, plus 68 KB (d = 128) / 36 KB (d = 64) of staging strips
  const size_t lds = std::max((size_t)g.G * (1024 + kBins + kInBin) * 4 + (size_t)kPrepWaves * 16 * (g.d * 2 + 16), (size_t)16384);
  const auto launch = [&](auto fn) {
    const hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) { set_error("hipFuncSetAttribute(%zu bytes of LDS): %s", lds, hipGetErrorString(e)); return; }
    TKPHI_LAUNCH(ST_PREP, fn, grid, dim3(kPrepThreads), lds, s, g, probs, ws);
  };
  if (g.d == 128) launch(decode_prep_kernel<128, 4>); else launch(decode_prep_kernel<64, 8>);
}

void launch_score_filtered(const Geom& g, const tkphi_problem* probs, char* ws, hipStream_t s) {
  if (g.max_mid == 0) {
    if (side_jobs(g) == 0) return;
    const auto launch_side = [&](auto fn) { TKPHI_LAUNCH(ST_PHIQ, fn, dim3(side_jobs(g), g.Hkv, g.n_problems), dim3(kThreads), 0, s, g, probs, ws); };
    if (g.d == 128) launch_side(decode_side_kernel<128>); else launch_side(decode_side_kernel<64>);
    return;
  }
  const int64_t blocks = (int64_t)(g.n_scan_chunks + side_jobs(g)) * g.Hkv * g.n_problems;
  constexpr int64_t row = 1 << 20;                   // (a row of 256-thread workgroups holds less than 2^32 threads)
  const dim3 grid((unsigned)std::min(blocks, row), (unsigned)((blocks + row - 1) / row));
  const size_t strips = g.head_strip ? (size_t)4 * g.G * g.cand_T * sizeof(uint2) : 0;   // the wavefronts' strips of list heads
  const size_t lds = std::max(strips, side_jobs(g) ? (size_t)kSideLds : 0);
  const auto launch = [&](auto fn) { TKPHI_LAUNCH(ST_SCORE, fn, grid, dim3(kThreads), lds, s, g, probs, ws); };
  const auto launch_as = [&](auto strip, auto stream) {
    if (g.d == 128) launch(score_filtered_kernel<128, 4, decltype(stream)::value, decltype(strip)::value>);
    else launch(score_filtered_kernel<64, 8, decltype(stream)::value, decltype(strip)::value>);
  };
  if (g.head_strip) { if (g.stream_keys) launch_as(std::true_type(), std::true_type()); else launch_as(std::true_type(), std::false_type()); }
  else { if (g.stream_keys) launch_as(std::false_type(), std::true_type()); else launch_as(std::false_type(), std::false_type()); }
}

}  // namespace tkphi
