// Decode back end.
//
// gather (exact_branch + residual_correct): one workgroup per tile of 64 retrieved tokens of
// a query head (and one per query head for the anchors) accumulates
//     m_loc = max s_i,  Z_loc = sum exp(s_i - m_loc),  nu_loc = sum exp(s_i - m_loc) v_i
// (eq. (exact_terms)), and the feature-space contributions to subtract from the summaries
// (eq. (subtraction)), kept as the already contracted sums
//     zsum = sum_i z_i,  zv = sum_i z_i v_i,   z_i = phi_q(q) . phi_k(k_i)
// with phi_k(k_i) recomputed from the gathered key, so that S_R is never materialised:
//     S_R^T phi_q = S_M^T phi_q - zv,      phi_q . u_R = phi_q . u_M - zsum.
// On the bf16 path phi_k(k_i) goes through the same arithmetic as in the summary build
// (bf16 MFMA with fp32 accumulation, fp32 exponent, result kept as a bf16 hi + lo pair),
// so what is subtracted is what was added.
//
// merge: combines the partials of a query head in a fixed order (log-sum-exp rescaling),
// evaluates the summary terms and applies the single-normalisation merge
// (eq. (hybrid_merge)) with the exact branch's max shift applied to the residual branch.
//
// All loops over tokens issue their (independent) row loads before consuming them: these
// kernels move little data and are bound by memory latency, not bandwidth.
#include "block_utils.h"
#include "gather_tile.h"
#include "merge_head.h"
#include "tkphi_internal.h"

namespace tkphi {

typedef GatherFrag Frag;

// ---- weighted sums of value rows ------------------------------------------------------------
// nu[c] = sum_i w[i] v_i[c], zv[c] = sum_i z[i] v_i[c] over `cnt` <= 64 rows given by tok[]
// (absolute token indices), rows of d elements.  Each row is read by LPR = d / (elements per
// 16 bytes) lanes with one 16-byte load; 256 threads cover 256 / LPR rows per pass and all
// passes' loads are issued together, as soon as the tokens are known: the rows arrive beside the keys or features that the
// weights are worked out from (64 sequences of 16K at 20 %: 866 us per step against 882 with the rows requested behind those at d = 64, 1276 against 1298
// at d = 128).  Results land in part[4 .. 4+d) and part[4+d .. 4+2d).
// LDS scratch `red` must hold 2 * 256 * 8 floats.
template <typename T, int D>   // rows of at most D elements
struct ValueRows {
  static constexpr int EPL = Elem<T>::per16, MAXP = 64 * D / (kThreads * EPL);   // passes
  u32x4 v[MAXP];
  __device__ __forceinline__ void request(const Geom& g, const tkphi_problem& pr, int64_t head_off, const int* tok, int cnt) {
    const int LPR = g.d / EPL, RPP = kThreads / LPR, seg = threadIdx.x % LPR, rsub = threadIdx.x / LPR;
#pragma unroll
    for (int ps = 0; ps < MAXP; ++ps)
      if (ps * RPP < cnt)
        v[ps] = gload128((const char*)pr.V + (head_off + (int64_t)tok[min(ps * RPP + rsub, cnt - 1)] * pr.stride_tok + seg * EPL) * sizeof(T));
  }
};
template <typename T, int D>
__device__ __forceinline__ void weighted_value_sums(const Geom& g, const ValueRows<T, D>& rows, const float* w, const float* z, int cnt,
                                                    float* red, float* part, bool with_z) {
  constexpr int EPL = Elem<T>::per16, MAXP = ValueRows<T, D>::MAXP;
  const int tid = threadIdx.x, d = g.d;
  const int LPR = d / EPL, RPP = kThreads / LPR;      // rows per pass
  const int seg = tid % LPR, rsub = tid / LPR;
  const int n_pass = (cnt + RPP - 1) / RPP;
  float an[EPL], az[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) { an[e] = 0.f; az[e] = 0.f; }
#pragma unroll
  for (int ps = 0; ps < MAXP; ++ps) {
    if (ps < n_pass) {
      const int i = ps * RPP + rsub;
      if (i < cnt) {
        float x[EPL];
        Elem<T>::unpack(make_uint4(rows.v[ps].x, rows.v[ps].y, rows.v[ps].z, rows.v[ps].w), x);
        const float wi = w[i], zi = with_z ? z[i] : 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) { an[e] = fmaf(wi, x[e], an[e]); az[e] = fmaf(zi, x[e], az[e]); }
      }
    }
  }
  // reduce over the RPP row groups: red[rsub][channel]
#pragma unroll
  for (int e = 0; e < EPL; ++e) {
    red[rsub * d + seg * EPL + e] = an[e];
    red[kThreads * 8 + rsub * d + seg * EPL + e] = az[e];
  }
  __syncthreads();
  if (tid < d) {
    float a0 = 0.f, a1 = 0.f;
    for (int k = 0; k < RPP; ++k) { a0 += red[k * d + tid]; a1 += red[kThreads * 8 + k * d + tid]; }
    part[4 + tid] += a0;
    part[4 + d + tid] += a1;
  }
  __syncthreads();
}

// Entry i0 + tid of a head's retrieved list, requested together with the length of the list (behind its end: any row of the
// mid-region, which counts for nothing)
struct ListEntry { int idx; float score; };
__device__ __forceinline__ ListEntry list_entry(const Geom& g, const char* blk, int gq, int i0) {
  const size_t at = (size_t)gq * g.max_K + min(i0 + min((int)threadIdx.x, kPairsPerWG - 1), g.max_K - 1);
  return ListEntry{((const int32_t*)(blk + g.off_selidx))[at], ((const float*)(blk + g.off_selscore))[at]};
}

// ---- anchors: exact terms over [0, n_sink) u [L - n_tail, L) (or every token if M is empty) --------
// One workgroup per batch of 64 anchors (`batch` = 0, 1, ...): scores with LPR lanes per key
// row (16-byte loads, butterfly sum), then the same weighted value sums as a retrieved tile.
template <typename T, int D>
__device__ void anchor_partial(const Geom& g, const tkphi_problem& pr, int gq, int n, int batch, float* part,
                               float* red) {
  constexpr int EPL = Elem<T>::per16;
  __shared__ int a_tok[64];
  __shared__ float a_s[64], a_w[64];
  __shared__ float a_acc[2 * kMaxDim + 4];           // [-, -, -, -, nu[d], zv[d]] in the partial's layout
  __shared__ float a_m;
  const int tid = threadIdx.x, d = g.d;
  const int h = gq / g.G;
  const int n_prefill = n > 0 ? g.n_sink + g.n_tail : pr.L;             // exact anchors of the prefill segment
  const int n_anchor = n_prefill + min(max(pr.n_gen, 0), g.max_gen);    // + generated tokens, rows [L, L + n_gen)
  const int base = batch * 64;
  if (base >= n_anchor) return;
  const int cnt = min(64, n_anchor - base);
  const int64_t head_off = (int64_t)h * pr.stride_head;
  const int LPR = d / EPL, RPP = kThreads / LPR;
  const int seg = tid % LPR, rsub = tid / LPR;
  float qreg[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) qreg[e] = Elem<T>::load1(pr.q, (int64_t)gq * d + seg * EPL + e);
  for (int i = tid; i < 2 * d + 4; i += kThreads) a_acc[i] = 0.f;
  if (tid < 64) {
    const int a = base + min(tid, cnt - 1);
    a_tok[tid] = a >= n_prefill ? pr.L + (a - n_prefill) : (n > 0 && a >= g.n_sink) ? (pr.L - g.n_tail + (a - g.n_sink)) : a;
  }
  __syncthreads();
  ValueRows<T, D> rows;
  rows.request(g, pr, head_off, a_tok, cnt);
  // scores of the batch
  constexpr int MAXP = ValueRows<T, D>::MAXP;
  const int n_pass = (cnt + RPP - 1) / RPP;
  uint4 kv[MAXP];
#pragma unroll
  for (int ps = 0; ps < MAXP; ++ps) {
    if (ps < n_pass) {
      const int i = min(ps * RPP + rsub, cnt - 1);
      const u32x4 t = gload128((const char*)pr.K + (head_off + (int64_t)a_tok[i] * pr.stride_tok + seg * EPL) * sizeof(T));
      kv[ps] = make_uint4(t.x, t.y, t.z, t.w);
    }
  }
#pragma unroll
  for (int ps = 0; ps < MAXP; ++ps) {
    if (ps < n_pass) {
      float x[EPL];
      Elem<T>::unpack(kv[ps], x);
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) s = fmaf(x[e], qreg[e], s);
      s = lanes_sum(s, LPR);
      const int i = ps * RPP + rsub;
      if (seg == 0 && i < cnt) a_s[i] = s * g.score_scale + 0.0f;
    }
  }
  __syncthreads();
  if (tid < 64) {
    float mb = tid < cnt ? a_s[tid] : -INFINITY;
    mb = wave_max(mb);
    a_w[tid] = tid < cnt ? __expf(a_s[tid] - mb) : 0.f;
    if (tid == 0) a_m = mb;
  }
  __syncthreads();
  weighted_value_sums(g, rows, a_w, a_w, cnt, red, a_acc, false);
  if (tid < 64) {
    const float Z = wave_sum(a_w[tid]);
    if (tid == 0) { part[0] = a_m; part[1] = Z; part[2] = 0.f; part[3] = (float)cnt; }
  }
  if (tid < d) { part[4 + tid] = a_acc[4 + tid]; part[4 + d + tid] = 0.f; }
}

// ---- summary terms: S_M^T phi_q and phi_q . u_M of a query head -> off_sphi, off_uphi ----------------------------------
// One workgroup per head of the gather launches, beside its tiles: at the head of the merge, whose few workgroups wait for 64 KB of S
// at d = 128, they took 4 of its 9.8 us.  Sums in a fixed order: features of a group in order, groups in order.  red: 1536 floats
// MAXF: rows of S that a thread requests together, no more than the head dimension calls for: these registers are the whole kernel's (with
// 16 at d = 64, where a thread has 4, and 8 value rows for the 2 there are, gather_mfma_kernel<64> held 5 wavefronts to a SIMD instead of 7
// and 64 sequences of 16K at 20 % took 976 us per step instead of 866)
template <int MAXF>
__device__ __forceinline__ void summary_terms(const Geom& g, const tkphi_problem& pr, char* blk, int gq, float* red) {
  const int tid = threadIdx.x, d = g.d, dphi = g.dphi, h = gq / g.G;
  float* sh_phiq = red + 1024;
  float* sh_u = red + 1280;
  const int QPR = d / 4, NG = kThreads / QPR;      // float4 per row of S; feature groups (8 for d = 128, 16 for d = 64)
  const int jg = tid / QPR, c4 = tid % QPR, per = (dphi + NG - 1) / NG, j0 = jg * per, j1 = min(dphi, j0 + per);
  const float* __restrict__ S = pr.S + (size_t)h * dphi * d;
  u32x4 sv[MAXF];
  auto request = [&](int jb) {
#pragma unroll
    for (int k = 0; k < MAXF; ++k)
      if (jb + k < j1) sv[k] = gload128(S + (size_t)(jb + k) * d + c4 * 4);
  };
  request(j0);
  if (tid < dphi) {                                // (d_phi <= kMaxDim = the threads)
    sh_phiq[tid] = ((const float*)(blk + g.off_phiq))[(size_t)gq * dphi + tid];
    sh_u[tid] = pr.u[(size_t)h * dphi + tid];
  }
  __syncthreads();
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int jb = j0; jb < j1; jb += MAXF) {
    if (jb != j0) request(jb);
#pragma unroll
    for (int k = 0; k < MAXF; ++k) {
      if (jb + k < j1) {
        const float pj = sh_phiq[jb + k];
        a.x = fmaf(pj, __uint_as_float(sv[k].x), a.x); a.y = fmaf(pj, __uint_as_float(sv[k].y), a.y);
        a.z = fmaf(pj, __uint_as_float(sv[k].z), a.z); a.w = fmaf(pj, __uint_as_float(sv[k].w), a.w);
      }
    }
  }
  *(float4*)(red + jg * d + c4 * 4) = a;           // (NG d = 1024 floats)
  __syncthreads();
  if (tid < d) {
    float x = 0.f;
    for (int k = 0; k < NG; ++k) x += red[k * d + tid];
    ((float*)(blk + g.off_sphi))[(size_t)gq * d + tid] = x;
  } else if (tid == kThreads - 64) {
    float x = 0.f;
    for (int j = 0; j < dphi; ++j) x = fmaf(sh_phiq[j], sh_u[j], x);     // feature order, products not rounded
    ((float*)(blk + g.off_uphi))[gq] = x;
  }
}

// ------------------------------------------------------------------------------------
// gather, bf16 on the matrix cores: grid (n_tiles + n_atiles + 1, Hq, n_problems); D == d_head == d_phi.
// Wavefront w owns 16 retrieved tokens: their key rows are the A operand (lane (r, kg): token
// r, 8 consecutive channels per k-step), Wk of the KV head is staged once per workgroup in
// LDS (rows padded by 16 B: conflict-free ds_read_b128) and provides the B operand per
// 16-feature tile.
// ------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(kThreads) void gather_mfma_kernel(Geom g, const tkphi_problem* __restrict__ probs,
                                                               char* __restrict__ ws, int mode) {
  constexpr int KS = D / 32;
  constexpr int WROW = wk_row_bytes(D);            // bytes per staged Wk row
  // the staged Wk and the reduction scratch of the value sums are never live together
  constexpr int kRedBytes = 2 * kThreads * 8 * (int)sizeof(float);
  constexpr int kBufBytes = D * WROW > kRedBytes ? D * WROW : kRedBytes;
  __shared__ __attribute__((aligned(16))) char lds_buf[kBufBytes];
  char* wk_lds = lds_buf;
  float* red = (float*)lds_buf;
  __shared__ int p_tok[kPairsPerWG];
  __shared__ float p_s[kPairsPerWG], p_w[kPairsPerWG], p_z[kPairsPerWG];
  __shared__ float acc_part[2 * D + 4];
  __shared__ float sh_m;

  const int tile = blockIdx.x, gq = blockIdx.y, p = blockIdx.z, tid = threadIdx.x;
  if (tile > g.n_tiles + g.n_atiles) return;
  const tkphi_problem pr = probs[p];
  if (pr.L < 1 || pr.L > g.max_L) return;
  const int n = mid_size(pr.L, g.n_sink, g.n_tail);
  char* blk = problem_block(g, ws, p);
  float* part = (float*)(blk + g.off_part) + ((size_t)gq * (g.n_tiles + g.n_atiles) + tile) * g.part_stride;
  if (tile == g.n_tiles + g.n_atiles) { if (has_residual(mode, n, retrieved_of(g, pr, n))) summary_terms<D * D / 4 / kThreads>(g, pr, blk, gq, red); return; }
  if (tile >= g.n_tiles) { anchor_partial<uint16_t, D>(g, pr, gq, n, tile - g.n_tiles, part, red); return; }
  const int i0 = tile * kPairsPerWG;
  const ListEntry le = list_entry(g, blk, gq, i0);
  const int Ksel = ((const SelPlan*)(blk + g.off_plan))[gq].n_sel;
  if (i0 >= Ksel) return;
  const int cnt = min(kPairsPerWG, Ksel - i0);
  const int h = gq / g.G;
  const int lane = tid & 63, wv = tid >> 6, r = lane & 15, kg = lane >> 4;

  // the tile's retrieved tokens
  if (tid < kPairsPerWG) {
    p_tok[tid] = g.n_sink + min(max(le.idx, 0), n - 1);
    p_s[tid] = tid < cnt ? le.score : -INFINITY;
  }
  for (int i = tid; i < 2 * D + 4; i += kThreads) acc_part[i] = 0.f;
  // stage Wk[h] ([D features][D channels] bf16) with padded rows
  {
    const char* wsrc = (const char*)pr.Wk + (size_t)h * D * D * 2;
    constexpr int SEGS = D * 2 / 16;               // 16-byte segments per row
    constexpr int PER = D * SEGS / kThreads;
    u32x4 t[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = tid + k * kThreads;
      t[k] = gload128(wsrc + (size_t)(i / SEGS) * D * 2 + (i % SEGS) * 16);
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = tid + k * kThreads;
      *(u32x4*)(wk_lds + (i / SEGS) * WROW + (i % SEGS) * 16) = t[k];
    }
  }
  __syncthreads();
  const int64_t head_off = (int64_t)h * pr.stride_head;
  ValueRows<uint16_t, D> rows;
  rows.request(g, pr, head_off, p_tok, cnt);
  if (tid < 64) {                                  // m_loc = max score of the tile
    float m = p_s[tid];
    m = wave_max(m);
    if (tid == 0) sh_m = m;
  }

  if (wv * 16 < cnt) {
    // A operand: key rows of this wavefront's 16 tokens
    const int tok = p_tok[wv * 16 + r];
    const char* rp = (const char*)pr.K + (head_off + (int64_t)tok * pr.stride_tok) * 2 + kg * 16;
    Frag a[KS];
#pragma unroll
    for (int j = 0; j < KS; ++j) a[j].u = gload128(rp + j * 64);
    const float* phiq = (const float*)(blk + g.off_phiq) + (size_t)gq * D;
    float zacc[4];
    wave_feature_dots<D>(a, wk_lds, pr.bk + (size_t)h * D, phiq, g.a, g.c, zacc);
    if (r == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) p_z[wv * 16 + 4 * kg + i] = zacc[i];
    }
  }
  __syncthreads();
  if (tid < kPairsPerWG) p_w[tid] = tid < cnt ? __expf(p_s[tid] - sh_m) : 0.f;
  __syncthreads();

  weighted_value_sums(g, rows, p_w, p_z, cnt, red, acc_part, true);
  if (tid < D) { part[4 + tid] = acc_part[4 + tid]; part[4 + D + tid] = acc_part[4 + D + tid]; }
  if (tid < 64) {
    const float Z = wave_sum(p_w[tid]), zs = wave_sum(tid < cnt ? p_z[tid] : 0.f);
    if (tid == 0) { part[0] = sh_m; part[1] = Z; part[2] = zs; part[3] = (float)cnt; }
  }
}

// ------------------------------------------------------------------------------------
// gather, generic (any storage type, fp32 arithmetic): same grid.  The key rows of the tile's
// (at most 64) tokens are staged in LDS as fp32; wavefront w evaluates the features of its 16 tokens with
// v_mfma_f32_16x16x4_f32, the arithmetic of the fp32 summary build (the inner indices of step (jj, e) are the channels
// 16 jj + 4 kg + e), Wk from global memory with the next feature tile's rows on their way.  Bound by latency: with a
// thread per (token, every fourth feature) on the vector ALU, one Wk row after the other, the kernel took 16 us for 40
// tokens at d = d_phi = 64; this one 10 us.
// ------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kThreads) void gather_kernel(Geom g, const tkphi_problem* __restrict__ probs,
                                                          char* __restrict__ ws, int mode) {
  constexpr int EPL = Elem<T>::per16;
  constexpr int KFS = 128 + 4;                     // padded row stride (d <= 128): conflict-free 16-byte reads
  __shared__ __attribute__((aligned(16))) float kf[kPairsPerWG * KFS];
  __shared__ __attribute__((aligned(16))) float red[2 * kThreads * 8];
  __shared__ int p_tok[kPairsPerWG];
  __shared__ float p_s[kPairsPerWG], p_w[kPairsPerWG], p_z[kPairsPerWG];
  __shared__ float acc_part[2 * 128 + 4];
  __shared__ float sh_m;
  const int tile = blockIdx.x, gq = blockIdx.y, p = blockIdx.z, tid = threadIdx.x;
  if (tile > g.n_tiles + g.n_atiles) return;
  const tkphi_problem pr = probs[p];
  if (pr.L < 1 || pr.L > g.max_L) return;
  const int n = mid_size(pr.L, g.n_sink, g.n_tail);
  char* blk = problem_block(g, ws, p);
  float* part = (float*)(blk + g.off_part) + ((size_t)gq * (g.n_tiles + g.n_atiles) + tile) * g.part_stride;
  if (tile == g.n_tiles + g.n_atiles) { if (has_residual(mode, n, retrieved_of(g, pr, n))) summary_terms<8>(g, pr, blk, gq, red); return; }
  if (tile >= g.n_tiles) { anchor_partial<T, 128>(g, pr, gq, n, tile - g.n_tiles, part, red); return; }
  const int i0 = tile * kPairsPerWG;
  const ListEntry le = list_entry(g, blk, gq, i0);
  const int Ksel = ((const SelPlan*)(blk + g.off_plan))[gq].n_sel;
  if (i0 >= Ksel) return;
  const int cnt = min(kPairsPerWG, Ksel - i0);
  const int h = gq / g.G, d = g.d, dphi = g.dphi;
  const float* phiq = (const float*)(blk + g.off_phiq) + (size_t)gq * dphi;
  const int64_t head_off = (int64_t)h * pr.stride_head;

  if (tid < kPairsPerWG) {
    p_tok[tid] = g.n_sink + min(max(le.idx, 0), n - 1);
    p_s[tid] = tid < cnt ? le.score : -INFINITY;
  }
  for (int i = tid; i < 2 * d + 4; i += kThreads) acc_part[i] = 0.f;
  __syncthreads();
  ValueRows<T, 128> rows;
  rows.request(g, pr, head_off, p_tok, cnt);
  {
    // key rows -> LDS (fp32): 16-byte pieces, (row, segment) pairs dealt over the threads
    const int SEGS = d / EPL;
    for (int idx = tid; idx < kPairsPerWG * SEGS; idx += kThreads) {
      const int row = idx / SEGS, seg = idx % SEGS;
      const u32x4 t = gload128((const char*)pr.K + (head_off + (int64_t)p_tok[row] * pr.stride_tok + seg * EPL) * sizeof(T));
      float x[EPL];
      Elem<T>::unpack(make_uint4(t.x, t.y, t.z, t.w), x);
#pragma unroll
      for (int e = 0; e < EPL; ++e) kf[row * KFS + seg * EPL + e] = x[e];
    }
  }
  __syncthreads();
  if (tid < 64) {                                  // m_loc = max score of the tile
    float m = p_s[tid];
    m = wave_max(m);
    if (tid == 0) sh_m = m;
  }
  // z_t = phi_q . phi_k(k_t) of this wavefront's 16 tokens
  const int lane = tid & 63, wv = tid >> 6, r = lane & 15, kg = lane >> 4;
  if (wv * 16 < cnt) {
    typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    constexpr int CTM = 8;                         // 16-channel steps of a row at d = 128
    const int CT = d / 16, NT = dphi / 16;
    // lane (r, kg): feature 16 nt + r, channels 16 jj + 4 kg ..
    auto load_w = [&](int nt, floatx4 (&w)[CTM], float* bias, float* pq) {
      const int j = min(nt, NT - 1) * 16 + r;
#pragma unroll
      for (int jj = 0; jj < CTM; ++jj) {
        if (jj >= CT) break;                       // (uniform)
        const char* src = (const char*)pr.Wk + (((int64_t)h * dphi + j) * d + jj * 16 + kg * 4) * sizeof(T);
        if (sizeof(T) == 4) {
          const u32x4 t = gload128(src);
          w[jj] = (floatx4){__uint_as_float(t.x), __uint_as_float(t.y), __uint_as_float(t.z), __uint_as_float(t.w)};
        } else {
          const u32x2 t = *(const __attribute__((address_space(1))) u32x2*)src;
          w[jj] = (floatx4){__uint_as_float(t.x << 16), __uint_as_float(t.x & 0xffff0000u), __uint_as_float(t.y << 16), __uint_as_float(t.y & 0xffff0000u)};
        }
      }
      *bias = pr.bk[(int64_t)h * dphi + j];
      *pq = phiq[j];
    };
    floatx4 a[CTM], w[2][CTM];
    float bias[2], pq[2];
    load_w(0, w[0], &bias[0], &pq[0]);
    float nrm = 0.f;
#pragma unroll
    for (int jj = 0; jj < CTM; ++jj) {
      if (jj >= CT) break;
      a[jj] = *(const floatx4*)(kf + (wv * 16 + r) * KFS + jj * 16 + kg * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) nrm = fmaf(a[jj][e], a[jj][e], nrm);
    }
    nrm = strided_sum(nrm, 16);                    // |k|^2 of token r
    float cn[4], z[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) { cn[i] = g.c * __shfl(nrm, 4 * kg + i); z[i] = 0.f; }
    for (int nt0 = 0; nt0 < NT; nt0 += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int nt = nt0 + u;
        load_w(nt + 1, w[u ^ 1], &bias[u ^ 1], &pq[u ^ 1]);
        if (nt >= NT) break;
        floatx4 acc[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int jj = 0; jj < CTM; ++jj) {
          if (jj >= CT) break;
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[jj][e], w[u][jj][e], acc[e], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float dot = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
          z[i] = fmaf(expf(g.a * dot - cn[i] + bias[u]), pq[u], z[i]);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      z[i] = lanes_sum(z[i], 16);
      if (r == 0) p_z[wv * 16 + 4 * kg + i] = wv * 16 + 4 * kg + i < cnt ? z[i] : 0.f;
    }
  }
  __syncthreads();
  if (tid < kPairsPerWG) p_w[tid] = tid < cnt ? __expf(p_s[tid] - sh_m) : 0.f;
  __syncthreads();

  weighted_value_sums(g, rows, p_w, p_z, cnt, red, acc_part, true);
  if (tid < d) { part[4 + tid] = acc_part[4 + tid]; part[4 + d + tid] = acc_part[4 + d + tid]; }
  if (tid < 64) {
    const float Z = wave_sum(p_w[tid]), zs = wave_sum(tid < cnt ? p_z[tid] : 0.f);
    if (tid == 0) { part[0] = sh_m; part[1] = Z; part[2] = zs; part[3] = (float)cnt; }
  }
}

// ------------------------------------------------------------------------------------
// gather from cached key features (cfg.cache_features): same grid and partial layout; instead
// of reading the key rows and recomputing phi_k, every retrieved token's feature row (d_phi
// fp32 values stored by the build) is read with 16-byte loads, d_phi / 4 lanes per row, all
// rows of the tile in flight together, and z_i = phi_q . phi_k(k_i) is a butterfly sum.
// ------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kThreads) void gather_cached_kernel(Geom g, const tkphi_problem* __restrict__ probs,
                                                                 char* __restrict__ ws, int mode) {
  __shared__ __attribute__((aligned(16))) float red[2 * kThreads * 8];
  __shared__ int p_tok[kPairsPerWG];
  __shared__ float p_s[kPairsPerWG], p_w[kPairsPerWG], p_z[kPairsPerWG];
  __shared__ float acc_part[2 * 128 + 4];
  __shared__ float sh_m;
  const int tile = blockIdx.x, gq = blockIdx.y, p = blockIdx.z, tid = threadIdx.x;
  if (tile > g.n_tiles + g.n_atiles) return;
  const tkphi_problem pr = probs[p];
  if (pr.L < 1 || pr.L > g.max_L) return;
  const int n = mid_size(pr.L, g.n_sink, g.n_tail);
  char* blk = problem_block(g, ws, p);
  float* part = (float*)(blk + g.off_part) + ((size_t)gq * (g.n_tiles + g.n_atiles) + tile) * g.part_stride;
  if (tile == g.n_tiles + g.n_atiles) { if (has_residual(mode, n, retrieved_of(g, pr, n))) summary_terms<8>(g, pr, blk, gq, red); return; }
  if (tile >= g.n_tiles) { anchor_partial<T, 128>(g, pr, gq, n, tile - g.n_tiles, part, red); return; }
  const int i0 = tile * kPairsPerWG;
  const ListEntry le = list_entry(g, blk, gq, i0);
  const int Ksel = ((const SelPlan*)(blk + g.off_plan))[gq].n_sel;
  if (i0 >= Ksel) return;
  const int cnt = min(kPairsPerWG, Ksel - i0);
  const int h = gq / g.G, d = g.d, dphi = g.dphi;
  const int64_t head_off = (int64_t)h * pr.stride_head;

  if (tid < kPairsPerWG) {
    p_tok[tid] = g.n_sink + min(max(le.idx, 0), n - 1);
    p_s[tid] = tid < cnt ? le.score : -INFINITY;
  }
  for (int i = tid; i < 2 * d + 4; i += kThreads) acc_part[i] = 0.f;
  __syncthreads();
  ValueRows<T, 128> rows;
  rows.request(g, pr, head_off, p_tok, cnt);
  if (tid < 64) {                                  // m_loc = max score of the tile
    float m = p_s[tid];
    m = wave_max(m);
    if (tid == 0) sh_m = m;
  }
  {
    // LPR lanes per feature row (a power of two <= 64; d_phi is a multiple of 16), RPP rows per pass
    int LPR = 4;
    while (LPR * 2 <= min(dphi / 4, 64)) LPR *= 2;
    const int RPP = kThreads / LPR, seg = tid % LPR, rsub = tid / LPR;
    const float* phiq = (const float*)(blk + g.off_phiq) + (size_t)gq * dphi;
    // feature row of tile entry `row`: the cached row of its token, or (MLP maps without a cache) row i0 + row of
    // the features the step recomputed for this head's retrieved list
    const float* cache_h = g.sel_feat ? (const float*)(blk + g.off_selphi) + ((size_t)gq * g.max_K + i0) * dphi
                                      : pr.phi_cache + (size_t)h * n * dphi;
    auto feat_row = [&](int row) -> size_t { return g.sel_feat ? (size_t)min(row, cnt - 1) : (size_t)(p_tok[row] - g.n_sink); };
    for (int r0 = 0; r0 < kPairsPerWG; r0 += RPP * 4) {
      float zz[4] = {0.f, 0.f, 0.f, 0.f};
      for (int c4 = seg; c4 < dphi / 4; c4 += LPR) {        // (one round when d_phi <= 256)
        const float4 pq = *(const float4*)(phiq + c4 * 4);
        float4 f[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int row = min(r0 + k * RPP + rsub, kPairsPerWG - 1);
          const u32x4 t = gload128(cache_h + feat_row(row) * dphi + c4 * 4);
          f[k] = make_float4(__uint_as_float(t.x), __uint_as_float(t.y), __uint_as_float(t.z), __uint_as_float(t.w));
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
          zz[k] = fmaf(pq.x, f[k].x, fmaf(pq.y, f[k].y, fmaf(pq.z, f[k].z, fmaf(pq.w, f[k].w, zz[k]))));
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        zz[k] = lanes_sum(zz[k], LPR);
        const int row = r0 + k * RPP + rsub;
        if (seg == 0 && row < kPairsPerWG) p_z[row] = row < cnt ? zz[k] : 0.f;
      }
    }
  }
  __syncthreads();
  if (tid < kPairsPerWG) p_w[tid] = tid < cnt ? __expf(p_s[tid] - sh_m) : 0.f;
  __syncthreads();

  weighted_value_sums(g, rows, p_w, p_z, cnt, red, acc_part, true);
  if (tid < d) { part[4 + tid] = acc_part[4 + tid]; part[4 + d + tid] = acc_part[4 + d + tid]; }
  if (tid < 64) {
    const float Z = wave_sum(p_w[tid]), zs = wave_sum(tid < cnt ? p_z[tid] : 0.f);
    if (tid == 0) { part[0] = sh_m; part[1] = Z; part[2] = zs; part[3] = (float)cnt; }
  }
}

// ------------------------------------------------------------------------------------
// merge: grid (Hq, n_problems); see merge_head.h
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void merge_kernel(Geom g, const tkphi_problem* __restrict__ probs,
                                                         char* __restrict__ ws, int mode) {
  merge_head<true, false>(g, probs, ws, (int)blockIdx.x, (int)blockIdx.y, mode);
}

// Blocks of a query head: the tiles, the anchor tiles, the summary terms, and an idle one if those are an even number.  Workgroups go to the 8 XCDs in
// turn; with 16 per head the light ones (anchors, summary terms) of all heads would share three XCDs and the others get two
// tiles of every head (16 fp32 sequences of 20K at 4 %, us per step with 16 blocks and with 17: d = 128 664 / 623, d = 64 386 / 367).
static int gather_blocks(const Geom& g) { return (g.n_tiles + g.n_atiles + 1) | 1; }
void launch_gather(const Geom& g, const tkphi_problem* probs, char* ws, int mode, hipStream_t s) {
  dim3 grid(gather_blocks(g), g.Hq, g.n_problems);
  if (g.cache || g.sel_feat) {
    if (g.dtype == TKPHI_BF16) TKPHI_LAUNCH(ST_GATHER, gather_cached_kernel<uint16_t>, grid, dim3(kThreads), 0, s, g, probs, ws, mode);
    else TKPHI_LAUNCH(ST_GATHER, gather_cached_kernel<float>, grid, dim3(kThreads), 0, s, g, probs, ws, mode);
  } else if (g.use_mfma) {
    if (g.d == 128) TKPHI_LAUNCH(ST_GATHER, gather_mfma_kernel<128>, grid, dim3(kThreads), 0, s, g, probs, ws, mode);
    else TKPHI_LAUNCH(ST_GATHER, gather_mfma_kernel<64>, grid, dim3(kThreads), 0, s, g, probs, ws, mode);
  } else if (g.dtype == TKPHI_BF16) {
    TKPHI_LAUNCH(ST_GATHER, gather_kernel<uint16_t>, grid, dim3(kThreads), 0, s, g, probs, ws, mode);
  } else {
    TKPHI_LAUNCH(ST_GATHER, gather_kernel<float>, grid, dim3(kThreads), 0, s, g, probs, ws, mode);
  }
}

void launch_merge(const Geom& g, const tkphi_problem* probs, char* ws, int mode, hipStream_t s) {
  TKPHI_LAUNCH(ST_MERGE, merge_kernel, dim3(g.Hq, g.n_problems), dim3(kThreads), 0, s, g, probs, ws, mode);
}

}  // namespace tkphi
