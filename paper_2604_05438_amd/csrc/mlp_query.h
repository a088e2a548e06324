// phi_q of the MLP feature maps, for its own launches and for spare workgroups of the score and select launches.
#pragma once

#include "tkphi_internal.h"

namespace tkphi {

// ------------------------------------------------------------------------------------
// phi_q of every query head (decode side): the same chain as matrix-vector products in fp32,
// three stages so that each layer is spread over the chip: a workgroup owns 64 output rows (`slice`) of its layer:
//   stage 0: g0 = Ws q + bs (every workgroup of the head recomputes it: 2 d d_emb bytes from L2),
//            h[rows] = GeLU(W1[rows] g0 + b1[rows]); slice 0 also stores g0
//   stage 1: g[rows] = g0[rows] + alpha (W2[rows] h + b2[rows])
//   stage 2: phi_q[rows] = exp(Wo[rows] g + bo[rows])
// ------------------------------------------------------------------------------------
// Every global load of a workgroup (weights of its first row groups, biases, input vector) is
// issued before anything is consumed: one memory round trip per stage.
constexpr int kQuerySliceLds = 128 + 2 * 1024 + 2 * 64;        // floats of LDS, the caller's
template <int STAGE, int SPL>   // SPL = 1 for d_emb <= 512, 2 for 1024
__device__ __forceinline__ void mlp_phi_q_slice(const Geom& g, const tkphi_problem& pr, char* __restrict__ blk, int gq, int slice, float* lds) {
  float *xs = lds, *vin = xs + 128, *sb = vin + 1024, *sb2 = sb + 1024, *sg = sb2 + 64;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int E = g.d_emb;
  float* gbuf = (float*)(blk + g.off_mlpq) + (size_t)gq * 2 * E;
  float* hbuf = gbuf + E;
  const tkphi_mlp mp = pr.mlp_q[gq];
  const int j0 = slice * 64;
  const int nrows = min(64, (STAGE == 2 ? g.dphi : E) - j0);
  const char* Wslice = (const char*)(STAGE == 0 ? mp.W1 : STAGE == 1 ? mp.W2 : mp.Wo) + (size_t)j0 * E * 2;
  const float* bslice = (STAGE == 0 ? mp.b1 : STAGE == 1 ? mp.b2 : mp.bo) + j0;
  u32x4 ts[8], tw[8];
  if (STAGE == 0) gemv_load<1>(mp.Ws, E, g.d, 0, ts);
  gemv_load<SPL>(Wslice, nrows, E, 0, tw);
  if (tid < 64) sb2[tid] = bslice[min(tid, nrows - 1)];
  if (STAGE == 0) {
    if (tid < g.d) xs[tid] = Elem<uint16_t>::load1(pr.q, (int64_t)gq * g.d + tid);
    for (int i = tid; i < E; i += nthr) sb[i] = mp.bs[i];
    __syncthreads();
    gemv_bf16_rows<1>(mp.Ws, E, g.d, xs, ts, [&](int j, float dot) { vin[j] = dot + sb[j]; });
    __syncthreads();
    if (slice == 0)
      for (int i = tid; i < E; i += nthr) gbuf[i] = vin[i];
    gemv_bf16_rows<SPL>(Wslice, nrows, E, vin, tw, [&](int j, float dot) { hbuf[j0 + j] = gelu_erf(dot + sb2[j]); });
  } else if (STAGE == 1) {
    for (int i = tid; i < E; i += nthr) vin[i] = hbuf[i];
    if (tid < 64) sg[tid] = gbuf[j0 + min(tid, nrows - 1)];
    __syncthreads();
    gemv_bf16_rows<SPL>(Wslice, nrows, E, vin, tw, [&](int j, float dot) { gbuf[j0 + j] = fmaf(mp.alpha, dot + sb2[j], sg[j]); });
  } else {
    for (int i = tid; i < E; i += nthr) vin[i] = gbuf[i];
    __syncthreads();
    float* phiq = (float*)(blk + g.off_phiq) + (size_t)gq * g.dphi;
    gemv_bf16_rows<SPL>(Wslice, nrows, E, vin, tw, [&](int j, float dot) { phiq[j0 + j] = expf(dot + sb2[j]); });
  }
}
// the same for the d_emb of the configuration
template <int STAGE>
__device__ __forceinline__ void mlp_phi_q_slice(const Geom& g, const tkphi_problem& pr, char* __restrict__ blk, int gq, int slice, float* lds) {
  if (g.d_emb <= 512) mlp_phi_q_slice<STAGE, 1>(g, pr, blk, gq, slice, lds);
  else mlp_phi_q_slice<STAGE, 2>(g, pr, blk, gq, slice, lds);
}

}  // namespace tkphi
