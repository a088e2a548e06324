// The key-side weights of the MLP feature maps in MFMA-fragment order: packed by a launch of their own (build, batches) or by
// spare workgroups of the select launch (a decode step of one problem).
#pragma once

#include "tkphi_internal.h"

namespace tkphi {

// ------------------------------------------------------------------------------------
// Weights in MFMA-fragment order.  A matrix W [N][Kd] (row-major bf16) is cut into blocks of 16
// outputs x 32 inputs; block (ct, ks) is stored as the 1 KB a wavefront loads as one operand:
// lane (r, kg) -> the 16 bytes W[16 ct + r][32 ks + 8 kg .. + 7], at byte 16 lane of the block.  Blocks of the d_emb-wide
// matrices lie in groups of four output tiles, K step by K step: block (ct, ks) at KB (ct / 4 Kd/32 + ks) 4 + ct mod 4
// (a wavefront's four operands of a K step are 4 KB in a row); those of Wo at KB ct Kd/32 + ks.
// `chain`: for W1, W2 and Wo lane (r, kg) takes the inputs 32 ks + 4 kg + {0 .. 3} and 32 ks + 16 + 4 kg + {0 .. 3} instead:
// the order in which a lane of the persistent chain holds the outputs of two neighbouring tiles.
// The GEMM's operand loads then are whole 1 KB lines instead of 16 pieces of 64 B (measured 19 %
// faster).  Per head Ws | W1 | W2 | Wo, in this order, in the workspace slot of its problem.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ size_t packed_bytes_per_head(const Geom& g) {
  return ((size_t)g.d_emb * g.d + (size_t)2 * g.d_emb * g.d_emb + (size_t)g.dphi * g.d_emb) * 2;
}

__device__ __forceinline__ const char* packed_weights(const Geom& g, const char* ws, int slot, int h) {
  return ws + g.off_wpack + ((size_t)slot * g.Hkv + h) * packed_bytes_per_head(g);
}
__device__ __forceinline__ size_t packed_pieces(const Geom& g) { return packed_bytes_per_head(g) / 16; }

// 16-byte piece q < packed_pieces of KV head h, whose weights are mp
__device__ __forceinline__ void pack_piece(const Geom& g, char* __restrict__ ws, const tkphi_mlp& mp, int slot, int h, size_t q, bool chain) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const int E = g.d_emb;
  const size_t n_s = (size_t)E * g.d / 8, n_1 = (size_t)E * E / 8;
  char* dst = ws + g.off_wpack + ((size_t)slot * g.Hkv + h) * packed_bytes_per_head(g) + q * 16;
  // (the layer says how a matrix is packed; two layers may share one buffer)
  const bool stem = q < n_s, out = q >= n_s + 2 * n_1;
  const char* W = (const char*)(stem ? mp.Ws : out ? mp.Wo : q < n_s + n_1 ? mp.W1 : mp.W2);
  const int Kd = stem ? g.d : E;
  q -= stem ? 0 : out ? n_s + 2 * n_1 : q < n_s + n_1 ? n_s : n_s + n_1;
  const int lane = (int)(q & 63), r = lane & 15, kg = lane >> 4;
  const size_t blk = q >> 6;
  const int KS = Kd / 32;
  const int ks = (int)(out ? blk % KS : blk / 4 % KS), ct = (int)(out ? blk / KS : blk / 4 / KS * 4 + blk % 4);
  const char* row = W + ((size_t)(ct * 16 + r) * Kd + ks * 32) * 2;
  if (chain && !stem) {
    const u32x2 a = *(const u32x2*)(row + kg * 8), b = *(const u32x2*)(row + 32 + kg * 8);
    *(u32x4*)dst = (u32x4){a.x, a.y, b.x, b.y};
  } else {
    *(u32x4*)dst = gload128(row + kg * 16);
  }
}

}  // namespace tkphi
