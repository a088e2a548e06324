// Prefill summary build (eq. (natural_cache)):
//   S[h][j][c] = sum_{i in M} phi_k(k_i)[j] v_i[c],   u[h][j] = sum_{i in M} phi_k(k_i)[j]
// with phi_k(k)[j] = exp(a * Wk[h][j] . k - c |k|^2 + bk[h][j]).
//
// The mid-region of each (problem, KV head) is split into chunks; one workgroup reduces a
// chunk into a partial [dphi][d] + [dphi], and a second kernel sums the partials of a head
// in chunk order, so the result does not depend on scheduling.
//
// bf16 caches with d_phi = d use bf16 matrix instructions for both contractions (features = K Wk^T, then
// S = Phi^T [V | 1]); other storage types and feature widths the fp32 ones.
#include "block_utils.h"
#include "tkphi_internal.h"

namespace tkphi {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
union Frag {
  u32x4 u;
  bf16x8 v;
};

// What the build kernels need of Geom, 88 bytes of arguments with the two pointers instead of 464 when they were handed all of it. A
// launch with 720 bytes costs the host 3.3 us, and the next launch follows after 3.8, with 64 bytes 2.8 both (short builds are bound by
// that: two launches with 4 and 7 us of work).
struct BuildGeom {
  int Hkv, d, dphi, n_sink, n_tail, n_problems, max_L, max_gen, build_chunk, n_build_chunks, cache;
  float a, c;
  size_t off_status, off_bpart;
  explicit BuildGeom(const Geom& g)
      : Hkv(g.Hkv), d(g.d), dphi(g.dphi), n_sink(g.n_sink), n_tail(g.n_tail), n_problems(g.n_problems), max_L(g.max_L),
        max_gen(g.max_gen), build_chunk(g.build_chunk), n_build_chunks(g.n_build_chunks), cache(g.cache), a(g.a), c(g.c),
        off_status(g.off_status), off_bpart(g.off_bpart) {}
};

// ------------------------------------------------------------------------------------
// bf16 on the matrix cores, d_head == d_phi == D = 128: grid (n_build_chunks, Hkv, n_problems), 4 wavefronts.
// Wavefront w owns the features [w D/4, (w+1) D/4): its slice of Wk stays in registers for the whole chunk.
//
// The chunk is cut into tiles of 32 tokens.  A stage of LDS holds one tile of keys and one of
// values, both row-major as they lie in the cache, brought in by loads that write LDS
// directly; NS stages form a ring, so NS - 1 tiles are on their way from HBM while one is
// contracted, and no register is spent on data in flight.  Per tile:
//   GEMM1  P[32 tokens][own features] = K Wk^T : A = key rows from LDS, B = Wk slice
//          -> exp -> bf16 hi + lo; the result registers (4 consecutive tokens per lane and
//          16-token tile) are already the A operand of GEMM2 over a fixed permutation of
//          the 32 tokens, so the features never touch LDS
//   GEMM2  S[own features][all channels] += Phi^T V : B = value tile read through the
//          transposing LDS read (same token permutation), hi and lo as two MFMAs
// u is summed from the same features.
//
// Each load instruction moves 64 x 16 bytes into 1 KB of consecutive LDS (lane l -> bytes
// 16 l ..), so a lane picks WHICH 16-byte granule of its row it fetches: granule slot s of row
// r holds granule s ^ f(r) of that row, with f chosen per tensor so that the reads spread
// over all banks:
//   keys    read as the A operand of GEMM1 (16 lanes = 16 rows, same granule): f = row mod 16
//   values  read by the transposing LDS read (16 lanes take 8 bytes each of 4 rows x 16
//           channels; lane j receives the 4 tokens of channel j): f = 2 (row mod 8)
// |k|^2: a wavefront reads back the rows its own loads brought (its own wait covers them), sums
// the squares with 16-bit dot products and leaves c |k|^2 per row in LDS before the tile's
// barrier: one barrier per tile.
// ------------------------------------------------------------------------------------
typedef short short4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c) {   // a.lo b.lo + a.hi b.hi + c
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  union { uint32_t u; bf16x2 v; } x, y;
  x.u = a; y.u = b;
  return __builtin_amdgcn_fdot2_f32_bf16(x.v, y.v, c, false);
}

template <bool CACHE, int NS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void build_mfma_kernel(BuildGeom g, const tkphi_problem* __restrict__ probs, char* __restrict__ ws) {
  constexpr int D = 128, NW = 4;
  constexpr int KS = D / 32;            // k-steps of GEMM1 (over channels)
  constexpr int FT = D / (16 * NW);     // feature tiles per wavefront
  constexpr int CT = D / 16;            // channel tiles of S
  constexpr int GR = D / 8;             // 16-byte granules per row
  constexpr int TT = 32;                // tokens per tile
  constexpr int ROWB = D * 2;           // bytes per row
  constexpr int TILEB = TT * ROWB;      // bytes per key (or value) tile
  constexpr int RPI = 64 / GR;          // rows one load instruction covers
  constexpr int NLD = TT / (RPI * NW);  // load instructions per wavefront, tile and tensor
  static_assert(NLD >= 1 && NS >= 3 && NS <= 6, "ring shape");
  extern __shared__ __attribute__((aligned(1024))) char ring[];   // [NS][keys, values][TT][ROWB], then norms [NS][TT]
  float* nrm_all = (float*)(ring + NS * 2 * TILEB);               // c |k|^2 log2(e); +inf past the chunk end

  const int ch = blockIdx.x, h = blockIdx.y, p = blockIdx.z, tid = threadIdx.x;
  const tkphi_problem pr = probs[p];
  if (pr.L < 1 || pr.L > g.max_L) return;
  const int n = mid_size(pr.L, g.n_sink, g.n_tail);
  const int c0 = ch * g.build_chunk;
  if (c0 >= n) return;
  const int c1 = min(n, c0 + g.build_chunk);
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 15, kg = lane >> 4;
  const float a2 = g.a * kLog2e, c2 = g.c * kLog2e;

  Frag wk[FT][KS];
  float bias[FT];
  {
    const uint16_t* wsrc = (const uint16_t*)pr.Wk + (size_t)h * D * D;
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      const int feat = wv * (D / NW) + ft * 16 + r;
#pragma unroll
      for (int j = 0; j < KS; ++j) wk[ft][j].u = gload128(wsrc + (size_t)feat * D + j * 32 + kg * 8);
      bias[ft] = pr.bk[(size_t)h * D + feat] * kLog2e;
    }
  }
  wait_vm_loads<0>();                    // (the tile loads below are counted by hand)
  floatx4 sacc[FT][CT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) sacc[ft][ct] = (floatx4){0.f, 0.f, 0.f, 0.f};
  float uacc[FT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) uacc[ft] = 0.f;

  const size_t row_bytes = (size_t)pr.stride_tok * 2;
  const size_t base_off = ((size_t)h * pr.stride_head + (size_t)g.n_sink * pr.stride_tok) * 2;
  const char* Kt = (const char*)pr.K + base_off;
  const char* Vt = (const char*)pr.V + base_off;
  const uint32_t ring_addr = (uint32_t)(size_t)(__attribute__((address_space(3))) char*)ring;

  auto f_key = [](int row) { return row & 15; };
  auto f_val = [](int row) { return (row & 7) << 1; };
  // loads: instruction i of wavefront wv fills rows (wv * NLD + i) * RPI .. + RPI of a tile
  int ld_row[NLD], ld_kg[NLD], ld_vg[NLD];
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    ld_row[i] = (wv * NLD + i) * RPI + lane / GR;
    ld_kg[i] = ((lane % GR) ^ f_key(ld_row[i])) * 16;
    ld_vg[i] = ((lane % GR) ^ f_val(ld_row[i])) * 16;
  }
  const int n_tiles = (c1 - c0 + TT - 1) / TT;
  // a full tile is fetched as uniform tile base + a lane's constant 32-bit offset (when a tile's rows span < 2 GiB)
  const bool near = (uint64_t)TT * row_bytes < (1ull << 31);
  uint32_t ld_ko[NLD], ld_vo[NLD];
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    ld_ko[i] = near ? (uint32_t)(ld_row[i] * row_bytes) + ld_kg[i] : 0u;
    ld_vo[i] = near ? (uint32_t)(ld_row[i] * row_bytes) + ld_vg[i] : 0u;
  }
  auto issue = [&](int ti) {             // tile ti of the chunk -> stage ti % NS
    const int t0 = c0 + ti * TT;
    const uint32_t st = ring_addr + (uint32_t)(ti % NS) * (2 * TILEB) + (uint32_t)(wv * NLD) * 1024;
    if (near && t0 + TT <= c1) {
      const char* kb = Kt + (size_t)t0 * row_bytes;
      const char* vb = Vt + (size_t)t0 * row_bytes;
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        load_to_lds16_stream(kb, ld_ko[i], st + i * 1024);
        load_to_lds16_stream(vb, ld_vo[i], st + TILEB + i * 1024);
      }
    } else {                             // rows past the end re-read the last row
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const size_t ro = (size_t)min(t0 + ld_row[i], c1 - 1) * row_bytes;
        load_to_lds16_stream(Kt + ro + ld_kg[i], st + i * 1024);
        load_to_lds16_stream(Vt + ro + ld_vg[i], st + TILEB + i * 1024);
      }
    }
  };
  // |k|^2 of the rows this wavefront loaded (lane l holds 16 bytes of row l / GR of each of its blocks)
  auto own_norms = [&](int ti) {
    const int t0 = c0 + ti * TT;
    const char* k_t = ring + (size_t)(ti % NS) * (2 * TILEB);
    float* nrm_t = nrm_all + (ti % NS) * TT;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const u32x4 w = *(const u32x4*)(k_t + (wv * NLD + i) * 1024 + lane * 16);
      float sq = dot2_bf16(w.x, w.x, 0.f);
      sq = dot2_bf16(w.y, w.y, sq);
      sq = dot2_bf16(w.z, w.z, sq);
      sq = dot2_bf16(w.w, w.w, sq);
      sq = lanes_sum(sq, GR);
      if (lane % GR == 0) nrm_t[ld_row[i]] = t0 + ld_row[i] < c1 ? c2 * sq : INFINITY;
    }
  };
  // reads: per-lane byte offsets inside a key tile (A operand of GEMM1, row r of a 16-token tile) and
  // inside a value tile (8 bytes of row 4 kg + s / 4, channels 16 ct + 4 (s mod 4) .., s = lane mod 16)
  uint32_t a_off[KS], v_off[CT];
#pragma unroll
  for (int j = 0; j < KS; ++j) a_off[j] = (uint32_t)(r * ROWB + (((j * 4 + kg) ^ f_key(r)) * 16));
  {
    const int vrow = 4 * kg + (r >> 2), b = r & 3, fv2 = f_val(vrow) >> 1;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) v_off[ct] = (uint32_t)(vrow * ROWB + ((ct ^ fv2) << 5) + b * 8);
  }
  float* cache_h = CACHE ? pr.phi_cache + (size_t)h * n * D : nullptr;   // [token of M][feature]

  auto contract = [&](int ti) {
    const int t0 = c0 + ti * TT;
    const char* k_t = ring + (size_t)(ti % NS) * (2 * TILEB);
    const char* v_t = k_t + TILEB;
    const float* nrm_t = nrm_all + (ti % NS) * TT;
    u32x2 phi_hi[2][FT], phi_lo[2][FT];
    float ut[FT];
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) ut[ft] = 0.f;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      Frag a[KS];
#pragma unroll
      for (int j = 0; j < KS; ++j) a[j].u = *(const u32x4*)(k_t + mt * 16 * ROWB + a_off[j]);
      const floatx4 cn = *(const floatx4*)(nrm_t + mt * 16 + 4 * kg);
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) {
        floatx4 acc = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < KS; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j].v, wk[ft][j].v, acc, 0, 0, 0);
        float f[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = phi_exp2(acc[i], a2, bias[ft] - cn[i]);
        ut[ft] += (f[0] + f[1]) + (f[2] + f[3]);
        uint32_t h01, l01, h23, l23;
        split_bf16_pair(f[0], f[1], &h01, &l01);
        split_bf16_pair(f[2], f[3], &h23, &l23);
        phi_hi[mt][ft] = (u32x2){h01, h23};
        phi_lo[mt][ft] = (u32x2){l01, l23};
        if (CACHE) {                     // the 16-bit values GEMM2 contracts, as fp32
          const int tok = t0 + mt * 16 + 4 * kg;
          float* cp = cache_h + (size_t)tok * D + wv * (D / NW) + ft * 16 + r;
          if (tok + 0 < c1) cp[0] = join_bf16_lo(h01, l01);
          if (tok + 1 < c1) cp[D] = join_bf16_hi(h01, l01);
          if (tok + 2 < c1) cp[2 * D] = join_bf16_lo(h23, l23);
          if (tok + 3 < c1) cp[3 * D] = join_bf16_hi(h23, l23);
        }
      }
    }
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) uacc[ft] += ut[ft];

    // GEMM2, one k-step: lane (., kg) holds tokens 4 kg + {0..3} and 16 + 4 kg + {0..3} in both operands
    Frag ahi[FT], alo[FT];
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      ahi[ft].u = (u32x4){phi_hi[0][ft].x, phi_hi[0][ft].y, phi_hi[1][ft].x, phi_hi[1][ft].y};
      alo[ft].u = (u32x4){phi_lo[0][ft].x, phi_lo[0][ft].y, phi_lo[1][ft].x, phi_lo[1][ft].y};
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      typedef short4v __attribute__((address_space(3)))* lds_s4;
      union { short4v s; u32x2 u; } b0, b1;
      b0.s = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(v_t + v_off[ct]));
      b1.s = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(v_t + 16 * ROWB + v_off[ct]));
      Frag vb;
      vb.u = (u32x4){b0.u.x, b0.u.y, b1.u.x, b1.u.y};
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) {
        sacc[ft][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo[ft].v, vb.v, sacc[ft][ct], 0, 0, 0);
        sacc[ft][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi[ft].v, vb.v, sacc[ft][ct], 0, 0, 0);
      }
    }
  };

#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < n_tiles) issue(s);
  constexpr int PER = 2 * NLD;           // load instructions per wavefront and tile
  for (int ti = 0; ti < n_tiles; ++ti) {
    // this wavefront's share of tile ti has landed once at most min(NS - 2, tiles issued after ti) tiles are in flight
    const int after = min(NS - 2, n_tiles - 1 - ti);
    if (after >= NS - 2) wait_vm_loads<(NS - 2) * PER>();
    else if (after == 3) wait_vm_loads<3 * PER>();
    else if (after == 2) wait_vm_loads<2 * PER>();
    else if (after == 1) wait_vm_loads<PER>();
    else wait_vm_loads<0>();
    own_norms(ti);
    lds_barrier();                       // every share of tile ti is in LDS; stage (ti - 1) % NS is free
    if (ti + NS - 1 < n_tiles) issue(ti + NS - 1);
    contract(ti);
  }

  float* bp = (float*)(ws + g.off_bpart) + ((size_t)(p * g.Hkv + h) * g.n_build_chunks + ch) * ((size_t)D * (D + 1));
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        bp[(size_t)(wv * (D / NW) + ft * 16 + 4 * kg + i) * D + ct * 16 + r] = sacc[ft][ct][i];
    float x = uacc[ft];
    x += __shfl_xor(x, 16);
    x += __shfl_xor(x, 32);
    if (kg == 0) bp[(size_t)D * D + wv * (D / NW) + ft * 16 + r] = x;
  }
}

// ------------------------------------------------------------------------------------
// bf16, d_head == d_phi == 64: grid (n_build_chunks, Hkv, n_problems), NW wavefronts, wavefront w with tokens of its own (the tiles
// w, w + NW, ... of the chunk) and all 64 features of them: S (64 registers), Wk (32) and a tile's features (32) of one
// wavefront fit the registers.  So the tiles of a wavefront are its own business: it waits for its own loads only, there is no barrier
// in the loop, a key row is read from LDS once instead of once per feature slice, and |k|^2 costs a wavefront eight dot products per 16
// tokens: their sums over a row's four lanes come from one fp32 matrix product with c in every element of B, which leaves
// c |k|^2 of the tokens 4 kg + i in every lane (r, kg), where the exponents need it.  The wavefronts' S and u are added at the
// end, through LDS, in wavefront order.  Contractions and operand layouts as in the kernel above (values: f = 2 ((row / 2) mod 4), keys:
// f = (row / 2) mod 8, rows of 128 bytes).  Two stages of 8 KB per wavefront; the keys' half of a stage is refilled as soon as
// its fragments are in registers.
// What bounds it: the memory pipeline.  Per call, with slices of 16 features per wavefront and a barrier per tile (the form of the kernel above, 4
// workgroups per CU) and so: 16 sequences of 64K (2.1 GB) 382 -> 369 us (343 without the arithmetic), 16 ragged ones of 16K..64K 314 ->
// 298, one of 128K 56.4 -> 48.9, of 32K 21.1 -> 18.5, of 12K 14.8 -> 12.5.  8 wavefronts per workgroup: 32K 26.6, ragged 321.
// ------------------------------------------------------------------------------------
template <int NW, bool CACHE>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void build_mfma64_kernel(BuildGeom g, const tkphi_problem* __restrict__ probs, char* __restrict__ ws) {
  constexpr int D = 64, KS = 2, FT = 4, CT = 4, TT = 32, ROWB = 128, TILEB = TT * ROWB, NLD = 4, STAGE = 2 * TILEB;
  extern __shared__ __attribute__((aligned(1024))) char ring[];   // [NW][2][keys, values][TT][ROWB], then Wk [D][ROWB], bias [D]
  const int ch = blockIdx.x, h = blockIdx.y, p = blockIdx.z, tid = threadIdx.x;
  const tkphi_problem pr = probs[p];
  if (pr.L < 1 || pr.L > g.max_L) return;
  const int n = mid_size(pr.L, g.n_sink, g.n_tail);
  const int c0 = ch * g.build_chunk;
  if (c0 >= n) return;
  const int c1 = min(n, c0 + g.build_chunk);
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 15, kg = lane >> 4;
  const float a2 = g.a * kLog2e, c2 = g.c * kLog2e;
  char* my = ring + wv * 2 * STAGE;      // this wavefront's stages
  char* w_s = ring + NW * 2 * STAGE;
  float* bias_s = (float*)(w_s + D * ROWB);
  const uint32_t ring_addr = (uint32_t)(size_t)(__attribute__((address_space(3))) char*)ring;
  const uint32_t my_addr = ring_addr + wv * 2 * STAGE;

  // Wk and the biases by way of LDS, ahead of the first tiles: no wait of their own
  {
    const char* wsrc = (const char*)pr.Wk + (size_t)h * D * ROWB;
#pragma unroll
    for (int i = 0; i < 8 / NW; ++i) {
      const uint32_t o = (wv * (8 / NW) + i) * 1024;
      load_to_lds16(wsrc, o + lane * 16, ring_addr + NW * 2 * STAGE + o);
    }
    load_to_lds4((const char*)(pr.bk + (size_t)h * D), lane * 4, ring_addr + NW * 2 * STAGE + D * ROWB);     // (D floats, no more aligned than those are)
  }
  const size_t row_bytes = (size_t)pr.stride_tok * 2;
  const size_t base_off = ((size_t)h * pr.stride_head + (size_t)g.n_sink * pr.stride_tok) * 2;
  const char* Kt = (const char*)pr.K + base_off;
  const char* Vt = (const char*)pr.V + base_off;
  auto f_key = [](int row) { return (row >> 1) & 7; };
  auto f_val = [](int row) { return ((row >> 1) & 3) << 1; };
  const int n_tiles = (c1 - c0 + TT - 1) / TT;
  const int n_my = n_tiles > wv ? (n_tiles - wv + NW - 1) / NW : 0;
  const bool near = (uint64_t)TT * row_bytes < (1ull << 31);
  // load instruction i of a tile: rows 8 i .. 8 i + 7
  const int lrow = lane >> 3;
  uint32_t ko[NLD], vo[NLD];
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    const int row = i * 8 + lrow;
    ko[i] = (near ? (uint32_t)(row * row_bytes) : 0u) + (((lane & 7) ^ f_key(row)) * 16);
    vo[i] = (near ? (uint32_t)(row * row_bytes) : 0u) + (((lane & 7) ^ f_val(row)) * 16);
  }
  auto issue = [&](int j, const char* T, const uint32_t (&off)[NLD], uint32_t dst) {      // this wavefront's tile j of K or V
    const int t0 = c0 + (wv + j * NW) * TT;
    if (near && t0 + TT <= c1) {
      const char* b = T + (size_t)t0 * row_bytes;
#pragma unroll
      for (int i = 0; i < NLD; ++i) load_to_lds16_stream(b, off[i], dst + i * 1024);
    } else {                             // rows past the end re-read the last row
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const int row = i * 8 + lrow;
        const size_t ro = (size_t)min(t0 + row, c1 - 1) * row_bytes;
        load_to_lds16_stream(T + ro + (off[i] - (near ? (uint32_t)(row * row_bytes) : 0u)), dst + i * 1024);
      }
    }
  };
#pragma unroll
  for (int j = 0; j < 2; ++j)
    if (j < n_my) {
      issue(j, Kt, ko, my_addr + j * STAGE);
      issue(j, Vt, vo, my_addr + j * STAGE + TILEB);
    }
  if (n_my >= 2) wait_vm_loads<4 * NLD>();
  else if (n_my == 1) wait_vm_loads<2 * NLD>();
  else wait_vm_loads<0>();
  lds_barrier();
  Frag wk[FT][KS];
  float bias[FT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
#pragma unroll
    for (int j = 0; j < KS; ++j) wk[ft][j].u = *(const u32x4*)(w_s + (ft * 16 + r) * ROWB + j * 64 + kg * 16);
    bias[ft] = bias_s[ft * 16 + r] * kLog2e;
  }
  floatx4 sacc[FT][CT];
  float uacc[FT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    uacc[ft] = 0.f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) sacc[ft][ct] = (floatx4){0.f, 0.f, 0.f, 0.f};
  }
  uint32_t a_off[KS], v_off[CT];
#pragma unroll
  for (int j = 0; j < KS; ++j) a_off[j] = (uint32_t)(r * ROWB + (((j * 4 + kg) ^ f_key(r)) * 16));
  {
    const int vrow = 4 * kg + (r >> 2), b = r & 3, fv2 = f_val(vrow) >> 1;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) v_off[ct] = (uint32_t)(vrow * ROWB + ((ct ^ fv2) << 5) + b * 8);
  }
  float* cache_h = CACHE ? pr.phi_cache + (size_t)h * n * D : nullptr;   // [token of M][feature]

  for (int j = 0; j < n_my; ++j) {
    const uint32_t so = (uint32_t)(j & 1) * STAGE;
    const char* k_t = my + so;
    const char* v_t = k_t + TILEB;
    const int t0 = c0 + (wv + j * NW) * TT;
    if (j + 1 < n_my) wait_vm_loads<3 * NLD>();
    else wait_vm_loads<NLD>();
    Frag a[2][KS];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int s = 0; s < KS; ++s) a[mt][s].u = *(const u32x4*)(k_t + mt * 16 * ROWB + a_off[s]);
    floatx4 cn[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      float part[KS];                    // (a chain per half row, as short as its rounding is then small)
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        part[s] = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) part[s] = dot2_bf16(a[mt][s].u[e], a[mt][s].u[e], part[s]);
      }
      float sq = part[0] + part[1];
      asm volatile("s_nop 4" : "+v"(sq));     // (a dot product's result needs wait states before a matrix instruction reads it)
      cn[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(sq, c2, (floatx4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
    // (the key fragments have left LDS: their stage takes the tile after the next)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (j + 2 < n_my) issue(j + 2, Kt, ko, my_addr + so);
    if (t0 + TT > c1) {                  // no features past the end
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (t0 + mt * 16 + 4 * kg + i >= c1) cn[mt][i] = INFINITY;
    }
    u32x2 phi_hi[2][FT], phi_lo[2][FT];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      floatx4 acc[FT];                   // (all tiles' products ahead of the first exponential)
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int ft = 0; ft < FT; ++ft)
          acc[ft] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt][s].v, wk[ft][s].v, s ? acc[ft] : (floatx4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) {
        float f[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = phi_exp2(acc[ft][i], a2, bias[ft] - cn[mt][i]);
        uacc[ft] += (f[0] + f[1]) + (f[2] + f[3]);
        uint32_t h01, l01, h23, l23;
        split_bf16_pair(f[0], f[1], &h01, &l01);
        split_bf16_pair(f[2], f[3], &h23, &l23);
        phi_hi[mt][ft] = (u32x2){h01, h23};
        phi_lo[mt][ft] = (u32x2){l01, l23};
        if (CACHE) {                     // the 16-bit values GEMM2 contracts, as fp32
          const int tok = t0 + mt * 16 + 4 * kg;
          float* cp = cache_h + (size_t)tok * D + ft * 16 + r;
          if (tok + 0 < c1) cp[0] = join_bf16_lo(h01, l01);
          if (tok + 1 < c1) cp[D] = join_bf16_hi(h01, l01);
          if (tok + 2 < c1) cp[2 * D] = join_bf16_lo(h23, l23);
          if (tok + 3 < c1) cp[3 * D] = join_bf16_hi(h23, l23);
        }
      }
    }
    if (CACHE) wait_vm_loads<0>();       // (stores count too)
    else if (j + 2 < n_my) wait_vm_loads<3 * NLD>();
    else if (j + 1 < n_my) wait_vm_loads<2 * NLD>();
    else wait_vm_loads<0>();
    Frag vb[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      typedef short4v __attribute__((address_space(3)))* lds_s4;
      union { short4v s; u32x2 u; } b0, b1;
      b0.s = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(v_t + v_off[ct]));
      b1.s = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(v_t + 16 * ROWB + v_off[ct]));
      vb[ct].u = (u32x4){b0.u.x, b0.u.y, b1.u.x, b1.u.y};
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // (so have the values)
    if (j + 2 < n_my) issue(j + 2, Vt, vo, my_addr + so + TILEB);
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      Frag ahi, alo;
      ahi.u = (u32x4){phi_hi[0][ft].x, phi_hi[0][ft].y, phi_hi[1][ft].x, phi_hi[1][ft].y};
      alo.u = (u32x4){phi_lo[0][ft].x, phi_lo[0][ft].y, phi_lo[1][ft].x, phi_lo[1][ft].y};
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) sacc[ft][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo.v, vb[ct].v, sacc[ft][ct], 0, 0, 0);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) sacc[ft][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi.v, vb[ct].v, sacc[ft][ct], 0, 0, 0);
    }
  }

  // the wavefronts' sums through LDS, added in wavefront order
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) *(floatx4*)(my + (ft * CT + ct) * 1024 + lane * 16) = sacc[ft][ct];
  float* u_s = (float*)w_s;              // [NW][D], over Wk
  lds_barrier();                         // every wavefront has taken its Wk and bias
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    float x = uacc[ft];
    x += __shfl_xor(x, 16);
    x += __shfl_xor(x, 32);
    if (kg == 0) u_s[wv * D + ft * 16 + r] = x;
  }
  lds_barrier();
  float* bp = (float*)(ws + g.off_bpart) + ((size_t)(p * g.Hkv + h) * g.n_build_chunks + ch) * ((size_t)D * (D + 1));
#pragma unroll
  for (int k = 0; k < FT * CT / NW; ++k) {
    const int t = wv * (FT * CT / NW) + k, ft = t / CT, ct = t % CT;
    floatx4 x = *(const floatx4*)(ring + t * 1024 + lane * 16);
#pragma unroll
    for (int w = 1; w < NW; ++w) x += *(const floatx4*)(ring + w * 2 * STAGE + t * 1024 + lane * 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) bp[(size_t)(ft * 16 + 4 * kg + i) * D + ct * 16 + r] = x[i];
  }
  if (tid < D) {
    float x = u_s[tid];
#pragma unroll
    for (int w = 1; w < NW; ++w) x += u_s[w * D + tid];
    bp[(size_t)D * D + tid] = x;
  }
}

// ------------------------------------------------------------------------------------
// fp32 arithmetic on the matrix cores (any storage type, any d_phi): grid (n_build_chunks, Hkv, n_problems),
// 4 wavefronts; wavefront w owns the feature tiles w, w + 4, ... (FTW = ceil(d_phi / 64) of them).
//
// Tiles of 64 tokens: the key and value rows are widened to fp32 into LDS (the next tile's loads are in flight while
// one is contracted).  Per 16 tokens:
//   GEMM1  P[16 tokens][16 features] = K Wk^T with v_mfma_f32_16x16x4_f32: the four inner indices of step
//          (jj, e) are the channels 16 jj + 4 kg + e, so one 16-byte read per lane feeds four steps
//   GEMM2  S[16 features][channels] += Phi^T V: GEMM1 leaves lane (r, kg) with feature r of the tokens
//          4 kg + i, which is the A operand of step i over the tokens {i, 4 + i, 8 + i, 12 + i}: the features never
//          touch LDS
// Rows are padded by 4 floats: the 16-byte reads of GEMM1 and the 4-byte reads of GEMM2 then spread over all banks.
// What bounds it: latency for the few tokens fp32 caches come with.  A VALU version with 16-token batches that read the
// Wk rows again for every batch, on chunks of 256 tokens, took 325 us for one head of 4028 tokens at d = 64
// (16 workgroups); this one, 63 chunks of 64 tokens, 8.5 us, and the call 328 -> 11.4 us.
// ------------------------------------------------------------------------------------
template <typename T, int D, int FTW>
__global__ __launch_bounds__(kThreads) void build_f32_kernel(BuildGeom g, const tkphi_problem* __restrict__ probs,
                                                             char* __restrict__ ws) {
  constexpr int TT = 64, ROWF = D + 4, EPL = Elem<T>::per16, SEGS = D / EPL, NLD = TT * SEGS / kThreads;
  constexpr int CT = D / 16;
  extern __shared__ __attribute__((aligned(16))) float lds_f[];      // keys [TT][ROWF], values [TT][ROWF]
  float* k_s = lds_f;
  float* v_s = lds_f + TT * ROWF;
  const int ch = blockIdx.x, h = blockIdx.y, p = blockIdx.z, tid = threadIdx.x;
  const tkphi_problem pr = probs[p];
  if (pr.L < 1 || pr.L > g.max_L) return;
  const int n = mid_size(pr.L, g.n_sink, g.n_tail);
  const int c0 = ch * g.build_chunk;
  if (c0 >= n) return;
  const int c1 = min(n, c0 + g.build_chunk);
  const int dphi = g.dphi, NFT = dphi / 16;
  const int lane = tid & 63, wv = tid >> 6, r = lane & 15, kg = lane >> 4;

  const int64_t base = (int64_t)h * pr.stride_head + (int64_t)g.n_sink * pr.stride_tok;
  u32x4 kr[NLD], vr[NLD];
  auto request = [&](int t0) {                       // rows past the end repeat the last one
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int idx = tid + i * kThreads;
      const int64_t off = base + (int64_t)min(t0 + idx / SEGS, c1 - 1) * pr.stride_tok + (idx % SEGS) * EPL;
      kr[i] = gload128((const char*)pr.K + off * sizeof(T));
      vr[i] = gload128((const char*)pr.V + off * sizeof(T));
    }
  };
  auto commit = [&](int t0) {                        // -> LDS as fp32; rows past the end as zeros
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int idx = tid + i * kThreads, row = idx / SEGS;
      const bool ok = t0 + row < c1;
      float x[EPL], y[EPL];
      Elem<T>::unpack(make_uint4(kr[i].x, kr[i].y, kr[i].z, kr[i].w), x);
      Elem<T>::unpack(make_uint4(vr[i].x, vr[i].y, vr[i].z, vr[i].w), y);
      float* kd = k_s + row * ROWF + (idx % SEGS) * EPL;
      float* vd = v_s + row * ROWF + (idx % SEGS) * EPL;
#pragma unroll
      for (int e = 0; e < EPL; e += 4) {
        *(floatx4*)(kd + e) = ok ? (floatx4){x[e], x[e + 1], x[e + 2], x[e + 3]} : (floatx4){0.f, 0.f, 0.f, 0.f};
        *(floatx4*)(vd + e) = ok ? (floatx4){y[e], y[e + 1], y[e + 2], y[e + 3]} : (floatx4){0.f, 0.f, 0.f, 0.f};
      }
    }
  };
  request(c0);

  // this wavefront's slice of Wk (lane (r, kg): feature r of a tile, channels 16 jj + 4 kg ..); at d_phi > 128 it does not
  // fit the registers beside S and is read again per 16 tokens (from L1 / L2)
  constexpr bool W_REG = FTW * D <= 256;
  constexpr int WN = W_REG ? FTW : 1;
  floatx4 wk[WN][CT];
  float bias[FTW];
  auto load_w = [&](int k, floatx4 (&w)[CT]) {
    const int64_t wrow = ((int64_t)h * dphi + min(wv + 4 * k, NFT - 1) * 16 + r) * D;
#pragma unroll
    for (int jj = 0; jj < CT; ++jj) {
      if (sizeof(T) == 4) {
        const u32x4 t = gload128((const char*)pr.Wk + (wrow + jj * 16 + kg * 4) * 4);
        w[jj] = (floatx4){__uint_as_float(t.x), __uint_as_float(t.y), __uint_as_float(t.z), __uint_as_float(t.w)};
      } else {
        const u32x2 t = *(const __attribute__((address_space(1))) u32x2*)((const char*)pr.Wk + (wrow + jj * 16 + kg * 4) * 2);
        w[jj] = (floatx4){__uint_as_float(t.x << 16), __uint_as_float(t.x & 0xffff0000u), __uint_as_float(t.y << 16),
                          __uint_as_float(t.y & 0xffff0000u)};
      }
    }
  };
#pragma unroll
  for (int k = 0; k < FTW; ++k) {
    if (W_REG) load_w(k, wk[W_REG ? k : 0]);
    bias[k] = pr.bk[(int64_t)h * dphi + min(wv + 4 * k, NFT - 1) * 16 + r];
  }
  floatx4 sacc[FTW][CT];
  float uacc[FTW];
#pragma unroll
  for (int k = 0; k < FTW; ++k) {
    uacc[k] = 0.f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) sacc[k][ct] = (floatx4){0.f, 0.f, 0.f, 0.f};
  }

  for (int t0 = c0; t0 < c1; t0 += TT) {
    if (t0 != c0) __syncthreads();                   // the previous tile's readers are done
    commit(t0);
    __syncthreads();
    if (t0 + TT < c1) request(t0 + TT);
    float ut[FTW];                                   // this tile's share of u
#pragma unroll
    for (int k = 0; k < FTW; ++k) ut[k] = 0.f;
#pragma unroll 1
    for (int mt = 0; mt < TT / 16; ++mt) {
      if (t0 + mt * 16 >= c1) break;
      floatx4 a[CT];
      float nrm = 0.f;
#pragma unroll
      for (int jj = 0; jj < CT; ++jj) {
        a[jj] = *(const floatx4*)(k_s + (mt * 16 + r) * ROWF + jj * 16 + kg * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) nrm = fmaf(a[jj][e], a[jj][e], nrm);
      }
      nrm += __shfl_xor(nrm, 16);
      nrm += __shfl_xor(nrm, 32);                    // |k|^2 of token r
      float cn[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) cn[i] = g.c * __shfl(nrm, 4 * kg + i);
      const int tok = t0 + mt * 16 + 4 * kg;
      floatx4 f[FTW];                                // feature (wv + 4 k) 16 + r of tokens 4 kg + i
#pragma unroll
      for (int k = 0; k < FTW; ++k) {
        if (!W_REG) load_w(k, wk[0]);
        // (four chains of D / 16 steps instead of one of D / 4: shorter to wait for, and less rounding in the exponent)
        floatx4 acc[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int jj = 0; jj < CT; ++jj)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[jj][e], wk[W_REG ? k : 0][jj][e], acc[e], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float dot = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
          f[k][i] = tok + i < c1 ? expf(g.a * dot - cn[i] + bias[k]) : 0.f;
        }
        ut[k] += (f[k][0] + f[k][1]) + (f[k][2] + f[k][3]);
        if (g.cache && wv + 4 * k < NFT) {
          float* cp = pr.phi_cache + ((size_t)h * n + tok) * dphi + (wv + 4 * k) * 16 + r;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (tok + i < c1) cp[(size_t)i * dphi] = f[k][i];
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float* vrow = v_s + (mt * 16 + 4 * kg + i) * ROWF + r;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const float v = vrow[ct * 16];
#pragma unroll
          for (int k = 0; k < FTW; ++k) sacc[k][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[k][i], v, sacc[k][ct], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < FTW; ++k) uacc[k] += ut[k];
  }

  float* bp = (float*)(ws + g.off_bpart) + ((size_t)(p * g.Hkv + h) * g.n_build_chunks + ch) * ((size_t)dphi * (D + 1));
#pragma unroll
  for (int k = 0; k < FTW; ++k) {
    const int ft = wv + 4 * k;
    if (ft < NFT) {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int i = 0; i < 4; ++i) bp[(size_t)(ft * 16 + 4 * kg + i) * D + ct * 16 + r] = sacc[k][ct][i];
      float x = uacc[k];
      x += __shfl_xor(x, 16);
      x += __shfl_xor(x, 32);
      if (kg == 0) bp[(size_t)dphi * D + ft * 16 + r] = x;
    }
  }
}

// sums the chunk partials of each (problem, KV head) in a fixed order.
// grid (ceil(dphi*(d+1)/4 / 64) + 1, Hkv, n_problems), 256 threads = 64 float4 elements x 4 chunk
// groups: group q sums chunks q*16 .. q*16+15 of every 64 (16 loads in flight), then the four
// group sums are added in group order.  The last workgroup of the first row writes the device status.
// What bounds it at one problem is a chain of round trips (arguments, problem record, partials, result): so the record's pointers
// are asked for with the length, and the first partials of a single problem before the length is there (its chunks nearly always
// fill the bounds; what lies behind them is not added): one fp32 head of 4K tokens 12.3 -> 11.4 us per call.
__global__ __launch_bounds__(kThreads) void build_reduce_kernel(BuildGeom g, const tkphi_problem* __restrict__ probs,
                                                                char* __restrict__ ws) {
  __shared__ float4 sh[4][64];
  const int h = blockIdx.y, p = blockIdx.z;
  if (blockIdx.x == gridDim.x - 1) {
    if (h == 0 && p == 0) write_device_status(g, probs, ws, false);
    return;
  }
  const int L = probs[p].L;
  float* S = probs[p].S;
  float* u = probs[p].u;
  const int d = g.d, dphi = g.dphi;
  const size_t per = (size_t)dphi * (d + 1);          // floats per partial (a multiple of 4)
  const int el = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const size_t e4 = (size_t)blockIdx.x * 64 + el;     // float4 index inside a partial
  const bool live = e4 * 4 < per;
  const float4* bp = (const float4*)((const float*)(ws + g.off_bpart) + ((size_t)(p * g.Hkv + h) * g.n_build_chunks) * per) +
                     (live ? e4 : 0);
  const size_t per4 = per / 4;
  auto request = [&](int c0, int last, float4 (&v)[16]) {
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = bp[(size_t)min(c0 + grp * 16 + k, last) * per4];
  };
  float4 v[16];
  if (g.n_problems == 1) request(0, g.n_build_chunks - 1, v);
  asm volatile("" : : "s"(L), "s"(S), "s"(u));
  if (L < 1 || L > g.max_L) return;
  const int n = mid_size(L, g.n_sink, g.n_tail);
  const int n_chunks = (n + g.build_chunk - 1) / g.build_chunk;
  if (g.n_problems != 1 && n_chunks > 0) request(0, n_chunks - 1, v);
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int c0 = 0; c0 < n_chunks; c0 += 64) {
    if (c0 > 0) request(c0, n_chunks - 1, v);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      if (c0 + grp * 16 + k < n_chunks) { acc.x += v[k].x; acc.y += v[k].y; acc.z += v[k].z; acc.w += v[k].w; }
    }
  }
  sh[grp][el] = acc;
  __syncthreads();
  if (grp != 0 || !live) return;
  float4 s = sh[0][el];
#pragma unroll
  for (int q = 1; q < 4; ++q) { s.x += sh[q][el].x; s.y += sh[q][el].y; s.z += sh[q][el].z; s.w += sh[q][el].w; }
  const size_t e = e4 * 4;
  if (e < (size_t)dphi * d) *(float4*)(S + (size_t)h * dphi * d + e) = s;
  else *(float4*)(u + (size_t)h * dphi + (e - (size_t)dphi * d)) = s;
}

template <bool CACHE, int NS>
static void launch_build_mfma_as(const Geom& g, const tkphi_problem* probs, char* ws, dim3 grid, hipStream_t s) {
  const size_t lds = (size_t)NS * (2 * 32 * 128 * 2 + 32 * 4);
  const hipError_t e = hipFuncSetAttribute((const void*)build_mfma_kernel<CACHE, NS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) { set_error("hipFuncSetAttribute(%zu bytes of LDS): %s", lds, hipGetErrorString(e)); return; }
  TKPHI_LAUNCH(ST_UNTIMED, (build_mfma_kernel<CACHE, NS>), grid, dim3(256), lds, s, BuildGeom(g), probs, ws);
}
template <int NW, bool CACHE>
static void launch_build_mfma64(const Geom& g, const tkphi_problem* probs, char* ws, dim3 grid, hipStream_t s) {
  constexpr size_t lds = NW * 16384 + 64 * 128 + 64 * 4;
  const hipError_t e = hipFuncSetAttribute((const void*)build_mfma64_kernel<NW, CACHE>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) { set_error("hipFuncSetAttribute(%zu bytes of LDS): %s", lds, hipGetErrorString(e)); return; }
  TKPHI_LAUNCH(ST_UNTIMED, (build_mfma64_kernel<NW, CACHE>), grid, dim3(64 * NW), lds, s, BuildGeom(g), probs, ws);
}
static void launch_build_mfma(const Geom& g, const tkphi_problem* probs, char* ws, dim3 grid, hipStream_t s) {
  constexpr int NS = 4;                  // ring stages: three tiles on their way while one is contracted
  if (g.d == 128 && g.cache) launch_build_mfma_as<true, NS>(g, probs, ws, grid, s);
  else if (g.d == 128) launch_build_mfma_as<false, NS>(g, probs, ws, grid, s);
  else if (g.cache) launch_build_mfma64<4, true>(g, probs, ws, grid, s);
  else launch_build_mfma64<4, false>(g, probs, ws, grid, s);
}

template <typename T, int D>
static void launch_build_f32_d(const Geom& g, const tkphi_problem* probs, char* ws, dim3 grid, hipStream_t s) {
  constexpr size_t lds = (size_t)2 * 64 * (D + 4) * sizeof(float);
  const int ftw = (g.dphi + 63) / 64;    // feature tiles per wavefront: 1, 2 or (3, 4 ->) 4
  const auto fn = ftw <= 1 ? build_f32_kernel<T, D, 1> : ftw == 2 ? build_f32_kernel<T, D, 2> : build_f32_kernel<T, D, 4>;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) { set_error("hipFuncSetAttribute(%zu bytes of LDS): %s", lds, hipGetErrorString(e)); return; }
  }
  TKPHI_LAUNCH(ST_UNTIMED, fn, grid, dim3(kThreads), lds, s, BuildGeom(g), probs, ws);
}
template <typename T>
static void launch_build_f32(const Geom& g, const tkphi_problem* probs, char* ws, dim3 grid, hipStream_t s) {
  if (g.d == 128) launch_build_f32_d<T, 128>(g, probs, ws, grid, s);
  else launch_build_f32_d<T, 64>(g, probs, ws, grid, s);
}

void launch_build(const Geom& g, const tkphi_problem* probs, char* ws, hipStream_t s) {
  if (g.max_mid > 0) {
    dim3 grid(g.n_build_chunks, g.Hkv, g.n_problems);
    if (g.phi_kind == TKPHI_PHI_MLP) {
      launch_mlp_build(g, probs, ws, s);            // phi_k of the mid-region, then S, u chunk partials from the features
    } else if (g.use_mfma) {
      launch_build_mfma(g, probs, ws, grid, s);
    } else if (g.dtype == TKPHI_BF16) {
      launch_build_f32<uint16_t>(g, probs, ws, grid, s);
    } else {
      launch_build_f32<float>(g, probs, ws, grid, s);
    }
  }
  const int per4 = g.dphi * (g.d + 1) / 4;
  dim3 rgrid((per4 + 63) / 64 + 1, g.Hkv, g.n_problems);
  TKPHI_LAUNCH(ST_UNTIMED, build_reduce_kernel, rgrid, dim3(kThreads), 0, s, BuildGeom(g), probs, ws);
}

}  // namespace tkphi
