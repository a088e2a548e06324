// Matrix-core score tiles shared by the filtered score pass and the select kernel's rescan:
// s_i = q . k_i / sqrt(d_h) (eq. (full_attention)) for the mid-region rows of one wavefront's share
// of a score chunk, with the candidates of the Top-K selection appended to per-wavefront lists.
#pragma once

#include "tkphi_internal.h"

namespace tkphi {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 st_bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float st_floatx4;
typedef unsigned int st_u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) st_u32x2* lds_u32x2;
typedef __attribute__((address_space(1))) st_u32x2* glb_u32x2;
typedef __attribute__((address_space(1))) float* glb_f32;
typedef __attribute__((address_space(3))) float* lds_f32;
typedef __attribute__((address_space(3))) st_floatx4* lds_f32x4;
union ScoreFrag {
  u32x4 u;
  st_bf16x8 v;
};

// The score contraction of 16 rows, in one of two layouts of the key loads.
// LINES: a load instruction covers 8 rows x 128 bytes, whole cache lines: lane (r, kg) takes 16 bytes of row r mod 8, in the first
// half of its line for r < 8, in the second for r >= 8; eight lanes of the first eight rows' register then change places with eight of
// the second eight rows', which makes the plain operands of both.
// Otherwise 16 rows x 64 bytes, the plain operand layout (lane (r, kg): row r, channels 32 j + 8 kg ..), which requests every line twice.
// Either way a score is the same sum in the same order, bit for bit: the bound that a call samples in one layout prunes what it scores in
// the other, and a mid-region that is sampled whole has its K-th score itself for a bound.
// Streaming 6 GB of 128- or 256-byte rows: whole lines 7.2 to 7.3 TB/s with non-temporal loads and 6.4 with plain ones, half lines 6.0
// and 6.4; so non-temporal loads come with LINES, and where plain ones are right (keys that the caches hold until the select
// kernel reads its share again) the plain layout saves the moves: 1B layer at 64K 33.7 us per step against 34.6.
template <int D> constexpr int kTileFrags = D / 32;
// the query heads' operand: lane (r, kg) holds the channels 32 j + 8 kg .. of head h G + r
template <int D>
__device__ __forceinline__ void load_query_frags(const Geom& g, const tkphi_problem& pr, int h, ScoreFrag (&bq)[kTileFrags<D>]) {
  const int lane = threadIdx.x & 63, r = lane & 15, kg = lane >> 4;
#pragma unroll
  for (int j = 0; j < kTileFrags<D>; ++j) {
    bq[j].u = (u32x4){0u, 0u, 0u, 0u};
    if (r < g.G) bq[j].u = gload128((const uint16_t*)pr.q + (size_t)(h * g.G + r) * D + j * 32 + kg * 8);
  }
}
// bytes that the lane adds to the address of its row
template <bool LINES>
__device__ __forceinline__ int score_lane_offset() {
  return (LINES ? ((threadIdx.x >> 3) & 1) * 64 : 0) + ((threadIdx.x >> 4) & 3) * 16;
}
// row_of(i): address of row i of the tile plus score_lane_offset(); LINES: non-temporal
template <int D, bool LINES, typename RowOf>
__device__ __forceinline__ void request_tile(ScoreFrag (&f)[kTileFrags<D>], RowOf&& row_of) {
  if constexpr (LINES) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const char* rp = row_of(u * 8 + (int)(threadIdx.x & 7));
#pragma unroll
      for (int j = 0; j < D / 64; ++j) f[2 * j + u].u = gload128_stream(rp + j * 128);
    }
  } else {
    const char* rp = row_of((int)(threadIdx.x & 15));
#pragma unroll
    for (int j = 0; j < D / 32; ++j) f[j].u = gload128(rp + j * 64);
  }
}
// unscaled scores: lane (r < G, kg) gets those of head r and the rows 4 kg + {0 .. 3}
template <int D, bool LINES>
__device__ __forceinline__ st_floatx4 score_tile(const ScoreFrag (&f)[kTileFrags<D>], const ScoreFrag (&bq)[kTileFrags<D>]) {
  st_floatx4 p = (st_floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < kTileFrags<D>; j += 2) {
    ScoreFrag a = f[j], b = f[j + 1];
    if constexpr (LINES) {
      // lanes 8 .. 15 of each row of 16 of the one <-> lanes 0 .. 7 of the other (row_ror:8 into two banks of four lanes)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        a.u[e] = (uint32_t)__builtin_amdgcn_update_dpp((int)f[j].u[e], (int)f[j + 1].u[e], 0x128, 0xf, 0xc, false);
        b.u[e] = (uint32_t)__builtin_amdgcn_update_dpp((int)f[j + 1].u[e], (int)f[j].u[e], 0x128, 0xf, 0x3, false);
      }
    }
    p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, bq[j].v, p, 0, 0, 0);
    p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b.v, bq[j + 1].v, p, 0, 0, 0);
  }
  return p;
}

// Candidate lists of the filtered selection.  A score chunk is scanned by four wavefront slots; slot
// `wslot` of chunk `chunk` appends, per query head, every token whose order-preserving score key is
// >= that head's lower bound to its own list (capacity: the slot's tokens, scan_chunk / 4), in the
// fixed order it visits them, and finally stores the list length.  No atomics: a list has one writer.
// Entry i of a list lives in a compact array (i < cand_T: what the select kernel reads in one sweep)
// or at position i of the list's full-capacity region.
__device__ __forceinline__ size_t cand_region(const Geom& g, int gq, int chunk, int wslot) {
  return (((size_t)gq * g.n_scan_chunks + chunk) * 4 + wslot) * (size_t)(g.scan_chunk / 4);
}

// One wavefront: slot `wslot` of chunk `chunk` of KV head h (n mid tokens, n_chunks chunks).
//   edge_r   lower bound of the score key for the query head of this lane's column r (ignored for r >= G)
//   strip    null, or this wavefront's LDS strip of G x cand_T entries: the compact heads of the G lists are
//            collected there and go to memory at the end as whole lines (a head is cand_T contiguous entries, the
//            four slots of a chunk adjoin), instead of one 8-byte store per candidate scattered through the scan:
//            fewer partly written lines for the L2 to write back in the middle of the read stream
// Lane (r, kg) ends up with the scores of head r for tokens base + t 16 + 4 kg + i, so each list is
// written by the four lanes of its column, in the order (unit, t, i, kg).
// SUB: 16-token tiles loaded and contracted together; NB: groups of SUB tiles in registers, NB - 1 of them on their way while one
// is contracted; STREAM: non-temporal loads of whole lines
// STRIP: `strip` is used (a template parameter, and address spaces spelled out on every pointer stored through: a store that
// might go to LDS or to memory becomes a flat store, after which the compiler waits for every load in flight)
// DIRECT: no bound and no lists; every score goes to the head's row of Geom::off_scores
template <int D, int TPI, int SUB, int NB, bool STREAM, bool STRIP, bool DIRECT = false>
__device__ __forceinline__ void scan_wave_slot(const Geom& g, const tkphi_problem& pr, char* blk, int h, int n, int n_chunks,
                                               int chunk, int wslot, const ScoreFrag (&bq)[kTileFrags<D>], uint32_t edge_r, lds_u32x2 strip) {
  constexpr int TOK = TPI * 16;         // tokens per wavefront and unit
  const int lane = threadIdx.x & 63, r = lane & 15, kg = lane >> 4;
  const int G = g.G;
  const bool col_live = r < G;
  const int gq = h * G + min(r, G - 1);
  const glb_u32x2 list = (glb_u32x2)(blk + g.off_candf) + cand_region(g, gq, chunk, wslot);
  const glb_u32x2 head = (glb_u32x2)(blk + g.off_candc) + (((size_t)gq * g.n_scan_chunks + chunk) * 4 + wslot) * (size_t)g.cand_T;
  const int cap = g.scan_chunk / 4, T = g.cand_T;
  const glb_f32 score_row = (glb_f32)(blk + g.off_scores) + (size_t)gq * g.mid_stride;   // (DIRECT)
  const uint64_t col_lanes = 0x0001000100010001ull << r;     // the four lanes of this column
  const uint64_t lanes_below = (1ull << lane) - 1ull;
  const size_t row_bytes = (size_t)pr.stride_tok * 2;
  const char* Kb = (const char*)pr.K + ((size_t)h * pr.stride_head + (size_t)g.n_sink * pr.stride_tok) * 2;
  const float scale = g.score_scale;
  const glb_f32 export_row = pr.scores ? (glb_f32)(pr.scores + (size_t)gq * n) : (glb_f32) nullptr;
  int cnt = 0;                          // length of this column's list (the same in its four lanes)

  // A score is first compared as a float with the bound: false for what cannot be a candidate (NaN and the columns of no
  // head aside), two instructions and a branch; the branch decides exactly, by key.
  float edge_s;
  auto float_bound = [&]() { edge_s = !col_live || edge_r == 0xffffffffu ? INFINITY : edge_r == 0u ? -INFINITY : key_score(edge_r); };

  ScoreFrag a[NB][SUB][kTileFrags<D>];
  const char* const Kl = Kb + score_lane_offset<STREAM>();
  auto request = [&](int base, ScoreFrag (&f)[SUB][kTileFrags<D>]) {
#pragma unroll
    for (int t = 0; t < SUB; ++t)          // (rows past the end repeat the last one)
      request_tile<D, STREAM>(f[t], [&](int i) { return Kl + (uint64_t)(uint32_t)min(base + t * 16 + i, n - 1) * row_bytes; });
  };
  auto contract = [&](int base, const ScoreFrag (&f)[SUB][kTileFrags<D>]) {
    st_floatx4 acc[SUB];
#pragma unroll
    for (int t = 0; t < SUB; ++t) acc[t] = score_tile<D, STREAM>(f[t], bq);
    if constexpr (DIRECT) {
#pragma unroll
      for (int t = 0; t < SUB; ++t) {
        const int tok = base + t * 16 + 4 * kg;
        if (col_live && tok < n) {
          uint32_t e[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float s = fmaf(acc[t][i], scale, 0.0f);        // + 0.0f: -0 -> +0, equal scores get equal keys
            e[i] = __float_as_uint(s);
            if (export_row && tok + i < n) export_row[tok + i] = s;
          }
          typedef __attribute__((address_space(1))) u32x4* glb_u32x4;
          *(glb_u32x4)(score_row + tok) = (u32x4){e[0], e[1], e[2], e[3]};       // (the row is padded to whole groups of 64)
        }
      }
      return;
    }
#pragma unroll
    for (int t = 0; t < SUB; ++t) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int tok = base + t * 16 + 4 * kg + i;
        const float s = fmaf(acc[t][i], scale, 0.0f);          // + 0.0f: -0 -> +0, equal scores get equal keys
        if (export_row && col_live && tok < n) export_row[tok] = s;
        if (__ballot(!(s < edge_s))) {
          const bool pass = col_live && tok < n && score_key(s) >= edge_r;
          const uint64_t mine = __ballot(pass) & col_lanes;
          const int at = cnt + __popcll(mine & lanes_below);
          if (pass) {
            const st_u32x2 e = (st_u32x2){__float_as_uint(s), (uint32_t)tok};
            if (at < T) { if constexpr (STRIP) strip[min(r, G - 1) * T + at] = e; else head[at] = e; }
            else if (at < cap) list[at] = e;
          }
          cnt += __popcll(mine);
        }
      }
    }
  };
  // groups of SUB tiles in the order (unit, group of the unit); units past the end of a chunk's tokens end the pass (their
  // first tokens only grow with k)
  constexpr int GPU = TPI / SUB;
  const int n_groups = g.scan_chunk / (4 * TOK) * GPU;
  auto group_base = [&](int q) { return q < n_groups ? chunk_unit_token(g, n_chunks, chunk, q / GPU) + wslot * TOK + (q % GPU) * SUB * 16 : n; };
  static_assert(NB > 1, "one group on its way while another is contracted");
  // (requests and contractions are unconditional - past the end they repeat the last row, whose tokens are then dead - so that
  // the compiler can count the loads in flight on every path)
  int bases[NB];
#pragma unroll
  for (int u = 0; u < NB - 1; ++u) { bases[u] = group_base(u); request(bases[u], a[u]); }
  float_bound();                         // (behind the first requests: the bound itself is still on its way)
  for (int q = 0; bases[0] < n; q += NB) {
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      constexpr int kAhead = NB - 1;
      bases[(u + kAhead) % NB] = group_base(q + u + kAhead);
      request(bases[(u + kAhead) % NB], a[(u + kAhead) % NB]);
      __builtin_amdgcn_sched_barrier(0);
      contract(bases[u], a[u]);
    }
  }
  if constexpr (STRIP) {                // (LDS operations of one wavefront execute in order: no barrier)
    for (int gl = 0; gl < G; ++gl) {
      const int c = min(__shfl(cnt, gl), T);          // lane gl is lane (r = gl, kg = 0) of column gl
      const glb_u32x2 hd = (glb_u32x2)(blk + g.off_candc) + (((size_t)(h * G + gl) * g.n_scan_chunks + chunk) * 4 + wslot) * (size_t)T;
      for (int i = lane; i < c; i += 64) hd[i] = strip[gl * T + i];
    }
  }
  if constexpr (DIRECT) return;
  if (col_live && kg == 0)
    ((uint32_t*)(blk + g.off_ccount))[((size_t)gq * g.n_scan_chunks + chunk) * 4 + wslot] = (uint32_t)min(cnt, cap);
}

// The score pass of a workgroup of NWV wavefronts that learns the bounds only at its end (Geom::fused): all unscaled scores of
// the chunk stay in LDS, keep[head of the group][position], position = token's place in the order of the chunk's units.
// The wavefronts draw groups of SUB tiles from a counter in LDS: of two workgroups that share a CU the older one gets its loads
// served first, so that with a fixed share for each the second half ran alone for the last quarter of the pass (3B layer at 128K: the
// older ones done after 33 us, the younger after 44).
// Non-temporal loads (above) also leave the lists, phi_q and the problem record in the caches for the select kernel.
template <int D, int SUB, int NWV, bool STREAM>
__device__ __forceinline__ void scan_keep(const Geom& g, const tkphi_problem& pr, int h, int n, int n_chunks, int chunk,
                                          const ScoreFrag (&bq)[kTileFrags<D>], lds_f32 keep, int* next /*LDS, NWV*/) {
  constexpr int GT = SUB * 16;
  const int lane = threadIdx.x & 63, r = lane & 15, kg = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const size_t row_bytes = (size_t)pr.stride_tok * 2;
  const char* const Kl = (const char*)pr.K + ((size_t)h * pr.stride_head + (size_t)g.n_sink * pr.stride_tok) * 2 + score_lane_offset<STREAM>();
  constexpr int per_unit = keep_unit(D) / GT;
  const int n_groups = g.scan_chunk / GT;
  auto group_base = [&](int q) { return q < n_groups ? chunk_unit_token(g, n_chunks, chunk, q / per_unit) + (q % per_unit) * GT : n; };
  auto draw = [&]() {
    int q = 0;
    if (lane == 0) q = atomicAdd(next, 1);
    return __builtin_amdgcn_readfirstlane(q);
  };
  ScoreFrag a[2][SUB][kTileFrags<D>];
  auto request = [&](int base, ScoreFrag (&f)[SUB][kTileFrags<D>]) {      // (unconditional: rows past the end repeat the last one)
#pragma unroll
    for (int t = 0; t < SUB; ++t)
      request_tile<D, STREAM>(f[t], [&](int i) { return Kl + (uint64_t)(uint32_t)min(base + t * 16 + i, n - 1) * row_bytes; });
  };
  auto contract = [&](int q, int base, const ScoreFrag (&f)[SUB][kTileFrags<D>]) {
    st_floatx4 acc[SUB];
#pragma unroll
    for (int t = 0; t < SUB; ++t) acc[t] = score_tile<D, STREAM>(f[t], bq);
    if (r < g.G && base < n) {
#pragma unroll
      for (int t = 0; t < SUB; ++t) *(lds_f32x4)(keep + r * g.scan_chunk + q * GT + t * 16 + 4 * kg) = acc[t];
    }
  };
  int q[2], base[2];
  q[0] = wv;
  base[0] = group_base(q[0]);
  request(base[0], a[0]);
  while (base[0] < n) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      q[u ^ 1] = draw();
      base[u ^ 1] = group_base(q[u ^ 1]);
      request(base[u ^ 1], a[u ^ 1]);
      __builtin_amdgcn_sched_barrier(0);
      contract(q[u], base[u], a[u]);
    }
  }
}

// The lists of a chunk whose scores scan_keep left in LDS, once the bounds are known (lane gl < G: the bound of head h G + gl):
// list (head, slot) takes the positions [slot, slot + 1) scan_chunk / 4, 1024 of them at a time: a lane marks which of its 16 (4 of
// every 256) pass, one prefix sum over the lanes places them (a ballot and a store per four positions took 5 us of the pass of
// a 3B layer at 128K instead of 1).  A list is in the order (1024 positions, lane, position).
// known_lane: false where the bound has not come: kNoList in the place of a count, whose head the select kernel rescans (lists without a
// bound beside lists with one could make up K candidates that are not the K best).
constexpr uint32_t kNoList = 0xffffffffu;
template <int D, int NWV>
__device__ __forceinline__ void list_kept(const Geom& g, const tkphi_problem& pr, char* blk, int h, int n, int n_chunks, int chunk,
                                          lds_f32 keep, uint32_t edge_lane, bool known_lane) {
  const int lane = threadIdx.x & 63, slot = g.scan_chunk / 4, T = g.cand_T;
  constexpr int U = keep_unit(D);        // = g.scan_unit
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int first = chunk_unit_token(g, n_chunks, chunk, 0), step = chunk_unit_token(g, n_chunks, chunk, 1) - first;
  auto token = [&](int pos) { return first + pos / U * step + pos % U; };
  auto score = [&](float x) { return fmaf(x, g.score_scale, 0.0f); };        // + 0.0f: -0 -> +0, equal scores get equal keys
  if (pr.scores) {
    for (int gl = 0; gl < g.G; ++gl)
      for (int pos = threadIdx.x; pos < g.scan_chunk; pos += NWV * 64)
        if (token(pos) < n) ((glb_f32)pr.scores)[(size_t)(h * g.G + gl) * n + token(pos)] = score(keep[gl * g.scan_chunk + pos]);
  }
  for (int job = wv; job < 4 * g.G; job += NWV) {
    const int gl = job >> 2, ws = job & 3, gq = h * g.G + gl, pos0 = ws * slot + 4 * lane;
    const uint32_t edge = (uint32_t)__builtin_amdgcn_readlane((int)edge_lane, gl);
    const size_t idx = ((size_t)gq * g.n_scan_chunks + chunk) * 4 + ws;
    if (!__builtin_amdgcn_readlane((int)known_lane, gl)) {
      if (lane == 0) ((uint32_t*)(blk + g.off_ccount))[idx] = kNoList;
      continue;
    }
    const glb_u32x2 list = (glb_u32x2)(blk + g.off_candf) + idx * (size_t)slot;
    const glb_u32x2 head = (glb_u32x2)(blk + g.off_candc) + idx * (size_t)T;
    const lds_f32 row = keep + gl * g.scan_chunk + ws * slot;
    const bool plain = edge >= 0x80000000u;      // the bound is a score >= 0: keys compare as the scores' bits do, as integers
    const int edge_bits = (int)(edge & 0x7fffffffu);
    int cnt = 0;
    for (int o = 0; o < slot; o += 1024) {
      st_floatx4 s4[4];
      uint32_t live = 0, pass = 0;         // bit 4 k + i: position o + 256 k + 4 lane + i
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int at4 = o + 256 * k + 4 * lane;
        s4[k] = *(lds_f32x4)(row + min(at4, slot - 4));
        const int left = at4 < slot ? n - token(pos0 + o + 256 * k) : 0;      // (positions of dead tokens may hold anything)
        live |= ((1u << min(max(left, 0), 4)) - 1u) << (4 * k);
      }
      if (plain) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int i = 0; i < 4; ++i) pass |= __float_as_int(score(s4[k][i])) >= edge_bits ? 1u << (4 * k + i) : 0u;
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int i = 0; i < 4; ++i) pass |= score_key(score(s4[k][i])) >= edge ? 1u << (4 * k + i) : 0u;
      }
      pass &= live;
      const int mine = __popc(pass), incl = wave_scan_incl(mine);
      int at = cnt + incl - mine;
      while (pass) {
        const int b = __builtin_ctz(pass), in_slot = o + 64 * (b & 12) + 4 * lane + (b & 3);
        const st_u32x2 e = (st_u32x2){__float_as_uint(score(row[in_slot])), (uint32_t)token(ws * slot + in_slot)};
        if (at < T) head[at] = e;
        else list[at] = e;
        ++at;
        pass &= pass - 1;
      }
      cnt += __builtin_amdgcn_readlane(incl, 63);
    }
    if (lane == 0) ((uint32_t*)(blk + g.off_ccount))[idx] = (uint32_t)cnt;
  }
}

// Smallest score key whose first-level bin is >= t (key_bin is monotone in the key), so that
// "bin(key) >= t" is the single comparison "key >= bin_lower_key(t)".  t <= 0: every key; t >= kBins: none.
__device__ __forceinline__ uint32_t bin_lower_key(int t) {
  auto mag_edge = [](int mb) { return ((uint32_t)(kExpLo + mb / 16) << 23) | ((uint32_t)(mb % 16) << 19); };
  if (t <= 0) return 0u;
  if (t >= kBins) return 0xffffffffu;
  if (t >= kMagBins) { const int mb = t - kMagBins; return 0x80000000u | (mb == 0 ? 0u : mag_edge(mb)); }
  const int M = kMagBins - 1 - t;       // negative scores: magnitude bins 0 .. M qualify
  return 0x7fffffffu - (mag_edge(M + 1) - 1u);
}

}  // namespace tkphi
