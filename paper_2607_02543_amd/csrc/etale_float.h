// Float embeddings (inner-product similarity) for the ETALE kernels on gfx950.
//
// Distance d(a, b) = 1 - <a, b>; for unit vectors this is half the squared L2
// distance, so RobustPrune's alpha^2 rule reads the same on either. The FP32
// master rows decide everything that is stored (neighbor order, slab
// distances, RobustPrune, the re-rank); traversal may read a bf16 copy or an
// FP8 e4m3 copy with one FP32 scale per vector, always accumulating in FP32
// against the FP32 query.
//
// Rows are split into 16-byte chunks; G lanes share a row, each lane taking 3
// chunks (t*G + lane%G, t = 0..2), so a dimension of 96 * 2^j (j <= 3) maps
// onto a power-of-two G for all three element widths.
#pragma once

#include "etale_dev.h"

namespace etale {

enum Trav { TRAV_NATIVE = 0, TRAV_BF16 = 1, TRAV_FP8 = 2 };

// Order-preserving map of an FP32 value onto uint32, so (distance, id) keys
// compare as integers.
__host__ __device__ inline uint32_t fkey(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__host__ __device__ inline float fkey_inv(uint32_t k) {
  uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
  return __builtin_bit_cast(float, u);
}

// ---- number formats -------------------------------------------------------------------

// bfloat16 by round-to-nearest-even of the dropped 16 bits (NaN stays NaN)
__device__ inline uint16_t to_bf16(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (uint16_t)((u >> 16) | 0x40u);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// OCP FP8 E4M3FN (bias 7, no infinities, largest finite 448): round to
// nearest even on the binary32 bit pattern, saturating to +-448.
__device__ inline uint8_t to_e4m3(float y) {
  const uint32_t u = __builtin_bit_cast(uint32_t, y);
  const uint32_t sign = (u >> 24) & 0x80u;
  const uint32_t a = u & 0x7FFFFFFFu;
  if (a > 0x7F800000u) return 0x7F;                 // NaN
  if (a >= 0x43E00000u) return (uint8_t)(sign | 0x7Eu);  // >= 448
  if (a < 0x3C800000u) {                            // below 2^-6: multiples of 2^-9
    const float m = __builtin_rintf(__builtin_bit_cast(float, a) * 512.0f);  // exact scaling, ties to even
    return (uint8_t)(sign | (uint32_t)m);           // m == 8 is the smallest normal
  }
  int e = (int)(a >> 23) - 127;                     // -6 .. 8
  uint32_t m3 = (a >> 20) & 7u;
  const uint32_t rem = a & 0xFFFFFu;
  if (rem > 0x80000u || (rem == 0x80000u && (m3 & 1u))) ++m3;
  if (m3 == 8u) {
    m3 = 0;
    ++e;
  }
  if (e > 8 || (e == 8 && m3 == 7u)) return (uint8_t)(sign | 0x7Eu);
  return (uint8_t)(sign | ((uint32_t)(e + 7) << 3) | m3);
}

// e4m3fn code -> value / 256, exact: the code's low 7 bits shifted into a
// binary16 exponent/mantissa pattern give the same value scaled by 2^-8
// (subnormals included).
__device__ inline float e4m3_div256(uint32_t c) {
  const uint16_t h = (uint16_t)(((c & 0x80u) << 8) | ((c & 0x7Fu) << 7));
  return (float)__builtin_bit_cast(_Float16, h);
}

// Eight per-lane partial sums reduced together over the G lanes of each group:
// lane l ends with the group's total of v[l % 8]. Three reduce-scatter steps
// (lanes l ^ 1, l ^ 2, l ^ 4, each halving the values a lane carries) and then
// the plain exchanges past 8 lanes: the pairs are added in group_sum's order,
// so every total has the bits group_sum gives, in a third of its instructions.
template <int G>
__device__ inline float group_sum8(const float (&v)[8]) {
  static_assert(G >= 8, "at least eight lanes share a row");
  const int l = lane_id();
  const bool b0 = l & 1, b1 = l & 2, b2 = l & 4;
  float w[4], x[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = (b0 ? v[2 * i + 1] : v[2 * i]) + lane_xor<1>(b0 ? v[2 * i] : v[2 * i + 1]);
#pragma unroll
  for (int i = 0; i < 2; ++i) x[i] = (b1 ? w[2 * i + 1] : w[2 * i]) + lane_xor<2>(b1 ? w[2 * i] : w[2 * i + 1]);
  float t = (b2 ? x[1] : x[0]) + lane_xor<4>(b2 ? x[0] : x[1]);
  if constexpr (G > 8) t += lane_xor<8>(t);
  if constexpr (G > 16) t += lane_xor<16>(t);
  if constexpr (G > 32) t += lane_xor<32>(t);
  return t;
}

// ---- traversal distance: G lanes per row, 3 chunks per lane --------------------------------
// UMAX: rows per lane group in flight at most (the re-rank, once per query, takes
// four, so that it does not set its kernel's registers)
template <int G, int TRAV, int UMAX = 8>
struct TravF {
  static constexpr int EPC = TRAV == TRAV_NATIVE ? 4 : (TRAV == TRAV_BF16 ? 8 : 16);  // elements per chunk
  static constexpr int CPL = 3;
  static constexpr int VPP = 64 / G;
  // rows per lane group in flight together: eight where eight lanes or more
  // share a row (their sums are then reduced together), 64 rows in all below
  static constexpr int U = G < UMAX ? G : UMAX;
  struct Q {
    float v[CPL][EPC];
  };

  __device__ static Q load_query(const float* q) {
    Q r;
    const int c = lane_id() % G;
#pragma unroll
    for (int t = 0; t < CPL; ++t)
#pragma unroll
      for (int e = 0; e < EPC; ++e) r.v[t][e] = q[(size_t)(t * G + c) * EPC + e];
    return r;
  }

  __device__ static const uint4* row(const Index& ix, uint32_t id) {
    if (TRAV == TRAV_NATIVE) return reinterpret_cast<const uint4*>(ix.xf + (size_t)id * ix.dim);
    if (TRAV == TRAV_BF16) return reinterpret_cast<const uint4*>(ix.xb + (size_t)id * ix.dim);
    return reinterpret_cast<const uint4*>(ix.x8 + (size_t)id * ix.dim);
  }

  // this lane's share of <q, row> (FP8: of <q, row/scale>/256). FP8 codes are
  // converted two at a time by the hardware, 1/256 with them (the query holds
  // every bit it came with: components below 2^-118 would lose some at 1/256),
  // which reads 0x7F and 0xFF as NaN: EXACT_CODES decodes them by their bit
  // pattern (to +-480) instead
  template <bool EXACT_CODES = false>
  __device__ static float partial(const Q& q, const uint4 (&w)[CPL]) {
    float acc = 0.f;
#pragma unroll
    for (int t = 0; t < CPL; ++t) {
      const uint32_t wd[4] = {w[t].x, w[t].y, w[t].z, w[t].w};
      if constexpr (TRAV == TRAV_NATIVE) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_fmaf(q.v[t][e], __builtin_bit_cast(float, wd[e]), acc);
      } else if constexpr (TRAV == TRAV_BF16) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc = __builtin_fmaf(q.v[t][2 * e], __builtin_bit_cast(float, wd[e] << 16), acc);
          acc = __builtin_fmaf(q.v[t][2 * e + 1], __builtin_bit_cast(float, wd[e] & 0xFFFF0000u), acc);
        }
      } else if constexpr (EXACT_CODES) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            acc = __builtin_fmaf(q.v[t][4 * e + b], e4m3_div256((wd[e] >> (8 * b)) & 0xFFu), acc);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const auto lo = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(wd[e], 0x1p-8f, false);
          const auto hi = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(wd[e], 0x1p-8f, true);
          acc = __builtin_fmaf(q.v[t][4 * e], lo[0], acc);
          acc = __builtin_fmaf(q.v[t][4 * e + 1], lo[1], acc);
          acc = __builtin_fmaf(q.v[t][4 * e + 2], hi[0], acc);
          acc = __builtin_fmaf(q.v[t][4 * e + 3], hi[1], acc);
        }
      }
    }
    return acc;
  }

  __device__ static float scale(const Index& ix, uint32_t id) {
    return TRAV == TRAV_FP8 ? ix.xs[id] * 256.0f : 1.0f;
  }

  // The keys of rows [from, to) of a batch with a NaN in it: from a NaN code, which
  // FP8 decodes by bit pattern, or from the vectors, and then its sign (by which it
  // sorts first or last) hangs on the order of the sum. Both are settled a row at
  // a time, as lane 0 of the row's group sums it. (The lane's number is read
  // again: kept for this it takes a register of the sum's, and some searches a
  // wave per SIMD.)
  __device__ static void settle_nans(const Index& ix, const Q& q, const uint32_t* ids, int from, int to, uint64_t* ck) {
    int ln;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
    const int cl = ln % G;
#pragma unroll 1
    for (int base = from; base < to; base += VPP) {
      const int vi = base + ln / G;
      uint4 x[CPL];
#pragma unroll
      for (int t = 0; t < CPL; ++t) x[t] = vi < to ? row(ix, ids[vi])[t * G + cl] : make_uint4(0, 0, 0, 0);
      const float d = group_sum_t<G, float>(partial<TRAV == TRAV_FP8>(q, x));
      if (cl == 0 && vi < to) ck[vi] = make_key(fkey(1.0f - scale(ix, ids[vi]) * d), ids[vi]);
    }
  }
  // looked for after every pass where a pass takes most of a batch, else at its end
  // (768-d FP32, 100 queries, L = 64: 575 us after every pass, 550; 96-d 161 and 165)
  static constexpr bool PER_PASS = G <= 16;

  // Keys (d, id) of ids[0..cnt) and, if cr, their reference words. The batch is
  // bound by the latency of its gathers, so U VPP rows are in flight together
  // (2 VPP before), and for FP8 was bound by decoding each code in six
  // instructions (now 1.5, two codes per conversion). Beam search of 2,000
  // queries, 768-d FP8, L = 96: 2.39 -> 0.90 ms (with the larger visited
  // table); 120 insert searches, 768-d FP32: 2.43 -> 1.08; 100 queries, bf16:
  // 1.72 -> 0.84; 3,001 queries, 96-d FP32: 0.49 -> 0.36 (2,000 rows of 384
  // bytes per query: 6.4 TB/s past L2).
  __device__ static void dist_batch(const Index& ix, const Q& q, const uint32_t* ids, int cnt, uint64_t* ck,
                                    uint64_t* cr) {
    const int l = lane_id();
    const int c = l % G, grp = l / G;
    bool nan = false;
    for (int base = 0; base < cnt; base += U * VPP) {
      const int used = min(U, (cnt - base + VPP - 1) / VPP);  // the others are skipped (uniform branches)
      uint4 w[U][CPL];
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int t = 0; t < CPL; ++t) w[u][t] = make_uint4(0, 0, 0, 0);
        if (u < used) {
          const int vi = base + u * VPP + grp;
          if (vi < cnt) {
            const uint4* rw = row(ix, ids[vi]);
#pragma unroll
            for (int t = 0; t < CPL; ++t) w[u][t] = rw[t * G + c];
          }
        }
      }
      // the row whose distance this lane writes, its scale and reference word
      // (U = 8: row l % 8 of the group's; otherwise one lane of the group per row)
      const int my = base + (U == 8 ? (l & 7) : c) * VPP + grp;
      const bool mine = c < U && my < cnt;
      const uint32_t id = mine ? ids[my] : 0u;
      float sc = 1.f;
      uint64_t r = 0;
      if (mine) {
        sc = scale(ix, id);
        if (cr) r = load_ref(ix, id);
      }
      float dot = 0.f;
      if constexpr (U == 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = u < used ? partial(q, w[u]) : 0.f;
        dot = group_sum8<G>(v);
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float d = group_sum_t<G, float>(partial(q, w[u]));
          if (c == u) dot = d;
        }
      }
      nan = nan || (mine && dot != dot);
      if (mine) {
        ck[my] = make_key(fkey(1.0f - sc * dot), id);
        if (cr) cr[my] = r;
      }
      if constexpr (PER_PASS) {
        if (__builtin_expect(ballot(nan) != 0, 0)) settle_nans(ix, q, ids, base, min(cnt, base + U * VPP), ck);
        nan = false;
      }
    }
    if constexpr (!PER_PASS) {
      if (__builtin_expect(ballot(nan) != 0, 0)) settle_nans(ix, q, ids, 0, cnt, ck);
    }
  }
};

// ---- exact FP32 rows (master copy): G lanes per row, 3 float4 chunks per lane --------------
template <int G>
struct RowF {
  static constexpr int CPL = 3;
  static constexpr int VPP = 64 / G;
  __device__ static void load(const Index& ix, uint32_t id, float4 (&f)[CPL]) {
    const float4* rw = reinterpret_cast<const float4*>(ix.xf + (size_t)id * ix.dim);
    const int c = lane_id() % G;
#pragma unroll
    for (int t = 0; t < CPL; ++t) f[t] = rw[t * G + c];
  }
  // this lane's share of <a, b>
  __device__ static float part(const float4 (&a)[CPL], const float4 (&b)[CPL]) {
    float acc = 0.f;
#pragma unroll
    for (int t = 0; t < CPL; ++t) {
      acc = __builtin_fmaf(a[t].x, b[t].x, acc);
      acc = __builtin_fmaf(a[t].y, b[t].y, acc);
      acc = __builtin_fmaf(a[t].z, b[t].z, acc);
      acc = __builtin_fmaf(a[t].w, b[t].w, acc);
    }
    return acc;
  }
  __device__ static float dotp(const float4 (&a)[CPL], const float4 (&b)[CPL]) {
    return group_sum_t<G, float>(part(a, b));
  }
};

// RobustPrune on FP32 rows, same selection rule as the uint8 variant: drop
// p, tombstones and duplicates; order by (d(p,c), id); keep at most
// prune_cap; keep c unless an earlier kept c' has a^2 d(c',c) <= b^2 d(p,c).
// The first nk candidates' keys (their distance to p, known to the caller) are
// already in s.keys.
//
// The ranked candidates are decided in blocks of eight: a block's rows stay in
// registers (every group of G lanes holds all eight, each lane its share), the
// kept rows pass by VPP at a time, and each step gives 8 x VPP distances; then
// the block against itself, and the eight are decided in order. A candidate is
// only ever compared with kept ones ranked before it, and nothing is computed
// past the R-th kept one, where testing every kept row against all later
// candidates costs three times the distances when few are covered. Each
// distance adds its products in the order of RowF::dotp, so the bits and with
// them the kept set are those of the one-at-a-time selection.
// Bound: the latency of the row loads (24 in flight per block) and FP32 issue
// (about 125 instructions per step); eight rows because sixteen would leave one
// wave per SIMD. Against one kept row at a time with its rows loaded VPP at a
// time: at 12,000 x 768-d, 120 deletes and inserts, repair 14.8 -> 1.57 ms,
// reverse edges 4.49 -> 0.78, forward 1.83 -> 0.12, refine 0.94 -> 0.12; at
// 100,000 x 96-d, 1,000 and 1,000, 2.38 -> 0.63, 0.92 -> 0.37, 0.16 -> 0.026,
// 0.079 -> 0.026.
template <int G>
__device__ inline int robust_prune_f32(const Index& ix, uint32_t p, const uint32_t* cand, int n, PruneLds& s,
                                       int nk = 0) {
  using RF = RowF<G>;
  constexpr int VPP = RF::VPP;
  const int l = lane_id();
  const int grp = l / G, i8 = l & 7;
  const int np = next_pow2_ge64(n);
  // 1. keys: flags first (64 candidates' in flight together), then the
  // distances not known yet, 8 x VPP rows in flight together
  for (int i = l; i < np; i += 64) {
    const uint32_t id = i < n ? cand[i] : NONE;
    const bool drop = id == NONE || id == p || del_bit(ix, id);
    if (drop) s.keys[i] = KEY_NONE;
    else if (i >= nk) s.keys[i] = 0;
  }
  wave_sync();
  if (nk < n) {
    float4 pf[3];
    RF::load(ix, p, pf);
    for (int base = nk; base < n; base += 8 * VPP) {
      float v[8];
      float4 xf[8][3];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int vi = base + u * VPP + grp;
#pragma unroll
        for (int t = 0; t < 3; ++t) xf[u][t] = make_float4(0, 0, 0, 0);
        if (vi < n && s.keys[vi] != KEY_NONE) RF::load(ix, cand[vi], xf[u]);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = RF::part(pf, xf[u]);
      const float dot = group_sum8<G>(v);
      const int vi = base + i8 * VPP + grp;
      const bool mine = (l % G) < 8 && vi < n && s.keys[vi] != KEY_NONE;
      const uint64_t nan = ballot(mine && dot != dot);
      if (mine) s.keys[vi] = make_key(fkey(1.0f - dot), cand[vi]);
      if (__builtin_expect(nan != 0, 0)) {  // a NaN's sign: as lane 0 of the row's group sums it
#pragma unroll 1
        for (int u = 0; u < 8; ++u) {
          const int vu = base + u * VPP + grp;
          const bool in = vu < n && s.keys[vu] != KEY_NONE;
          if (in) RF::load(ix, cand[vu], xf[0]);
          const float d = RF::dotp(pf, xf[0]);
          if (in && l % G == 0) s.keys[vu] = make_key(fkey(1.0f - d), cand[vu]);
        }
      }
    }
    wave_sync();
  }
  // 2. order, drop duplicates (equal keys are adjacent), at most prune_cap
  int m = 0;
  auto compact = [&](uint64_t k, uint64_t prev, bool first) {
    const bool keep = k != KEY_NONE && (first || prev != k);
    const uint64_t bm = ballot(keep);
    const int at = m + (int)lanes_below(bm);
    if (keep && at < s.rows) s.keys2[at] = k;
    m += __popcll(bm);
  };
  if (np <= 128) {  // in registers, one or two keys per lane
    uint64_t v[2] = {s.keys[l], np > 64 ? s.keys[64 + l] : KEY_NONE};
    if (np > 64) {
      wave_sort_regs<2>(v);
    } else {
      uint64_t (&v1)[1] = *reinterpret_cast<uint64_t(*)[1]>(&v[0]);
      wave_sort_regs<1>(v1);
    }
    // every lane takes part in the shifts: a DPP reads nothing from an inactive one
    const uint64_t last = bcast_lane64(v[0], 63), p0 = lane_shr1_64(v[0]), p1 = lane_shr1_64(v[1]);
    compact(v[0], p0, l == 0);
    if (np > 64) compact(v[1], l == 0 ? last : p1, false);
  } else {
    wave_bitonic_sort(s.keys, np);
    for (int base = 0; base < np; base += 64) {
      const int i = base + l;
      compact(s.keys[i], i ? s.keys[i - 1] : 0ull, i == 0);
    }
  }
  wave_sync();
  if (m > (int)ix.prune_cap) m = (int)ix.prune_cap;
  if (m > s.rows) m = s.rows;
  // 3. the selection, eight candidates at a time
  const float a2 = (float)ix.a2, b2 = (float)ix.b2;
  const int R = (int)ix.R;
  int cnt = 0;
  for (int r0 = 0; r0 < m && cnt < R; r0 += 8) {
    const int nb = min(8, m - r0);
    const uint64_t ki = r0 + i8 < m ? s.keys2[r0 + i8] : KEY_NONE;  // lane l: the block's candidate l % 8
    const uint32_t idi = key_id(ki);
    const float thr = b2 * fkey_inv(key_dist(ki));
    float4 a[8][3];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t id = (uint32_t)__builtin_amdgcn_readlane((int)idi, i);
#pragma unroll
      for (int t = 0; t < 3; ++t) a[i][t] = make_float4(0, 0, 0, 0);
      if (i < nb) RF::load(ix, id, a[i]);
    }
    // the kept rows against the block
    bool cov = false;
    float4 b[3], bn[3];
    auto load_kept = [&](int k0, float4 (&f)[3]) {
      const int k = k0 + grp;
#pragma unroll
      for (int t = 0; t < 3; ++t) f[t] = make_float4(0, 0, 0, 0);
      if (k < cnt) RF::load(ix, s.out_ids[k], f);
    };
    if (cnt) load_kept(0, b);
    for (int k0 = 0; k0 < cnt; k0 += VPP) {
      if (k0 + VPP < cnt) load_kept(k0 + VPP, bn);
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = RF::part(a[i], b);
      const float dji = 1.0f - group_sum8<G>(v);
      if (k0 + grp < cnt && a2 * dji <= thr) cov = true;
#pragma unroll
      for (int t = 0; t < 3; ++t) b[t] = bn[t];
    }
    uint64_t cm = ballot(cov);
    cm |= cm >> 32;
    cm |= cm >> 16;
    cm |= cm >> 8;
    uint32_t alive = ((1u << nb) - 1u) & ~(uint32_t)cm;
    // the block against itself: row j = st VPP + group against all eight. The
    // first eight lanes of a group hold the eight results of its row
    uint64_t by[8 / VPP];  // bits of group g: the block's candidates its row covers
#pragma unroll
    for (int st = 0; st < 8 / VPP; ++st) {
      if constexpr (VPP == 1) {
#pragma unroll
        for (int t = 0; t < 3; ++t) b[t] = a[st][t];
      } else {
        const uint32_t id = (uint32_t)__shfl((int)idi, st * VPP + grp, 64);
#pragma unroll
        for (int t = 0; t < 3; ++t) b[t] = make_float4(0, 0, 0, 0);
        if (st * VPP + grp < nb) RF::load(ix, id, b);
      }
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = RF::part(a[i], b);
      const float dji = 1.0f - group_sum8<G>(v);
      by[st] = ballot(a2 * dji <= thr);
    }
    // the eight in order: a kept one drops the later ones it covers
    uint32_t kept = 0;
    int left = R - cnt;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t later = ((uint32_t)(by[j / VPP] >> ((j % VPP) * G)) & 0xFFu) & ~((2u << j) - 1u);
      if (((alive >> j) & 1u) && left > 0) {
        kept |= 1u << j;
        --left;
        alive &= ~later;
      }
    }
    if (l < 8 && ((kept >> l) & 1u)) {
      const int at = cnt + __popc(kept & ((1u << l) - 1u));
      s.out_ids[at] = idi;
      s.out_d[at] = __builtin_bit_cast(uint32_t, fkey_inv(key_dist(ki)));
    }
    cnt += __popc(kept);
    wave_sync();
  }
  wave_sync();
  return cnt;
}

// exact FP32 d(w, v) between stored rows, as the bit pattern stored in a slab
template <int G>
__device__ inline uint32_t dist1_f32(const Index& ix, uint32_t w, uint32_t v) {
  float4 a[3], b[3];
  RowF<G>::load(ix, w, a);
  RowF<G>::load(ix, v, b);
  const float d = 1.0f - RowF<G>::dotp(a, b);
  return __builtin_bit_cast(uint32_t, d);
}

}  // namespace etale
