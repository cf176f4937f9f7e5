// Gates and reverse steps on a tile of amplitudes in LDS, on the FP32 matrix
// cores: the code shared by the whole-circuit evaluation of small states
// (small_eval.hip) and the fused runs of gates on larger ones (tile_runs.hip).
//
// A tile holds the amplitudes over a few modes (all D levels each, local index
// a = sum_k n_k D^k).  A two-mode gate on tile modes (i, j) mixes, in each of
// the tile's D^(modes - 2) fibres, the conserved blocks of Sec. II.B: blocks s
// and s + D of the 2D - 1 (sizes s + 1 and D - 1 - s) together hold one member
// for every n_i, at n_j = (s - n_i) mod D (kind SUM) or (n_i - s - 1) mod D
// (kind DIFF).  A fibre is thus D groups of D members, each under one D x D
// block-diagonal matrix.
//
// Eight member slots (one group at D > 4, two at D = 3, 4, four at D = 2) form
// a unit: a 16 x 16 real matrix on (re, im) rows, applied to 16 fibres by four
// v_mfma_f32_16x16x4_f32.  The reduction index is permuted so that lane l
// supplies and receives the same two slots 2 (l / 16) and 2 (l / 16) + 1 of
// fibre l % 16: it reads its two members, and writes them back in place, with
// no exchange between lanes.  The matrix operand is two table entries per
// lane, the same for every fibre, so it is loaded from global memory one gate
// ahead and needs no LDS.  With the block tables broadcast from LDS instead, a
// gate on vector ALUs reads b^2 table entries a block beside its 2 b members
// (LDS-bound), and packed FP32, the other way to the full FP32 rate, is off in
// this build.
#pragma once

#include "gate_kernels.h"

namespace fock {

constexpr int kTileWaves = 16;  // wavefronts of a workgroup, at most

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Levels per group slot (2, 4 or 8) and units per gate.
__host__ __device__ inline int tile_slots(int D) { return D <= 2 ? 2 : (D <= 4 ? 4 : 8); }
__host__ __device__ inline int tile_units(int D) {
  const int per = 8 / tile_slots(D);
  return (D + per - 1) / per;
}

// Wavefronts for a tile of T amplitudes: 16, or fewer when its fibre chunks
// cannot keep them busy (every wave issues each gate's description, operand and
// barrier; a wave takes one unit at least).
inline int tile_waves(int D, int T) {
  const int work = tile_units(D) * ((T / (D * D) + 15) / 16);
  return work > 8 ? 16 : tile_units(D) > 4 ? 8 : 4;
}

// LDS position of local index a.  At power-of-two D (P2) the five low bits are
// mixed with higher ones, so that fibres whose index strides are multiples of
// 32 float2 fall in different banks (mean conflict factor over all pairs of a
// 4-mode tile at D = 8: 5.0 without, 1.25 with; 6 modes at D = 4: 2.7 and 1.3;
// other D need no mixing: 1.7).  The mixing is linear over bits, and a fibre's
// base and a member's offset then have no bits in common: tile_at combines
// their positions.
template <bool P2>
__device__ __forceinline__ int tile_pos(int a) { return P2 ? a ^ (((a >> 3) ^ (a >> 5)) & 31) : a; }
template <bool P2>
__device__ __forceinline__ int tile_at(int base, int off) { return P2 ? base ^ off : base + off; }

// q = n / d for 0 <= n < 2^14 and d >= 1, with r = 1 / d: (n + 0.5) / d is at
// least 0.5 / d away from an integer, more than its rounding error.
__device__ __forceinline__ int tile_div(int n, float r) { return (int)(((float)n + 0.5f) * r); }

// What a lane does in every gate: its unit's two slots and, as a matrix row,
// the dword offsets of its entries in the packed blocks.
struct TileLane {
  int unit, c0, cstep;     // unit of the wave, its first fibre chunk and the chunk stride
  int ni[2], nj_s[2], nj_d[2];
  bool ok[2];
  int of[2], od[2];        // entry (row, slot), entry (slot, row): the part the row's (re or im) starts with
  unsigned keep[2];        // 0: zero entry (row and slot in different blocks)
  unsigned neg_f, neg_d;   // sign bits of the forward and the adjoint operand
};

__device__ __forceinline__ int tile_block_off(int s, int D) {  // packed offset of block s
  int off = 0;
  for (int t = 0; t < s; ++t) {
    const int b = t < D ? t + 1 : 2 * D - 1 - t;
    off += b * b;
  }
  return off;
}

__device__ __forceinline__ TileLane tile_lane(int D, int nwaves) {
  TileLane t;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int units = tile_units(D), dp = tile_slots(D), per = 8 / dp;
  t.unit = wave % units;
  t.cstep = nwaves / units > 0 ? nwaves / units : 1;
  t.c0 = wave / units < t.cstep ? wave / units : 1 << 20;  // waves beyond the last whole round rest
  const int g = lane >> 4, row = lane & 15;
  const int im = row & 1;
  t.neg_f = im ? 0u : 0x80000000u;
  t.neg_d = im ? 0x80000000u : 0u;
  const int ps = row >> 1, pg = t.unit * per + ps / dp, pm = ps % dp;  // the row's group and member
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int q = 2 * g + e, qg = t.unit * per + q / dp, qm = q % dp;
    t.ok[e] = qg < D && qm < D;
    t.ni[e] = t.ok[e] ? qm : 0;
    t.nj_s[e] = t.ok[e] ? (qg - qm + D) % D : 0;
    t.nj_d[e] = t.ok[e] ? (qm - qg - 1 + D) % D : 0;
    t.of[e] = t.od[e] = 0;
    t.keep[e] = 0u;
    if (t.ok[e] && pg == qg && pm < D && (pm <= pg) == (qm <= pg)) {
      const bool lo = pm <= pg;
      const int s = lo ? pg : pg + D, b = lo ? pg + 1 : D - 1 - pg;
      const int p0 = lo ? pm : pm - pg - 1, q0 = lo ? qm : qm - pg - 1;
      const int off = tile_block_off(s, D);
      t.of[e] = 2 * (off + p0 * b + q0) + im;
      t.od[e] = 2 * (off + q0 * b + p0) + im;
      t.keep[e] = ~0u;
    }
  }
  return t;
}

// A lane's matrix operand for the four reduction steps: row (re or im) times
// (re, im) of its two slots.
struct TileMat {
  float a[4];
};
template <bool DAG>
__device__ __forceinline__ TileMat tile_mat(const float2 *U, const TileLane &t) {
  const unsigned *u = reinterpret_cast<const unsigned *>(U);
  TileMat m;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int o = DAG ? t.od[e] : t.of[e];
    m.a[2 * e] = __uint_as_float((u[o] & t.keep[e]) ^ (DAG ? t.neg_d : 0u));
    m.a[2 * e + 1] = __uint_as_float((u[o ^ 1] & t.keep[e]) ^ (DAG ? 0u : t.neg_f));
  }
  return m;
}

__device__ __forceinline__ f32x4 tile_mul(const TileMat &m, float2 v0, float2 v1) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(m.a[0], v0.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(m.a[1], v0.y, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(m.a[2], v1.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(m.a[3], v1.y, acc, 0, 0, 0);
  return acc;
}

// Fibre decomposition of a gate on tile modes with strides si < sj: fibre
// f = low + si (mid + dm high), dm = sj / (si D).  Computed once per gate and
// launch (the divisions cost more than the gate on a small tile).
struct TilePair {
  int si, sj, dm;
  float rsi, rdm;
};
__device__ __forceinline__ TilePair tile_pair(int si, int sj, int D) {
  TilePair p;
  p.si = si;
  p.sj = sj;
  p.dm = sj / (si * D);
  p.rsi = 1.0f / (float)si;
  p.rdm = 1.0f / (float)p.dm;
  return p;
}
__device__ __forceinline__ int tile_fibre(int f, const TilePair &p, int D) {
  const int t = tile_div(f, p.rsi), low = f - __mul24(t, p.si);
  const int high = tile_div(t, p.rdm), mid = t - __mul24(high, p.dm);
  return low + __mul24(__mul24(mid, p.si) + __mul24(high, p.sj), D);
}

// A gate as a wave applies it: the positions of the lane's two members relative
// to a fibre's, and of the wave's first chunk of fibres.
struct TileStep {
  int d0, d1, base;
};
template <bool P2>
__device__ __forceinline__ TileStep tile_step(const TilePair &p, const TileLane &t, int kind, int nfib, int D) {
  TileStep s;
  s.d0 = tile_pos<P2>(__mul24(t.ni[0], p.si) + __mul24(kind == KIND_SUM ? t.nj_s[0] : t.nj_d[0], p.sj));
  s.d1 = tile_pos<P2>(__mul24(t.ni[1], p.si) + __mul24(kind == KIND_SUM ? t.nj_s[1] : t.nj_d[1], p.sj));
  const int f = t.c0 * 16 + (threadIdx.x & 15);
  s.base = tile_pos<P2>(tile_fibre(f < nfib ? f : 0, p, D));
  return s;
}

// phi <- U phi on the tile (m: the wave's operand of U).  Slots without a
// member and lanes beyond the last fibre read some amplitude of the tile: their
// matrix columns are zero, resp. their column is not written.
template <bool P2>
__device__ __forceinline__ void tile_gate(float2 *phi, const TilePair &p, const TileLane &t, const TileStep &s,
                                          const TileMat &m, int nfib, int D) {
  int f0 = t.c0 * 16;
  int a0 = tile_at<P2>(s.base, s.d0), a1 = tile_at<P2>(s.base, s.d1);
  float2 v0 = phi[a0], v1 = phi[a1];
  while (true) {
    const f32x4 r = tile_mul(m, v0, v1);
    const bool in = f0 + (int)(threadIdx.x & 15) < nfib;
    if (in && t.ok[0]) phi[a0] = make_float2(r[0], r[1]);
    if (in && t.ok[1]) phi[a1] = make_float2(r[2], r[3]);
    f0 += t.cstep * 16;
    if (f0 >= nfib) break;
    const int f = f0 + (threadIdx.x & 15);
    const int base = tile_pos<P2>(tile_fibre(f < nfib ? f : 0, p, D));
    a0 = tile_at<P2>(base, s.d0);
    a1 = tile_at<P2>(base, s.d1);
    v0 = phi[a0];
    v1 = phi[a1];
  }
}

// Reverse step: returns this lane's share of Re<lam|A phi>, then phi <- U^+ phi
// and lam <- U^+ lam (m: operand of U^+, ma: of A).
template <bool P2>
__device__ __forceinline__ float tile_gate_adj(float2 *phi, float2 *lam, const TilePair &p, const TileLane &t,
                                               const TileStep &s, const TileMat &m, const TileMat &ma, int nfib,
                                               int D) {
  int f0 = t.c0 * 16;
  int a0 = tile_at<P2>(s.base, s.d0), a1 = tile_at<P2>(s.base, s.d1);
  float2 v0 = phi[a0], v1 = phi[a1], l0 = lam[a0], l1 = lam[a1];
  float g = 0.f;
  while (true) {
    const f32x4 ap = tile_mul(ma, v0, v1);
    const f32x4 r = tile_mul(m, v0, v1);
    const f32x4 q = tile_mul(m, l0, l1);
    const bool in = f0 + (int)(threadIdx.x & 15) < nfib;
    const float c = fmaf(l0.x, ap[0], fmaf(l0.y, ap[1], fmaf(l1.x, ap[2], l1.y * ap[3])));
    g += in ? c : 0.f;
    if (in && t.ok[0]) {
      phi[a0] = make_float2(r[0], r[1]);
      lam[a0] = make_float2(q[0], q[1]);
    }
    if (in && t.ok[1]) {
      phi[a1] = make_float2(r[2], r[3]);
      lam[a1] = make_float2(q[2], q[3]);
    }
    f0 += t.cstep * 16;
    if (f0 >= nfib) break;
    const int f = f0 + (threadIdx.x & 15);
    const int base = tile_pos<P2>(tile_fibre(f < nfib ? f : 0, p, D));
    a0 = tile_at<P2>(base, s.d0);
    a1 = tile_at<P2>(base, s.d1);
    v0 = phi[a0];
    v1 = phi[a1];
    l0 = lam[a0];
    l1 = lam[a1];
  }
  return g;
}

// Sum over the wavefront in double by DPP moves (no LDS traffic), valid in lane 63.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add_d(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false);
  return v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double wave_total_d(double v) {
  v = dpp_add_d<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8: lane 15 of each row of 16 holds the row's sum
  v = dpp_add_d<0x112, 0xf>(v);
  v = dpp_add_d<0x114, 0xf>(v);
  v = dpp_add_d<0x118, 0xf>(v);
  v = dpp_add_d<0x142, 0xa>(v);  // row_bcast 15 into rows 1 and 3
  v = dpp_add_d<0x143, 0xc>(v);  // row_bcast 31 into rows 2 and 3
  return v;
}

}  // namespace fock
