// Gates and reverse steps on a tile of amplitudes in LDS, on the FP32 matrix
// cores: the code of the whole-circuit evaluation of small states
// (small_eval.hip), which have too few fibres for a lane each (fibre_gate.h), and
// the sums that it shares with the fused runs of gates on larger ones.
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
// no exchange between lanes.  The matrix operand is two table entries per lane,
// the same for every fibre, so a wavefront reads it once a gate.  On vector ALUs,
// with the block tables broadcast from LDS, a gate reads b^2 table entries a block
// beside its 2 b members (LDS-bound), and packed FP32, the other way to the full
// FP32 rate, is off in this build.
#pragma once

#include "gate_kernels.h"
#include "tile_pair.h"

namespace fock {

constexpr int kTileWaves = 16;  // wavefronts of a workgroup, at most

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Levels per group slot (2, 4 or 8) and units per gate.
__host__ __device__ constexpr int tile_slots(int D) { return D <= 2 ? 2 : (D <= 4 ? 4 : 8); }
__host__ __device__ constexpr int tile_units(int D) {
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

// What a lane does in every gate, by cutoff and unit: a compile-time table (its
// divisions and block sums would cost a workgroup more than a gate).  Offsets
// are dwords into a packed two-mode table (0xffff: none).
struct TileLaneWord {
  uint32_t fwd, dag;    // operand entry (row, slot) and (slot, row) of slots 2g, 2g + 1
  uint32_t link, diag;  // generator entries: links (2g, 2g + 1), (2g + 1, 2g + 2); slots 2g, 2g + 1
  uint32_t levels;      // 3-bit levels and flags, see tile_lane
};
constexpr int kTileMinD = 2, kTileMaxD = 8;

constexpr int tile_block_off(int s, int D) {  // packed offset (entries) of block s
  int off = 0;
  for (int t = 0; t < s; ++t) {
    const int b = t < D ? t + 1 : 2 * D - 1 - t;
    off += b * b;
  }
  return off;
}
// Packed entry (m + up, m) of group g, or -1: member m is n_i = m, in block g
// (m <= g) or g + D.
constexpr int tile_entry(int D, int g, int p, int q) {
  if (g >= D || p >= D || q >= D || (p <= g) != (q <= g)) return -1;
  const bool lo = p <= g;
  const int b = lo ? g + 1 : D - 1 - g, o = lo ? 0 : g + 1;
  return tile_block_off(lo ? g : g + D, D) + (p - o) * b + (q - o);
}
constexpr TileLaneWord tile_lane_word(int D, int unit, int lane) {
  TileLaneWord w{0, 0, 0, 0, 0};
  const int dp = tile_slots(D), per = 8 / dp, g = lane >> 4, row = lane & 15, im = row & 1;
  const int pg = unit * per + (row >> 1) / dp, pm = (row >> 1) % dp;
  uint32_t lv = im ? 1u << 31 : 0u;
  for (int e = 0; e < 3; ++e) {  // slots 2g, 2g + 1 and, for the second link, 2g + 2
    const int q = 2 * g + e, qg = unit * per + q / dp, qm = q % dp;
    const bool ok = q < 8 && qg < D && qm < D;
    const uint32_t ni = ok ? qm : 0, njs = ok ? (qg - qm + D) % D : 0, njd = ok ? (qm - qg - 1 + D) % D : 0;
    lv |= ni << (3 * e) | njs << (9 + 3 * e) | njd << (18 + 3 * e);
    if (e == 2) break;
    if (ok) lv |= 1u << (27 + e);
    const int f = ok && pg == qg ? tile_entry(D, qg, pm, qm) : -1, r = ok && pg == qg ? tile_entry(D, qg, qm, pm) : -1;
    if (f >= 0) lv |= 1u << (29 + e);
    w.fwd |= (uint32_t)(f >= 0 ? 2 * f + im : 0) << (16 * e);
    w.dag |= (uint32_t)(r >= 0 ? 2 * r + im : 0) << (16 * e);
    const int k = ok && (q + 1) / dp == q / dp ? tile_entry(D, qg, qm + 1, qm) : -1, d = ok ? tile_entry(D, qg, qm, qm) : -1;
    w.link |= (uint32_t)(k >= 0 ? 2 * k : 0xffff) << (16 * e);
    w.diag |= (uint32_t)(d >= 0 ? 2 * d : 0xffff) << (16 * e);
  }
  w.levels = lv;
  return w;
}
struct TileLaneTable {
  TileLaneWord w[kTileMaxD - kTileMinD + 1][8][64];
  constexpr TileLaneTable() : w() {
    for (int D = kTileMinD; D <= kTileMaxD; ++D)
      for (int u = 0; u < tile_units(D); ++u)
        for (int l = 0; l < 64; ++l) w[D - kTileMinD][u][l] = tile_lane_word(D, u, l);
  }
};
static __device__ const TileLaneTable kTileLanes{};

struct TileLane {
  TileLaneWord w;
  int c0, cstep;           // the wave's first fibre chunk and the chunk stride
  bool ok0, ok1;           // slots 2g, 2g + 1 hold members
  bool whole;              // every lane's do
  unsigned keep0, keep1;   // 0: zero entry (row and slot in different blocks)
  unsigned neg_f, neg_d;   // sign bits of the forward and the adjoint operand
};
// The wave's unit is wave % units and its chunks are wave / units, + cstep, ..;
// nwaves / units whole rounds of waves work, the rest have no chunk.
__device__ __forceinline__ TileLane tile_lane(int D, int nwaves) {
  TileLane t;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int units = tile_units(D), round = wave / units;
  t.cstep = nwaves / units > 0 ? nwaves / units : 1;
  t.c0 = round < t.cstep ? round : 1 << 20;
  t.w = kTileLanes.w[D - kTileMinD][wave - round * units][lane];
  t.ok0 = t.w.levels & (1u << 27);
  t.ok1 = t.w.levels & (1u << 28);
  t.whole = D == 8 || D == 4;  // slots = groups x members
  t.keep0 = t.w.levels & (1u << 29) ? ~0u : 0u;
  t.keep1 = t.w.levels & (1u << 30) ? ~0u : 0u;
  t.neg_f = ~t.w.levels & 0x80000000u;
  t.neg_d = t.w.levels & 0x80000000u;
  return t;
}

// A lane's matrix operand for the four reduction steps: row (re or im) times
// (re, im) of its two slots.  Read as table entries (TileRaw) and finished by
// tile_mat.
struct TileRaw {
  unsigned e00, e01, e10, e11;
};
struct TileMat {
  float a0, a1, a2, a3;
};
template <bool DAG>
__device__ __forceinline__ TileRaw tile_raw(const float2 *U, const TileLane &t) {
  const unsigned *u = reinterpret_cast<const unsigned *>(U);
  const uint32_t o = DAG ? t.w.dag : t.w.fwd, o0 = o & 0xffffu, o1 = o >> 16;
  return {u[o0], u[o0 ^ 1], u[o1], u[o1 ^ 1]};
}
template <bool DAG>
__device__ __forceinline__ TileMat tile_mat(const TileRaw &r, const TileLane &t) {
  const unsigned n0 = DAG ? t.neg_d : 0u, n1 = DAG ? 0u : t.neg_f;
  return {__uint_as_float((r.e00 & t.keep0) ^ n0), __uint_as_float((r.e01 & t.keep0) ^ n1),
          __uint_as_float((r.e10 & t.keep1) ^ n0), __uint_as_float((r.e11 & t.keep1) ^ n1)};
}

// The generator's part of a reverse step.  A is tridiagonal in a block's
// members and its entries are all real (HR, PR) or all imaginary (HI, DH, PI,
// and the diagonal CK), anti-Hermitian: a link (m, m + 1) with entry a = A[m+1][m]
// gives Re(conj(l[m+1]) a p[m] - conj(l[m]) conj(a) p[m+1]).  A few FMAs per
// fibre, so this stays on the vector ALUs beside the products.
enum TileGen { TG_REAL, TG_IMAG, TG_DIAG };
__device__ __forceinline__ int tile_gen_kind(int type) {
  return type == FOCK_CK ? TG_DIAG : type == FOCK_HR || type == FOCK_PR ? TG_REAL : TG_IMAG;
}
struct TileGenW {
  float w0, w1;
};
__device__ __forceinline__ TileGenW tile_gen_raw(const float2 *A, const TileLane &t, int kind) {
  const uint32_t o = kind == TG_DIAG ? t.w.diag : t.w.link, o0 = o & 0xffffu, o1 = o >> 16;
  const float *a = reinterpret_cast<const float *>(A) + (kind == TG_REAL ? 0 : 1);
  return {a[o0 != 0xffffu ? o0 : 0u], a[o1 != 0xffffu ? o1 : 0u]};
}
__device__ __forceinline__ TileGenW tile_gen(const TileGenW &r, const TileLane &t, int kind) {
  const uint32_t o = kind == TG_DIAG ? t.w.diag : t.w.link;
  return {(o & 0xffffu) != 0xffffu ? r.w0 : 0.f, (o >> 16) != 0xffffu ? r.w1 : 0.f};
}
// The lane's terms at one fibre: slots 0, 1, 2 of phi (v) and lambda (l).
template <int kind>
__device__ __forceinline__ float tile_gen_sum(const TileGenW &w, float2 v0, float2 v1, float2 v2, float2 l0, float2 l1,
                                              float2 l2) {
  if (kind == TG_REAL) {
    const float s0 = fmaf(l1.x, v0.x, fmaf(l1.y, v0.y, -fmaf(l0.x, v1.x, l0.y * v1.y)));
    const float s1 = fmaf(l2.x, v1.x, fmaf(l2.y, v1.y, -fmaf(l1.x, v2.x, l1.y * v2.y)));
    return fmaf(w.w0, s0, w.w1 * s1);
  }
  if (kind == TG_IMAG) {  // -a (Im conj(l1) v0 + Im conj(l0) v1)
    const float s0 = fmaf(l1.x, v0.y, fmaf(-l1.y, v0.x, fmaf(l0.x, v1.y, -l0.y * v1.x)));
    const float s1 = fmaf(l2.x, v1.y, fmaf(-l2.y, v1.x, fmaf(l1.x, v2.y, -l1.y * v2.x)));
    return -fmaf(w.w0, s0, w.w1 * s1);
  }
  return -fmaf(w.w0, fmaf(l0.x, v0.y, -l0.y * v0.x), w.w1 * fmaf(l1.x, v1.y, -l1.y * v1.x));
}

__device__ __forceinline__ f32x4 tile_mul(const TileMat &m, float2 v0, float2 v1) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(m.a0, v0.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(m.a1, v0.y, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(m.a2, v1.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(m.a3, v1.y, acc, 0, 0, 0);
  return acc;
}

__device__ __forceinline__ int tile_fibre(int f, const TilePair &p, int D) {
  const int t = tile_div(f, p.rsi), low = f - __mul24(t, p.si);
  const int high = tile_div(t, p.rdm), mid = t - __mul24(high, p.dm);
  return low + __mul24(__mul24(mid, p.si) + __mul24(high, p.sj), D);
}

// A gate as a wave applies it: the byte offsets of the lane's members (slots 2g,
// 2g + 1, 2g + 2) relative to a fibre's.  Offsets are positions times 8, so that
// an LDS address is one exclusive or (sum) and the state's base.
struct TileStep {
  int d0, d1, d2;
};
template <bool P2>
__device__ __forceinline__ TileStep tile_step(const TilePair &p, const TileLane &t, int kind) {
  const uint32_t ni = t.w.levels, nj = ni >> (kind == KIND_SUM ? 9 : 18);
  auto off = [&](int e) {
    return 8 * tile_pos<P2>(__mul24((ni >> (3 * e)) & 7, p.si) + __mul24((nj >> (3 * e)) & 7, p.sj));
  };
  TileStep s;
  s.d0 = off(0);
  s.d1 = off(1);
  s.d2 = off(2);
  return s;
}
__device__ __forceinline__ float2 &tile_amp(float2 *x, int byte) {
  return *reinterpret_cast<float2 *>(reinterpret_cast<char *>(x) + byte);
}

// phi <- U phi on the tile (m: the wave's operand of U; at(f): byte offset of
// fibre f).  Slots without a member and lanes beyond the last fibre read some
// amplitude of the tile: their matrix columns are zero, resp. their column is
// not written.
template <bool P2, class At>
__device__ __forceinline__ void tile_gate(float2 *phi, const TileLane &t, const TileStep &s, const TileMat &m, int nfib,
                                          At at) {
  for (int f0 = t.c0 * 16; f0 < nfib; f0 += t.cstep * 16) {
    const int f = f0 + (threadIdx.x & 15);
    const bool in = f < nfib;
    const int base = at(in ? f : 0);
    const int a0 = tile_at<P2>(base, s.d0), a1 = tile_at<P2>(base, s.d1);
    const f32x4 r = tile_mul(m, tile_amp(phi, a0), tile_amp(phi, a1));
    if (t.whole && f0 + 16 <= nfib) {  // every lane holds two members
      tile_amp(phi, a0) = make_float2(r[0], r[1]);
      tile_amp(phi, a1) = make_float2(r[2], r[3]);
    } else {
      if (in && t.ok0) tile_amp(phi, a0) = make_float2(r[0], r[1]);
      if (in && t.ok1) tile_amp(phi, a1) = make_float2(r[2], r[3]);
    }
  }
}

// Reverse step: returns this lane's share of Re<lam|A phi>, then phi <- U^+ phi
// and lam <- U^+ lam (m: operand of U^+; w: the generator's weights).
template <bool P2, int GEN, class At>
__device__ __forceinline__ float tile_adj_loop(float2 *phi, float2 *lam, const TileLane &t, const TileStep &s,
                                               const TileMat &m, const TileGenW &w, int nfib, At at) {
  float g = 0.f;
  for (int f0 = t.c0 * 16; f0 < nfib; f0 += t.cstep * 16) {
    const int f = f0 + (threadIdx.x & 15);
    const bool in = f < nfib;
    const int base = at(in ? f : 0);
    const int a0 = tile_at<P2>(base, s.d0), a1 = tile_at<P2>(base, s.d1), a2 = tile_at<P2>(base, s.d2);
    const float2 v0 = tile_amp(phi, a0), v1 = tile_amp(phi, a1), l0 = tile_amp(lam, a0), l1 = tile_amp(lam, a1);
    const float2 v2 = tile_amp(phi, a2), l2 = tile_amp(lam, a2);
    const f32x4 r = tile_mul(m, v0, v1);
    const f32x4 q = tile_mul(m, l0, l1);
    const float c = tile_gen_sum<GEN>(w, v0, v1, v2, l0, l1, l2);
    if (t.whole && f0 + 16 <= nfib) {
      g += c;
      tile_amp(phi, a0) = make_float2(r[0], r[1]);
      tile_amp(lam, a0) = make_float2(q[0], q[1]);
      tile_amp(phi, a1) = make_float2(r[2], r[3]);
      tile_amp(lam, a1) = make_float2(q[2], q[3]);
    } else {
      g += in ? c : 0.f;
      if (in && t.ok0) {
        tile_amp(phi, a0) = make_float2(r[0], r[1]);
        tile_amp(lam, a0) = make_float2(q[0], q[1]);
      }
      if (in && t.ok1) {
        tile_amp(phi, a1) = make_float2(r[2], r[3]);
        tile_amp(lam, a1) = make_float2(q[2], q[3]);
      }
    }
  }
  return g;
}
template <bool P2, class At>
__device__ __forceinline__ float tile_gate_adj(float2 *phi, float2 *lam, const TileLane &t, const TileStep &s,
                                               const TileMat &m, const TileGenW &raw, int gen, int nfib, At at) {
  const TileGenW w = tile_gen(raw, t, gen);
  if (gen == TG_REAL) return tile_adj_loop<P2, TG_REAL>(phi, lam, t, s, m, w, nfib, at);
  if (gen == TG_IMAG) return tile_adj_loop<P2, TG_IMAG>(phi, lam, t, s, m, w, nfib, at);
  return tile_adj_loop<P2, TG_DIAG>(phi, lam, t, s, m, w, nfib, at);
}

// Per-lane shares of up to 16 gates, summed in double over the wavefront by one
// FP64 matrix instruction a gate: row q of the 16 x 16 accumulator gathers gate
// q's 64 values in 16 column sums, which tile_sums_flush adds up once.
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kTileSums = 16;
__device__ __forceinline__ void tile_sums_add(f64x4 &acc, int q, float v) {
  const double sel = (int)(threadIdx.x & 15) == q ? 1.0 : 0.0;
  acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sel, (double)v, acc, 0, 0, 0);
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

// part[q][wave] = gate q's sum over the wave.  A product with the row numbers
// tells which row each lane's accumulator registers hold.
__device__ __forceinline__ void tile_sums_flush(const f64x4 &acc, double (*part)[kTileWaves]) {
  f64x4 row = {0.0, 0.0, 0.0, 0.0};
  row = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(threadIdx.x & 15), (threadIdx.x & 63) < 16 ? 1.0 : 0.0, row, 0, 0,
                                             0);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    double v = acc[r];
    v = dpp_add_d<0x111, 0xf>(v);
    v = dpp_add_d<0x112, 0xf>(v);
    v = dpp_add_d<0x114, 0xf>(v);
    v = dpp_add_d<0x118, 0xf>(v);
    if ((threadIdx.x & 15) == 15) part[(int)row[r]][threadIdx.x >> 6] = v;
  }
}

}  // namespace fock
