// Two-mode gates and reverse steps on a tile of amplitudes in LDS, one fibre a
// lane: the code of the fused runs (tile_runs.hip).
//
// A gate on tile modes (i, j) mixes, in each of the tile's D^(modes - 2) fibres,
// the conserved blocks of Sec. II.B: blocks s = g and g + D of the 2 D - 1 hold
// together one member for every n_i, at n_j = (g - n_i) mod D (kind SUM) or
// (n_i - g - 1) mod D (kind DIFF).  A wavefront takes group g of 64 fibres: every
// lane holds its fibre's D members in registers, and the matrix of both blocks
// is the same for all lanes, so it is read through the scalar cache into scalar
// registers and costs neither LDS reads nor vector registers.  Blocks, sizes and
// parities are compile-time constants (one body per g).
//
// A matrix entry is one float: a generator links neighbouring levels only and is
// real antisymmetric (HR, PR) or i times real symmetric with no diagonal (HI, DH,
// PI), so an entry of exp(theta A) with an even number of links between row and
// column is real, with an odd number real or i times real (fuse_table).  A gate
// is then 2 fused multiply-adds for each of the 344 (D = 8; 146 at D = 6) entries
// of a fibre's blocks, at 64 lanes.  On the FP32 matrix cores the same gate
// needs the full 16 x 16 operand for 8 members (2.9, D = 6: 5.3 times the
// products at twice the rate, in cycles that the vector ALUs cannot use).
#pragma once

#include "fuse_internal.h"
#include "tile_gate.h"

namespace fock {

// Uniform data of earlier launches, read by scalar loads.
typedef const float __attribute__((address_space(4))) KFloat;
__device__ __forceinline__ KFloat *scalar_ptr(const void *p) {
  const uint64_t a = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  return (KFloat *)(((uint64_t)hi << 32) | lo);
}

template <int D>
__device__ __forceinline__ constexpr int run_pos(int a) { return run_pos(D, a); }
// Byte offset of a member of a fibre.
template <int D>
__device__ __forceinline__ int run_at(int base, int off) {
  return (D & (D - 1)) == 0 ? base ^ off : base + off;
}
// An amplitude at an LDS address: phi's start plus its byte offset, so that a
// member costs one instruction (an exclusive or combines positions because phi
// starts at 0: dynamic LDS is all that the kernels have, which the build checks in
// their assembly).  As pointers a member
// cost an addition more: 30 gates with gradients at 8^6 250 us, now 235, at 8^8
// 1,720 and 1,630.
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) f2 LdsAmp;
__device__ __forceinline__ float2 amp_load(int byte) {
  const f2 v = *(const LdsAmp *)(uint32_t)byte;
  return make_float2(v.x, v.y);
}
__device__ __forceinline__ void amp_store(int byte, float2 v) { *(LdsAmp *)(uint32_t)byte = f2{v.x, v.y}; }

// A gate's modes: byte offsets of 1, 2 and 4 levels of mode i and of mode j
// (other D: of one level).  Scalars.
template <int D>
struct ModeStep {
  static constexpr bool P2 = (D & (D - 1)) == 0;
  int i[3], j[3];
};
// Keeps what is computed from the steps beside its use: the offsets of every
// group's members, computed ahead for all cases, cost a wavefront more than its
// group.
template <int D>
__device__ __forceinline__ void pin_steps(ModeStep<D> &s) {
  if constexpr (ModeStep<D>::P2)
    asm volatile("" : "+s"(s.i[0]), "+s"(s.i[1]), "+s"(s.i[2]), "+s"(s.j[0]), "+s"(s.j[1]), "+s"(s.j[2]));
  else
    asm volatile("" : "+s"(s.i[0]), "+s"(s.j[0]));
}
// Byte offset of member m of group g (sum: kind SUM) relative to its fibre.
template <int D>
__device__ __forceinline__ int member_off(const ModeStep<D> &s, int g, int m, bool sum) {
  const int a = g - m + (m > g ? D : 0), b = m - g - 1 + (m > g ? 0 : D);
  if constexpr (ModeStep<D>::P2) {
    int o = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) o ^= ((m >> k) & 1 ? s.i[k] : 0) ^ (((sum ? a : b) >> k) & 1 ? s.j[k] : 0);
    return o;
  } else {
    return m * s.i[0] + (sum ? a : b) * s.j[0];
  }
}

// First entry of block s in a packed table.
template <int D>
__device__ __forceinline__ constexpr int block_off(int s) {
  const int t = D * (2 * D * D + 1) / 3, k = s < D ? s : 2 * D - 1 - s, q = k * (k + 1) * (2 * k + 1) / 6;
  return s < D ? q : t - q;
}

// y = rows of one block (members M0 .. M0 + B - 1) on x.  IM: entries of odd
// distance are i times the table's; DAG: the conjugate transpose.
template <int D, int M0, int B, bool IM, bool DAG>
__device__ __forceinline__ void block_rows(const float (&u)[B * B], const float2 (&x)[D], float2 (&y)[D]) {
#pragma unroll
  for (int r = 0; r < B; ++r) {
    float a = 0.f, b = 0.f;
#pragma unroll
    for (int c = 0; c < B; ++c) {
      const float w = DAG ? u[c * B + r] : u[r * B + c];
      const float2 v = x[M0 + c];
      const bool swap = IM && ((r - c) & 1);
      const float p = swap ? (DAG ? v.y : -v.y) : v.x, q = swap ? (DAG ? -v.x : v.x) : v.y;
      a = c == 0 ? w * p : fmaf(w, p, a);
      b = c == 0 ? w * q : fmaf(w, q, b);
    }
    y[M0 + r] = make_float2(a, b);
  }
}

// The links' share of Re<l|A x> in one block; A: the block's packed generator.
template <int D, int M0, int B, bool IM>
__device__ __forceinline__ float block_links(KFloat *A, const float2 (&x)[D], const float2 (&l)[D]) {
  float s = 0.f;
#pragma unroll
  for (int p = 0; p + 1 < B; ++p) {
    const float w = A[2 * ((p + 1) * B + p) + (IM ? 1 : 0)];
    const float2 x0 = x[M0 + p], x1 = x[M0 + p + 1], l0 = l[M0 + p], l1 = l[M0 + p + 1];
    const float t = IM ? fmaf(l1.y, x0.x, fmaf(-l1.x, x0.y, fmaf(l0.y, x1.x, -l0.x * x1.y)))
                       : fmaf(l1.x, x0.x, fmaf(l1.y, x0.y, -fmaf(l0.x, x1.x, l0.y * x1.y)));
    s = fmaf(w, t, s);
  }
  return s;
}

// Group G of one wavefront's fibres: phi <- U phi, or (REV) phi, lam <- U^+ and
// this lane's share of Re<lam|A phi>.  lam: distance from phi in bytes; u: the group's table; A: the generator's
// packed blocks; base: the lane's fibre (in: it has one).
template <int D, int G, bool SUM, bool IM, bool REV>
__device__ __forceinline__ float fibre_group(int lam, KFloat *u, KFloat *A, ModeStep<D> st,
                                             int base, bool in) {
  pin_steps<D>(st);
  constexpr int B0 = G + 1, B1 = D - 1 - G;
  float u0[B0 * B0], u1[B1 * B1 > 0 ? B1 * B1 : 1];
#pragma unroll
  for (int e = 0; e < B0 * B0; ++e) u0[e] = u[e];
#pragma unroll
  for (int e = 0; e < B1 * B1; ++e) u1[e] = u[B0 * B0 + e];
  int at[D];
  float2 x[D], y[D];
#pragma unroll
  for (int m = 0; m < D; ++m) {
    at[m] = run_at<D>(base, member_off<D>(st, G, m, SUM));
    x[m] = amp_load(at[m]);
  }
  float s = 0.f;
  if constexpr (REV) {
    float2 l[D], z[D];
#pragma unroll
    for (int m = 0; m < D; ++m) l[m] = amp_load(at[m] + lam);
    s = block_links<D, 0, B0, IM>(A + 2 * block_off<D>(G), x, l);
    if constexpr (B1 > 0) s += block_links<D, B0, B1, IM>(A + 2 * block_off<D>(G + D), x, l);
    block_rows<D, 0, B0, IM, true>(u0, x, y);
    block_rows<D, 0, B0, IM, true>(u0, l, z);
    if constexpr (B1 > 0) {
      block_rows<D, B0, B1, IM, true>(u1, x, y);
      block_rows<D, B0, B1, IM, true>(u1, l, z);
    }
    if (in) {
#pragma unroll
      for (int m = 0; m < D; ++m) {
        amp_store(at[m], y[m]);
        amp_store(at[m] + lam, z[m]);
      }
    }
  } else {
    block_rows<D, 0, B0, IM, false>(u0, x, y);
    if constexpr (B1 > 0) block_rows<D, B0, B1, IM, false>(u1, x, y);
    if (in) {
#pragma unroll
      for (int m = 0; m < D; ++m) amp_store(at[m], y[m]);
    }
  }
  return in ? s : 0.f;
}

// The same for CK = exp(i theta n_i n_j): one complex entry a member.
template <int D, bool REV>
__device__ __forceinline__ float fibre_diag(int lam, KFloat *u, int g, const ModeStep<D> &st, int base, bool in) {
  float s = 0.f;
#pragma unroll
  for (int m = 0; m < D; ++m) {
    const int at = run_at<D>(base, member_off<D>(st, g, m, true));
    const float2 w = make_float2(u[2 * m], u[2 * m + 1]), x = amp_load(at);
    float2 y = make_float2(0.f, 0.f);
    if constexpr (REV) {
      const float2 l = amp_load(at + lam);
      float2 z = y;
      s = fmaf(-(float)(m * ((g - m) + (m > g ? D : 0))), fmaf(l.x, x.y, -l.y * x.x), s);
      cmac_conj(y, w, x);
      cmac_conj(z, w, l);
      if (in) amp_store(at + lam, z);
    } else {
      cmac(y, w, x);
    }
    if (in) amp_store(at, y);
  }
  return in ? s : 0.f;
}

template <int D, bool SUM, bool IM, bool REV>
__device__ __forceinline__ float fibre_any(int g, int lam, KFloat *u, KFloat *A,
                                           const ModeStep<D> &st, int base, bool in) {
  switch (g) {
#define FOCK_GROUP(G) \
  case G:             \
    if constexpr (G < D) return fibre_group<D, (G < D ? G : 0), SUM, IM, REV>(lam, u, A, st, base, in); \
    break;
    FOCK_GROUP(0) FOCK_GROUP(1) FOCK_GROUP(2) FOCK_GROUP(3) FOCK_GROUP(4) FOCK_GROUP(5) FOCK_GROUP(6) FOCK_GROUP(7)
#undef FOCK_GROUP
  }
  return 0.f;
}

// A wavefront's units of a gate (group unit % D of fibres 64 (unit / D) ..) and
// its lanes' share of Re<lam|A phi>.  lam: its distance from phi in bytes; rt: the
// gate's fuse_table; fib: byte offset
// of every fibre.
template <int D, bool REV>
__device__ __forceinline__ float fibre_gate(const FuseGate &gt, float2 *phi, int lam, const float *rt,
                                            const float2 *A, const uint16_t *fib, int nfib) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6, lane = threadIdx.x & 63;
  const int type = gt.type;
  const int origin = (int)(uint32_t)(uintptr_t)(LdsAmp *)phi;
  ModeStep<D> st;
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    st.i[b] = gt.bi[b];
    st.j[b] = gt.bj[b];
  }
  KFloat *const u = scalar_ptr(rt), *const a = scalar_ptr(A);
  float s = 0.f;
  for (int c = wave; c < D * ((nfib + 63) >> 6); c += nw) {
    const int g = c % D, f = (c / D) * 64 + lane;
    const bool in = f < nfib;
    const int base = origin + fib[in ? f : 0];
    KFloat *const ug = u + g * (D * D);
    switch (type) {
      case FOCK_CK: s += fibre_diag<D, REV>(lam, ug, g, st, base, in); break;
      case FOCK_HR: s += fibre_any<D, true, false, REV>(g, lam, ug, a, st, base, in); break;
      case FOCK_PR: s += fibre_any<D, false, false, REV>(g, lam, ug, a, st, base, in); break;
      case FOCK_PI: s += fibre_any<D, false, true, REV>(g, lam, ug, a, st, base, in); break;
      default: s += fibre_any<D, true, true, REV>(g, lam, ug, a, st, base, in); break;  // HI, DH
    }
  }
  return s;
}

}  // namespace fock
