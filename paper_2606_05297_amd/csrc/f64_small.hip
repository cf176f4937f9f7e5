// Energy and all dE/dtheta of a circuit on a small complex128 state in one
// launch (adapt64_energy_grad and the FP64 ADAPT driver): one workgroup keeps
// phi and lam in LDS from psi0 to the last gradient.
//
// These states (both in one workgroup's LDS, d <= 8) take microseconds of
// arithmetic; gate by gate a circuit of n gates was 2n + 5 launches of
// 5.6-6.1 us each.  Here a gate is one pass over LDS.  Blocks s and s + D of a
// two-mode gate hold together one member for every n_i (tile_gate.h): a thread
// takes such a group of one fibre, D amplitudes in registers, and the D x D
// block-diagonal matrix of the group from LDS (a single-mode gate: the D levels
// of one fibre).  It stores over what it read, so a gate needs one barrier.
// States of one wave of groups are split by rows over P = 4 threads a group,
// which adds a barrier between reading and storing.
//
// A matrix entry is one double.  A generator links neighbouring levels only and
// is real antisymmetric (HR, PR, SR) or i times real symmetric with no diagonal
// (HI, DH, PI, SI), so with an even number of links between r and c the entry of
// exp(theta A) is real, with an odd number it is real or i times real; and the
// inverse is the same matrix with the entries of odd distance negated.  That
// halves the table reads (which set the time of a gate here) and the products.
// CK, KERR and ROT are diagonal: one complex number a member.
//
// The gate tables are built here as well, as many gates at a time as fit beside
// the states, from one sine-cosine per eigenvalue.  Re<lam|A phi> takes the
// diagonal of a generator and the links between neighbouring levels only.
// Angles and gates are read from, and the results written to, host memory.
//
// Bound by LDS reads and latency of the one CU (four waves at most have groups).
// Per gate, its table included, forward / reverse: 1.0 / 0.9 us at 256 amplitudes
// (d = 4), 2.5 / 2.7 at 512 (d = 8; 8 KB of states, but 4 KB of table a gate),
// 1.8 / 1.8 at 1,296 (d = 6), 2.7 / 3.4 at 2,401 (d = 7).  40 gates at 1,296:
// 122 us, 85 launches before of 500 us; with complex entries 194.  One thread an
// output, block sums from LDS: 208.
#include "f64_internal.h"

#include <algorithm>
#include <map>
#include <mutex>
#include <type_traits>
#include <vector>

#include "tile_gate.h"

namespace fock {

namespace {

constexpr int kThreads64 = 512;  // 2 waves a SIMD: 256 registers a thread
constexpr int kWaves64 = kThreads64 / 64;
constexpr int kBuild64 = 16;  // gates whose phases are in LDS at a time
constexpr int kLeast64 = 4;   // gates in LDS at a time: below, the builds would cost more than launches
constexpr size_t kLds64 = 163840 - 1024;

enum { KIND_ONE = 2 };  // Gate64::kind beside KIND_SUM and KIND_DIFF: single mode

struct Gate64 {
  int type, kind, row;  // row: of its generator's first group in the links
  int sj;               // stride of mode j, 0: single mode
  TilePair p;          // as tile_fibre takes it; single mode: p.sj = p.si, p.dm = 1
  double th;
};

// Doubles of a gate's table: d groups of d x d entries, or d^2 complex ones of a
// diagonal gate, read as double2: an even number, so that every table starts on 16
// bytes.
__host__ __device__ constexpr int table64(int d) { return (d * d * d + 1) & ~1; }

__host__ __device__ constexpr int links64(int d) { return kTwoModeTypes * d * d + 4 * d; }

__host__ __device__ inline int link_row(int type, int d) {
  const int two = kTwoModeTypes * d * d;
  return type == FOCK_SR ? two : type == FOCK_SI ? two + d : type == FOCK_KERR ? two + 2 * d
       : type == FOCK_ROT ? two + 3 * d : table_slot(type) * d * d;
}

// A = i c with c real and symmetric, or (HR, PR, SR) real and antisymmetric.
__host__ __device__ inline bool imaginary(int type) { return type != FOCK_HR && type != FOCK_PR && type != FOCK_SR; }

// Place of amplitude a.  d a power of two: the low three bits folded with the
// higher ones, or the fibres of a gate (strides 8, 64, ..) would share a bank.
template <int D>
__device__ __forceinline__ int at64(int a) {
  return (D & (D - 1)) == 0 ? a ^ (((a >> 3) ^ (a >> 6) ^ (a >> 9)) & 7) : a;
}

// y += u x with u real; y = u x, u^* x with u complex.
__device__ __forceinline__ void mac(double2 &y, double u, double2 x) {
  y.x = fma(u, x.x, y.x);
  y.y = fma(u, x.y, y.y);
}
__device__ __forceinline__ double2 mul(double2 u, double2 x) {
  return make_double2(fma(-u.y, x.y, u.x * x.x), fma(u.y, x.x, u.x * x.y));
}
__device__ __forceinline__ double2 mul_conj(double2 u, double2 x) {
  return make_double2(fma(u.y, x.y, u.x * x.x), fma(-u.y, x.x, u.x * x.y));
}

// Re(conj(l) x) and Re(conj(l) i x).
__device__ __forceinline__ double re_dot(double2 l, double2 x) { return l.x * x.x + l.y * x.y; }
__device__ __forceinline__ double im_dot(double2 l, double2 x) { return l.y * x.x - l.x * x.y; }

// A link's share of Re<l|A x>, c between members (l0, x0) and (l1, x1).
__device__ __forceinline__ double link(bool im, double c, double2 l0, double2 x0, double2 l1, double2 x1) {
  return im ? c * (im_dot(l0, x1) + im_dot(l1, x0)) : c * (re_dot(l0, x1) - re_dot(l1, x0));
}

__device__ __forceinline__ bool diagonal(int type) { return type == FOCK_CK || type == FOCK_KERR || type == FOCK_ROT; }
__device__ __forceinline__ bool squeezer(int type) { return type == FOCK_SR || type == FOCK_SI; }

// Phase of eigenvalue m (of D^2, or D) of a gate.
template <int D>
__device__ __forceinline__ double2 phase64(const Gate64 &q, int m, const EigTables &T) {
  double f = 0.0;
  if (q.type == FOCK_CK) f = (double)((m / D) * (m % D));  // member (n_i, n_j) = (m / D, m % D)
  else if (q.kind != KIND_ONE) f = T.lam[table_slot(q.type)][m];
  else if (m < D)
    f = squeezer(q.type) ? T.lam1[q.type == FOCK_SR ? 0 : 1][m] : q.type == FOCK_KERR ? (double)m * m : (double)m;
  double2 v;
  sincos(q.th * f, &v.y, &v.x);
  return v;
}

// Entry (group g, row r, column c) of a gate's table: Re U where r and c are an
// even number of links apart, else Re U or, A imaginary, Im U.  z: its phases.
template <int D>
__device__ __forceinline__ double entry64(const Gate64 &q, const double2 *z, int e, const EigTables &T) {
  const int g = e / (D * D), r = e / D % D, c = e % D;
  const double *V;
  int b = D, pr = r, pc = c, apart = r - c;
  if (q.kind == KIND_ONE) {
    if (g > 0 || (apart & 1)) return 0.0;
    apart >>= 1;
    V = T.V1[q.type == FOCK_SR ? 0 : 1];
  } else {
    if ((r <= g) != (c <= g)) return 0.0;
    const bool low = r <= g;  // block g, else g + D
    b = low ? g + 1 : D - 1 - g;
    const int k = low ? g : b, sq = k * (k + 1) * (2 * k + 1) / 6, ln = k * (k + 1) / 2;
    V = T.V[table_slot(q.type)] + 2 * (low ? sq : D * (2 * D * D + 1) / 3 - sq);
    z += low ? ln : D * D - ln;
    pr = low ? r : r - g - 1;
    pc = low ? c : c - g - 1;
  }
  const double2 *vr = (const double2 *)V + pr * b, *vc = (const double2 *)V + pc * b;
  const bool im = (apart & 1) && imaginary(q.type);
  double u = 0.0;
#pragma unroll
  for (int m = 0; m < D; ++m)
    if (m < b) {
      const double2 p = vr[m], s = vc[m], w = z[m];
      const double tx = fma(-p.y, w.y, p.x * w.x), ty = fma(p.y, w.x, p.x * w.y);
      u = im ? fma(-tx, s.y, fma(ty, s.x, u)) : fma(ty, s.y, fma(tx, s.x, u));
    }
  return u;
}

template <int D, int P>
__global__ __launch_bounds__(kThreads64) void k64_small(Small64 it, H64 h, EigTables T) {
  extern __shared__ double2 lds[];
  __shared__ double en[2][kWaves64], root[D + 1];
  constexpr int ne = D * D * D, us = table64(D), rows = (D + P - 1) / P;
  static_assert(us % 2 == 0 && us >= ne && us >= 2 * D * D, "tables are read as double2");
  const int N = (int)h.n_amp, n = it.n, cap = it.cap;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  double2 *const phi = lds, *const lam = phi + N, *const links = lam + N;
  double2 *const ph = links + links64(D);
  double *const tab = (double *)(ph + it.batch * D * D), *const part = tab + (size_t)cap * us;  // [cap][kWaves64]
  Gate64 *const gates = (Gate64 *)(part + cap * kWaves64);

  if (tid <= D) root[tid] = sqrt((double)tid);
  // The states carry a global phase.  E, gradients and scores do not depend on
  // it, but a real psi0 would stay real to the last bit under HR, PR and SR here,
  // and an optimisation that starts on a saddle of real states (the phases of
  // two-parameter gates at 0) would never leave it.  Rounding makes it do so, as
  // in the launches of larger states, whose complex tables round off the real axis.
  for (int a = tid; a < N; a += kThreads64) phi[at64<D>(a)] = mul(make_double2(0.8, 0.6), it.psi0[a]);
  for (int k = tid; k < n; k += kThreads64) {
    const int g = it.gates[k], type = g & 0xff, i = (g >> 8) & 0xff, j = (g >> 16) & 0xff;
    int si = 1, sj = 1;
    for (int r = 0; r < i; ++r) si *= D;
    Gate64 q;
    q.type = type;
    q.row = link_row(type, D);
    q.th = it.theta[k];
    if (j == 0xff) {
      q.kind = KIND_ONE;
      q.p = tile_pair(si, si * D, D);
      q.p.sj = si;
      q.sj = 0;
    } else {
      for (int r = 0; r < j; ++r) sj *= D;
      q.kind = type == FOCK_PR || type == FOCK_PI ? KIND_DIFF : KIND_SUM;
      q.p = tile_pair(si, sj, D);
      q.sj = sj;
    }
    gates[k] = q;
  }
  if (it.grad)
    for (int e = tid; e < links64(D); e += kThreads64) links[e] = it.links[e];

  // This thread's groups fg = g nfib + f (two-mode) or fibres fg (single mode):
  // one in kThreads64 (P = 1), or one, of which it has rows part, part + P, ..
  const int nfg = N / D, nfib = N / (D * D), per = (nfg + 63) / 64;
  const float rfib = 1.0f / (float)(nfib > 0 ? nfib : 1);
  const int part_of = P == 1 ? 0 : wave / per;
  const int first = P == 1 ? tid : part_of < P ? tid - part_of * per * 64 : nfg;
  __syncthreads();

  // Tables of gates [k0, k0 + cap).
  int k0 = 0;
  auto build = [&](int k) {
    k0 = k / cap * cap;
    const int end = min(k0 + cap, n);
    for (int g0 = k0; g0 < end; g0 += it.batch) {
      const int cnt = min(it.batch, end - g0);
      for (int x = tid; x < cnt * D * D; x += kThreads64) {
        const Gate64 &q = gates[g0 + x / (D * D)];
        const double2 v = phase64<D>(q, x % (D * D), T);
        ph[x] = v;
        if (diagonal(q.type)) {  // entry of its member, see diag below
          const int m = x % (D * D);
          double2 *u = (double2 *)(tab + (size_t)(g0 - k0 + x / (D * D)) * us);
          u[m] = v;
        }
      }
      __syncthreads();
      for (int x = tid; x < cnt * ne; x += kThreads64) {
        const int g = x / ne, e = x - g * ne;
        if (!diagonal(gates[g0 + g].type))
          tab[(size_t)(g0 - k0 + g) * us + e] = entry64<D>(gates[g0 + g], ph + g * D * D, e, T);
      }
      __syncthreads();
    }
  };

  // Member m of group fg of a gate is at base + m si + n_j sj, n_j = t mod D
  // with t in [-D, D) linear in m.
  struct Group {
    int base, t0, table, row;
  };
  auto group = [&](const Gate64 &q, int fg) {
    Group o;
    const bool two = q.sj > 0;
    const int g = two ? tile_div(fg, rfib) : 0;
    o.base = tile_fibre(two ? fg - g * nfib : fg, q.p, D);
    o.t0 = q.kind == KIND_SUM ? g : -g - 1;
    o.table = g * D * D;
    o.row = q.row + g * D;
    return o;
  };
  auto level_j = [&](const Gate64 &q, const Group &o, int m) {
    const unsigned t = (unsigned)(o.t0 + (q.kind == KIND_SUM ? -m : m));
    return (int)min(t, t + D);
  };
  auto place = [&](const Gate64 &q, const Group &o, int m) {
    return at64<D>(o.base + m * q.p.si + level_j(q, o, m) * q.sj);
  };
  auto gate = [&](int k) {
    Gate64 q = gates[k];
    q.type = __builtin_amdgcn_readfirstlane(q.type);
    q.kind = __builtin_amdgcn_readfirstlane(q.kind);
    q.row = __builtin_amdgcn_readfirstlane(q.row);
    q.sj = __builtin_amdgcn_readfirstlane(q.sj);
    q.p.si = __builtin_amdgcn_readfirstlane(q.p.si);
    return q;
  };
  auto load = [&](const double2 *s, const Gate64 &q, const Group &o, double2 (&x)[D]) {
#pragma unroll
    for (int m = 0; m < D; ++m) x[m] = s[place(q, o, m)];
  };
  // The level of this thread's row t (rows past the last repeat it).
  auto level = [&](int t) { return P == 1 ? t : min(part_of + t * P, D - 1); };
  // Entry of member m of a diagonal gate.
  auto diag = [&](const double *U, const Gate64 &q, const Group &o, int m) {
    return ((const double2 *)U)[q.sj > 0 ? m * D + level_j(q, o, m) : m];
  };
  // The rows of U (dag: of U^+) on W states: sums over the columns whose class
  // (even or odd distance from level 0, in links of `hop` levels) is the row's,
  // and over the others.  The next row's entries are read before a row's
  // products: one wave on a SIMD has nothing else to hide their latency.
  auto products = [&](auto hop, auto dag, const double *u0, int type, auto &y, const auto &x) {
    constexpr int W = sizeof(x) / sizeof(x[0]);
    double u[2][D];
    const bool im = imaginary(type);
#pragma unroll
    for (int c = 0; c < D; ++c) u[0][c] = u0[level(0) * D + c];
#pragma unroll
    for (int t = 0; t < rows; ++t) {
      if (t + 1 < rows) {
#pragma unroll
        for (int c = 0; c < D; ++c) u[(t + 1) & 1][c] = u0[level(t + 1) * D + c];
      }
      __builtin_amdgcn_sched_barrier(0);
      const bool odd = (level(t) / hop) & 1;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        double2 s[2] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
#pragma unroll
        for (int c = 0; c < D; ++c) mac(s[(c / hop) & 1], u[t & 1][c], x[w][c]);
        const double2 own = odd ? s[1] : s[0];
        double2 off = odd ? s[0] : s[1];
        if (im) off = make_double2(-off.y, off.x);
        y[w][t] = dag ? make_double2(own.x - off.x, own.y - off.y) : make_double2(own.x + off.x, own.y + off.y);
      }
    }
  };
  constexpr std::integral_constant<int, 1> hop1{};
  constexpr std::integral_constant<int, 2> hop2{};
  auto forward = [&](const double *U, const Gate64 &q, const Group &o, double2 (&y)[1][rows]) {
    if (diagonal(q.type)) {
#pragma unroll
      for (int t = 0; t < rows; ++t) y[0][t] = mul(diag(U, q, o, level(t)), phi[place(q, o, level(t))]);
      return;
    }
    double2 x[1][D];
    load(phi, q, o, x[0]);
    if (q.kind != KIND_ONE) products(hop1, std::false_type(), U + o.table, q.type, y, x);
    else products(hop2, std::false_type(), U, q.type, y, x);
  };
  // U^+ on both states, and this thread's share of Re<lam|A phi>.
  auto reverse = [&](const double *U, const Gate64 &q, const Group &o, double2 (&y)[2][rows]) {
    const bool im = imaginary(q.type);
    const double2 *c = links + o.row;
    double acc = 0.0;
    if (diagonal(q.type)) {
#pragma unroll
      for (int t = 0; t < rows; ++t) {
        const int r = level(t), at = place(q, o, r);
        const double2 w = diag(U, q, o, r), x = phi[at], l = lam[at];
        y[0][t] = mul_conj(w, x);
        y[1][t] = mul_conj(w, l);
        if (P == 1 || part_of + t * P < D) acc = fma(c[r].x, im_dot(l, x), acc);
      }
      return acc;
    }
    double2 x[2][D];
    load(phi, q, o, x[0]);
    load(lam, q, o, x[1]);
    auto links_of = [&](auto hop) {
      if constexpr (P == 1) {
        double2 v[D];
#pragma unroll
        for (int m = 0; m + hop < D; ++m) v[m] = c[m];
#pragma unroll
        for (int m = 0; m + hop < D; ++m) acc += link(im, v[m].y, x[1][m], x[0][m], x[1][m + hop], x[0][m + hop]);
      } else {
#pragma unroll
        for (int t = 0; t < rows; ++t) {
          const int m = level(t), a0 = place(q, o, m), a1 = place(q, o, min(m + hop, D - 1));
          if (part_of + t * P < D) acc += link(im, c[m].y, lam[a0], phi[a0], lam[a1], phi[a1]);
        }
      }
    };
    if (q.kind != KIND_ONE) {
      links_of(hop1);
      products(hop1, std::true_type(), U + o.table, q.type, y, x);
    } else {
      links_of(hop2);
      products(hop2, std::true_type(), U, q.type, y, x);
    }
    return acc;
  };
  auto store = [&](double2 *s, const Gate64 &q, const Group &o, const double2 (&y)[rows]) {
#pragma unroll
    for (int t = 0; t < rows; ++t)
      if (P == 1 || part_of + t * P < D) s[place(q, o, level(t))] = y[t];
  };
  const bool on = first < nfg;

  if (n > 0) build(0);
  for (int k = 0; k < n; ++k) {
    if (k >= k0 + cap) build(k);
    const Gate64 q = gate(k);
    const double *U = tab + (size_t)(k - k0) * us;
    double2 y[1][rows];
    if constexpr (P == 1) {
      for (int fg = first; fg < nfg; fg += kThreads64) {
        const Group o = group(q, fg);
        forward(U, q, o, y);
        store(phi, q, o, y[0]);
      }
    } else {
      const Group o = group(q, on ? first : 0);
      if (on) forward(U, q, o, y);
      __syncthreads();
      if (on) store(phi, q, o, y[0]);
    }
    __syncthreads();
  }

  // lam = H phi: the terms of a bond in the order of k64_apply_h
  double e = 0.0, nn = 0.0;
  constexpr float rd = 1.0f / (float)D;
  for (int idx = tid; idx < N; idx += kThreads64) {
    const double2 x = phi[at64<D>(idx)];
    double2 y;
    {
      double dg = 0.0;
      for (int r = 0, t = idx; r < h.L; ++r) {
        const int q = tile_div(t, rd), m = t - q * D;
        t = q;
        dg += h.c2 * m * (m - 1.0) - h.mu * m;
      }
      y = make_double2(dg * x.x, dg * x.y);
    }
    auto add = [&](double c, int at) {
      const double2 v = phi[at64<D>(at)];
      y.x += c * v.x;
      y.y += c * v.y;
    };
    auto bond = [&](int ni, int si, int nj, int sj) {
      if (h.J != 0.0) {
        if (ni >= 1 && nj <= D - 2) add(-h.J * root[ni] * root[nj + 1], idx - si + sj);
        if (ni <= D - 2 && nj >= 1) add(-h.J * root[ni + 1] * root[nj], idx + si - sj);
      }
      if (h.Delta != 0.0) {
        if (ni <= D - 2 && nj <= D - 2) add(h.Delta * root[ni + 1] * root[nj + 1], idx + si + sj);
        if (ni >= 1 && nj >= 1) add(h.Delta * root[ni] * root[nj], idx - si - sj);
      }
    };
    int t = tile_div(idx, rd), ni = idx - t * D, si = 1;
    const int n0 = ni;
    for (int r = 1; r < h.L; ++r) {
      const int q = tile_div(t, rd), nj = t - q * D;
      t = q;
      bond(ni, si, nj, si * D);
      if (h.wrap && r == h.L - 1) bond(n0, 1, nj, si * D);
      ni = nj;
      si *= D;
    }
    lam[at64<D>(idx)] = y;
    e += x.x * y.x + x.y * y.y;
    nn += x.x * x.x + x.y * x.y;
  }
  e = wave_total_d(e);
  nn = wave_total_d(nn);
  if (lane == 63) {
    en[0][wave] = e;
    en[1][wave] = nn;
  }
  __syncthreads();
  if (tid < 2) {
    double s = 0.0;
    for (int w = 0; w < kWaves64; ++w) s += en[tid][w];
    it.res[tid] = s;
  }
  if (!it.grad) {
    for (int a = tid; a < N; a += kThreads64) {
      it.phi[a] = phi[at64<D>(a)];
      it.lam[a] = lam[at64<D>(a)];
    }
    return;
  }

  for (int k = n - 1; k >= 0; --k) {
    if (k < k0) build(k);
    const Gate64 q = gate(k);
    const double *U = tab + (size_t)(k - k0) * us;
    double2 y[2][rows];
    double acc = 0.0;
    if constexpr (P == 1) {
      for (int fg = first; fg < nfg; fg += kThreads64) {
        const Group o = group(q, fg);
        acc += reverse(U, q, o, y);
        store(phi, q, o, y[0]);
        store(lam, q, o, y[1]);
      }
    } else {
      const Group o = group(q, on ? first : 0);
      if (on) acc = reverse(U, q, o, y);
      __syncthreads();
      if (on) {
        store(phi, q, o, y[0]);
        store(lam, q, o, y[1]);
      }
    }
    acc = wave_total_d(acc);
    if (lane == 63) part[(k - k0) * kWaves64 + wave] = acc;
    __syncthreads();
    if (k == k0) {  // the sums of this chunk's gates
      for (int x = tid; x < min(cap, n - k0); x += kThreads64) {
        double s = 0.0;
        for (int w = 0; w < kWaves64; ++w) s += part[x * kWaves64 + w];
        it.res[2 + k0 + x] = s;
      }
      __syncthreads();
    }
  }
}

// LDS beside the gate tables; of one gate's table and sums; of its phases.
size_t small64_fixed(int d, uint32_t namp, int n) {
  return sizeof(double2) * (2 * (size_t)namp + links64(d)) + sizeof(Gate64) * n;
}
size_t small64_gate(int d) { return sizeof(double) * (table64(d) + kWaves64); }
size_t small64_phase(int d) { return sizeof(double2) * d * d; }

// Gates in LDS at a time (0: none fit), of which `batch` are built at a time.
int small64_cap(int d, uint32_t namp, int n, int *batch) {
  const size_t fixed = small64_fixed(d, namp, n), gate = small64_gate(d), phase = small64_phase(d);
  *batch = std::min(n, kBuild64);
  if (fixed >= kLds64) return 0;
  const size_t left = kLds64 - fixed;
  while (*batch > 1 && *batch * (gate + phase) > left) *batch /= 2;
  return *batch * phase >= left ? 0 : (int)std::min<size_t>(n, (left - *batch * phase) / gate);
}

template <int D>
void launch_d(dim3 grid, size_t lds, const Small64 &it, const H64 &h, const EigTables &T, hipStream_t s) {
  // Four threads a group where its groups would be one wave on one SIMD: 40 gates
  // and their gradients at d = 4, 5, 7, 8 and 256, 125, 343, 512 amplitudes take
  // 101, 120, 150, 226 us, else 105, 128, 172, 255.  At two waves (625, d = 5)
  // 140 against 129; two threads a group lose everywhere.
  if ((int)h.n_amp / D <= 64 && D >= 4) hipLaunchKernelGGL((k64_small<D, 4>), grid, dim3(kThreads64), lds, s, it, h, T);
  else hipLaunchKernelGGL((k64_small<D, 1>), grid, dim3(kThreads64), lds, s, it, h, T);
}

}  // namespace

bool small64_ok(int d, uint32_t namp, int n) {
  if (d > 8 || namp > (1u << 14) || n > kGates64) return false;
  int batch = 0;
  return n == 0 ? small64_fixed(d, namp, 0) < kLds64 : small64_cap(d, namp, n, &batch) >= std::min(n, kLeast64);
}

// The energy of two gates or fewer on many bonds is all H psi, which the chip has
// sooner than one CU: 4,096 amplitudes of twelve modes, one gate, 47 us by launches,
// 60 in one (with the gradient 72 and 64); 2,048 of eleven 47 and 41.
bool small64_used(const H64 &h, int n, bool grad) {
  const bool all_h = n == 0 || (n <= 2 && !grad);
  return small64_ok(h.d, h.n_amp, n) && !(all_h && (long)h.n_amp * (h.L - 1) > 30000);
}

// (diagonal, link to the next level) of every generator's groups, in the order
// of link_row; zero where a link would leave its block.
static std::vector<double> build_links(int d) {
  std::vector<double> out((size_t)2 * links64(d), 0.0);
  std::vector<double> A;
  auto put = [&](int row, int type, int M, int p, int up) {
    const int im = imaginary(type) ? 1 : 0;
    out[(size_t)2 * row] = A[2 * ((size_t)p * M + p) + im];
    if (up >= 0) out[(size_t)2 * row + 1] = A[2 * ((size_t)p * M + up) + im];
  };
  for (int type : {FOCK_HR, FOCK_HI, FOCK_DH, FOCK_PR, FOCK_PI, FOCK_CK}) {
    generator_dense(type, d, A);
    const bool sum = gate_kind(type) == KIND_SUM;
    for (int g = 0; g < d; ++g)
      for (int m = 0; m < d; ++m) {
        auto index = [&](int a) { return a * d + ((sum ? g - a : a - g - 1) + d) % d; };
        put(link_row(type, d) + g * d + m, type, d * d, index(m), m != g && m + 1 < d ? index(m + 1) : -1);
      }
  }
  for (int type : {FOCK_SR, FOCK_SI, FOCK_KERR, FOCK_ROT}) {
    generator_dense(type, d, A);
    for (int p = 0; p < d; ++p)
      put(link_row(type, d) + p, type, d, p, (type == FOCK_SR || type == FOCK_SI) && p + 2 < d ? p + 2 : -1);
  }
  return out;
}

int small64_links(int d, const double2 **out) {
  static std::mutex mu;
  static std::map<std::pair<int, int>, const double2 *> made;
  int dev = 0;
  FOCK_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(mu);
  const double2 *&p = made[{dev, d}];
  if (!p) {
    const std::vector<double> h = build_links(d);
    void *b = nullptr;
    FOCK_HIP(hipMalloc(&b, sizeof(double) * h.size()));
    if (hipMemcpy(b, h.data(), sizeof(double) * h.size(), hipMemcpyHostToDevice) != hipSuccess) {
      (void)hipFree(b);
      return set_error(FOCK_ERR_HIP, "upload of the generator links failed");
    }
    p = (const double2 *)b;
  }
  *out = p;
  return FOCK_OK;
}

int launch64_small(const Small64 &item, const H64 &h, const EigTables &T, hipStream_t s) {
  Small64 it = item;
  if (!small64_ok(h.d, h.n_amp, it.n))
    return set_error(FOCK_ERR_SIZE, "small complex128 evaluation: L=%d d=%d n=%d", h.L, h.d, it.n);
  it.batch = it.cap = 0;
  if (it.n > 0) it.cap = small64_cap(h.d, h.n_amp, it.n, &it.batch);
  const size_t lds = small64_fixed(h.d, h.n_amp, it.n) + it.batch * small64_phase(h.d) + it.cap * small64_gate(h.d);
  const dim3 grid(1);
  switch (h.d) {
    case 2: launch_d<2>(grid, lds, it, h, T, s); break;
    case 3: launch_d<3>(grid, lds, it, h, T, s); break;
    case 4: launch_d<4>(grid, lds, it, h, T, s); break;
    case 5: launch_d<5>(grid, lds, it, h, T, s); break;
    case 6: launch_d<6>(grid, lds, it, h, T, s); break;
    case 7: launch_d<7>(grid, lds, it, h, T, s); break;
    default: launch_d<8>(grid, lds, it, h, T, s); break;
  }
  FOCK_HIP(hipGetLastError());
  return FOCK_OK;
}

}  // namespace fock
