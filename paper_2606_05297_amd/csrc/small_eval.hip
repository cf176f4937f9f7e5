// Energy and all dE/dtheta of a circuit on a small state in one launch
// (fock_energy_grad_adjoint, the ADAPT, HVA and sweep drivers): one workgroup
// keeps phi and lam in LDS from psi0 to the last gradient.
//
// These states (LDS takes both of up to about 9,500 amplitudes; the plan gives it
// those of up to 4,096, small_planned) are far too small to fill the chip, and gate
// by gate a circuit of n gates is 2n + 5 launches of 2-6 us each, most of it launch
// gap and memory latency.  Here a
// gate is one pass over LDS (the matrix-core tile code of tile_gate.h) and one
// barrier; a reverse step is the same on two states plus one wave reduction.
// The gate tables come into LDS in bulk, as many gates at a time as fit beside
// the states (all of them in most circuits): loaded one gate ahead from global
// memory they cost 1-2 us each, several times the gate itself.  The results go
// straight into host-visible memory.
//
// Bound by instruction issue and LDS latency of the one CU.  Per gate forward /
// reverse: 0.48 / 0.78 us at 64-256 amplitudes (d = 4), 1.1 / 2.1 at 1,296
// (d = 6), 1.5 / 2.6 at 4,096 (d = 8), 2.6 / 5.5 at 7,776 (d = 6), against
// 1.8-6 / 2.6-8 us and a launch gap each for the per-gate kernels.  A squeezer is
// dense work of one thread a fibre: 3 us forward and 8 in reverse at d = 8.  With 8
// instead of 16 waves from 1,296 amplitudes on it ran 10-35 % slower; with the
// next gate's operands held in registers, 20-60 % slower (spills).
#include "small_eval.h"

#include <algorithm>

#include "tile_gate.h"

namespace fock {

namespace {

// A gate's description, decoded once per launch (p.sj = 0: single mode).
struct SGate {
  int type;
  TilePair p;
};

struct SmallShared {
  double part[kTileSums][kTileWaves];
  double en[2][kTileWaves];
  float4 w[64];
  SGate gate[kSmallGates];
};

__device__ __forceinline__ bool gate_is_phase(int t) { return t == FOCK_KERR || t == FOCK_ROT; }
__device__ __forceinline__ bool gate_is_squeeze(int t) { return t == FOCK_SR || t == FOCK_SI; }
__device__ __forceinline__ int gate_kind_dev(int t) { return t == FOCK_PR || t == FOCK_PI ? KIND_DIFF : KIND_SUM; }

__device__ __forceinline__ int mode_stride(int r, int d) {
  int s = 1;
  for (int k = 0; k < r; ++k) s *= d;
  return s;
}

// Phase gate: forward, or the reverse step's share of Re<lam|A phi>.
template <bool REV, bool P2>
__device__ __forceinline__ float small_phase(float2 *phi, float2 *lam, const float2 *U, const SGate &g, int N, int d) {
  const int nt = blockDim.x;
  const float rd = 1.0f / (float)d;
  float acc = 0.f;
  for (int a = threadIdx.x; a < N; a += nt) {
    const int t = tile_div(a, g.p.rsi), n = t - tile_div(t, rd) * d;
    const float2 p = U[n];
    const int x = tile_pos<P2>(a);
    if (!REV) {
      float2 o = make_float2(0.f, 0.f);
      cmac(o, p, phi[x]);
      phi[x] = o;
    } else {
      const float2 pv = phi[x], lv = lam[x];
      const float f = g.type == FOCK_KERR ? (float)(n * n) : (float)n;
      acc = fmaf(-f, lv.x * pv.y - lv.y * pv.x, acc);
      float2 np = make_float2(0.f, 0.f), nl = make_float2(0.f, 0.f);
      cmac_conj(np, p, pv);
      cmac_conj(nl, p, lv);
      phi[x] = np;
      lam[x] = nl;
    }
  }
  return acc;
}

// Squeezer gate (dense d x d on mode i, nonzero between levels of equal parity).
template <bool REV, bool P2>
__device__ __forceinline__ float small_squeeze(float2 *phi, float2 *lam, const float2 *U, const float2 *__restrict__ A,
                                               const SGate &g, int N, int d) {
  const int nt = blockDim.x;
  const int s = g.p.si;
  float acc = 0.f;
  for (int f = threadIdx.x; f < N / d; f += nt) {
    const int t = tile_div(f, g.p.rsi), base = t * s * d + (f - t * s);
    // phi first, then lam: one state's members in registers at a time
#pragma unroll
    for (int w = 0; w < (REV ? 2 : 1); ++w) {
      float2 *x = w == 0 ? phi : lam;
      float2 v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = q < d ? x[tile_pos<P2>(base + q * s)] : make_float2(0.f, 0.f);
#pragma unroll 1
      for (int p = 0; p < d; ++p) {
        float2 o = make_float2(0.f, 0.f), ap = o;
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (q < d && ((p + q) & 1) == 0) {
            if (!REV) cmac(o, U[p * d + q], v[q]);
            else cmac_conj(o, U[q * d + p], v[q]);
            if (REV && w == 0) cmac(ap, A[p * d + q], v[q]);
          }
        const int xp = tile_pos<P2>(base + p * s);
        x[xp] = o;
        if (REV && w == 0) {
          const float2 l = lam[xp];
          acc = fmaf(l.x, ap.x, fmaf(l.y, ap.y, acc));
        }
      }
    }
  }
  return acc;
}

// lam = H phi (Sec. III; every neighbour from LDS), this thread's shares of
// <phi|H phi> and <phi|phi>.  w[m d + n]: the weights of the four neighbours of
// a bond at levels (m, n), zero where the neighbour does not exist (its index
// is clamped then).
template <bool P2>
__device__ __forceinline__ void small_h(const SmallItem &it, const float2 *phi, float2 *lam, const float4 *w, double &e,
                                        double &nn) {
  const int d = it.d, L = it.L, top = it.N - 1, nt = blockDim.x;
  const float rd = 1.0f / (float)d;
  const bool hop = it.J != 0.f, pair = it.Delta != 0.f;
  e = nn = 0.0;
  for (int a = threadIdx.x; a < it.N; a += nt) {
    const float2 own = phi[tile_pos<P2>(a)];
    float2 acc = make_float2(0.f, 0.f);
    auto add = [&](int at, float c) {
      const float2 v = phi[tile_pos<P2>(min(max(at, 0), top))];
      acc.x = fmaf(c, v.x, acc.x);
      acc.y = fmaf(c, v.y, acc.y);
    };
    auto bond = [&](int m, int sm, int n, int sn) {
      const float4 c = w[m * d + n];
      if (hop) {
        add(a - sm + sn, c.x);
        add(a + sm - sn, c.y);
      }
      if (pair) {
        add(a + sm + sn, c.z);
        add(a - sm - sn, c.w);
      }
    };
    int q = tile_div(a, rd), t = q, ni = a - q * d, si = 1, sj = d;
    const int n0 = ni;
    float dg = it.c2 * (float)ni * ((float)ni - 1.f) - it.mu * (float)ni;
    for (int r = 1; r < L; ++r) {
      q = tile_div(t, rd);
      const int n = t - q * d;
      t = q;
      dg += it.c2 * (float)n * ((float)n - 1.f) - it.mu * (float)n;
      bond(ni, si, n, sj);
      if (it.wrap && r == L - 1) bond(n0, 1, n, sj);
      ni = n;
      si = sj;
      sj *= d;
    }
    acc.x = fmaf(dg, own.x, acc.x);
    acc.y = fmaf(dg, own.y, acc.y);
    lam[tile_pos<P2>(a)] = acc;
    e += (double)fmaf(own.x, acc.x, own.y * acc.y);
    nn += (double)fmaf(own.x, own.x, own.y * own.y);
  }
}

template <bool P2>
__global__ __launch_bounds__(64 * kTileWaves) void k_small_eval(SmallItem one, const SmallItem *__restrict__ items,
                                                             EigTables T, const int *__restrict__ active) {
  extern __shared__ float2 lds[];
  __shared__ SmallShared sh;
  SmallItem it = items ? items[blockIdx.x] : one;
  if (it.point >= 0 && active && active[it.point] == 0) return;
  // one item per workgroup: its numbers are uniform
  const int d = __builtin_amdgcn_readfirstlane(it.d), N = __builtin_amdgcn_readfirstlane(it.N);
  const int n = __builtin_amdgcn_readfirstlane(it.n), us = __builtin_amdgcn_readfirstlane(it.ustride);
  const int cap = __builtin_amdgcn_readfirstlane(it.chunk);
  it.d = d;
  it.N = N;
  it.L = __builtin_amdgcn_readfirstlane(it.L);
  const int nt = blockDim.x, nw = nt >> 6;
  const int NP = (N + 31) & ~31;
  float2 *const phi = lds, *const lam = lds + NP, *const gen = lam + NP, *const tab = gen + kTwoModeTypes * us;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const TileLane tl = tile_lane(d, nw);
  const int nfib = N / (d * d);
  const bool busy = tl.c0 * 16 < nfib;  // this wave has fibres
  if ((int)threadIdx.x < d * d) {
    const int m = threadIdx.x / d, q = threadIdx.x % d;
    const float sm = sqrtf((float)m), sm1 = m < d - 1 ? sqrtf((float)(m + 1)) : 0.f;
    const float sn = sqrtf((float)q), sn1 = q < d - 1 ? sqrtf((float)(q + 1)) : 0.f;
    sh.w[threadIdx.x] = make_float4(-it.J * sm * sn1, -it.J * sm1 * sn, it.Delta * sm1 * sn1, it.Delta * sm * sn);
  }
  for (int a = threadIdx.x; a < N; a += nt) phi[tile_pos<P2>(a)] = it.psi0[a];
  for (int k = threadIdx.x; k < n; k += nt) {
    const GateRec r = it.recs[k];
    const int j = (r.modes >> 8) & 0xff;
    const int si = mode_stride(r.modes & 0xff, d);
    SGate g;
    g.type = r.type;
    if (j == 0xff) {
      g.p = tile_pair(si, si * d, d);
      g.p.sj = 0;
    } else {
      g.p = tile_pair(si, mode_stride(j, d), d);
    }
    sh.gate[k] = g;
  }
  if (it.grad && n > 0)
    for (int t = 0; t < kTwoModeTypes; ++t)
      for (int e = threadIdx.x; e < us; e += nt) gen[t * us + e] = T.A[t][e];
  // Gate tables [k0, k0 + cap) in LDS.
  int k0 = 0;
  auto load_tables = [&](int k) {
    k0 = k / cap * cap;
    const int cnt = (k0 + cap < n ? cap : n - k0) * us;
    const float2 *src = it.U + (size_t)k0 * us;
    for (int e = threadIdx.x; e < cnt; e += nt) tab[e] = src[e];
    __syncthreads();
  };
  auto held = [&](int k) { return k >= k0 && k < k0 + cap; };
  if (n > 0) load_tables(0);
  else __syncthreads();
  for (int k = 0; k < n; ++k) {
    const SGate g = sh.gate[k];
    const int type = __builtin_amdgcn_readfirstlane(g.type), pair = __builtin_amdgcn_readfirstlane(g.p.sj);
    if (!held(k)) load_tables(k);
    const float2 *U = tab + (k - k0) * us;
    if (pair > 0) {
      if (busy)
        tile_gate<P2>(phi, tl, tile_step<P2>(g.p, tl, gate_kind_dev(type)), tile_mat<false>(tile_raw<false>(U, tl), tl), nfib,
                      [&](int f) { return 8 * tile_pos<P2>(tile_fibre(f, g.p, d)); });
    } else if (gate_is_phase(type)) {
      small_phase<false, P2>(phi, lam, U, g, N, d);
    } else {
      small_squeeze<false, P2>(phi, lam, U, nullptr, g, N, d);
    }
    __syncthreads();
  }
  double e, nn;
  small_h<P2>(it, phi, lam, sh.w, e, nn);
  e = wave_total_d(e);
  nn = wave_total_d(nn);
  if (lane == 63) {
    sh.en[0][wave] = e;
    sh.en[1][wave] = nn;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += sh.en[threadIdx.x][w];
    it.res[threadIdx.x] = s;
  }
  if (!it.grad) {
    for (int a = threadIdx.x; a < N; a += nt) {
      it.phi[a] = phi[tile_pos<P2>(a)];
      it.lam[a] = lam[tile_pos<P2>(a)];
    }
    return;
  }
  // reverse; the sums of up to kTileSums gates are added up together
  f64x4 sums = {0.0, 0.0, 0.0, 0.0};
  int done = 0;
  for (int k = n - 1; k >= 0; --k) {
    const SGate g = sh.gate[k];
    const int type = __builtin_amdgcn_readfirstlane(g.type), pair = __builtin_amdgcn_readfirstlane(g.p.sj);
    if (!held(k)) load_tables(k);
    const float2 *U = tab + (k - k0) * us;
    float acc = 0.f;
    if (pair > 0) {
      if (busy)
        acc = tile_gate_adj<P2>(phi, lam, tl, tile_step<P2>(g.p, tl, gate_kind_dev(type)), tile_mat<true>(tile_raw<true>(U, tl), tl),
                                tile_gen_raw(gen + table_slot(type) * us, tl, tile_gen_kind(type)), tile_gen_kind(type), nfib,
                                [&](int f) { return 8 * tile_pos<P2>(tile_fibre(f, g.p, d)); });
    } else if (gate_is_phase(type)) {
      acc = small_phase<true, P2>(phi, lam, U, g, N, d);
    } else {
      acc = small_squeeze<true, P2>(phi, lam, U, T.A1[type == FOCK_SR ? 0 : 1], g, N, d);
    }
    if (busy || pair == 0) tile_sums_add(sums, done, acc);
    ++done;
    if (done == kTileSums || k == 0) {  // a full accumulator
      tile_sums_flush(sums, sh.part);
      sums = f64x4{0.0, 0.0, 0.0, 0.0};
      __syncthreads();
      if ((int)threadIdx.x < done) {
        double s = 0.0;
        for (int w = 0; w < nw; ++w) s += sh.part[threadIdx.x][w];
        it.res[2 + k + done - 1 - threadIdx.x] = s;
      }
      done = 0;
    }
    __syncthreads();
  }
}

// Dynamic LDS a workgroup may take beside the static part, of the 160 KB per CU.
constexpr size_t kSmallLds = 163840 - sizeof(SmallShared) - 256;

// LDS of the states and generators; the gate tables take the rest.
size_t small_lds(int d, uint32_t namp) {
  return sizeof(float2) * (2 * (size_t)((namp + 31) & ~31u) + (size_t)kTwoModeTypes * gate_stride(d));
}

}  // namespace

bool small_eval_ok(int L, int d, uint32_t namp, int n) {
  return d <= 8 && n <= kSmallGates && L >= 1 && L <= kSmallModes && namp <= (1u << 14) &&
         small_lds(d, namp) + sizeof(float2) * 8 * gate_stride(d) <= kSmallLds;
}

int small_chunk(int d, uint32_t namp, int n) {
  const size_t left = kSmallLds - small_lds(d, namp), one = sizeof(float2) * (size_t)gate_stride(d);
  return std::max(1, (int)std::min<size_t>((size_t)n, left / one));
}

size_t small_lds_bytes(const SmallItem &it) {
  return small_lds(it.d, (uint32_t)it.N) + sizeof(float2) * (size_t)it.chunk * gate_stride(it.d);
}

int small_waves(const SmallItem &it) {
  return tile_waves(it.d, it.N);
}

int launch_small_eval(const SmallItem &one, const SmallItem *items, int count, size_t lds, int waves, const EigTables &T,
                      const int *active, hipStream_t s) {
  if (lds > kSmallLds) return set_error(FOCK_ERR_SIZE, "small-state evaluation: %zu bytes of LDS", lds);
  const dim3 grid(count > 0 ? count : 1), block(64 * waves);
  if (count == 0) items = nullptr;
  if ((one.d & (one.d - 1)) == 0)
    hipLaunchKernelGGL((k_small_eval<true>), grid, block, lds, s, one, items, T, active);
  else
    hipLaunchKernelGGL((k_small_eval<false>), grid, block, lds, s, one, items, T, active);
  FOCK_HIP(hipGetLastError());
  return FOCK_OK;
}

}  // namespace fock
