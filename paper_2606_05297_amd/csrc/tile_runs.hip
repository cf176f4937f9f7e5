// Fused runs of gates on complex64 states: consecutive gates whose modes fit
// one tile of s modes (mode 0 always included, so that rows stay contiguous)
// run as one pass over the state.  Tile t holds the amplitudes whose digits of
// the tile modes take all values for fixed digits of the other modes; the run's
// gates are applied one after another in LDS by the matrix-core tile code
// (tile_gate.h), so the state is read and written once per run instead of once
// per gate.
//
// Forward: dst <- U_k1-1 ... U_k0 src.  Reverse (adjoint sweep, Sec. IV.B
// gradient identity): for k = k1-1 .. k0, this tile's share of Re<lam|A_k phi>
// goes to partial[k * rs + t], then phi <- U_k^+ phi and lam <- U_k^+ lam.
//
// Bound: the copies (5.7 TB/s) plus the gates' FP32 arithmetic, which on this
// chip includes the FP32 matrix instructions (their cycles and the vector ALUs'
// add up to the kernel's time; 47 % and 46 % of a 16-gate forward run at 8^8).
// Measured forward / reverse: 59 + 9 per gate / 92 + 24 us at 8^8 (134 MB),
// 11.3 + 2.4 / 13.6 + 4.7 us at 6^8, 7 + 1.4 / 8 + 2.3 us at 8^6, against 37 / 84,
// 8 / 11 and 5 / 6.4 us (11 / 18 on mode 0) for each gate on its own.  The tile's
// loads are all in flight together, and the tables a lane needs are made at
// compile time: with one load at a time and the divisions in the kernel the
// fixed parts were 10-20 us longer.
#include <algorithm>

#include "fuse_internal.h"
#include "sweep_internal.h"
#include "tile_gate.h"

namespace fock {

namespace {

static_assert(kMaxFuseGates <= kTileSums, "one accumulator row per gate of a run");

struct RunGate {
  int type, kj, u_off, k;
  const float2 *A;
  TilePair p;
};
struct RunShared {
  RunGate g[kMaxFuseGates];
  double red[kTileSums][kTileWaves];
};

// Global index, relative to the tile's base, of row r of the tile (its d
// amplitudes along mode 0 are contiguous).
__device__ __forceinline__ uint32_t run_row_offset(const FuseArgs &a, int r, float rd) {
  uint32_t g = 0;
  for (int k = 1; k < a.s; ++k) {
    const int q = tile_div(r, rd);
    g += (uint32_t)(r - __mul24(q, a.d)) * a.tstride[k];
    r = q;
  }
  return g;
}

// The digits of the tile index are those of the other modes; the highest one
// takes what is left (it has d / 2 levels in the parity-halved layout).
__device__ __forceinline__ uint32_t run_base(const FuseArgs &a, uint32_t t) {
  uint32_t base = 0;
  for (int k = 0; k < a.nc; ++k) {
    const uint32_t q = k + 1 < a.nc ? fdiv(t, a.dd) : 0u;
    base += (t - q * (uint32_t)a.d) * a.cstride[k];
    t = q;
  }
  return base;
}

// Phase gate on tile position ki.
template <bool P2, bool REV>
__device__ __forceinline__ float run_phase(float2 *tp, float2 *tl, const float2 *__restrict__ U, bool kerr, int si,
                                           int T, int d, float rd) {
  const float rs = 1.0f / (float)si;
  float acc = 0.f;
  for (int la = threadIdx.x; la < T; la += blockDim.x) {
    const int t = tile_div(la, rs), n = t - __mul24(tile_div(t, rd), d);
    const float2 p = U[n];
    const int x = tile_pos<P2>(la);
    float2 o = make_float2(0.f, 0.f);
    if (!REV) {
      cmac(o, p, tp[x]);
      tp[x] = o;
    } else {
      const float2 pv = tp[x], lv = tl[x];
      acc = fmaf(-(kerr ? (float)(n * n) : (float)n), lv.x * pv.y - lv.y * pv.x, acc);
      float2 ol = make_float2(0.f, 0.f);
      cmac_conj(o, p, pv);
      cmac_conj(ol, p, lv);
      tp[x] = o;
      tl[x] = ol;
    }
  }
  return acc;
}

// Tile <-> global; rows: the offsets of the tile's rows (LDS).  Even d: pairs
// (n_0 even, n_0 + 1) as one 16-byte access.  All of a thread's loads (up to
// kBatch at a time) are in flight together.
constexpr int kBatch = 4;
template <bool P2, bool TWO>
__device__ __forceinline__ void run_load(float2 *tp, float2 *tl, const float2 *__restrict__ p,
                                         const float2 *__restrict__ l, const FuseArgs &a, const uint32_t *rows) {
  const int nt = blockDim.x;
  if ((a.d & 1) == 0) {
    const int h = a.d / 2, n = a.T / 2;
    const float rh = 1.0f / (float)h;
    for (int w0 = threadIdx.x; w0 < n; w0 += kBatch * nt) {
      float4 v[kBatch], u[kBatch];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int w = min(w0 + k * nt, n - 1), r = tile_div(w, rh);
        const uint32_t o = rows[r] + 2 * (w - __mul24(r, h));
        v[k] = *reinterpret_cast<const float4 *>(p + o);
        if (TWO) u[k] = *reinterpret_cast<const float4 *>(l + o);
      }
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int w = w0 + k * nt;
        if (w >= n) break;
        const int x = tile_pos<P2>(2 * w), y = tile_pos<P2>(2 * w + 1);
        tp[x] = make_float2(v[k].x, v[k].y);
        tp[y] = make_float2(v[k].z, v[k].w);
        if (TWO) {
          tl[x] = make_float2(u[k].x, u[k].y);
          tl[y] = make_float2(u[k].z, u[k].w);
        }
      }
    }
  } else {
    const float rd = 1.0f / (float)a.d;
    for (int w0 = threadIdx.x; w0 < a.T; w0 += kBatch * nt) {
      float2 v[kBatch], u[kBatch];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int w = min(w0 + k * nt, a.T - 1), r = tile_div(w, rd);
        const uint32_t o = rows[r] + (w - __mul24(r, a.d));
        v[k] = p[o];
        if (TWO) u[k] = l[o];
      }
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int w = w0 + k * nt;
        if (w >= a.T) break;
        tp[tile_pos<P2>(w)] = v[k];
        if (TWO) tl[tile_pos<P2>(w)] = u[k];
      }
    }
  }
}

template <bool P2>
__device__ __forceinline__ void run_store(const float2 *tile, float2 *__restrict__ dst, const FuseArgs &a,
                                          const uint32_t *rows) {
  if ((a.d & 1) == 0) {
    const int h = a.d / 2;
    const float rh = 1.0f / (float)h;
    for (int w = threadIdx.x; w < a.T / 2; w += blockDim.x) {
      const int r = tile_div(w, rh), e = 2 * (w - __mul24(r, h));
      const float2 x = tile[tile_pos<P2>(2 * w)], y = tile[tile_pos<P2>(2 * w + 1)];
      *reinterpret_cast<float4 *>(dst + rows[r] + e) = make_float4(x.x, x.y, y.x, y.y);
    }
  } else {
    const float rd = 1.0f / (float)a.d;
    for (int w = threadIdx.x; w < a.T; w += blockDim.x) {
      const int r = tile_div(w, rd);
      dst[rows[r] + (w - __mul24(r, a.d))] = tile[tile_pos<P2>(w)];
    }
  }
}

// One tile.  src: the run's input (forward); phi, lam: updated in place
// (reverse; forward writes phi).
template <bool P2, bool REV>
__device__ __forceinline__ void run_tile(const FuseArgs &a, int t, const float2 *__restrict__ src,
                                         float2 *__restrict__ phi, float2 *__restrict__ lam,
                                         const float2 *__restrict__ utab, double *__restrict__ partial, int rs,
                                         float2 *lds, RunShared &sh) {
  const int d = a.d, T = a.T, nw = blockDim.x >> 6, nfib = T / (d * d);
  const float rd = 1.0f / (float)d;
  // LDS: the states, the rows' offsets and, per gate, the fibres' positions
  const int TP = (T + 31) & ~31;
  float2 *const tp = lds, *const tl = lds + TP;
  uint32_t *const rows = (uint32_t *)(lds + (REV ? 2 : 1) * TP);
  uint16_t *const fib = (uint16_t *)(rows + T / d);
  const TileLane lc = tile_lane(d, nw);
  const bool busy = lc.c0 * 16 < nfib;
  const uint32_t base = run_base(a, (uint32_t)t);
  for (int r = threadIdx.x; r < T / d; r += blockDim.x) rows[r] = run_row_offset(a, r, rd);
  if ((int)threadIdx.x < a.ng) {
    const FuseGate &g = a.g[threadIdx.x];
    RunGate o;
    o.type = g.type;
    o.kj = g.kj;
    o.u_off = g.u_off;
    o.k = g.k;
    o.A = a.A[table_slot(g.type == FOCK_KERR || g.type == FOCK_ROT ? 0 : g.type)];
    o.p = g.p;
    sh.g[threadIdx.x] = o;
  }
  __syncthreads();
  // The next gate's operands come from L2 while the current gate is applied.
  f64x4 sums = {0.0, 0.0, 0.0, 0.0};
  TileRaw u = {}, un = {};
  TileGenW w = {}, wn = {};
  auto operands = [&](int q) {
    const RunGate &g = sh.g[q];
    if (__builtin_amdgcn_readfirstlane(g.kj) < 0 || !busy) return;
    un = tile_raw<REV>(utab + __builtin_amdgcn_readfirstlane(g.u_off), lc);
    if constexpr (REV) {
      const int type = __builtin_amdgcn_readfirstlane(g.type);
      const uint64_t A = (uint64_t)g.A;
      const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)A), hi = __builtin_amdgcn_readfirstlane((uint32_t)(A >> 32));
      wn = tile_gen_raw((const float2 *)(((uint64_t)hi << 32) | lo), lc, tile_gen_kind(type));
    }
  };
  const int q0 = REV ? a.ng - 1 : 0, dq = REV ? -1 : 1;
  operands(q0);
  run_load<P2, REV>(tp, tl, (REV ? phi : src) + base, REV ? lam + base : nullptr, a, rows);
  for (int q = 0; q < a.ng; ++q) {
    const RunGate g = sh.g[q];
    if (g.kj >= 0)
      for (int f = threadIdx.x; f < nfib; f += blockDim.x)
        fib[q * nfib + f] = (uint16_t)(8 * tile_pos<P2>(tile_fibre(f, g.p, d)));
  }
  __syncthreads();
  for (int c = 0, q = q0; c < a.ng; ++c, q += dq) {
    const RunGate g = sh.g[q];
    const int kj = __builtin_amdgcn_readfirstlane(g.kj), type = __builtin_amdgcn_readfirstlane(g.type);
    u = un;
    w = wn;
    if (c + 1 < a.ng) operands(q + dq);
    float acc = 0.f;
    if (kj < 0) {
      acc = run_phase<P2, REV>(tp, tl, utab + g.u_off, type == FOCK_KERR, g.p.si, T, d, rd);
    } else if (busy) {
      const TileStep st = tile_step<P2>(g.p, lc, type == FOCK_PR || type == FOCK_PI ? KIND_DIFF : KIND_SUM);
      const uint16_t *fq = fib + q * nfib;
      auto at = [&](int f) { return (int)fq[f]; };
      const TileMat m = tile_mat<REV>(u, lc);
      if constexpr (REV) acc = tile_gate_adj<P2>(tp, tl, lc, st, m, w, tile_gen_kind(type), nfib, at);
      else tile_gate<P2>(tp, lc, st, m, nfib, at);
    }
    if constexpr (REV) {
      if (busy || kj < 0) tile_sums_add(sums, q, acc);
      if (c + 1 == a.ng) tile_sums_flush(sums, sh.red);
    }
    __syncthreads();
  }
  run_store<P2>(tp, phi + base, a, rows);
  if (REV) {
    run_store<P2>(tl, lam + base, a, rows);
    if ((int)threadIdx.x < a.ng) {
      double s = 0.0;
      for (int w = 0; w < nw; ++w) s += sh.red[threadIdx.x][w];
      partial[(size_t)a.g[threadIdx.x].k * rs + t] = s;
    }
  }
}

template <bool P2, bool REV>
__global__ __launch_bounds__(64 * kTileWaves) void k_tile_run(FuseArgs a, const float2 *__restrict__ src,
                                                              float2 *__restrict__ phi, float2 *__restrict__ lam,
                                                              const float2 *__restrict__ utab,
                                                              double *__restrict__ partial, int rs) {
  extern __shared__ float2 lds[];
  __shared__ RunShared sh;
  run_tile<P2, REV>(a, xcd_remap(blockIdx.x, gridDim.x), src, phi, lam, utab, partial, rs, lds, sh);
}

// The same for the runs of many sweep points; tiles of points whose BFGS is idle
// this round are skipped.
template <bool P2, bool REV>
__global__ __launch_bounds__(64 * kTileWaves) void k_sweep_runs(const SweepRun *__restrict__ runs,
                                                                const int2 *__restrict__ tiles,
                                                                const int *__restrict__ active) {
  extern __shared__ float2 lds[];
  __shared__ RunShared sh;
  const int2 t = tiles[blockIdx.x];
  const SweepRun &r = runs[t.x];
  if (!active[r.p]) return;
  run_tile<P2, REV>(r.a, t.y, r.src, r.phi, r.lam, r.utab, r.partial, r.rs, lds, sh);
}

}  // namespace

bool fuse_supported(int d) { return d >= kTileMinD && d <= kTileMaxD; }

// Wavefronts of a run's workgroups: as many whole rounds of units as fit 8
// waves, or 16 when the tiles are so large that a CU holds one workgroup, and no
// more than the fibre chunks keep busy.  Measured forward / reverse, four gates:
// d = 8 (4,096 amplitudes a tile, 8^8) 95 / 188 us with 8 waves, 133 / 191 with
// 16; d = 6 (7,776 a tile, 6^8) 28 / 41 with 6 waves, 21 / 33 with 12.
int fuse_waves(int D, int T) {
  const int u = tile_units(D), chunks = (T / (D * D) + 15) / 16, want = T > 4096 ? 16 : 8;
  return u * std::max(1, std::min(want / u, chunks));
}

size_t fuse_lds(const FuseArgs &a, bool rev) {
  return sizeof(float2) * (size_t)((a.T + 31) & ~31) * (rev ? 2 : 1) + sizeof(uint32_t) * (a.T / a.d) +
         sizeof(uint16_t) * (size_t)(a.ng * (a.T / (a.d * a.d)));
}

template <bool REV>
static int launch_run(const FuseArgs &a, const float2 *src, float2 *phi, float2 *lam, const float2 *utab,
                      double *partial, int rs, hipStream_t s) {
  const size_t lds = fuse_lds(a, REV);
  const dim3 grid(a.ntile), block(64 * fuse_waves(a.d, a.T));
  if ((a.d & (a.d - 1)) == 0)
    hipLaunchKernelGGL((k_tile_run<true, REV>), grid, block, lds, s, a, src, phi, lam, utab, partial, rs);
  else
    hipLaunchKernelGGL((k_tile_run<false, REV>), grid, block, lds, s, a, src, phi, lam, utab, partial, rs);
  FOCK_HIP(hipGetLastError());
  return FOCK_OK;
}

int launch_fuse_fwd(const FuseArgs &a, const float2 *src, float2 *dst, const float2 *utab, hipStream_t s) {
  return launch_run<false>(a, src, dst, nullptr, utab, nullptr, 0, s);
}

int launch_fuse_adj(const FuseArgs &a, float2 *phi, float2 *lam, const float2 *utab, double *partial, int rs,
                    hipStream_t s) {
  if (a.ntile > rs) return set_error(FOCK_ERR_SIZE, "fused run: %d partials per gate exceed the row stride %d", a.ntile, rs);
  return launch_run<true>(a, nullptr, phi, lam, utab, partial, rs, s);
}

int sweep_launch_runs(int d, bool rev, const SweepRun *runs, const int2 *tiles, int n, int waves, size_t lds,
                      const int *active, hipStream_t s) {
  if (n <= 0) return FOCK_OK;
  const dim3 grid(n), block(64 * waves);
  const bool p2 = (d & (d - 1)) == 0;
  if (rev) {
    if (p2) hipLaunchKernelGGL((k_sweep_runs<true, true>), grid, block, lds, s, runs, tiles, active);
    else hipLaunchKernelGGL((k_sweep_runs<false, true>), grid, block, lds, s, runs, tiles, active);
  } else {
    if (p2) hipLaunchKernelGGL((k_sweep_runs<true, false>), grid, block, lds, s, runs, tiles, active);
    else hipLaunchKernelGGL((k_sweep_runs<false, false>), grid, block, lds, s, runs, tiles, active);
  }
  FOCK_HIP(hipGetLastError());
  return FOCK_OK;
}

}  // namespace fock
