// Fused runs of gates on complex64 states: consecutive gates whose modes fit
// one tile of s modes (mode 0 always included, so that rows stay contiguous)
// run as one pass over the state.  Tile t holds the amplitudes whose digits of
// the tile modes take all values for fixed digits of the other modes; the run's
// gates are applied one after another in LDS (fibre_gate.h), so the state is read and written once per run instead of once
// per gate.
//
// Forward: dst <- U_k1-1 ... U_k0 src.  Reverse (adjoint sweep, Sec. IV.B
// gradient identity): for k = k1-1 .. k0, this tile's share of Re<lam|A_k phi>
// goes to partial[k * rs + t], then phi <- U_k^+ phi and lam <- U_k^+ lam.
//
// Bound: the copies (5.7 TB/s) plus the vector ALUs, which overlap in part only (a
// CU's workgroups, four forward and two in reverse at 8^8, run in step).  Measured
// forward / reverse: 58 + 8 per gate / 75 + 19 us at 8^8 (134 MB; a gate's fused
// multiply-adds alone take 4.6 / 11), 10 + 1.8 / 11 + 3.0 us at 6^8, against 37 /
// 84 and 8 / 11 us for each gate on its own, and 59 + 9 / 92 + 24, 11 + 2.4 / 14 +
// 4.7 on the FP32 matrix cores.  The next tile read ahead into registers made the
// forward run 10 us shorter alone, but not in a circuit, and the reverse one
// longer (spills); workgroups started a quarter of a tile apart changed nothing.
#include <algorithm>

#include "fibre_gate.h"
#include "sweep_internal.h"

namespace fock {

namespace {

static_assert(kMaxFuseGates <= kTileSums, "one accumulator row per gate of a run");

// The gates' sums of a reverse run, per wavefront.
typedef double RunSums[kTileSums][kTileWaves];
static_assert(sizeof(RunSums) == sizeof(double) * 16 * 16, "fuse_lds");

// Global index, relative to the tile's base, of row r of the tile (its d
// amplitudes along mode 0 are contiguous).
template <int D>
__device__ __forceinline__ uint32_t run_row_offset(const FuseArgs &a, int r) {
  constexpr float rd = 1.0f / (float)D;
  uint32_t g = 0;
  for (int k = 1; k < a.s; ++k) {
    const int q = tile_div(r, rd);
    g += (uint32_t)(r - q * D) * a.tstride[k];
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
template <int D, bool REV>
__device__ __forceinline__ float run_phase(float2 *tp, float2 *tl, const float2 *__restrict__ U, bool kerr, int si,
                                           int T) {
  constexpr float rd = 1.0f / (float)D;
  const float rs = 1.0f / (float)si;
  float acc = 0.f;
  for (int la = threadIdx.x; la < T; la += blockDim.x) {
    const int t = tile_div(la, rs), n = t - tile_div(t, rd) * D;
    const float2 p = U[n];
    const int x = run_pos<D>(la);
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
template <int D, bool TWO>
__device__ __forceinline__ void run_load(float2 *tp, float2 *tl, const float2 *__restrict__ p,
                                         const float2 *__restrict__ l, const FuseArgs &a, const uint32_t *rows) {
  const int nt = blockDim.x;
  if constexpr ((D & 1) == 0) {
    constexpr int h = D / 2;
    constexpr float rh = 1.0f / (float)h;
    const int n = a.T / 2;
    for (int w0 = threadIdx.x; w0 < n; w0 += kBatch * nt) {
      float4 v[kBatch], u[kBatch];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int w = min(w0 + k * nt, n - 1), r = tile_div(w, rh);
        const uint32_t o = rows[r] + 2 * (w - r * h);
        v[k] = *reinterpret_cast<const float4 *>(p + o);
        if (TWO) u[k] = *reinterpret_cast<const float4 *>(l + o);
      }
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int w = w0 + k * nt;
        if (w >= n) break;
        const int x = run_pos<D>(2 * w), y = run_pos<D>(2 * w + 1);
        tp[x] = make_float2(v[k].x, v[k].y);
        tp[y] = make_float2(v[k].z, v[k].w);
        if (TWO) {
          tl[x] = make_float2(u[k].x, u[k].y);
          tl[y] = make_float2(u[k].z, u[k].w);
        }
      }
    }
  } else {
    constexpr float rd = 1.0f / (float)D;
    for (int w0 = threadIdx.x; w0 < a.T; w0 += kBatch * nt) {
      float2 v[kBatch], u[kBatch];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int w = min(w0 + k * nt, a.T - 1), r = tile_div(w, rd);
        const uint32_t o = rows[r] + (w - r * D);
        v[k] = p[o];
        if (TWO) u[k] = l[o];
      }
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int w = w0 + k * nt;
        if (w >= a.T) break;
        tp[run_pos<D>(w)] = v[k];
        if (TWO) tl[run_pos<D>(w)] = u[k];
      }
    }
  }
}

template <int D>
__device__ __forceinline__ void run_store(const float2 *tile, float2 *__restrict__ dst, const FuseArgs &a,
                                          const uint32_t *rows) {
  if constexpr ((D & 1) == 0) {
    constexpr int h = D / 2;
    constexpr float rh = 1.0f / (float)h;
    for (int w = threadIdx.x; w < a.T / 2; w += blockDim.x) {
      const int r = tile_div(w, rh), e = 2 * (w - r * h);
      const float2 x = tile[run_pos<D>(2 * w)], y = tile[run_pos<D>(2 * w + 1)];
      *reinterpret_cast<float4 *>(dst + rows[r] + e) = make_float4(x.x, x.y, y.x, y.y);
    }
  } else {
    constexpr float rd = 1.0f / (float)D;
    for (int w = threadIdx.x; w < a.T; w += blockDim.x) {
      const int r = tile_div(w, rd);
      dst[rows[r] + (w - r * D)] = tile[run_pos<D>(w)];
    }
  }
}

// One tile.  src: the run's input (forward); phi, lam: updated in place
// (reverse; forward writes phi).
template <int D, bool REV>
__device__ __forceinline__ void run_tile(const FuseArgs &a, int t, const float2 *__restrict__ src,
                                         float2 *__restrict__ phi, float2 *__restrict__ lam, const FuseTables &tab,
                                         double *__restrict__ partial, int rs, float2 *lds) {
  const int T = a.T, nw = blockDim.x >> 6, nfib = T / (D * D);
  // LDS: the states (from address 0: a member's address is then one instruction),
  // the sums, the rows' offsets and, per gate, the fibres' positions
  const int TP = (T + 31) & ~31;
  float2 *const tp = lds, *const tl = lds + TP;
  RunSums *const sums_of = (RunSums *)(lds + (REV ? 2 : 1) * TP);
  uint32_t *const rows = (uint32_t *)(sums_of + (REV ? 1 : 0));
  uint16_t *const fib = (uint16_t *)(rows + T / D);
  const uint32_t base = run_base(a, (uint32_t)t);
  for (int r = threadIdx.x; r < T / D; r += blockDim.x) rows[r] = run_row_offset<D>(a, r);
  __syncthreads();
  run_load<D, REV>(tp, tl, (REV ? phi : src) + base, REV ? lam + base : nullptr, a, rows);
  for (int q = 0; q < a.ng; ++q)
    if (a.g[q].kj >= 0) {
      const TilePair p = a.g[q].p;
      for (int f = threadIdx.x; f < nfib; f += blockDim.x)
        fib[q * nfib + f] = (uint16_t)(8 * run_pos<D>(tile_fibre(f, p, D)));
    }
  __syncthreads();
  f64x4 sums = {0.0, 0.0, 0.0, 0.0};
  for (int c = 0; c < a.ng; ++c) {
    const int q = REV ? a.ng - 1 - c : c;
    const FuseGate &g = a.g[q];
    float acc;
    if (g.kj < 0)
      acc = run_phase<D, REV>(tp, tl, tab.u + g.u_off, g.type == FOCK_KERR, g.p.si, T);
    else
      acc = fibre_gate<D, REV>(g, tp, 8 * TP, tab.r + (size_t)g.k * fuse_table(D), a.A[table_slot(g.type)], fib + q * nfib,
                               nfib);
    if constexpr (REV) {
      tile_sums_add(sums, q, acc);
      if (c + 1 == a.ng) tile_sums_flush(sums, *sums_of);
    }
    __syncthreads();
  }
  run_store<D>(tp, phi + base, a, rows);
  if (REV) {
    run_store<D>(tl, lam + base, a, rows);
    if ((int)threadIdx.x < a.ng) {
      double s = 0.0;
      for (int w = 0; w < nw; ++w) s += (*sums_of)[threadIdx.x][w];
      partial[(size_t)a.g[threadIdx.x].k * rs + t] = s;
    }
  }
}

template <int D, bool REV>
__global__ __launch_bounds__(64 * kTileWaves) void k_tile_run(FuseArgs a, const float2 *__restrict__ src,
                                                              float2 *__restrict__ phi, float2 *__restrict__ lam,
                                                              FuseTables tab, double *__restrict__ partial, int rs) {
  extern __shared__ float2 lds[];
  run_tile<D, REV>(a, xcd_remap(blockIdx.x, gridDim.x), src, phi, lam, tab, partial, rs, lds);
}

// The same for the runs of many sweep points; tiles of points whose BFGS is idle
// this round are skipped.
template <int D, bool REV>
__global__ __launch_bounds__(64 * kTileWaves) void k_sweep_runs(const SweepRun *__restrict__ runs,
                                                                const int2 *__restrict__ tiles,
                                                                const int *__restrict__ active) {
  extern __shared__ float2 lds[];
  const int2 t = tiles[blockIdx.x];
  // read by scalar loads, like a kernel's arguments
  const SweepRun &r = *(const SweepRun *)(const SweepRun __attribute__((address_space(4))) *)(runs + t.x);
  if (!active[r.p]) return;
  run_tile<D, REV>(r.a, t.y, r.src, r.phi, r.lam, FuseTables{r.utab, r.rtab}, r.partial, r.rs, lds);
}

}  // namespace

bool fuse_supported(int d) { return d >= kTileMinD && d <= kTileMaxD; }

// Wavefronts of a run's workgroups: one for every unit (group of 64 fibres), in
// equal rounds where they are more than 16; at least four for the copies.
int fuse_waves(int D, int T) {
  const int units = D * ((T / (D * D) + 63) / 64), rounds = (units + kTileWaves - 1) / kTileWaves;
  return std::max(4, (units + rounds - 1) / rounds);
}

#define FOCK_RUN_SWITCH(d, STMT)                                              \
  switch (d) {                                                                \
    case 2: { constexpr int D = 2; STMT; } break;                             \
    case 3: { constexpr int D = 3; STMT; } break;                             \
    case 4: { constexpr int D = 4; STMT; } break;                             \
    case 5: { constexpr int D = 5; STMT; } break;                             \
    case 6: { constexpr int D = 6; STMT; } break;                             \
    case 7: { constexpr int D = 7; STMT; } break;                             \
    case 8: { constexpr int D = 8; STMT; } break;                             \
    default: return set_error(FOCK_ERR_UNSUPPORTED, "fused runs: d=%d", d);   \
  }

template <bool REV>
static int launch_run(const FuseArgs &a, const float2 *src, float2 *phi, float2 *lam, const FuseTables &tab,
                      double *partial, int rs, hipStream_t s) {
  const size_t lds = fuse_lds(a, REV);
  const dim3 grid(a.ntile), block(64 * fuse_waves(a.d, a.T));
  FOCK_RUN_SWITCH(a.d, hipLaunchKernelGGL((k_tile_run<D, REV>), grid, block, lds, s, a, src, phi, lam, tab, partial, rs));
  FOCK_HIP(hipGetLastError());
  return FOCK_OK;
}

int launch_fuse_fwd(const FuseArgs &a, const float2 *src, float2 *dst, const FuseTables &tab, hipStream_t s) {
  return launch_run<false>(a, src, dst, nullptr, tab, nullptr, 0, s);
}

int launch_fuse_adj(const FuseArgs &a, float2 *phi, float2 *lam, const FuseTables &tab, double *partial, int rs,
                    hipStream_t s) {
  if (a.ntile > rs) return set_error(FOCK_ERR_SIZE, "fused run: %d partials per gate exceed the row stride %d", a.ntile, rs);
  return launch_run<true>(a, nullptr, phi, lam, tab, partial, rs, s);
}

int sweep_launch_runs(int d, bool rev, const SweepRun *runs, const int2 *tiles, int n, int waves, size_t lds,
                      const int *active, hipStream_t s) {
  if (n <= 0) return FOCK_OK;
  const dim3 grid(n), block(64 * waves);
  if (rev) {
    FOCK_RUN_SWITCH(d, hipLaunchKernelGGL((k_sweep_runs<D, true>), grid, block, lds, s, runs, tiles, active));
  } else {
    FOCK_RUN_SWITCH(d, hipLaunchKernelGGL((k_sweep_runs<D, false>), grid, block, lds, s, runs, tiles, active));
  }
  FOCK_HIP(hipGetLastError());
  return FOCK_OK;
}

}  // namespace fock
