// Passes over a circuit on complex64 states: planning and the fused runs' launchers.
#pragma once

#include <vector>

#include "tile_pair.h"

namespace fock {

constexpr int kMaxFuseModes = 13;   // tile modes
constexpr int kMaxFuseGates = 16;   // gates per run
constexpr int kTileMaxAmps = 8192;  // amplitudes of a tile

struct FuseGate {
  int type;
  int ki, kj;  // tile positions of the gate's modes (kj = -1: single-mode gate on ki)
  int u_off;   // offset of the gate's table in the gate-table block
  int k;       // index of the gate in the circuit (row of its gradient partials)
  TilePair p;  // local strides of its modes (tile_pair; a single mode with its next stride)
};

struct FuseArgs {
  int d, s, nc, ng, ntile, T;       // T = d^s amplitudes of a tile
  FastDiv dd;                       // divides by d
  uint32_t tstride[kMaxFuseModes];  // d^m of the tile modes, ascending (tile position 0 = mode 0)
  uint32_t cstride[kMaxL];          // d^m of the other modes, ascending (digits of the tile index)
  const float2 *A[kTwoModeTypes];   // packed generator blocks of the two-mode types by table_slot (gradients)
  FuseGate g[kMaxFuseGates];
};

// One pass: the gates k (indices into the circuit, in the order applied) as a
// fused run on the tile modes m[0..s) (s > 0), as a run of single-mode phase
// gates in one diagonal pass (diag; consecutive indices), or one gate on its own
// kernel.
struct GateGroup {
  std::vector<int> k;
  int s = 0;
  int m[kMaxFuseModes] = {};
  bool diag = false;
};

bool fuse_supported(int d);
// Passes of ops[0..n) in the order they run; fuse: with fused runs.
std::vector<GateGroup> plan_gate_groups(const Geometry &g, const fock_op_t *ops, int n, bool fuse);
int fuse_modes(const Geometry &g);
// Workgroups (tiles) of a fused run.
int fuse_tiles(const Geometry &g, const GateGroup &gr);
FuseArgs make_fuse_args(const Geometry &g, const EigTables &T, const GateGroup &gr, const fock_op_t *ops);
// Wavefronts and dynamic LDS of a run's workgroups.
int fuse_waves(int D, int T);
size_t fuse_lds(const FuseArgs &a, bool rev);
int launch_fuse_fwd(const FuseArgs &a, const float2 *src, float2 *dst, const float2 *utab, hipStream_t s);
int launch_fuse_adj(const FuseArgs &a, float2 *phi, float2 *lam, const float2 *utab, double *partial, int rs,
                    hipStream_t s);

}  // namespace fock
