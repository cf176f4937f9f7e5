// Passes over a circuit on complex64 states: planning and the fused runs' launchers.
#pragma once

#include <vector>

#include "tile_pair.h"

namespace fock {

constexpr int kMaxFuseModes = 13;   // tile modes
constexpr int kMaxFuseGates = 16;   // gates per run
constexpr int kTileMaxAmps = 8192;  // amplitudes of a tile

// LDS position of a tile's local index a.  At power-of-two d the five low bits are
// mixed with higher ones: 32 consecutive fibres of any mode pair of a 4-mode tile
// at d = 8 then lie in 32 different 8-byte banks (6 modes at d = 4: 1.3 to a
// bank).  Linear over bits, and a fibre's base and a member's offset have no bits
// in common: their positions combine by exclusive or.
__host__ __device__ constexpr int run_pos(int d, int a) {
  return (d & (d - 1)) == 0 ? a ^ (((a >> 3) ^ (a >> 5) ^ (a >> 6)) & 31) : a;
}

struct FuseGate {
  int type;
  int ki, kj;  // tile positions of the gate's modes (kj = -1: single-mode gate on ki)
  int u_off;   // offset of the gate's table in the gate-table block
  int k;       // index of the gate in the circuit (row of its gradient partials)
  TilePair p;  // local strides of its modes (tile_pair; a single mode with its next stride)
  // LDS byte offsets (8 run_pos) of 1, 2 and 4 levels of its modes
  int bi[3], bj[3];
};

// A gate's entries as a fused run reads them (fibre_gate.h): group g's at g d^2,
// the block of rows n_i <= g, then the other, one float an entry (the real part,
// or where A is imaginary and row and column are an odd number of levels apart
// the imaginary one); CK: (re, im) of the group's d members.
__host__ __device__ constexpr int fuse_table(int d) { return d * d * d; }
// The gate tables of a circuit: u by FuseGate::u_off, r by FuseGate::k.
struct FuseTables {
  const float2 *u;
  const float *r;
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

// Dynamic LDS of a run's workgroup: states, sums, row offsets and fibre positions
// of ng gates (tile_runs.hip), and the most there is.
constexpr size_t kFuseLds = 163840;
inline size_t fuse_lds(int d, int T, int ng, bool rev) {
  return sizeof(float2) * (size_t)((T + 31) & ~31) * (rev ? 2 : 1) + (rev ? sizeof(double) * 16 * 16 : 0) +
         sizeof(uint32_t) * (size_t)(T / d) + sizeof(uint16_t) * (size_t)ng * (T / (d * d));
}

bool fuse_supported(int d);
// The items that run together with item a: a, and later ones that `joins` takes (asked
// in order) and whose modes meet no item left behind: those commute with all of them
// and may move up.  all: every mode; cap: items at most.  Marks them done.
template <class Joins>
std::vector<int> take_run(int a, const std::vector<unsigned> &modes, unsigned all, size_t cap, std::vector<char> &done,
                          Joins joins) {
  std::vector<int> take{a};
  done[a] = 1;
  unsigned behind = 0u;
  for (int b = a + 1; b < (int)modes.size() && take.size() < cap && (~behind & all); ++b) {
    if (done[b]) continue;
    if (!(modes[b] & behind) && joins(b)) {
      take.push_back(b);
      done[b] = 1;
    } else {
      behind |= modes[b];
    }
  }
  return take;
}
// Passes of ops[0..n) in the order they run; fuse: with fused runs.
std::vector<GateGroup> plan_gate_groups(const Geometry &g, const fock_op_t *ops, int n, bool fuse);
int fuse_modes(const Geometry &g);
// Workgroups (tiles) of a fused run.
int fuse_tiles(const Geometry &g, const GateGroup &gr);
FuseArgs make_fuse_args(const Geometry &g, const EigTables &T, const GateGroup &gr, const fock_op_t *ops);
// Wavefronts of a run's workgroups.
int fuse_waves(int D, int T);
inline size_t fuse_lds(const FuseArgs &a, bool rev) { return fuse_lds(a.d, a.T, a.ng, rev); }
int launch_fuse_fwd(const FuseArgs &a, const float2 *src, float2 *dst, const FuseTables &tab, hipStream_t s);
int launch_fuse_adj(const FuseArgs &a, float2 *phi, float2 *lam, const FuseTables &tab, double *partial, int rs,
                    hipStream_t s);

}  // namespace fock
