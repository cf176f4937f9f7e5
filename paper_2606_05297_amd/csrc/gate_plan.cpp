// How a circuit on complex64 states is cut into passes: runs of single-mode
// phase gates (one diagonal pass), fused runs of gates inside one tile
// (tile_runs.hip) and single gates on their own kernels.  Host only; the
// single-point drivers and the batched sweep plan with this one function.
#include <algorithm>
#include <cstring>

#include "fuse_internal.h"
#include "small_eval.h"

namespace fock {

namespace {

// A gate, or a run of single-mode phase gates, to be placed as a whole.
struct Item {
  int k0, k1;
  bool fusable;
};

unsigned mode_mask(const fock_op_t &o) { return (1u << o.i) | (op_j(o) >= 0 ? 1u << o.j : 0u); }

}  // namespace

// Modes of a fused run's tile: as many as the LDS of one workgroup holds (both
// states of the reverse sweep, kTileMaxAmps each) while 100 tiles are left to
// keep the chip busy, but never so few that a wavefront's lanes (a fibre each,
// d^(s - 2) of them) stay empty: half of them filled on a handful of CUs is faster
// than many CUs with few, and the longer runs save passes.  Measured, an
// evaluation in us by modes (tiles): 8^5 4 (8) 217, 3 (64) 293; 5^6 5 (5) 137,
// 4 (25) 153, 3 (125) 184; 7^5 4 (7) 158, 3 (49) 198; 3^9 6 (27) 200, 5 (81) 219;
// 4^8 5 (64) 215, 4 (256) 240; 5^8 5 (125) 206, 4 (625) 220; 6^8 5 (216) 455, 4
// (1296) 603; but 6^7 5 (36) 315, 4 (216) 276; 6^6 5 (6) 290, 4 (36) 237.
int fuse_modes(const Geometry &g) {
  const int Lf = g.half ? g.L - 1 : g.L;
  int many = 0, full = 0, s = 1;
  for (long T = g.d; s <= Lf && s <= kMaxFuseModes && T <= kTileMaxAmps; T *= g.d, ++s) {
    if (fuse_lds(g.d, (int)T, kMaxFuseGates, true) > kFuseLds) break;  // d = 2, 8,192 amplitudes: fibre positions
    if ((long)g.n_amp / T >= 100) many = s;
    if (!full && T / (g.d * g.d) >= 32 && (long)g.n_amp / T >= 4) full = s;
  }
  return std::max(many, full);
}

// Whether the library's plan evaluates a circuit on a small state whole, in one
// workgroup (small_eval.hip), rather than pass by pass.
//
// Above 4,096 amplitudes (d = 2: 2,048) not where fused runs are at hand: the chip
// is faster than one CU there.  30 gates with gradients, us, fused / whole: 8,192
// amplitudes at d = 2 164 / 407, 4,096 166 / 244, 6,561 (d = 3) 164 / 294, 7,776
// (d = 6) 207 / 298; but 4,096 at d = 4 with a warm-up layer 142 / 135, and 1,024
// at d = 2 147 / 121.  With one or two gates on 4,096 amplitudes of six modes H psi
// is most of the call, 37 us by its own kernel, 41 whole.
//
// Elsewhere a two-mode gate saves 4 us at least against a pass forward and one in
// reverse, and the call 4 us by itself, but two things cost more than in passes:
// a squeezer (dense: one thread a fibre) at d >= 6, 1, 2.5 and 5 us, and each phase
// gate that a diagonal pass would take along, up to N / 2000 us.  Pass by pass /
// whole: 30 squeezers at d = 8, 512 amplitudes 241 / 358, one or two alone 39 / 42 at
// 3,125 (d = 5), 30 phase gates at 4,096 amplitudes (d = 8) 80 / 116, ten at 1,024
// (d = 4) 50 / 54.
bool small_planned(const Geometry &g, const fock_op_t *ops, int n) {
  if (g.half || !small_eval_ok(g.L, g.d, g.n_amp, n)) return false;
  if (fuse_supported(g.d) && fuse_modes(g) >= 3) {
    if (g.n_amp > (g.d == 2 ? 2048u : 4096u)) return false;
    if (g.n_amp == 4096 && n > 0 && n <= 2) return false;
  }
  double saved = 4.0, lost = 0.0;
  int squeezers = 0;
  for (int k = 0; k < n;) {
    const int end = std::max(diag_run_end(ops, n, k), k + 1);
    if (is_squeeze(ops[k].type)) {
      ++squeezers;
      lost += g.d == 8 ? 5.0 : g.d == 7 ? 2.5 : g.d == 6 ? 1.0 : 0.0;
    } else if (!is_single_mode(ops[k].type)) {
      saved += 4.0;
    }
    lost += (end - k - 1) * (double)g.n_amp / 2000.0;
    k = end;
  }
  return saved >= lost && (n == 0 || n > 2 || squeezers < n);
}

std::vector<GateGroup> plan_gate_groups(const Geometry &g, const fock_op_t *ops, int n, bool fuse) {
  const int Lf = g.half ? g.L - 1 : g.L, smax = fuse_modes(g);
  const bool on = fuse && fuse_supported(g.d) && smax >= 3;
  std::vector<Item> items;
  std::vector<unsigned> modes;
  for (int k = 0; k < n;) {
    Item it{k, std::max(diag_run_end(ops, n, k), k + 1), false};
    unsigned m = 0u;
    for (int q = it.k0; q < it.k1; ++q) m |= mode_mask(ops[q]);
    it.fusable = on && it.k1 == it.k0 + 1 && !is_squeeze(ops[k].type) && !(m >> Lf);
    items.push_back(it);
    modes.push_back(m);
    k = it.k1;
  }
  std::vector<GateGroup> out;
  std::vector<char> done(items.size(), 0);
  for (size_t a = 0; a < items.size(); ++a) {
    if (done[a]) continue;
    GateGroup gr;
    unsigned mask = 1u | modes[a];  // mode 0 always, so that rows stay contiguous
    const bool open = items[a].fusable && __builtin_popcount(mask) <= smax;
    // later gates join while the union of modes fits the tile
    const std::vector<int> take = take_run((int)a, modes, (1u << g.L) - 1, open ? kMaxFuseGates : 1, done, [&](int b) {
      const unsigned u = mask | modes[b];
      if (!items[b].fusable || __builtin_popcount(u) > smax) return false;
      mask = u;
      return true;
    });
    if (take.size() > 1)  // the tile's other modes: the lowest
      for (int r = 0; r < Lf && __builtin_popcount(mask) < smax; ++r) mask |= 1u << r;
    for (int b : take)
      for (int k = items[b].k0; k < items[b].k1; ++k) gr.k.push_back(k);
    gr.diag = take.size() == 1 && gr.k.size() > 1;
    if (take.size() > 1)
      for (int r = 0; r < Lf; ++r)
        if (mask & (1u << r)) gr.m[gr.s++] = r;
    out.push_back(gr);
  }
  return out;
}

int fuse_tiles(const Geometry &g, const GateGroup &gr) {
  int T = 1;
  for (int r = 0; r < gr.s; ++r) T *= g.d;
  return (int)(g.n_amp / (uint32_t)T);
}

FuseArgs make_fuse_args(const Geometry &g, const EigTables &T, const GateGroup &gr, const fock_op_t *ops) {
  FuseArgs a;
  memset(&a, 0, sizeof(a));
  const int L = g.L, d = g.d;
  std::vector<uint32_t> pw(L, 1);
  for (int r = 1; r < L; ++r) pw[r] = pw[r - 1] * (uint32_t)d;
  a.d = d;
  a.dd = make_fastdiv((uint32_t)d);
  a.s = gr.s;
  a.T = 1;
  std::vector<int> pos(L, -1);
  for (int k = 0; k < gr.s; ++k) {
    a.tstride[k] = pw[gr.m[k]];
    pos[gr.m[k]] = k;
    a.T *= d;
  }
  a.ntile = fuse_tiles(g, gr);
  for (int r = 0; r < L; ++r)
    if (pos[r] < 0) a.cstride[a.nc++] = pw[r];
  for (int t = 0; t < kTwoModeTypes; ++t) a.A[t] = T.A[t];
  a.ng = (int)gr.k.size();
  for (int q = 0; q < a.ng; ++q) {
    const int k = gr.k[q];
    const fock_op_t &o = ops[k];
    FuseGate &f = a.g[q];
    f.type = o.type;
    f.ki = pos[o.i];
    f.kj = op_j(o) < 0 ? -1 : pos[o.j];
    f.u_off = k * gate_stride(d);
    f.k = k;
    int si = 1, sj = 1;
    for (int e = 0; e < f.ki; ++e) si *= d;
    for (int e = 0; e < (f.kj < 0 ? f.ki + 1 : f.kj); ++e) sj *= d;
    f.p = tile_pair(si, sj, d);
    for (int b = 0; b < 3; ++b) {
      f.bi[b] = 8 * run_pos(d, si << b);
      f.bj[b] = 8 * run_pos(d, sj << b);
    }
  }
  return a;
}

}  // namespace fock
