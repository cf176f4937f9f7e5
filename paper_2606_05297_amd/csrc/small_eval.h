// Whole-circuit evaluation of small states by one workgroup (small_eval.hip).
#pragma once

#include "fock_internal.h"

namespace fock {

constexpr int kSmallModes = 16;
constexpr int kSmallGates = 256;

// One evaluation: phi = O_n..O_1 psi0, lam = H phi, (<phi|H phi>, <phi|phi>)
// into res[0..1] and, with grad, Re<lam_k|A_k phi_k> into res[2 + k].  Without
// grad the states are written to phi and lam; with it they stay on chip.
struct SmallItem {
  const float2 *psi0;
  float2 *phi, *lam;
  const float2 *U;      // table of gate 0; gate k at k * ustride
  const GateRec *recs;  // type and modes (GateRec::modes) of the n gates
  double *res;
  int n, grad, point;   // point: index into the active flags (sweep), or -1
  int L, d, N, wrap, ustride;
  int chunk;            // gate tables in LDS at a time (small_chunk)
  float J, Delta, c2, mu;
};

// States this evaluation takes: both states of the reverse sweep, complex64, in
// the LDS of one workgroup, and d <= 8 (a group of d members fills one matrix
// operand), circuits of up to kSmallGates gates (their descriptions in LDS).
bool small_eval_ok(int L, int d, uint32_t namp, int n);
// Those the library's plan gives to it (gate_plan.cpp).
bool small_planned(const Geometry &g, const fock_op_t *ops, int n);
int small_chunk(int d, uint32_t namp, int n);
// LDS of one item's workgroup.
size_t small_lds_bytes(const SmallItem &it);
// Its wavefronts (a function of d and N alone).
int small_waves(const SmallItem &it);
// One workgroup per item: `one`, or items[0..count) (device) when count > 0;
// lds: the largest small_lds_bytes among them; waves: their common
// small_waves.  active (device, nullable):
// items whose flag is 0 are skipped.
int launch_small_eval(const SmallItem &one, const SmallItem *items, int count, size_t lds, int waves, const EigTables &T,
                      const int *active, hipStream_t s);

}  // namespace fock
