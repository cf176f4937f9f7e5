// FP64-state path: parameters and launchers (f64_kernels.hip, f64_small.hip).
#pragma once

#include "device_common.h"

namespace fock {

// Hamiltonian in double precision (same terms and signs as HamArgs).
struct H64 {
  int L, d, wrap;  // wrap: the ring bond (0, L-1) exists
  uint32_t n_amp;
  double J, Delta, c2, mu;  // c2 = U/2 + K
};

// Fibres of one op: M local amplitudes (d^2 over modes i < j, or d over mode i
// when j = -1), nfib fibres, fpw fibres per 256-thread workgroup.
struct Fib64 {
  int L, d, i, j, M, fpw;
  uint32_t si, sj, nfib;
};

Fib64 make_fib64(int L, int d, const fock_op_t &op);
int fib64_blocks(const Fib64 &a);
int launch64_apply_h(const H64 &h, const double2 *psi, double2 *hpsi, double *partial, int *nblocks, hipStream_t s);
int launch64_fib_apply(const Fib64 &a, const double2 *src, double2 *dst, const double2 *U, bool dag, hipStream_t s);
int launch64_fib_adj(const Fib64 &a, double2 *phi, double2 *lam, const double2 *U, const double2 *A,
                     double *partial, hipStream_t s);
int launch64_fib_pool(const Fib64 &a, const double2 *psi, const double2 *hpsi, const double2 *A, double *partial,
                      hipStream_t s);
// Dense M x M tables of n gates at utab + recs[k].u_off (Mmax = largest M).
int launch64_build(const double *theta, const GateRec *recs, int n, const EigTables &T, int Mmax, double2 *utab,
                   hipStream_t s);

// One evaluation of a small state by one workgroup (f64_small.hip): psi0 through
// the n gates, then (<phi|H phi>, <phi|phi>) into res[0..1] and, with grad,
// Re<lam_k|A_k phi_k> into res[2 + k]; without grad the states go to phi and
// lam, both times the global phase 0.8 + 0.6 i (f64_small.hip: why), which no
// energy, gradient or score depends on.  theta, gates (type | gate_modes << 8) and res are
// host-visible; links: small64_links.
struct Small64 {
  const double2 *psi0;
  double2 *phi, *lam;
  const double *theta;
  const double2 *links;
  const int *gates;
  double *res;
  int n, grad;
  int cap, batch;  // gate tables in LDS at a time, built `batch` at a time (set by the launcher)
};

// States and circuits it takes: both states and a few gate tables in one
// workgroup's LDS.
bool small64_ok(int d, uint32_t namp, int n);
// Those that are faster in it than gate by gate.
bool small64_used(const H64 &h, int n, bool grad);
// The diagonal and the links between levels of every generator at cutoff d <= 8, on
// the current device: made on first use and kept, like the gate eigendata (13 kB).
int small64_links(int d, const double2 **out);
int launch64_small(const Small64 &it, const H64 &h, const EigTables &T, hipStream_t s);
// Circuits of at most so many gates.
constexpr int kGates64 = 256;

}  // namespace fock
