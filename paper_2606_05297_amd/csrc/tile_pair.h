// Fibre decomposition of a gate on an LDS tile (tile_gate.h).
#pragma once

#include "device_common.h"

namespace fock {

// Fibre decomposition of a gate on tile modes with strides si < sj: fibre
// f = low + si (mid + dm high), dm = sj / (si D).  Computed once per gate and
// launch (the divisions cost more than the gate on a small tile).
struct TilePair {
  int si, sj, dm;
  float rsi, rdm;
};
__host__ __device__ inline TilePair tile_pair(int si, int sj, int D) {
  TilePair p;
  p.si = si;
  p.sj = sj;
  p.dm = sj / (si * D);
  p.rsi = 1.0f / (float)si;
  p.rdm = 1.0f / (float)p.dm;
  return p;
}

}  // namespace fock
