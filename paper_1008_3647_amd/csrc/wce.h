// Weak-coupling applications in the block-ordered eigenbasis of T (wce.hip).
#pragma once

#include "ops.h"

namespace ufg {

// y = W_d x (adjoint: W_d^T x) of the plan on a lattice with the block form of
// U (dimension 3, nx = 6 to 16); with `src`, x is formed as described at
// PcSource. Counts its M0^{-1} applications.
template <typename R>
int wce_modes_apply(Lattice& L, const PcPlan& pc, bool adjoint, const C2<R>* x, C2<R>* y,
                    int nrhs, const int* gate, Counters* cnt, const PcSource<R>* src);

// Time slices per workgroup of those launches.
int wce_slab(const Lattice& L, int nrhs, int order, bool fp64, bool fused_source);

}  // namespace ufg
