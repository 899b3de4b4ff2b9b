// Block coefficients of the symmetric-circulant T in the basis of its two
// reflection symmetries, and the streaming M / M^T launcher.
#pragma once

#include "ufg_internal.h"

namespace ufg {

// Sizes of the four blocks of a line of even NX: even / odd under i -> -i (E, O),
// then symmetric / antisymmetric under i -> NX/2 - i (S, A).
template <int NX>
struct SplitSize {
  static constexpr int H = NX / 2;
  static constexpr bool odd = H % 2 != 0;
  static constexpr int ES = odd ? (H + 1) / 2 : H / 2 + 1;
  static constexpr int EA = odd ? (H + 1) / 2 : H / 2;
  static constexpr int OS = odd ? (H - 1) / 2 : H / 2;
  static constexpr int OA = odd ? (H - 1) / 2 : H / 2 - 1;
};

template <typename R, int NX>
struct SplitCoef {
  using Z = SplitSize<NX>;
  R es[Z::ES * Z::ES];
  R ea[Z::EA * Z::EA];
  R os[Z::OS * Z::OS];
  R oa[Z::OA * Z::OA];
};

// Host: the blocks for even nx of 6 to 16 in the order es, ea, os, oa
// (row-major each); empty for other nx. Returns the largest off-block entry
// of the transformed matrix (a self-check).
double split_coefficients(int nx, const std::vector<double>& T, std::vector<double>* out);

// Host: the block-diagonal forward (U^T) and backward (U) maps of the
// eigenbasis of T, with the block ordering of the modes (perm); empty for nx
// below 6. Returns the largest off-block entry (a self-check).
double mode_split_coefficients(int nx, const std::vector<double>& U, std::vector<double>* fwd,
                               std::vector<double>* bwd, std::vector<int>* perm);

int stream_slab(const Lattice& L);
// Slabs per right-hand side: slab s of nslab covers slices [s ntau / nslab,
// (s + 1) ntau / nslab), so every slab holds floor or ceil of ntau / nslab.
int stream_nslab(const Lattice& L);
// Slab groups per XCD of the workgroup numbering (0: contiguous (slab, rhs)
// runs per XCD with the rhs fastest), and the grid of a launch over nrhs.
int stream_group(const Lattice& L);
int stream_grid(const Lattice& L, int nrhs);
// 1: an XCD takes every rhs of a slab group in turn (default or lattice_tune_order)
int stream_inner(const Lattice& L);
bool stream_supported(const Lattice& L);
template <typename R>
int launch_hop_stream(const Lattice& L, const HopArgs<R>& a);

// y = alpha Q x + beta x, Q = M^T M, in one launch (hop_q.hip; stream_supported
// lattices; hop_q_pays: where that is faster than two). y must not alias x.
bool hop_q_pays(const Lattice& L, int nrhs, bool fp64);
template <typename R>
int launch_hop_q(const Lattice& L, const C2<R>* x, C2<R>* y, double2 alpha, double2 beta, int nrhs,
                 const int* gate);

}  // namespace ufg
