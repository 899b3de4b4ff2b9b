// One line of the symmetric-circulant factor T applied in registers through
// its reflection-symmetry block form (the blocks are SplitCoef, built on the
// host by split_coefficients). Shared by the streaming operator and the
// batched operator.
#pragma once

#include "hop_stream.h"

namespace ufg {
namespace splitk {

// Line elements El: complex (C2<R>) or one real component (R) of it.
__device__ __forceinline__ float add(float a, float b) { return a + b; }
__device__ __forceinline__ double add(double a, double b) { return a + b; }
__device__ __forceinline__ float sub(float a, float b) { return a - b; }
__device__ __forceinline__ double sub(double a, double b) { return a - b; }
__device__ __forceinline__ float2 add(float2 a, float2 b) { return float2{a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ float2 sub(float2 a, float2 b) { return float2{a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ double2 add(double2 a, double2 b) {
  return double2{a.x + b.x, a.y + b.y};
}
__device__ __forceinline__ double2 sub(double2 a, double2 b) {
  return double2{a.x - b.x, a.y - b.y};
}
// s + m a
__device__ __forceinline__ float madd(float m, float a, float s) { return fma(m, a, s); }
__device__ __forceinline__ double madd(double m, double a, double s) { return fma(m, a, s); }
__device__ __forceinline__ float2 madd(float m, float2 a, float2 s) {
  return float2{fma(m, a.x, s.x), fma(m, a.y, s.y)};
}
__device__ __forceinline__ double2 madd(double m, double2 a, double2 s) {
  return double2{fma(m, a.x, s.x), fma(m, a.y, s.y)};
}
template <typename El>
__device__ __forceinline__ El zero_of() {
  return El{};
}

// y = T a for one line held in registers (in place), through the butterflies.
// The four blocks of a line in the reflection-symmetry basis (Q = NX/4):
// es[0..Q], ea[0..Q-1], os[1..Q], oa[1..Q-1].
template <typename El, int NX>
struct Parts {
  static constexpr int Q = NX / 4;
  El es[Q + 1], ea[Q + 1], os[Q + 1], oa[Q + 1];
};

// positions -> reflection-symmetry components (two butterfly levels)
template <typename R, int NX, typename El>
__device__ __forceinline__ void butterflies(const El (&a)[NX], Parts<El, NX>& p) {
  constexpr int H = NX / 2, Q = NX / 4;
  El E[H + 1], O[H + 1];
  E[0] = a[0];
  E[H] = a[H];
#pragma unroll
  for (int j = 1; j < H; ++j) {
    E[j] = add(a[j], a[NX - j]);
    O[j] = sub(a[j], a[NX - j]);
  }
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    p.es[j] = add(E[j], E[H - j]);
    p.ea[j] = sub(E[j], E[H - j]);
  }
  p.es[Q] = E[Q];
#pragma unroll
  for (int j = 1; j < Q; ++j) {
    p.os[j] = add(O[j], O[H - j]);
    p.oa[j] = sub(O[j], O[H - j]);
  }
  p.os[Q] = O[Q];
}

// out = blockdiag(c) in, block by block
template <typename R, int NX, typename Coef, typename El>
__device__ __forceinline__ void blockmul(const Coef& c, const Parts<El, NX>& in,
                                         Parts<El, NX>& out) {
  constexpr int Q = NX / 4;
#pragma unroll
  for (int i = 0; i <= Q; ++i) {
    El s = zero_of<El>();
#pragma unroll
    for (int k = 0; k <= Q; ++k) {
      const R m = c.es[i * (Q + 1) + k];
      s = madd(m, in.es[k], s);
    }
    out.es[i] = s;
  }
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    El s = zero_of<El>();
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      const R m = c.ea[i * Q + k];
      s = madd(m, in.ea[k], s);
    }
    out.ea[i] = s;
  }
#pragma unroll
  for (int i = 1; i <= Q; ++i) {
    El s = zero_of<El>();
#pragma unroll
    for (int k = 1; k <= Q; ++k) {
      const R m = c.os[(i - 1) * Q + (k - 1)];
      s = madd(m, in.os[k], s);
    }
    out.os[i] = s;
  }
#pragma unroll
  for (int i = 1; i < Q; ++i) {
    El s = zero_of<El>();
#pragma unroll
    for (int k = 1; k < Q; ++k) {
      const R m = c.oa[(i - 1) * (Q - 1) + (k - 1)];
      s = madd(m, in.oa[k], s);
    }
    out.oa[i] = s;
  }
}

// reflection-symmetry components -> positions (additions only)
template <typename R, int NX, typename El>
__device__ __forceinline__ void unbutterflies(const Parts<El, NX>& p, El (&a)[NX]) {
  constexpr int H = NX / 2, Q = NX / 4;
  El E[H + 1], O[H + 1];
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    E[j] = add(p.es[j], p.ea[j]);
    E[H - j] = sub(p.es[j], p.ea[j]);
  }
  E[Q] = p.es[Q];
#pragma unroll
  for (int j = 1; j < Q; ++j) {
    O[j] = add(p.os[j], p.oa[j]);
    O[H - j] = sub(p.os[j], p.oa[j]);
  }
  O[Q] = p.os[Q];
  a[0] = E[0];
  a[H] = E[H];
#pragma unroll
  for (int j = 1; j < H; ++j) {
    a[j] = add(E[j], O[j]);
    a[NX - j] = sub(E[j], O[j]);
  }
}

// y = T a for one line held in registers (in place)
template <typename R, int NX, typename Coef, typename El>
__device__ __forceinline__ void split_line(const Coef& c, El (&a)[NX]) {
  Parts<El, NX> u, w;
  butterflies<R, NX, El>(a, u);
  blockmul<R, NX>(c, u, w);
  unbutterflies<R, NX>(w, a);
}

// Mode-space packing of a line: the blocks in the order es, ea, os, oa.
template <typename R, int NX, typename El>
__device__ __forceinline__ void pack_modes(const Parts<El, NX>& p, El (&a)[NX]) {
  constexpr int Q = NX / 4;
#pragma unroll
  for (int j = 0; j <= Q; ++j) a[j] = p.es[j];
#pragma unroll
  for (int j = 0; j < Q; ++j) a[Q + 1 + j] = p.ea[j];
#pragma unroll
  for (int j = 1; j <= Q; ++j) a[2 * Q + j] = p.os[j];
#pragma unroll
  for (int j = 1; j < Q; ++j) a[3 * Q + j] = p.oa[j];
}
template <typename R, int NX, typename El>
__device__ __forceinline__ void unpack_modes(const El (&a)[NX], Parts<El, NX>& p) {
  constexpr int Q = NX / 4;
#pragma unroll
  for (int j = 0; j <= Q; ++j) p.es[j] = a[j];
#pragma unroll
  for (int j = 0; j < Q; ++j) p.ea[j] = a[Q + 1 + j];
#pragma unroll
  for (int j = 1; j <= Q; ++j) p.os[j] = a[2 * Q + j];
#pragma unroll
  for (int j = 1; j < Q; ++j) p.oa[j] = a[3 * Q + j];
}

// c = U^T a in the block-ordered eigenbasis of T (positions -> modes)
template <typename R, int NX, typename Coef, typename El>
__device__ __forceinline__ void modes_fwd(const Coef& c, El (&a)[NX]) {
  Parts<El, NX> u, w;
  butterflies<R, NX, El>(a, u);
  blockmul<R, NX>(c, u, w);
  pack_modes<R, NX, El>(w, a);
}

// a = U c from block-ordered modes (modes -> positions)
template <typename R, int NX, typename Coef, typename El>
__device__ __forceinline__ void modes_bwd(const Coef& c, El (&a)[NX]) {
  Parts<El, NX> u, w;
  unpack_modes<R, NX>(a, u);
  blockmul<R, NX>(c, u, w);
  unbutterflies<R, NX>(w, a);
}

}  // namespace splitk
}  // namespace ufg
