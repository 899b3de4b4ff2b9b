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
// The four blocks of a line in the reflection-symmetry basis (os and oa start
// with index 1 of the line).
template <typename El, int NX>
struct Parts {
  using Z = SplitSize<NX>;
  El es[Z::ES], ea[Z::EA], os[Z::OS], oa[Z::OA];
};

// positions -> reflection-symmetry components (two butterfly levels)
template <typename R, int NX, typename El>
__device__ __forceinline__ void butterflies(const El (&a)[NX], Parts<El, NX>& p) {
  using Z = SplitSize<NX>;
  constexpr int H = NX / 2;
  El E[H + 1], O[H + 1];
  E[0] = a[0];
  E[H] = a[H];
#pragma unroll
  for (int j = 1; j < H; ++j) {
    E[j] = add(a[j], a[NX - j]);
    O[j] = sub(a[j], a[NX - j]);
  }
#pragma unroll
  for (int j = 0; j < Z::EA; ++j) {
    p.es[j] = add(E[j], E[H - j]);
    p.ea[j] = sub(E[j], E[H - j]);
  }
#pragma unroll
  for (int j = 1; j <= Z::OA; ++j) {
    p.os[j - 1] = add(O[j], O[H - j]);
    p.oa[j - 1] = sub(O[j], O[H - j]);
  }
  if constexpr (!Z::odd) {  // the fixed point of i -> NX/2 - i
    p.es[H / 2] = E[H / 2];
    p.os[H / 2 - 1] = O[H / 2];
  }
}

// out = m in for one N x N block
template <int N, typename M, typename El>
__device__ __forceinline__ void one_block(const M& m, const El (&in)[N], El (&out)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    El s = zero_of<El>();
#pragma unroll
    for (int k = 0; k < N; ++k) s = madd(m[i * N + k], in[k], s);
    out[i] = s;
  }
}

// out = blockdiag(c) in, block by block
template <typename R, int NX, typename Coef, typename El>
__device__ __forceinline__ void blockmul(const Coef& c, const Parts<El, NX>& in,
                                         Parts<El, NX>& out) {
  using Z = SplitSize<NX>;
  one_block<Z::ES>(c.es, in.es, out.es);
  one_block<Z::EA>(c.ea, in.ea, out.ea);
  one_block<Z::OS>(c.os, in.os, out.os);
  one_block<Z::OA>(c.oa, in.oa, out.oa);
}

// reflection-symmetry components -> positions (additions only)
template <typename R, int NX, typename El>
__device__ __forceinline__ void unbutterflies(const Parts<El, NX>& p, El (&a)[NX]) {
  using Z = SplitSize<NX>;
  constexpr int H = NX / 2;
  El E[H + 1], O[H + 1];
#pragma unroll
  for (int j = 0; j < Z::EA; ++j) {
    E[j] = add(p.es[j], p.ea[j]);
    E[H - j] = sub(p.es[j], p.ea[j]);
  }
#pragma unroll
  for (int j = 1; j <= Z::OA; ++j) {
    O[j] = add(p.os[j - 1], p.oa[j - 1]);
    O[H - j] = sub(p.os[j - 1], p.oa[j - 1]);
  }
  if constexpr (!Z::odd) {
    E[H / 2] = p.es[H / 2];
    O[H / 2] = p.os[H / 2 - 1];
  }
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
  using Z = SplitSize<NX>;
#pragma unroll
  for (int j = 0; j < Z::ES; ++j) a[j] = p.es[j];
#pragma unroll
  for (int j = 0; j < Z::EA; ++j) a[Z::ES + j] = p.ea[j];
#pragma unroll
  for (int j = 0; j < Z::OS; ++j) a[Z::ES + Z::EA + j] = p.os[j];
#pragma unroll
  for (int j = 0; j < Z::OA; ++j) a[Z::ES + Z::EA + Z::OS + j] = p.oa[j];
}
template <typename R, int NX, typename El>
__device__ __forceinline__ void unpack_modes(const El (&a)[NX], Parts<El, NX>& p) {
  using Z = SplitSize<NX>;
#pragma unroll
  for (int j = 0; j < Z::ES; ++j) p.es[j] = a[j];
#pragma unroll
  for (int j = 0; j < Z::EA; ++j) p.ea[j] = a[Z::ES + j];
#pragma unroll
  for (int j = 0; j < Z::OS; ++j) p.os[j] = a[Z::ES + Z::EA + j];
#pragma unroll
  for (int j = 0; j < Z::OA; ++j) p.oa[j] = a[Z::ES + Z::EA + Z::OS + j];
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
