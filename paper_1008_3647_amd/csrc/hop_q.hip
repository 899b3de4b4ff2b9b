// Q = M^T M (paper, Sec. 1, Eq. 1) in one launch, with the complex scaling of a
// Chebyshev factor: y = alpha Q x + beta x.
//
// With m = M x,
//   m_t = x_t + s_{t-1} T^3 (b_{t-1} x_{t-1}),   y_t = m_t + s_t b_t T^3 m_{t+1}.
// A workgroup of G groups of Nx^2 threads produces G - 1 slices of y: group g forms
// m_{t0+g} in registers, transforms it in its own LDS slice, and takes T^3 m_{t+1}
// from the slice of group g + 1. The G slices of m run side by side, so the
// chain is two transforms long whatever G, and m never goes to memory: x is read
// once (its neighbours' slices through the cache) and y written once, instead of
// five vector passes in two launches.
#include <algorithm>

#include "slice_t3.h"

namespace ufg {
namespace {

template <typename R>
struct QArgs {
  const C2<R>* x;
  C2<R>* y;
  const R* b;
  double2 alpha, beta;
  const int* gate;
  int nrhs;
};

// Blocks of up to 40 SGPRs (Nx = 8, complex64 Nx = 12) come in the kernel argument and
// stay in the scalar registers (degree 16 on 12^3 x 200, 8 rhs complex64 375 -> 336
// us, 8^3 x 160, 4 rhs 98.5 -> 96.1 us), larger ones are reloaded per stage (complex128
// Nx = 12 643 us, 678 us as an argument).
template <typename R, int NX>
using QCoef = typename std::conditional<(sizeof(SplitCoef<R, NX>) <= 160), SplitCoef<R, NX>,
                                        CoefPtr<R, NX>>::type;
template <typename R, int NX>
void set_coef(const Lattice& L, SplitCoef<R, NX>* c) {
  int k = 0;
  for (auto& v : c->es) v = R(L.split_host[k++]);
  for (auto& v : c->ea) v = R(L.split_host[k++]);
  for (auto& v : c->os) v = R(L.split_host[k++]);
  for (auto& v : c->oa) v = R(L.split_host[k++]);
}
template <typename R, int NX>
void set_coef(const Lattice& L, CoefPtr<R, NX>* c) {
  c->p = reinterpret_cast<const SplitCoef<R, NX>*>(fields<R>(L).split);
}

// alpha q + beta i
template <typename R>
__device__ __forceinline__ C2<R> q_epilogue(double2 alpha, double2 beta, C2<R> q, C2<R> i) {
  const R ar = R(alpha.x), ai = R(alpha.y), br = R(beta.x), bi = R(beta.y);
  C2<R> o;
  o.x = ar * q.x - ai * q.y;
  o.y = ar * q.y + ai * q.x;
  o.x += br * i.x - bi * i.y;
  o.y += br * i.y + bi * i.x;
  return o;
}

template <typename R, int NX, int G>
__global__ void __launch_bounds__(NX* NX* G)
    hop_q_kernel(QArgs<R> a, QCoef<R, NX> c, int ntau) {
  constexpr int P = NX * NX, V = NX * NX * NX, ES = sizeof(C2<R>), RS = sizeof(R);
  constexpr int SL = lds_slice_elems<NX>();
  extern __shared__ __align__(16) unsigned char smem_raw[];
  // contiguous runs of (slab, rhs) per XCD with the rhs fastest: the field and
  // the neighbouring slices come through one XCD's L2
  int lid = blockIdx.x;
  const int full = (int)gridDim.x & ~7;
  if (lid < full) lid = (lid & 7) * (full >> 3) + (lid >> 3);
  const int r = lid % a.nrhs, t0 = lid / a.nrhs * (G - 1);
  if (a.gate && a.gate[r] == 0) return;
  const int g = threadIdx.x / P, l = threadIdx.x - g * P;
  C2<R>* lds = reinterpret_cast<C2<R>*>(smem_raw) + g * SL;
  const int t = (t0 + g) % ntau, ts = t == 0 ? ntau - 1 : t - 1;
  const long long rbase = (long long)r * ntau * V;
  const auto rx = make_rsrc(a.x + rbase, (unsigned)ntau * V * ES);
  const auto rb = make_rsrc(a.b, (unsigned)ntau * V * RS);
  const auto ry = make_rsrc(a.y + rbase, (unsigned)ntau * V * ES);
  const int vo = (t * V + l) * ES;
  C2<R> X[NX], I[NX];
  {
    const int vs = (ts * V + l) * ES, fs = (ts * V + l) * RS;
#pragma unroll
    for (int z = 0; z < NX; ++z) X[z] = bload<R>(rx, vs, z * P * ES);
#pragma unroll
    for (int z = 0; z < NX; ++z) I[z] = bload<R>(rx, vo, z * P * ES);
#pragma unroll
    for (int z = 0; z < NX; ++z) {
      const R f = bload_real<R>(rb, fs, z * P * RS);
      X[z].x *= f;
      X[z].y *= f;
    }
  }
  slice_T3<R, NX>(c, lds, l, X);
  // m_t, kept in M; the identity term x_t stays in I
  const R sm = t == 0 ? R(1) : R(-1);
  C2<R> M[NX];
#pragma unroll
  for (int z = 0; z < NX; ++z) {
    M[z] = C2<R>{sm * X[z].x + I[z].x, sm * X[z].y + I[z].y};
    X[z] = M[z];
  }
  // the first slice's T^3 m is not needed: where a wave belongs to one group, its
  // waves only take part in the barriers (slice_T3 has two for 64 % Nx == 0)
  if (P % 64 == 0 && __builtin_amdgcn_readfirstlane(g) == 0) {
    slice_sync<NX>();
    slice_sync<NX>();
  } else {
    slice_T3<R, NX, 0, true>(c, lds, l, X);
  }
  if constexpr (P == 64) __syncthreads();  // the groups meet
  if (g == G - 1 || t0 + g >= ntau) return;
  const C2<R>* nb = lds + SL;
  const int y = l / NX, x = l - y * NX;
  const R sg = t == ntau - 1 ? R(1) : R(-1);
  R F[NX];
#pragma unroll
  for (int z = 0; z < NX; ++z) F[z] = sg * bload_real<R>(rb, (t * V + l) * RS, z * P * RS);
#pragma unroll
  for (int z = 0; z < NX; ++z) {
    const C2<R> w = nb[lds_at<NX>(z * NX + y, x)];
    const C2<R> q = C2<R>{F[z] * w.x + M[z].x, F[z] * w.y + M[z].y};
    bstore<R, false>(q_epilogue<R>(a.alpha, a.beta, q, I[z]), a.y + rbase, ry, vo,
                     z * P * ES);
  }
}

template <typename R, int NX, int G>
int launch_q(const Lattice& L, const QArgs<R>& a) {
  const size_t lds = size_t(G) * lds_slice_elems<NX>() * sizeof(C2<R>);
  static bool attr = false;
  if (!attr) {
    UFG_HIP(hipFuncSetAttribute((const void*)hop_q_kernel<R, NX, G>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    attr = true;
  }
  const int nblk = (L.ntau + G - 2) / (G - 1);
  QCoef<R, NX> c;
  set_coef<R, NX>(L, &c);
  hipLaunchKernelGGL((hop_q_kernel<R, NX, G>), dim3((unsigned)(nblk * a.nrhs)), dim3(NX * NX * G),
                     lds, L.stream, a, c, L.ntau);
  UFG_HIP(hipGetLastError());
  return UFG_OK;
}

}  // namespace

bool hop_q_pays(const Lattice& L, int nrhs, bool fp64) {
  // complex128 slices of Nx = 14 (47 KB of LDS each, two of them leave one
  // workgroup per CU): two launches once the chip is full (degree 8 on 14^3 x
  // 400, 8 rhs 1164 us against 1267 us; 14^3 x 100, 1 rhs 104 us fused)
  return stream_supported(L) && !(fp64 && L.nx == 14 && (long long)L.ntau * nrhs > 512);
}

template <typename R>
int launch_hop_q(const Lattice& L, const C2<R>* x, C2<R>* y, double2 alpha, double2 beta, int nrhs,
                 const int* gate) {
  if (!stream_supported(L) || fields<R>(L).split == nullptr || x == y) {
    set_error("fused M^T M: needs a lattice of the streaming kernels and distinct vectors");
    return UFG_EINVAL;
  }
  const QArgs<R> a{x, y, fields<R>(L).b, alpha, beta, gate, nrhs};
  // Groups per workgroup. More groups share the transforms of m (2 G - 1 for G - 1
  // slices of y) but fill fewer CUs: us for degree 16 at G = 2 / 3 / 4 / 5 or 8,
  // 8^3 x 160, 4 rhs complex128 130 / - / 98 / 119 (6), 8^3 x 400, 8 rhs 243 / - / 255 / 241
  // (8); 12^3 x 200, 1 rhs complex128 157 / 182 / 250 / 268, 8 rhs 896 / 722 / 842 / 647;
  // 16^3 x 400, 8 rhs complex64 1184 / 1423 / 1324 / - (complex128: two slices fill the
  // LDS); degree 8, 10^3 x 200, 1 rhs complex128 61 / 67 / 77 / 90 (6), 10^3 x 400, 8 rhs 338 /
  // 410 / 381 / 316 (6). In two launches a factor (M, then M^T with the scaling): 168, 437, 213, 776,
  // 1670 us, and complex128 16^3 x 400, 8 rhs 3492 -> 2960 us.
  const long long n = (long long)L.ntau * nrhs;  // slices
  switch (L.nx) {
    case 6: return n < 2048 ? launch_q<R, 6, 4>(L, a) : launch_q<R, 6, 8>(L, a);
    case 8: return n < 2048 ? launch_q<R, 8, 4>(L, a) : launch_q<R, 8, 8>(L, a);
    case 10:
      return n <= 512 ? launch_q<R, 10, 2>(L, a) : launch_q<R, 10, sizeof(R) == 4 ? 5 : 6>(L, a);
    case 12:
      // complex128: one workgroup per CU while that is enough (degree 8, us, two
      // launches / G = 2 / G = 3: 110 slices, 3 rhs 128 / 140 / 95; 400, 1 rhs 131 / 141 /
      // 98; 60, 8 rhs 139 / 145 / 105)
      if constexpr (sizeof(R) == 8) {
        if (n > 256 && n <= 512) return launch_q<R, 12, 3>(L, a);
      }
      return n <= 512 ? launch_q<R, 12, 2>(L, a) : launch_q<R, 12, 5>(L, a);
    case 14:
      if (sizeof(R) == 4 && n > 1024) return launch_q<R, 14, 4>(L, a);
      return launch_q<R, 14, 2>(L, a);
    case 16: return launch_q<R, 16, 2>(L, a);
    default: set_error("fused M^T M: unsupported nx"); return UFG_EINVAL;
  }
}

template int launch_hop_q<float>(const Lattice&, const float2*, float2*, double2, double2, int,
                                 const int*);
template int launch_hop_q<double>(const Lattice&, const double2*, double2*, double2, double2, int,
                                  const int*);

}  // namespace ufg
