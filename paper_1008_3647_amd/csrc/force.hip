// Force contraction (paper, Sec. 1) on lattices with the block form of T
// (dimension 3, Nx = 6 to 16): per site of slice t,
//   grad = -2 A cos sigma * s_t * sum_r Re[X_t conj((T^3 y_{t+1}))].
#include "slice_t3.h"

namespace ufg {
namespace {

// A complex64 lattice has its force in double precision too, and the rounding of
// its FP32 transform stays what the dense product gives: the same terms in the
// same order, one component at a time (16^3 x 400, 8 rhs 94 -> 72 us; the block form
// 55 us, but 1.6e-7 away from the dense product's rounding).
template <typename R, int NX>
struct DenseT {
  const R* p;  // T, row by row
};
template <int MODE, typename R, int NX>
__device__ __forceinline__ void line_op(const DenseT<R, NX>& c, R (&v)[NX]) {
  using CC = const __attribute__((address_space(4))) R;
  CC* m = (CC*)c.p;
  asm volatile("" : "+s"(m));
  R w[NX];
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    R acc = R(0);
#pragma unroll
    for (int j = 0; j < NX; ++j) acc = fma(m[i * NX + j], v[j], acc);
    w[i] = acc;
  }
#pragma unroll
  for (int i = 0; i < NX; ++i) v[i] = w[i];
}
template <typename R, int NX>
using ForceT = std::conditional_t<sizeof(R) == 4, DenseT<R, NX>, CoefPtr<R, NX>>;

// A workgroup takes one slice t and all right-hand sides, one real component of
// y and X per Nx^2 threads (T is real, and the real part of the product is the
// sum over components), the two sums added through LDS at the end. One or a few
// slices per CU, so the launch is bound by the latency of a slice: half the work
// per thread, the operands of X loaded before the transform, cos sigma read
// from the installed field instead of computed. force_dS_dsigma, us, complex
// slices with dense lines and a cosine per site -> this: 12^3 x 200 complex128
// 11.8 -> 6.0 (bound by the host), 16^3 x 400, 8 rhs complex128 149 -> 118 (71 at
// 5.9 TB/s).
template <typename R, int NX>
__global__ void __launch_bounds__(2 * NX * NX)
    force_block_kernel(const C2<R>* __restrict__ X, const C2<R>* __restrict__ y, ForceT<R, NX> cf,
                       const double* __restrict__ cs, double A, int ntau, int nrhs,
                       double* __restrict__ grad) {
  constexpr int P = NX * NX, V = NX * NX * NX, RS = sizeof(R);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int comp = threadIdx.x >= P ? 1 : 0;
  const int l = threadIdx.x - comp * P;
  R* lds = reinterpret_cast<R*>(smem_raw) + comp * lds_slice_elems<NX>();
  const int t = blockIdx.x;
  const int tp = t + 1 == ntau ? 0 : t + 1;
  const int vo = (2 * l + comp) * RS;
  double acc[NX];
#pragma unroll
  for (int z = 0; z < NX; ++z) acc[z] = 0.0;
  for (int r = 0; r < nrhs; ++r) {
    const auto ry = make_rsrc(y + ((long long)r * ntau + tp) * V, 2 * V * RS);
    const auto rx = make_rsrc(X + ((long long)r * ntau + t) * V, 2 * V * RS);
    R v[NX], q[NX];
#pragma unroll
    for (int z = 0; z < NX; ++z) v[z] = bload_real<R>(ry, vo, 2 * z * P * RS);
#pragma unroll
    for (int z = 0; z < NX; ++z) q[z] = bload_real<R>(rx, vo, 2 * z * P * RS);
    slice_T3<R, NX>(cf, lds, l, v);
#pragma unroll
    for (int z = 0; z < NX; ++z) acc[z] += double(q[z]) * v[z];
  }
  // component 0 finishes the lower half of the z-line, component 1 the upper
  constexpr int H = NX / 2;
  double* ex = reinterpret_cast<double*>(smem_raw);
  __syncthreads();  // the slices' last reads, before their LDS is reused
#pragma unroll
  for (int z = 0; z < H; ++z) ex[(comp * H + z) * P + l] = comp ? acc[z] : acc[H + z];
  __syncthreads();
  const double c = (t == ntau - 1 ? -2.0 : 2.0) * A;
#pragma unroll
  for (int z = 0; z < H; ++z) {
    const double s = (comp ? acc[H + z] : acc[z]) + ex[((1 - comp) * H + z) * P + l];
    const long long i = (long long)t * V + (comp * H + z) * P + l;
    grad[i] = c * cs[i] * s;
  }
}

template <typename R, int NX>
int launch_nx(const Lattice& L, const C2<R>* X, const C2<R>* y, int nrhs, double* grad) {
  const size_t lds =
      std::max(size_t(2) * lds_slice_elems<NX>() * sizeof(R), size_t(NX) * NX * NX * sizeof(double));
  static bool attr = false;
  if (!attr) {
    UFG_HIP(hipFuncSetAttribute((const void*)force_block_kernel<R, NX>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    attr = true;
  }
  ForceT<R, NX> cf;
  if constexpr (sizeof(R) == 4)
    cf.p = fields<R>(L).T;
  else
    cf.p = reinterpret_cast<const SplitCoef<R, NX>*>(fields<R>(L).split);
  hipLaunchKernelGGL((force_block_kernel<R, NX>), dim3((unsigned)L.ntau), dim3(2 * NX * NX), lds,
                     L.stream, X, y, cf, L.f64.cs, L.A, L.ntau, nrhs, grad);
  UFG_HIP(hipGetLastError());
  return UFG_OK;
}

}  // namespace

template <typename R>
int launch_force_block(const Lattice& L, const C2<R>* X, const C2<R>* y, int nrhs, double* grad) {
  switch (L.nx) {
    case 6: return launch_nx<R, 6>(L, X, y, nrhs, grad);
    case 8: return launch_nx<R, 8>(L, X, y, nrhs, grad);
    case 10: return launch_nx<R, 10>(L, X, y, nrhs, grad);
    case 12: return launch_nx<R, 12>(L, X, y, nrhs, grad);
    case 14: return launch_nx<R, 14>(L, X, y, nrhs, grad);
    case 16: return launch_nx<R, 16>(L, X, y, nrhs, grad);
    default: set_error("force: unsupported nx"); return UFG_EINVAL;
  }
}

template int launch_force_block<float>(const Lattice&, const float2*, const float2*, int, double*);
template int launch_force_block<double>(const Lattice&, const double2*, const double2*, int,
                                        double*);

}  // namespace ufg
