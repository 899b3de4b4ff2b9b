// M and M^T on lattices of spatial dimension 1 and 2 with the block form of T
// (Nx = 6, dimension 1, and 8 to 16): y = alpha (x + s f T^d (f' x')) (+ beta aux), the operand
// conventions of the general slice kernels (HopArgs).
#include <type_traits>

#include "hop_common.h"
#include "slice_t3.h"

namespace ufg {
namespace {

// A thread holds a whole line of T in registers. A wave takes 64 / Nx slices
// (dimension 2; thread (slice, x) loads the y-line of column x) or 64 slices
// (dimension 1; elements loaded in memory order), so that its loads and stores
// cover whole contiguous pieces, and the lines along x are exchanged through an
// LDS tile: no block barrier, a wave is a workgroup (four to a workgroup: 16 x 100,
// 1 rhs complex128 4.5 -> 5.7 us, 8 x 8000, 16 rhs 43 -> 50). An element makes four LDS
// accesses and about Nx / 4 multiply-adds per axis; one thread per site with its
// row of T in registers makes 2 Nx + 2 accesses in dimension 2 and is bound by
// them. M / M^T, us, that -> this: 2D 16 x 1000, 8 rhs complex64 14.3 / 13.1 -> 8.6 /
// 8.5, complex128 24.4 / 22.8 -> 15.0 / 15.8 (11.5 at 5.9 TB/s); 2D 8 x 8000, 16 rhs
// complex128 50 / 44 -> 43 / 43; 1D 16 x 16000, 8 rhs complex64 10.4 / 9.1 -> 7.8 / 7.7,
// complex128 20.7 / 18.1 -> 14.7 / 14.3.
template <int NX, int D>
struct LineShape {
  static constexpr int V = D == 1 ? NX : NX * NX;    // sites per slice
  static constexpr int G = D == 1 ? 64 : 64 / NX;    // slices per wave
  static constexpr int STR = D == 1 ? 64 : NX;       // elements between a thread's elements
  static constexpr int ROWS = D == 1 ? 64 : G * NX;  // LDS rows of a wave
  static constexpr int TILE = ROWS * (NX + 1);
};

template <typename R, int NX, int D, int DIR, bool GENERAL, bool RED>
__global__ void __launch_bounds__(64)
    hop_line_kernel(HopArgs<R> a, CoefPtr<R, NX> cf, int ntau) {
  using S = LineShape<NX, D>;
  constexpr int V = S::V, STR = S::STR, ES = sizeof(C2<R>), RS = sizeof(R);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int nblk = (ntau + S::G - 1) / S::G;
  const int r = blockIdx.x / nblk, b = blockIdx.x - r * nblk;
  if (a.gate && a.gate[r] == 0) return;  // uniform over the block
  const int lane = threadIdx.x;
  C2<R>* lds = reinterpret_cast<C2<R>*>(smem_raw);
  const int N = ntau * V;
  const int sub = D == 1 ? 0 : lane / NX, x = D == 1 ? lane : lane - sub * NX;
  const bool act = lane < S::ROWS;
  // position of element i of this thread: p0 + i STR, past the end (its buffer
  // accesses are dropped) where the tile is not full
  const int p0 = act ? (b * S::G + sub) * V + x : N;
  // and of its source, one slice before (M) or after (M^T), antiperiodic: a
  // thread's elements share their slice in dimension 2
  auto source = [&](int i) {
    const int p = p0 + i * STR, w = D == 1 ? p : p0;
    if (DIR < 0) return w >= N ? N : (w < V ? p + N - V : p - V);
    return w >= N ? N : (w >= N - V ? p + V - N : p + V);
  };
  auto flips = [&](int i) {  // the term crosses the boundary, where s = +1
    const int w = D == 1 ? p0 + i * STR : p0;
    return DIR < 0 ? w < V : w >= N - V;
  };
  const auto rs = make_rsrc(a.src + (long long)r * N, N * ES);
  const auto rf = make_rsrc(DIR < 0 ? a.pre : a.post, N * RS);
  const auto ri = make_rsrc(a.id + (long long)r * N, a.id ? N * ES : 0);
  C2<R> v[NX], I[NX];
  R F[NX];
  // the identity term before the sources in FP64 M^T: its lines are those of the
  // tile before, read a moment ago (1D 10 x 16000, 16 rhs 16.2 -> 15.2 us, 2D 8 x
  // 8000, 16 rhs 45.3 -> 43.3; M no difference, complex64 7.7 -> 8.2 on 1D 16)
  constexpr bool kIdFirst = DIR > 0 && sizeof(R) == 8;
  if constexpr (kIdFirst) {
#pragma unroll
    for (int i = 0; i < NX; ++i) I[i] = bload<R>(ri, (p0 + i * STR) * ES, 0);
  }
#pragma unroll
  for (int i = 0; i < NX; ++i) v[i] = bload<R>(rs, source(i) * ES, 0);
#pragma unroll
  for (int i = 0; i < NX; ++i)
    F[i] = bload_real<R>(rf, (DIR < 0 ? source(i) : p0 + i * STR) * RS, 0);
  if constexpr (!kIdFirst) {
#pragma unroll
    for (int i = 0; i < NX; ++i) I[i] = bload<R>(ri, (p0 + i * STR) * ES, 0);
  }
#pragma unroll
  for (int i = 0; i < NX; ++i) F[i] = flips(i) ? F[i] : -F[i];
  if constexpr (DIR < 0) {
#pragma unroll
    for (int i = 0; i < NX; ++i) v[i] = C2<R>{F[i] * v[i].x, F[i] * v[i].y};
  }
  if constexpr (D == 2) line_op<0, R, NX>(cf, v);  // along y
  // element i in memory order, and element i of this thread's x-line
  auto slot = [&](int i) {
    if constexpr (D == 2) return (sub * NX + i) * (NX + 1) + x;
    const int e = i * 64 + lane;
    return (e / NX) * (NX + 1) + e % NX;
  };
  const int line = lane * (NX + 1);
  if (act) {
#pragma unroll
    for (int i = 0; i < NX; ++i) lds[slot(i)] = v[i];
  }
  // RED: the reduction's operand in flight during the lines along x, in instances of
  // their own for its registers. Loaded behind the output it was a wait of its own:
  // BiCGStab, us an iteration, 1D 16 x 400, 8 rhs complex128 M^T 38.8 -> 37.0 (a thread per
  // site: 37.2), 2D 16 x 400, 8 rhs 81 -> 73.5, 2D 8 x 200, 1 rhs 32.8 -> 31.2.
  C2<R> Q[RED ? NX : 1];
  if constexpr (RED) {
    const auto rw = make_rsrc(a.red_w + (long long)r * N, N * ES);
#pragma unroll
    for (int i = 0; i < NX; ++i) Q[i] = bload<R>(rw, (p0 + i * STR) * ES, 0);
  }
  wave_order();
  if (act) {
#pragma unroll
    for (int i = 0; i < NX; ++i) v[i] = lds[line + i];
  }
  line_op<0, R, NX>(cf, v);  // along x
  if (act) {
#pragma unroll
    for (int i = 0; i < NX; ++i) lds[line + i] = v[i];
  }
  wave_order();
  if (act) {
#pragma unroll
    for (int i = 0; i < NX; ++i) v[i] = lds[slot(i)];
  }
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    if constexpr (DIR < 0)
      v[i] = C2<R>{I[i].x + v[i].x, I[i].y + v[i].y};
    else
      v[i] = C2<R>{I[i].x + F[i] * v[i].x, I[i].y + F[i] * v[i].y};
  }
  if constexpr (GENERAL) {
    const R ar = R(a.alpha.x), ai = R(a.alpha.y), br = R(a.beta.x), bi = R(a.beta.y);
    const auto ra = make_rsrc(a.aux + (long long)r * N, a.aux ? N * ES : 0);
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const C2<R> q = bload<R>(ra, (p0 + i * STR) * ES, 0);  // zero without aux
      v[i] = C2<R>{ar * v[i].x - ai * v[i].y + (br * q.x - bi * q.y),
                   ar * v[i].y + ai * v[i].x + (br * q.y + bi * q.x)};
    }
  }
  C2<R>* dst = a.dst + (long long)r * N;
#pragma unroll
  for (int i = 0; i < NX; ++i)
    if (p0 + i * STR < N) dst[p0 + i * STR] = v[i];
  // The plain instances keep the late form, which the launcher does not use: without it
  // the compiler orders their loads differently (2D 16 x 1000, 8 rhs complex128 M 14.1 -> 14.5 us).
  if (!a.red_mode) return;
  // outside the lattice both factors are zero: w by its range check, v by its operands'
  double acc0 = 0, acc1 = 0, acc2 = 0, acc3 = 0;
  const auto rw = make_rsrc(a.red_w + (long long)r * N, N * ES);
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    const C2<R> q = RED ? Q[RED ? i : 0] : bload<R>(rw, (p0 + i * STR) * ES, 0);
    if (p0 + i * STR >= N) v[i] = C2<R>{R(0), R(0)};
    if (a.red_mode == 1) {  // <w, out> = sum conj(w) out
      acc0 += double(q.x) * v[i].x + double(q.y) * v[i].y;
      acc1 += double(q.x) * v[i].y - double(q.y) * v[i].x;
    } else {  // <out, w>, <out, out>, <w, w>
      acc0 += double(v[i].x) * q.x + double(v[i].y) * q.y;
      acc1 += double(v[i].x) * q.y - double(v[i].y) * q.x;
      acc2 += double(v[i].x) * v[i].x + double(v[i].y) * v[i].y;
      acc3 += double(q.x) * q.x + double(q.y) * q.y;
    }
  }
  hopc::block_sum4(acc0, acc1, acc2, acc3, a.red_out + ((long long)r * nblk + b) * 4,
                   reinterpret_cast<double*>(smem_raw));
}

template <typename R, int NX, int D, int DIR, bool GENERAL, bool RED>
int launch_one(const Lattice& L, const HopArgs<R>& a) {
  using S = LineShape<NX, D>;
  const size_t lds = size_t(S::TILE) * sizeof(C2<R>);
  static bool attr = false;
  if (!attr) {
    UFG_HIP(hipFuncSetAttribute((const void*)hop_line_kernel<R, NX, D, DIR, GENERAL, RED>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    attr = true;
  }
  const CoefPtr<R, NX> cf{reinterpret_cast<const SplitCoef<R, NX>*>(fields<R>(L).split)};
  const int nblk = (L.ntau + S::G - 1) / S::G;
  hipLaunchKernelGGL((hop_line_kernel<R, NX, D, DIR, GENERAL, RED>), dim3((unsigned)(nblk * a.nrhs)),
                     dim3(64), lds, L.stream, a, cf, L.ntau);
  UFG_HIP(hipGetLastError());
  return UFG_OK;
}

template <typename R, int NX, int D>
int launch_line(const Lattice& L, const HopArgs<R>& args) {
  HopArgs<R> a = args;
  if (a.beta.x == 0.0 && a.beta.y == 0.0) a.aux = nullptr;  // never read an unused operand
  const bool general = a.alpha.x != 1.0 || a.alpha.y != 0.0 || a.aux != nullptr;
  const bool red = a.red_mode != 0;
  auto launch = [&](auto dir) {
    constexpr int DIR = decltype(dir)::value;
    if (red)
      return general ? launch_one<R, NX, D, DIR, true, true>(L, a)
                     : launch_one<R, NX, D, DIR, false, true>(L, a);
    return general ? launch_one<R, NX, D, DIR, true, false>(L, a)
                   : launch_one<R, NX, D, DIR, false, false>(L, a);
  };
  return a.shift < 0 ? launch(std::integral_constant<int, -1>())
                     : launch(std::integral_constant<int, 1>());
}

}  // namespace

bool lowd_line_supported(const Lattice& L) {
  // buffer offsets are 32-bit: one rhs block of complex128 must stay below 2 GiB
  // (less what the last tile reaches past the end)
  // 2D Nx = 6 keeps a thread per site: pieces of 96 bytes, and 60 of 64 lanes
  // (4000 slices, 16 rhs complex128 M / M^T 16.2 / 14.2 us, lines 15.2 / 15.0)
  return L.dim < 3 && !L.split_host.empty() && !(L.dim == 2 && L.nx == 6) &&
         (long long)L.ntau * L.V * (long long)sizeof(double2) < (1ll << 31) - (1 << 20);
}

int lowd_line_blocks(const Lattice& L) {
  const int per = L.dim == 1 ? 64 : 64 / L.nx;  // slices per workgroup
  return (L.ntau + per - 1) / per;
}

template <typename R>
int launch_hop_lowd_line(const Lattice& L, const HopArgs<R>& a) {
  const bool fields_ok = a.shift < 0 ? (a.pre != nullptr && a.post == nullptr)
                                     : (a.post != nullptr && a.pre == nullptr);
  if (!lowd_line_supported(L) || a.shift == 0 || !fields_ok) {
    set_error("line kernel: M-type (field on the source) or M^T-type (field on the output) of a "
              "lattice of dimension 1 or 2 with a block form");
    return UFG_EINVAL;
  }
#define CALL_LINE(N) (L.dim == 1 ? launch_line<R, N, 1>(L, a) : launch_line<R, N, 2>(L, a))
  switch (L.nx) {
    case 6: return launch_line<R, 6, 1>(L, a);
    case 8: return CALL_LINE(8);
    case 10: return CALL_LINE(10);
    case 12: return CALL_LINE(12);
    case 14: return CALL_LINE(14);
    case 16: return CALL_LINE(16);
    default: set_error("line kernel: unsupported nx"); return UFG_EINVAL;
  }
#undef CALL_LINE
}

template int launch_hop_lowd_line<float>(const Lattice&, const HopArgs<float>&);
template int launch_hop_lowd_line<double>(const Lattice&, const HopArgs<double>&);

}  // namespace ufg
