// Weak-coupling series W_d (paper, Sec. 3) on lattices with the block form of
// the eigenbasis U of T (dimension 3, Nx = 6 to 16).
//
// M0^{-1} = U^3 (1 - lam Z)^{-1} U^3T: a basis change per time slice, the
// antiperiodic recurrence u_t = v_t + lam u_{t-1}, u_{-1} = -u_{Ntau-1} per mode,
// and the change back. The recurrence is not a pass of its own: a workgroup
// walks a slab of consecutive slices in sweep order, a thread keeps one z-line
// of modes, so
//   - the launch that changes to the modes writes v_t and, in registers, runs
//     the slab's recurrence from zero; only its last value g (one slice per
//     slab) is stored;
//   - wce_scan_kernel turns the g of all slabs into the value before each slab
//     (U_j = g_j + lam^len U_{j-1}, closed antiperiodically), in FP64;
//   - the launch that changes back runs the recurrence from that value while
//     it loads v_t.
// (1 - lam Z)^{-1} - 1, which the series needs, is lam u_{t-1} directly. The
// adjoint runs the same on reversed time. Consecutive orders of the series
// meet as "change back, per-site factors, change to the modes", one launch
// (PAIR). The order-2 application is FIRST, PAIR, PAIR, LAST with a scan
// between them: 11 vector passes and 3 small scans, where a temporal solve as
// a launch of its own (3 passes each) needed 20.
#include <algorithm>
#include <cmath>

#include "slice_t3.h"
#include "wce.h"

namespace ufg {
namespace {

// Every map of the series is real, so the two components of a vector are
// independent problems: between the first and the last change the vectors (v,
// u_0, the carries) are planar, [rhs][t][component][site], and a PAIR workgroup
// takes one component of a slab. That halves its registers and its LDS slice
// against complex elements, and its slices are latency-bound otherwise (16^3 x
// 400, 8 rhs, complex: 2 (complex64) or 1 (complex128) workgroups per CU).

// What a PAIR launch does between its two changes.
enum PairEpi {
  kStore = 0,  // forward, first order: z = alpha w stored, sin sigma z goes on
  kFwd = 1,    // forward: sin sigma (alpha w + beta aux) goes on
  kAdj = 2     // adjoint: alpha sin sigma w + beta aux goes on (aux complex)
};

template <typename R>
struct WceArgs {
  R* carry = nullptr;         // [nrhs][nslab][2][V]: in before a slab, out after it; null: none
  R* modes = nullptr;         // [nrhs][ntau][2][V]
  const R* lam = nullptr;     // mode eigenvalues [V]
  int subtract = 0;           // (1 - lam Z)^{-1} - 1 instead of (1 - lam Z)^{-1}
  int adjoint = 0;
  int nrhs = 1;
  int slab = 1;
  const int* gate = nullptr;
  // FIRST: source, or the fused BiCGStab source (PcSource)
  const C2<R>* src = nullptr;
  const C2<R>* fr = nullptr;
  const C2<R>* fp = nullptr;
  const C2<R>* fv = nullptr;
  C2<R>* fpnew = nullptr;
  const void* st = nullptr;
  // PAIR, LAST
  R alpha = R(1), beta = R(0);
  const R* field = nullptr;     // sin sigma
  const R* u0 = nullptr;        // planar auxiliary term
  R* zout = nullptr;            // planar z
  const C2<R>* aux = nullptr;   // complex auxiliary term (kAdj)
  C2<R>* dst = nullptr;         // LAST
};

// Workgroup -> (column of `ncol`, slab): contiguous runs of (slab, column) per
// XCD with the column fastest, so that a slab's field is read through one
// XCD's L2.
__device__ __forceinline__ void wce_item(int ncol, int& c, int& sb) {
  int lid = blockIdx.x;
  const int full = (int)gridDim.x & ~7;
  if (lid < full) lid = (lid & 7) * (full >> 3) + (lid >> 3);
  c = lid % ncol;
  sb = lid / ncol;
}

// U^3T x per slice, and the slab's recurrence from zero. AHEAD: the next slice's
// operands in flight during the transform, for FP64 slices of Nx = 16 only, two
// workgroups of which fill a CU's LDS (16^3 x 400, 8 rhs: 103 -> 87 us; complex64 57 -> 56
// us, Nx = 12 slower by the registers it takes). With a fused source they take 302 and 366
// registers, one workgroup per CU, and still gain where a slab has a next slice: 16^3 x
// 100, 4 rhs (slabs of 2) 38.8 / 41.2 (SRC 1 / 2) -> 32.0 / 28.4 us, 400 slices 128 / 119 -> 127 / 110.
template <typename R, int NX, int SRC, bool AHEAD>
__global__ void __launch_bounds__(NX * NX, sizeof(R) == 8 && NX == 16 && !(SRC && AHEAD) ? 2 : 1)
    wce_first_kernel(WceArgs<R> a, CoefPtr<R, NX> cf, int ntau, int nslab) {
  constexpr int P = NX * NX, V = NX * NX * NX;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  C2<R>* lds = reinterpret_cast<C2<R>*>(smem_raw);
  int r, sb;
  wce_item(a.nrhs, r, sb);
  if (a.gate && a.gate[r] == 0) return;
  const unsigned l = threadIdx.x;
  const int t0 = sb * a.slab, t1 = min(t0 + a.slab, ntau);
  const SrcScal<R> q = src_scalars<R, SRC>(a.st, r);
  constexpr int RS = sizeof(R);
  const auto rl = make_rsrc(a.lam, V * RS);
  C2<R> W[NX];
#pragma unroll
  for (int z = 0; z < NX; ++z) W[z] = zero_of<C2<R>>();
  constexpr int ES = sizeof(C2<R>);
  // element z of a slice at offset o: x, or r, v and, for SRC 1, p
  struct Operands {
    C2<R> x, v, p;
  };
  auto load = [&](long long o, int z) {
    Operands e;
    e.x = bload<R>(make_rsrc((SRC ? a.fr : a.src) + o, V * ES), l * ES, z * P * ES);
    if constexpr (SRC != 0) e.v = bload<R>(make_rsrc(a.fv + o, V * ES), l * ES, z * P * ES);
    if constexpr (SRC == 1) e.p = bload<R>(make_rsrc(a.fp + o, V * ES), l * ES, z * P * ES);
    return e;
  };
  auto form = [&](const Operands& e) {
    if constexpr (SRC == 1) {
      const R dx = e.p.x - (q.wr * e.v.x - q.wi * e.v.y);
      const R dy = e.p.y - (q.wr * e.v.y + q.wi * e.v.x);
      return C2<R>{e.x.x + q.br * dx - q.bi * dy, e.x.y + q.br * dy + q.bi * dx};
    } else if constexpr (SRC == 2) {
      return C2<R>{e.x.x - (q.ar * e.v.x - q.ai * e.v.y), e.x.y - (q.ar * e.v.y + q.ai * e.v.x)};
    } else {
      return e.x;
    }
  };
  auto offset = [&](int k) {
    return ((long long)r * ntau + (a.adjoint ? t1 - 1 - (k - t0) : k)) * V;
  };
  Operands N[AHEAD ? NX : 1];
  if constexpr (AHEAD) {
#pragma unroll
    for (int z = 0; z < NX; ++z) N[z] = load(offset(t0), z);
  }
  for (int k = t0; k < t1; ++k) {
    const long long o = offset(k);
    C2<R> X[NX];
#pragma unroll
    for (int z = 0; z < NX; ++z) X[z] = form(AHEAD ? N[AHEAD ? z : 0] : load(o, z));
    if constexpr (SRC != 0) {
      const auto rn = make_rsrc(a.fpnew + o, V * ES);
#pragma unroll
      for (int z = 0; z < NX; ++z) bstore<R, false>(X[z], a.fpnew + o, rn, l * ES, z * P * ES);
    }
    if constexpr (AHEAD) {
      if (k + 1 < t1) {
#pragma unroll
        for (int z = 0; z < NX; ++z) N[z] = load(offset(k + 1), z);
      }
    }
    slice_T3<R, NX, 1>(cf, lds, l, X);
    const auto rd = make_rsrc(a.modes + 2 * o, 2 * V * RS);
#pragma unroll
    for (int z = 0; z < NX; ++z) {
      const R lam = bload_real<R>(rl, l * RS, z * P * RS);
      W[z] = C2<R>{X[z].x + lam * W[z].x, X[z].y + lam * W[z].y};
    }
#pragma unroll
    for (int z = 0; z < NX; ++z) {
      bstore_real<R>(X[z].x, rd, l * RS, z * P * RS);
      bstore_real<R>(X[z].y, rd, l * RS, (V + z * P) * RS);
    }
  }
  if (!a.carry) return;
  const auto rc = make_rsrc(a.carry + ((long long)r * nslab + sb) * 2 * V, 2 * V * RS);
#pragma unroll
  for (int z = 0; z < NX; ++z) {
    bstore_real<R>(W[z].x, rc, l * RS, z * P * RS);
    bstore_real<R>(W[z].y, rc, l * RS, (V + z * P) * RS);
  }
}

// The recurrence of one component from the slab's carry, U^3, the factors
// between two orders, U^3T, and the next recurrence from zero; in place.
template <typename R, int NX, int EPI>
__global__ void __launch_bounds__(NX * NX)
    wce_pair_kernel(WceArgs<R> a, CoefPtr<R, NX> cb, CoefPtr<R, NX> cf, int ntau, int nslab) {
  constexpr int P = NX * NX, V = NX * NX * NX;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  R* lds = reinterpret_cast<R*>(smem_raw);
  int rc, sb;
  wce_item(2 * a.nrhs, rc, sb);
  const int r = rc >> 1, comp = rc & 1;
  if (a.gate && a.gate[r] == 0) return;
  const unsigned l = threadIdx.x;
  const int t0 = sb * a.slab, t1 = min(t0 + a.slab, ntau);
  constexpr int RS = sizeof(R);
  const int vo = threadIdx.x * RS;
  const auto rl = make_rsrc(a.lam, V * RS);
  const auto rcar = make_rsrc(a.carry + (((long long)r * nslab + sb) * 2 + comp) * V, V * RS);
  R U[NX], W[NX];
#pragma unroll
  for (int z = 0; z < NX; ++z) {
    U[z] = bload_real<R>(rcar, vo, z * P * RS);
    W[z] = R(0);
  }
  for (int k = t0; k < t1; ++k) {
    const int t = a.adjoint ? t1 - 1 - (k - t0) : k;
    const long long o = ((long long)r * ntau + t) * V;
    const long long op = 2 * o + comp * V;  // planar offset
    const auto rm = make_rsrc(a.modes + op, V * RS);
    R X[NX];
#pragma unroll
    for (int z = 0; z < NX; ++z) X[z] = bload_real<R>(rm, vo, z * P * RS);
#pragma unroll
    for (int z = 0; z < NX; ++z) {
      const R d = bload_real<R>(rl, vo, z * P * RS) * U[z];
      U[z] = X[z] + d;
      X[z] = a.subtract ? d : U[z];
    }
    R F[NX], A[EPI != kStore ? NX : 1];
    const auto rf = make_rsrc(a.field + (long long)t * V, V * RS);
#pragma unroll
    for (int z = 0; z < NX; ++z) F[z] = bload_real<R>(rf, vo, z * P * RS);
    if constexpr (EPI == kFwd) {
      const auto ru = make_rsrc(a.u0 + op, V * RS);
#pragma unroll
      for (int z = 0; z < NX; ++z) A[z] = bload_real<R>(ru, vo, z * P * RS);
    } else if constexpr (EPI == kAdj) {
      const auto ru = make_rsrc(reinterpret_cast<const R*>(a.aux + o) + comp, 2 * V * RS);
#pragma unroll
      for (int z = 0; z < NX; ++z) A[z] = bload_real<R>(ru, 2 * vo, 2 * z * P * RS);
    }
    slice_T3<R, NX, 2>(cb, lds, l, X);  // U^3
#pragma unroll
    for (int z = 0; z < NX; ++z) {
      R w = (EPI == kAdj ? a.alpha * F[z] : a.alpha) * X[z];
      if constexpr (EPI != kStore) w += a.beta * A[EPI != kStore ? z : 0];
      X[z] = EPI == kAdj ? w : F[z] * w;
      if constexpr (EPI == kStore) {
        const auto rz = make_rsrc(a.zout + op, V * RS);
        bstore_real<R>(w, rz, vo, z * P * RS);
      }
    }
    slice_T3<R, NX, 1>(cf, lds, l, X);  // U^3T
#pragma unroll
    for (int z = 0; z < NX; ++z) W[z] = X[z] + bload_real<R>(rl, vo, z * P * RS) * W[z];
#pragma unroll
    for (int z = 0; z < NX; ++z) bstore_real<R>(X[z], rm, vo, z * P * RS);
  }
#pragma unroll
  for (int z = 0; z < NX; ++z) bstore_real<R>(W[z], rcar, vo, z * P * RS);
}

// The recurrence from the slab's carry and U^3: y = alpha U^3 u (+ beta u0).
// Without CARRY the modes are u already (order 0 with one slice a slab).
template <typename R, int NX, bool AUX, bool CARRY>
__global__ void __launch_bounds__(NX * NX, sizeof(R) == 8 && NX == 16 ? 2 : 1)
    wce_last_kernel(WceArgs<R> a, CoefPtr<R, NX> cb, int ntau, int nslab) {
  constexpr int P = NX * NX, V = NX * NX * NX;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  C2<R>* lds = reinterpret_cast<C2<R>*>(smem_raw);
  int r, sb;
  wce_item(a.nrhs, r, sb);
  if (a.gate && a.gate[r] == 0) return;
  const unsigned l = threadIdx.x;
  const int t0 = sb * a.slab, t1 = min(t0 + a.slab, ntau);
  constexpr int RS = sizeof(R), ES = sizeof(C2<R>);
  const int vo = threadIdx.x * RS;
  const auto rl = make_rsrc(a.lam, V * RS);
  C2<R> U[CARRY ? NX : 1];
  if constexpr (CARRY) {
    const auto rc = make_rsrc(a.carry + ((long long)r * nslab + sb) * 2 * V, 2 * V * RS);
#pragma unroll
    for (int z = 0; z < NX; ++z)
      U[z] = C2<R>{bload_real<R>(rc, vo, z * P * RS), bload_real<R>(rc, vo, (V + z * P) * RS)};
  }
  auto load = [&](int k, auto& Y) {
    const int t = a.adjoint ? t1 - 1 - (k - t0) : k;
    const auto rm = make_rsrc(a.modes + 2 * ((long long)r * ntau + t) * V, 2 * V * RS);
#pragma unroll
    for (int z = 0; z < NX; ++z)
      Y[z] = C2<R>{bload_real<R>(rm, vo, z * P * RS), bload_real<R>(rm, vo, (V + z * P) * RS)};
  };
  // the next slice in flight as in FIRST (16^3 x 400, 8 rhs complex128: 132 -> 98 us, 16^3
  // x 100, 4 rhs 25.2 -> 19.2); with the auxiliary term no difference (150 us)
  constexpr bool kPre = !AUX && sizeof(R) == 8 && NX == 16;
  C2<R> N[kPre ? NX : 1];
  if constexpr (kPre) load(t0, N);
  for (int k = t0; k < t1; ++k) {
    const int t = a.adjoint ? t1 - 1 - (k - t0) : k;
    const long long o = ((long long)r * ntau + t) * V;
    C2<R> X[NX];
    if constexpr (kPre) {
#pragma unroll
      for (int z = 0; z < NX; ++z) X[z] = N[z];
      if (k + 1 < t1) load(k + 1, N);
    } else {
      load(k, X);
    }
    if constexpr (CARRY) {
#pragma unroll
      for (int z = 0; z < NX; ++z) {
        const R lam = bload_real<R>(rl, vo, z * P * RS);
        const C2<R> d = C2<R>{lam * U[z].x, lam * U[z].y};
        U[z] = C2<R>{X[z].x + d.x, X[z].y + d.y};
        X[z] = a.subtract ? d : U[z];
      }
    }
    slice_T3<R, NX, 2>(cb, lds, l, X);
    C2<R> A[AUX ? NX : 1];
    if constexpr (AUX) {
      const auto ru = make_rsrc(a.u0 + 2 * o, 2 * V * RS);
#pragma unroll
      for (int z = 0; z < NX; ++z)
        A[z] = C2<R>{bload_real<R>(ru, vo, z * P * RS), bload_real<R>(ru, vo, (V + z * P) * RS)};
    }
    const auto rd = make_rsrc(a.dst + o, V * ES);
#pragma unroll
    for (int z = 0; z < NX; ++z) {
      C2<R> w = C2<R>{a.alpha * X[z].x, a.alpha * X[z].y};
      if constexpr (AUX) {
        w.x += a.beta * A[AUX ? z : 0].x;
        w.y += a.beta * A[AUX ? z : 0].y;
      }
      bstore<R, false>(w, a.dst + o, rd, threadIdx.x * ES, z * P * ES);
    }
  }
}

__device__ __forceinline__ double ipow(double x, int n) {
  double r = 1.0;
  for (; n > 0; n >>= 1) {
    if (n & 1) r *= x;
    x *= x;
  }
  return r;
}

// Per (rhs, component, mode): the slab ends g_j (each slab's recurrence from
// zero, in sweep order) become the values before each slab: U_j = g_j +
// lam^len_j U_{j-1}, U_{-1} = -U_last. MODES columns along the lanes x CHUNKS
// chunks of slabs per workgroup; a chunk of up to KEEP slabs stays in registers
// between the two sweeps. Every thread walks all chunk sums by itself (one
// barrier, no serial section of one chunk's threads), from sums that are all
// read at once. FP64 whatever the vector type. Small and bound by its latency:
// a column per (grid.y, lane), no division, buffer loads whose range check does
// for the ends of a chunk (a launch at 12^3 x 200: 6.5 us with 64-bit column
// numbers and addresses, 32 chunks and a loop over their sums; 4.0 us so).
template <typename R, int MODES, int CHUNKS, int KEEP, bool INCLUSIVE>
__global__ void __launch_bounds__(MODES* CHUNKS)
    wce_scan_kernel(R* carry, const double* __restrict__ lam_mode, int V, int ntau, int slab,
                    int nslab, int adjoint, const int* gate) {
  __shared__ double cend[CHUNKS][MODES];
  __shared__ double cpow[CHUNKS][MODES];
  constexpr int RS = sizeof(R);
  const int r = blockIdx.y >> 1, comp = blockIdx.y & 1;
  if (gate && gate[r] == 0) return;
  const int ml = threadIdx.x % MODES, c = threadIdx.x / MODES;
  const int n = blockIdx.x * MODES + ml;
  const bool inb = n < V;
  const int Lc = (nslab + CHUNKS - 1) / CHUNKS;
  const int k0 = c * Lc, k1 = min(k0 + Lc, nslab);
  const int short_k = adjoint ? 0 : nslab - 1;  // sweep position of the slab that may be short
  // out of range (k >= k1, n >= V) is past the end of the buffer: reads zero, stores nothing
  const auto rc = make_rsrc(carry + (long long)r * nslab * 2 * V, nslab * 2 * V * RS);
  const int step = (adjoint ? -2 : 2) * V * RS;
  const int o0 = (((adjoint ? nslab - 1 - k0 : k0) * 2 + comp) * V + n) * RS;
  const int none = nslab * 2 * V * RS;
  auto at = [&](int k) { return inb && k < k1 ? o0 + (k - k0) * step : none; };
  R G[KEEP];
#pragma unroll
  for (int i = 0; i < KEEP; ++i) G[i] = bload_real<R>(rc, at(k0 + i), 0);
  const double lam = inb ? lam_mode[n] : 0.0;
  const double lamS = ipow(lam, slab), lamL = ipow(lam, ntau - (nslab - 1) * slab);
  double pw = 1.0, w = 0.0;
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    if (k0 + i < k1) {
      const double p = k0 + i == short_k ? lamL : lamS;
      w = double(G[i]) + p * w;
      pw *= p;
    }
  }
#pragma unroll 4
  for (int k = k0 + KEEP; k < k1; ++k) {
    const double p = k == short_k ? lamL : lamS;
    w = double(bload_real<R>(rc, at(k), 0)) + p * w;
    pw *= p;
  }
  cend[c][ml] = w;
  cpow[c][ml] = pw;
  __syncthreads();
  // U: the scan over all chunks from zero; v, pv: its value and power before chunk c
  double U = 0.0, v = 0.0, lamN = 1.0, pv = 1.0;
#pragma unroll
  for (int j = 0; j < CHUNKS; ++j) {
    if (j == c) {
      v = U;
      pv = lamN;
    }
    const double p = cpow[j][ml];
    U = cend[j][ml] + p * U;
    lamN *= p;
  }
  v -= pv * U / (1.0 + lamN);  // U_{-1} = -U / (1 + lam^Ntau), carried to chunk c
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    const double p = k0 + i == short_k ? lamL : lamS, u = double(G[i]) + p * v;
    bstore_real<R>(R(INCLUSIVE ? u : v), rc, at(k0 + i), 0);
    v = u;
  }
#pragma unroll 4
  for (int k = k0 + KEEP; k < k1; ++k) {
    const R g = bload_real<R>(rc, at(k), 0);
    const double p = k == short_k ? lamL : lamS, u = double(g) + p * v;
    bstore_real<R>(R(INCLUSIVE ? u : v), rc, at(k), 0);
    v = u;
  }
}

template <typename R, int MODES, int CHUNKS, int KEEP, bool INCLUSIVE>
int launch_scan_shape(const Lattice& L, R* carry, int slab, int nslab, int nrhs, bool adjoint,
                      const int* gate) {
  constexpr int kMost = 32767;  // right-hand sides a launch: grid.y ends at 65535
  for (int r0 = 0; r0 < nrhs; r0 += kMost) {
    hipLaunchKernelGGL((wce_scan_kernel<R, MODES, CHUNKS, KEEP, INCLUSIVE>),
                       dim3((unsigned)((L.V + MODES - 1) / MODES),
                            (unsigned)(2 * std::min(kMost, nrhs - r0))),
                       dim3(MODES * CHUNKS), 0, L.stream, carry + (long long)r0 * nslab * 2 * L.V,
                       L.f64.lam, L.V, L.ntau, slab, nslab, adjoint ? 1 : 0,
                       gate ? gate + r0 : nullptr);
    UFG_HIP(hipGetLastError());
  }
  return UFG_OK;
}

template <bool INCLUSIVE, typename R>
int launch_scan(const Lattice& L, R* carry, int slab, int nslab, int nrhs, bool adjoint,
                const int* gate) {
  // Many columns: wide rows, short chunks. Few: 16 modes a row to have more
  // workgroups, and chunks that fit the registers. Order-2 application, us, with
  // 32 x 8 keeping 8 / 16 x 8 keeping 16 / 16 x 16 keeping 16: 16^3 x 400, 8 rhs (80
  // slabs) complex64 274 / 293 / 285 (32 x 16); 8^3 x 160, 4 rhs (80 slabs) 42.0 / 39.8 /
  // 41.3; 6^3 x 50 (50) 20.9 / 21.1 / 23.4; 12^3 x 200 (200) 65.5 / 58.6 / 53.0.
  if (2ll * L.V * nrhs >= 64 * 256)
    return launch_scan_shape<R, 32, 8, 8, INCLUSIVE>(L, carry, slab, nslab, nrhs, adjoint, gate);
  if (nslab <= 128)
    return launch_scan_shape<R, 16, 8, 16, INCLUSIVE>(L, carry, slab, nslab, nrhs, adjoint, gate);
  return launch_scan_shape<R, 16, 16, 16, INCLUSIVE>(L, carry, slab, nslab, nrhs, adjoint, gate);
}

// The blocks of U^T and U, adjacent on the device.
template <typename R, int NX>
CoefPtr<R, NX> coef_fwd(const Lattice& L) {
  return {reinterpret_cast<const SplitCoef<R, NX>*>(fields<R>(L).modes)};
}
template <typename R, int NX>
CoefPtr<R, NX> coef_bwd(const Lattice& L) {
  return {reinterpret_cast<const SplitCoef<R, NX>*>(fields<R>(L).modes) + 1};
}

// One instantiation per kernel: the LDS attribute is set once.
#define WCE_LAUNCH(KERNEL, ES, GRID, ...)                                                      \
  do {                                                                                         \
    const size_t lds = size_t(lds_slice_elems<NX>()) * (ES);                                   \
    static bool attr = false;                                                                  \
    if (!attr) {                                                                               \
      UFG_HIP(hipFuncSetAttribute((const void*)KERNEL,                                         \
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));      \
      attr = true;                                                                             \
    }                                                                                          \
    hipLaunchKernelGGL(KERNEL, dim3((unsigned)(GRID)), dim3(NX * NX), lds, L.stream,           \
                       __VA_ARGS__, L.ntau, nslab);                                            \
    UFG_HIP(hipGetLastError());                                                                \
    return UFG_OK;                                                                             \
  } while (0)

template <typename R, int NX, int SRC, bool AHEAD>
int launch_first_kernel(const Lattice& L, const WceArgs<R>& a, int nslab) {
  WCE_LAUNCH((wce_first_kernel<R, NX, SRC, AHEAD>), sizeof(C2<R>), nslab * a.nrhs, a,
             (coef_fwd<R, NX>(L)));
}
template <typename R, int NX, int SRC>
int launch_first(const Lattice& L, const WceArgs<R>& a, int nslab) {
  constexpr bool kAhead = sizeof(R) == 8 && NX == 16;
  if constexpr (SRC != 0 && kAhead) {
    if (a.slab == 1) return launch_first_kernel<R, NX, SRC, false>(L, a, nslab);
  }
  return launch_first_kernel<R, NX, SRC, kAhead>(L, a, nslab);
}
template <typename R, int NX, int EPI>
int launch_pair(const Lattice& L, const WceArgs<R>& a, int nslab) {
  WCE_LAUNCH((wce_pair_kernel<R, NX, EPI>), sizeof(R), nslab * a.nrhs * 2, a,
             (coef_bwd<R, NX>(L)), (coef_fwd<R, NX>(L)));
}
template <typename R, int NX, bool AUX, bool CARRY>
int launch_last_kernel(const Lattice& L, const WceArgs<R>& a, int nslab) {
  WCE_LAUNCH((wce_last_kernel<R, NX, AUX, CARRY>), sizeof(C2<R>), nslab * a.nrhs, a,
             (coef_bwd<R, NX>(L)));
}
template <typename R, int NX, bool AUX>
int launch_last(const Lattice& L, const WceArgs<R>& a, int nslab) {
  if constexpr (NX == 16 && !AUX) {  // see wce_direct
    if (!a.carry) return launch_last_kernel<R, NX, AUX, false>(L, a, nslab);
  }
  return launch_last_kernel<R, NX, AUX, true>(L, a, nslab);
}
#undef WCE_LAUNCH

#define WCE_NX(CALL)                                                             \
  switch (L.nx) {                                                                \
    case 6: return CALL(6);                                                      \
    case 8: return CALL(8);                                                      \
    case 10: return CALL(10);                                                    \
    case 12: return CALL(12);                                                    \
    case 14: return CALL(14);                                                    \
    case 16: return CALL(16);                                                    \
    default: set_error("weak-coupling kernels: unsupported nx"); return UFG_EINVAL; \
  }

template <typename R>
int first_change(const Lattice& L, const WceArgs<R>& a, int src_mode, int nslab) {
#define WCE_F(N)                                                       \
  (src_mode == 1   ? launch_first<R, N, 1>(L, a, nslab)                \
   : src_mode == 2 ? launch_first<R, N, 2>(L, a, nslab)                \
                   : launch_first<R, N, 0>(L, a, nslab))
  WCE_NX(WCE_F)
#undef WCE_F
}
template <typename R>
int pair_change(const Lattice& L, const WceArgs<R>& a, int epi, int nslab) {
#define WCE_P(N)                                                       \
  (epi == kStore ? launch_pair<R, N, kStore>(L, a, nslab)              \
   : epi == kFwd ? launch_pair<R, N, kFwd>(L, a, nslab)                \
                 : launch_pair<R, N, kAdj>(L, a, nslab))
  WCE_NX(WCE_P)
#undef WCE_P
}
template <typename R>
int last_change(const Lattice& L, const WceArgs<R>& a, int nslab) {
#define WCE_L(N) (a.u0 ? launch_last<R, N, true>(L, a, nslab) : launch_last<R, N, false>(L, a, nslab))
  WCE_NX(WCE_L)
#undef WCE_L
}

}  // namespace

// With one slice a slab the slab ends are the modes themselves, and at order 0 nothing
// but (1 - lam Z)^{-1} is wanted of them: the scan turns the modes into it in place, and
// FIRST and LAST leave the carry out. Order 0 on 16^3 x 100, 4 rhs complex128: 43 us with
// a carry at one or two slices a slab, 39 so; 60 slices, 8 rhs 47 / 42. For Nx = 16
// only, and complex64 only beyond 512 slices (70 slices, 8 rhs 35 -> 33): where FIRST and
// LAST are short the scan of the modes, whose lines FIRST has just spread over the XCDs'
// L2s, takes longer than that of a carry (16^3 x 100, 4 rhs complex64 8.4 -> 11.6 us).
static bool wce_direct(const Lattice& L, long long n, int order, bool fp64, int slab) {
  return order == 0 && L.nx == 16 && slab == 1 && (fp64 || n > 512);
}

int wce_slab(const Lattice& L, int nrhs, int order, bool fp64, bool fused_source) {
  // the scan addresses one rhs's slab ends by 32-bit byte offsets: keep them below 2 GiB
  const int least = 1 + (int)(((long long)L.ntau * 2 * L.V * 8) >> 30);
  // Not the operator's slab, which is best at 1 there (453 us below): a lattice tuned
  // for M took 462 us instead of 287 for order 2 at 16^3 x 400, 8 rhs complex64.
  if (L.wce_slab > 0) return std::max(least, L.wce_slab);  // at most ntau
  // Longer slabs make the scan cheaper (its traffic is 1 / slab of a pass) and
  // each launch longer (a slab's slices run one after the other); with n slices
  // in all the balance lies near sqrt(n / 128). Order-2 application, us at slab
  // 1 / 2 / 4 / 5 / 8: 16^3 x 400, 8 rhs (n = 3200) complex64 453 / 345 / 293 /
  // 275 / 287, complex128 985 / 726 / 652 / 610 / 636; 12^3 x 200, 8 rhs (1600)
  // complex128 180 / 148 / 144 / 153 / 180; 8^3 x 160, 4 rhs (640) 44 / 40 / 46 /
  // 48 / 64; 16^3 x 400, 1 rhs (400) complex64 89 / 81 / 96 / 108 / 150; 12^3 x
  // 200, 1 rhs (200) complex128 55 / 57 / 83 / 93 / 139.
  const long long n = (long long)L.ntau * nrhs;
  if (wce_direct(L, n, order, fp64, 1) && n <= 600) return least;
  // A FIRST that also forms its source is bound by its traffic, and slabs of two leave
  // CUs without a workgroup below 512 slices. BiCGStab with order 0, us an iteration at slab 1 / 2:
  // FP32-refined 16^3 x 100, 4 rhs 146 / 158, 60 slices, 8 rhs 156 / 171, 12^3 x 100, 4 rhs
  // 104 / 109; FP64 12^3 121 / 128, 10^3 101 / 108, 6^3 64 / 67.
  if (fused_source && order == 0 && n <= 512) return least;
  const int s = std::max(1, std::min(8, (int)std::lround(std::sqrt(n / 128.0))));
  // From 3 on, a neighbour that leaves fewer slices to the CU with most workgroups
  // (256 CUs; a longer slab for Nx of 12 and more only: 8^3 at n = 2400 prefers 4, 72 us,
  // to 5, 76). us at slab 2 / 3 for n = 800: 16^3 complex64 order 0 / 2 39 / 44, 98 /
  // 108, complex128 62 / 71, 177 / 191; 12^3 complex128 order 0 36 / 43; at 4 / 5 for n =
  // 2400, 16^3 complex128 order 2 483 / 449.
  auto most = [&](int k) {
    const long long wg = (long long)((L.ntau + k - 1) / k) * nrhs;
    return (wg + 255) / 256 * k;
  };
  int best = s;
  for (int k : {s - 1, s + 1})
    if (s >= 3 && k <= 8 && (k < s || L.nx >= 12) && most(k) < most(best)) best = k;
  return std::max(least, best);
}

template <typename R>
int wce_modes_apply(Lattice& L, const PcPlan& pc, bool adjoint, const C2<R>* x, C2<R>* y,
                    int nrhs, const int* gate, Counters* cnt, const PcSource<R>* src) {
  const Fields<R>& F = fields<R>(L);
  const int d = pc.order;
  int rc = 0;
  WceArgs<R> a;
  a.modes = reinterpret_cast<R*>(slot_vec<R>(L, SLOT_PC0 + 0, nrhs, &rc));
  UFG_TRY(rc);
  a.slab = wce_slab(L, nrhs, d, sizeof(R) == 8, src != nullptr);
  const bool direct = wce_direct(L, (long long)L.ntau * nrhs, d, sizeof(R) == 8, a.slab);
  if (!direct) {  // one slice per slab: at most a vector
    a.carry = reinterpret_cast<R*>(slot_vec<R>(L, SLOT_PC0 + 1, nrhs, &rc));
    UFG_TRY(rc);
  }
  R* u0 = nullptr;
  if (!adjoint && d > 0) {
    u0 = reinterpret_cast<R*>(slot_vec<R>(L, SLOT_PC0 + 2, nrhs, &rc));
    UFG_TRY(rc);
  }
  a.lam = F.lam;
  a.field = F.sn;
  a.nrhs = nrhs;
  a.adjoint = adjoint ? 1 : 0;
  a.gate = gate;
  const int nslab = (L.ntau + a.slab - 1) / a.slab;
  auto scan = [&]() -> int {
    cnt->m0inv += 1;
    if (direct) return launch_scan<true>(L, a.modes, a.slab, nslab, nrhs, adjoint, gate);
    return launch_scan<false>(L, a.carry, a.slab, nslab, nrhs, adjoint, gate);
  };
  a.src = x;
  if (src) {
    if (src->out != x) {
      set_error("weak-coupling apply: the fused source must be stored to x");
      return UFG_EINVAL;
    }
    a.fr = src->r;
    a.fp = src->p;
    a.fv = src->v;
    a.fpnew = src->out;
    a.st = src->st;
  }
  UFG_TRY(first_change<R>(L, a, src ? src->mode : 0, nslab));
  UFG_TRY(scan());
  a.dst = y;
  a.alpha = R(1);
  if (d == 0) {
    a.alpha = R(pc.w[0]);
    return last_change<R>(L, a, nslab);
  }
  double scale = pc.w[d];
  if (!adjoint) {
    // u_0 = M0^{-1} x, kept for z_m = w_m u_0 + K z_{m+1}; the modes then hold
    // U^3T (sin sigma z_{m+1}) up to `scale`
    a.zout = u0;
    UFG_TRY(pair_change<R>(L, a, kStore, nslab));
    UFG_TRY(scan());
    a.u0 = u0;
    a.subtract = 1;
    for (int m = d - 1; m >= 0; --m) {
      cnt->mv += 1;
      a.alpha = R(L.A * scale);
      a.beta = R(pc.w[m]);
      if (m == 0) break;
      UFG_TRY(pair_change<R>(L, a, kFwd, nslab));
      UFG_TRY(scan());
      scale = 1.0;
    }
    return last_change<R>(L, a, nslab);
  }
  // z_m = w_m x + K' z_{m+1}, K' v = A S U^3 [(1 - lam Z^T)^{-1} - 1] U^3T v; y = M0^{-T} z_0
  a.aux = x;
  a.subtract = 1;
  for (int m = d - 1; m >= 0; --m) {
    cnt->mv += 1;
    a.alpha = R(L.A * scale);
    a.beta = R(pc.w[m]);
    UFG_TRY(pair_change<R>(L, a, kAdj, nslab));
    UFG_TRY(scan());
    scale = 1.0;
  }
  a.alpha = R(1);
  a.subtract = 0;
  return last_change<R>(L, a, nslab);
}

template int wce_modes_apply<float>(Lattice&, const PcPlan&, bool, const float2*, float2*, int,
                                    const int*, Counters*, const PcSource<float>*);
template int wce_modes_apply<double>(Lattice&, const PcPlan&, bool, const double2*, double2*, int,
                                     const int*, Counters*, const PcSource<double>*);

}  // namespace ufg
