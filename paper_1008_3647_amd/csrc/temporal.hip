// Kernels that run along Euclidean time at fixed spatial site or mode:
//   * field setup: 1 + A sin sigma, sin sigma, cos sigma (paper, Sec. 1)
//   * strong-coupling factorisation and its two sweeps (paper, Sec. 4), the time
//     line split into chunks that threads hold in registers
//   * the temporal part of M0^{-1} in the eigenbasis of exp(-tau K)
//     (paper, Sec. 3: M0 is diagonal in frequency-momentum space; per spatial
//     mode the antiperiodic time problem (1 - lam Z) u = v has the closed form
//     u = (1 + lam^Ntau)^{-1} sum_m lam^m Z^m v, evaluated by two sweeps), for the
//     lattices without the block form of U (wce.hip has the others)
// Consecutive threads take consecutive sites so every access along t is a
// coalesced row.
#include <cmath>

#include "slice_t3.h"
#include "ufg_internal.h"

namespace ufg {
namespace {

// `sigma` is copied to `own` on the way (null: it is the library's copy already).
__global__ void field_setup_kernel(const double* __restrict__ sigma, double* own, double A,
                                   long long n, double* b64, double* s64, double* c64, float* b32, float* s32,
                                   double* bmax_part) {
  double m = 0.0;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const double sg = sigma[i];
    if (own) own[i] = sg;
    double s, c;
    sincos(sg, &s, &c);
    const double b = 1.0 + A * s;
    b64[i] = b;
    s64[i] = s;
    c64[i] = c;
    b32[i] = float(b);
    s32[i] = float(s);
    m = fmax(m, fabs(b));
  }
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
  __shared__ double sm[16];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) sm[wid] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) r = fmax(r, sm[w]);
    bmax_part[blockIdx.x] = r;
  }
}

// D_0 = alpha + b_0^2; D_t = alpha + b_t^2 - b_{t-1}^2 / D_{t-1};
// D_{Ntau-1} additionally loses b_{Ntau-1}^2 / D_0 (the antiperiodic corner);
// L_t = b_t / D_t for t < Ntau-1 and L_{Ntau-1} = b_{Ntau-1} / D_0.
// The chain of one FP64 division per slice (0.14 us each) is what bounds one
// thread per site (12^3 x 200: 114 us with a load wait in every step, 28 us with
// the loads ahead of the chain), so a site's time line is split into chunks.
// With D_t = b_t^2 + E_t and q = b_{t-1}^2 a step is the projective map E -> (alpha
// E + (alpha - 1) q) / (E + q), whose terms are all positive for alpha >= 1:
// every chunk multiplies its 2 x 2 matrices (no division, no cancellation), the
// products of the chunks before are applied to (E_0 = alpha, 1), and the
// recursion as printed runs from there. Matrices and vectors are rescaled by
// powers of two by the lower row, which bounds the upper one (E <= alpha) but not the
// other way round (alpha = 1 keeps the upper one at (1, 0) while the lower one is a
// product of all q). Between chunks E is kept at 2^-54 alpha or more, the rounding of
// the recursion's own term q / D: an E that is exact down to 2^-1000 would give factors
// L whose products leave the range of complex64 where b^2 falls below 1 again.
// Against 300 digits over Ntau = 200..4000, alpha = 1..3, tau g = 0.25..40: error no
// larger than the recursion's from D_0 (alpha = 1, Ntau = 200: 3e-13 against 6e-11;
// equal where that is at rounding level or, tau g = 1.1, lost altogether).
// chunks = 1: the recursion as printed from D_0 alone, see launch_sca_setup.
// The last workgroup instead writes the largest of the nblk partial maxima to
// bmax_host (pinned host memory; none when null).
constexpr int kSetupSites = 16, kSetupChunks = 32;
__global__ void __launch_bounds__(kSetupSites* kSetupChunks)
    sca_setup_kernel(const double* __restrict__ b, int V, int ntau, double alpha, int chunks,
                     double* __restrict__ D64, double* __restrict__ L64, float* __restrict__ D32,
                     float* __restrict__ L32, const double* __restrict__ bmax_part, int nblk,
                     double* bmax_host) {
  __shared__ double sm[4][kSetupChunks][kSetupSites];
  if (bmax_host && blockIdx.x == gridDim.x - 1) {
    if (threadIdx.x >= 64) return;
    double m = 0.0;
    for (int i = threadIdx.x; i < nblk; i += 64) m = fmax(m, bmax_part[i]);
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
    if (threadIdx.x == 0) *bmax_host = m;
    return;
  }
  const int ml = threadIdx.x % kSetupSites, c = threadIdx.x / kSetupSites;
  const int n = blockIdx.x * kSetupSites + ml;
  const bool act = n < V;
  const int K = (ntau - 1 + chunks - 1) / chunks;  // steps t = 1 .. ntau - 1
  const int s0 = min(1 + c * K, ntau), s1 = min(s0 + K, ntau);
  auto bat = [&](int t) -> double { return b[(long long)t * V + n]; };
  // exponent that brings v to [1, 2); zero, infinity and NaN stay as they are
  auto scale_of = [](double v) -> int {
    return v > 0.0 && v < HUGE_VAL ? max(-1000, min(1000, -ilogb(v))) : 0;
  };
  double m00 = 1.0, m01 = 0.0, m10 = 0.0, m11 = 1.0;
  const double b0 = act ? bat(0) : 0.0;
  if (act && chunks > 1) {  // (the last chunk too: its b is then near for the recursion)
#pragma unroll 8
    for (int t = s0; t < s1; ++t) {
      const double bp = bat(t - 1), q = bp * bp, f = (alpha - 1.0) * q;
      const double u0 = alpha * m00 + f * m10, u1 = alpha * m01 + f * m11;
      m10 = m00 + q * m10;
      m11 = m01 + q * m11;
      m00 = u0;
      m01 = u1;
      if (((t - s0) & 7) == 7) {
        const int x = scale_of(fmax(m10, m11));
        m00 = ldexp(m00, x);
        m01 = ldexp(m01, x);
        m10 = ldexp(m10, x);
        m11 = ldexp(m11, x);
      }
    }
  }
  sm[0][c][ml] = m00;
  sm[1][c][ml] = m01;
  sm[2][c][ml] = m10;
  sm[3][c][ml] = m11;
  __syncthreads();
  if (!act) return;
  const double D0 = alpha + b0 * b0, least = 0x1p-54 * alpha;
  double v0 = alpha, v1 = 1.0;
  for (int j = 0; j < c; ++j) {
    const double u0 = sm[0][j][ml] * v0 + sm[1][j][ml] * v1;
    const double u1 = sm[2][j][ml] * v0 + sm[3][j][ml] * v1;
    const int x = scale_of(u1);
    v0 = ldexp(u0, x);
    v1 = ldexp(u1, x);
    if (v0 < least) v0 = least;  // v1 is in [1, 2); a NaN stays
  }
  if (c == 0) {
    D64[n] = D0;
    D32[n] = float(D0);
  }
  if (s0 >= s1) return;
  double bp = bat(s0 - 1);
  double Dp = c == 0 ? D0 : bp * bp + v0 / v1;
#pragma unroll 8
  for (int t = s0; t < s1; ++t) {
    const long long i = (long long)t * V + n;
    const double bt = bat(t);
    double D = alpha + bt * bt - bp * bp / Dp;
    if (t == ntau - 1) D -= bt * bt / D0;
    const double Lp = bp / Dp;
    D64[i] = D;
    D32[i] = float(D);
    L64[i - V] = Lp;
    L32[i - V] = float(Lp);
    Dp = D;
    bp = bt;
  }
  if (s1 == ntau) {
    const double Ll = bp / D0;
    L64[(long long)(ntau - 1) * V + n] = Ll;
    L32[(long long)(ntau - 1) * V + n] = float(Ll);
  }
}

// x = L^{-1} D^{-1} L^{dagger -1} v per site. x may alias v.
//   forward : w_0 = v_0, w_t = v_t + L_{t-1} w_{t-1}, w_{Ntau-1} also - L_{Ntau-1} w_0
//   backward: x_{Ntau-1} = w_{Ntau-1} / D, x_t = w_t / D_t + L_t x_{t+1}, x_0 also
//             - L_{Ntau-1} x_{Ntau-1}
// Every factor is real, so a thread owns one real component; a column's time
// line is split into CHUNKS chunks. Each sweep runs a chunk from zero, the
// chunk ends are combined (in FP64) through LDS into the value before each
// chunk, and the chunk runs again from it. KMAX > 0: a chunk of at most KMAX
// slices stays in registers from the load of v to the store of x, one read and
// one write of the vector; KMAX = 0 (longer time lines): the sweeps re-read v
// and x. A single thread per column (the earlier form) was bound by its chain
// of 2 Ntau dependent accesses on few waves.
template <typename R, int LANES, int CHUNKS, int KMAX>
__global__ void __launch_bounds__(LANES* CHUNKS)
    sca_apply_kernel(const R* v, R* x, const R* __restrict__ D, const R* __restrict__ Lb, int V,
                     int ntau, int nrhs, const int* gate) {
  __shared__ double cend[2][CHUNKS][LANES], cpow[2][CHUNKS][LANES];
  __shared__ R xlast[LANES];
  constexpr bool kReg = KMAX > 0;
  constexpr int KA = kReg ? KMAX : 1;
  const int ml = threadIdx.x % LANES, c = threadIdx.x / LANES;
  const long long gid = (long long)blockIdx.x * LANES + ml;
  const bool inb = gid < 2ll * V * nrhs;
  const int r = inb ? int(gid / (2 * V)) : 0;
  const int e = inb ? int(gid - 2ll * V * r) : 0;
  const int n = e >> 1;
  const bool act = inb && !(gate && gate[r] == 0);
  const int K = (ntau + CHUNKS - 1) / CHUNKS;
  const int s0 = min(c * K, ntau), cnt = act ? min(s0 + K, ntau) - s0 : 0;
  const bool first = s0 == 0, last = cnt > 0 && s0 + cnt == ntau;
  // Register path: raw buffer accesses, the thread's byte offset in one VGPR and
  // the slice's in an SGPR (the launcher checks that a vector stays below 4 GiB).
  const long long nv = 2ll * V * ntau * nrhs, nf = (long long)V * ntau;
  const auto bv = make_rsrc(v, (unsigned)(nv * sizeof(R))), bx = make_rsrc(x, (unsigned)(nv * sizeof(R)));
  const auto bl = make_rsrc(Lb, (unsigned)(nf * sizeof(R))), bd = make_rsrc(D, (unsigned)(nf * sizeof(R)));
  const long long v0 = ((long long)r * ntau + s0) * 2 * V + e, f0 = (long long)s0 * V + n;
  const int vo = (int)(unsigned)(v0 * sizeof(R)), fo = (int)(unsigned)(f0 * sizeof(R));
  const int vs = 2 * V * (int)sizeof(R), fs = V * (int)sizeof(R);  // one slice
  auto vin = [&](int i) -> R {
    if constexpr (kReg)
      return bload_real<R>(bv, vo, i * vs);
    else
      return v[v0 + (long long)i * 2 * V];
  };
  auto xin = [&](int i) -> R { return x[v0 + (long long)i * 2 * V]; };
  auto xout = [&](int i, R u) {
    if constexpr (kReg)
      bstore_real<R>(u, bx, vo, i * vs);
    else
      x[v0 + (long long)i * 2 * V] = u;
  };
  // L_{t-1} and L_t of slice s0 + i (0 outside the line), D_t
  auto lprev = [&](int i) -> R { return first && i == 0 ? R(0) : Lb[f0 + (long long)(i - 1) * V]; };
  auto lnext = [&](int i) -> R {
    if (last && i == cnt - 1) return R(0);
    if constexpr (kReg)
      return bload_real<R>(bl, fo, i * fs);
    else
      return Lb[f0 + (long long)i * V];
  };
  auto dval = [&](int i) -> R {
    if constexpr (kReg)
      return bload_real<R>(bd, fo, i * fs);
    else
      return D[f0 + (long long)i * V];
  };
  R w[KA], l[KA + 1], d[KA];
  if constexpr (kReg) {
#pragma unroll
    for (int i = 0; i < KA; ++i)
      if (i < cnt) w[i] = vin(i);
    if (cnt > 0) l[0] = lprev(0);
#pragma unroll
    for (int i = 0; i < KA; ++i)
      if (i < cnt) {
        l[i + 1] = lnext(i);
        d[i] = dval(i);
      }
  }
  const R lc = act && (first || last) ? Lb[(long long)(ntau - 1) * V + n] : R(0);
  const R corner = last ? lc * v[(long long)r * ntau * 2 * V + e] : R(0);  // read before any store of x
  if constexpr (kReg) {
#pragma unroll
    for (int i = 0; i < KA; ++i)
      if (last && i == cnt - 1) w[i] -= corner;
  }
  // element i of the chunk's right-hand side of the forward sweep
  auto rhs = [&](int i) -> R {
    if constexpr (kReg)
      return w[i];
    else
      return last && i == cnt - 1 ? vin(i) - corner : vin(i);
  };
#define SCA_UP(BODY)                                   \
  if constexpr (kReg) {                                \
    _Pragma("unroll") for (int i = 0; i < KA; ++i) {   \
      if (i < cnt) { BODY }                            \
    }                                                  \
  } else {                                             \
    for (int i = 0; i < cnt; ++i) { BODY }             \
  }
#define SCA_DOWN(BODY)                                    \
  if constexpr (kReg) {                                   \
    _Pragma("unroll") for (int i = KA - 1; i >= 0; --i) { \
      if (i < cnt) { BODY }                               \
    }                                                     \
  } else {                                                \
    for (int i = cnt - 1; i >= 0; --i) { BODY }           \
  }
  {
    R g = R(0);
    R p = R(1);
    SCA_UP({
      const R a = kReg ? l[kReg ? i : 0] : lprev(i);
      g = rhs(i) + a * g;
      p *= a;
    })
    cend[0][c][ml] = double(g);
    cpow[0][c][ml] = double(p);
  }
  __syncthreads();
  {
    double U = 0.0;
    for (int j = 0; j < c; ++j) U = cend[0][j][ml] + cpow[0][j][ml] * U;
    R u = R(U);
    SCA_UP({
      const R a = kReg ? l[kReg ? i : 0] : lprev(i);
      u = rhs(i) + a * u;
      const R o = u / (kReg ? d[kReg ? i : 0] : dval(i));
      if constexpr (kReg)
        w[kReg ? i : 0] = o;
      else
        xout(i, o);
      if (last && i == cnt - 1) xlast[ml] = o;
    })
  }
  {
    R g = R(0);
    R p = R(1);
    SCA_DOWN({
      const R b = kReg ? l[kReg ? i + 1 : 0] : lnext(i);
      g = (kReg ? w[kReg ? i : 0] : xin(i)) + b * g;
      p *= b;
    })
    cend[1][c][ml] = double(g);
    cpow[1][c][ml] = double(p);
  }
  __syncthreads();
  {
    double U = 0.0;
    for (int j = CHUNKS - 1; j > c; --j) U = cend[1][j][ml] + cpow[1][j][ml] * U;
    R u = R(U);
    SCA_DOWN({
      const R b = kReg ? l[kReg ? i + 1 : 0] : lnext(i);
      u = (kReg ? w[kReg ? i : 0] : xin(i)) + b * u;
      if (first && i == 0) u -= lc * xlast[ml];
      xout(i, u);
    })
  }
#undef SCA_UP
#undef SCA_DOWN
}

// Per spatial mode n with eigenvalue lam of exp(-tau K):
//   forward : (1 - lam Z) u = v,   (Z w)_t = w_{t-1}, (Z w)_0 = -w_{Ntau-1}
//   adjoint : (1 - lam Z^T) u = v
// Temporal part of M0^{-1} per (rhs, spatial mode): the cyclic first-order
// recurrence u_t = v_t + lam u_{t-1} with the antiperiodic closure
// u_{-1} = -u_{Ntau-1}, split into kChunks time chunks so that 8x more threads
// share the sweep (a thread's chain is Ntau/8 long instead of Ntau):
// workgroup = 64 modes x kChunks chunks (one chunk per wave, modes along the
// lanes). Pass 1: every chunk sweeps its slices from a zero carry (g = last
// value). Then per mode: the chunk carries U_c = g_c + lam^{L_c} U_{c-1} with
// the antiperiodic closure U_{-1} = -U_{last}, i.e. U_last = G / (1 + lam^N)
// where G is the scan from a zero start. Pass 2: every chunk sweeps again from
// its carry. The adjoint runs the same recurrence on reversed time. u may
// alias v (each thread reads and writes only its own chunk).
constexpr int kChunks = 8;
constexpr int kModes = 64;

template <typename R>
__global__ void __launch_bounds__(kModes* kChunks)
    m0_chunked_kernel(const C2<R>* v, C2<R>* u, const R* __restrict__ lam_mode, int V, int ntau,
                      int nrhs, int adjoint, int subtract, const int* gate) {
  __shared__ C2<R> carry[kChunks][kModes];
  const int ml = threadIdx.x % kModes, c = threadIdx.x / kModes;
  const long long gid = (long long)blockIdx.x * kModes + ml;
  const bool inb = gid < (long long)V * nrhs;
  const int r = inb ? int(gid / V) : 0;
  const int n = inb ? int(gid - (long long)r * V) : 0;
  const bool act = inb && !(gate && gate[r] == 0);
  const int Lc = (ntau + kChunks - 1) / kChunks;
  const int s0 = min(c * Lc, ntau), s1 = min(s0 + Lc, ntau);  // chunk [s0, s1) in sweep order
  const long long base = (long long)r * ntau * V + n;
  const R lam = act ? lam_mode[n] : R(0);
  auto at = [&](int k) -> long long {  // sweep position -> element index
    const int t = adjoint ? ntau - 1 - k : k;
    return base + (long long)t * V;
  };
  // pass 1: zero-carry sweep of the chunk
  C2<R> w = C2<R>{R(0), R(0)};
  if (act) {
#pragma unroll 8
    for (int k = s0; k < s1; ++k) {
      const C2<R> q = v[at(k)];
      w = C2<R>{q.x + lam * w.x, q.y + lam * w.y};
    }
  }
  carry[c][ml] = w;
  __syncthreads();
  if (c == 0 && act) {
    R lamL[kChunks];
    R lamN = R(1);
    for (int j = 0; j < kChunks; ++j) {
      const int L = min((j + 1) * Lc, ntau) - min(j * Lc, ntau);
      R p = R(1);
      for (int i = 0; i < L; ++i) p *= lam;
      lamL[j] = p;
      lamN *= p;
    }
    // scan from a zero start: G = carry out of the last chunk
    C2<R> U = C2<R>{R(0), R(0)};
    for (int j = 0; j < kChunks; ++j) {
      const C2<R> g = carry[j][ml];
      U = C2<R>{g.x + lamL[j] * U.x, g.y + lamL[j] * U.y};
    }
    const R inv = R(1) / (R(1) + lamN);
    // carry into chunk 0 is U_{-1} = -U_last
    C2<R> cin = C2<R>{-U.x * inv, -U.y * inv};
    for (int j = 0; j < kChunks; ++j) {
      const C2<R> g = carry[j][ml];
      carry[j][ml] = cin;  // carry into chunk j
      cin = C2<R>{g.x + lamL[j] * cin.x, g.y + lamL[j] * cin.y};
    }
  }
  __syncthreads();
  if (act) {
    C2<R> prev = carry[c][ml];
#pragma unroll 8
    for (int k = s0; k < s1; ++k) {
      // last use of v here, and u is not re-read by this launch
      const long long i = at(k);
      const C2<R> q =
          C2<R>{__builtin_nontemporal_load(&v[i].x), __builtin_nontemporal_load(&v[i].y)};
      prev = C2<R>{q.x + lam * prev.x, q.y + lam * prev.y};
      const C2<R> o = subtract ? C2<R>{prev.x - q.x, prev.y - q.y} : prev;
      __builtin_nontemporal_store(o.x, &u[i].x);
      __builtin_nontemporal_store(o.y, &u[i].y);
    }
  }
}

}  // namespace

int launch_field_setup(Lattice& L, const double* sigma, double* bmax_part, int nblk) {
  hipLaunchKernelGGL(field_setup_kernel, dim3(nblk), dim3(256), 0, L.stream, sigma,
                     sigma == L.sigma ? nullptr : L.sigma, L.A, L.N, L.f64.b, L.f64.sn, L.f64.cs,
                     L.f32.b, L.f32.sn, bmax_part);
  UFG_HIP(hipGetLastError());
  return UFG_OK;
}

int launch_sca_setup(Lattice& L, double alpha, const double* bmax_part, int nblk,
                     double* bmax_host) {
  // In chunks where every term of the maps is positive and eight steps, each growing
  // their entries by at most alpha + b^2, stay within the exponent's range.
  // Otherwise one thread per site runs the recursion as printed: alpha < 1 (terms
  // cancel, errors up to 15 times the recursion's) and magnitudes of no
  // preconditioner in use (alpha above 1e33, or tau g above 75). 12^3 x 200: 10 us in
  // chunks, 41 us so.
  const double bm = 1.0 + std::fabs(L.A);
  const int chunks = alpha >= 1.0 && alpha * (1.0 + bm * bm) < 0x1p110 ? kSetupChunks : 1;
  hipLaunchKernelGGL(sca_setup_kernel, dim3((L.V + kSetupSites - 1) / kSetupSites + (bmax_host ? 1 : 0)),
                     dim3(kSetupSites * kSetupChunks), 0,
                     L.stream, L.f64.b, L.V, L.ntau, alpha, chunks, L.f64.scaD, L.f64.scaL,
                     L.f32.scaD, L.f32.scaL, bmax_part, nblk, bmax_host);
  UFG_HIP(hipGetLastError());
  L.sca_alpha = alpha;
  return UFG_OK;
}

namespace {
template <typename R, int LANES, int CHUNKS, int KMAX>
int launch_sca_shape(const Lattice& L, const C2<R>* v, C2<R>* x, int nrhs, const int* gate) {
  const Fields<R>& F = fields<R>(L);
  const long long n = 2ll * L.V * nrhs;
  hipLaunchKernelGGL((sca_apply_kernel<R, LANES, CHUNKS, KMAX>),
                     dim3((unsigned)((n + LANES - 1) / LANES)), dim3(LANES * CHUNKS), 0, L.stream,
                     reinterpret_cast<const R*>(v), reinterpret_cast<R*>(x), F.scaD, F.scaL, L.V,
                     L.ntau, nrhs, gate);
  UFG_HIP(hipGetLastError());
  return UFG_OK;
}
}  // namespace

template <typename R>
int launch_sca_apply(const Lattice& L, const C2<R>* v, C2<R>* x, int nrhs, const int* gate) {
  const int k32 = (L.ntau + 31) / 32, k16 = (L.ntau + 15) / 16;
  if (sizeof(C2<R>) * (double)L.N * nrhs >= 4294967296.0)  // beyond 32-bit offsets
    return launch_sca_shape<R, 16, 32, 0>(L, v, x, nrhs, gate);
  // 512 threads: 16 columns x 32 chunks, or, for complex64 with enough columns
  // for 1024 workgroups, 32 columns (128-byte rows instead of 64) x 16 chunks:
  // 16^3 x 400, 8 rhs complex64 117 -> 75 us, complex128 143 -> 142 us. One thread
  // a column took 319 / 410 us there and 63 us on 8^3 x 160, 4 rhs complex128 (7.3
  // us now; 16 x 4000, 8 rhs, memory path, 2818 -> 120 us).
  if (sizeof(R) == 4 && 2ll * L.V * nrhs >= 32 * 1024 && k16 <= 32) {
    if (k16 <= 16) return launch_sca_shape<R, 32, 16, 16>(L, v, x, nrhs, gate);
    return launch_sca_shape<R, 32, 16, 32>(L, v, x, nrhs, gate);
  }
  if (k32 <= 8) return launch_sca_shape<R, 16, 32, 8>(L, v, x, nrhs, gate);
  if (k32 <= 16) return launch_sca_shape<R, 16, 32, 16>(L, v, x, nrhs, gate);
  if (k32 <= 32) return launch_sca_shape<R, 16, 32, 32>(L, v, x, nrhs, gate);
  return launch_sca_shape<R, 16, 32, 0>(L, v, x, nrhs, gate);
}

template <typename R>
int launch_m0_temporal(const Lattice& L, const C2<R>* v, C2<R>* u, int nrhs, bool adjoint,
                       bool subtract_input, const int* gate) {
  const Fields<R>& F = fields<R>(L);
  const long long n = (long long)L.V * nrhs;
  hipLaunchKernelGGL((m0_chunked_kernel<R>), dim3((unsigned)((n + kModes - 1) / kModes)),
                     dim3(kModes * kChunks), 0, L.stream, v, u, F.lam, L.V, L.ntau, nrhs,
                     adjoint ? 1 : 0, subtract_input ? 1 : 0, gate);
  UFG_HIP(hipGetLastError());
  return UFG_OK;
}

template int launch_sca_apply<float>(const Lattice&, const float2*, float2*, int, const int*);
template int launch_sca_apply<double>(const Lattice&, const double2*, double2*, int, const int*);
template int launch_m0_temporal<float>(const Lattice&, const float2*, float2*, int, bool, bool,
                                       const int*);
template int launch_m0_temporal<double>(const Lattice&, const double2*, double2*, int, bool, bool,
                                        const int*);

}  // namespace ufg
