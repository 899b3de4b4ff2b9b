// Streaming slice operator for M and M^T (paper, Sec. 1, Eq. MatrixM) on gfx950.
//
// One workgroup owns a slab of S consecutive time slices of one right-hand
// side and walks it in the direction that reuses loads: upwards for M (output
// t reads source t-1), downwards for M^T (output t reads source t+1). The
// slice loaded for the identity term of output t is the source of the next
// output, so every input slice of the slab is loaded once; only one halo
// slice per slab is loaded twice (at two slices per slab the L2 misses come to
// about 1.2 times the algorithmic bytes).
//
// Workgroup numbering (see stream_item): by default consecutive slabs are
// gathered into groups of G that go round-robin to the eight XCDs, and each
// XCD walks its groups right-hand side by right-hand side. Every rhs of a slab
// then runs on the same XCD (the field slab is read from HBM once), the halo
// slice of a slab is the last slice of the previous slab on the same XCD
// (except at group edges), and the workgroups resident at any moment cover one
// contiguous address window of each vector. The earlier numbering, contiguous
// runs of (slab, rhs) pairs per XCD with the rhs fastest (G = 0), spreads the
// resident workgroups over the eight rhs blocks of every vector.
//
// exp(-tau K) along one axis is the symmetric circulant T. T commutes with the
// reflections i -> -i and i -> Nx/2 - i (mod Nx), so in the basis of their
// joint eigenvectors (built by two levels of add/subtract butterflies) T is
// block diagonal with four blocks of about Nx/4 (SplitSize). A line of Nx values
// then costs about 4 Nx additions for the butterflies and sum(block^2)
// multiply-adds (56 + 66 for Nx = 16) instead of Nx^2 = 256 multiply-adds.
//
// Memory access: raw buffer instructions with one resource per array (base =
// the rhs block), the lane offset in a VGPR and the slice / z offset in an
// SGPR, so a z-line costs no 64-bit address arithmetic. The operands of an
// output slice (field, aux, reduction weights) are loaded before its stores
// start, because loads cannot be moved across buffer stores.
//
// Fused BiCGStab sources: the kernel can build its source on the fly from the
// Krylov vectors (p = r + beta (p_old - omega v_old), or s = r - alpha v) so
// that BiCGStab's vector updates ride on the operator's memory stream, and
// reduce FP64 dot products of its output, its source and a weight vector into
// one partial per workgroup.
#include "hop_stream.h"
#include "krylov.h"
#include "krylov_fin.h"
#include "slice_t3.h"

namespace ufg {
namespace {
using namespace splitk;

// The y and x stages of T^3 as 16x16x4 FP32 MFMA contractions (Nx = 16,
// complex64; lattice_tune_transform route 1). A wave owns z-planes 4w..4w+3,
// as in the VALU stages. For one plane and axis, the lines of the plane form
// the 16 columns of B and T the 16x16 A operand: lane holds
// ta[s] = T[lane % 16][4 s + lane / 16] for k-block s, and B[k][c] = the
// plane's element k of line c (real and imaginary parts separately); the
// product lands as D[4 (lane / 16) + j][lane % 16], element 4 (lane / 16) + j
// of line lane % 16. AX = 1: lines along y (c = x); AX = 0: along x (c = y).
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int AX>
__device__ __forceinline__ void stage_mfma16(const float (&ta)[4], float2* lds, int l) {
  constexpr int NX = 16;
  const int w = l >> 6, lane = l & 63, g = lane >> 4, cc = lane & 15;
#pragma unroll
  for (int zz = 0; zz < 4; ++zz) {
    const int z = 4 * w + zz;
    f32x4 dre = {0.f, 0.f, 0.f, 0.f}, dim = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = 4 * s + g;
      const float2 v = AX == 0 ? lds[lds_at<NX>(z * NX + cc, k)] : lds[lds_at<NX>(z * NX + k, cc)];
      dre = __builtin_amdgcn_mfma_f32_16x16x4f32(ta[s], v.x, dre, 0, 0, 0);
      dim = __builtin_amdgcn_mfma_f32_16x16x4f32(ta[s], v.y, dim, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int o = 4 * g + j;
      const float2 r = make_float2(dre[j], dim[j]);
      if (AX == 0)
        lds[lds_at<NX>(z * NX + cc, o)] = r;
      else
        lds[lds_at<NX>(z * NX + o, cc)] = r;
    }
  }
}

// slice_T3 with the y and x stages on MFMA (z stays on the VALU, in registers);
// the result stays in LDS as for slice_T3<..., KEEP = true>.
__device__ __forceinline__ void slice_T3_mfma16(const SplitCoef<float, 16>& c,
                                                const float (&ta)[4], float2* lds, int l,
                                                float2 (&v)[16]) {
  constexpr int NX = 16;
  const int y = l / NX, x = l - (l / NX) * NX;
  split_line<float, NX>(c, v);  // along z
#pragma unroll
  for (int z = 0; z < NX; ++z) lds[lds_at<NX>(z * NX + y, x)] = v[z];
  __syncthreads();
  stage_mfma16<1>(ta, lds, l);  // along y: planes of this wave only
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  stage_mfma16<0>(ta, lds, l);  // along x
  __syncthreads();
}

// T^3 through Fourier transforms (complex64, Nx = 16; lattice_tune_transform
// route 2): T is a symmetric circulant, so along each axis T = F^-1 diag(lam) F
// with F the 16-point DFT and lam_k = sum_j T_0j cos(2 pi j k / 16). Each
// stage is a forward DFT of the line, the scaling by lam_k / 16 and an
// inverse DFT, the DFT in radix 4 x 4 (index n = 4 n1 + n2, k = k1 + 4 k2:
// 4-point DFTs over n1, twiddles W^(n2 k1), 4-point DFTs over n2).
template <int M, bool INV>
__device__ __forceinline__ float2 twiddle16(float2 a) {
  // a * exp(-+2 pi i M / 16) (INV: +)
  constexpr float c1 = 0.92387953251128674f, s1 = 0.38268343236508978f,
                  r2 = 0.70710678118654752f;
  constexpr float cs[10] = {1.f, c1, r2, s1, 0.f, -s1, -r2, -c1, -1.f, -c1};
  constexpr float sn[10] = {0.f, s1, r2, c1, 1.f, c1, r2, s1, 0.f, -s1};
  if constexpr (M == 0) {
    return a;
  } else if constexpr (M == 4) {  // -i (forward) or +i (inverse)
    return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
  } else if constexpr (M == 8) {
    return make_float2(-a.x, -a.y);
  } else {
    const float c = cs[M], sg = INV ? sn[M] : -sn[M];
    return make_float2(a.x * c - a.y * sg, a.x * sg + a.y * c);
  }
}

template <bool INV>
__device__ __forceinline__ void dft4(float2& a0, float2& a1, float2& a2, float2& a3) {
  const float2 t0 = make_float2(a0.x + a2.x, a0.y + a2.y);
  const float2 t1 = make_float2(a0.x - a2.x, a0.y - a2.y);
  const float2 t2 = make_float2(a1.x + a3.x, a1.y + a3.y);
  const float2 t3 = make_float2(a1.x - a3.x, a1.y - a3.y);
  a0 = make_float2(t0.x + t2.x, t0.y + t2.y);
  a2 = make_float2(t0.x - t2.x, t0.y - t2.y);
  // forward: A1 = t1 - i t3, A3 = t1 + i t3 (inverse: the other way round)
  const float2 m = make_float2(t1.x + t3.y, t1.y - t3.x);
  const float2 p = make_float2(t1.x - t3.y, t1.y + t3.x);
  a1 = INV ? p : m;
  a3 = INV ? m : p;
}

template <bool INV>
__device__ __forceinline__ void dft16(float2 (&v)[16]) {
  float2 y[16];  // y[4 n2 + k1]
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
    float2 a0 = v[n2], a1 = v[4 + n2], a2 = v[8 + n2], a3 = v[12 + n2];
    dft4<INV>(a0, a1, a2, a3);
    y[4 * n2 + 0] = a0;
    y[4 * n2 + 1] = a1;
    y[4 * n2 + 2] = a2;
    y[4 * n2 + 3] = a3;
  }
  y[5] = twiddle16<1, INV>(y[5]);
  y[6] = twiddle16<2, INV>(y[6]);
  y[7] = twiddle16<3, INV>(y[7]);
  y[9] = twiddle16<2, INV>(y[9]);
  y[10] = twiddle16<4, INV>(y[10]);
  y[11] = twiddle16<6, INV>(y[11]);
  y[13] = twiddle16<3, INV>(y[13]);
  y[14] = twiddle16<6, INV>(y[14]);
  y[15] = twiddle16<9, INV>(y[15]);
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    float2 a0 = y[k1], a1 = y[4 + k1], a2 = y[8 + k1], a3 = y[12 + k1];
    dft4<INV>(a0, a1, a2, a3);
    v[k1] = a0;
    v[k1 + 4] = a1;
    v[k1 + 8] = a2;
    v[k1 + 12] = a3;
  }
}

__device__ __forceinline__ void fft_line16(const float (&lam)[16], float2 (&v)[16]) {
  dft16<false>(v);
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    v[k].x *= lam[k];
    v[k].y *= lam[k];
  }
  dft16<true>(v);
}

// lam_k / 16 from the first row of T (row-major Nx x Nx on the device).
__device__ __forceinline__ void fft_lambda16(const float* __restrict__ T, float (&lam)[16]) {
  constexpr float c1 = 0.92387953251128674f, s1 = 0.38268343236508978f,
                  r2 = 0.70710678118654752f;
  constexpr float cs[16] = {1.f, c1, r2, s1, 0.f, -s1, -r2, -c1,
                            -1.f, -c1, -r2, -s1, 0.f, s1, r2, c1};
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < 16; ++j) acc = fmaf(T[j], cs[(j * k) & 15], acc);
    lam[k] = acc * (1.f / 16.f);
  }
}

// slice_T3<float, 16, 0, true> with each line through fft_line16.
__device__ __forceinline__ void slice_T3_fft16(const float (&lam)[16], float2* lds, int l,
                                               float2 (&v)[16]) {
  constexpr int NX = 16;
  const int y = l / NX, x = l - (l / NX) * NX;
  fft_line16(lam, v);  // along z
#pragma unroll
  for (int z = 0; z < NX; ++z) lds[lds_at<NX>(z * NX + y, x)] = v[z];
  __syncthreads();
  float2 w[NX];
  {
    const int z = l / NX, xx = l - (l / NX) * NX;
#pragma unroll
    for (int yy = 0; yy < NX; ++yy) w[yy] = lds[lds_at<NX>(z * NX + yy, xx)];
    fft_line16(lam, w);  // along y
#pragma unroll
    for (int yy = 0; yy < NX; ++yy) lds[lds_at<NX>(z * NX + yy, xx)] = w[yy];
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  {
    const int z = l / NX, yy = l - (l / NX) * NX;
#pragma unroll
    for (int xx = 0; xx < NX; ++xx) w[xx] = lds[lds_at<NX>(z * NX + yy, xx)];
    fft_line16(lam, w);  // along x
#pragma unroll
    for (int xx = 0; xx < NX; ++xx) lds[lds_at<NX>(z * NX + yy, xx)] = w[xx];
  }
  __syncthreads();
}

struct Rsrc {
  __amdgpu_buffer_rsrc_t src, fr, fp, fv, fpnew, dst, aux, rw, pre, post;
};

// z-line of the source slice at byte offset so (uniform); vo = lane byte offset.
// AUX: cache policy of the loads (kAuxNT for slices that no other workgroup reads).
template <typename R, int NX, int SRC, int AUX>
__device__ __forceinline__ void load_source(const Rsrc& b, const SrcScal<R>& q, int so, int vo,
                                            C2<R> (&X)[NX]) {
  constexpr int ZB = NX * NX * (int)sizeof(C2<R>);
#pragma unroll
  for (int z = 0; z < NX; ++z) {
    const int s = so + z * ZB;
    if (SRC == 0) {
      X[z] = bload<R, AUX>(b.src, vo, s);
    } else if (SRC == 1) {
      const C2<R> rv = bload<R, AUX>(b.fr, vo, s), pv = bload<R, AUX>(b.fp, vo, s),
                  vv = bload<R, AUX>(b.fv, vo, s);
      const R dx = pv.x - (q.wr * vv.x - q.wi * vv.y);
      const R dy = pv.y - (q.wr * vv.y + q.wi * vv.x);
      X[z].x = rv.x + q.br * dx - q.bi * dy;
      X[z].y = rv.y + q.br * dy + q.bi * dx;
    } else {
      const C2<R> rv = bload<R, AUX>(b.fr, vo, s), vv = bload<R, AUX>(b.fv, vo, s);
      X[z].x = rv.x - (q.ar * vv.x - q.ai * vv.y);
      X[z].y = rv.y - (q.ar * vv.y + q.ai * vv.x);
    }
  }
}

// z-line of a real field slice times X (in place).
template <typename R, int NX>
__device__ __forceinline__ void scale_field(__amdgpu_buffer_rsrc_t f, int so, int vo,
                                            C2<R> (&X)[NX]) {
  constexpr int ZB = NX * NX * (int)sizeof(R);
#pragma unroll
  for (int z = 0; z < NX; ++z) {
    const R fz = bload_real<R>(f, vo, so + z * ZB);
    X[z].x *= fz;
    X[z].y *= fz;
  }
}

// Block -> (rhs r, slab sb); false if the block has no item (it exits).
// xg = 0: contiguous runs of (slab, rhs) per XCD, rhs fastest (grid nslab*nrhs).
// xg > 0: slab groups of xg go round-robin to the XCDs (blocks are dispatched
// to XCD blockIdx % 8); the q-th block of XCD j takes item q of the list
// "for r: for the slabs of XCD j's groups" (ri = 0) or "for XCD j's groups:
// for r: for the group's slabs" (ri = 1); grid stream_grid().
__device__ __forceinline__ bool stream_item(int nslab, int nrhs, int xg, int ri, int& r,
                                            int& sb) {
  const int b = blockIdx.x;
  if (xg <= 0) {
    const int full = (int)gridDim.x & ~7;
    int lid = b;
    if (lid < full) lid = (lid & 7) * (full >> 3) + (lid >> 3);
    r = lid % nrhs;
    sb = lid / nrhs;
    return true;
  }
  const int j = b & 7, q = b >> 3;
  if (ri) {
    const int per = nrhs * xg;  // blocks per group
    const int m = q / per, k = q - m * per;
    r = k / xg;
    sb = (8 * m + j) * xg + (k - r * xg);
    return sb < nslab;
  }
  const int F = nslab / xg, rem = nslab - F * xg;  // full groups, slabs of the partial one
  int nj = xg * (F / 8 + ((j < (F & 7)) ? 1 : 0));
  if (rem > 0 && (F & 7) == j) nj += rem;
  if (q >= nrhs * nj) return false;
  r = q / nj;
  const int k = q - r * nj;
  sb = (k / xg) * 8 * xg + j * xg + (k % xg);
  return true;
}

__device__ __forceinline__ double wsum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// DIR = -1: M-type, output t reads source t-1; the slab is walked upwards.
// DIR = +1: M^T-type, output t reads source t+1; the slab is walked downwards.
// Either way the slice loaded for the identity term of output t is the source
// of the next output: each thread holds one z-line X (current source) in
// registers, and the transform of the previous source stays in the LDS slice,
// from which the output phase reads the thread's own z-line.
// TR = 1: the transform's y and x stages on MFMA (complex64, Nx = 16, plain
// operator only; see slice_T3_mfma16); TR = 2: every stage through 16-point
// DFTs (same restriction; see slice_T3_fft16).
// Waves per SIMD the compiler may aim at.
// Three for the complex64 Nx = 16 M^T with scaling and auxiliary term: aiming at the
// four that its LDS slice allows, the compiler spills (123 VGPRs and scratch; a degree-8
// Chebyshev application on 16^3 x 217, 5 rhs 347 -> 367 us).
// Two for the complex128 Nx = 16 operators that form their source while loading: the 68 KB
// slice admits two workgroups a CU, and registers saved for a third wave only put the
// loads of a slice one behind the other. t = A s on 16^3 x 400, 8 rhs, M / M^T: 146 and 166
// VGPRs 206.5 / 204.4 us, 182 and 185 VGPRs 195.6 / 192.6, the FP64 solve 2.697 ->
// 2.642 s; an iteration on 16^3 x 64, 1 rhs 45.3 / 48.3 -> 42.4 / 45.1 us. The plain source
// has no such gain (v = A p 124.4 / 122.3 -> 125.7 / 122.9).
template <typename R, int NX, int DIR, bool GENERAL, int SRC>
constexpr int hop_max_waves() {
  if (NX == 16 && sizeof(R) == 8 && SRC != 0) return 2;
  return sizeof(R) == 4 && NX == 16 && DIR > 0 && GENERAL ? 3 : 8;
}

template <typename R, int NX, int DIR, bool GENERAL, int SRC, int RED, int TR = 0>
__global__ void __launch_bounds__(NX * NX)
    __attribute__((amdgpu_waves_per_eu(1, hop_max_waves<R, NX, DIR, GENERAL, SRC>())))
    hop_stream_kernel(HopArgs<R> a, SplitCoef<R, NX> c, int ntau, int nslab, int xg, int ri) {
  static_assert(TR == 0 || (sizeof(R) == 4 && NX == 16 && SRC == 0 && RED == 0 && !GENERAL),
                "the MFMA and DFT transform routes exist for the plain complex64 Nx = 16 "
                "operator");
  constexpr int P = NX * NX, V = NX * NX * NX;
  constexpr int ES = sizeof(C2<R>), FS = sizeof(R);
  // Single-use operand slices are loaded non-temporal (measured: faster for
  // every complex64 variant and the fused complex128 ones, slower for the
  // plain complex128 operator, which keeps the default policy).
  constexpr int kNTA = (sizeof(R) == 4 || SRC != 0 || RED != 0) ? kAuxNT : 0;
  // plain operator: the first output slice's source (and, for M^T, its field) is
  // loaded together with the halo, before the halo's transform (one more z-line
  // of registers; the fused variants would lose a wave per SIMD to it).
  // complex128 up to Nx = 10, M^T also at Nx = 12: 8^3 x 400, 8 rhs 10.2 / 10.7 (M / M^T)
  // -> 9.7 / 9.6 us, 12^3 x 400, 8 rhs M^T 41.9 -> 40.2 but M 41.5 -> 43.6.
  constexpr bool EARLY = (sizeof(R) == 4 || NX <= 10 || (NX == 12 && DIR > 0)) && SRC == 0 && RED == 0 && !GENERAL;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  C2<R>* lds = reinterpret_cast<C2<R>*>(smem_raw);

  int r, sb;
  if (!stream_item(nslab, a.nrhs, xg, ri, r, sb)) return;
  // M^T walks time downwards: with slab groups the XCD takes its slabs in
  // decreasing order, so a slab's halo (the next slab) was loaded first
  if (DIR > 0 && xg > 0) sb = nslab - 1 - sb;
  if (a.gate && a.gate[r] == 0) return;
  constexpr bool kCoefLds = sizeof(R) == 8 && DIR < 0 && (SRC != 0 || RED != 0);
  __shared__ CoefSlot<kCoefLds, R, NX> coef_lds[1];
  const SplitCoef<R, NX>& cc = *coef_copy<kCoefLds, R, NX>(c, coef_lds);

  const int l = threadIdx.x;
  float ta[TR == 1 ? 4 : 1];
  if constexpr (TR == 1) {
    const int lane = l & 63;
#pragma unroll
    for (int j = 0; j < 4; ++j) ta[j] = float(a.mat[(lane & 15) * NX + 4 * j + (lane >> 4)]);
  }
  float lam[TR == 2 ? 16 : 1];
  if constexpr (TR == 2) fft_lambda16(a.mat, lam);
  const int t0 = (int)((long long)sb * ntau / nslab);
  const int t1 = (int)((long long)(sb + 1) * ntau / nslab);  // exclusive
  const long long rbase = (long long)r * ntau * V;
  const unsigned vbytes = (unsigned)ntau * V * ES;
  const unsigned fbytes = (unsigned)ntau * V * FS;
  Rsrc b;
  b.src = make_rsrc(a.src + rbase, vbytes);
  b.fr = make_rsrc(a.fr + rbase, vbytes);
  b.fp = make_rsrc(a.fp + rbase, vbytes);
  b.fv = make_rsrc(a.fv + rbase, vbytes);
  b.fpnew = make_rsrc(a.fpnew + rbase, vbytes);
  b.dst = make_rsrc(a.dst + rbase, vbytes);
  b.aux = make_rsrc(a.aux + rbase, vbytes);
  b.rw = make_rsrc(a.red_w + rbase, vbytes);
  b.pre = make_rsrc(a.pre, fbytes);
  b.post = make_rsrc(a.post, fbytes);
  const int vo = l * ES, fo = l * FS;
  SrcScal<R> q = src_scalars<R, SRC>(a.st, r);
  if constexpr (SRC == 2 && RED == 4) {
    if (a.fin_part) {  // the alpha step of the rhs state, see HopArgs
      // thread 0 fetches the state and flags while every thread sums partials
      RhsState* st = reinterpret_cast<RhsState*>(const_cast<void*>(a.st));
      int* fl = a.fin_flags;
      RhsState qs{};
      int act = 0, upd = 0, rst = 0;
      if (l == 0) {
        qs = st[r];
        act = fl[r];
        upd = fl[a.nrhs + r];
        rst = fl[2 * a.nrhs + r];
      }
      double v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = 0.0;
      for (int bi = l; bi < a.fin_nblk; bi += P) {
        const double* pp = a.fin_part + ((long long)r * a.fin_nblk + bi) * 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] += pp[j];
      }
      for (int bi = l; bi < a.fin_nblk2; bi += P) {
        const double* pp = a.fin_part2 + ((long long)r * a.fin_nblk2 + bi) * 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[4 + j] += pp[j];
      }
      constexpr int NW = (P + 63) / 64;
      double* sm = reinterpret_cast<double*>(smem_raw);
      const int lane = l & 63, wid = l >> 6;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const double w = wsum(v[j]);
        if (lane == 0) sm[wid * 8 + j] = w;
      }
      __syncthreads();
      if (l == 0) {
        double s8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int w = 0; w < NW; ++w)
#pragma unroll
          for (int j = 0; j < 8; ++j) s8[j] += sm[w * 8 + j];
        apply_fin(FIN_ALPHA_XR, s8, qs, act, upd, rst, a.fin_prm);
        if (sb == 0) {
          st[r] = qs;
          fl[r] = act;
          fl[a.nrhs + r] = upd;
          fl[2 * a.nrhs + r] = rst;
        }
        sm[NW * 8] = qs.alpha.x;
        sm[NW * 8 + 1] = qs.alpha.y;
        sm[NW * 8 + 2] = act ? 1.0 : 0.0;
      }
      __syncthreads();
      const double alx = sm[NW * 8], aly = sm[NW * 8 + 1];
      const bool live = sm[NW * 8 + 2] != 0.0;
      __syncthreads();  // the LDS slice is written next
      if (!live) return;
      q.ar = R(alx);
      q.ai = R(aly);
    }
  }
  const int count = t1 - t0;
  // first output slice, step, and the halo slice that feeds it
  const int tfirst = (DIR < 0) ? t0 : t1 - 1;
  const int step = (DIR < 0) ? 1 : -1;
  const int th = (DIR < 0) ? ((t0 == 0) ? ntau - 1 : t0 - 1) : ((t1 == ntau) ? 0 : t1);

  double acc0 = 0, acc1 = 0, acc2 = 0, acc3 = 0, acc4 = 0, acc5 = 0, acc6 = 0, acc7 = 0;
  // X: the z-line of the current source slice. The T^3 of the previous one
  // stays in the LDS slice (each thread reads back only its own z-line, which
  // is also the first thing it writes in the next transform).
  C2<R> X[NX];
  C2<R> Y[EARLY ? NX : 1];
  const int ly = l / NX, lx = l - (l / NX) * NX;
  load_source<R, NX, SRC, 0>(b, q, th * V * ES, vo, X);
  R F0[EARLY && DIR > 0 ? NX : 1];
  if constexpr (EARLY) {
    if (count > 1)
      load_source<R, NX, SRC, kNTA>(b, q, tfirst * V * ES, vo, Y);
    else
      load_source<R, NX, SRC, 0>(b, q, tfirst * V * ES, vo, Y);
    if constexpr (DIR > 0) {  // and its output field
#pragma unroll
      for (int z = 0; z < NX; ++z)
        F0[z] = bload_real<R>(b.post, fo, tfirst * V * FS + z * P * FS);
    }
  }
  // plain complex64 operator: once its loads are issued, the workgroup runs
  // the transform and the output at raised wave priority, so that the
  // workgroups started earlier finish (and free their slots) first (measured:
  // apply_Mdag 45.9 -> 43.6 us, apply_M unchanged; the fused and complex128
  // variants ran slower that way)
  if constexpr (EARLY && sizeof(R) == 4) __builtin_amdgcn_s_setprio(2);
  if (DIR < 0) scale_field<R, NX>(b.pre, th * V * FS, fo, X);
  if constexpr (TR == 1)
    slice_T3_mfma16(cc, ta, lds, l, X);
  else if constexpr (TR == 2)
    slice_T3_fft16(lam, lds, l, X);
  else
    slice_T3<R, NX, 0, true>(cc, lds, l, X);
  for (int k = 0; k < count; ++k) {
    const int t = tfirst + k * step;
    const int so = t * V * ES;  // slice byte offset (uniform)
    // the last slice of the slab is the halo of the neighbouring slab: it
    // stays cacheable, the others are streamed
    bool have = false;
    if constexpr (EARLY) {
      if (k == 0) {
#pragma unroll
        for (int z = 0; z < NX; ++z) X[z] = Y[z];
        have = true;
      }
    }
    if (!have) {
      if (k + 1 < count)
        load_source<R, NX, SRC, kNTA>(b, q, so, vo, X);
      else
        load_source<R, NX, SRC, 0>(b, q, so, vo, X);
    }
    if (SRC == 1) {
#pragma unroll
      for (int z = 0; z < NX; ++z) bstore<R, false>(X[z], a.fpnew + rbase, b.fpnew, vo, so + z * P * ES);
    }
    // sign of the block that connects the source slice to slice t
    R sgn;
    if (DIR < 0)
      sgn = (t == 0) ? R(1) : R(-1);
    else
      sgn = (t == ntau - 1) ? R(1) : R(-1);
    // The output slice is written in chunks of ZC z-planes; the operands of a
    // chunk (field, aux, reduction weights) are loaded ahead of its stores
    // (loads cannot be moved across buffer stores). complex128 with a
    // reduction uses half-slice chunks to stay within the register file.
    constexpr int ZC = (sizeof(R) == 8 && (GENERAL || RED != 0)) ? NX / 2 : NX;
#pragma unroll
    for (int z0 = 0; z0 < NX; z0 += ZC) {
      R F[DIR > 0 ? ZC : 1];
      if (DIR > 0) {  // M^T-type: the field multiplies the output slice
        if (EARLY && k == 0) {
#pragma unroll
          for (int j = 0; j < ZC; ++j) F[j] = sgn * F0[EARLY && DIR > 0 ? z0 + j : 0];
        } else {
#pragma unroll
          for (int j = 0; j < ZC; ++j)
            F[j] = sgn * bload_real<R>(b.post, fo, t * V * FS + (z0 + j) * P * FS);
        }
      }
      C2<R> U[GENERAL ? ZC : 1];
      if (GENERAL && a.aux) {
#pragma unroll
        for (int j = 0; j < ZC; ++j) U[j] = bload<R, kNTA>(b.aux, vo, so + (z0 + j) * P * ES);
      }
      C2<R> Wr[(RED == 1 || RED == 2 || RED == 4) ? ZC : 1];
      if (RED == 1 || RED == 2 || RED == 4) {
#pragma unroll
        for (int j = 0; j < ZC; ++j) Wr[j] = bload<R, kNTA>(b.rw, vo, so + (z0 + j) * P * ES);
      }
#pragma unroll
      for (int j = 0; j < ZC; ++j) {
        const int z = z0 + j;
        const int s = so + z * P * ES;
        const C2<R> id = X[z];
        const C2<R> wz = lds[lds_at<NX>(z * NX + ly, lx)];
        C2<R> base;
        const R f = (DIR > 0) ? F[DIR > 0 ? j : 0] : sgn;
        base.x = f * wz.x;
        base.y = f * wz.y;
        if (a.id) {
          base.x += id.x;
          base.y += id.y;
        }
        C2<R> out = base;
        if (GENERAL) {
          const R ar = R(a.alpha.x), ai = R(a.alpha.y);
          out.x = ar * base.x - ai * base.y;
          out.y = ar * base.y + ai * base.x;
          if (a.aux) {
            const C2<R> u = U[GENERAL ? j : 0];
            const R br = R(a.beta.x), bi = R(a.beta.y);
            out.x += br * u.x - bi * u.y;
            out.y += br * u.y + bi * u.x;
          }
        }
        // streaming store: y is not re-read by this launch, keep L2 for the
        // halo slices and the field
        bstore<R, true>(out, a.dst + rbase, b.dst, vo, s);
        if (RED == 1) {  // <w, out>
          const C2<R> u = Wr[RED == 1 ? j : 0];
          acc0 += double(u.x) * out.x + double(u.y) * out.y;
          acc1 += double(u.x) * out.y - double(u.y) * out.x;
        } else if (RED == 2) {  // <out, w>, |out|^2, |w|^2
          const C2<R> u = Wr[RED == 2 ? j : 0];
          acc0 += double(out.x) * u.x + double(out.y) * u.y;
          acc1 += double(out.x) * u.y - double(out.y) * u.x;
          acc2 += double(out.x) * out.x + double(out.y) * out.y;
          acc3 += double(u.x) * u.x + double(u.y) * u.y;
        } else if (RED == 3 || RED == 4) {  // <out, source>, |out|^2, |source|^2
          acc0 += double(out.x) * id.x + double(out.y) * id.y;
          acc1 += double(out.x) * id.y - double(out.y) * id.x;
          acc2 += double(out.x) * out.x + double(out.y) * out.y;
          acc3 += double(id.x) * id.x + double(id.y) * id.y;
          if (RED == 4) {  // <w, out>, <w, source>
            const C2<R> u = Wr[RED == 4 ? j : 0];
            acc4 += double(u.x) * out.x + double(u.y) * out.y;
            acc5 += double(u.x) * out.y - double(u.y) * out.x;
            acc6 += double(u.x) * id.x + double(u.y) * id.y;
            acc7 += double(u.x) * id.y - double(u.y) * id.x;
          }
        }
      }
    }
    if (RED != 0) {
      // the reductions of this slice are complete here: without this point the
      // compiler sinks them below the next transform and keeps the slice's
      // operands live across it
      asm volatile("" ::"v"(acc0), "v"(acc1), "v"(acc2), "v"(acc3));
      if (RED == 4) asm volatile("" ::"v"(acc4), "v"(acc5), "v"(acc6), "v"(acc7));
    }
    if (k + 1 < count) {
      // transform source slice t for the next output slice
      if (DIR < 0) scale_field<R, NX>(b.pre, t * V * FS, fo, X);
      if constexpr (TR == 1)
        slice_T3_mfma16(cc, ta, lds, l, X);
      else if constexpr (TR == 2)
        slice_T3_fft16(lam, lds, l, X);
      else
        slice_T3<R, NX, 0, true>(cc, lds, l, X);
    }
  }
  if (RED != 0) {
    constexpr int NR = (RED == 4) ? 8 : 4;
    double acc[NR];
    acc[0] = wsum(acc0);
    acc[1] = wsum(acc1);
    acc[2] = wsum(acc2);
    acc[3] = wsum(acc3);
    if (RED == 4) {
      acc[NR - 4] = wsum(acc4);
      acc[NR - 3] = wsum(acc5);
      acc[NR - 2] = wsum(acc6);
      acc[NR - 1] = wsum(acc7);
    }
    __syncthreads();
    double* sm = reinterpret_cast<double*>(smem_raw);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) {
#pragma unroll
      for (int j = 0; j < NR; ++j) sm[wid * NR + j] = acc[j];
    }
    __syncthreads();
    if (threadIdx.x < NR) {
      const int j = threadIdx.x;
      double v = 0;
      for (int w = 0; w < (P + 63) / 64; ++w) v += sm[w * NR + j];
      a.red_out[((long long)r * nslab + sb) * NR + j] = v;
    }
  }
}

template <typename R, int NX, int DIR, bool GENERAL, int SRC, int RED, int TR = 0>
int launch_one(const Lattice& L, const HopArgs<R>& a, const SplitCoef<R, NX>& c, dim3 grid,
               size_t lds, int nslab) {
  static bool attr = false;
  if (!attr) {
    UFG_HIP(hipFuncSetAttribute((const void*)hop_stream_kernel<R, NX, DIR, GENERAL, SRC, RED, TR>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    attr = true;
  }
  hipLaunchKernelGGL((hop_stream_kernel<R, NX, DIR, GENERAL, SRC, RED, TR>), grid, dim3(NX * NX),
                     lds, L.stream, a, c, L.ntau, nslab, stream_group(L), stream_inner(L));
  UFG_HIP(hipGetLastError());
  return UFG_OK;
}

template <typename R, int NX, int DIR>
int launch_dir(const Lattice& L, const HopArgs<R>& a, const SplitCoef<R, NX>& c) {
  const int nslab = stream_nslab(L);
  const size_t lds = size_t(lds_slice_elems<NX>()) * sizeof(C2<R>);
  const bool general = (a.alpha.x != 1.0 || a.alpha.y != 0.0 || a.aux != nullptr);
  const dim3 grid(stream_grid(L, a.nrhs));
  // instantiated combinations: plain apply (any reduction), the residual form
  // b - A x, and the two fused BiCGStab sources with their reductions
  if (a.src_mode == 1 && a.red_mode == 1 && !general)
    return launch_one<R, NX, DIR, false, 1, 1>(L, a, c, grid, lds, nslab);
  if (a.src_mode == 2 && a.red_mode == 3 && !general)
    return launch_one<R, NX, DIR, false, 2, 3>(L, a, c, grid, lds, nslab);
  if (a.src_mode == 2 && a.red_mode == 4 && !general && a.red_w != nullptr)
    return launch_one<R, NX, DIR, false, 2, 4>(L, a, c, grid, lds, nslab);
  if (a.src_mode == 0 && general && a.red_mode == 0)
    return launch_one<R, NX, DIR, true, 0, 0>(L, a, c, grid, lds, nslab);
  if (a.src_mode == 0 && !general) {
    switch (a.red_mode) {
      case 0:
        if constexpr (sizeof(R) == 4 && NX == 16) {
          if (L.t3_route == 1)
            return launch_one<R, NX, DIR, false, 0, 0, 1>(L, a, c, grid, lds, nslab);
          if (L.t3_route == 2)
            return launch_one<R, NX, DIR, false, 0, 0, 2>(L, a, c, grid, lds, nslab);
        }
        return launch_one<R, NX, DIR, false, 0, 0>(L, a, c, grid, lds, nslab);
      case 1: return launch_one<R, NX, DIR, false, 0, 1>(L, a, c, grid, lds, nslab);
      case 2: return launch_one<R, NX, DIR, false, 0, 2>(L, a, c, grid, lds, nslab);
      case 3: return launch_one<R, NX, DIR, false, 0, 3>(L, a, c, grid, lds, nslab);
      default: break;
    }
  }
  set_error("streaming kernel: unsupported combination of source, reduction and scaling");
  return UFG_EINVAL;
}

template <typename R, int NX>
int launch_nx(const Lattice& L, const HopArgs<R>& a) {
  SplitCoef<R, NX> c;
  const std::vector<double>& h = L.split_host;
  int k = 0;
  for (auto& v : c.es) v = R(h[k++]);
  for (auto& v : c.ea) v = R(h[k++]);
  for (auto& v : c.os) v = R(h[k++]);
  for (auto& v : c.oa) v = R(h[k++]);
  if (a.shift < 0) return launch_dir<R, NX, -1>(L, a, c);
  return launch_dir<R, NX, +1>(L, a, c);
}

}  // namespace

int stream_slab(const Lattice& L) {
  if (L.slab > 0) return std::min(L.slab, L.ntau);
  // One slice per workgroup throughout (with the slab groups of stream_group):
  // complex64 apply_M at 16^3 x 400, 8 rhs: 48.8 us at two slices per
  // workgroup in the contiguous numbering, 43.1 us at one in groups of 10;
  // complex128: 102.9 / 95.3 us (M / M^T) at two slices, 95.4 / 95.8 us at
  // one in groups of 10 taken rhs-inner (16^3 x 800: 200.1 / 177.9 against
  // 178.7 / 178.9 us), the FP64 solve within 0.5 %.
  return 1;
}

int stream_nslab(const Lattice& L) {
  if (L.nslab > 0) return std::min(L.nslab, L.ntau);
  const int slab = stream_slab(L);
  return (L.ntau + slab - 1) / slab;
}

int stream_group(const Lattice& L) {
  if (L.xcd_group >= 0) return std::min(L.xcd_group, stream_nslab(L));
  // Groups of ten slabs per XCD. complex64 walks a group's slabs for one rhs
  // after the other; complex128 lattices of 2^20 sites and more take every rhs
  // of a group in turn (stream_inner), so a field slice is read while the same
  // XCD still holds it. Smaller complex128 lattices (short launches,
  // few slabs) keep the contiguous numbering.
  if (L.dtype == UFG_C64) return std::min(10, stream_nslab(L));
  if ((long long)L.V * L.ntau >= (1ll << 20)) return std::min(10, stream_nslab(L));
  return 0;
}

int stream_inner(const Lattice& L) {
  if (L.xcd_group >= 0) return L.xcd_rhs_inner;
  return (L.dtype == UFG_C128 && (long long)L.V * L.ntau >= (1ll << 20)) ? 1 : 0;
}

int stream_grid(const Lattice& L, int nrhs) {
  const int nslab = stream_nslab(L), xg = stream_group(L);
  if (xg <= 0) return nslab * nrhs;
  if (stream_inner(L)) {
    const int groups = (nslab + xg - 1) / xg;
    return 8 * ((groups + 7) / 8) * nrhs * xg;
  }
  const int F = nslab / xg, rem = nslab - F * xg;
  int most = 0;
  for (int j = 0; j < 8; ++j) {
    int nj = xg * (F / 8 + ((j < (F & 7)) ? 1 : 0));
    if (rem > 0 && (F & 7) == j) nj += rem;
    most = std::max(most, nj);
  }
  return 8 * nrhs * most;
}

bool stream_supported(const Lattice& L) {
  // buffer offsets are 32-bit: one rhs block of complex128 must stay below 2 GiB
  const long long block = (long long)L.ntau * L.nx * L.nx * L.nx * (long long)sizeof(double2);
  // Every Nx with a block form (6 to 16). Nx = 6, 10 and 14 ran in the general slice
  // kernel before (dense lines, every slice loaded twice), M / M^T us: 10^3 x 201, 3
  // rhs complex128 13.3 / 15.1 -> 6.7 / 7.1, 10^3 x 400, 8 rhs complex64 20.4 / 22.7 -> 11.2 /
  // 11.1, 14^3 x 400, 8 rhs complex128 100 / 108 -> 64 / 64, 6^3 x 800, 64 rhs complex64
  // 46.6 / 50.8 -> 42.9 / 43.1 (36 of a wave's 64 lanes hold a line there), 6^3 x 50
  // complex128 6.5 / 6.7 -> 6.2 / 6.3. Nx = 2 and 4 keep it: several slices to a wave.
  return L.dim == 3 && !L.split_host.empty() && block < (1ll << 31);
}

template <typename R>
int launch_hop_stream(const Lattice& L, const HopArgs<R>& args) {
  HopArgs<R> a = args;
  if (a.beta.x == 0.0 && a.beta.y == 0.0) a.aux = nullptr;
  if (a.fin_part && !(a.src_mode == 2 && a.red_mode == 4 && a.fin_part2 && a.fin_flags &&
                      a.st && a.fin_nblk > 0 && a.fin_nblk2 > 0)) {
    set_error("streaming kernel: the fused alpha step needs source 2, reduction 4 and its "
              "partials, state and flags");
    return UFG_EINVAL;
  }
  // M-type applies the field to the source slice, M^T-type to the output slice
  const bool fields_ok = (a.shift < 0) ? (a.pre != nullptr && a.post == nullptr)
                                       : (a.post != nullptr && a.pre == nullptr);
  if (!fields_ok) {
    set_error("streaming kernel: field must multiply the source (M) or the output (M^T)");
    return UFG_EINVAL;
  }
  switch (L.nx) {
    case 6: return launch_nx<R, 6>(L, a);
    case 8: return launch_nx<R, 8>(L, a);
    case 10: return launch_nx<R, 10>(L, a);
    case 14: return launch_nx<R, 14>(L, a);
    case 12: return launch_nx<R, 12>(L, a);
    case 16: return launch_nx<R, 16>(L, a);
    default: set_error("streaming kernel: unsupported nx"); return UFG_EINVAL;
  }
}

template int launch_hop_stream<float>(const Lattice&, const HopArgs<float>&);
template int launch_hop_stream<double>(const Lattice&, const HopArgs<double>&);

}  // namespace ufg
