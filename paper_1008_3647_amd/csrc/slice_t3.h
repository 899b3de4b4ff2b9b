// T^3 (or a basis change U^3, U^3T) of one time slice by a workgroup of Nx^2
// threads, z in registers, y and x through one LDS slice, and the pieces the
// kernels built on it share. Used by the streaming operator (hop_stream.hip)
// and by the weak-coupling kernels (wce.hip).
#pragma once

#include "hop_stream.h"
#include "krylov.h"
#include "split_line.h"

namespace ufg {
namespace {
using namespace splitk;

// LDS slot of element (row, col) of a slice stored as NX*NX rows of NX + 1: the
// pad column spreads the banks for all three line directions (Nx = 8, 16: no
// conflicts at 4, 8 or 16 bytes an element), and every slot of a line is one
// base plus an immediate. An XOR swizzle needs one address register for each of
// the 2 Nx slots of the y and x lines (plain complex64 Nx = 16 operator: 116
// VGPRs for M and 137 for M^T, 87 and 112 with the pad), and the z-planes of a
// wave shared banks: complex128 M^T at 16^3 x 800, 8 rhs 179.6 -> 176.1 us,
// complex64 M at 16^3 x 400 43.0 -> 42.5 us.
template <int NX>
__device__ __forceinline__ int lds_at(int row, int col) {
  return row * (NX + 1) + col;
}
template <int NX>
constexpr int lds_slice_elems() {
  return NX * NX * (NX + 1);
}

// T^3 of the slice held as z-lines in v (thread (y, x)); result left in v.
// Barriers: stage 1 (thread (y, x) writes its z-line) feeds the y-lines of
// other waves, and the x-lines feed the z-lines of other waves. The y-lines
// (z, x) and x-lines (z, y) of one z-plane belong to the same NX consecutive
// threads, which sit in one wave when NX divides 64: there a wave-level
// ordering point replaces the block barrier. Each thread's last read and its
// next first write touch only its own z-line, so no barrier guards the reuse
// of the buffer by the next slice.
// MODE 0: T (positions -> positions); 1: U^T (positions -> block-ordered
// modes); 2: U (modes -> positions). The same three passes serve all three.
// El: complex, or one real component (every map is real).
template <int MODE, typename R, int NX, typename Coef, typename El>
__device__ __forceinline__ void line_op(const Coef& c, El (&v)[NX]) {
  if constexpr (MODE == 0)
    split_line<R, NX>(c, v);
  else if constexpr (MODE == 1)
    modes_fwd<R, NX>(c, v);
  else
    modes_bwd<R, NX>(c, v);
}

// The blocks in device memory, read as scalars (constant address space, so the
// loads go through the scalar cache). The empty asm makes the pointer opaque
// once per stage, so that the compiler neither keeps all blocks in SGPRs across
// a slice nor spills them to VGPR lanes (66 numbers a set at Nx = 16; kept
// instead, order-2 WCE on 8^3 x 160, 4 rhs: 47 -> 51 us, 16^3 x 400, 8 rhs
// complex64 282 -> 284 us).
template <typename R, int NX>
struct CoefPtr {
  const SplitCoef<R, NX>* p;
};
template <int MODE, typename R, int NX, typename El>
__device__ __forceinline__ void line_op(const CoefPtr<R, NX>& c, El (&v)[NX]) {
  using CC = const __attribute__((address_space(4))) SplitCoef<R, NX>;
  CC* q = (CC*)c.p;
  asm volatile("" : "+s"(q));
  line_op<MODE, R, NX>(*q, v);
}

// Ordering point inside one wave: LDS operations of a wave are performed in
// order; the fences keep the compiler from moving reads above writes.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Barrier among the threads of one slice: the slice of Nx = 8 is one wave.
template <int NX>
__device__ __forceinline__ void slice_sync() {
  if constexpr (NX * NX == 64)
    wave_order();
  else
    __syncthreads();
}

template <typename R, int NX, int MODE = 0, bool KEEP = false, typename Coef, typename El>
__device__ __forceinline__ void slice_T3(const Coef& c, El* lds, int l, El (&v)[NX]) {
  const int y = l / NX, x = l - (l / NX) * NX;
  line_op<MODE, R, NX>(c, v);  // along z
#pragma unroll
  for (int z = 0; z < NX; ++z) lds[lds_at<NX>(z * NX + y, x)] = v[z];
  slice_sync<NX>();
  El w[NX];
  {
    const int z = l / NX, xx = l - (l / NX) * NX;
#pragma unroll
    for (int yy = 0; yy < NX; ++yy) w[yy] = lds[lds_at<NX>(z * NX + yy, xx)];
    line_op<MODE, R, NX>(c, w);  // along y
#pragma unroll
    for (int yy = 0; yy < NX; ++yy) lds[lds_at<NX>(z * NX + yy, xx)] = w[yy];
  }
  if constexpr (64 % NX == 0) {
    wave_order();
  } else {
    __syncthreads();
  }
  {
    const int z = l / NX, yy = l - (l / NX) * NX;
#pragma unroll
    for (int xx = 0; xx < NX; ++xx) w[xx] = lds[lds_at<NX>(z * NX + yy, xx)];
    line_op<MODE, R, NX>(c, w);  // along x
#pragma unroll
    for (int xx = 0; xx < NX; ++xx) lds[lds_at<NX>(z * NX + yy, xx)] = w[xx];
  }
  slice_sync<NX>();
  if (KEEP) return;  // the result stays in LDS: z-line of thread (y, x) at lds_at(z NX + y, x)
#pragma unroll
  for (int z = 0; z < NX; ++z) v[z] = lds[lds_at<NX>(z * NX + y, x)];
}

// Raw buffer access: one 128-bit resource per array (base = the rhs block),
// a 32-bit lane offset in a VGPR and the slice / z offset in an SGPR.
// Out-of-range accesses are dropped by the hardware (loads return 0).
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int kRsrcWord3 = 0x00020000;  // gfx9 raw buffer, 32-bit data format
constexpr int kAuxNT = 2;               // non-temporal

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, kRsrcWord3);
}

template <typename R, int AUX = 0>
__device__ __forceinline__ C2<R> bload(__amdgpu_buffer_rsrc_t rs, int vo, int so) {
  if constexpr (sizeof(R) == 4) {
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, vo, so, AUX);
    return __builtin_bit_cast(C2<R>, v);
  } else {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, vo, so, AUX);
    return __builtin_bit_cast(C2<R>, v);
  }
}

// Store of one element at byte offset so + vo from base (rsrc describes the
// same block). 16-byte elements go through a FLAT store: the compiler's
// wait-state handling for a VALU overwrite of store-data registers does not
// cover buffer stores with an SGPR offset, and 128-bit buffer stores were
// seen to write registers already overwritten by the next instruction.
template <typename R, bool NT>
__device__ __forceinline__ void bstore(C2<R> v, C2<R>* base, __amdgpu_buffer_rsrc_t rs, int vo,
                                       int so) {
  if constexpr (sizeof(R) == 4) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rs, vo, so,
                                          NT ? kAuxNT : 0);
  } else {
    C2<R>* p = reinterpret_cast<C2<R>*>(reinterpret_cast<char*>(base) + so + vo);
    if (NT) {
      __builtin_nontemporal_store(v.x, &p->x);
      __builtin_nontemporal_store(v.y, &p->y);
    } else {
      *p = v;
    }
  }
}

template <typename R>
__device__ __forceinline__ R bload_real(__amdgpu_buffer_rsrc_t rs, int vo, int so) {
  if constexpr (sizeof(R) == 4) {
    return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b32(rs, vo, so, 0));
  } else {
    return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b64(rs, vo, so, 0));
  }
}

template <typename R>
__device__ __forceinline__ void bstore_real(R v, __amdgpu_buffer_rsrc_t rs, int vo, int so) {
  if constexpr (sizeof(R) == 4)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, vo, so, 0);
  else
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rs, vo, so, 0);
}

// Per-rhs scalars of the fused BiCGStab sources.
template <typename R>
struct SrcScal {
  R br, bi, wr, wi, ar, ai;
};

template <typename R, int SRC>
__device__ __forceinline__ SrcScal<R> src_scalars(const void* st, int r) {
  SrcScal<R> q{};
  if (SRC == 0) return q;
  const RhsState s = reinterpret_cast<const RhsState*>(st)[r];
  if (SRC == 1) {
    q.br = R(s.beta.x);  // beta = (rho / rho_old)(alpha / omega), set by the finalize
    q.bi = R(s.beta.y);
    q.wr = R(s.omega.x);
    q.wi = R(s.omega.y);
  } else {
    q.ar = R(s.alpha.x);
    q.ai = R(s.alpha.y);
  }
  return q;
}

// Where the transform reads the blocks of T (or U) from. The Nx = 16 blocks
// are 66 numbers. In FP64 (132 SGPRs) they exceed the scalar register file and
// the compiler spills them to VGPR lanes (a v_readlane before each use); with
// IN_LDS the workgroup copies them into LDS once and the transform reads them
// from there (broadcast reads). Measured per kernel: the fused FP64 M-type
// operator gains (t = A s: 227 -> 206 us); the plain FP64 operator (103 -> 122
// us), the M^T-type fused ones and every complex64 operator keep the
// kernel-argument copy.
template <bool IN_LDS, typename R, int NX>
using CoefSlot = typename std::conditional<IN_LDS, SplitCoef<R, NX>, char>::type;

template <bool IN_LDS, typename R, int NX>
__device__ __forceinline__ const SplitCoef<R, NX>* coef_copy(const SplitCoef<R, NX>& c,
                                                            CoefSlot<IN_LDS, R, NX>* lds_slot) {
  if constexpr (IN_LDS) {
    constexpr int NC = sizeof(SplitCoef<R, NX>) / sizeof(R);
    for (int i = threadIdx.x; i < NC; i += blockDim.x)
      reinterpret_cast<R*>(lds_slot)[i] = reinterpret_cast<const R*>(&c)[i];
    __syncthreads();
    return lds_slot;
  } else {
    return &c;
  }
}

}  // namespace
}  // namespace ufg
