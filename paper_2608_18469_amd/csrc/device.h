// Device helpers shared by the GEMM kernels: element conversions, MFMA operand
// fragments, the XCD-aware tile order, direct-to-LDS loads.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "internal.h"

namespace erase {

#define ERASE_LAUNCH(KERNEL, GRID, BLOCK, SHMEM, STREAM, EV, ...)                                   \
  do {                                                                                             \
    if ((EV).e0 || (EV).e1)                                                                        \
      hipExtLaunchKernelGGL(KERNEL, GRID, BLOCK, SHMEM, STREAM, (EV).e0, (EV).e1, 0, __VA_ARGS__); \
    else                                                                                           \
      hipLaunchKernelGGL(KERNEL, GRID, BLOCK, SHMEM, STREAM, __VA_ARGS__);                        \
  } while (0)

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));  // 16-byte chunk in registers

// ---------------------------------------------------------------------------
// element conversions (bf16 is carried as uint16_t)
// ---------------------------------------------------------------------------
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// gfx950 converts in hardware (v_cvt_pk_bf16_f32): round to nearest, ties to
// even, NaN stays NaN, no branch.
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

template <typename T> __device__ __forceinline__ float ldf(const T* p);
template <> __device__ __forceinline__ float ldf<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float ldf<uint16_t>(const uint16_t* p) { return bf2f(*p); }

template <typename T> __device__ __forceinline__ T cvt(float f);
template <> __device__ __forceinline__ float cvt<float>(float f) { return f; }
template <> __device__ __forceinline__ uint16_t cvt<uint16_t>(float f) { return f2bf(f); }

template <typename T> __device__ __forceinline__ float asf(T v);
template <> __device__ __forceinline__ float asf<float>(float v) { return v; }
template <> __device__ __forceinline__ float asf<uint16_t>(uint16_t v) { return bf2f(v); }

// Four consecutive elements of one feature-major row: one 8- or 16-byte store.
__device__ __forceinline__ void st4(uint16_t* p, const uint16_t v[4]) {
  uint2 w;
  w.x = (uint32_t)v[0] | ((uint32_t)v[1] << 16);
  w.y = (uint32_t)v[2] | ((uint32_t)v[3] << 16);
  *reinterpret_cast<uint2*>(p) = w;
}
__device__ __forceinline__ void st4(float* p, const float v[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}

// Pointers read from device memory (not kernel arguments) are generic to the
// compiler; this marks them global so loads and stores use the global path.
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T* gmem(T* p) {
  return (__attribute__((address_space(1))) T*)p;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// An MFMA operand fragment (8 consecutive contraction indices of one row) from
// a k-major bf16 LDS tile: two transposing 8-byte reads, rows p and p + 4*pitch.
typedef short s16x4_t __attribute__((ext_vector_type(4)));
template <typename T>
__device__ __forceinline__ u32x4_t tr_frag(const T* p, int pitch) {
  typedef __attribute__((address_space(3))) s16x4_t lds_s16x4;
  const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
  const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * pitch));
  const uint2 a = __builtin_bit_cast(uint2, lo), b = __builtin_bit_cast(uint2, hi);
  return u32x4_t{a.x, a.y, b.x, b.y};
}

// GELU in its tanh form, 0.5 u (1 + tanh(c (u + a u^3))) with c = sqrt(2/pi),
// a = 0.044715, and its derivative
// 0.5 (1 + t) + 0.5 u (1 - t^2) c (1 + 3 a u^2), t = tanh(c (u + a u^3)).
constexpr float kGeluC = 0.7978845608028654f, kGeluA = 0.044715f;
// tanh(y) = 1 - 2 / (exp(2y) + 1) with the hardware exp2 and reciprocal
// (absolute error about 1e-7; +-1 in the limits, where exp2 gives inf or 0)
__device__ __forceinline__ float tanh_hw(float y) {
  const float e = __builtin_amdgcn_exp2f(y * 2.8853900817779268f);  // 2 log2(e)
  return 1.f - 2.f * __builtin_amdgcn_rcpf(e + 1.f);
}
__device__ __forceinline__ float gelu_f(float u) {
  const float t = tanh_hw(kGeluC * fmaf(kGeluA * u * u, u, u));
  return 0.5f * u * (1.f + t);
}
__device__ __forceinline__ float gelu_grad_f(float u) {
  const float t = tanh_hw(kGeluC * fmaf(kGeluA * u * u, u, u));
  return 0.5f * (1.f + t) + 0.5f * u * (1.f - t * t) * kGeluC * fmaf(3.f * kGeluA, u * u, 1.f);
}

// XCD-aware tile order.  A launch's workgroup i runs on XCD (i + c) % 8 for
// some c, so the workgroups i = r (mod 8) share one XCD and its L2.
// xcd_linear() renumbers them so that each XCD owns one contiguous range of
// logical tiles; tile_from() walks logical tiles in groups of `group` M-tiles
// (M fastest inside a group, then N, then the next group; split-K slices
// last), so each range is a compact block of output tiles whose A and B rows
// are fetched into that XCD's L2 once and reused there.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_linear(int bid, int total) {
  const int q = total / kXcds, r = total % kXcds;
  const int x = bid % kXcds, loc = bid / kXcds;
  return x * q + min(x, r) + loc;
}
struct TileIdx {
  int m, n, z;
};
__device__ __forceinline__ TileIdx tile_from(int t, int gm, int gn, int group) {
  const int per = gm * gn;
  const int z = t / per;
  int u = t - z * per;
  const int gsz = group * gn;
  const int gi = u / gsz;
  const int mf = gi * group;
  const int gh = min(group, gm - mf);
  u -= gi * gsz;
  return {mf + u % gh, u / gh, z};
}

// One 16-byte chunk per lane from global memory straight into LDS: lane l
// writes bytes [lds + 16 l, lds + 16 l + 16) of the wave's 1 KB block at the
// LDS byte address `lds` (wave-uniform, through M0).  The load counts in the
// wave's vector-memory counter like any load; the caller waits for it before
// reading the block.  The compiler reserves M0 and keeps nothing in it across
// these statements: no other instruction of the kernel reads it.
__device__ __forceinline__ void lds_dma16(const void* src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(src) : "memory");
}
// The same with a wave-uniform base address in scalar registers and the
// lane's 32-bit byte offset from it (no 64-bit address per lane and load).
__device__ __forceinline__ void lds_dma16s(const void* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "memory");
}


// Arguments of a batched launch (BlockJob in device memory, written at
// init): scalar loads through the constant address space, pointers typed as
// global so that every access through them takes the global path.
typedef const __attribute__((address_space(4))) char* cmem_t;
template <typename T>
__device__ __forceinline__ void ld_field(cmem_t p, T& v) {
  v = *reinterpret_cast<const __attribute__((address_space(4))) T*>(p);
}
template <typename T>
__device__ __forceinline__ void ld_field(cmem_t p, T*& v) {
  typedef __attribute__((address_space(1))) T* gptr;
  v = (T*)*reinterpret_cast<const __attribute__((address_space(4))) gptr*>(p);
}
__device__ __forceinline__ cmem_t job_of(const BlockJob* jobs) { return (cmem_t)(uintptr_t)(jobs + blockIdx.y); }
#define ERASE_LD(S, F) ld_field(p + offsetof(S, F), v.F)
__device__ __forceinline__ void ld_gemm(cmem_t p, GemmDesc& v, const StepPtrs& st) {
  ERASE_LD(GemmDesc, A), ERASE_LD(GemmDesc, lda), ERASE_LD(GemmDesc, B), ERASE_LD(GemmDesc, ldb);
  ERASE_LD(GemmDesc, M), ERASE_LD(GemmDesc, N), ERASE_LD(GemmDesc, K), ERASE_LD(GemmDesc, kps);
  ERASE_LD(GemmDesc, split), ERASE_LD(GemmDesc, bm), ERASE_LD(GemmDesc, bn), ERASE_LD(GemmDesc, group);
  ERASE_LD(GemmDesc, kgroups);
  if (v.A == reinterpret_cast<const void*>(uintptr_t(16))) v.A = st.x;
  if (v.B == reinterpret_cast<const void*>(uintptr_t(16))) v.B = st.x;
}
__device__ __forceinline__ void ld_epi(cmem_t p, EpiParams& v, const StepPtrs& st) {
  ERASE_LD(EpiParams, bias), ERASE_LD(EpiParams, y), ERASE_LD(EpiParams, ldy), ERASE_LD(EpiParams, x0);
  ERASE_LD(EpiParams, ldx0), ERASE_LD(EpiParams, xl), ERASE_LD(EpiParams, ldxl), ERASE_LD(EpiParams, part);
  ERASE_LD(EpiParams, ldp), ERASE_LD(EpiParams, pstride), ERASE_LD(EpiParams, bpart), ERASE_LD(EpiParams, res);
  ERASE_LD(EpiParams, ldres), ERASE_LD(EpiParams, mask), ERASE_LD(EpiParams, ldmask), ERASE_LD(EpiParams, gout);
  ERASE_LD(EpiParams, ldgout), ERASE_LD(EpiParams, dmn), ERASE_LD(EpiParams, lddmn);
  ERASE_LD(EpiParams, below_cross), ERASE_LD(EpiParams, hw), ERASE_LD(EpiParams, hc), ERASE_LD(EpiParams, lam);
  ERASE_LD(EpiParams, inv_m), ERASE_LD(EpiParams, pdw), ERASE_LD(EpiParams, pdc), ERASE_LD(EpiParams, ploss);
  ERASE_LD(EpiParams, ap), ERASE_LD(EpiParams, am), ERASE_LD(EpiParams, av), ERASE_LD(EpiParams, ag);
  ERASE_LD(EpiParams, ash), ERASE_LD(EpiParams, ldash), ERASE_LD(EpiParams, b1), ERASE_LD(EpiParams, b2);
  ERASE_LD(EpiParams, eps), ERASE_LD(EpiParams, bp), ERASE_LD(EpiParams, bm), ERASE_LD(EpiParams, bv);
  ERASE_LD(EpiParams, bg);
  v.labels = st.labels;
  v.hyper = st.hyper;
  if (v.x0 == reinterpret_cast<const void*>(uintptr_t(16))) v.x0 = st.x;
  if (v.xl == reinterpret_cast<const void*>(uintptr_t(16))) v.xl = st.x;
}
// (not the first chunks of the segments: adam_chunk's search reads them
// from the table)
__device__ __forceinline__ void ld_adam(cmem_t p, AdamArgs& v, const StepPtrs& st, int64_t block) {
  ERASE_LD(AdamArgs, seg), ERASE_LD(AdamArgs, nseg), ERASE_LD(AdamArgs, nchunks), ERASE_LD(AdamArgs, beta1);
  ERASE_LD(AdamArgs, beta2), ERASE_LD(AdamArgs, eps), ERASE_LD(AdamArgs, ploss), ERASE_LD(AdamArgs, nloss);
  ERASE_LD(AdamArgs, inv_m), ERASE_LD(AdamArgs, status);
  v.hyper = st.hyper;
  v.loss_out = st.losses + block;
}
__device__ __forceinline__ void ld_head(cmem_t p, HeadArgs& v, const StepPtrs& st) {
  ERASE_LD(HeadArgs, z), ERASE_LD(HeadArgs, ldz), ERASE_LD(HeadArgs, w), ERASE_LD(HeadArgs, c);
  ERASE_LD(HeadArgs, lam), ERASE_LD(HeadArgs, inv_m), ERASE_LD(HeadArgs, M), ERASE_LD(HeadArgs, N);
  ERASE_LD(HeadArgs, rows), ERASE_LD(HeadArgs, dmn), ERASE_LD(HeadArgs, lddmn), ERASE_LD(HeadArgs, pdw);
  ERASE_LD(HeadArgs, pdc), ERASE_LD(HeadArgs, ploss);
  v.y = st.labels;
}
#undef ERASE_LD
__device__ __forceinline__ int64_t ld_block(cmem_t j) {
  int64_t b;
  ld_field(j + offsetof(BlockJob, block), b);
  return b;
}

}  // namespace erase
