// GEMM tiles with direct-to-LDS operands (bf16, gfx950).  First, for launches
// that fill the chip with them: 256 x 256 outputs per workgroup of eight waves, one workgroup per compute
// unit (128 KB of LDS stages).
//
// What bounds the GEMM core's 128 x 128 tiles is operand movement: a byte
// loaded feeds 64 multiply-adds, through registers and an LDS store, and one
// barrier per k-step drains the loads in flight.  Here
//  * a byte loaded feeds 128, and goes from global memory straight into LDS
//    (global_load_lds_dwordx4: no registers, no LDS store instructions);
//  * a 64-wide k-step is four phases, one per 128 x 128 quadrant of the tile:
//    the quadrant's fragments are read, one half of an operand of a later
//    k-step is issued, then the 16 MFMAs of each wave run.  A half is free as
//    soon as its quadrants are done, so up to the tile's end a whole k-step (64 KB
//    per compute unit) is in flight and no wait drains the loads: the waits
//    count the newest halves off;
//  * the two rows of waves run half a phase apart (one barrier more at the
//    start of the second): while one row's MFMAs run, the other's LDS reads
//    and loads are issued on the same SIMDs;
//  * the MFMA computes the transposed block (weight rows as the A operand),
//    and the two 16-row blocks of a quadrant take interleaved groups of four
//    weight rows, so a lane ends with eight consecutive output columns:
//    16-byte loads and stores in the epilogue, no LDS pass.
// Measured on one MI355X against the core's best tile: 16384 x 1677 x 1677
// 94 us (979 TFLOP/s) and 138 us, 16384 x 1024 x 1677 50 and 78 us,
// 8192 x 8192 x 8192 930 us (1182 TFLOP/s) and 1274 us; weight gradients
// 1677 x 1677 over 16384 rows 112 us (5 slices) and 165 us, 512 x 1677 over
// 32768 rows 73 us (16 slices) and 88 us.  A 128 x 256 form (8 MFMAs per
// phase) reached 771 TFLOP/s where this reaches 1116.
//
// Rows (columns, k-major) past the operands' logical extent are read clamped
// to the last one: they only reach outputs that are not stored.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "device.h"
#include "wide_plan.h"

namespace erase {

namespace wide {
constexpr int BK = 64, NW = 8, NT = 64 * NW;

// A half of an operand's tile is H rows (forward, input gradient: "NT", both
// operands contiguous along the contraction) or columns (weight gradient:
// k-major, both operands row-major over the contraction).  A stage is
// A0 | A1 | B0 | B1; two stages.  NT rows are 128 bytes with 16-byte chunk c at
// c ^ (3 bits of the row); k-major rows hold H elements with the chunks
// permuted by kperm16: fragment reads are conflict-free both ways.
constexpr int H = 128, BM = 2 * H, BN = 2 * H;
constexpr int HB = H * BK * 2;        // bytes of a half
constexpr int STAGE = 4 * HB, BYTES = 2 * STAGE;
constexpr int LD = HB / 1024 / NW;    // 1 KB loads per wave and half
constexpr int TA = H / 32, TB = H / 64;  // a wave's 16-wide blocks of a half

template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void bar() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// permutation of the 16 chunks of 16 bytes of a k-major row
__device__ __forceinline__ int kperm16(int r) { return 2 * ((r >> 1) & 1) + 4 * ((r >> 3) & 1) + 8 * (r & 1); }

// Output tile t of a GEMM's ntiles.
//
// Order of a wave's loads, LD per half: k-step p + 1's B1 in phase 0 of p and
// A1 in phase 1, p + 2's A0 in phase 2 and B0 in phase 3.  A half is
// overwritten two phases or more after its last read (A0, B0 are read in phase
// 0 of the k-step that used the stage, B1 in 1, A1 in 2): both wave rows are
// then past the MFMAs that waited for those reads.  A half read in phase q has
// been waited for by every wave in phase q - 1 or before, in front of a
// barrier: the waits leave the four newest halves in flight, fewer at the end.
template <bool KM, class Epi>
__device__ __forceinline__ void run(const GemmDesc& g, int t, int ntiles, bool want_rows, char* smem, Epi&& epi) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wv >> 2, wn = wv & 3;
  const int fr = lane & 15, fg = lane >> 4;
  const int M = g.M, N = g.N;
  const int64_t lda = g.lda, ldb = g.ldb;
  const TileIdx ti = tile_from(xcd_linear(t, ntiles), (M + BM - 1) / BM, (N + BN - 1) / BN, g.group);
  const int m0 = ti.m * BM, n0 = ti.n * BN, kb = ti.z * g.kps;
  const int nk = (min(g.K, kb + g.kps) - kb + BK - 1) / BK;
  const uint32_t lbase = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char*)smem);

  // ---- loads: of half h, of the k-step that pa[h], pb[h] point at
  const char* pa[2];
  const char* pb[2];
  uint32_t oa[2][LD], ob[2][LD];
  if constexpr (KM) {
    constexpr int CH = H / 8;  // chunks per k-major row
    pa[0] = pa[1] = static_cast<const char*>(g.A) + ((int64_t)kb * lda + m0) * 2;
    pb[0] = pb[1] = static_cast<const char*>(g.B) + ((int64_t)kb * ldb + n0) * 2;
    const int ml = ((M + 63) & ~63) - 8 - m0, nl = ((N + 63) & ~63) - 8 - n0;  // last whole chunk
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int u = 0; u < LD; ++u) {
        const int r = (wv * LD + u) * (64 / CH) + lane / CH, ch = (lane % CH) ^ kperm16(r);
        oa[h][u] = (uint32_t)((int64_t)r * lda + min(h * H + ch * 8, ml)) * 2;
        ob[h][u] = (uint32_t)((int64_t)r * ldb + min(h * H + ch * 8, nl)) * 2;
      }
  } else {
    pa[0] = pa[1] = static_cast<const char*>(g.A) + ((int64_t)m0 * lda + kb) * 2;
    pb[0] = pb[1] = static_cast<const char*>(g.B) + ((int64_t)n0 * ldb + kb) * 2;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int u = 0; u < LD; ++u) {
        const int r = (wv * LD + u) * 8 + (lane >> 3);
        oa[h][u] = (uint32_t)(min(h * H + r, M - 1 - m0) * (int)lda + ((lane & 7) ^ (r & 7)) * 8) * 2;
        ob[h][u] = (uint32_t)(min(h * H + r, N - 1 - n0) * (int)ldb + ((lane & 7) ^ ((r & 3) | ((r >> 1) & 4))) * 8) * 2;
      }
  }
  auto load_a = [&](int h, int st) {
#pragma unroll
    for (int u = 0; u < LD; ++u) lds_dma16s(pa[h], oa[h][u], lbase + st * STAGE + h * HB + (wv * LD + u) * 1024);
  };
  auto load_b = [&](int h, int st) {
#pragma unroll
    for (int u = 0; u < LD; ++u) lds_dma16s(pb[h], ob[h][u], lbase + st * STAGE + (2 + h) * HB + (wv * LD + u) * 1024);
  };
  auto next = [&](int h) {
    pa[h] += KM ? BK * lda * 2 : BK * 2;
    pb[h] += KM ? BK * ldb * 2 : BK * 2;
  };

  // ---- fragments
  const int tq = (lane & 15) >> 2, tc = lane & 3, trow = 8 * fg + tq;
  // NT: row of the 16-row block and permuted chunk; k half 1 flips bit 6
  const int fa0 = fr * 128 + ((fg ^ (fr & 7)) * 16);
  const int fb0o = (8 * (fr >> 2) + (fr & 3)) * 128 + ((fg ^ (fr & 7)) * 16);
  int ka[TA], kb_[TB];
#pragma unroll
  for (int i = 0; i < TA; ++i)
    ka[i] = KM ? (trow * H + (((((wm * H / 2) + i * 16) >> 3) + (tc >> 1)) ^ kperm16(trow)) * 8 + (tc & 1) * 4) * 2 : 0;
#pragma unroll
  for (int j = 0; j < TB; ++j)
    kb_[j] = KM ? (trow * H + (((((wn * H / 4) + j * 16) >> 3) + (tc >> 1)) ^ kperm16(trow)) * 8 + (tc & 1) * 4) * 2 : 0;

  u32x4_t fa[TA][2], fb[2][TB][2];
  auto read_a = [&](int h, int st) {
    const char* p = smem + st * STAGE + h * HB;
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int i = 0; i < TA; ++i) {
        if constexpr (KM)
          fa[i][kh] = tr_frag(reinterpret_cast<const uint16_t*>(p + ka[i] + kh * 32 * H * 2), H);
        else
          fa[i][kh] = *reinterpret_cast<const u32x4_t*>(p + (wm * (H / 2) + i * 16) * 128 + (fa0 ^ (kh * 64)));
      }
  };
  auto read_b = [&](int h, int st) {
    const char* p = smem + st * STAGE + (2 + h) * HB;
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int j = 0; j < TB; ++j) {
        if constexpr (KM)
          fb[h][j][kh] = tr_frag(reinterpret_cast<const uint16_t*>(p + kb_[j] + kh * 32 * H * 2), H);
        else
          fb[h][j][kh] = *reinterpret_cast<const u32x4_t*>(p + (wn * 32 + 4 * j) * 128 + (fb0o ^ (kh * 64)));
      }
  };

  f32x4_t acc[2][2][TA][TB];
  f32x4_t accr[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    accr[a] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[a][b][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  const bool rows = want_rows && ti.n == 0;
  auto mma = [&](auto ac, auto bc) {
    constexpr int a = decltype(ac)::value, b = decltype(bc)::value;
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
          acc[a][b][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fb[b][j][kh]),
                                                                    __builtin_bit_cast(bf16x8_t, fa[i][kh]),
                                                                    acc[a][b][i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };
  // row sums of A half a: ones times the block of this wave (blocks over wn)
  auto rowsum = [&](int a) {
    if constexpr (KM) {
      if (rows) {
        const u32x4_t one = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
#pragma unroll
        for (int i = 0; i < TA; ++i)
          if (wn == i) {
#pragma unroll
            for (int kh = 0; kh < 2; ++kh)
              accr[a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, one),
                                                                __builtin_bit_cast(bf16x8_t, fa[i][kh]), accr[a], 0, 0, 0);
          }
      }
    }
  };
  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};

  load_a(0, 0);
  load_b(0, 0);
  next(0);
  load_b(1, 0);
  load_a(1, 0);
  next(1);
  if (nk > 1) {
    load_a(0, 1);
    load_b(0, 1);
    next(0);
    wait_vm<4 * LD>();
  } else {
    wait_vm<2 * LD>();
  }
  bar();
  if (wm == 1) bar();  // the two wave rows run half a phase apart

  int st = 0;
  for (int k = nk; k > 0; --k, st ^= 1) {
    const bool more = k > 1, more2 = k > 2;  // a next k-step, and one after it
    // phase 0: A0 x B0; waits for B1
    read_b(0, st);
    read_a(0, st);
    if (more) {
      load_b(1, st ^ 1);
      wait_vm<4 * LD>();
    } else {
      wait_vm<LD>();
    }
    bar();
    wait_lds();
    mma(c0, c0);
    rowsum(0);
    bar();
    // phase 1: A0 x B1; waits for A1
    read_b(1, st);
    if (more) {
      load_a(1, st ^ 1);
      next(1);
      wait_vm<4 * LD>();
    } else {
      wait_vm<0>();
    }
    bar();
    wait_lds();
    mma(c0, c1);
    bar();
    // phase 2: A1 x B1
    read_a(1, st);
    if (more2) load_a(0, st);
    bar();
    wait_lds();
    mma(c1, c1);
    rowsum(1);
    bar();
    // phase 3: A1 x B0 (in registers); waits for the next k-step's A0, B0
    if (more2) {
      load_b(0, st);
      next(0);
      wait_vm<4 * LD>();
    } else if (more) {
      wait_vm<2 * LD>();
    }
    bar();
    mma(c1, c0);
    bar();
  }
  epi(acc, accr, ti, rows, wm, wn, fr, fg);
  if (wm == 0) bar();
}

__device__ __forceinline__ void unpack8(const u32x4_t& w, float f[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(w[i] << 16);
    f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ u32x4_t pack8(const float f[8]) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  u32x4_t o;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    o[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{f[2 * i], f[2 * i + 1]}), bf16x2_t));
  return o;
}
// eight columns from n of a row; the operands' rows are padded to whole chunks
__device__ __forceinline__ u32x4_t ld8(const void* p, int64_t ld, int m, int n) {
  return *reinterpret_cast<const __attribute__((address_space(1))) u32x4_t*>(
      gmem(static_cast<const uint16_t*>(p)) + (int64_t)m * ld + n);
}
__device__ __forceinline__ void stn(void* p, int64_t ld, int m, int n, int N, const u32x4_t& v) {
  uint16_t* d = static_cast<uint16_t*>(p) + (int64_t)m * ld + n;
  if (n + 8 <= N) {
    *reinterpret_cast<u32x4_t*>(d) = v;
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (n + k < N) d[k] = (uint16_t)(k & 1 ? v[k / 2] >> 16 : v[k / 2] & 0xffffu);
  }
}

// Epilogue operands of eight columns from (m, n), and the values stored there.
template <int KIND>
__device__ __forceinline__ void epi_load(const EpiParams& e, int m, int n, u32x4_t& r0, u32x4_t& r1) {
  if constexpr (KIND == GK_FWD_CROSS) {
    r0 = ld8(e.x0, e.ldx0, m, n);
    r1 = ld8(e.xl, e.ldxl, m, n);
  }
  if constexpr (KIND == GK_FWD_LIN) {
    if (e.res) r0 = ld8(e.res, e.ldres, m, n);
  }
  if constexpr (KIND == GK_DGRAD_GELU) r0 = ld8(e.mask, e.ldmask, m, n);
  if constexpr (KIND == GK_DGRAD) {
    if (e.res) r0 = ld8(e.res, e.ldres, m, n);
    if (e.below_cross)
      r1 = ld8(e.x0, e.ldx0, m, n);
    else if (e.mask)
      r1 = ld8(e.mask, e.ldmask, m, n);
  }
}
template <int KIND>
__device__ __forceinline__ void epi_bias(const EpiParams& e, int n, int N, float bias[8]) {
  if constexpr (KIND == GK_FWD_RELU || KIND == GK_FWD_CROSS) {
#pragma unroll
    for (int k = 0; k < 8; ++k) bias[k] = n + k < N ? e.bias[n + k] : 0.f;
  }
}
template <int KIND>
__device__ __forceinline__ void epi_store(const EpiParams& e, float v[8], const float bias[8], int m, int n, int N,
                                          const u32x4_t& r0, const u32x4_t& r1) {
  float p[8], q[8];
  if constexpr (KIND == GK_FWD_RELU) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      v[k] += bias[k];
      v[k] = v[k] < 0.f ? 0.f : v[k];  // keeps NaN
    }
    stn(e.y, e.ldy, m, n, N, pack8(v));
  } else if constexpr (KIND == GK_FWD_CROSS) {
    unpack8(r0, p);
    unpack8(r1, q);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = fmaf(p[k], v[k] + bias[k], q[k]);
    stn(e.y, e.ldy, m, n, N, pack8(v));
  } else if constexpr (KIND == GK_FWD_LIN) {
    if (e.res) {
      unpack8(r0, p);
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] += p[k];
    }
    stn(e.y, e.ldy, m, n, N, pack8(v));
  } else if constexpr (KIND == GK_FWD_GELU) {
    if (e.gout) stn(e.gout, e.ldgout, m, n, N, pack8(v));
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = gelu_f(v[k]);
    stn(e.y, e.ldy, m, n, N, pack8(v));
  } else if constexpr (KIND == GK_DGRAD_GELU) {
    unpack8(r0, p);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] *= gelu_grad_f(p[k]);
    stn(e.dmn, e.lddmn, m, n, N, pack8(v));
  } else {
    if (e.res) {
      unpack8(r0, p);
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] += p[k];
    }
    if (e.below_cross) {
      const u32x4_t gq = pack8(v);
      if (e.gout) stn(e.gout, e.ldgout, m, n, N, gq);
      unpack8(gq, p);
      unpack8(r1, q);
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = p[k] * q[k];
    } else if (e.mask) {
      unpack8(r1, q);
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = q[k] > 0.f ? v[k] : 0.f;
    }
    stn(e.dmn, e.lddmn, m, n, N, pack8(v));
  }
}

// Eight columns of an fp32 slice (rows are a multiple of 64 wide).
__device__ __forceinline__ void st_part(const EpiParams& e, const float v[8], int m, int n, int z) {
  f32x4_t* d = reinterpret_cast<f32x4_t*>(e.part + (int64_t)z * e.pstride + (int64_t)m * e.ldp + n);
  d[0] = f32x4_t{v[0], v[1], v[2], v[3]};
  d[1] = f32x4_t{v[4], v[5], v[6], v[7]};
}

// Epilogue of an NT tile: a lane holds eight consecutive columns of TA rows
// per quadrant.  The operands of one quadrant are loaded together.
template <int KIND, class A>
__device__ __forceinline__ void epi_nt(const EpiParams& e, const A& acc, int M, int N, const TileIdx& ti, int wm,
                                       int wn, int fr, int fg) {
  const int m0 = ti.m * BM, n0 = ti.n * BN;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int n = n0 + b * H + wn * 32 + fg * 8;
    if (n >= N) continue;
    float bias[8];
    epi_bias<KIND>(e, n, N, bias);
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      u32x4_t r0[TA], r1[TA];
#pragma unroll
      for (int i = 0; i < TA; ++i)
        epi_load<KIND>(e, min(m0 + a * H + wm * (H / 2) + i * 16 + fr, M - 1), n, r0[i], r1[i]);
#pragma unroll
      for (int i = 0; i < TA; ++i) {
        const int m = m0 + a * H + wm * (H / 2) + i * 16 + fr;
        if (m >= M) continue;
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = acc[a][b][i][k >> 2][k & 3];
        epi_store<KIND>(e, v, bias, m, n, N, r0[i], r1[i]);
      }
    }
  }
}

// Weight-gradient slice: fp32 partials (a lane holds four consecutive columns
// of a row per block) and the bias row sums.
template <class A, class R>
__device__ __forceinline__ void epi_wgrad(const EpiParams& e, const A& acc, const R& accr, int M, int N,
                                          const TileIdx& ti, bool rows, int wm, int wn, int fr, int fg) {
  const int m0 = ti.m * BM, n0 = ti.n * BN;
  float* out = e.part + (int64_t)ti.z * e.pstride;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int i = 0; i < TA; ++i) {
      const int m = m0 + a * H + wm * (H / 2) + i * 16 + fr;
      if (m >= M) continue;
      float* row = out + (int64_t)m * e.ldp;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int j = 0; j < TB; ++j) {
          const int n = n0 + b * H + wn * (H / 4) + j * 16 + 4 * fg;
          if (n < N) *reinterpret_cast<f32x4_t*>(row + n) = acc[a][b][i][j];  // rows padded to 64 columns
        }
      if (rows && wn == i && fg == 0) e.bpart[(int64_t)ti.z * M + m] = accr[a][0];
    }
}
}  // namespace wide

// ---------------------------------------------------------------------------
// 128 x 128 tiles, from about half a workgroup per compute unit on: the
// operands straight into NST LDS stages of a 64-wide k-step (32 KB), NST - 1
// k-steps in flight, one barrier per k-step.  Eight waves in two k-groups:
// each group computes the whole tile over its half of every k-step (a wave
// 64 x 64), so every SIMD runs two waves of one tile; the groups exchange
// halves of their partial tiles through LDS and each finishes 32 of a wave's
// 64 rows.  Bound by the latency of a k-step (load, barrier, fragment reads,
// MFMAs) when alone on its unit, by L2 and LDS traffic with two workgroups.
// The order of every sum is the same for any NST.
// Measured on one MI355X, against the best tile of the register-staged core:
// 8192 x 512 x 1677 18.3 us (769 TFLOP/s) and 25.7 us, 16384 x 512 x 2048 34.1
// (1008) and 46.0, 3001 x 1003 x 1003 12.1 and 15.8, 16384 x 512 x 512 14.3
// and 20.1 us; weight gradients 512 x 1677 over 4096 rows 15.8 and 19.6 us,
// 1003 x 1003 over 3001 rows 14.3 and 18.8 us.
// ---------------------------------------------------------------------------
namespace mid {
constexpr int BM = 128, BN = 128, BK = 64, NW = 8, NT = 64 * NW;
constexpr int OPB = BM * BK * 2, STAGE = 2 * OPB;  // bytes of an operand's k-step, of a stage
constexpr int XCH = 4 * 2 * 8 * 64 * 16;           // exchanged halves: 4 wave pairs x 2 directions x 8 tiles (64 KB)
template <int NST>
constexpr int bytes() {
  return (NST * STAGE > XCH ? NST * STAGE : XCH) + 2 * BM * 4;  // and the groups' bias row sums
}

// Partial tile of this workgroup; on return acc[0..1] of k-group kg hold the
// finished rows 32 kg .. 32 kg + 31 of the wave's 64, in all their columns.
template <int NST, bool KM>
__device__ __forceinline__ void run(const GemmDesc& g, const TileIdx& ti, bool rows, char* smem, f32x4_t (&out)[2][4],
                                    const EpiParams& e) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wv >> 2, wm = (wv >> 1) & 1, wn = wv & 1;
  const int fr = lane & 15, fg = lane >> 4;
  const int M = g.M, N = g.N, m0 = ti.m * BM, n0 = ti.n * BN, kb = ti.z * g.kps;
  const int nk = (min(g.K, kb + g.kps) - kb + BK - 1) / BK;
  const int64_t lda = g.lda, ldb = g.ldb;
  const uint32_t lbase = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char*)smem);
  const char *ga, *gb;
  uint32_t oa[2], ob[2];
  if constexpr (KM) {
    ga = static_cast<const char*>(g.A) + ((int64_t)kb * lda + m0) * 2;
    gb = static_cast<const char*>(g.B) + ((int64_t)kb * ldb + n0) * 2;
    const int ml = ((M + 63) & ~63) - 8 - m0, nl = ((N + 63) & ~63) - 8 - n0;  // last whole chunk
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = (wv * 2 + u) * 4 + (lane >> 4), ch = (lane & 15) ^ wide::kperm16(r);
      oa[u] = (uint32_t)((int64_t)r * lda + min(ch * 8, ml)) * 2;
      ob[u] = (uint32_t)((int64_t)r * ldb + min(ch * 8, nl)) * 2;
    }
  } else {
    ga = static_cast<const char*>(g.A) + ((int64_t)m0 * lda + kb) * 2;
    gb = static_cast<const char*>(g.B) + ((int64_t)n0 * ldb + kb) * 2;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = (wv * 2 + u) * 8 + (lane >> 3);
      oa[u] = (uint32_t)(min(r, M - 1 - m0) * (int)lda + ((lane & 7) ^ (r & 7)) * 8) * 2;
      ob[u] = (uint32_t)(min(r, N - 1 - n0) * (int)ldb + ((lane & 7) ^ ((r & 3) | ((r >> 1) & 4))) * 8) * 2;
    }
  }
  const int64_t sa = KM ? BK * lda * 2 : BK * 2, sb = KM ? BK * ldb * 2 : BK * 2;
  auto load = [&](int kt, int st) {
    const uint32_t l = lbase + st * STAGE + wv * 2048;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      lds_dma16s(ga + kt * sa, oa[u], l + u * 1024);
      lds_dma16s(gb + kt * sb, ob[u], l + OPB + u * 1024);
    }
  };
  const int tq = (lane & 15) >> 2, tc = lane & 3, trow = 8 * fg + tq;
  int ao[4], bo[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (KM) {
      const int hp = wide::kperm16(trow);
      ao[i] = ((kg * 32 + trow) * BM + ((((wm * 64 + i * 16) >> 3) + (tc >> 1)) ^ hp) * 8 + (tc & 1) * 4) * 2;
      bo[i] = OPB + ((kg * 32 + trow) * BN + ((((wn * 64 + i * 16) >> 3) + (tc >> 1)) ^ hp) * 8 + (tc & 1) * 4) * 2;
    } else {
      const int sl = ((4 * kg + fg) ^ (fr & 7)) * 16;
      ao[i] = (wm * 64 + i * 16 + fr) * 128 + sl;
      bo[i] = OPB + (wn * 64 + 32 * (i >> 1) + 4 * (i & 1) + 8 * (fr >> 2) + (fr & 3)) * 128 + sl;
    }
  }
  f32x4_t acc[4][4], accr[2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  accr[0] = accr[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int s = 0; s < NST - 1; ++s)
    if (s < nk) load(s, s);
  int st = 0;
  for (int kt = 0; kt < nk; ++kt) {
    // k-step kt has landed: at most the loads of the NST - 2 after it are in
    // flight; behind the barrier that holds for every wave, and every wave is
    // done with the stage the next loads overwrite (k-step kt - 1's)
    const int left = nk - 1 - kt;
    if (left >= NST - 2)
      wide::wait_vm<4 * (NST - 2)>();
    else
      wide::wait_vm<0>();
    wide::bar();
    if (kt + NST - 1 < nk) load(kt + NST - 1, st == 0 ? NST - 1 : st - 1);
    const char* p = smem + st * STAGE;
    u32x4_t fa[4], fb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (KM) {
        fb[i] = tr_frag(reinterpret_cast<const uint16_t*>(p + bo[i]), BN);
        fa[i] = tr_frag(reinterpret_cast<const uint16_t*>(p + ao[i]), BM);
      } else {
        fb[i] = *reinterpret_cast<const u32x4_t*>(p + bo[i]);
        fa[i] = *reinterpret_cast<const u32x4_t*>(p + ao[i]);
      }
    }
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fb[j]),
                                                            __builtin_bit_cast(bf16x8_t, fa[i]), acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    if constexpr (KM) {
      if (rows) {  // row sums of A: ones times the wave's two blocks (blocks over wn)
        const u32x4_t one = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (wn == i >> 1)
            accr[i & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8_t, one), __builtin_bit_cast(bf16x8_t, fa[i]), accr[i & 1], 0, 0, 0);
      }
    }
    st = st + 1 == NST ? 0 : st + 1;
  }
  // exchange: group kg keeps row blocks 2 kg, 2 kg + 1 and hands over the
  // other two
  __syncthreads();
  f32x4_t* xc = reinterpret_cast<f32x4_t*>(smem) + (wv & 3) * (2 * 8 * 64) + lane;
  float* rsum = reinterpret_cast<float*>(smem + (NST * STAGE > XCH ? NST * STAGE : XCH));
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (kg == 0)
        xc[(i * 4 + j) * 64] = acc[2 + i][j];
      else
        xc[(8 + i * 4 + j) * 64] = acc[i][j];
    }
  if constexpr (KM) {
    if (rows && fg == 0) {
#pragma unroll
      for (int i = 0; i < 2; ++i) rsum[kg * BM + wm * 64 + (2 * wn + i) * 16 + fr] = accr[i][0];
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) out[i][j] = kg == 0 ? acc[i][j] + xc[(8 + i * 4 + j) * 64] : xc[(i * 4 + j) * 64] + acc[2 + i][j];
  if constexpr (KM) {
    if (rows && tid < BM && m0 + tid < M) e.bpart[(int64_t)ti.z * M + m0 + tid] = rsum[tid] + rsum[BM + tid];
  }
}

template <int NST, int KIND>
__device__ __forceinline__ void nt_tile(const GemmDesc& g, const EpiParams& e, int b, int ntiles, char* smem) {
  const int gm = (g.M + BM - 1) / BM, gn = (g.N + BN - 1) / BN;
  const TileIdx ti = tile_from(xcd_linear(b, ntiles), gm, gn, g.group);
  f32x4_t acc[2][4];
  run<NST, false>(g, ti, false, smem, acc, e);
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int fr = lane & 15, fg = lane >> 4;
  const int mb = ti.m * BM + ((wv >> 1) & 1) * 64 + (wv >> 2) * 32 + fr, nb = ti.n * BN + (wv & 1) * 64 + fg * 8;
  const int M = g.M, N = g.N;
  u32x4_t r0[2][2], r1[2][2];
  float bias[2][8];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int n = nb + 32 * h;
    if (n >= N) continue;
    wide::epi_bias<KIND>(e, n, N, bias[h]);
#pragma unroll
    for (int i = 0; i < 2; ++i) wide::epi_load<KIND>(e, min(mb + 16 * i, M - 1), n, r0[h][i], r1[h][i]);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int n = nb + 32 * h;
    if (n >= N) continue;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int m = mb + 16 * i;
      if (m >= M) continue;
      float v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = acc[i][2 * h + (k >> 2)][k & 3];
      if constexpr (KIND == GK_DGRAD_PART)
        wide::st_part(e, v, m, n, ti.z);
      else
        wide::epi_store<KIND>(e, v, bias[h], m, n, N, r0[h][i], r1[h][i]);
    }
  }
}

template <int NST>
__device__ __forceinline__ void wgrad_tile(const GemmDesc& g, const EpiParams& e, int b, int ntiles, char* smem) {
  const int gm = (g.M + BM - 1) / BM, gn = (g.N + BN - 1) / BN;
  const TileIdx ti = tile_from(xcd_linear(b, ntiles), gm, gn, g.group);
  f32x4_t acc[2][4];
  run<NST, true>(g, ti, e.bpart != nullptr && ti.n == 0, smem, acc, e);
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int fr = lane & 15, fg = lane >> 4;
  float* out = e.part + (int64_t)ti.z * e.pstride;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = ti.m * BM + ((wv >> 1) & 1) * 64 + (wv >> 2) * 32 + 16 * i + fr;
    if (m >= g.M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = ti.n * BN + (wv & 1) * 64 + 16 * j + 4 * fg;
      if (n < g.N) *reinterpret_cast<f32x4_t*>(out + (int64_t)m * e.ldp + n) = acc[i][j];  // rows padded to 64 columns
    }
  }
}
}  // namespace mid

template <int NST, int DK = GK_DGRAD>
__device__ __forceinline__ void mid_bwd(const GemmDesc& gd, const EpiParams& ed, const GemmDesc& gw,
                                        const EpiParams& ew, int nd, int nw, int first, char* smem) {
  const int b = (int)blockIdx.x - (first ? 0 : nd);
  if (b >= 0 && b < nw)
    mid::wgrad_tile<NST>(gw, ew, b, nw, smem);
  else
    mid::nt_tile<NST, DK>(gd, ed, first ? b - nw : (int)blockIdx.x, nd, smem);
}

template <int NST, int KIND>
__global__ __launch_bounds__(mid::NT) void erase_mid_nt(GemmDesc g, EpiParams e, int ntiles) {
  __shared__ __attribute__((aligned(16))) char smem[mid::bytes<NST>()];
  mid::nt_tile<NST, KIND>(g, e, (int)blockIdx.x, ntiles, smem);
}
template <int NST>
__global__ __launch_bounds__(mid::NT) void erase_mid_wgrad(GemmDesc g, EpiParams e, int ntiles) {
  __shared__ __attribute__((aligned(16))) char smem[mid::bytes<NST>()];
  mid::wgrad_tile<NST>(g, e, (int)blockIdx.x, ntiles, smem);
}
// Both backward GEMMs of a layer, the longer contraction first (`first`: the
// weight gradient's).
template <int NST, int DK>
__global__ __launch_bounds__(mid::NT) void erase_mid_bwd(GemmDesc gd, EpiParams ed, GemmDesc gw, EpiParams ew, int nd,
                                                         int nw, int first) {
  __shared__ __attribute__((aligned(16))) char smem[mid::bytes<NST>()];
  mid_bwd<NST, DK>(gd, ed, gw, ew, nd, nw, first, smem);
}
// the same for several blocks (grid row j: job j)
template <int NST, int KIND>
__global__ __launch_bounds__(mid::NT) void erase_mid_nt_b(const BlockJob* jobs, StepPtrs st, int ntiles) {
  __shared__ __attribute__((aligned(16))) char smem[mid::bytes<NST>()];
  GemmDesc g;
  EpiParams e;
  const cmem_t jb = job_of(jobs);
  ld_gemm(jb + offsetof(BlockJob, g), g, st);
  ld_epi(jb + offsetof(BlockJob, e), e, st);
  mid::nt_tile<NST, KIND>(g, e, (int)blockIdx.x, ntiles, smem);
}
template <int NST>
__global__ __launch_bounds__(mid::NT) void erase_mid_wgrad_b(const BlockJob* jobs, StepPtrs st, int ntiles) {
  __shared__ __attribute__((aligned(16))) char smem[mid::bytes<NST>()];
  GemmDesc g;
  EpiParams e;
  const cmem_t jb = job_of(jobs);
  ld_gemm(jb + offsetof(BlockJob, g), g, st);
  ld_epi(jb + offsetof(BlockJob, e), e, st);
  mid::wgrad_tile<NST>(g, e, (int)blockIdx.x, ntiles, smem);
}
template <int NST>
__global__ __launch_bounds__(mid::NT) void erase_mid_bwd_b(const BlockJob* jobs, StepPtrs st, int nd, int nw, int first) {
  __shared__ __attribute__((aligned(16))) char smem[mid::bytes<NST>()];
  GemmDesc gd, gw;
  EpiParams ed, ew;
  const cmem_t jb = job_of(jobs);
  ld_gemm(jb + offsetof(BlockJob, g), gd, st);
  ld_epi(jb + offsetof(BlockJob, e), ed, st);
  ld_gemm(jb + offsetof(BlockJob, g2), gw, st);
  ld_epi(jb + offsetof(BlockJob, e2), ew, st);
  mid_bwd<NST>(gd, ed, gw, ew, nd, nw, first, smem);
}

template <int KIND>
__device__ __forceinline__ void wide_nt(const GemmDesc& g, const EpiParams& e, int t, int ntiles, char* smem) {
  wide::run<false>(g, t, ntiles, false, smem,
                   [&](const auto& acc, const auto&, const TileIdx& ti, bool, int wm, int wn, int fr, int fg) {
                     wide::epi_nt<KIND>(e, acc, g.M, g.N, ti, wm, wn, fr, fg);
                   });
}
__device__ __forceinline__ void wide_wgrad(const GemmDesc& g, const EpiParams& e, int t, int ntiles, char* smem) {
  wide::run<true>(g, t, ntiles, e.bpart != nullptr, smem,
                  [&](const auto& acc, const auto& accr, const TileIdx& ti, bool rows, int wm, int wn, int fr, int fg) {
                    wide::epi_wgrad(e, acc, accr, g.M, g.N, ti, rows, wm, wn, fr, fg);
                  });
}
// Both backward GEMMs of a layer.  The workgroups of the longer contraction
// come first (`first`: the weight gradient's).
__device__ __forceinline__ void wide_bwd(const GemmDesc& gd, const EpiParams& ed, const GemmDesc& gw,
                                         const EpiParams& ew, int nd, int nw, int first, char* smem) {
  const int b = (int)blockIdx.x - (first ? 0 : nd);
  if (b >= 0 && b < nw)
    wide_wgrad(gw, ew, b, nw, smem);
  else
    wide_nt<GK_DGRAD>(gd, ed, first ? b - nw : (int)blockIdx.x, nd, smem);
}

template <int KIND>
__global__ __launch_bounds__(wide::NT) void erase_wide_nt(GemmDesc g, EpiParams e, int ntiles) {
  __shared__ __attribute__((aligned(16))) char smem[wide::BYTES];
  wide_nt<KIND>(g, e, (int)blockIdx.x, ntiles, smem);
}
__global__ __launch_bounds__(wide::NT) void erase_wide_wgrad(GemmDesc g, EpiParams e, int ntiles) {
  __shared__ __attribute__((aligned(16))) char smem[wide::BYTES];
  wide_wgrad(g, e, (int)blockIdx.x, ntiles, smem);
}
__global__ __launch_bounds__(wide::NT) void erase_wide_bwd(GemmDesc gd, EpiParams ed, GemmDesc gw, EpiParams ew, int nd,
                                                           int nw, int first) {
  __shared__ __attribute__((aligned(16))) char smem[wide::BYTES];
  wide_bwd(gd, ed, gw, ew, nd, nw, first, smem);
}
// the same for several blocks (grid row j: job j)
template <int KIND>
__global__ __launch_bounds__(wide::NT) void erase_wide_nt_b(const BlockJob* jobs, StepPtrs st, int ntiles) {
  __shared__ __attribute__((aligned(16))) char smem[wide::BYTES];
  GemmDesc g;
  EpiParams e;
  const cmem_t jb = job_of(jobs);
  ld_gemm(jb + offsetof(BlockJob, g), g, st);
  ld_epi(jb + offsetof(BlockJob, e), e, st);
  wide_nt<KIND>(g, e, (int)blockIdx.x, ntiles, smem);
}
__global__ __launch_bounds__(wide::NT) void erase_wide_wgrad_b(const BlockJob* jobs, StepPtrs st, int ntiles) {
  __shared__ __attribute__((aligned(16))) char smem[wide::BYTES];
  GemmDesc g;
  EpiParams e;
  const cmem_t jb = job_of(jobs);
  ld_gemm(jb + offsetof(BlockJob, g), g, st);
  ld_epi(jb + offsetof(BlockJob, e), e, st);
  wide_wgrad(g, e, (int)blockIdx.x, ntiles, smem);
}
__global__ __launch_bounds__(wide::NT) void erase_wide_bwd_b(const BlockJob* jobs, StepPtrs st, int nd, int nw, int first) {
  __shared__ __attribute__((aligned(16))) char smem[wide::BYTES];
  GemmDesc gd, gw;
  EpiParams ed, ew;
  const cmem_t jb = job_of(jobs);
  ld_gemm(jb + offsetof(BlockJob, g), gd, st);
  ld_epi(jb + offsetof(BlockJob, e), ed, st);
  ld_gemm(jb + offsetof(BlockJob, g2), gw, st);
  ld_epi(jb + offsetof(BlockJob, e2), ew, st);
  wide_bwd(gd, ed, gw, ew, nd, nw, first, smem);
}

#define ERASE_WIDE(ONE, MANY)                                          \
  if (bt)                                                             \
    ERASE_LAUNCH(MANY, grid, block, 0, s, ev, bt->jobs, bt->st, nt);   \
  else                                                                \
    ERASE_LAUNCH(ONE, grid, block, 0, s, ev, g, e, nt)

static hipError_t launch_256(int kind, const GemmDesc& g, const EpiParams& e, hipStream_t s, const LaunchEv& ev,
                             const Batch* bt) {
  const int nt = (int)wide_tiles(g.M, g.N) * g.split;
  const dim3 grid((unsigned)nt, bt ? (unsigned)bt->n : 1u), block(wide::NT);
  switch (kind) {
    case GK_FWD_RELU: ERASE_WIDE((erase_wide_nt<GK_FWD_RELU>), (erase_wide_nt_b<GK_FWD_RELU>)); break;
    case GK_FWD_CROSS: ERASE_WIDE((erase_wide_nt<GK_FWD_CROSS>), (erase_wide_nt_b<GK_FWD_CROSS>)); break;
    case GK_DGRAD: ERASE_WIDE((erase_wide_nt<GK_DGRAD>), (erase_wide_nt_b<GK_DGRAD>)); break;
    case GK_WGRAD: ERASE_WIDE(erase_wide_wgrad, erase_wide_wgrad_b); break;
    case GK_FWD_LIN: ERASE_LAUNCH((erase_wide_nt<GK_FWD_LIN>), grid, block, 0, s, ev, g, e, nt); break;
    case GK_FWD_GELU: ERASE_LAUNCH((erase_wide_nt<GK_FWD_GELU>), grid, block, 0, s, ev, g, e, nt); break;
    case GK_DGRAD_GELU: ERASE_LAUNCH((erase_wide_nt<GK_DGRAD_GELU>), grid, block, 0, s, ev, g, e, nt); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// 128x128 tiles: three stages for launches of at most one workgroup per
// compute unit, else two (two workgroups per unit).  4096 x 512 x 1677 (128
// tiles) 16.2 and 16.4 us, 8192 rows (256) 18.3 and 22.2, 24576 (768) 50.0
// and 47.3, 16384 x 512 x 2048 (512) 38.5 and 34.1 us; four stages were
// never faster than three.
template <int NST>
static hipError_t launch_128_t(int kind, const GemmDesc& g, const EpiParams& e, hipStream_t s, const LaunchEv& ev,
                               const Batch* bt) {
  const int nt = (int)mid_tiles(g.M, g.N) * g.split;
  const dim3 grid((unsigned)nt, bt ? (unsigned)bt->n : 1u), block(mid::NT);
  switch (kind) {
    case GK_FWD_RELU: ERASE_WIDE((erase_mid_nt<NST, GK_FWD_RELU>), (erase_mid_nt_b<NST, GK_FWD_RELU>)); break;
    case GK_FWD_CROSS: ERASE_WIDE((erase_mid_nt<NST, GK_FWD_CROSS>), (erase_mid_nt_b<NST, GK_FWD_CROSS>)); break;
    case GK_DGRAD: ERASE_WIDE((erase_mid_nt<NST, GK_DGRAD>), (erase_mid_nt_b<NST, GK_DGRAD>)); break;
    case GK_WGRAD: ERASE_WIDE((erase_mid_wgrad<NST>), (erase_mid_wgrad_b<NST>)); break;
    case GK_FWD_LIN: ERASE_LAUNCH((erase_mid_nt<NST, GK_FWD_LIN>), grid, block, 0, s, ev, g, e, nt); break;
    case GK_FWD_GELU: ERASE_LAUNCH((erase_mid_nt<NST, GK_FWD_GELU>), grid, block, 0, s, ev, g, e, nt); break;
    case GK_DGRAD_GELU: ERASE_LAUNCH((erase_mid_nt<NST, GK_DGRAD_GELU>), grid, block, 0, s, ev, g, e, nt); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
#undef ERASE_WIDE

static GemmDesc with_order(const GemmDesc& g0) {
  GemmDesc g = g0;
  if (g.group <= 0) g.group = xcd_group((g.M + g.bm - 1) / g.bm, (g.N + g.bn - 1) / g.bn, g.split, g.bm, g.bn);
  return g;
}
static bool operands_ok(const GemmDesc& g) { return g.K % 64 == 0 && g.kps > 0 && g.kps % 64 == 0 && g.lda % 8 == 0 && g.ldb % 8 == 0; }

hipError_t launch_wide(int kind, const GemmDesc& g0, const EpiParams& e, hipStream_t s, const LaunchEv& ev,
                       const Batch* bt) {
  const GemmDesc g = with_order(g0);
  if (!operands_ok(g) || (kind != GK_WGRAD && g.split != 1)) return hipErrorInvalidValue;
  if (bt && (kind == GK_FWD_LIN || kind == GK_FWD_GELU || kind == GK_DGRAD_GELU)) return hipErrorInvalidValue;
  if (g.bm == 256 && g.bn == 256) return launch_256(kind, g, e, s, ev, bt);
  if (g.bm != 128 || g.bn != 128) return hipErrorInvalidValue;
  if (mid_tiles(g.M, g.N) * g.split * (bt ? bt->n : 1) <= kWideCus) return launch_128_t<3>(kind, g, e, s, ev, bt);
  return launch_128_t<2>(kind, g, e, s, ev, bt);
}

hipError_t launch_wide_bwd(const GemmDesc& gd, const EpiParams& ed, const GemmDesc& gw, const EpiParams& ew,
                           hipStream_t s, const LaunchEv& ev, const Batch* bt) {
  const GemmDesc d = with_order(gd), w = with_order(gw);
  if (!operands_ok(d) || !operands_ok(w) || d.bm != w.bm || d.bn != w.bn || d.bm != d.bn)
    return hipErrorInvalidValue;
  // an input gradient in fp32 slices (the vocabulary head's, in 128x128 tiles), else whole
  const bool big = d.bm == 256, part = ed.part != nullptr;
  if (!big && d.bm != 128) return hipErrorInvalidValue;
  if (part ? (big || bt || d.split < 1 || (int64_t)d.split * d.kps < d.K || d.N % 64) : (d.split != 1 || d.kps < d.K))
    return hipErrorInvalidValue;
  const int nd = (int)(big ? wide_tiles(d.M, d.N) : mid_tiles(d.M, d.N)) * d.split;
  const int nw = (int)(big ? wide_tiles(w.M, w.N) : mid_tiles(w.M, w.N)) * w.split;
  const dim3 grid((unsigned)(nd + nw), bt ? (unsigned)bt->n : 1u), block(512);
  const int first = w.kps >= std::min(d.K, d.kps) ? 1 : 0;
#define ERASE_MID_BWD(NST)                                                                                   \
  do {                                                                                                       \
    if (bt)                                                                                                  \
      ERASE_LAUNCH((erase_mid_bwd_b<NST>), grid, block, 0, s, ev, bt->jobs, bt->st, nd, nw, first);           \
    else if (part)                                                                                           \
      ERASE_LAUNCH((erase_mid_bwd<NST, GK_DGRAD_PART>), grid, block, 0, s, ev, d, ed, w, ew, nd, nw, first);   \
    else                                                                                                     \
      ERASE_LAUNCH((erase_mid_bwd<NST, GK_DGRAD>), grid, block, 0, s, ev, d, ed, w, ew, nd, nw, first);        \
  } while (0)
  if (big && bt)
    ERASE_LAUNCH(erase_wide_bwd_b, grid, block, 0, s, ev, bt->jobs, bt->st, nd, nw, first);
  else if (big)
    ERASE_LAUNCH(erase_wide_bwd, grid, block, 0, s, ev, d, ed, w, ew, nd, nw, first);
  else if ((int64_t)grid.x * grid.y <= kWideCus)
    ERASE_MID_BWD(3);
  else
    ERASE_MID_BWD(2);
#undef ERASE_MID_BWD
  return hipGetLastError();
}

}  // namespace erase
