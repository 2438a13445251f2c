// Embedding-bag input stage of the CTR workload, written for gfx950.
//
// x[m] = [ log1p(dense[m][0 .. n_dense)) |  sum over the bag of table 0 |
//          ... | sum over the bag of table T-1 | zeros up to x_ld ]
//
// Each bag is summed in fp32 in the order of its index list.  A wave pools
// 64 / G bags at once: G = dim / 4 (rounded up to a power of two) lanes per
// bag, each lane one 16-byte column chunk, so every row load is one
// contiguous, coalesced read of the row.  The lanes of a bag read its ids
// together, one id per lane, and pass them round by lane shifts; up to 8 rows
// per bag are in flight before they are added.  Out-of-range offsets or
// indices read nothing: they contribute zero and set the status word.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>

#include "erase.h"
#include "internal.h"

namespace erase {

// Scratch of erase_embed_bags_backward_noalloc: one array per GPU, created
// with the code object on that GPU and held until the process ends.  In host
// code `scratch` names a host-side stand-in; kernels get its device address
// from bag_scratch_device_ptr().
static __device__ __align__(256) char scratch[ERASE_BAG_SCRATCH_MAX];

hipError_t bag_scratch_device_ptr(void** ptr, size_t* bytes) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  *bytes = sizeof(scratch);
  return hipSuccess;
}

typedef float f32x4e_t __attribute__((ext_vector_type(4)));
// output columns start after the dense features, so stores are aligned only
// to the element size (gfx950 serves unaligned vector accesses)
typedef float f32x4s_t __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2s_t __attribute__((ext_vector_type(2), aligned(2)));

__device__ __forceinline__ uint16_t bag_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// The stage is bound by the row gathers: 286 MB of rows for 4096 rows of 26
// bags of 1..20 ids, most of them hits of the hot rows.  Workgroups are dealt
// out to the 8 XCDs in turn, so XCD x is given the x-th eighth of the bags,
// table after table: its L2 holds the hot rows of its own tables instead of a
// share of everyone's (44.8 -> 37.7 us).  At most 64 VGPRs, so that eight waves
// share a SIMD: 27.4 us.
template <typename T, int G>
__global__ __launch_bounds__(256, 8) void erase_embed_bags_k(EmbedArgs a, uint32_t chunk) {
  constexpr int BPW = 64 / G;               // bags per wave
  constexpr int IPL = G >= 8 ? 1 : 8 / G;   // ids per lane and round
  constexpr int CH = G * IPL;               // ids of a bag per round
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane / G, q = lane % G;  // bag of this lane within the wave, column chunk
  const uint32_t wg = (blockIdx.x & 7u) * chunk + (blockIdx.x >> 3);
  const int64_t bag0 = (int64_t)wg * 4 * BPW;  // uniform: the workgroup's first bag
  const int64_t nbags = (int64_t)a.M * a.T;    // < 2^31
  const bool live = bag0 + wave * BPW + g < nbags;
  const uint32_t bag = live ? (uint32_t)bag0 + wave * BPW + g : 0u;
  const int t = (int)(bag / (uint32_t)a.M), m = (int)(bag - (uint32_t)t * (uint32_t)a.M);
  const bool col = live && 4 * q < a.dim;

  int64_t beg = 0, end = 0;
  bool bad = false;
  if (live) {
    beg = a.offsets[(int64_t)t * (a.M + 1) + m];
    end = a.offsets[(int64_t)t * (a.M + 1) + m + 1];
    if (!(beg >= 0 && beg <= end && end <= a.nnz)) {
      bad = true;
      beg = end = 0;
    }
  }
  const int n = (int)(end - beg);
  const float* tab = a.tables + (int64_t)t * a.rows * a.dim + 4 * q;
  f32x4e_t acc = {0.f, 0.f, 0.f, 0.f};
  // the longest bag of the wave bounds the loop; shorter bags idle
  int nmax = n;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) nmax = max(nmax, __shfl_xor(nmax, o, 64));
  for (int j0 = 0; j0 < nmax; j0 += CH) {
    int32_t id[IPL];  // ids j0 + q + G i; -1: none, or out of range
#pragma unroll
    for (int i = 0; i < IPL; ++i) {
      const int j = j0 + q + G * i;
      id[i] = -1;
      if (j < n) {
        id[i] = a.indices[beg + j];
        if (id[i] < 0 || id[i] >= a.rows) {
          bad = true;
          id[i] = -1;
        }
      }
    }
#pragma unroll 1
    for (int u0 = 0; u0 < CH && j0 + u0 < nmax; u0 += 8) {
      f32x4e_t v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        // with fewer than 8 lanes per bag a round has exactly 8 ids
        const int32_t r = __shfl(id[IPL > 1 ? u / G : 0], g * G + (IPL > 1 ? u % G : u0 + u), 64);
        v[u] = f32x4e_t{0.f, 0.f, 0.f, 0.f};
        if (col && r >= 0) v[u] = *reinterpret_cast<const f32x4e_t*>(tab + (int64_t)r * a.dim);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (j0 + u0 + u < n) acc += v[u];  // in index order
    }
  }
  if (bad && a.status) a.status[0] = 1;
  if (col) {
    T* dst = static_cast<T*>(a.x) + (int64_t)m * a.ldx + a.n_dense + (int64_t)t * a.dim + 4 * q;
    if constexpr (sizeof(T) == 2) {
      const uint32_t lo = (uint32_t)bag_bf16(acc[0]) | ((uint32_t)bag_bf16(acc[1]) << 16);
      const uint32_t hi = (uint32_t)bag_bf16(acc[2]) | ((uint32_t)bag_bf16(acc[3]) << 16);
      *reinterpret_cast<u32x2s_t*>(dst) = u32x2s_t{lo, hi};
    } else {
      *reinterpret_cast<f32x4s_t*>(dst) = f32x4s_t{acc[0], acc[1], acc[2], acc[3]};
    }
  }
  // the lanes of a row's first table also write its dense features and the
  // zero padding beyond the pooled columns
  if (live && t == 0) {
    T* row = static_cast<T*>(a.x) + (int64_t)m * a.ldx;
    for (int j = q; j < a.n_dense; j += G) {
      const float d = log1pf(a.dense[(int64_t)m * a.n_dense + j]);
      if constexpr (sizeof(T) == 2)
        row[j] = bag_bf16(d);
      else
        row[j] = d;
    }
    const int64_t k0 = a.n_dense + (int64_t)a.T * a.dim;
    for (int64_t k = k0 + q; k < a.ldx; k += G) row[k] = T(0);
  }
}

hipError_t launch_embed_bags(int bf16, const EmbedArgs& a, hipStream_t s) {
  const int c = (a.dim + 3) / 4;
  int G = 1;
  while (G < c) G *= 2;
  const int64_t nbags = (int64_t)a.M * a.T;
  const int64_t per_wg = 4 * (64 / G);
  const uint32_t chunk = (uint32_t)(((nbags + per_wg - 1) / per_wg + 7) / 8);  // workgroups per XCD
  dim3 grid(8 * chunk), block(256);
#define ERASE_BAGS(GG)                                                                     \
  case GG:                                                                                 \
    if (bf16)                                                                              \
      hipLaunchKernelGGL((erase_embed_bags_k<uint16_t, GG>), grid, block, 0, s, a, chunk);        \
    else                                                                                   \
      hipLaunchKernelGGL((erase_embed_bags_k<float, GG>), grid, block, 0, s, a, chunk);           \
    break;
  switch (G) {
    ERASE_BAGS(1)
    ERASE_BAGS(2)
    ERASE_BAGS(4)
    ERASE_BAGS(8)
    ERASE_BAGS(16)
    ERASE_BAGS(32)
    ERASE_BAGS(64)
    default: return hipErrorInvalidValue;
  }
#undef ERASE_BAGS
  return hipGetLastError();
}

constexpr int kLightBucket = 4;   // entries a lane group sums
constexpr int kSmallBucket = 64;  // entries a wave sorts in its registers
constexpr int kWaveBucket = 512;  // entries a wave sorts where many rows have over kSmallBucket
constexpr int kSortCap = 16384;   // entries held in LDS at a time (64 KB)
// A workgroup takes about 7 us for a row, however short (a chain of sorts, scans
// and barriers), and 256 of them run at a time; a wave takes longer for rows of
// over kSmallBucket entries, but 4096 run.  So beyond two rows per workgroup the
// rows of up to kWaveBucket entries go to waves.  The whole backward of 26 tables
// of 4096 bags of 1..20 ids, dim 64, with a workgroup for every such row and so:
// 500 rows (83 entries each) 446 and 116 us, 300 rows 300 and 103, 100 rows (430
// entries) 164 and 112, 1000 rows with Zipf ids 210 and 168.  With waves
// always, 4 tables of 512 bags, 1000 rows (44 such rows) took 63 instead of 42.
constexpr int kFewRows = 512;

// ---------------------------------------------------------------------------
// Backward: table gradients from the gradient at x.  Entry i (an index
// position) belongs to the bag (t, m) whose range holds it; its global row
// is t * rows + indices[i].  Entries are bucketed by global row (counts,
// a place for each bucket, then each entry to its slot), every bucket is put
// in increasing entry order, and each row is summed in a fixed order of its
// entries, so the result does not depend on scheduling:
//  * rows of at most 4 entries: one lane group of G lanes (4 columns each);
//  * rows of 5..64 entries: one wave; entries sorted across its lanes,
//    entry k to lane group k mod (64/G), each group adding its entries in
//    order, the groups then combined by a fixed butterfly;
//  * rows of 65..512 entries, where more than kFewRows rows have over 64: one
//    wave in the same way, its entries in LDS;
//  * larger rows, and those where they are few: one workgroup of 1024
//    threads; entries put in order in LDS (a bitmap over their range, a
//    bitonic sort, or above 16384 entries one bitmap after another), entry
//    k to lane group k mod (1024/G), the groups of a wave then combined by a
//    fixed butterfly and the 16 waves' partial rows added in order;
//  * rows no entry selects: zero.
// One launch does them all (erase_bags_bwd_sums).  The buckets of rows that a
// wave sums hold the entries' bag rows m, the larger ones the entries:
// within a table a later entry never has a smaller m, so the order is the
// same.
//
// Workgroups are dealt out to the 8 XCDs in turn; the passes over entries and
// over table rows give XCD x the x-th eighth of their range, so that the
// counters, places and buckets of a table stay in one XCD's L2.
// ---------------------------------------------------------------------------
// Workgroup of the x-th eighth of n (at most n + 7 launched: results >= n do nothing)
__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t n) { return (b & 7u) * ((n + 7) / 8) + (b >> 3); }

__global__ __launch_bounds__(256) void erase_bags_bwd_clear(EmbedBwdArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i == 0) {
    a.nlarge[0] = 0;  // rows of more than kSmallBucket entries
    a.nlarge[1] = 0;  // rows listed in large: more entries than wave_bucket()
    a.nlarge[2] = 0;  // entries with a place in a bucket
    a.nlarge[3] = 0;  // rows listed in mid: kLightBucket + 1..wave_bucket() entries
  }
  if (i < a.trows) a.count[i] = 0;
  if (i < a.nnz) a.owner[i] = -1;
}

// one thread per bag: its entries' owner
__global__ __launch_bounds__(256) void erase_bags_bwd_owner(EmbedBwdArgs a) {
  const int64_t nbags = (int64_t)a.M * a.T;  // < 2^31
  const int64_t bag = (int64_t)xcd_block(blockIdx.x, (uint32_t)((nbags + 255) / 256)) * 256 + threadIdx.x;
  if (bag >= nbags) return;
  const int t = (int)((uint32_t)bag / (uint32_t)a.M), m = (int)((uint32_t)bag % (uint32_t)a.M);
  const int64_t beg = a.offsets[(int64_t)t * (a.M + 1) + m], end = a.offsets[(int64_t)t * (a.M + 1) + m + 1];
  if (!(beg >= 0 && beg <= end && end <= a.nnz)) {
    if (a.status) a.status[0] = 1;
    return;
  }
  for (int64_t i = beg; i < end; ++i) a.owner[i] = (int32_t)bag;
}

// Each entry's global row, and its slot in the row's bucket.  A workgroup
// takes kCountTile entries (kCountPer per thread) and first counts their
// rows in an LDS hash table, so each row it holds takes one addition to its
// global counter per workgroup (Zipf-hot rows occur in most workgroups, and
// the additions to one counter are serialised).  Slots need only be distinct
// within a bucket (every bucket is sorted by entry before it is summed): an
// entry's slot is its row's base from that addition plus its rank from the
// LDS count.
constexpr int kCountPer = 8, kCountTile = 256 * kCountPer, kHashSlots = 2 * kCountTile;
__global__ __launch_bounds__(256) void erase_bags_bwd_count(EmbedBwdArgs a) {
  __shared__ int32_t hkey[kHashSlots];  // global row, -1: empty
  __shared__ int32_t hval[kHashSlots];  // the row's entries in this tile, then its base
  const int tid = threadIdx.x;
  for (int h = tid; h < kHashSlots; h += 256) {
    hkey[h] = -1;
    hval[h] = 0;
  }
  __syncthreads();
  const uint32_t tile = xcd_block(blockIdx.x, (uint32_t)((a.nnz + kCountTile - 1) / kCountTile));
  const int64_t i0 = (int64_t)tile * kCountTile + tid;
  int32_t gid[kCountPer], hs[kCountPer], rk[kCountPer];
#pragma unroll
  for (int u = 0; u < kCountPer; ++u) {
    const int64_t i = i0 + u * 256;
    gid[u] = -1;
    hs[u] = 0;
    rk[u] = 0;
    if (i < a.nnz) {
      const int32_t o = a.owner[i];
      if (o >= 0) {
        const int32_t r = a.indices[i];
        if (r >= 0 && r < a.rows) {
          gid[u] = (int32_t)((o / a.M) * a.rows + r);
        } else if (a.status) {
          a.status[0] = 1;
        }
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kCountPer; ++u) {
    if (gid[u] < 0) continue;
    // open addressing: at most kCountTile keys in 2 kCountTile slots
    int h = (int)(((uint32_t)gid[u] * 0x9E3779B1u) >> 20) & (kHashSlots - 1);
    while (true) {
      const int32_t prev = atomicCAS(&hkey[h], -1, gid[u]);
      if (prev == -1 || prev == gid[u]) break;
      h = (h + 1) & (kHashSlots - 1);
    }
    hs[u] = h;
    rk[u] = atomicAdd(&hval[h], 1);
  }
  __syncthreads();
  // the additions of a thread's slots in flight together: the whole backward of
  // 3 tables of 5000 x 16 and 200 rows 30 us, against 36 one after another
  // (equal on the CTR shape, where the counters' memory bounds them)
  constexpr int kSlotPer = kHashSlots / 256;
  int32_t key[kSlotPer], cnt[kSlotPer], base[kSlotPer];
#pragma unroll
  for (int u = 0; u < kSlotPer; ++u) {
    key[u] = hkey[tid + 256 * u];
    cnt[u] = hval[tid + 256 * u];
  }
#pragma unroll
  for (int u = 0; u < kSlotPer; ++u) base[u] = key[u] >= 0 ? atomicAdd(&a.count[key[u]], cnt[u]) : 0;
  int over = 0;  // rows whose count passes kSmallBucket: exactly one addition to each crosses it
#pragma unroll
  for (int u = 0; u < kSlotPer; ++u) {
    over += __popcll(__ballot(key[u] >= 0 && base[u] <= kSmallBucket && base[u] + cnt[u] > kSmallBucket));
    if (key[u] >= 0) hval[tid + 256 * u] = base[u];
  }
  if ((tid & 63) == 0 && over) atomicAdd(a.nlarge, over);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kCountPer; ++u) {
    const int64_t i = i0 + u * 256;
    if (i < a.nnz) {
      a.gid[i] = gid[u];
      a.slot[i] = gid[u] >= 0 ? hval[hs[u]] + rk[u] : 0;
    }
  }
}

// Most entries of a row that a wave sums (known once the rows are counted).
__device__ __forceinline__ int wave_bucket(const EmbedBwdArgs& a) {
  return a.nlarge[0] > kFewRows ? kWaveBucket : kSmallBucket;
}

// A place for every bucket, the list of the rows of kLightBucket + 1 ..
// wave_bucket() entries and that of the larger ones: a workgroup scans the
// counts and the flags of kScanBlock rows and takes its room behind the counters
// with one 64-bit addition (two additions: 21 us at 2.6 M rows, they wait for
// one another) and, where it has larger rows, one more.  Which workgroup comes
// first changes where a bucket lies and the order of the lists, but no row's sum.
constexpr int kScanBlock = 4096;  // 256 threads x 16 rows

__device__ __forceinline__ int block_exclusive_scan(int v, int* part) {
  // exclusive scan of one value per thread over 256 threads: inclusive scans
  // within the waves (lane shifts), then the wave totals through LDS
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) part[w] = x;
  __syncthreads();
  int base = 0;
  for (int k = 0; k < w; ++k) base += part[k];
  __syncthreads();
  return base + x - v;
}

// a thread's 16 consecutive rows: four 16-byte accesses when all exist
__device__ __forceinline__ void load16(const int32_t* p, int64_t base, int64_t n, int v[16]) {
  if (base + 16 <= n) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int4 x = reinterpret_cast<const int4*>(p + base)[q];
      v[4 * q] = x.x;
      v[4 * q + 1] = x.y;
      v[4 * q + 2] = x.z;
      v[4 * q + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = base + k < n ? p[base + k] : 0;
  }
}
__device__ __forceinline__ void store16(int32_t* p, int64_t base, int64_t n, const int v[16]) {
  if (base + 16 <= n) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      reinterpret_cast<int4*>(p + base)[q] = make_int4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
  } else {
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (base + k < n) p[base + k] = v[k];
  }
}

__global__ __launch_bounds__(256) void erase_bags_bwd_place(EmbedBwdArgs a) {
  __shared__ int part[4];
  __shared__ int room[3];
  const uint32_t part_of = xcd_block(blockIdx.x, (uint32_t)((a.trows + kScanBlock - 1) / kScanBlock));
  const int64_t base = (int64_t)part_of * kScanBlock + threadIdx.x * 16;
  int v[16], st[16], s = 0, f = 0;
  load16(a.count, base, a.trows, v);
  const int wb = wave_bucket(a);
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    s += v[k];
    f += v[k] > wb ? 0x10000 : v[k] > kLightBucket ? 1 : 0;  // at most 4096 of either in a workgroup
  }
  const int sx = block_exclusive_scan(s, part), fx = block_exclusive_scan(f, part);
  if (threadIdx.x == 255) {
    // both counters stay below 2^31: no carry from the low one
    const int nm = (fx + f) & 0xffff;
    const unsigned long long r = atomicAdd(reinterpret_cast<unsigned long long*>(a.nlarge + 2),
                                           ((unsigned long long)(uint32_t)nm << 32) | (uint32_t)(sx + s));
    room[0] = (int)(uint32_t)r;
    room[1] = (int)(uint32_t)(r >> 32);
  } else if (threadIdx.x == 0) {  // another wave: at the same time; part[] holds the waves' flags
    const int nl = (part[0] + part[1] + part[2] + part[3]) >> 16;
    room[2] = nl ? atomicAdd(a.nlarge + 1, nl) : 0;
  }
  __syncthreads();
  int run = room[0] + sx, pos = room[1] + (fx & 0xffff), lpos = room[2] + (fx >> 16);
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    st[k] = run;
    run += v[k];
    if (v[k] > wb)
      a.large[lpos++] = (int32_t)(base + k);
    else if (v[k] > kLightBucket)
      a.mid[pos++] = (int32_t)(base + k);
  }
  store16(a.start, base, a.trows, st);
}

// one thread per entry: into its slot of its row's bucket (no atomics)
__global__ __launch_bounds__(256) void erase_bags_bwd_scatter(EmbedBwdArgs a) {
  const int64_t i = (int64_t)xcd_block(blockIdx.x, (uint32_t)((a.nnz + 255) / 256)) * 256 + threadIdx.x;
  if (i >= a.nnz) return;
  const int32_t gid = a.gid[i];
  if (gid >= 0) {
    const int32_t m = (int32_t)((uint32_t)a.owner[i] % (uint32_t)a.M);
    const int c = a.count[gid], to = a.start[gid] + a.slot[i];
    a.bucket[to] = c <= kSmallBucket || c <= wave_bucket(a) ? m : (int32_t)i;
  }
}

// 4 consecutive dx columns of bag row m, as fp32
template <typename T>
__device__ __forceinline__ float4 dx4(const EmbedBwdArgs& a, int m, int64_t xc) {
  const T* src = static_cast<const T*>(a.dx) + (int64_t)m * a.lddx + xc;
  if constexpr (sizeof(T) == 2) {
    const u32x2s_t w = *reinterpret_cast<const u32x2s_t*>(src);
    return make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                       __uint_as_float(w.y & 0xffff0000u));
  } else {
    const f32x4s_t v = *reinterpret_cast<const f32x4s_t*>(src);
    return make_float4(v[0], v[1], v[2], v[3]);
  }
}
__device__ __forceinline__ void add4(float4& a, const float4& b) {
  a.x += b.x;
  a.y += b.y;
  a.z += b.z;
  a.w += b.w;
}

// A bucket of more than wave_bucket() entries: the workgroup's NT threads put its
// entries in order in LDS, turn them into their bag rows, and sum the row: lane
// group q (G lanes, 4 columns each) takes entries q, q + NT / G, ... in order,
// the groups of a wave are combined by a fixed butterfly and the waves'
// partial rows added in order.  Up to kSortCap entries are sorted at once: a
// bitmap over the bucket's entry range when it spans at most 32 kBitWords
// entries, as on the CTR shape, else a bitonic sort.  Larger buckets take the
// bitmap over one range of 32 kBitWords entries after another (each from the
// first entry past the last, so every pass over the bucket lists some), and
// sum each range kSortCap entries at a time.
constexpr int kSumThreads = 1024;
constexpr int kBitWords = 2048;  // bitmap of the bitmap sort: buckets whose entries span <= 64 Ki

// The lane, opaque: else the lane shifts' indexes are kept over the rows of a
// workgroup, more of them than registers.
__device__ __forceinline__ int opaque_lane() {
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  return lane;
}
__device__ __forceinline__ int32_t lane_read(int32_t v, int lane) { return __builtin_amdgcn_ds_bpermute(lane << 2, v); }
// Minimum over the NT threads of a workgroup (every thread gets it).
template <int NT>
__device__ __forceinline__ int32_t block_min_nt(int32_t v, int32_t* sel) {
  const int lane = opaque_lane();
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = min(v, lane_read(v, lane ^ o));
  if ((threadIdx.x & 63) == 0) sel[threadIdx.x >> 6] = v;
  __syncthreads();
  v = sel[0];
  for (int w = 1; w < NT / 64; ++w) v = min(v, sel[w]);
  __syncthreads();
  return v;
}
// Exclusive prefix sum of one value per thread over the NT threads (and the
// total into *all, when set).
template <int NT>
__device__ __forceinline__ int block_exclusive_scan_nt(int v, int32_t* sel, int* all = nullptr) {
  const int lane = opaque_lane(), w = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = lane_read(x, lane - o);
    if (lane >= o) x += y;
  }
  if (lane == 63) sel[w] = x;
  __syncthreads();
  int base = 0;
  for (int k = 0; k < w; ++k) base += sel[k];
  if (all) {
    *all = base;
    for (int k = w; k < NT / 64; ++k) *all += sel[k];
  }
  __syncthreads();
  return base + x - v;
}
// Adds n bag rows of key[], entries number first .. first + n - 1 of the bucket,
// to the lane groups' sums (entry k to group k mod NG).
template <typename T, int NG>
__device__ __forceinline__ void add_bag_rows(const EmbedBwdArgs& a, const int32_t* key, int first, int n, int q, bool col,
                                             int64_t xc, float4& acc) {
  for (int k0 = (q - first) & (NG - 1); k0 < n; k0 += 8 * NG) {
    float4 v[8];  // all in flight; entries past the end add zero
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = k0 + u * NG;
      v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (k < n && col) v[u] = dx4<T>(a, key[k], xc);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) add4(acc, v[u]);
  }
}
// The row's sum from the lane groups' sums; part: LDS for [NT / 64][4 G] floats.
template <int G>
__device__ __forceinline__ void store_row_sum(const EmbedBwdArgs& a, int32_t g, float4 acc, float* part) {
  const int tid = threadIdx.x, cq = tid % G;
#pragma unroll
  for (int o = G; o < 64; o <<= 1) {
    acc.x += __shfl_xor(acc.x, o, 64);
    acc.y += __shfl_xor(acc.y, o, 64);
    acc.z += __shfl_xor(acc.z, o, 64);
    acc.w += __shfl_xor(acc.w, o, 64);
  }
  __syncthreads();  // the LDS is reused for the partial rows
  if (4 * cq < a.dim && (tid & 63) < G) *reinterpret_cast<float4*>(part + (tid >> 6) * 4 * G + 4 * cq) = acc;
  __syncthreads();
  if (tid < a.dim) {
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < kSumThreads / 64; ++w) sum += part[w * 4 * G + tid];
    a.grad[(int64_t)g * a.dim + tid] = sum;
  }
}

template <typename T, int G>
__device__ __forceinline__ void bag_row_large(const EmbedBwdArgs& a, int32_t g, int32_t* key, uint32_t* bits, int32_t* sel) {
  constexpr int NT = kSumThreads, NG = NT / G;  // lane groups of the workgroup
  const int c = a.count[g];
  const int32_t* bucket = a.bucket + a.start[g];
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int q = tid / G, cq = tid % G;
  const bool col = 4 * cq < a.dim;
  const int64_t xc = a.n_dense + (int64_t)(g / a.rows) * a.dim + 4 * cq;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  // n entries in key[], number `first` and on of the bucket: to their bag rows,
  // in place (each thread its own keys), and those rows to the sums
  auto add = [&](int first, int n) {
    for (int i = tid; i < n; i += 4 * NT) {
      int32_t m[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) m[u] = i + u * NT < n ? a.owner[key[i + u * NT]] % a.M : 0;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i + u * NT < n) key[i + u * NT] = m[u];
    }
    __syncthreads();
    add_bag_rows<T, NG>(a, key, first, n, q, col, xc, acc);
  };
  // the bucket's entry range
  int32_t lo = INT32_MAX, hi = -1;
  for (int i = tid; i < c; i += NT) {
    const int32_t p = bucket[i];
    lo = min(lo, p);
    hi = max(hi, p);
  }
  lo = block_min_nt<NT>(lo, sel);
  hi = -block_min_nt<NT>(-hi, sel);
  constexpr int WIN = 32 * kBitWords;
  if (c <= kSortCap && hi - lo >= WIN) {
    // bitonic sort of the bucket in LDS
    int n2 = 1;
    while (n2 < c) n2 <<= 1;
    for (int i = tid; i < n2; i += 4 * NT) {
      int32_t e[4];  // the loads in flight before the LDS stores
#pragma unroll
      for (int u = 0; u < 4; ++u) e[u] = i + u * NT < c ? bucket[i + u * NT] : INT32_MAX;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i + u * NT < n2) key[i + u * NT] = e[u];
    }
    __syncthreads();
    for (int k = 2; k <= n2; k <<= 1)
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int i = tid; i < n2; i += NT) {
          const int l = i ^ j;
          if (l > i) {
            const int32_t x = key[i], y = key[l];
            if (((i & k) == 0) == (x > y)) {
              key[i] = y;
              key[l] = x;
            }
          }
        }
        __syncthreads();
      }
    add(0, c);
  } else {
    // Bitmap sort (the entries of a bucket are distinct): one bit per entry of
    // the range [lo, lo + WIN), then every thread lists the set bits of its run
    // of words, in order, at its place from a scan of the runs' bit counts:
    // all words at once, or of larger buckets as many as key[] surely holds.
    const int cw = c <= kSortCap ? kBitWords : kSortCap / 32;
    int done = 0;  // entries summed
    int32_t next;  // the first entry past the range
    do {
      const int nw = min(kBitWords, (hi - lo) / 32 + 1);
      for (int w = tid; w < nw; w += NT) bits[w] = 0u;
      __syncthreads();
      next = INT32_MAX;
      for (int i = tid; i < c; i += NT) {
        const int32_t p = bucket[i];
        if (p < lo) continue;
        if (p - lo < WIN)
          atomicOr(&bits[(p - lo) >> 5], 1u << ((p - lo) & 31));
        else
          next = min(next, p);
      }
      __syncthreads();
#pragma unroll 1
      for (int wc = 0; wc < nw; wc += cw) {
        const int we = min(nw, wc + cw), per = (we - wc + NT - 1) / NT;
        const int w0 = min(we, wc + tid * per), w1 = min(we, w0 + per);
        int cnt = 0;
        for (int w = w0; w < w1; ++w) cnt += __popc(bits[w]);
        int n = c;
        int pos = block_exclusive_scan_nt<NT>(cnt, sel, c > kSortCap ? &n : nullptr);  // and key[] is free again
        for (int w = w0; w < w1; ++w)
          for (uint32_t b = bits[w]; b; b &= b - 1u) key[pos++] = lo + 32 * w + (__ffs(b) - 1);
        __syncthreads();
        add(done, n);
        done += n;
      }
    } while (done < c && (lo = block_min_nt<NT>(next, sel)) < INT32_MAX);
  }
  store_row_sum<G>(a, g, acc, reinterpret_cast<float*>(key));
}

// Bitonic sort (ascending) of 64 R values across a wave, value 64 r + lane in
// v[r] of that lane.
template <int R>
__device__ __forceinline__ void wave_sort(int32_t (&v)[R], int lane) {
#pragma unroll
  for (int k = 2; k <= 64 * R; k <<= 1)
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
      if (j >= 64) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int p = r | (j >> 6);
          if (r & (j >> 6)) continue;
          const int32_t lo = min(v[r], v[p]), hi = max(v[r], v[p]);
          const bool up = ((64 * r) & k) == 0;
          v[r] = up ? lo : hi;
          v[p] = up ? hi : lo;
        }
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int32_t o = __shfl_xor(v[r], j, 64);
          const bool lower = (lane & j) == 0, up = ((64 * r + lane) & k) == 0;
          v[r] = (lower == up) ? min(v[r], o) : max(v[r], o);
        }
      }
    }
}

__device__ __forceinline__ void sort2(int32_t& x, int32_t& y) {
  const int32_t lo = min(x, y), hi = max(x, y);
  x = lo;
  y = hi;
}

// 64 consecutive table rows by one wave: zeros for the rows no entry selects,
// then the rows of at most kLightBucket entries (92% of the rows with entries
// on the CTR shape, 73% have one), 64 / G at once, one per lane group: its bag
// rows sorted in registers, the dx slices loaded by the group's lanes, added
// as the wave path associates them: ((0 + v0) + (0 + v1)) + ((0 + v2) + (0 + v3)).
template <typename T, int G>
__device__ __forceinline__ void bag_rows_light(const EmbedBwdArgs& a, int64_t r0) {
  constexpr int NGW = 64 / G;  // lane groups per wave
  const int lane = threadIdx.x & 63;
  const int q = lane / G, cq = lane % G;  // lane group, column quad
  const bool col = 4 * cq < a.dim, in = r0 + lane < a.trows;
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  const int cnt = in ? a.count[r0 + lane] : INT32_MAX;
  const int st = in ? a.start[r0 + lane] : 0;
  const uint64_t some = __ballot(cnt >= 1 && cnt <= kLightBucket);
  if (__ballot(cnt == 0)) {
    for (int r = q; r < 64; r += NGW) {
      // streaming stores: the zeros are not read again by this launch sequence
      typedef float f32x4v_t __attribute__((ext_vector_type(4)));
      if (__shfl(cnt, r, 64) == 0 && col)
        __builtin_nontemporal_store(f32x4v_t{0.f, 0.f, 0.f, 0.f},
                                    reinterpret_cast<f32x4v_t*>(a.grad + (r0 + r) * a.dim + 4 * cq));
    }
  }
  const int n = __popcll(some);
  // lane k gets the lane of the k-th such row (unlisted lanes send to the top end)
  const int below = __popcll(some & ((1ull << lane) - 1));
  const int to = ((some >> lane) & 1) ? below : 63 - (lane - below);
  const int list = __builtin_amdgcn_ds_permute(to << 2, lane);
  for (int k0 = 0; k0 < n; k0 += NGW) {
    const bool has = k0 + q < n;
    const int r = __shfl(list, has ? k0 + q : 0, 64);
    const int cs = __shfl(cnt, r, 64), ss = __shfl(st, r, 64);
    const int cn = has ? cs : 0;
    int32_t e[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) e[k] = k < cn ? a.bucket[ss + k] : INT32_MAX;
    sort2(e[0], e[1]);
    sort2(e[2], e[3]);
    sort2(e[0], e[2]);
    sort2(e[1], e[3]);
    sort2(e[1], e[2]);
    const uint32_t g = (uint32_t)(r0 + r);  // < 2^31
    const int64_t xc = a.n_dense + (int64_t)(g / (uint32_t)a.rows) * a.dim + 4 * cq;
    float4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = (k < cn && col) ? dx4<T>(a, e[k], xc) : zero;
    float4 s01 = zero, s1 = zero, s23 = zero, s3 = zero;
    add4(s01, v[0]);
    add4(s1, v[1]);
    add4(s01, s1);
    add4(s23, v[2]);
    add4(s3, v[3]);
    add4(s23, s3);
    add4(s01, s23);
    if (has && col) *reinterpret_cast<float4*>(a.grad + (int64_t)g * a.dim + 4 * cq) = s01;
  }
}

// A row of kLightBucket + 1..kSmallBucket entries by one wave: the bag rows
// sorted across the lanes, lane group q adding entries q, q + 64/G, ... in
// order (eight loads in flight), the groups combined by a fixed butterfly.
template <typename T, int G>
__device__ __forceinline__ void bag_row_mid(const EmbedBwdArgs& a, int32_t g) {
  constexpr int NGW = 64 / G;
  const int lane = threadIdx.x & 63;
  const int q = lane / G, cq = lane % G;
  const bool col = 4 * cq < a.dim;
  const int c = a.count[g], s0 = a.start[g];  // the same in every lane
  int32_t m[1] = {lane < c ? a.bucket[s0 + lane] : INT32_MAX};
  wave_sort<1>(m, lane);
  const int64_t xc = a.n_dense + (int64_t)(g / a.rows) * a.dim + 4 * cq;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int k0 = 0; k0 < c; k0 += 8 * NGW) {
    float4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = k0 + u * NGW + q;
      const int mk = __shfl(m[0], k & 63, 64);
      v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (k < c && col) v[u] = dx4<T>(a, mk, xc);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) add4(acc, v[u]);
  }
#pragma unroll
  for (int o = G; o < 64; o <<= 1) {
    acc.x += __shfl_xor(acc.x, o, 64);
    acc.y += __shfl_xor(acc.y, o, 64);
    acc.z += __shfl_xor(acc.z, o, 64);
    acc.w += __shfl_xor(acc.w, o, 64);
  }
  if (col && q == 0) *reinterpret_cast<float4*>(a.grad + (int64_t)g * a.dim + 4 * cq) = acc;
}

// The bag rows of a bucket of at most 64 R entries in order.
template <int R>
__device__ __forceinline__ void sort_bucket(const int32_t* bucket, int c, int32_t* key) {
  const int lane = opaque_lane();
  int32_t m[R];
#pragma unroll
  for (int r = 0; r < R; ++r) m[r] = 64 * r + lane < c ? bucket[64 * r + lane] : INT32_MAX;
  wave_sort<R>(m, lane);
#pragma unroll
  for (int r = 0; r < R; ++r) key[64 * r + lane] = m[r];
}

// A row of kSmallBucket + 1..kWaveBucket entries by one wave.  key: kWaveBucket
// words of LDS of its own (a wave's stores and loads are served in order).
template <typename T, int G>
__device__ __forceinline__ void bag_row_wave(const EmbedBwdArgs& a, int32_t g, int32_t* key) {
  constexpr int NGW = 64 / G;
  static_assert(kWaveBucket == 512, "the longest sort");
  const int lane = opaque_lane();
  const int q = lane / G, cq = lane % G;
  const bool col = 4 * cq < a.dim;
  const int c = a.count[g];
  const int32_t* bucket = a.bucket + a.start[g];
  if (c <= 128)
    sort_bucket<2>(bucket, c, key);
  else if (c <= 256)
    sort_bucket<4>(bucket, c, key);
  else
    sort_bucket<8>(bucket, c, key);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const int64_t xc = a.n_dense + (int64_t)(g / a.rows) * a.dim + 4 * cq;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  add_bag_rows<T, NGW>(a, key, 0, c, q, col, xc, acc);
#pragma unroll
  for (int o = G; o < 64; o <<= 1) {
    acc.x += __shfl_xor(acc.x, o, 64);
    acc.y += __shfl_xor(acc.y, o, 64);
    acc.z += __shfl_xor(acc.z, o, 64);
    acc.w += __shfl_xor(acc.w, o, 64);
  }
  if (col && q == 0) *reinterpret_cast<float4*>(a.grad + (int64_t)g * a.dim + 4 * cq) = acc;
}

// Every row of the gradient, in one launch of three kinds of workgroups: the
// first nlist take the rows of more than wave_bucket() entries (a serial chain
// of sorts and sums, so they start first), then nmid the rows of 5 entries and
// more up to that, a wave each, then nlight all the others, 64 consecutive rows per
// wave: the chains of dependent loads of the rows with entries run beside the
// stores of the zeros (665 MB of gradient for 26 tables of 100000 x 64: 145 to
// 165 us, against 220 for the same work as four launches).  At that shape the
// whole backward went from 308 to 239 us, at 3 tables of 5000 x 16 and 200 rows
// from 79 to 31, at 10 of 30000 x 32 (fp32, 1500 rows) from 95 to 53.  One
// workgroup per compute unit for the listed rows: with two 251 us.
template <typename T, int G>
__global__ __launch_bounds__(kSumThreads, 8) void erase_bags_bwd_sums(EmbedBwdArgs a, uint32_t nlist, uint32_t nmid, uint32_t nlight) {
  __shared__ int32_t key[kSortCap];
  __shared__ int32_t sel[kSumThreads / 64];
  __shared__ uint32_t bits[kBitWords];
  const uint32_t b = blockIdx.x, wave = threadIdx.x >> 6;
  if (b < nlist) {
    const int nl = a.nlarge[1];
    for (int i = (int)b; i < nl; i += (int)nlist) {
      bag_row_large<T, G>(a, a.large[i], key, bits, sel);
      __syncthreads();  // the next row reuses the arrays
    }
  } else if (b < nlist + nmid) {
    const uint32_t n = (uint32_t)a.nlarge[3], i0 = (b - nlist) * (kSumThreads / 64) + wave, ni = nmid * (kSumThreads / 64);
    // two loops: the longer sorts' lane masks are not kept in the first one
    if (wave_bucket(a) == kSmallBucket) {
      for (uint32_t i = i0; i < n; i += ni) bag_row_mid<T, G>(a, a.mid[i]);
    } else {
      for (uint32_t i = i0; i < n; i += ni) {
        const int32_t g = a.mid[i];
        if (a.count[g] <= kSmallBucket)
          bag_row_mid<T, G>(a, g);
        else
          bag_row_wave<T, G>(a, g, key + wave * kWaveBucket);
      }
    }
  } else {
    const int64_t r0 = ((int64_t)xcd_block(b - nlist - nmid, nlight) * (kSumThreads / 64) + wave) * 64;
    if (r0 < a.trows) bag_rows_light<T, G>(a, r0);
  }
}

hipError_t launch_embed_bags_backward(int bf16, const EmbedBwdArgs& a, hipStream_t s) {
  if (a.dim % 4 || a.dim > 256 || a.trows <= 0) return hipErrorInvalidValue;
  const int64_t nmax = a.trows > a.nnz ? a.trows : a.nnz;
  auto g8 = [](int64_t n) { return (uint32_t)((n + 7) / 8 * 8); };  // workgroups for xcd_block()
  hipLaunchKernelGGL(erase_bags_bwd_clear, dim3((unsigned)((nmax + 255) / 256)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(erase_bags_bwd_owner, dim3(g8(((int64_t)a.M * a.T + 255) / 256)), dim3(256), 0, s, a);
  if (a.nnz > 0) {
    hipLaunchKernelGGL(erase_bags_bwd_count, dim3(g8((a.nnz + kCountTile - 1) / kCountTile)), dim3(256), 0,
                       s, a);
    hipLaunchKernelGGL(erase_bags_bwd_place, dim3(g8((a.trows + kScanBlock - 1) / kScanBlock)), dim3(256), 0,
                       s, a);
    hipLaunchKernelGGL(erase_bags_bwd_scatter, dim3(g8((a.nnz + 255) / 256)), dim3(256), 0, s, a);
  }
  int G = 1;  // lanes per row: dim / 4 rounded up to a power of two
  while (G < a.dim / 4) G *= 2;
  // at most nnz / (kSmallBucket + 1) rows pass the small-bucket count.  One
  // workgroup per compute unit takes them in turn, so that the other one that
  // fits there writes meanwhile (multiples of 8: the light rows' workgroups go
  // to the XCDs by their number)
  const uint32_t nlist = g8(std::min<int64_t>(a.nnz / (kSmallBucket + 1), 256));
  const int64_t nw = kSumThreads / 64, nmid_max = std::min<int64_t>(a.trows, a.nnz / (kLightBucket + 1));
  const uint32_t nmid = g8(std::min<int64_t>((nmid_max + nw - 1) / nw, 256));
  const uint32_t nlight = (uint32_t)((a.trows + 64 * nw - 1) / (64 * nw));
  const dim3 grid(nlist + nmid + g8(nlight)), block(kSumThreads);
#define ERASE_BAG_ROWS(GG)                                                                              \
  case GG:                                                                                              \
    if (bf16)                                                                                           \
      hipLaunchKernelGGL((erase_bags_bwd_sums<uint16_t, GG>), grid, block, 0, s, a, nlist, nmid, nlight); \
    else                                                                                                \
      hipLaunchKernelGGL((erase_bags_bwd_sums<float, GG>), grid, block, 0, s, a, nlist, nmid, nlight);    \
    break;
  switch (G) {
    ERASE_BAG_ROWS(1)
    ERASE_BAG_ROWS(2)
    ERASE_BAG_ROWS(4)
    ERASE_BAG_ROWS(8)
    ERASE_BAG_ROWS(16)
    ERASE_BAG_ROWS(32)
    ERASE_BAG_ROWS(64)
    default: return hipErrorInvalidValue;
  }
#undef ERASE_BAG_ROWS
  return hipGetLastError();
}

}  // namespace erase
