// Device helpers shared by the gfx950 kernels of libzf (row-major and
// channel-major): bf16 conversions, wave bit counts, descriptor lookup, raw
// buffer resources and the Adam element update.
#pragma once

#include "zf_internal.hpp"

namespace zf {

__device__ __forceinline__ float widen_bf16(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// fp32 -> bf16, round to nearest, ties to even; NaN stays a (quiet) NaN.
__device__ __forceinline__ uint16_t round_bf16(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<uint16_t>((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

// A value every lane of the wave holds (loaded from the same address, e.g.
// the selection word of a block's channel) moved to scalar registers.
// Buffer resources built from it are then scalar as the hardware requires,
// instead of being wrapped by the compiler in per-access lane loops.
__device__ __forceinline__ uint64_t uniform_u64(uint64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x >> 32));
  return (static_cast<uint64_t>(hi) << 32) | lo;
}
__device__ __forceinline__ int32_t uniform_i32(int32_t x) {
  return __builtin_amdgcn_readfirstlane(x);
}

// A plan's device tables (matrix descriptors, block offsets) are written by
// the host before a launch and only read by the kernels.  Reading one
// through the constant address space lets the compiler use scalar loads:
// the values land in scalar registers without waiting for the vector loads
// in flight, and buffer resources built from them need no per-lane loop.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* const_table(const T* p) {
  return (const __attribute__((address_space(4))) T*)(p);
}

// Number of set bits of `mask` at lane positions below the calling lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// Workgroups are dispatched to the 8 XCDs of the chip round-robin by block
// id.  The id is remapped so that, within each window of 8 * RUN blocks, XCD x
// handles RUN consecutive ones (a power of two; the blocks after the last full
// window, or the whole grid where RUN is 0, are split into one contiguous
// range per XCD): each XCD and its L2 stream contiguous addresses.  A bijection
// on [0, B) for any B.
//
// One range per XCD (4-5% faster than no remapping) hands whole matrices to an
// XCD when the set is small, and the matrices' blocks differ in work: a score
// wave's channel is as long as its matrix has rows.  Windows balance that, and
// keep the XCDs in one neighbourhood of every stream; over tens of GB a pass
// separate ranges are the faster again.  Measured, RUN 64 / 256 / one range, in
// us:
//   column scores        7B layer 66 / 64 / 89, 70B layer 252 / 253 / 460, two
//                        embeddings and 12 7B layers (118 K blocks) 797 / 785 /
//                        868, ten 70B layers (195 K) 2600 / - / 2510; with the
//                        hand-over, 13B layer (11 K) 361 / 384 / 502, the 13B set
//                        (460 K) 13200 / 13100 / 12530
//   hand-over, deferred  7B layer (52 K blocks) 423 / 430 / 441, 3 layers and
//                        embeddings (220 K) 2210 / 2190 / 2196, 12 (690 K) 6915 /
//                        6757 / 6778, 20 (1.1 M) 11170 / 10930 / 10900
//   row-major update     7B layer (15 K larger blocks) 696 / 700 / 727, the 7B
//                        set's deferred hand-over (490 K) - / 23300 / 22400
//   Adam, selected grid  13B layer (79 K) 457 / 451 / 469, 70B (84 K) 450 / 436 /
//                        440, 12 7B layers (265 K) 1405 / 1383 / 1381, 20 (430 K)
//                        2273 / 2240 / 2222
// (runs of 16 are within 2% of 64; 1024 lose the balance).  What decides is the
// size of the pass, `work`: the grid's blocks, or what a smaller grid of larger
// blocks walks: row-major blocks count their rows in sixteens (Zen-auto's blocks
// of 256 rows on the 7B set, 30 K of them, RUN 64 / one range: 19.5 / 19.0 ms),
// the gated hand-over's fixed grid its units (8.7 / 8.3 ms).
#ifndef ZF_XCD_REMAP
#define ZF_XCD_REMAP 1
#endif
constexpr uint32_t kXcds = 8;

enum XcdOrder { kOrderScores, kOrderStream, kOrderSelected, kOrderRowMajor };

template <int ORDER = kOrderStream>
__device__ __forceinline__ int64_t xcd_remap(uint32_t b, uint32_t B, int64_t work) {
  if constexpr (ZF_XCD_REMAP == 0) return b;
  uint32_t lg;  // log2 RUN, or 0: one range per XCD
  if constexpr (ORDER == kOrderScores) lg = work <= (1 << 17) ? 6 : 0;
  else if constexpr (ORDER == kOrderRowMajor) lg = work <= (1 << 17) ? 6 : 0;
  else if constexpr (ORDER == kOrderSelected) lg = work <= (1 << 18) ? 8 : 0;
  else lg = work <= (1 << 17) ? 6 : work <= (1 << 20) ? 8 : 0;
  const uint32_t full = lg != 0 ? B >> (lg + 3) << (lg + 3) : 0;
  if (b < full) {
    const uint32_t i = b & ((kXcds << lg) - 1);
    return b - i + ((i % kXcds) << lg) + i / kXcds;
  }
  const uint32_t rest = B - full, t = b - full;
  const uint32_t q = rest / kXcds, r = rest % kXcds;
  const uint32_t x = t % kXcds, i = t / kXcds;
  return full + (x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i);
}

template <int ORDER = kOrderStream>
__device__ __forceinline__ int64_t xcd_remap(uint32_t b, uint32_t B) {
  return xcd_remap<ORDER>(b, B, B);
}

// Descriptor of the matrix the (remapped) block belongs to.  BATCHED kernels
// read it from the plan's device table (scalar loads); single-matrix kernels
// take it by value.  Keeping the two apart avoids a generic pointer that
// would turn the descriptor loads into flat vector loads.
template <bool BATCHED, int ORDER = kOrderStream>
__device__ __forceinline__ const DevMat& get_mat(const DevMat* __restrict__ mats,
                                                 const int64_t* __restrict__ off, int32_t nmats,
                                                 const DevMat& one, int64_t& local,
                                                 int32_t& index) {
  int64_t work = gridDim.x;
  if constexpr (ORDER == kOrderRowMajor)  // (blocks of 8 rows, on small grids, count as 16)
    work *= max(1, (BATCHED ? mats[0].rv_rows : one.rv_rows) / 16);
  const int64_t b = xcd_remap<ORDER>(blockIdx.x, gridDim.x, work);
  if constexpr (!BATCHED) {
    local = b;
    index = 0;
    return one;
  } else {
    int lo = 0, hi = nmats - 1;
    while (lo < hi) {  // largest q with off[q] <= b
      const int mid = (lo + hi + 1) >> 1;
      if (off[mid] <= b) lo = mid; else hi = mid - 1;
    }
    local = b - off[lo];
    index = lo;
    return mats[lo];
  }
}

template <bool BATCHED, int ORDER = kOrderStream>
__device__ __forceinline__ const DevMat& get_mat(const DevMat* __restrict__ mats,
                                                 const int64_t* __restrict__ off, int32_t nmats,
                                                 const DevMat& one, int64_t& local) {
  int32_t index;
  return get_mat<BATCHED, ORDER>(mats, off, nmats, one, local, index);
}

// Raw buffer resources (gfx9 family word 3).  A resource is based at the
// first row a block touches; lanes pass one 32-bit byte offset that is the
// same for every row, the row part goes in the scalar offset.  num_records
// is the exact byte span of the block's rows, so an access outside them is
// dropped by the hardware rather than reaching other memory.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr int kRsrcWord3 = 0x00020000;

__device__ __forceinline__ rsrc_t make_rsrc(const void* base, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), static_cast<short>(0),
                                           static_cast<int>(bytes), kRsrcWord3);
}

// Resource over rows [i0, i1) of a row-major [.][ld] array of `width` used
// elements of T per row.
template <typename T>
__device__ __forceinline__ rsrc_t rows_rsrc(const T* base, int64_t i0, int64_t i1, int64_t ld,
                                            int64_t width) {
  const int64_t rows = i1 - i0;
  const int64_t bytes = rows > 0 ? ((rows - 1) * ld + width) * static_cast<int64_t>(sizeof(T)) : 0;
  return make_rsrc(base + i0 * ld, bytes);
}

// Cache policy of a buffer access.  Every stream of the hot path is read or
// written once per kernel, so the kernels mark their traffic non-temporal
// (kStream); kCached is the default policy.
constexpr int kCached = 0;
constexpr int kStream = 2;  // "nt"

template <int AUX = kCached>
__device__ __forceinline__ float buf_f32(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, AUX));
}
template <int AUX = kCached>
__device__ __forceinline__ uint16_t buf_u16(rsrc_t r, uint32_t voff, uint32_t soff) {
  return static_cast<uint16_t>(__builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, AUX));
}
template <int AUX = kCached>
__device__ __forceinline__ void buf_put_f32(float v, rsrc_t r, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, voff, soff, AUX);
}
template <int AUX = kCached>
__device__ __forceinline__ void buf_put_u16(uint16_t v, rsrc_t r, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_buffer_store_b16(v, r, voff, soff, AUX);
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <int AUX = kCached>
__device__ __forceinline__ u32x4 buf_b128(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, AUX);
}
template <int AUX = kCached>
__device__ __forceinline__ void buf_put_b128(u32x4 v, rsrc_t r, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, soff, AUX);
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Wide non-temporal accesses to bf16 rows of any alignment (rows of an odd
// number of elements start at odd multiples of 2 bytes).  The target runs in
// unaligned access mode, so a type of 2-byte alignment still compiles to one
// global access; streaming 8 bytes a lane at offsets of 2 to 6 bytes measured
// 5.6-6.2 TB/s (copy), 6.4 when aligned and 3.0 element by element.  (A buffer
// access wants 4-byte alignment, which every fp32 row has.)  In bounds only:
// nothing checks a range here.
typedef u32x4 u32x4_h __attribute__((aligned(2)));
typedef u32x2 u32x2_h __attribute__((aligned(2)));

__device__ __forceinline__ u32x4 load8_bf16(const uint16_t* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4_h*>(p));
}
__device__ __forceinline__ void store8_bf16(uint16_t* p, u32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4_h*>(p));
}
__device__ __forceinline__ u32x2 load4_bf16(const uint16_t* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x2_h*>(p));
}
__device__ __forceinline__ void store4_bf16(uint16_t* p, u32x2 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<u32x2_h*>(p));
}

template <int AUX = kCached>
__device__ __forceinline__ u32x2 buf_b64(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, AUX);
}
template <int AUX = kCached>
__device__ __forceinline__ void buf_put_b64(u32x2 v, rsrc_t r, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_buffer_store_b64(v, r, voff, soff, AUX);
}

// Second stage of the row-major column sums: column j's cn_rb row-block
// partials (rows of m doubles at p) added in a fixed order -- wave w of the
// block's SEGS the w-th contiguous share of them, in row-block order, then the
// waves' sums in wave order through `red`.  Every thread of the block calls it;
// the result is valid in the first kFinCols threads.
template <int SEGS>
__device__ __forceinline__ double finalize_sum(const double* __restrict__ p, int32_t rb, int64_t m,
                                               int64_t j, double (&red)[SEGS][kFinCols]) {
  constexpr int kBatch = kFinBatch;  // loads in flight per lane
  const int lane = threadIdx.x & 63;
  const int wave = uniform_i32(threadIdx.x >> 6);
  const int32_t per = (rb + SEGS - 1) / SEGS;
  const int32_t r1 = min(rb, (wave + 1) * per);
  double s = 0.0;
  if (j < m) {
    for (int32_t r = wave * per; r < r1; r += kBatch) {
      double v[kBatch];
#pragma unroll
      for (int b = 0; b < kBatch; ++b)
        v[b] = r + b < r1 ? p[static_cast<int64_t>(r + b) * m + j] : 0.0;
#pragma unroll
      for (int b = 0; b < kBatch; ++b) s += v[b];
    }
  }
  if constexpr (SEGS == 1) return s;
  red[wave][lane] = s;
  __syncthreads();
  s = red[0][lane];
#pragma unroll
  for (int w = 1; w < SEGS; ++w) s += red[w][lane];
  return s;
}

// One Adam/AdamW element update; each line is one fp32 operation (the
// library is compiled without contraction, with correctly rounded sqrt and
// division).
__device__ __forceinline__ void adam_step(float g, float& p, float& m, float& v, const AdamK& c) {
  m = c.b1 * m + c.c1 * g;
  v = c.b2 * v + c.c2 * (g * g);
  const float den = sqrtf(v * c.ib2) + c.eps;
  const float u = (m * c.ib1) / den;
  if (c.wd != 0.0f) p = p - c.wd * p;
  p = p - c.lr * u;
}

}  // namespace zf
