// gfx950 kernels of the selective-update hot path.
//
// All kernels are bandwidth-bound streaming passes (no contraction, so no
// MFMA).  Every kernel reads its matrix descriptor from a batch table (one
// grid over many matrices; block -> matrix by binary search over the
// per-kernel block offsets) or from a single descriptor passed by value.
//
// Compiled with -ffp-contract=off and correctly rounded fp32 division and
// square root, so that each arithmetic line below is one IEEE operation.
#include "zf_device.hpp"

namespace zf {
namespace {

// ---------------------------------------------------------------------------
// a1: column scores.  Stage 1: a block sums the squares of a 512-column x
// cn_rpb-row tile in fp64 (squares of bf16 values are exact), each lane
// owning 8 adjacent columns and reading them with one 16-byte load per row;
// the four waves take interleaved rows and are combined in LDS in fixed
// order.  Stage 2 adds the row-block partials of each column in a fixed order
// and rounds once to fp32.  No atomics: the result is deterministic.
// ---------------------------------------------------------------------------

constexpr int kCnBatch = 4;  // rows per wave loaded before they are added

// G (rows of any alignment) is read once and the stage (16-byte rows) written
// once per pass: both non-temporal
__device__ __forceinline__ void cn_store(uint16_t* p, u32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
}

__device__ __forceinline__ void accum8(double (&acc)[8], u32x4 v) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const double lo = static_cast<double>(__uint_as_float(w[h] << 16));
    const double hi = static_cast<double>(__uint_as_float(w[h] & 0xffff0000u));
    acc[2 * h] = __builtin_fma(lo, lo, acc[2 * h]);
    acc[2 * h + 1] = __builtin_fma(hi, hi, acc[2 * h + 1]);
  }
}

// STAGE (a refresh step that starts an interval, plans with the bf16
// first-step stage): the pass also copies every element it reads to the
// same place of the stage (one bf16 row per gradient row), the packing of
// whichever columns the selection leaves unselected, so that the step's
// update runs the Adam part alone.
template <bool BATCHED, bool STAGE>
__global__ __launch_bounds__(kThreads) void colnorm_partial_kernel(const DevMat* __restrict__ mats, const int64_t* __restrict__ off, int32_t nmats, DevMat one,
                                                                   double* __restrict__ ws) {
  int64_t local;
  const DevMat d = get_mat<BATCHED>(mats, off, nmats, one, local);
  const bool st = STAGE && d.acc1 != nullptr;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t cblk = local % d.cn_cb;
  const int64_t rblk = local / d.cn_cb;
  const int64_t c0 = cblk * kColnormCols + lane * 8;
  const int64_t r0 = rblk * d.cn_rpb;
  const int64_t r1 = min(r0 + static_cast<int64_t>(d.cn_rpb), d.n);

  double acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = 0.0;

  if (c0 < d.m) {
    const uint16_t* __restrict__ base = d.grad + c0;
    const int64_t ld = d.ld_grad;
    uint16_t* __restrict__ sbase = st ? d.acc1 + c0 : nullptr;
    const int64_t sld = d.ld_acc1;
    if (c0 + 8 <= d.m) {
      int64_t i = r0 + wave;
      for (; i + 4 * (kCnBatch - 1) < r1; i += 4 * kCnBatch) {
        u32x4 v[kCnBatch];
#pragma unroll
        for (int b = 0; b < kCnBatch; ++b) v[b] = load8_bf16(base + (i + 4 * b) * ld);
        if (st) {
#pragma unroll
          for (int b = 0; b < kCnBatch; ++b) cn_store(sbase + (i + 4 * b) * sld, v[b]);
        }
#pragma unroll
        for (int b = 0; b < kCnBatch; ++b) accum8(acc, v[b]);
      }
      for (; i < r1; i += 4) {
        const u32x4 v = load8_bf16(base + i * ld);
        if (st) cn_store(sbase + i * sld, v);
        accum8(acc, v);
      }
    } else {
      const int64_t nc = min(static_cast<int64_t>(8), d.m - c0);
      for (int64_t i = r0 + wave; i < r1; i += 4) {
        const uint16_t* row = base + i * ld;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          if (c < nc) {
            if (st) sbase[i * sld + c] = row[c];
            const double x = static_cast<double>(widen_bf16(row[c]));
            acc[c] = __builtin_fma(x, x, acc[c]);
          }
        }
      }
    }
  }

  __shared__ double red[4][kColnormCols];
#pragma unroll
  for (int c = 0; c < 8; ++c) red[wave][lane * 8 + c] = acc[c];
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int col = threadIdx.x + h * kThreads;
    const int64_t j = cblk * kColnormCols + col;
    if (j < d.m) {
      const double s = ((red[0][col] + red[1][col]) + red[2][col]) + red[3][col];
      ws[d.cn_ws + rblk * d.m + j] = s;
    }
  }
}

// Stage 2 is a chain of dependent fp64 additions behind loads that are m
// doubles apart, so what bounds it is latency: one thread per column walking
// its cn_rb partials took 62.7 us for a 4096 x 4096 weight (256 partials a
// column, 16 blocks on the chip), seven times the pass over G itself.  Here
// the kFinSegs waves of a block take a contiguous share of the partials of 64
// columns each, 8 loads in flight (finalize_sum): 4.3 us, and 5.8 us against 27.9 us for the layer of
// seven Llama-2-7B weights (16 to 43 partials a column).  Few partials are one
// round of loads for a single wave (SEGS 1).
template <bool BATCHED, int SEGS>
__global__ __launch_bounds__(kFinCols * SEGS) void colnorm_finalize_kernel(
    const DevMat* __restrict__ mats, const int64_t* __restrict__ off, int32_t nmats, DevMat one, const double* __restrict__ ws) {
  int64_t local;
  const DevMat& d = get_mat<BATCHED>(mats, off, nmats, one, local);
  const int64_t j = local * kFinCols + (threadIdx.x & 63);
  __shared__ double red[SEGS][kFinCols];
  const double s = finalize_sum<SEGS>(ws + d.cn_ws, d.cn_rb, d.m, j, red);
  if (threadIdx.x < kFinCols && j < d.m) d.norms[j] = static_cast<float>(s);
}

// ---------------------------------------------------------------------------
// a2: selection.  One 1024-thread block per matrix.  Scores are mapped to
// unsigned keys that order like the float values (with -0.0 == +0.0); an
// MSB-first radix select over digits of 11, 11 and 10 bits finds the k-th
// largest key T and how many keys equal to T are taken; a pass in ascending
// column order then emits sel / unsel, the 64-bit mask words (one wave ballot
// each) and their prefix counts.  Among keys equal to T the lowest columns win.
//
// One block on one CU, where 64 lanes execute one instruction a cycle: what
// bounds it is latency (loads, barriers) for a few thousand columns and the
// instructions spent per column beyond, not the 12 bytes a column.  So
//   - each wave owns one contiguous range of mask words and, up to
//     64 * 16 * kTopkMaxWords columns, keeps its keys in registers: the scores
//     are read once, all loads in flight;
//   - the first digit holds two mantissa bits besides the exponent, so scores
//     of a few binades spread over many LDS counters, and the later digits
//     touch the few keys that share the digits before; a digit whose keys are
//     all taken ends the search (two digits nearly always);
//   - the output pass needs one barrier: the waves count what they hold first
//     and then write their ranges independently.
// Measured (10% selected, one launch): 512 columns 5.8 -> 3.8 us, 4096 11.5 ->
// 5.4, 11008 28.4 -> 12.5, 28672 61.1 -> 21.1, against four 8-bit digits that
// read the scores again each time and an output pass with four barriers per
// 1024 columns.
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t order_key(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u << 1) == 0u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr int kTopkWaves = kTopkThreads / 64;
constexpr int kTopkBins = 2048;
constexpr int kTopkMaxWords = 32;  // words a wave holds in registers
static_assert(kTopkBins == 2 * kTopkThreads && kTopkWaves == 16, "two bins a thread, one row of waves");

struct TopkShared {
  uint32_t hist[3][kTopkBins];
  uint32_t wave_a[kTopkWaves], wave_b[kTopkWaves];
  uint32_t digit, above, here;
};

// Inclusive sum over the lanes of the wave up to this one.
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return x;
}

// Sum of v[0 .. wave - 1] (v: one value per wave, in LDS).
__device__ __forceinline__ uint32_t waves_before(const uint32_t* v, int lane, int wave) {
  const uint32_t incl = wave_scan(lane < kTopkWaves ? v[lane] : 0u);
  return wave > 0 ? __builtin_amdgcn_readlane(incl, wave - 1) : 0u;
}

// After a digit's counts are complete: the digit in which the rem-th largest
// of the counted keys falls (sh.digit), the keys in larger ones (sh.above) and
// in it (sh.here).  Thread t holds the t-th pair of bins from the top.
__device__ __forceinline__ void topk_digit(const uint32_t* hist, uint32_t rem, TopkShared& sh,
                                           int tid, int lane, int wave) {
  const uint32_t h0 = hist[kTopkBins - 1 - 2 * tid], h1 = hist[kTopkBins - 2 - 2 * tid];
  const uint32_t incl = wave_scan(h0 + h1);
  if (lane == 63) sh.wave_a[wave] = incl;
  __syncthreads();
  const uint32_t excl = waves_before(sh.wave_a, lane, wave) + incl - (h0 + h1);
  if (excl < rem && rem <= excl + h0 + h1) {
    const bool second = excl + h0 < rem;
    sh.digit = static_cast<uint32_t>(kTopkBins - 1 - 2 * tid - (second ? 1 : 0));
    sh.above = second ? excl + h0 : excl;
    sh.here = second ? h1 : h0;
  }
  __syncthreads();
}

// The selection of matrix d.  WORDS > 0: a wave's words (at most WORDS) are
// held in registers; 0: any number of columns, the keys read again each time.
template <int WORDS>
__device__ __forceinline__ void topk_block(const DevMat& d, TopkShared& sh) {
  const int64_t m = d.m, k = d.k;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = uniform_i32(tid >> 6);
  const int32_t words = static_cast<int32_t>((m + 63) >> 6);
  const int32_t per = (words + kTopkWaves - 1) / kTopkWaves;
  const int32_t w0 = min(wave * per, words);
  const int32_t nw = min(per, words - w0);  // this wave's words
  // word i holds this lane's column iff 64 * i < left
  const int32_t left = static_cast<int32_t>(m) - w0 * 64 - lane;
  const float* __restrict__ sw = d.norms + (static_cast<int64_t>(w0) * 64 + lane);

  // A lane without a column holds key 0, the smallest: it changes neither the
  // k-th largest key nor how many keys lie above it.
  uint32_t reg[WORDS > 0 ? WORDS : 1];
  float x[WORDS > 0 ? WORDS : 1];
  if constexpr (WORDS > 0) {
#pragma unroll
    for (int i = 0; i < WORDS; ++i) x[i] = (i < nw && 64 * i < left) ? sw[64 * i] : 0.0f;
  }
  for (int b = tid; b < 3 * kTopkBins; b += kTopkThreads) (&sh.hist[0][0])[b] = 0u;
  if (tid == 0) sh.digit = sh.above = sh.here = 0u;
  if constexpr (WORDS > 0) {
#pragma unroll
    for (int i = 0; i < WORDS; ++i) reg[i] = 64 * i < left ? order_key(x[i]) : 0u;
  }
  // fn(i, key) over the wave's words
  const auto each = [&](auto fn) {
    if constexpr (WORDS > 0) {
#pragma unroll
      for (int i = 0; i < WORDS; ++i)
        if (i < nw) fn(i, reg[i]);
    } else {
      for (int32_t i = 0; i < nw; ++i)
        fn(i, 64 * i < left ? order_key(sw[64 * static_cast<int64_t>(i)]) : 0u);
    }
  };

  // taken: the keys above thr, and the first `need` equal to it
  uint32_t thr, need;
  if (k == 0) {
    thr = 0xffffffffu;
    need = 0u;
  } else if (k == m) {
    thr = 0u;
    need = static_cast<uint32_t>(m);
  } else {
    uint32_t rem = static_cast<uint32_t>(k);
    __syncthreads();
    each([&](int, uint32_t key) { atomicAdd(&sh.hist[0][key >> 21], 1u); });
    __syncthreads();
    topk_digit(sh.hist[0], rem, sh, tid, lane, wave);
    uint32_t prefix = sh.digit;
    rem -= sh.above;
    uint32_t here = sh.here;
    int bits = 11;  // of the key in prefix
#pragma unroll 1
    for (int pass = 1; pass < 3 && (here != rem || prefix == 0u); ++pass) {
      // (the next write of digit, above and here comes after two barriers)
      const int next = pass == 1 ? 11 : 10;
      uint32_t* hist = sh.hist[pass];
      each([&](int, uint32_t key) {
        if ((key >> (32 - bits)) == prefix)
          atomicAdd(&hist[(key >> (32 - bits - next)) & ((1u << next) - 1u)], 1u);
      });
      __syncthreads();
      topk_digit(hist, rem, sh, tid, lane, wave);
      prefix = (prefix << next) | sh.digit;
      rem -= sh.above;
      here = sh.here;
      bits += next;
    }
    const uint32_t low = prefix << (32 - bits);  // smallest key with these digits
    if (here == rem && low != 0u) {  // all of them are taken
      thr = low - 1u;
      need = 0u;
    } else {  // (all 32 bits known)
      thr = low;
      need = rem;
    }
  }

  // what the wave holds above the threshold and at it
  uint32_t gt = 0u, eq = 0u;
  each([&](int i, uint32_t key) {
    gt += __popcll(__ballot(key > thr));
    if (need != 0u) eq += __popcll(__ballot(key == thr && 64 * i < left));
  });
  __syncthreads();  // (the last digit's wave sums are read)
  if (lane == 0) {
    sh.wave_a[wave] = gt;
    sh.wave_b[wave] = eq;
  }
  __syncthreads();
  uint32_t carry_eq = waves_before(sh.wave_b, lane, wave);
  uint32_t carry_sel = waves_before(sh.wave_a, lane, wave) + min(carry_eq, need);
  uint64_t my_mask = 0u;
  int32_t my_prefix = 0;
  int32_t* __restrict__ out_sel = d.sel_idx;
  int32_t* __restrict__ out_uns = d.unsel_idx;
  const uint32_t n_sel = static_cast<uint32_t>(k), n_uns = static_cast<uint32_t>(m - k);
  each([&](int i, uint32_t key) {
    bool take = key > thr;
    if (need != 0u) {
      const uint64_t b_eq = __ballot(key == thr && 64 * i < left);
      take = take || (key == thr && 64 * i < left && carry_eq + lanes_below(b_eq) < need);
      carry_eq += static_cast<uint32_t>(__popcll(b_eq));
    }
    const uint64_t b_sel = __ballot(take);
    const uint32_t rank = carry_sel + lanes_below(b_sel);
    const uint32_t j = static_cast<uint32_t>((w0 + i) * 64 + lane);
    // The ranks are in range whenever the select above is right; the guards
    // keep a wrong count from ever writing outside the outputs.
    int32_t* to = take ? out_sel : out_uns;
    const uint32_t at = take ? rank : j - rank;
    if (64 * i < left && at < (take ? n_sel : n_uns)) to[at] = static_cast<int32_t>(j);
    if constexpr (WORDS > 0) {
      if (lane == i) {
        my_mask = b_sel;
        my_prefix = static_cast<int32_t>(carry_sel);
      }
    } else if (lane == 0) {
      d.mask[w0 + i] = b_sel;
      d.prefix[w0 + i] = static_cast<int32_t>(carry_sel);
    }
    carry_sel += static_cast<uint32_t>(__popcll(b_sel));
  });
  if constexpr (WORDS > 0) {
    if (lane < nw) {
      d.mask[w0 + lane] = my_mask;
      d.prefix[w0 + lane] = my_prefix;
    }
  }
}

template <bool BATCHED>
__global__ __launch_bounds__(kTopkThreads) void topk_kernel(const DevMat* __restrict__ mats, const int64_t* __restrict__ off, int32_t nmats, DevMat one) {
  int64_t local;
  const DevMat& d = get_mat<BATCHED>(mats, off, nmats, one, local);
  __shared__ TopkShared sh;
  if (d.m == 0) return;
  // the words a wave owns decide the variant (unrolled over that many)
  const int64_t per = (((d.m + 63) >> 6) + kTopkWaves - 1) / kTopkWaves;
  if (per <= 1) topk_block<1>(d, sh);
  else if (per <= 4) topk_block<4>(d, sh);
  else if (per <= 8) topk_block<8>(d, sh);
  else if (per <= 16) topk_block<16>(d, sh);
  else if (per <= kTopkMaxWords) topk_block<kTopkMaxWords>(d, sh);
  else topk_block<0>(d, sh);
}

// ---------------------------------------------------------------------------
// a3-a5: selective Adam with bf16 write-back, and packing of the unselected
// columns, in one pass over G.  A block owns a 256-column tile (four mask
// words) and a range of rows.  Its columns split into cu unselected slots
// [us, us+cu) of the accumulation buffer and cs selected slots [rs, rs+cs)
// of the compact states, both contiguous; thread t < cu owns unselected
// slot us+t, thread cu <= t < cu+cs owns selected slot rs+t-cu.  Each
// thread reads its column index once and then walks the rows: consecutive
// lanes touch consecutive slots (fully coalesced A and P/M/V traffic), the
// G gathers of a wave fall in one or two cache lines, and only the one or
// two waves holding selected slots execute the Adam arithmetic.  Rows are
// processed kRowBatch at a time with all loads issued before use.
// ---------------------------------------------------------------------------


#ifndef ZF_PACK_BATCH
#define ZF_PACK_BATCH 8
#endif
#ifndef ZF_ADAM_BATCH
#define ZF_ADAM_BATCH 8
#endif
#ifndef ZF_RM_AUX_RO
#define ZF_RM_AUX_RO kCached
#endif
#ifndef ZF_RM_AUX_W
#define ZF_RM_AUX_W kCached
#endif
constexpr int kRowBatch = ZF_PACK_BATCH;   // rows in flight per pack lane (and unpack)
constexpr int kAdamBatch = ZF_ADAM_BATCH;  // rows in flight per Adam lane

// Selected and unselected slot ranges of the tile starting at column c0.
struct TileSlots {
  int64_t rs, cs, us, cu, width;
};

__device__ __forceinline__ TileSlots tile_slots(const DevMat& d, int64_t c0) {
  TileSlots ts;
  ts.width = min(static_cast<int64_t>(kUpdateCols), d.m - c0);
  const int64_t words = (d.m + 63) >> 6;
  const int64_t w1 = (c0 + ts.width + 63) >> 6;
  ts.rs = d.prefix[c0 >> 6];
  const int64_t re = (w1 < words) ? static_cast<int64_t>(d.prefix[w1]) : d.k;
  ts.cs = re - ts.rs;
  ts.cu = ts.width - ts.cs;
  ts.us = c0 - ts.rs;
  return ts;
}

// Pack lane: A[i][u] (+)= G[i][j] over the block's rows.  HAND (last step
// of an interval, fused hand-over): scale * the new sum goes to D[i][j] (rD,
// vD, sD) and A is not written.  A16 (the bf16 first-step stage, element
// (i, j) at rS/vS/sS): 1 -- the first step stores the gradient's bits there
// instead of fp32 A; 2 -- the second step reads its previous values there.
template <bool FIRST, bool HAND = false, int A16 = 0>
__device__ __forceinline__ void pack_rows(rsrc_t rG, uint32_t vG, uint32_t sG, rsrc_t rA,
                                          uint32_t vA, uint32_t sA, int32_t rows,
                                          rsrc_t rD = rsrc_t(), uint32_t vD = 0, uint32_t sD = 0,
                                          float scale = 1.0f, rsrc_t rS = rsrc_t(),
                                          uint32_t vS = 0, uint32_t sS = 0) {
  int32_t i = 0;
  for (; i + kRowBatch <= rows; i += kRowBatch) {
    uint16_t gb[kRowBatch];
    float a[kRowBatch];
#pragma unroll
    for (int b = 0; b < kRowBatch; ++b) gb[b] = buf_u16<ZF_RM_AUX_RO>(rG, vG, (i + b) * sG);
    if constexpr (!FIRST) {
#pragma unroll
      for (int b = 0; b < kRowBatch; ++b)
        a[b] = A16 == 2 ? widen_bf16(buf_u16(rS, vS, (i + b) * sS)) : buf_f32(rA, vA, (i + b) * sA);
#pragma unroll
      for (int b = 0; b < kRowBatch; ++b) a[b] = a[b] + widen_bf16(gb[b]);
    } else {
#pragma unroll
      for (int b = 0; b < kRowBatch; ++b) a[b] = widen_bf16(gb[b]);
    }
#pragma unroll
    for (int b = 0; b < kRowBatch; ++b) {
      if constexpr (HAND) buf_put_f32(a[b] * scale, rD, vD, (i + b) * sD);
      else if constexpr (FIRST && A16 == 1) buf_put_u16(gb[b], rS, vS, (i + b) * sS);
      else buf_put_f32(a[b], rA, vA, (i + b) * sA);
    }
  }
  for (; i < rows; ++i) {
    const uint16_t gb = buf_u16<ZF_RM_AUX_RO>(rG, vG, i * sG);
    const float g = widen_bf16(gb);
    float a = g;
    if constexpr (!FIRST)
      a = (A16 == 2 ? widen_bf16(buf_u16(rS, vS, i * sS)) : buf_f32(rA, vA, i * sA)) + g;
    if constexpr (HAND) buf_put_f32(a * scale, rD, vD, i * sD);
    else if constexpr (FIRST && A16 == 1) buf_put_u16(gb, rS, vS, i * sS);
    else buf_put_f32(a, rA, vA, i * sA);
  }
}

// Where an Adam lane's (p, m, v) come from; see zf_state_mode.
struct AdamSrc {
  rsrc_t rP, rM, rV, rW;        // states and weight being written
  uint32_t vS, sS, vG, sW;      // slot / column byte offsets, row strides
  rsrc_t rSP, rSM, rSV;         // previous states (remap)
  uint32_t vPrev, sPrev;
  bool was;                     // column was selected before (remap)
  rsrc_t rI;                    // fp32 init master (init from master)
  uint32_t vI, sI;
  rsrc_t rTP, rTM, rTV;         // full-state store (swap-in)
  uint32_t vT, sT;
  rsrc_t rPA;                   // owed deferred update: previous interval's sums
  uint32_t vPA, sPA;
};

enum SrcKind {
  kSrcInplace = 0, kSrcRemapW, kSrcRemapMaster, kSrcInitW, kSrcInitMaster,
  kSrcRemapStore, kSrcInitStore,  // swap-in of new columns from the full-state store
  kSrcRemapStorePend              // the same, after the owed deferred step (Pending)
};

template <int SRC>
__device__ __forceinline__ void load_state(const AdamSrc& a, int32_t i, float& p, float& m,
                                           float& v, const Pending* pd = nullptr) {
  if constexpr (SRC == kSrcInplace) {
    p = buf_f32(a.rP, a.vS, i * a.sS);
    m = buf_f32(a.rM, a.vS, i * a.sS);
    v = buf_f32(a.rV, a.vS, i * a.sS);
  } else if constexpr (SRC == kSrcRemapStore || SRC == kSrcInitStore ||
                       SRC == kSrcRemapStorePend) {
    // Only the lanes of entering columns read the store (it may be pinned
    // host memory, where every lane's 4-byte read is its own PCIe request);
    // the others read their previous compact states.
    if (SRC != kSrcInitStore && a.was) {
      p = buf_f32(a.rSP, a.vPrev, i * a.sPrev);
      m = buf_f32(a.rSM, a.vPrev, i * a.sPrev);
      v = buf_f32(a.rSV, a.vPrev, i * a.sPrev);
    } else {
      p = buf_f32(a.rTP, a.vT, i * a.sT);
      m = buf_f32(a.rTM, a.vT, i * a.sT);
      v = buf_f32(a.rTV, a.vT, i * a.sT);
      if constexpr (SRC == kSrcRemapStorePend)  // the owed deferred step first
        adam_step(buf_f32(a.rPA, a.vPA, i * a.sPA) * pd->scale, p, m, v, pd->c);
    }
  } else {
    // A column that stays reads its previous states, an entering one the fp32
    // master: only the lanes that need a master line touch it (reading both and keeping
    // one took 494 us against 324 for the Adam pass of a Llama-2-7B layer's
    // refresh: almost every line of a 4-byte master holds a selected column).
    if constexpr (SRC == kSrcRemapMaster) {
      if (a.was) {
        p = buf_f32(a.rSP, a.vPrev, i * a.sPrev);
        m = buf_f32(a.rSM, a.vPrev, i * a.sPrev);
        v = buf_f32(a.rSV, a.vPrev, i * a.sPrev);
      } else {
        p = buf_f32(a.rI, a.vI, i * a.sI);
        m = v = 0.0f;
      }
      return;
    }
    // init value of p for a newly selected column
    float pi;
    if constexpr (SRC == kSrcInitMaster)
      pi = buf_f32(a.rI, a.vI, i * a.sI);
    else
      pi = widen_bf16(buf_u16(a.rW, a.vG, i * a.sW));
    if constexpr (SRC == kSrcRemapW) {
      // both sources are read; the lane keeps the one that applies
      const float pp = buf_f32(a.rSP, a.vPrev, i * a.sPrev);
      const float mp = buf_f32(a.rSM, a.vPrev, i * a.sPrev);
      const float vp = buf_f32(a.rSV, a.vPrev, i * a.sPrev);
      p = a.was ? pp : pi;
      m = a.was ? mp : 0.0f;
      v = a.was ? vp : 0.0f;
    } else {
      p = pi;
      m = 0.0f;
      v = 0.0f;
    }
  }
}

template <int SRC>
__device__ __forceinline__ void adam_rows(const AdamSrc& a, rsrc_t rG, uint32_t sG,
                                          const AdamK& c, int32_t rows,
                                          const Pending* pd = nullptr) {
  int32_t i = 0;
  for (; i + kAdamBatch <= rows; i += kAdamBatch) {
    uint16_t gb[kAdamBatch];
    float p[kAdamBatch], mm[kAdamBatch], vv[kAdamBatch];
#pragma unroll
    for (int b = 0; b < kAdamBatch; ++b) gb[b] = buf_u16<ZF_RM_AUX_RO>(rG, a.vG, (i + b) * sG);
#pragma unroll
    for (int b = 0; b < kAdamBatch; ++b) load_state<SRC>(a, i + b, p[b], mm[b], vv[b], pd);
#pragma unroll
    for (int b = 0; b < kAdamBatch; ++b) {
      adam_step(widen_bf16(gb[b]), p[b], mm[b], vv[b], c);
      const uint32_t so = (i + b) * a.sS;
      buf_put_f32(p[b], a.rP, a.vS, so);
      buf_put_f32(mm[b], a.rM, a.vS, so);
      buf_put_f32(vv[b], a.rV, a.vS, so);
      buf_put_u16<ZF_RM_AUX_W>(round_bf16(p[b]), a.rW, a.vG, (i + b) * a.sW);
    }
  }
  for (; i < rows; ++i) {
    float p, mm, vv;
    const float g = widen_bf16(buf_u16<ZF_RM_AUX_RO>(rG, a.vG, i * sG));
    load_state<SRC>(a, i, p, mm, vv, pd);
    adam_step(g, p, mm, vv, c);
    buf_put_f32(p, a.rP, a.vS, i * a.sS);
    buf_put_f32(mm, a.rM, a.vS, i * a.sS);
    buf_put_f32(vv, a.rV, a.vS, i * a.sS);
    buf_put_u16<ZF_RM_AUX_W>(round_bf16(p), a.rW, a.vG, i * a.sW);
  }
}

// PEND (fused Adam + pack in kRemap against the store only): a column that
// enters the selection takes the owed deferred step pd first, from its slot
// among the previous selection's unselected columns.
template <bool BATCHED, bool ADAM, bool PACK, bool HAND, bool PEND>
__global__ __launch_bounds__(kThreads) void update_kernel(const DevMat* __restrict__ mats,
                                                          const int64_t* __restrict__ off,
                                                          int32_t nmats, DevMat one, AdamK c,
                                                          int32_t mode, int32_t first,
                                                          float scale, Pending pd,
                                                          const ZenState* __restrict__ zst) {
  // Zen-auto with the interval driven on the device: a refresh step, or
  // any step after an ended interval, overwrites; else it accumulates
  if (zst != nullptr)
    first = (mode != kInplace || uniform_i32(zst->ended)) ? 1 : uniform_i32(zst->length) + 1;
  int64_t local;
  const DevMat d = get_mat<BATCHED>(mats, off, nmats, one, local);
  const int64_t cblk = local % d.up_cb;
  const int64_t rblk = local / d.up_cb;
  const int64_t c0 = cblk * kUpdateCols;
  const TileSlots ts = tile_slots(d, c0);
  const int tid = threadIdx.x;
  const bool swap_out = mode == kRemap && d.st_P != nullptr;
  const bool is_unsel = (PACK || swap_out) && tid < ts.cu;
  const bool is_adam = ADAM && tid >= ts.cu && tid < ts.width;
  if (!is_unsel && !is_adam) return;

  const int64_t i0 = rblk * d.up_rows;
  const int64_t i1 = min(i0 + static_cast<int64_t>(d.up_rows), d.n);
  const int32_t rows = static_cast<int32_t>(i1 - i0);
  const rsrc_t rG = rows_rsrc(d.grad, i0, i1, d.ld_grad, d.m);
  const uint32_t sG = static_cast<uint32_t>(d.ld_grad * 2);  // bytes per G row

  if (is_unsel) {
    const uint32_t u = static_cast<uint32_t>(ts.us + tid);
    const uint32_t j = static_cast<uint32_t>(d.unsel_idx[u]);
    if (swap_out) {
      // a column that left the selection: previous compact (p, m, v) -> store
      const uint64_t pm = d.prev_mask[j >> 6];
      if ((pm >> (j & 63u)) & 1ull) {
        const int64_t ro = static_cast<int64_t>(d.prev_prefix[j >> 6]) +
                           __popcll(pm & ((uint64_t(1) << (j & 63u)) - 1));
        for (int64_t i = i0; i < i1; ++i) {
          d.st_P[i * d.ld_store + j] = d.prev_P[i * d.ld_prev + ro];
          d.st_M[i * d.ld_store + j] = d.prev_M[i * d.ld_prev + ro];
          d.st_V[i * d.ld_store + j] = d.prev_V[i * d.ld_prev + ro];
        }
      }
    }
    if constexpr (PACK) {
      const uint32_t vG = j * 2u;
      const rsrc_t rA = rows_rsrc(d.acc, i0, i1, d.ld_acc, d.m - d.k);
      const uint32_t sA = static_cast<uint32_t>(d.ld_acc * 4);
      // the bf16 first-step stage at element (i, j): first == 1 on an
      // interval's first step, 2 on its second (a matrix without a stage
      // takes 2 as any later step)
      const bool a16 = d.acc1 != nullptr;
      const rsrc_t rS = a16 ? rows_rsrc(d.acc1, i0, i1, d.ld_acc1, d.m) : rA;
      const uint32_t sS = a16 ? static_cast<uint32_t>(d.ld_acc1 * 2) : 0u;
      if constexpr (HAND) {
        const rsrc_t rD = rows_rsrc(d.out, i0, i1, d.ld_out, d.m);
        const uint32_t sD = static_cast<uint32_t>(d.ld_out * 4);
        if (first == 1)
          pack_rows<true, true>(rG, vG, sG, rA, u * 4u, sA, rows, rD, j * 4u, sD, scale);
        else if (a16 && first == 2)
          pack_rows<false, true, 2>(rG, vG, sG, rA, u * 4u, sA, rows, rD, j * 4u, sD, scale, rS,
                                    vG, sS);
        else pack_rows<false, true>(rG, vG, sG, rA, u * 4u, sA, rows, rD, j * 4u, sD, scale);
      } else {
        if (first == 1) {
          if (a16)
            pack_rows<true, false, 1>(rG, vG, sG, rA, u * 4u, sA, rows, rsrc_t(), 0, 0, 1.0f, rS,
                                      vG, sS);
          else pack_rows<true>(rG, vG, sG, rA, u * 4u, sA, rows);
        } else if (a16 && first == 2) {
          pack_rows<false, false, 2>(rG, vG, sG, rA, u * 4u, sA, rows, rsrc_t(), 0, 0, 1.0f, rS,
                                     vG, sS);
        } else {
          pack_rows<false>(rG, vG, sG, rA, u * 4u, sA, rows);
        }
      }
    }
    return;
  }

  // Adam lane: selected slot r, column j.
  AdamSrc a;
  const uint32_t r = static_cast<uint32_t>(ts.rs + (tid - ts.cu));
  const uint32_t j = static_cast<uint32_t>(d.sel_idx[r]);
  a.vS = r * 4u;
  a.vG = j * 2u;
  a.rP = rows_rsrc(d.P, i0, i1, d.ld_state, d.k);
  a.rM = rows_rsrc(d.M, i0, i1, d.ld_state, d.k);
  a.rV = rows_rsrc(d.V, i0, i1, d.ld_state, d.k);
  a.sS = static_cast<uint32_t>(d.ld_state * 4);
  a.rW = rows_rsrc(d.weight, i0, i1, d.ld_weight, d.m);
  a.sW = static_cast<uint32_t>(d.ld_weight * 2);
  a.rSP = a.rP;
  a.rSM = a.rM;
  a.rSV = a.rV;
  a.vPrev = 0;
  a.sPrev = 0;
  a.was = false;
  a.rI = a.rW;
  a.vI = 0;
  a.sI = 0;
  const bool master = d.init_P != nullptr;
  const bool store = d.st_P != nullptr;
  if (mode != kInplace && master) {
    a.rI = rows_rsrc(d.init_P, i0, i1, d.ld_init, d.m);
    a.vI = j * 4u;
    a.sI = static_cast<uint32_t>(d.ld_init * 4);
  }
  a.rTP = a.rTM = a.rTV = a.rPA = a.rP;
  a.vT = a.vPA = 0;
  a.sT = a.sPA = 0;
  if (mode != kInplace && store) {
    a.rTP = rows_rsrc(d.st_P, i0, i1, d.ld_store, d.m);
    a.rTM = rows_rsrc(d.st_M, i0, i1, d.ld_store, d.m);
    a.rTV = rows_rsrc(d.st_V, i0, i1, d.ld_store, d.m);
    a.vT = j * 4u;
    a.sT = static_cast<uint32_t>(d.ld_store * 4);
  }
  if (mode == kRemap) {
    const uint32_t w = j >> 6;
    const uint64_t pm = d.prev_mask[w];
    a.was = (pm >> (j & 63u)) & 1ull;
    const uint32_t ro = static_cast<uint32_t>(d.prev_prefix[w]) +
                        static_cast<uint32_t>(__popcll(pm & ((uint64_t(1) << (j & 63u)) - 1)));
    // a column that was not selected reads slot 0 (any valid slot), unused
    a.vPrev = (a.was ? ro : 0u) * 4u;
    a.sPrev = static_cast<uint32_t>(d.ld_prev * 4);
    a.rSP = rows_rsrc(d.prev_P, i0, i1, d.ld_prev, d.m);
    a.rSM = rows_rsrc(d.prev_M, i0, i1, d.ld_prev, d.m);
    a.rSV = rows_rsrc(d.prev_V, i0, i1, d.ld_prev, d.m);
    if constexpr (PEND) {
      // (no unselected columns: an empty resource, every read returns 0)
      a.rPA = d.m > d.k ? rows_rsrc(d.pend_acc, i0, i1, d.ld_pend, d.m - d.k)
                        : make_rsrc(d.pend_acc, 0);
      a.vPA = (a.was ? 0u : j - ro) * 4u;
      a.sPA = static_cast<uint32_t>(d.ld_pend * 4);
    }
  }
  if constexpr (HAND) {
    // the hand-over buffer is +0.0 at a selected column
    const rsrc_t rD = rows_rsrc(d.out, i0, i1, d.ld_out, d.m);
    const uint32_t sD = static_cast<uint32_t>(d.ld_out * 4);
    for (int32_t i = 0; i < rows; ++i) buf_put_f32(0.0f, rD, j * 4u, i * sD);
  }
  if (mode == kInplace) adam_rows<kSrcInplace>(a, rG, sG, c, rows);
  else if (mode == kRemap) {
    if (PEND) adam_rows<kSrcRemapStorePend>(a, rG, sG, c, rows, &pd);
    else if (store) adam_rows<kSrcRemapStore>(a, rG, sG, c, rows);
    else if (master) adam_rows<kSrcRemapMaster>(a, rG, sG, c, rows);
    else adam_rows<kSrcRemapW>(a, rG, sG, c, rows);
  } else {
    if (store) adam_rows<kSrcInitStore>(a, rG, sG, c, rows);
    else if (master) adam_rows<kSrcInitMaster>(a, rG, sG, c, rows);
    else adam_rows<kSrcInitW>(a, rG, sG, c, rows);
  }
}

// ---------------------------------------------------------------------------
// a6: hand-over.  Same column mapping as the update pass.
// ---------------------------------------------------------------------------

// One block's share of the hand-over: the block-th tile (rows x 256
// columns) of matrix d.
__device__ __forceinline__ void unpack_unit(const DevMat& d, int64_t local, float scale) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t cblk = local % d.up_cb;
  const int64_t rblk = local / d.up_cb;
  const int64_t word = cblk * (kUpdateCols / 64) + wave;
  const int64_t j = word * 64 + lane;
  if (j >= d.m) return;
  const uint64_t mw = d.mask[word];
  const bool sel = (mw >> lane) & 1ull;
  const uint32_t u =
      static_cast<uint32_t>(j - (static_cast<int64_t>(d.prefix[word]) + lanes_below(mw)));
  const int64_t i0 = rblk * d.up_rows;
  const int64_t i1 = min(i0 + static_cast<int64_t>(d.up_rows), d.n);
  const int32_t rows = static_cast<int32_t>(i1 - i0);
  const rsrc_t rA = rows_rsrc(d.acc, i0, i1, d.ld_acc, d.m - d.k);
  const rsrc_t rD = rows_rsrc(d.out, i0, i1, d.ld_out, d.m);
  const uint32_t sA = static_cast<uint32_t>(d.ld_acc * 4);
  const uint32_t sD = static_cast<uint32_t>(d.ld_out * 4);
  const uint32_t vD = static_cast<uint32_t>(j) * 4u;
  int32_t i = 0;
  if (d.m == d.k) {  // every column selected: no accumulated data to read
    for (; i < rows; ++i) buf_put_f32(0.0f, rD, vD, i * sD);
    return;
  }
  // A selected lane reads a neighbouring valid slot (same cache lines as its
  // wave) and writes +0.0, so the wave runs one uniform loop.
  const uint32_t vA = min(u, static_cast<uint32_t>(d.m - d.k - 1)) * 4u;
  for (; i + kRowBatch <= rows; i += kRowBatch) {
    float a[kRowBatch];
#pragma unroll
    for (int b = 0; b < kRowBatch; ++b) a[b] = buf_f32(rA, vA, (i + b) * sA);
#pragma unroll
    for (int b = 0; b < kRowBatch; ++b)
      buf_put_f32(sel ? 0.0f : a[b] * scale, rD, vD, (i + b) * sD);
  }
  for (; i < rows; ++i) {
    const float a = buf_f32(rA, vA, i * sA);
    buf_put_f32(sel ? 0.0f : a * scale, rD, vD, i * sD);
  }
}

template <bool BATCHED>
__global__ __launch_bounds__(kThreads) void unpack_kernel(const DevMat* __restrict__ mats,
                                                          const int64_t* __restrict__ off,
                                                          int32_t nmats, DevMat one,
                                                          float scale) {
  int64_t local;
  const DevMat d = get_mat<BATCHED>(mats, off, nmats, one, local);
  unpack_unit(d, local, scale);
}

// The hand-over of an interval that Zen-auto ended on the device: nothing
// unless zst->ended == 1; then scale = fp32(1 / length) (a correctly rounded
// fp32 division, the value the host passes as fp32(1.0 / length)).  A fixed
// grid walks the table's unpack tiles, so that a step that does not end its
// interval costs one short launch.
__global__ __launch_bounds__(kThreads) void unpack_zen_kernel(const DevMat* __restrict__ mats,
                                                             const int64_t* __restrict__ off,
                                                             int32_t nmats, int64_t units,
                                                             const ZenState* __restrict__ zst) {
  if (uniform_i32(zst->ended) != 1) return;  // (2: already handed over)
  const float scale = 1.0f / static_cast<float>(uniform_i32(zst->length));
  const int64_t b = xcd_remap(blockIdx.x, gridDim.x);
  int lo = 0;
  for (int64_t u = b; u < units; u += gridDim.x) {
    int hi = nmats - 1;
    while (lo < hi) {  // largest q with off[q] <= u (u only grows)
      const int mid = (lo + hi + 1) >> 1;
      if (off[mid] <= u) lo = mid; else hi = mid - 1;
    }
    unpack_unit(mats[lo], u - off[lo], scale);
  }
}

// a3-a6 with deferred packing, row-major buffers off the 16-byte path: the
// interval's hand-over from the gradients it kept (the earlier steps' plans,
// then this step's), summed in step order in fp32 and scaled, +0.0 at a
// selected column.  Same column mapping as the hand-over above; the Adam
// part of the step is the per-column update's.
__global__ __launch_bounds__(kThreads) void rm_handover_deferred_kernel(
    const DevMat* __restrict__ mats, const int64_t* __restrict__ off, int32_t nmats, float scale,
    HistTable hist) {
  int64_t local;
  const DevMat& d = get_mat<true>(mats, off, nmats, mats[0], local);
  const int32_t q = static_cast<int32_t>(&d - mats);
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t cblk = local % d.up_cb;
  const int64_t rblk = local / d.up_cb;
  const int64_t word = cblk * (kUpdateCols / 64) + wave;
  const int64_t j = word * 64 + lane;
  if (j >= d.m) return;
  const bool sel = (d.mask[word] >> lane) & 1ull;
  const int64_t i0 = rblk * d.up_rows;
  const int64_t i1 = min(i0 + static_cast<int64_t>(d.up_rows), d.n);
  const int32_t rows = static_cast<int32_t>(i1 - i0);
  const rsrc_t rG = rows_rsrc(d.grad, i0, i1, d.ld_grad, d.m);
  const rsrc_t rD = rows_rsrc(d.out, i0, i1, d.ld_out, d.m);
  const uint32_t sG = static_cast<uint32_t>(d.ld_grad * 2);
  const uint32_t sD = static_cast<uint32_t>(d.ld_out * 4);
  const uint32_t vG = static_cast<uint32_t>(j) * 2u;
  const uint32_t vD = static_cast<uint32_t>(j) * 4u;
  for (int32_t i = 0; i < rows; ++i) {
    float a = 0.0f;
    for (int32_t st = 0; st < hist.n; ++st) {
      const auto& hd = const_table(hist.mats[st])[q];
      const rsrc_t rE = rows_rsrc(hd.grad, i0, i1, hd.ld_grad, d.m);
      const float g = widen_bf16(buf_u16<kStream>(
          rE, vG, static_cast<uint32_t>(i) * static_cast<uint32_t>(hd.ld_grad * 2)));
      a = st == 0 ? g : a + g;
    }
    const float g = widen_bf16(buf_u16<kStream>(rG, vG, static_cast<uint32_t>(i) * sG));
    a = hist.n > 0 ? a + g : g;
    buf_put_f32(sel ? 0.0f : a * scale, rD, vD, static_cast<uint32_t>(i) * sD);
  }
}

}  // namespace

#define ZF_LAUNCH(KERNEL, GRID, BLOCK, STREAM, T, ...)                                      \
  do {                                                                                     \
    if ((T).mats != nullptr)                                                               \
      hipLaunchKernelGGL((KERNEL<true>), GRID, BLOCK, 0, STREAM, (T).mats, (T).off,          \
                         (T).nmats, __VA_ARGS__);                                          \
    else                                                                                   \
      hipLaunchKernelGGL((KERNEL<false>), GRID, BLOCK, 0, STREAM, (T).mats, (T).off,         \
                         (T).nmats, __VA_ARGS__);                                          \
  } while (0)

template <int SEGS>
static void launch_fin(const Table& t, const DevMat& one, int64_t blocks, const double* ws,
                       hipStream_t s) {
  const dim3 grid(static_cast<uint32_t>(blocks)), block(kFinCols * SEGS);
  if (t.mats != nullptr)
    hipLaunchKernelGGL((colnorm_finalize_kernel<true, SEGS>), grid, block, 0, s, t.mats, t.off,
                       t.nmats, one, ws);
  else
    hipLaunchKernelGGL((colnorm_finalize_kernel<false, SEGS>), grid, block, 0, s, t.mats, t.off,
                       t.nmats, one, ws);
}

hipError_t launch_colnorm(const Table& t, const DevMat& one, int64_t blocks, const Table& tf,
                          int64_t fin_blocks, int segs, double* ws, hipStream_t s, bool stage) {
  (void)hipGetLastError();
  if (blocks > 0) {
    const dim3 grid(static_cast<uint32_t>(blocks));
    if (stage) {
      if (t.mats != nullptr)
        hipLaunchKernelGGL((colnorm_partial_kernel<true, true>), grid, dim3(kThreads), 0, s,
                           t.mats, t.off, t.nmats, one, ws);
      else
        hipLaunchKernelGGL((colnorm_partial_kernel<false, true>), grid, dim3(kThreads), 0, s,
                           t.mats, t.off, t.nmats, one, ws);
    } else {
      if (t.mats != nullptr)
        hipLaunchKernelGGL((colnorm_partial_kernel<true, false>), grid, dim3(kThreads), 0, s,
                           t.mats, t.off, t.nmats, one, ws);
      else
        hipLaunchKernelGGL((colnorm_partial_kernel<false, false>), grid, dim3(kThreads), 0, s,
                           t.mats, t.off, t.nmats, one, ws);
    }
  }
  if (fin_blocks > 0 && segs == 1)
    launch_fin<1>(tf, one, fin_blocks, ws, s);
  else if (fin_blocks > 0)
    launch_fin<kFinSegs>(tf, one, fin_blocks, ws, s);
  return hipGetLastError();
}

hipError_t launch_topk(const Table& t, const DevMat& one, int64_t blocks, hipStream_t s) {
  (void)hipGetLastError();
  if (blocks > 0)
    ZF_LAUNCH(topk_kernel, dim3(static_cast<uint32_t>(blocks)), dim3(kTopkThreads), s, t, one);
  return hipGetLastError();
}

template <bool ADAM, bool PACK, bool HAND, bool PEND = false>
static void launch_update_t(const Table& t, const DevMat& one, dim3 grid, const AdamK& c,
                            int32_t mode, int32_t first, float scale, hipStream_t s,
                            const Pending& pd = Pending{}, const ZenState* zst = nullptr) {
  if (t.mats != nullptr)
    hipLaunchKernelGGL((update_kernel<true, ADAM, PACK, HAND, PEND>), grid, dim3(kThreads), 0, s,
                       t.mats, t.off, t.nmats, one, c, mode, first, scale, pd, zst);
  else
    hipLaunchKernelGGL((update_kernel<false, ADAM, PACK, HAND, PEND>), grid, dim3(kThreads), 0, s,
                       t.mats, t.off, t.nmats, one, c, mode, first, scale, pd, zst);
}

hipError_t launch_update(const Table& t, const DevMat& one, int64_t blocks, const AdamK& c,
                         int32_t mode, int32_t first, bool adam, bool pack, bool handover,
                         float scale, hipStream_t s, const Pending* pend, const ZenState* zst) {
  (void)hipGetLastError();
  if (blocks <= 0) return hipSuccess;
  const dim3 grid(static_cast<uint32_t>(blocks));
  if (handover && !(adam && pack)) return hipErrorInvalidValue;
  if (zst != nullptr && (pend != nullptr || handover || !pack)) return hipErrorInvalidValue;
  if (pend != nullptr) {
    if (!(adam && pack) || handover || mode != kRemap) return hipErrorInvalidValue;
    launch_update_t<true, true, false, true>(t, one, grid, c, mode, first, 1.0f, s, *pend);
  } else if (handover) launch_update_t<true, true, true>(t, one, grid, c, mode, first, scale, s);
  else if (adam && pack)
    launch_update_t<true, true, false>(t, one, grid, c, mode, first, 1.0f, s, Pending{}, zst);
  else if (adam) launch_update_t<true, false, false>(t, one, grid, c, mode, first, 1.0f, s);
  else if (pack)
    launch_update_t<false, true, false>(t, one, grid, c, mode, first, 1.0f, s, Pending{}, zst);
  return hipGetLastError();
}

hipError_t launch_unpack(const Table& t, const DevMat& one, int64_t blocks, float scale,
                         hipStream_t s) {
  (void)hipGetLastError();
  if (blocks > 0)
    ZF_LAUNCH(unpack_kernel, dim3(static_cast<uint32_t>(blocks)), dim3(kThreads), s, t, one,
              scale);
  return hipGetLastError();
}

// A step that does not end its interval should exit in a short launch, one
// that does keep enough tiles in flight.  On a Llama-2-7B layer (98.8 K tiles)
// 65536 blocks take 15.3 us to exit and 292 us to hand over, 16384 5.0 and 305,
// 4096 4.9 and 330: eight tiles a block from 16384 blocks on, and 65536 for the
// large sets, where a hand-over takes milliseconds and 10 us do not count.
constexpr int64_t kUnpackZenMin = 16384, kUnpackZenMax = 65536;

hipError_t launch_unpack_zen(const Table& t, int64_t units, const ZenState* zst, hipStream_t s) {
  (void)hipGetLastError();
  if (units <= 0 || t.mats == nullptr) return hipSuccess;
  const int64_t want = units / 8 < kUnpackZenMin ? kUnpackZenMin
                       : units / 8 > kUnpackZenMax ? kUnpackZenMax : units / 8;
  const dim3 grid(static_cast<uint32_t>(units < want ? units : want));
  hipLaunchKernelGGL(unpack_zen_kernel, grid, dim3(kThreads), 0, s, t.mats, t.off, t.nmats, units,
                     zst);
  return hipGetLastError();
}

hipError_t launch_rm_handover_deferred(const Table& t, int64_t blocks, float scale,
                                       const HistTable& h, hipStream_t s) {
  (void)hipGetLastError();
  if (blocks <= 0 || t.mats == nullptr) return hipSuccess;
  hipLaunchKernelGGL(rm_handover_deferred_kernel, dim3(static_cast<uint32_t>(blocks)),
                     dim3(kThreads), 0, s, t.mats, t.off, t.nmats, scale, h);
  return hipGetLastError();
}

}  // namespace zf
