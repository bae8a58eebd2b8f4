// plas_kernels.hip -- gfx950 kernels of one PLAS sort (Sec. 3.1 of arXiv
// 2312.13299): start arrangement, ingest with the range, separable box blur,
// grouping table, blockwise assignment with its energy, and the controller.
//
// Working layout: a grid is [n][DP], cell-major, DP a power of two (4..64)
// with zero padding beyond the d real channels, stored as float32 or as
// bfloat16 (S = float or S = uint16_t holding bfloat16 bits). A cell of
// DP = 64 is 256 bytes in float32 (two 128-byte lines) or 128 bytes in
// bfloat16 (one line), so the assignment kernel's random cell reads waste
// nothing, and a blur line is read as whole cells. All arithmetic is float32:
// bfloat16 values widen exactly, and results are rounded to bfloat16 (nearest,
// ties to even) only when they are stored.
//
// Floating point: compiled without contraction (-ffp-contract=off) and with
// denormals kept, so every float operation below is one IEEE-rounded add,
// subtract or multiply in the order written. That is what makes the results
// equal, bit for bit, to a CPU that evaluates the same expressions.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <mutex>

#include "plas_launch.h"
#include "plas_random.h"

namespace plas {
namespace {

constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / 64;
constexpr int kIngestTile = 4096;   // values of an ingest tile
constexpr int kFinishBlock = 1024;  // threads of the ingest's last fold
constexpr int kMaxGridBlocks = 4096;
constexpr int kVadBlocks = 1024;    // blocks of a VAD over a grid
constexpr int kVadRows = 16;        // rows of a chunk there
constexpr int kEnergyBlocks = 512;  // blocks of an energy sum
constexpr int kEnergyFlight = 4;    // cells in flight per lane there

inline int blocks_for(int64_t threads, int64_t cap = kMaxGridBlocks) {
  int64_t b = (threads + kBlock - 1) / kBlock;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return static_cast<int>(b);
}

// ---------------------------------------------------------------- storage

// bfloat16 is the high half of a float32: widening is exact.
__device__ __forceinline__ float bf16_to_float(uint32_t bits) { return __uint_as_float(bits << 16); }

// Nearest bfloat16, ties to even: gfx950 converts in one instruction
// (v_cvt_pk_bf16_f32). Every finite value and both infinities round as the
// integer form (add 0x7fff plus the kept part's lowest bit, keep the high
// half) does; a NaN stays a NaN with its sign, so the quiet NaNs that
// arithmetic produces keep their high half too.
__device__ __forceinline__ uint32_t float_to_bf16(float f) {
  return __builtin_bit_cast(unsigned short, static_cast<__bf16>(f));
}

template <typename S>
struct Storage;

template <>
struct Storage<float> {
  using Quad = float4;  // four channels
  __device__ static __forceinline__ float widen(float v) { return v; }
  __device__ static __forceinline__ float narrow(float v) { return v; }
  __device__ static __forceinline__ float4 widen4(float4 q) { return q; }
};

template <>
struct Storage<uint16_t> {
  using Quad = uint2;  // four channels
  __device__ static __forceinline__ float widen(uint16_t v) { return bf16_to_float(v); }
  __device__ static __forceinline__ uint16_t narrow(float v) { return static_cast<uint16_t>(float_to_bf16(v)); }
  __device__ static __forceinline__ float4 widen4(uint2 q) {
    return make_float4(bf16_to_float(q.x & 0xffffu), bf16_to_float(q.x >> 16), bf16_to_float(q.y & 0xffffu),
                       bf16_to_float(q.y >> 16));
  }
};

// ------------------------------------------------- arrangement and ingest

// Before an ingest: clears the query's results, fills the 1/c table (if
// `counts` is given: c = 0..w) and inverts a caller's permutation (if given).
// Entries that no in-range value of perm names keep what inv held before;
// the ingest finds them (arranged_place).
__global__ __launch_bounds__(kBlock) void k_begin(QueryOut* __restrict__ out, const int32_t* __restrict__ perm,
                                                  int64_t n, int32_t* __restrict__ inv, float* __restrict__ counts,
                                                  int w) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
  const int64_t first = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (first == 0) {
    out->bad_value = 0;
    out->bad_perm = 0;
    out->energy = 0;
  }
  if (counts != nullptr)
    for (int64_t c = first; c <= w; c += stride) counts[c] = c == 0 ? 0.0f : 1.0f / static_cast<float>(c);
  if (perm != nullptr)
    for (int64_t p = first; p < n; p += stride) {
      const int32_t v = perm[p];
      if (v >= 0 && v < n) inv[v] = static_cast<int32_t>(p);
    }
}

// P[p] = f(p), the keyed bijection of the start arrangement, and its inverse
// (inv NULL: not).
__global__ __launch_bounds__(kBlock) void k_start_perm(int32_t* __restrict__ P, int32_t* __restrict__ inv, int64_t n,
                                                       Words4 keys) {
  const Bijection f(static_cast<uint64_t>(n), keys.v);
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
  for (int64_t p = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; p < n; p += stride) {
    const int32_t v = static_cast<int32_t>(f(static_cast<uint64_t>(p)));
    P[p] = v;
    if (inv != nullptr) inv[v] = static_cast<int32_t>(p);
  }
}

// Cell i's place under perm, from the inverse k_begin wrote: `at` = inv[i] if
// perm really holds i there, else -1. If that succeeds for all n cells, perm
// takes all n values, so it is a bijection; if perm is one, k_begin wrote
// every entry and it succeeds for all. No counting, no atomics (1024^2 cells:
// 41 us of counters alone before).
__device__ __forceinline__ int32_t arranged_place(const int32_t* __restrict__ perm, int64_t n, int64_t i,
                                                  int32_t at) {
  return at >= 0 && at < n && perm[at] == i ? at : -1;
}

// The check alone: sets *bad if perm is not a bijection.
__global__ __launch_bounds__(kBlock) void k_check_inverse(const int32_t* __restrict__ perm,
                                                          const int32_t* __restrict__ inv, int64_t n,
                                                          int32_t* __restrict__ bad) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
  bool wrong = false;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < n; i += stride)
    wrong |= arranged_place(perm, n, i, inv[i]) < 0;
  if (__any(wrong) && (threadIdx.x & 63) == 0) atomicOr(bad, 1);
}

// features -> G: G[inv[i]] = features[i] (inv NULL: G[i]), padded to DP
// channels and rounded to the storage, with the range of the stored values
// per channel and the check of perm (NULL: not checked) on the way. Tiles of
// 4096 / DP cells go through LDS, so that the reads (64 consecutive cells of
// one channel, or whole cells one after the other) and the writes (whole
// cells) are both contiguous; a block loads its next tile while it stores
// this one. A thread stores one channel, so a block's range reduces over
// every DP-th thread; a NaN counts as an infinite maximum.
//
// Bound by memory: each value is read once and written once, at its place in
// the arranged grid, and the check's random reads ride along (1024^2 x 59
// float32 under a permutation: 112 us and 6 for the fold of the ranges, 4.6
// TB/s; ingest, range, its fold, permutation check and gather took 130, 380,
// 65, 41 and more, and 83 us as passes of their own).
template <int DP, typename SI, typename SO, int LAYOUT>
__global__ __launch_bounds__(kBlock) void k_ingest(const SI* __restrict__ F, int64_t n, int d,
                                                   const int32_t* __restrict__ inv, const int32_t* __restrict__ perm,
                                                   SO* __restrict__ G, float* __restrict__ part,
                                                   QueryOut* __restrict__ out) {
  constexpr int kTile = kIngestTile / DP;             // cells
  constexpr int kEach = kIngestTile / kBlock;         // values per thread
  constexpr int kPlaces = (kTile + kBlock - 1) / kBlock;
  constexpr int kPitch = LAYOUT == 0 ? kTile + 1 : DP;
  __shared__ float tile[LAYOUT == 0 ? DP * kPitch : kIngestTile];
  __shared__ int32_t s_at[kTile];
  __shared__ float s_lo[kBlock], s_hi[kBlock];
  const int t = threadIdx.x;
  const int64_t tiles = (n + kTile - 1) / kTile;
  SI value[kEach];
  int32_t at[kPlaces];
  // CN: thread t loads cells t % kTile of channels t / kTile + ..; NC: the
  // tile's d values per cell are one run.
  auto load = [&](int64_t index) {
    const int64_t n0 = index * kTile;
    const int cells = static_cast<int>(n - n0 < kTile ? n - n0 : kTile);
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
      const int e = k * kBlock + t;
      value[k] = SI(0);
      if constexpr (LAYOUT == 0) {
        const int c = e / kTile, i = e % kTile;
        if (c < d && i < cells) value[k] = F[static_cast<int64_t>(c) * n + n0 + i];
      } else {
        if (e < cells * d) value[k] = F[n0 * d + e];
      }
    }
#pragma unroll
    for (int k = 0; k < kPlaces; ++k) {
      const int i = k * kBlock + t;
      at[k] = -1;
      if (i < cells) at[k] = inv != nullptr ? inv[n0 + i] : static_cast<int32_t>(n0 + i);
    }
  };
  const int c = t % DP;
  float lo = INFINITY, hi = -INFINITY;
  bool wrong = false;
  int64_t index = blockIdx.x;
  if (index < tiles) load(index);
  for (; index < tiles; index += gridDim.x) {
    const int64_t n0 = index * kTile;
    const int cells = static_cast<int>(n - n0 < kTile ? n - n0 : kTile);
    if (perm != nullptr) {
#pragma unroll
      for (int k = 0; k < kPlaces; ++k) {
        const int i = k * kBlock + t;
        if (i < cells) {
          at[k] = arranged_place(perm, n, n0 + i, at[k]);
          wrong |= at[k] < 0;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
      const int e = k * kBlock + t;
      const float v = Storage<SI>::widen(value[k]);
      if constexpr (LAYOUT == 0)
        tile[(e / kTile) * kPitch + e % kTile] = v;
      else
        tile[e] = v;
    }
#pragma unroll
    for (int k = 0; k < kPlaces; ++k)
      if (k * kBlock + t < kTile) s_at[k * kBlock + t] = at[k];
    __syncthreads();
    if (index + gridDim.x < tiles) load(index + gridDim.x);
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
      const int i = k * (kBlock / DP) + t / DP;
      if (i < cells) {
        float v;
        if constexpr (LAYOUT == 0)
          v = tile[c * kPitch + i];
        else
          v = c < d ? tile[i * d + c] : 0.0f;
        const SO stored = Storage<SO>::narrow(v);
        const float r = Storage<SO>::widen(stored);
        lo = fminf(lo, r);
        hi = r == r ? fmaxf(hi, r) : INFINITY;
        const int32_t place = s_at[i];
        if (place >= 0) G[static_cast<int64_t>(place) * DP + c] = stored;
      }
    }
    __syncthreads();
  }
  s_lo[t] = lo;
  s_hi[t] = hi;
  __syncthreads();
  if (t < DP) {
    for (int i = t + DP; i < kBlock; i += DP) {
      lo = fminf(lo, s_lo[i]);
      hi = fmaxf(hi, s_hi[i]);
    }
    float* mine = part + static_cast<int64_t>(blockIdx.x) * 2 * DP;
    mine[t] = lo;
    mine[DP + t] = hi;
  }
  if (__any(wrong) && (t & 63) == 0) atomicOr(&out->bad_perm, 1);
}

// The blocks' ranges to the features' range and its energy scale, by one
// block: a thread folds every R-th block's four minima or maxima, then the R
// rows fold in LDS. QueryOut's ranges hold d channels.
template <int DP>
__global__ __launch_bounds__(kFinishBlock) void k_ingest_finish(const float* __restrict__ part, int nparts, int d,
                                                                int64_t n, QueryOut* __restrict__ out) {
  constexpr int kCols = DP / 2;  // quads of one block's 2 DP values
  constexpr int kRows = kFinishBlock / kCols;
  __shared__ float4 s_fold[kFinishBlock];
  const int t = threadIdx.x, col = t % kCols;
  const bool minimum = col < kCols / 2;
  const float none = minimum ? INFINITY : -INFINITY;
  auto fold = [minimum](float4 a, const float4 b) {
    a.x = minimum ? fminf(a.x, b.x) : fmaxf(a.x, b.x);
    a.y = minimum ? fminf(a.y, b.y) : fmaxf(a.y, b.y);
    a.z = minimum ? fminf(a.z, b.z) : fmaxf(a.z, b.z);
    a.w = minimum ? fminf(a.w, b.w) : fmaxf(a.w, b.w);
    return a;
  };
  const float4* __restrict__ rows = reinterpret_cast<const float4*>(part);
  float4 v = make_float4(none, none, none, none);
#pragma unroll 8
  for (int b = t / kCols; b < nparts; b += kRows) v = fold(v, rows[static_cast<int64_t>(b) * kCols + col]);
  s_fold[t] = v;
  __syncthreads();
  for (int step = kFinishBlock / 2; step >= kCols; step >>= 1) {
    if (t < step) s_fold[t] = fold(s_fold[t], s_fold[t + step]);
    __syncthreads();
  }
  const float* lo = reinterpret_cast<const float*>(s_fold);
  const float* hi = lo + DP;
  if (t < d) {
    out->lo[t] = lo[t];
    out->hi[t] = hi[t];
    if (!__builtin_isfinite(lo[t]) || !__builtin_isfinite(hi[t])) atomicOr(&out->bad_value, 1);
  }
  if (t == 0) out->s = scale_shift(lo, hi, d, n);
}

// ------------------------------------------------------------------- blur

// The radius of a pass over lines of w positions: st->r, or the fixed radius
// when st is NULL. Every window of half-width w - 1 or more is the whole line,
// so it is clipped there, for every kernel: callers may give any radius, and
// the walks take r / 16 steps more than the line has and add r to positions.
// Returns false when the sort has ended (every kernel queued after the end
// returns at once).
__device__ __forceinline__ bool pass_radius(const DevState* __restrict__ st, int radius, int w, int& r) {
  if (st != nullptr && st->done) return false;
  r = st != nullptr ? st->r : radius;
  if (r > w - 1) r = w - 1;
  return true;
}

// table[t] = pi(t) packed as (ly << 16) | lx, pi the grouping bijection of
// a reorder over the beta^2 block-local cells, filled by all blocks of a
// launch (NT threads each). The first row pass of a reorder runs it after
// its lines, from the state's beta and keys.
template <int NT>
__device__ __forceinline__ void fill_group_table(int32_t* __restrict__ table, int beta, const uint64_t keys[4],
                                                 int64_t bid, int64_t nblocks) {
  const uint64_t cells = static_cast<uint64_t>(beta) * beta;
  const Bijection f(cells, keys);
  const uint64_t stride = static_cast<uint64_t>(nblocks) * NT;
  for (uint64_t t = static_cast<uint64_t>(bid) * NT + threadIdx.x; t < cells; t += stride) {
    const uint32_t v = static_cast<uint32_t>(f(t));
    const uint32_t ly = v / static_cast<uint32_t>(beta);
    const uint32_t lx = v - ly * static_cast<uint32_t>(beta);
    table[t] = static_cast<int32_t>((ly << 16) | lx);
  }
}

// Orders this wave's LDS writes before its later LDS reads (lanes of one
// wave exchange data through LDS without a block barrier).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}


// One separable box-blur pass. Lane = (line, channel): DP consecutive lanes
// walk one line, 64 / DP lines per wave. Along the line the window sum is
// kept as a running sum: it starts as the ascending sum of the first
// r + 1 values; at each next position the entering value is added
// and then the leaving value subtracted, and the output is the running sum
// times float32(1 / count) for the window clipped to the grid.
//
// The running sum is a serial chain per (line, channel), so a wave cannot
// hide memory latency by switching lines. Instead each lane keeps the loads
// of the next kBlurUnroll positions in flight while it adds up the current
// ones (two register buffers used in turn). The line is cut into ranges where
// "a value enters" and "a value leaves" are fixed, which keeps the unrolled
// loops free of per-position tests; the position x is the same for all lanes
// of a wave, so every remaining branch is uniform.
#ifndef PLAS_BLUR_UNROLL
#define PLAS_BLUR_UNROLL 12
#endif
constexpr int kBlurUnroll = PLAS_BLUR_UNROLL;

template <typename S>
struct BlurLine {
  const S* __restrict__ src;
  S* __restrict__ dst;
  int64_t step;
  const float* __restrict__ inv;
  int w;
  int r;

  __device__ __forceinline__ float load(int t) const {
    return Storage<S>::widen(src[static_cast<int64_t>(t) * step]);
  }
  // float32(1/count) of output position x (window clipped to the line).
  __device__ __forceinline__ float mult(int x) const {
    const int hi = x + r < w - 1 ? x + r : w - 1;
    const int lo = x - r > 0 ? x - r : 0;
    return inv[hi - lo + 1];
  }
  __device__ __forceinline__ void store(int x, float s, float m) const {
    dst[static_cast<int64_t>(x) * step] = Storage<S>::narrow(s * m);
  }
  __device__ static __forceinline__ float widen(S v) { return Storage<S>::widen(v); }
  __device__ static __forceinline__ S narrow(float v) { return Storage<S>::narrow(v); }
};

// kBlurUnroll positions' entering values, leaving values and multipliers.
struct BlurBlock {
  float enter[kBlurUnroll];
  float leave[kBlurUnroll];
  float mult[kBlurUnroll];
};

// Addresses advance by one step per position (a 64-bit add) instead of
// being recomputed from the position (a 64-bit multiply each).
template <bool ENTER, bool LEAVE, typename L_t>
__device__ __forceinline__ void blur_fetch(const L_t& L, int x0, BlurBlock& B) {
  const auto* pe = L.src;
  const auto* pl = L.src;
  if (ENTER) pe += static_cast<int64_t>(x0 + L.r) * L.step;
  if (LEAVE) pl += static_cast<int64_t>(x0 - L.r - 1) * L.step;
#pragma unroll
  for (int i = 0; i < kBlurUnroll; ++i) {
    if (ENTER) {
      B.enter[i] = L.widen(*pe);
      pe += L.step;
    }
    if (LEAVE) {
      B.leave[i] = L.widen(*pl);
      pl += L.step;
    }
    B.mult[i] = L.mult(x0 + i);
  }
}

template <bool ENTER, bool LEAVE, typename L_t>
__device__ __forceinline__ void blur_apply(const L_t& L, int x0, const BlurBlock& B, float& s) {
  auto* pd = L.dst + static_cast<int64_t>(x0) * L.step;
#pragma unroll
  for (int i = 0; i < kBlurUnroll; ++i) {
    if (ENTER) s = s + B.enter[i];
    if (LEAVE) s = s - B.leave[i];
    *pd = L.narrow(s * B.mult[i]);
    pd += L.step;
  }
}

// Wait until every vector memory operation of this wave has completed
// (s_waitcnt vmcnt(0); expcnt and lgkmcnt left at their maxima).
__device__ __forceinline__ void wait_vmem() {
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __builtin_amdgcn_sched_barrier(0);
}


// Positions [xb, xe) where entering/leaving values exist as ENTER/LEAVE say.
// Loads and stores share one memory counter, so with the previous block's
// stores in flight the compiler can only wait for all outstanding memory
// operations before a block's values are used; left to itself it would do
// so after the next block's loads were issued and wait for those too. The
// explicit wait comes first, the next block's fetch is issued after it and
// flies while the current block is summed and stored.
template <bool ENTER, bool LEAVE, typename L_t>
__device__ __forceinline__ void blur_range(const L_t& L, int xb, int xe, float& s) {
  const int full = (xe - xb) / kBlurUnroll;
  int x = xb;
  if (full > 0) {
    BlurBlock next, cur;
    blur_fetch<ENTER, LEAVE>(L, x, next);
    for (int c = 0; c < full; ++c) {
      wait_vmem();
      cur = next;
      if (c + 1 < full) blur_fetch<ENTER, LEAVE>(L, x + kBlurUnroll, next);
      blur_apply<ENTER, LEAVE>(L, x, cur, s);
      x += kBlurUnroll;
    }
  }
  for (; x < xe; ++x) {
    if (ENTER) s = s + L.load(x + L.r);
    if (LEAVE) s = s - L.load(x - L.r - 1);
    L.store(x, s, L.mult(x));
  }
}

// Lines wave * 64/DP .. of one pass, by wave `wave` of the pass.
template <int DP, typename S>
__device__ __forceinline__ void blur_reg_lines(const S* __restrict__ in, S* __restrict__ out, int w, int r,
                                               int vertical, const float* __restrict__ inv, int64_t wave,
                                               int lane) {
  constexpr int LPW = 64 / DP;
  const int64_t line = wave * LPW + lane / DP;
  const int c = lane % DP;
  if (line >= w) return;
  const int64_t base = vertical ? line * DP + c : line * w * DP + c;
  BlurLine<S> L;
  L.src = in + base;
  L.dst = out + base;
  L.step = vertical ? static_cast<int64_t>(w) * DP : DP;
  L.inv = inv;
  L.w = w;
  L.r = r;
  if (r == 0) {
    for (int x = 0; x < w; ++x) L.dst[x * L.step] = L.src[x * L.step];
    return;
  }
  // Start: ascending sum of positions 0 .. r, loaded kBlurUnroll at a time.
  float s = L.load(0);
  int t = 1;
  for (; t + kBlurUnroll - 1 <= r; t += kBlurUnroll) {
    float v[kBlurUnroll];
#pragma unroll
    for (int i = 0; i < kBlurUnroll; ++i) v[i] = L.load(t + i);
#pragma unroll
    for (int i = 0; i < kBlurUnroll; ++i) s = s + v[i];
  }
  for (; t <= r; ++t) s = s + L.load(t);
  L.store(0, s, L.mult(0));
  // Position x has an entering value iff x + r <= w - 1 and a leaving value
  // iff x - r - 1 >= 0. Both bounds split [1, w) into at most three ranges.
  const int enter_end = w - r;    // x < enter_end: entering
  const int leave_begin = r + 1;  // x >= leave_begin: leaving
  if (enter_end <= leave_begin) {
    blur_range<true, false>(L, 1, enter_end, s);
    blur_range<false, false>(L, enter_end, leave_begin, s);
    blur_range<false, true>(L, leave_begin, w, s);
  } else {
    blur_range<true, false>(L, 1, leave_begin, s);
    blur_range<true, true>(L, leave_begin, enter_end, s);
    blur_range<false, true>(L, enter_end, w, s);
  }
}

// Waves of one pass for DP < 64 (64 / DP lines per wave).
template <int DP>
inline int64_t blur_reg_waves(int w) {
  return (w + 64 / DP - 1) / (64 / DP);
}

template <int DP, typename S>
__global__ __launch_bounds__(kBlock) void k_blur(const S* __restrict__ in, S* __restrict__ out,
                                                 int w, const DevState* __restrict__ st, int radius,
                                                 int vertical, const float* __restrict__ inv,
                                                 int32_t* __restrict__ table) {
  int r;
  if (!pass_radius(st, radius, w, r)) return;
  const int64_t wave = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) >> 6;
  blur_reg_lines<DP, S>(in, out, w, r, vertical, inv, wave, threadIdx.x & 63);
  if (table != nullptr) fill_group_table<kBlock>(table, st->beta, st->keys, blockIdx.x, gridDim.x);
}

// Cache hint, measured on whole sorts. The assignment reads every cell of G
// and T once per reorder, in random group order: streaming (non-temporal)
// loads keep those reads from evicting what the next blur pass reads (1024^2
// float32 with normal loads: assignment 109 -> 132 us). Cells smaller than a
// 128-byte line share it with neighbours that other groups read, so there the
// lines stay (2091^2 x 16 float32: 198 -> 187 us; 512^2 x 4: 15.8 -> 14.5).
template <typename S, int DP>
constexpr bool assign_stream_loads() {
  return DP * static_cast<int>(sizeof(S)) >= 128;
}

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

// Streaming-hint load / store of a Quad (float4 or uint2), as above.
template <bool nt, typename Q>
__device__ __forceinline__ Q load_quad(const Q* p) {
  if constexpr (nt && sizeof(Q) == 16) {
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return __builtin_bit_cast(Q, v);
  } else if constexpr (nt && sizeof(Q) == 8) {
    const u32x2_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t*>(p));
    return __builtin_bit_cast(Q, v);
  } else {
    return *p;
  }
}

template <bool nt>
__device__ __forceinline__ void store_quad(float* p, const float4& v) {
  if constexpr (nt)
    __builtin_nontemporal_store(__builtin_bit_cast(u32x4_t, v), reinterpret_cast<u32x4_t*>(p));
  else
    *reinterpret_cast<float4*>(p) = v;
}

// Blur pass for cells of at least 16 bytes: same arithmetic as k_blur (one
// running sum per line and channel, same operation order), with the work of a
// group of 64 / DP lines split over three waves of a block that meet at a
// barrier once per chunk of 16 positions:
//
//  - the loading wave moves 16-byte pieces from global memory straight to an
//    LDS ring (gfx950's direct loads: the data never passes through
//    registers). A ring row holds one position of all the group's lines
//    (element l * DP + c is channel c of line l). It does nothing else, so its
//    waits never hold up the sums, and it runs kDepth chunks ahead of them;
//  - the summing wave runs the chains, lane l * DP + c that of channel c of
//    line l: per position one addition, one subtraction and one LDS write of
//    the sum. It reads a step's values during the step before, because an LDS
//    read beside the direct loads' writes takes hundreds of cycles;
//  - the storing wave multiplies the sums of the step before by 1 / count and
//    stores them as 16-byte pieces.
//
// What bounds it: with few lines (small or narrow grids) the serial chain,
// about 41 cycles per position; with many, memory. One wave that did all three
// in turn took 135 cycles per position, waiting for its own LDS round trips:
// 512^2 x 4 float32 33 -> 12 us per pass (r = 1; 42 -> 22 us at r = 255), 700^2
// x 16 float32 45 -> 18 us, 300^2 x 64 float32 23 -> 12 us, 724^2 x 64 bfloat16
// 57 -> 26 us, 2091^2 x 64 float32 641 -> 455 us (r = 20; with streaming
// stores about 430). Two waves (the sums stored by the summing wave) reached 15
// us on the first of these.
//
// Steps walk t = 0 .. w - 1 + r. Every t < w adds value t to the sum (up to t
// = r that is the starting sum, from then on the entering value of output
// x = t - r), every t >= 2r + 1 subtracts value t - 2r - 1 (the leaving value
// of x), and every t >= r gives output x. So the values a step adds are
// exactly one loaded chunk. While the ring holds the leaving values beside
// the chunks in flight they are read back from it; otherwise its second half
// holds leaving chunks, loaded a second time (the same positions, cut so that
// a step's leaving values are exactly one chunk).
//
// Loads are issued at positions clamped into the line (a clamped load fetches
// a value the sums never use), so every chunk is exactly kVec instructions.
// Vector memory operations of a wave complete in issue order, so "slot u has
// arrived" is "at most as many operations are outstanding as were issued
// after slot u". The loads are written as asm so that the compiler does not
// add its own wait for all of them; M0 (the LDS base of a load) is set in the
// same asm statement, and no compiler-generated code of these kernels uses M0.
constexpr int kRelayRows = 128;  // ring rows
constexpr int kRelayWaves = 3;   // waves per line group
template <typename S>
struct RelayShape {
  static constexpr int kRowBytes = 64 * static_cast<int>(sizeof(S));  // one position of the group's lines
  static constexpr int kLanesPerRow = kRowBytes / 16;
  static constexpr int kPos = 64 / kLanesPerRow;  // positions per load instruction: 4 (float32), 8 (bfloat16)
  static constexpr int kChunk = 16;               // positions per chunk
  static constexpr int kVec = kChunk / kPos;      // load instructions per chunk
  static constexpr int kSlots = kRelayRows / kChunk;      // chunks of the whole ring
  static constexpr int kHalf = kSlots / 2;        // chunks of each region of the split ring
  // Chunks the loads run ahead of the sums.
  static constexpr int kDepth = kHalf;
  static_assert(kRelayRows % kChunk == 0 && kDepth >= 2, "ring shape");
  static_assert(2 * kVec * (kDepth - 2) < 64, "loads in flight fit the wait counter");
};

// LDS of one line group: the ring, and the sums of two steps (40 KB float32,
// 24 KB bfloat16: four float32 groups share a CU).
template <typename S>
struct alignas(16) RelayLds {
  S ring[kRelayRows][64];
  float sums[2 * RelayShape<S>::kChunk][64];
};

// Cache hints of the load streams. The leaving stream (a second read of
// positions the entering stream read 2r + 1 positions earlier) streams
// through, so that it does not evict entering data the L2 still holds for
// it. The entering stream streams in the column pass when the grids in
// flight exceed 128 MiB (blur_large_working_set): its input H is dead after
// that pass, and keeping H out of the Infinity Cache leaves room for G and
// T, which the assignment reads next (1024^2 float32: column pass 98 -> 87
// us, assignment 110 -> 104 us at r <= 15). Streaming the row pass's loads
// of G as well made the column pass slower again (101 us); grids the cache
// holds whole ran 1-2 % slower with streaming column loads.
constexpr bool kBlurLeaveStream = true;

// One direct load: 16 bytes per lane from `src` to LDS byte address
// m0 + 16 * lane, with a streaming hint (the data is not read again through
// the cache) when `nt`.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // M0 is named as clobbered on purpose
template <bool nt>
__device__ __forceinline__ void dma16_load(const void* src, uint32_t m0) {
  if constexpr (nt)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
                 :
                 : "v"(src), "s"(m0)
                 : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :
                 : "v"(src), "s"(m0)
                 : "memory", "m0");
}
#pragma clang diagnostic pop

template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// s_waitcnt vmcnt(n) for n = chunks * VEC loads, n uniform.
template <int VEC, int MAXC>
__device__ __forceinline__ void wait_chunks(int chunks) {
  if constexpr (MAXC == 0) {
    wait_vm<0>();
  } else {
    if (chunks >= MAXC)
      wait_vm<VEC * MAXC>();
    else
      wait_chunks<VEC, MAXC - 1>(chunks);
  }
}

// All of this wave's LDS accesses done, then the block's barrier.
__device__ __forceinline__ void relay_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); }

// One chunk's stored values of a lane, widened where they are used (not where
// they are read: that would wait for the reads).
template <typename S>
struct ChunkValues;
template <>
struct ChunkValues<float> {
  float v[16];
  __device__ __forceinline__ void set(int i, float x) { v[i] = x; }
  __device__ __forceinline__ float get(int i) const { return v[i]; }
};

template <>
struct ChunkValues<uint16_t> {
  uint32_t v[16];
  __device__ __forceinline__ void set(int i, uint16_t x) { v[i] = x; }
  __device__ __forceinline__ float get(int i) const { return bf16_to_float(v[i]); }
};

template <typename S, int DP, bool NTS>
struct RelayLine {
  using Sh = RelayShape<S>;
  static constexpr int kChunk = Sh::kChunk;
  static constexpr int kPiecesPerCell = DP * static_cast<int>(sizeof(S)) / 16;
  static_assert(kPiecesPerCell >= 1, "a cell must hold at least one 16-byte piece");
  int w, r;
  int n_chunks;  // chunks of the line
  int n_steps;   // chunks of t = 0 .. w - 1 + r
  bool split;    // the leaving values have their own region (the ring's second half)
  bool stream;   // the entering loads stream
  int lane;
  S (*ring)[64];
  float (*sums)[64];

  __device__ __forceinline__ void init(int w_, int r_, bool stream_, int lane_, RelayLds<S>& lds) {
    w = w_;
    r = r_;
    lane = lane_;
    stream = stream_;
    ring = lds.ring;
    sums = lds.sums;
    n_chunks = (w + kChunk - 1) / kChunk;
    n_steps = (w + r + kChunk - 1) / kChunk;
    split = (2 * r + kChunk) / kChunk > Sh::kSlots - Sh::kDepth;  // ceil((2r + 1) / kChunk)
  }

  // ---- loading wave

  // kVec loads of positions pos0 .. pos0 + kChunk - 1 (clamped into the
  // line) into slot `slot`. p0: this lane's piece at position 0; step:
  // elements between positions.
  template <bool nt>
  __device__ __forceinline__ void load_chunk(const S* p0, int64_t step, int pos0, int slot, uint32_t ring_m0) const {
    const int q = lane / Sh::kLanesPerRow;
    const uint32_t m0 = ring_m0 + static_cast<uint32_t>(slot * kChunk * Sh::kRowBytes);
    if (pos0 >= 0 && pos0 + kChunk - 1 <= w - 1) {
      const S* p = p0 + static_cast<int64_t>(pos0 + q) * step;
      const int64_t inc = static_cast<int64_t>(Sh::kPos) * step;
#pragma unroll
      for (int i = 0; i < Sh::kVec; ++i) dma16_load<nt>(p + i * inc, m0 + i * 1024u);
    } else {
#pragma unroll
      for (int i = 0; i < Sh::kVec; ++i) {
        const int t = pos0 + Sh::kPos * i + q;
        dma16_load<nt>(p0 + static_cast<int64_t>(t < 0 ? 0 : t < w ? t : w - 1) * step, m0 + i * 1024u);
      }
    }
  }

  __device__ __forceinline__ void load_side(const S* p0, int64_t step, uint32_t ring_m0) const {
    const int enter_slots = split ? Sh::kHalf : Sh::kSlots;
    const int lag = (2 * r + 1) / kChunk;  // the first step with a leaving value
    int enter_slot = 0, leave_slot = 0;
    auto issue = [&](int u) {
      if (u < n_chunks) {
        if (stream)
          load_chunk<true>(p0, step, u * kChunk, enter_slot, ring_m0);
        else
          load_chunk<false>(p0, step, u * kChunk, enter_slot, ring_m0);
        enter_slot = enter_slot + 1 == enter_slots ? 0 : enter_slot + 1;
      }
      if (split && u < n_steps) {
        if (u >= lag)
          load_chunk<kBlurLeaveStream>(p0, step, u * kChunk - 2 * r - 1, Sh::kHalf + leave_slot, ring_m0);
        leave_slot = leave_slot + 1 == Sh::kHalf ? 0 : leave_slot + 1;
      }
    };
    // Chunks issued by slots u0 .. u1.
    auto issued = [&](int u0, int u1) {
      const int e = min(u1, n_chunks - 1) - u0 + 1;
      const int l = split ? min(u1, n_steps - 1) - max(u0, lag) + 1 : 0;
      return max(e, 0) + max(l, 0);
    };
    for (int u = 0; u < Sh::kDepth; ++u) issue(u);
    wait_chunks<Sh::kVec, 2 * (Sh::kDepth - 2)>(issued(2, Sh::kDepth - 1));
    relay_barrier();
    relay_barrier();
    for (int e = 0; e < n_steps; ++e) {
      issue(e + Sh::kDepth);
      wait_chunks<Sh::kVec, 2 * (Sh::kDepth - 2)>(issued(e + 3, e + Sh::kDepth));
      relay_barrier();
    }
    relay_barrier();
  }

  // ---- summing wave

  // What a step adds (e) and subtracts (l).
  static_assert(kChunk == 16, "ChunkValues holds 16 positions");
  struct Values {
    ChunkValues<S> e, l;
  };
  // Where the summing wave stands: the step, the region rows of its chunk and
  // of its first leaving position, and the running sum.
  struct Cursor {
    int e, row, lb, erows, lbase;
    float s;
  };

  // kChunk rows from row b of the region of `rows` rows at `base`.
  __device__ __forceinline__ void read_rows(ChunkValues<S>& v, int base, int b, int rows) const {
    if (b + kChunk <= rows) {
      const S* p = &ring[base + b][lane];
#pragma unroll
      for (int i = 0; i < kChunk; ++i) v.set(i, p[i * 64]);
      asm volatile("" : : : "memory");  // keeps the two ways apart
    } else {
      // Byte offsets from the region's start: past its end the smaller of
      // the offset and the (unsigned) offset less the region's size.
      const char* from = reinterpret_cast<const char*>(&ring[base][0]);
      const uint32_t size = static_cast<uint32_t>(rows) * Sh::kRowBytes;
      uint32_t at = static_cast<uint32_t>(b) * Sh::kRowBytes + static_cast<uint32_t>(lane * sizeof(S));
      asm volatile("" : "+v"(at));  // the offsets below are made here, not kept in registers all along
#pragma unroll
      for (int i = 0; i < kChunk; ++i) {
        const uint32_t o = at + i * Sh::kRowBytes;
        v.set(i, *reinterpret_cast<const S*>(from + min(o, o - size)));
      }
      asm volatile("" : : : "memory");
    }
  }
  // The values of the step at c.row / c.lb, which then moves on.
  __device__ __forceinline__ void read_values(Cursor& c, Values& v) const {
    const S* p = &ring[c.row][lane];
#pragma unroll
    for (int i = 0; i < kChunk; ++i) v.e.set(i, p[i * 64]);
    read_rows(v.l, c.lbase, c.lb, c.erows);
    c.row = c.row + kChunk == c.erows ? 0 : c.row + kChunk;
    c.lb = c.lb + kChunk >= c.erows ? c.lb + kChunk - c.erows : c.lb + kChunk;
  }

  // One step whose every t adds (ADD) and subtracts (SUB) a value, or none does.
  template <bool ADD, bool SUB>
  __device__ __forceinline__ void even_step(const Values& cur, Values& next, Cursor& c) const {
    read_values(c, next);
    __builtin_amdgcn_sched_barrier(0);
    float* o = &sums[(c.e & 1) * kChunk][lane];
#pragma unroll
    for (int p = 0; p < kChunk; ++p) {
      if (ADD) c.s = c.s + cur.e.get(p);
      if (SUB) c.s = c.s - cur.l.get(p);
      o[p * 64] = c.s;
    }
    ++c.e;
    relay_barrier();
  }
  // n such steps; the values of the first are in a, and so are in the end
  // those of the step after the last.
  template <bool ADD, bool SUB>
  __device__ __forceinline__ void even_steps(int n, Values& a, Values& b, Cursor& c) const {
    for (; n >= 2; n -= 2) {
      even_step<ADD, SUB>(a, b, c);
      even_step<ADD, SUB>(b, a, c);
    }
    if (n == 1) {
      even_step<ADD, SUB>(a, b, c);
      a = b;
    }
  }
  // Any step. Where no value enters, -0 is added and where none leaves, +0
  // is subtracted: both leave every sum as it is.
  __device__ __forceinline__ void mixed_step(Values& a, Cursor& c) const {
    const int t0 = c.e * kChunk;
    const int no_add = w - t0, sub_from = 2 * r + 1 - t0;
    float* o = &sums[(c.e & 1) * kChunk][lane];
#pragma unroll
    for (int p = 0; p < kChunk; ++p) {
      c.s = c.s + (p < no_add ? a.e.get(p) : -0.0f);
      c.s = c.s - (p >= sub_from ? a.l.get(p) : 0.0f);
      o[p * 64] = c.s;
    }
    read_values(c, a);
    ++c.e;
    relay_barrier();
  }

  __device__ __forceinline__ void sum_side() const {
    // Chunks wholly below these bounds of t: every t adds, no t subtracts yet.
    const int adds = w / kChunk, no_sub = (2 * r + 1) / kChunk;
    Cursor c;
    c.e = 0;
    c.row = 0;
    c.erows = (split ? Sh::kHalf : Sh::kSlots) * kChunk;
    c.lbase = split ? Sh::kHalf * kChunk : 0;
    // Split: step e reads slot e of the second region. Else the position's row.
    c.lb = split ? 0 : c.erows - 2 * r - 1;
    c.s = -0.0f;  // adding the first value to it gives that value
    Values a, b;
    relay_barrier();
    read_values(c, a);
    relay_barrier();  // the first chunk may be overwritten
    while (c.e < n_steps) {
      const int t0 = c.e * kChunk;
      const bool all_sub = t0 >= 2 * r + 1;
      if (c.e < adds && all_sub)
        even_steps<true, true>(adds - c.e, a, b, c);
      else if (c.e < min(adds, no_sub))
        even_steps<true, false>(min(adds, no_sub) - c.e, a, b, c);
      else if (t0 >= w && all_sub)
        even_steps<false, true>(n_steps - c.e, a, b, c);
      else
        mixed_step(a, c);
    }
    relay_barrier();
  }

  // ---- storing wave

  // Output x = t - r of a sum is s / count. Lane (q, j) stores the 16-byte
  // piece j of positions q, q + kPos, ..; dst0: its address at position 0.
  __device__ __forceinline__ void store_side(S* dst0, int64_t step, bool ok) const {
    constexpr int kPiece = 16 / static_cast<int>(sizeof(S));  // values of a piece
    const int q = lane / Sh::kLanesPerRow, j = lane % Sh::kLanesPerRow;
    const float m_inner = 1.0f / static_cast<float>(2 * r + 1);
    S* at = dst0 + static_cast<int64_t>(q - r) * step;
    const int64_t inc = Sh::kPos * step;
    const float* from = &sums[q][kPiece * j];
    relay_barrier();
    relay_barrier();
    for (int e = 0; e < n_steps; ++e) {
      const int x0 = e * kChunk - r;
      const bool inner = x0 >= r && x0 + kChunk - 1 + r <= w - 1;
      float m[Sh::kVec];
#pragma unroll
      for (int i = 0; i < Sh::kVec; ++i) m[i] = m_inner;
      if (!inner) {
#pragma unroll
        for (int i = 0; i < Sh::kVec; ++i) {
          const int t = x0 + Sh::kPos * i + q;
          const int x = t < 0 ? 0 : t < w - 1 ? t : w - 1;
          m[i] = 1.0f / static_cast<float>((x + r < w - 1 ? x + r : w - 1) - (x - r > 0 ? x - r : 0) + 1);
        }
      }
      relay_barrier();
      const float* rows = from + (e & 1) * kChunk * 64;
      float v[Sh::kVec][kPiece];
#pragma unroll
      for (int i = 0; i < Sh::kVec; ++i)
#pragma unroll
        for (int k = 0; k < kPiece; k += 4) {
          const float4 f = *reinterpret_cast<const float4*>(rows + i * Sh::kPos * 64 + k);
          v[i][k] = f.x * m[i];
          v[i][k + 1] = f.y * m[i];
          v[i][k + 2] = f.z * m[i];
          v[i][k + 3] = f.w * m[i];
        }
      S* p = at;
      if (inner) {
        if (ok) {
#pragma unroll
          for (int i = 0; i < Sh::kVec; ++i, p += inc) store_piece(p, v[i]);
        }
      } else {
#pragma unroll
        for (int i = 0; i < Sh::kVec; ++i, p += inc) {
          const int x = x0 + Sh::kPos * i + q;
          if (x >= 0 && x < w && ok) store_piece(p, v[i]);
        }
      }
      at += kChunk * step;
    }
    relay_barrier();
  }
  __device__ static __forceinline__ void store_piece(S* dst, const float (&v)[16 / sizeof(S)]) {
    if constexpr (sizeof(S) == 4) {
      store_quad<NTS>(dst, make_float4(v[0], v[1], v[2], v[3]));
    } else {
      uint4 u;
      u.x = float_to_bf16(v[0]) | (float_to_bf16(v[1]) << 16);
      u.y = float_to_bf16(v[2]) | (float_to_bf16(v[3]) << 16);
      u.z = float_to_bf16(v[4]) | (float_to_bf16(v[5]) << 16);
      u.w = float_to_bf16(v[6]) | (float_to_bf16(v[7]) << 16);
      *reinterpret_cast<uint4*>(dst) = u;
    }
  }
};

// Lines of one relay blur pass, GPB line groups (GPB * kRelayWaves waves) per
// block: group `sub` of block `bid` takes lines (bid * GPB + sub) * 64/DP ..
// and walks on with a stride. Every group of a block takes the same number of
// steps (past the last line it repeats that line without storing), so that
// all its waves meet at the same barriers. NTS: streaming stores (see
// relay_streams_stores).
template <typename S, int DP, int GPB, bool NTS>
__device__ __forceinline__ void blur_relay_lines(const S* __restrict__ in, S* __restrict__ out, int w, int r,
                                                 int vertical, bool stream, int64_t bid, int64_t nblocks,
                                                 RelayLds<S>* lds) {
  constexpr int kLines = 64 / DP;
  using Sh = RelayShape<S>;
  using L_t = RelayLine<S, DP, NTS>;
  const int wib = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int sub = wib / kRelayWaves, role = wib % kRelayWaves;
  const int64_t step = vertical ? static_cast<int64_t>(w) * DP : DP;       // elements between positions of a line
  const int64_t line_step = vertical ? DP : static_cast<int64_t>(w) * DP;  // and between lines
  if (r == 0) {
    if (role != 0) return;
    for (int64_t g = bid * GPB + sub; g * kLines < w; g += nblocks * GPB) {
      const int64_t line = g * kLines + lane / DP;
      if (line >= w) continue;
      const int64_t base = line * line_step + lane % DP;
      for (int x = 0; x < w; ++x) out[base + x * step] = in[base + x * step];
    }
    return;
  }
  L_t L;
  L.init(w, r, stream, lane, lds[sub]);
  const int j = lane % Sh::kLanesPerRow;
  // Each role has its own loop over the line groups, so that a wave holds its
  // own role's values only.
  auto each_group = [&](auto&& work) __attribute__((always_inline)) {
    for (int64_t g0 = bid * GPB; g0 * kLines < w; g0 += nblocks * GPB) {
      const int64_t want = (g0 + sub) * kLines + j / L_t::kPiecesPerCell;
      const int64_t line = want < w ? want : w - 1;
      work(line * line_step + (j % L_t::kPiecesPerCell) * (16 / static_cast<int>(sizeof(S))), want < w);
    }
  };
  if (role == 0) {
    const uint32_t ring_m0 = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(
        reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) S*)(&lds[sub].ring[0][0]))));
    each_group([&](int64_t piece, bool) { L.load_side(in + piece, step, ring_m0); });
  } else if (role == 1) {
    each_group([&](int64_t, bool) { L.sum_side(); });
  } else {
    each_group([&](int64_t piece, bool ok) { L.store_side(out + piece, step, ok); });
  }
}

// Waves per SIMD of a relay kernel: what its LDS lets share a CU (four
// float32 groups; six bfloat16 groups, or one block of four). At five the
// bfloat16 kernels spill five to seven registers, outside the steps.
template <typename S, int GPB>
constexpr int relay_waves_per_eu() {
  return sizeof(S) == 4 || GPB == 4 ? 3 : 5;
}

template <typename S, int DP, int GPB, bool NTS>
__global__ __launch_bounds__(GPB * kRelayWaves * 64) __attribute__((amdgpu_waves_per_eu(relay_waves_per_eu<S, GPB>())))
void k_blur_relay(const S* __restrict__ in, S* __restrict__ out, int w, const DevState* __restrict__ st, int radius,
                  int vertical, int stream, int32_t* __restrict__ table) {
  __shared__ RelayLds<S> s_lds[GPB];
  int r;
  if (!pass_radius(st, radius, w, r)) return;
  blur_relay_lines<S, DP, GPB, NTS>(in, out, w, r, vertical, stream != 0, blockIdx.x, gridDim.x, s_lds);
  if (table != nullptr) fill_group_table<GPB * kRelayWaves * 64>(table, st->beta, st->keys, blockIdx.x, gridDim.x);
}

// Blur pass of large float32 grids (see ring_rows and batch_ring): one wave
// per group of 64 / DP lines loads, sums and stores, and keeps leaving values
// in registers. Same arithmetic, LDS rows and direct loads as the relay pass.
//
// The line is loaded chunk by chunk (16 positions aligned to multiples of 16)
// into a ring of rows (row = position modulo the ring). Step e takes chunk e:
// first its positions up to r go into the starting sum, then, from
// step A = ceil(r / kChunk) on, the outputs x of chunk e - A (x + r lies in
// chunk e or e - 1). While the ring also holds every leaving position
// x - r - 1 still to come beside the chunks in flight, leaving values are read
// back from it; otherwise the ring is split in two halves and the leaving
// chunks reach the upper half from register slots, where each chunk was kept
// since it entered (ring of 128 rows, one wave per SIMD: 24 slots, 48 <= r <=
// 192; ring of 64 rows, two waves per SIMD: 8 slots, 16 <= r <= 64), or from a
// second load stream (the same positions again). Loads are issued at positions
// clamped into the line, so every chunk is exactly kVec load instructions.
//
// Waits. Every step issues, in this order, the stores of the chunk it summed
// and then the loads of issue slot e + kDepth - 1 (entering chunk, then leaving
// chunk); the number of operations issued after a chunk's last load follows
// from that schedule (ops_after).
template <int RR>
struct RingShape {
  static constexpr int kRowBytes = 256;  // one position of the wave's lines
  static constexpr int kLanesPerRow = kRowBytes / 16;
  static constexpr int kPos = 64 / kLanesPerRow;  // positions per load instruction
  static constexpr int kChunk = 16;               // positions per chunk
  static constexpr int kVec = kChunk / kPos;      // load instructions per chunk
  static constexpr int kDepth = RR >= 128 ? 3 : 2;  // issue slots in flight, the one being summed included
  static constexpr int kRingRows = RR;
  static constexpr int kSlots = kRingRows / kChunk;
  static constexpr int kRegChunks = RR >= 128 ? 24 : 8;  // register slots of leaving chunks
  static constexpr int kRegWords = kChunk;   // registers per chunk
  static constexpr int kHalfRows = kRingRows / 2;  // rows of each stream when the ring is split
  static_assert((kRingRows & (kRingRows - 1)) == 0, "ring shape");
  static_assert(kHalfRows / kChunk >= kDepth, "a split half holds the chunks in use and in flight");
};

// LDS of one wave: 36 KB with 128 rows, 20 KB with 64.
template <int RR>
struct alignas(16) RingLds {
  float ring[RingShape<RR>::kRingRows][64];
  float out[RingShape<RR>::kChunk][64];
};

// Leaving values come from the entering ring when, at every step, the chunk
// issued then does not overwrite a leaving position still to come: with A =
// ceil(r / kChunk) chunks between a step's chunk and its outputs and
// ceil((r + 1) / kChunk) between an output chunk and its leaving positions,
// A + ceil((r + 1) / kChunk) <= kSlots + 1 - kDepth.
template <int RR>
__device__ __forceinline__ bool ring_leave(int r) {
  using Sh = RingShape<RR>;
  const int a = (r + Sh::kChunk - 1) / Sh::kChunk;
  const int b = (r + Sh::kChunk) / Sh::kChunk;
  return a + b <= Sh::kSlots + 1 - Sh::kDepth;
}

// One direct load whose LDS rows this wave may still be reading: those reads
// must have completed first.
template <bool nt>
__device__ __forceinline__ void dma16(const void* src, uint32_t m0) {
  asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
  dma16_load<nt>(src, m0);
}

// s_waitcnt vmcnt(n) for a run-time n (rounded down, which only waits
// longer).
__device__ __forceinline__ void wait_vm_dyn(int n) {
  switch (n < 0 ? 0 : n) {
    case 0: wait_vm<0>(); break;
    case 1: wait_vm<1>(); break;
    case 2: wait_vm<2>(); break;
    case 3: wait_vm<3>(); break;
    case 4: wait_vm<4>(); break;
    case 5: wait_vm<5>(); break;
    case 6: wait_vm<6>(); break;
    case 7: wait_vm<7>(); break;
    case 8: wait_vm<8>(); break;
    case 9: wait_vm<9>(); break;
    case 10: wait_vm<10>(); break;
    case 11: wait_vm<11>(); break;
    case 12: wait_vm<12>(); break;
    case 13: wait_vm<13>(); break;
    case 14: wait_vm<14>(); break;
    case 15: wait_vm<15>(); break;
    default: wait_vm<16>(); break;
  }
}

template <int DP, int RR, bool NT>
struct RingLine {
  using Sh = RingShape<RR>;
  static constexpr int kChunk = Sh::kChunk;
  static constexpr int kPiecesPerCell = DP / 4;
  const float* __restrict__ src;  // the pass's input grid
  float* __restrict__ dst;        // and output grid
  int64_t step;     // elements between consecutive positions of a line
  int64_t ld_off;   // element offset of this lane's load piece at position 0
  bool ld_ok;       // the load piece's line exists (else its loads are clamped and its stores skipped)
  int w, r;
  int n_chunks;  // M: chunks of the line
  int ahead;     // A = ceil(r / kChunk): step e sums the outputs of chunk e - A
  int lag;       // the leaving chunk needed at step e is e - lag (split ring)
  int n_steps;   // A + M
  int q, j, lane;
  bool split;        // the leaving values have their own region (the ring's upper half)
  bool regs;         // split, and the leaving chunks come from registers instead of a second load stream
  int enter_mask;    // ring rows of the entering stream - 1
  uint32_t ring_m0;  // LDS byte address of ring row 0 (the same for all lanes)
  RingLds<RR>* lds;

  __device__ __forceinline__ int clamp_pos(int t) const { return t < 0 ? 0 : (t > w - 1 ? w - 1 : t); }

  // kVec loads of chunk m (positions kChunk m ..) into rows row0 ..
  template <bool nt>
  __device__ __forceinline__ void load_chunk(int m, int row0) const {
    const int pos0 = m * kChunk;
    const uint32_t m0 = ring_m0 + static_cast<uint32_t>(row0 * Sh::kRowBytes);
    if (pos0 + kChunk - 1 <= w - 1) {
      const float* p = src + ld_off + static_cast<int64_t>(pos0 + q) * step;
      const int64_t inc = static_cast<int64_t>(Sh::kPos) * step;
#pragma unroll
      for (int i = 0; i < Sh::kVec; ++i) dma16<nt>(p + i * inc, m0 + i * 1024u);
    } else {
#pragma unroll
      for (int i = 0; i < Sh::kVec; ++i)
        dma16<nt>(src + ld_off + static_cast<int64_t>(clamp_pos(pos0 + Sh::kPos * i + q)) * step, m0 + i * 1024u);
    }
  }

  // Issue slot u: entering chunk u and, when split, leaving chunk u - lag.
  __device__ __forceinline__ bool slot_enter(int u) const { return u < n_chunks; }
  __device__ __forceinline__ bool slot_leave(int u) const {
    return split && !regs && u - lag >= 0 && u - lag < n_chunks;
  }
  __device__ __forceinline__ void issue(int u) const {
    if (slot_enter(u)) load_chunk<NT>(u, (u * kChunk) & enter_mask);
    if (slot_leave(u))
      load_chunk<kBlurLeaveStream>(u - lag, Sh::kHalfRows + (((u - lag) * kChunk) & (Sh::kHalfRows - 1)));
  }
  __device__ __forceinline__ int slot_loads(int u) const {
    return Sh::kVec * ((slot_enter(u) ? 1 : 0) + (slot_leave(u) ? 1 : 0));
  }
  // Stores of step s: a whole output chunk (every output chunk but the last
  // lies inside the line, and only the last step stores the last one).
  __device__ __forceinline__ int step_stores(int s) const { return s >= ahead ? Sh::kVec : 0; }
  // Operations issued after slot e's loads, as of the start of step e: the
  // loads of slots e + 1 .. e + kDepth - 2 and the stores of the steps that
  // came after slot e was issued.
  __device__ __forceinline__ int ops_after(int e) const {
    int n = 0;
#pragma unroll
    for (int u = 1; u <= Sh::kDepth - 2; ++u) n += slot_loads(e + u);
    const int first = e - Sh::kDepth + 2;
    const int s0 = first > 0 ? first : 0;
    for (int s = s0; s < e; ++s) n += step_stores(s);
    return n;
  }

  __device__ __forceinline__ int enter_row(int x) const { return (x + r) & enter_mask; }
  __device__ __forceinline__ int leave_row(int x) const {
    const int t = x - r - 1;
    return split ? Sh::kHalfRows + (t & (Sh::kHalfRows - 1)) : (t & (Sh::kRingRows - 1));
  }
  __device__ __forceinline__ float enter_val(int x) const {
    return lds->ring[enter_row(x)][lane];
  }
  __device__ __forceinline__ float leave_val(int x) const {
    return lds->ring[leave_row(x)][lane];
  }

  // Outputs x0 .. x0 + kChunk - 1, all inside the grid, all with (ENTER) or
  // without an entering value and all with (LEAVE) or without a leaving one:
  // no per-position tests. With both at every position the window holds
  // 2r + 1 cells, and with neither it is the whole line: one multiplier
  // serves all positions. Otherwise each position takes its own from lane p.
  template <bool ENTER, bool LEAVE>
  __device__ __forceinline__ void run_uniform(int x0, float mult, float& s) const {
    constexpr bool kConstMult = ENTER == LEAVE;
    const int mult_bits = __float_as_int(mult);
    float e[kChunk], l[kChunk];
    // The chunk's entering rows and its leaving rows are each kChunk
    // consecutive ring rows unless they wrap around the end of their region:
    // then one base address with constant offsets reads them.
    const int eb = enter_row(x0), lb = leave_row(x0);
    const bool e_flat = !ENTER || eb + kChunk <= enter_mask + 1;
    const bool l_flat = !LEAVE || (lb & (split ? Sh::kHalfRows - 1 : Sh::kRingRows - 1)) + kChunk <=
                                      (split ? Sh::kHalfRows : Sh::kRingRows);
    if (e_flat && l_flat) {
      const float* ep = &lds->ring[ENTER ? eb : 0][lane];
      const float* lp = &lds->ring[LEAVE ? lb : 0][lane];
#pragma unroll
      for (int p = 0; p < kChunk; ++p) {
        if (ENTER) e[p] = ep[p * 64];
        if (LEAVE) l[p] = lp[p * 64];
      }
    } else {
#pragma unroll
      for (int p = 0; p < kChunk; ++p) {
        if (ENTER) e[p] = enter_val(x0 + p);
        if (LEAVE) l[p] = leave_val(x0 + p);
      }
    }
    const float m_const = kConstMult ? __int_as_float(__builtin_amdgcn_readfirstlane(mult_bits)) : 0.0f;
#pragma unroll
    for (int p = 0; p < kChunk; ++p) {
      if (ENTER) s = s + e[p];
      if (LEAVE) s = s - l[p];
      const float m = kConstMult ? m_const : __int_as_float(__builtin_amdgcn_readlane(mult_bits, p));
      lds->out[p][lane] = s * m;
    }
  }

  // Any outputs (x = 0 included: the starting sum as it is): the tests of
  // each position select the update.
  __device__ __forceinline__ void run_mixed(int x0, float mult, float& s) const {
    const int mult_bits = __float_as_int(mult);
    float e[kChunk], l[kChunk];
#pragma unroll
    for (int p = 0; p < kChunk; ++p) {
      e[p] = enter_val(x0 + p);
      l[p] = leave_val(x0 + p);
    }
#pragma unroll
    for (int p = 0; p < kChunk; ++p) {
      const int x = x0 + p;
      const bool inside = x >= 1 && x < w;
      const float with_enter = s + e[p];
      s = (inside && x + r <= w - 1) ? with_enter : s;
      const float with_leave = s - l[p];
      s = (inside && x - r - 1 >= 0) ? with_leave : s;
      lds->out[p][lane] = s * __int_as_float(__builtin_amdgcn_readlane(mult_bits, p));
    }
  }

  // The positions of chunk e up to r, in ascending order, into the
  // starting sum (position 0 starts it).
  __device__ __forceinline__ void start_sum(int e, float& s) const {
    const int t0 = e * kChunk;
    float v[kChunk];
#pragma unroll
    for (int p = 0; p < kChunk; ++p) v[p] = lds->ring[(t0 + p) & enter_mask][lane];
    if (t0 > 0 && t0 + kChunk - 1 <= r) {
#pragma unroll
      for (int p = 0; p < kChunk; ++p) s = s + v[p];
    } else {
#pragma unroll
      for (int p = 0; p < kChunk; ++p) {
        const int t = t0 + p;
        const float added = t == 0 ? v[p] : s + v[p];
        s = t <= r ? added : s;
      }
    }
  }

  // Output chunk k (positions x0 = k kChunk ..): sum, then store the chunk's
  // rows as 16-byte pieces, with a streaming hint where the grids are beyond
  // the Infinity Cache (the 64-row ring; 1448^2 x 64: whole sort 5568 against
  // 5668 ms).
  __device__ __forceinline__ void outputs(int k, float& s) const {
    const int x0 = k * kChunk;
    const int x1 = x0 + kChunk - 1;
    // Lane p < kChunk: float32(1 / count) of position x0 + p (correctly
    // rounded, as the host table 1.0f / c).
    float mult;
    {
      const int x = clamp_pos(x0 + (lane & (kChunk - 1)));
      const int hi = x + r < w - 1 ? x + r : w - 1;
      const int lo = x - r > 0 ? x - r : 0;
      mult = 1.0f / static_cast<float>(hi - lo + 1);
    }
    const bool all_in = x0 >= 1 && x1 < w;
    const bool enter_all = x1 + r <= w - 1, enter_none = x0 + r > w - 1;
    const bool leave_all = x0 - r - 1 >= 0, leave_none = x1 - r - 1 < 0;
    if (all_in && enter_all && leave_all)
      run_uniform<true, true>(x0, mult, s);
    else if (all_in && enter_all && leave_none)
      run_uniform<true, false>(x0, mult, s);
    else if (all_in && enter_none && leave_all)
      run_uniform<false, true>(x0, mult, s);
    else if (all_in && enter_none && leave_none)
      run_uniform<false, false>(x0, mult, s);
    else
      run_mixed(x0, mult, s);
#pragma unroll
    for (int i = 0; i < Sh::kVec; ++i) {
      const int x = x0 + Sh::kPos * i + q;
      if (x < w && ld_ok)
        store_quad<(RR < 128)>(dst + ld_off + static_cast<int64_t>(x) * step,
                               *reinterpret_cast<const float4*>(&lds->out[Sh::kPos * i + q][4 * j]));
    }
  }

  // Register ring of the leaving values: step e reads chunk e back from the
  // entering half and swaps it with register slot e mod lag, which holds
  // chunk e - lag, the newest leaving chunk of the step; that chunk goes to
  // its rows of the leaving half. A chunk is used as leaving values at steps
  // e and e + 1 only, and the leaving half holds at least two. A chunk's rows
  // are contiguous in both halves, so it moves as 16-byte pieces (lane l
  // holds bytes 16 l .. of each KB) in whatever order: only its place in the
  // leaving half matters. Past the last chunk the rows read are stale; what
  // they push is never popped (a chunk pushed at step e >= M would pop at
  // e + lag >= M + A, after the last step).
  using Word = uint32_t;
  static constexpr int kWords = Sh::kRegWords;  // per lane and chunk
  static constexpr int kPieces = kWords / 4;    // 16-byte pieces per lane and chunk
  template <int K>
  __device__ __forceinline__ void exchange(Word (&keep)[K][kWords], int slot, int e) const {
    Word in[kWords], out[kWords];
    const char* ep = reinterpret_cast<const char*>(&lds->ring[(e * kChunk) & enter_mask][0]) + 16 * lane;
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const uint4 v = *reinterpret_cast<const uint4*>(ep + 1024 * i);
      in[4 * i] = v.x;
      in[4 * i + 1] = v.y;
      in[4 * i + 2] = v.z;
      in[4 * i + 3] = v.w;
    }
    // The uniform slot is found in two levels of scalar branches: its group
    // of kGroup slots, then the slot.
    constexpr int kGroup = 6;
#pragma unroll
    for (int g = 0; g < K; g += kGroup) {
      if (slot >= g && slot < g + kGroup) {
#pragma unroll
        for (int k = g; k < g + kGroup && k < K; ++k) {
          if (k == slot) {
#pragma unroll
            for (int p = 0; p < kWords; ++p) {
              out[p] = keep[k][p];
              keep[k][p] = in[p];
            }
          }
        }
      }
    }
    if (e >= lag) {
      char* lp = reinterpret_cast<char*>(&lds->ring[Sh::kHalfRows + (((e - lag) * kChunk) & (Sh::kHalfRows - 1))][0]) +
                 16 * lane;
#pragma unroll
      for (int i = 0; i < kPieces; ++i)
        *reinterpret_cast<uint4*>(lp + 1024 * i) = make_uint4(out[4 * i], out[4 * i + 1], out[4 * i + 2], out[4 * i + 3]);
    }
  }

  __device__ __forceinline__ void run_regs() const {
    // Zeroed: the first lag steps read a slot (and drop the value) before
    // its first chunk arrives.
    Word keep[Sh::kRegChunks][kWords] = {};
    for (int u = 0; u <= Sh::kDepth - 2; ++u) issue(u);
    float s = 0.0f;
    int slot = 0;
    for (int e = 0; e < n_steps; ++e) {
      if (slot_loads(e) > 0) wait_vm_dyn(ops_after(e));
      exchange<Sh::kRegChunks>(keep, slot, e);
      if (e * kChunk <= r) start_sum(e, s);
      if (e >= ahead) outputs(e - ahead, s);
      issue(e + Sh::kDepth - 1);
      slot = slot + 1 == lag ? 0 : slot + 1;
    }
  }

  __device__ __forceinline__ void run() const {
    if (regs) {
      run_regs();
      return;
    }
    for (int u = 0; u <= Sh::kDepth - 2; ++u) issue(u);
    float s = 0.0f;
    for (int e = 0; e < n_steps; ++e) {
      if (slot_loads(e) > 0) wait_vm_dyn(ops_after(e));
      if (e * kChunk <= r) start_sum(e, s);
      if (e >= ahead) outputs(e - ahead, s);
      issue(e + Sh::kDepth - 1);
    }
  }
};

// Lines line0 .. line0 + 64/DP - 1 of a ring pass (those below w), by one wave.
template <int DP, int RR, bool NT>
__device__ __forceinline__ void blur_ring_line(const float* __restrict__ in, float* __restrict__ out, int w, int r,
                                               int vertical, int64_t line0, int lane, RingLds<RR>* lds) {
  using Sh = RingShape<RR>;
  using L_t = RingLine<DP, RR, NT>;
  L_t L;
  // Element offset of line l at position 0, and between positions.
  auto line_off = [&](int64_t l) { return vertical ? l * DP : l * w * DP; };
  L.src = in;
  L.dst = out;
  L.step = vertical ? static_cast<int64_t>(w) * DP : DP;
  L.w = w;
  L.r = r;
  L.q = lane / Sh::kLanesPerRow;
  L.j = lane % Sh::kLanesPerRow;
  const int64_t ld_line = line0 + L.j / L_t::kPiecesPerCell;
  L.ld_ok = ld_line < w;
  L.ld_off = line_off(L.ld_ok ? ld_line : w - 1) + (L.j % L_t::kPiecesPerCell) * 4;
  L.lane = lane;
  L.lds = lds;
  if (r == 0) {
    const int64_t own_line = line0 + lane / DP;
    const int64_t own_off = line_off(own_line < w ? own_line : w - 1) + lane % DP;
    if (own_line < w)
      for (int x = 0; x < w; ++x) L.dst[own_off + x * L.step] = L.src[own_off + x * L.step];
    return;
  }
  L.n_chunks = (w + Sh::kChunk - 1) / Sh::kChunk;
  L.ahead = (r + Sh::kChunk - 1) / Sh::kChunk;
  L.n_steps = L.ahead + L.n_chunks;
  L.split = !ring_leave<RR>(r);
  // Step e sums outputs of chunk k = e - A, whose leaving positions reach
  // up to k kChunk + kChunk - 2 - r: chunk e - lag.
  L.lag = L.ahead - ((Sh::kChunk - 2 - r) >= 0 ? (Sh::kChunk - 2 - r) / Sh::kChunk
                                               : -((r - Sh::kChunk + 2 + Sh::kChunk - 1) / Sh::kChunk));
  L.regs = L.split && L.lag <= Sh::kRegChunks;
  L.enter_mask = (L.split ? Sh::kHalfRows : Sh::kRingRows) - 1;
  L.ring_m0 = __builtin_amdgcn_readfirstlane(
      static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) float*)(&lds->ring[0][0]))));
  L.run();
}

// One group of 64/DP lines per wave, in two-wave blocks; block `bid` of
// `nblocks` takes groups 2 bid and 2 bid + 1 and walks on with a stride. With
// 128 rows (72 KB LDS) four waves share a CU, one per SIMD with all its
// registers; with 64 rows (40 KB) eight do.
constexpr int kRingWavesPerBlock = 2;
template <int DP, int RR, bool NT>
__device__ __forceinline__ void blur_ring_lines(const float* __restrict__ in, float* __restrict__ out, int w, int r,
                                                int vertical, int64_t bid, int64_t nblocks, RingLds<RR>* lds) {
  const int wib = threadIdx.x >> 6;
  for (int64_t g = bid * kRingWavesPerBlock + wib; g * (64 / DP) < w; g += nblocks * kRingWavesPerBlock)
    blur_ring_line<DP, RR, NT>(in, out, w, r, vertical, g * (64 / DP), threadIdx.x & 63, lds + wib);
}

template <int DP, int RR, bool NT>
__global__ __launch_bounds__(kRingWavesPerBlock * 64) __attribute__((amdgpu_waves_per_eu(RR >= 128 ? 1 : 2)))
void k_blur_ring(const float* __restrict__ in, float* __restrict__ out, int w, const DevState* __restrict__ st,
                 int radius, int vertical, int32_t* __restrict__ table) {
  __shared__ RingLds<RR> s_ring[kRingWavesPerBlock];
  int r;
  if (!pass_radius(st, radius, w, r)) return;
  blur_ring_lines<DP, RR, NT>(in, out, w, r, vertical, blockIdx.x, gridDim.x, s_ring);
  if (table != nullptr)
    fill_group_table<kRingWavesPerBlock * 64>(table, st->beta, st->keys, blockIdx.x, gridDim.x);
}

// Cells of DP * sizeof(S) bytes are moved in 16-byte pieces when they hold
// at least one (every float32 width, bfloat16 from 8 channels up).
template <typename S, int DP>
constexpr bool staged_cells() {
  return DP * static_cast<int>(sizeof(S)) >= 16;
}

// Groups of 64/DP lines of a pass over w lines.
template <int DP>
inline int64_t staged_groups(int w) {
  return (w + 64 / DP - 1) / (64 / DP);
}

// ---------------------------------------------------------- group table

__global__ __launch_bounds__(kBlock) void k_group_table(int32_t* __restrict__ table,
                                                        const DevState* __restrict__ st) {
  if (st->done) return;
  fill_group_table<kBlock>(table, st->beta, st->keys, blockIdx.x, gridDim.x);
}

// Squared distance partial over one lane's 4 channels, as the two lowest
// levels of the pairwise tree: (c0^2 + c1^2) + (c2^2 + c3^2).
__device__ inline float chunk_sq(const float4 a, const float4 b) {
  const float e0 = a.x - b.x, e1 = a.y - b.y, e2 = a.z - b.z, e3 = a.w - b.w;
  return (e0 * e0 + e1 * e1) + (e2 * e2 + e3 * e3);
}

// Channels per lane in the assignment: 8 bfloat16 channels (one 16-byte
// load) when a cell holds at least 8, else 4 (a float4, or 8 bytes of
// bfloat16). Eight channels per lane add the tree's third level, (first
// four) + (last four), inside the lane; the lanes then reduce the rest.
template <typename S, int DP>
constexpr int assign_channels() {
  return (sizeof(S) == 2 && DP >= 8) ? 8 : 4;
}

template <typename S, int DP>
struct AssignVec {
  using Quad = typename Storage<S>::Quad;
  using T = Quad;
  __device__ static __forceinline__ float sq(const T& a, const T& b) {
    return chunk_sq(Storage<S>::widen4(a), Storage<S>::widen4(b));
  }
};

template <>
struct AssignVec<uint16_t, 64> {
  using T = uint4;
  __device__ static __forceinline__ float sq(const T& a, const T& b) {
    const float lo = chunk_sq(Storage<uint16_t>::widen4(make_uint2(a.x, a.y)),
                              Storage<uint16_t>::widen4(make_uint2(b.x, b.y)));
    const float hi = chunk_sq(Storage<uint16_t>::widen4(make_uint2(a.z, a.w)),
                              Storage<uint16_t>::widen4(make_uint2(b.z, b.w)));
    return lo + hi;
  }
};
template <>
struct AssignVec<uint16_t, 32> : AssignVec<uint16_t, 64> {};
template <>
struct AssignVec<uint16_t, 16> : AssignVec<uint16_t, 64> {};
template <>
struct AssignVec<uint16_t, 8> : AssignVec<uint16_t, 64> {};

__device__ inline unsigned long long wave_sum_u64(unsigned long long v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
  return v;
}

// The 24 orderings of (0,1,2,3) in lexicographic order as position codes
// (sigma(i) in bits 2i..2i+1), eight codes per 64-bit word, ordering m in
// byte m mod 8 of word m / 8:
//   0123 0132 0213 0231 0312 0321 1023 1032 | 1203 1230 1302 1320 2013 2031
//   2103 2130 | 2301 2310 3012 3021 3102 3120 3201 3210
// Ordering 2p + 1 is ordering 2p with its last two places swapped.
__device__ __forceinline__ uint32_t order_code(int m) {
  constexpr uint64_t kOrders0 = 0xB1E16C9C78D8B4E4ull;
  constexpr uint64_t kOrders1 = 0x36C672D22D8D39C9ull;
  constexpr uint64_t kOrders2 = 0x1B4B278763931E4Eull;
  const uint64_t word = m < 8 ? kOrders0 : (m < 16 ? kOrders1 : kOrders2);
  return static_cast<uint32_t>((word >> (8 * (m & 7))) & 0xff);
}

// a / d for 0 <= a < 2^31 (Divisor: made by the host).
__device__ __forceinline__ uint32_t quotient(uint32_t a, Divisor d) { return __umulhi(a << 1, d.mul) >> d.shift; }

// A value all lanes hold, in a scalar register (the compiler cannot know that
// of what it loads from the state).
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint32_t uniform(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int32_t>(v)));
}
__device__ __forceinline__ Divisor uniform(Divisor d) { return Divisor{uniform(d.mul), uniform(d.shift)}; }

// Geometry of one reorder's items, read once per thread. Items are the
// groups of every block (item < groups), then packs of four cells in no group
// (singles), whose distance still counts towards the energy. Item indices,
// cell indices and counts stay below 2^31 (side <= 46340).
struct ItemGeometry {
  const int32_t* __restrict__ table;
  int w, beta, nb, dy, dx, s;
  uint32_t gpb, groups, singles, total;
  Divisor by_gpb, by_nb, by_rest, by_w;

  __device__ __forceinline__ void init(const DevState* __restrict__ st, const int32_t* __restrict__ tbl) {
    table = tbl;
    w = uniform(st->w);
    beta = uniform(st->beta);
    nb = uniform(st->nb);
    dy = uniform(st->dy);
    dx = uniform(st->dx);
    s = uniform(st->s);
    gpb = uniform(static_cast<uint32_t>(st->groups_per_block));
    groups = uniform(static_cast<uint32_t>(st->groups));
    singles = uniform(static_cast<uint32_t>(st->singles));
    total = groups + (singles + 3) / 4;
    by_gpb = uniform(st->by_gpb);
    by_nb = uniform(st->by_nb);
    by_rest = uniform(st->by_rest);
    by_w = uniform(st->by_w);
  }

  __device__ __forceinline__ int32_t wrapped(int y, int x) const {
    if (y >= w) y -= w;
    if (x >= w) x -= w;
    return y * w + x;
  }
  // Where the grid block of group `item` starts (rolled grid), and the
  // group's first table entry.
  __device__ __forceinline__ void group_origin(uint32_t item, int& y0, int& x0, uint32_t& entry) const {
    const uint32_t b = quotient(item, by_gpb);
    const uint32_t by = quotient(b, by_nb);
    y0 = dy + static_cast<int>(by) * beta;
    x0 = dx + static_cast<int>(b - by * static_cast<uint32_t>(nb)) * beta;
    entry = 4 * (item - b * gpb);
  }
  __device__ __forceinline__ int32_t group_cell(int y0, int x0, int32_t t) const {
    return wrapped(y0 + (t >> 16), x0 + (t & 0xffff));
  }
  // Single t: first the rolled-grid rows below the nb*beta square, then the
  // columns right of it, then the left-over cell pi(beta^2 - 1) of each block
  // when beta is odd. 0 past the last single.
  __device__ __forceinline__ int32_t single_cell(uint32_t t) const {
    if (t >= singles) return 0;
    const uint32_t R = static_cast<uint32_t>(nb) * beta, W = static_cast<uint32_t>(w);
    const uint32_t strip_rows = (W - R) * W, strip = W * W - R * R;
    uint32_t u, v;
    if (t < strip_rows) {
      const uint32_t qy = quotient(t, by_w);
      u = R + qy;
      v = t - qy * W;
    } else if (t < strip) {
      const uint32_t t2 = t - strip_rows;
      u = quotient(t2, by_rest);
      v = R + t2 - u * (W - R);
    } else {
      const uint32_t b = t - strip;
      const uint32_t by = quotient(b, by_nb);
      const int32_t tt = table[static_cast<int64_t>(beta) * beta - 1];
      u = by * beta + static_cast<uint32_t>(tt >> 16);
      v = (b - by * static_cast<uint32_t>(nb)) * beta + static_cast<uint32_t>(tt & 0xffff);
    }
    return wrapped(static_cast<int>(u) + dy, static_cast<int>(v) + dx);
  }
};

// Cross-lane moves within quads (DPP): the value of lane i ^ (1 << B).
template <int B>
__device__ __forceinline__ int quad_xor(int v) {
  static_assert(B == 0 || B == 1, "within a quad");
  return __builtin_amdgcn_mov_dpp(v, B == 0 ? 0xB1 : 0x4E, 0xF, 0xF, true);  // quad_perm [1,0,3,2], [2,3,0,1]
}
template <int I>
__device__ __forceinline__ int quad_lane(int v) {  // the value of lane I of the quad
  return __builtin_amdgcn_mov_dpp(v, I * 0x55, 0xF, 0xF, true);
}
// The same for the lane 16 (ROW = 16) or 32 lanes away, as an exchange of
// whole rows: row halves of a and b meet, so that afterwards a holds, for the
// lanes with the ROW bit clear, a of both lanes of each pair in a and b.
template <int ROW>
__device__ __forceinline__ void row_swap(uint32_t& a, uint32_t& b) {
  if constexpr (ROW == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  }
}

// How the lanes of a wave serve items: LG lanes per item, IPW items per wave.
// Lane bits 0 and 1 are the two lowest bits of the lane's chunk of the cell
// (so that a quad reads 64 consecutive bytes); the next one or two bits of
// the chunk are whole rows of lanes (bit 4 and 5), which exchange data with
// one instruction for two values. The item slot takes the bits between.
template <int LG>
struct ItemLanes {
  static constexpr int kQuad = LG < 4 ? LG : 4;
  static constexpr int IPW = 64 / LG;
  static constexpr int kRowA = LG == 16 ? 16 : 32;  // lanes between the halves of chunk bit 2
  __device__ static __forceinline__ int chunk(int lane) {
    if constexpr (LG <= 4) return lane % LG;
    else if constexpr (LG == 8) return (lane & 3) | ((lane >> 3) & 4);
    else return (lane & 3) | ((lane >> 2) & 12);
  }
  __device__ static __forceinline__ int slot(int lane) {
    if constexpr (LG <= 4) return lane / LG;
    else if constexpr (LG == 8) return (lane >> 2) & 7;
    else return (lane >> 2) & 3;
  }
};

// One level of the transposed butterfly over the item's pair partials, chunk
// bit B: lanes with the bit clear keep the even pairs, the others the odd
// ones, each adding its partner's partial of the kept pair.
template <int LG, int B, int N>
__device__ __forceinline__ void transpose_level(float* part, int lane) {
#pragma unroll
  for (int t = 0; t < N; ++t) {
    if constexpr (B < 2) {
      const float lo = part[2 * t], hi = part[2 * t + 1];
      const float sum_lo = lo + __int_as_float(quad_xor<B>(__float_as_int(lo)));
      const float sum_hi = hi + __int_as_float(quad_xor<B>(__float_as_int(hi)));
      part[t] = (lane & (1 << B)) ? sum_hi : sum_lo;
    } else {
      uint32_t a = __float_as_uint(part[2 * t]), b = __float_as_uint(part[2 * t + 1]);
      row_swap<B == 2 ? ItemLanes<LG>::kRowA : 32>(a, b);
      part[t] = __uint_as_float(a) + __uint_as_float(b);
    }
  }
}

// The smaller of the two keys of each pair of lanes that differ in chunk bit B.
template <int LG, int B>
__device__ __forceinline__ unsigned long long min_level(unsigned long long key) {
  uint32_t lo = static_cast<uint32_t>(key), hi = static_cast<uint32_t>(key >> 32);
  uint32_t lo2, hi2;
  if constexpr (B < 2) {
    lo2 = static_cast<uint32_t>(quad_xor<B>(static_cast<int>(lo)));
    hi2 = static_cast<uint32_t>(quad_xor<B>(static_cast<int>(hi)));
  } else {
    lo2 = lo;
    hi2 = hi;
    row_swap<B == 2 ? ItemLanes<LG>::kRowA : 32>(lo, lo2);
    row_swap<B == 2 ? ItemLanes<LG>::kRowA : 32>(hi, hi2);
  }
  const unsigned long long a = (static_cast<unsigned long long>(hi) << 32) | lo;
  const unsigned long long b = (static_cast<unsigned long long>(hi2) << 32) | lo2;
  return b < a ? b : a;
}
template <int LG>
__device__ __forceinline__ unsigned long long item_min(unsigned long long key) {
  if constexpr (LG > 1) key = min_level<LG, 0>(key);
  if constexpr (LG > 2) key = min_level<LG, 1>(key);
  if constexpr (LG > 4) key = min_level<LG, 2>(key);
  if constexpr (LG > 8) key = min_level<LG, 3>(key);
  return key;
}

// floor(v 2^s) for 0 <= v with v 2^s < 2^57: v = f 2^e, f in [1/2, 1), f a
// 24-bit fraction.
__device__ __forceinline__ unsigned long long quantise(float v, int s) {
  const uint32_t f = static_cast<uint32_t>(__builtin_amdgcn_frexp_mantf(v) * 4294967296.0f);
  const int k = 64 - s - __builtin_amdgcn_frexp_expf(v);  // v 2^s = f 2^32 / 2^k (f as 32 bits), k >= 7
  const unsigned long long q = (static_cast<unsigned long long>(f) << 32) >> (k & 63);
  return k < 64 ? q : 0ull;
}

// Blocks are handed to the eight chiplets (each with its own L2) in turn:
// the place of block `bid` when every chiplet takes a contiguous eighth.
// Neighbouring groups share the 128-byte lines of their cells' permutation
// entries and, below 32 channels, of the cells themselves (assignment inside
// sorts, in turn / contiguous: 512^2 x 4 14.5 / 13.6 us, 723^2 x 64 52.5 /
// 50.8, 1024^2 x 64 98.6 / 95.7, 2091^2 x 16 187 / 182; 1448^2 x 64 bfloat16
// 110.5 / 111.8).
__device__ __forceinline__ int64_t chiplet_order(int64_t bid, int64_t nblocks) {
  const int64_t each = nblocks >> 3, more = nblocks & 7, chiplet = bid & 7;
  return chiplet * each + (chiplet < more ? chiplet : more) + (bid >> 3);
}

// One reorder's blockwise assignment, block `bid` of `nblocks` blocks that
// share its items. LG = DP / C lanes serve one item, C = assign_channels<S,
// DP>() (4, or 8 for bfloat16 cells of 8 or more channels): each lane holds C
// channels of the item's four grid cells and four target cells and forms all
// 16 pair partials as the lowest levels of the channel tree. The rest of the
// work is split across the LG lanes:
//  - a transposed butterfly finishes the tree level by level (each still left
//    half + right half): after log2(LG) levels the lane with chunk L holds the
//    exact distances of pairs q = t*LG + L;
//  - the quantised pair costs go to LDS; chunk L takes the ordered pairs p =
//    L, L + LG, .. of places for the first two cells, each of which leaves two
//    orderings (2p, 2p + 1) of the last two, and the lanes pick the first
//    minimum as the smallest key (cost, ordering).
// Keys are cost * 32 + ordering. Costs that this would not hold (tiny grids,
// or distances that are no finite numbers) take a slower way, chosen for a
// whole wave.
//
// What bounds it: on grids beyond the Infinity Cache the grid's and target's
// cells, read and written at random 4 DP-byte places (1024^2 x 64: 0.75 GB in
// 95.7 us); below, a wave's chain of dependent loads (table, permutation,
// cells) and its VALU work per item, which three waves per SIMD and a few
// long-lived blocks per CU hide best: a block of a single item costs several
// microseconds of launch and tear-down. Pairs of places instead of all 24
// orderings, quantising in integers instead of float64, one packed key per
// ordering and lane swaps in registers instead of LDS shuffles took the VALU
// work per item to under half (inside sorts, before and after: 64^2 x 64 9.5
// -> 8.5 us, 512^2 x 4 18.5 -> 13.6, 723^2 x 64 77.6 -> 50.8, 1024^2 x 64
// 109.7 -> 95.7, 2091^2 x 16 207 -> 182, 1448^2 x 64 bfloat16 129 -> 111).
template <int DP, typename S>
__device__ __forceinline__ void assign_items(S* __restrict__ G, const S* __restrict__ T, int32_t* __restrict__ P,
                                             const ItemGeometry& geo, DevState* __restrict__ st, int64_t bid,
                                             int64_t nblocks) {
  using V = AssignVec<S, DP>;
  using Vec = typename V::T;
  constexpr int LG = DP / assign_channels<S, DP>();
  static_assert(sizeof(Vec) * LG == DP * sizeof(S), "lane vectors must tile a cell");
  using Lanes = ItemLanes<LG>;
  constexpr int IPW = Lanes::IPW;
  constexpr int KEEP = 16 / LG;  // pair distances held per lane after the reduction
  constexpr int kRounds = (12 + LG - 1) / LG;
  constexpr int kOwn = 4 / Lanes::kQuad;  // cells whose permutation entry a lane moves
  __shared__ unsigned long long s_q[kWavesPerBlock][IPW][16];
  const int lane = threadIdx.x & 63;
  const int wib = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int sub = Lanes::chunk(lane), slot = Lanes::slot(lane);
  const int ql = lane % Lanes::kQuad;           // this lane's place in its quad (or pair, or alone)
  const bool owns = sub < Lanes::kQuad;         // one quad of an item moves its permutation entries
  unsigned long long* q_item = s_q[wib][slot];
  const int64_t wave = chiplet_order(bid, nblocks) * kWavesPerBlock + wib;
  const int64_t nwaves = nblocks * kWavesPerBlock;
  const Vec* __restrict__ G4 = reinterpret_cast<const Vec*>(G) + sub;
  const Vec* __restrict__ T4 = reinterpret_cast<const Vec*>(T) + sub;
  Vec* __restrict__ Gout = reinterpret_cast<Vec*>(G) + sub;
  // Distances from this on take the slower way.
  const uint32_t slow_from = __float_as_uint(fminf(ldexpf(1.0f, 57 - geo.s), INFINITY));
  unsigned long long e_acc = 0;
  uint32_t m_acc = 0;

  // The item's cells: each lane of a quad finds one and the quad shares them.
  auto find_cells = [&](int64_t first, int32_t (&cell)[4]) {
    const uint32_t item = static_cast<uint32_t>(first) + slot;
    int32_t own[kOwn];
    if (static_cast<uint32_t>(first) + IPW <= geo.groups) {
      int y0, x0;
      uint32_t entry;
      geo.group_origin(item, y0, x0, entry);
      int32_t t[kOwn];
      if constexpr (kOwn == 4) {
        const int4 t4 = *reinterpret_cast<const int4*>(geo.table + entry);
        t[0] = t4.x, t[1] = t4.y, t[2] = t4.z, t[3] = t4.w;
      } else {
#pragma unroll
        for (int k = 0; k < kOwn; ++k) t[k] = geo.table[entry + ql * kOwn + k];
      }
#pragma unroll
      for (int k = 0; k < kOwn; ++k) own[k] = geo.group_cell(y0, x0, t[k]);
    } else {
#pragma unroll
      for (int k = 0; k < kOwn; ++k) {
        own[k] = 0;
        if (item < geo.groups) {
          int y0, x0;
          uint32_t entry;
          geo.group_origin(item, y0, x0, entry);
          own[k] = geo.group_cell(y0, x0, geo.table[entry + ql * kOwn + k]);
        } else if (item < geo.total) {
          own[k] = geo.single_cell(4 * (item - geo.groups) + ql * kOwn + k);
        }
      }
    }
    if constexpr (kOwn == 4) {
#pragma unroll
      for (int i = 0; i < 4; ++i) cell[i] = own[i];
    } else if constexpr (kOwn == 2) {
      const int32_t other0 = quad_xor<0>(own[0]), other1 = quad_xor<0>(own[1]);
      cell[0] = ql ? other0 : own[0];
      cell[1] = ql ? other1 : own[1];
      cell[2] = ql ? own[0] : other0;
      cell[3] = ql ? own[1] : other1;
    } else {
      cell[0] = quad_lane<0>(own[0]);
      cell[1] = quad_lane<1>(own[0]);
      cell[2] = quad_lane<2>(own[0]);
      cell[3] = quad_lane<3>(own[0]);
    }
  };

  // Software pipeline: the next item's cells (table reads) are resolved
  // while the current item's grid and target cells are in flight.
  int64_t first = wave * IPW;
  int32_t cell[4];
  if (first < geo.total) find_cells(first, cell);
  for (; first < geo.total; first += nwaves * IPW) {
    const uint32_t item = static_cast<uint32_t>(first) + slot;
    const bool is_group = item < geo.groups;
    Vec g[4], tg[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      g[i] = load_quad<assign_stream_loads<S, DP>()>(G4 + static_cast<int64_t>(cell[i]) * LG);
      tg[i] = load_quad<assign_stream_loads<S, DP>()>(T4 + static_cast<int64_t>(cell[i]) * LG);
    }
    int32_t own_perm[kOwn];
    if (owns && is_group) {
#pragma unroll
      for (int k = 0; k < kOwn; ++k) {
        const int i = ql * kOwn + k;
        own_perm[k] = P[i == 0 ? cell[0] : i == 1 ? cell[1] : i == 2 ? cell[2] : cell[3]];
      }
    }
    int32_t next_cell[4] = {0, 0, 0, 0};
    if (first + nwaves * IPW < geo.total) find_cells(first + nwaves * IPW, next_cell);

    // Pair q = 4i + j: grid cell i against target cell j.
    float part[16];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) part[4 * i + j] = V::sq(g[i], tg[j]);
    if constexpr (LG > 1) transpose_level<LG, 0, 8>(part, lane);
    if constexpr (LG > 2) transpose_level<LG, 1, 4>(part, lane);
    if constexpr (LG > 4) transpose_level<LG, 2, 2>(part, lane);
    if constexpr (LG > 8) transpose_level<LG, 3, 1>(part, lane);
    uint32_t most = 0;
#pragma unroll
    for (int t = 0; t < KEEP; ++t) most = max(most, __float_as_uint(part[t]));

    unsigned long long cost;  // of the ordering taken
    int best_m;
    if (__builtin_expect(__ballot(most >= slow_from) == 0, 1)) {
#pragma unroll
      for (int t = 0; t < KEEP; ++t) q_item[t * LG + sub] = quantise(part[t], geo.s);
      wave_lds_sync();
      unsigned long long key = ~0ull;
#pragma unroll
      for (int k = 0; k < kRounds; ++k) {
        const int p = k * LG + sub;
        const uint32_t code = order_code(2 * (p < 12 ? p : 0));
        const unsigned long long* qa = q_item + (code & 3);
        const unsigned long long* qb = q_item + 4 + ((code >> 2) & 3);
        const unsigned long long* qc = q_item + 8 + ((code >> 4) & 3);
        const unsigned long long* qd = q_item + 8 + ((code >> 6) & 3);
        const unsigned long long straight = qc[0] + qd[4], swapped = qd[0] + qc[4];
        const bool swap = swapped < straight;
        const unsigned long long k_p = ((qa[0] + qb[0] + (swap ? swapped : straight)) << 5) | (2 * p + (swap ? 1 : 0));
        if (p < 12 && k_p < key) key = k_p;
      }
      key = item_min<LG>(key);
      best_m = static_cast<int>(key & 31);
      cost = key >> 5;
      if (static_cast<uint32_t>(first) + IPW > geo.groups && !is_group) {
        // Four singles (or fewer, or none) keep their places.
        best_m = 0;
        cost = 0;
        if (item < geo.total)
          for (int i = 0; i < 4; ++i)
            if (4 * (item - geo.groups) + i < geo.singles) cost += q_item[5 * i];
      }
    } else {
      const double scale = ldexp(1.0, geo.s);
      for (int t = 0; t < KEEP; ++t)
        q_item[t * LG + sub] = static_cast<unsigned long long>(static_cast<double>(part[t]) * scale);
      wave_lds_sync();
      cost = ~0ull;
      best_m = 24;
      if (is_group) {
        for (int m = 0; m < 24; ++m) {
          const uint32_t code = order_code(m);
          const unsigned long long c = q_item[code & 3] + q_item[4 + ((code >> 2) & 3)] +
                                       q_item[8 + ((code >> 4) & 3)] + q_item[12 + ((code >> 6) & 3)];
          if (c < cost) {
            cost = c;
            best_m = m;
          }
        }
      } else {
        best_m = 0;
        cost = 0;
        if (item < geo.total)
          for (int i = 0; i < 4; ++i)
            if (4 * (item - geo.groups) + i < geo.singles) cost += q_item[5 * i];
      }
    }
    wave_lds_sync();

    if (best_m != 0) {
      const uint32_t code = order_code(best_m);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int to = (code >> (2 * i)) & 3;
        if (to != i) {
          const int32_t dst = to == 0 ? cell[0] : to == 1 ? cell[1] : to == 2 ? cell[2] : cell[3];
          Gout[static_cast<int64_t>(dst) * LG] = g[i];
        }
      }
      if (owns) {
#pragma unroll
        for (int k = 0; k < kOwn; ++k) {
          const int i = ql * kOwn + k;
          const int to = (code >> (2 * i)) & 3;
          if (to != i) {
            P[to == 0 ? cell[0] : to == 1 ? cell[1] : to == 2 ? cell[2] : cell[3]] = own_perm[k];
            ++m_acc;
          }
        }
      }
    }
    e_acc += cost;
#pragma unroll
    for (int i = 0; i < 4; ++i) cell[i] = next_cell[i];
  }
  // One pair of atomics per block: waves reduce, then the block.
  __shared__ unsigned long long s_sum[2][kWavesPerBlock];
  e_acc = wave_sum_u64(sub == 0 ? e_acc : 0ull);
  const unsigned long long moved = wave_sum_u64(m_acc);
  if (lane == 0) {
    s_sum[0][wib] = e_acc;
    s_sum[1][wib] = moved;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long e = 0, m = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) {
      e += s_sum[0][i];
      m += s_sum[1][i];
    }
    const int slot_acc = static_cast<int>(bid % kAccSlots);
    const unsigned long long e_old =
        __hip_atomic_fetch_add(&st->energy_acc[slot_acc], e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long m_old =
        __hip_atomic_fetch_add(&st->moved_acc[slot_acc], m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // Wait for both results (and every earlier memory operation of this
    // wave): once they have returned, both additions have been made where
    // every block's atomics meet, before anything this thread does next
    // (the control step's ticket).
    asm volatile("s_waitcnt vmcnt(0)" : : "v"(e_old), "v"(m_old) : "memory");
  }
}

// The preparation and the control step of a reorder's assignment (defined
// with the controller below).
__device__ void prepare_step(DevState* __restrict__ st, const LevelInfo* __restrict__ levels);
__device__ void reorder_done(DevState* __restrict__ st, const LevelInfo* __restrict__ levels,
                             plas_level_out* __restrict__ trace, uint32_t nblocks);

// Waves per SIMD the assignment kernels keep room for in registers: more do
// not help (see assign_blocks_cap), and with four many lane layouts spill. At
// three those of two lanes per item do, by four to eight registers (16
// bfloat16 channels, and in batches 8 float32 ones).
constexpr int kAssignWavesPerEu = 3;

template <int DP, typename S>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kAssignWavesPerEu)))
void k_assign(S* __restrict__ G, const S* __restrict__ T, int32_t* __restrict__ P,
              const int32_t* __restrict__ table, DevState* __restrict__ st,
              const LevelInfo* __restrict__ levels, plas_level_out* __restrict__ trace, int control) {
  ItemGeometry geo;
  geo.init(st, table);
  if (st->done) return;
  // With control, block 0 prepares the control step and the others assign.
  const int64_t bid = static_cast<int64_t>(blockIdx.x) - control;
  if (bid >= 0)
    assign_items<DP, S>(G, T, P, geo, st, bid, static_cast<int64_t>(gridDim.x) - control);
  else if (threadIdx.x < 64)
    prepare_step(st, levels);
  if (control && threadIdx.x < 64) reorder_done(st, levels, trace, gridDim.x);
}

// ----------------------------------------------------------------- energy

// out += sum over cells of floor(d(G[p], T[p]) 2^s), s read from device
// memory where the host does not have it yet. Bound by reading G and T once:
// the launch is few blocks with several cells in flight per lane, since every
// block's atomic on the one sum costs 15 ns (1024^2 x 64: 130 us, 4.1 TB/s;
// with one cell in flight and an atomic per wave of 4096 blocks 252 us).
template <int DP, typename S>
__global__ __launch_bounds__(kBlock) void k_energy(const S* __restrict__ G, const S* __restrict__ T,
                                                   int64_t n, int s_host, const int32_t* __restrict__ s_device,
                                                   unsigned long long* __restrict__ out) {
  constexpr int LG = DP / 4;
  constexpr int IPW = 64 / LG;
  __shared__ unsigned long long s_sum[kWavesPerBlock];
  const double scale = ldexp(1.0, s_device != nullptr ? *s_device : s_host);
  const int lane = threadIdx.x & 63;
  const int sub = lane % LG, slot = lane / LG;
  const int wib = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int64_t wave = static_cast<int64_t>(blockIdx.x) * kWavesPerBlock + wib;
  const int64_t nwaves = static_cast<int64_t>(gridDim.x) * kWavesPerBlock;
  using Quad = typename Storage<S>::Quad;
  const Quad* __restrict__ G4 = reinterpret_cast<const Quad*>(G);
  const Quad* __restrict__ T4 = reinterpret_cast<const Quad*>(T);
  unsigned long long acc = 0;
  for (int64_t first = wave * IPW; first < n; first += kEnergyFlight * nwaves * IPW) {
    Quad g[kEnergyFlight], t[kEnergyFlight];
    bool in[kEnergyFlight];
#pragma unroll
    for (int k = 0; k < kEnergyFlight; ++k) {
      const int64_t p = first + k * nwaves * IPW + slot;
      in[k] = p < n;
      const int64_t at = (in[k] ? p : 0) * LG + sub;
      g[k] = G4[at];
      t[k] = T4[at];
    }
#pragma unroll
    for (int k = 0; k < kEnergyFlight; ++k) {
      float v = chunk_sq(Storage<S>::widen4(g[k]), Storage<S>::widen4(t[k]));
#pragma unroll
      for (int m = 1; m < LG; m <<= 1) v = v + __shfl_xor(v, m);
      if (in[k] && sub == 0) acc += static_cast<unsigned long long>(static_cast<double>(v) * scale);
    }
  }
  acc = wave_sum_u64(acc);
  if (lane == 0) s_sum[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < kWavesPerBlock; ++i) acc += s_sum[i];
    atomicAdd(out, acc);
  }
}

// -------------------------------------------------------------------- VAD

// The quality measure of App. C: the population variance of |a - b| over the
// right and down neighbour pairs of the arranged grid, every channel, in
// float64. Partial results are merged in a fixed order, so the result does
// not depend on scheduling.

// A set of values by count, mean and sum of squared deviations from it.
struct Moments {
  double count, mean, dev;
};

// The union of two disjoint sets (Chan, Golub and LeVeque's pairwise update).
// Only terms of one sign are added to dev, so nothing cancels.
__device__ __forceinline__ Moments merge(const Moments& a, const Moments& b) {
  if (b.count == 0.0) return a;
  if (a.count == 0.0) return b;
  const double delta = b.mean - a.mean, count = a.count + b.count, share = b.count / count;
  return Moments{count, a.mean + delta * share, a.dev + b.dev + delta * delta * a.count * share};
}

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m);
  return v;
}

// The moments of an arranged grid [n][DP] (padding channels zero). A wave
// takes chunks of 64 / (DP / 4) columns by kVadRows rows, one quad of channels
// of one column per lane, and walks each chunk down twice: first for the
// chunk's mean, then, out of the caches, for the deviations from it; chunks
// merge by their moments. Pairs that leave the grid and padding channels add
// zero to both sums and are not counted.
//
// Bound by reading the grid once from memory and by the float64 arithmetic,
// about a third of the time (1024^2 x 59: 97 us; 96 with chunks of 32 rows,
// 108 with 2048 blocks, 145 with 512; reading the features in place took 2 x
// 3.1 ms).
template <int DP, typename S>
__global__ __launch_bounds__(kBlock) void k_vad_grid(const S* __restrict__ G, int d, int w, int row_chunks,
                                                     int chunks, Moments* __restrict__ part) {
  constexpr int LG = DP / 4;
  constexpr int kCols = 64 / LG;
  using Quad = typename Storage<S>::Quad;
  __shared__ Moments s_m[kWavesPerBlock];
  const int lane = threadIdx.x & 63;
  const int wib = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int sub = lane % LG, slot = lane / LG;
  const Quad* __restrict__ G4 = reinterpret_cast<const Quad*>(G) + sub;
  Moments total{0.0, 0.0, 0.0};
  double dev = 0.0;  // this lane's squared deviations, all chunks
  const int nwaves = static_cast<int>(gridDim.x) * kWavesPerBlock;
  for (int chunk = static_cast<int>(blockIdx.x) * kWavesPerBlock + wib; chunk < chunks; chunk += nwaves) {
    // Chunks run along the rows first: neighbours share the row below.
    const int x0 = chunk / row_chunks * kCols, y0 = chunk % row_chunks * kVadRows;
    const int x = x0 + slot, xc = x < w ? x : w - 1;
    const int rows = w - y0 < kVadRows ? w - y0 : kVadRows;
    const int downs = w - 1 - y0 < kVadRows ? w - 1 - y0 : kVadRows;  // rows with a row below
    const int cols = w - x0 < kCols ? w - x0 : kCols;
    const int rights = w - 1 - x0 < kCols ? w - 1 - x0 : kCols;       // columns with a column to the right
    const bool right = x + 1 < w, down = x < w;
    const int64_t to_right = right ? LG : 0;
    // visit(|a - b| of each pair of this lane's column), rows y0 .. y0 + rows.
    auto walk = [&](auto&& visit) {
      const Quad* at = G4 + (static_cast<int64_t>(y0) * w + xc) * LG;
      const int64_t pitch = static_cast<int64_t>(w) * LG;
      float4 a = Storage<S>::widen4(at[0]);
#pragma unroll 4
      for (int i = 0; i < rows; ++i) {
        const float4 b = Storage<S>::widen4(at[to_right]);
        if (i < downs) at += pitch;
        const float4 c = Storage<S>::widen4(at[0]);
        visit(a, b, right);
        visit(a, c, down && i < downs);
        a = c;
      }
    };
    const double count = static_cast<double>(d) * (static_cast<double>(rows) * rights +
                                                   static_cast<double>(downs) * cols);
    if (count == 0.0) continue;  // the grid's last cell alone
    double sum = 0.0;
    walk([&](const float4& p, const float4& q, bool valid) {
      const double v = (fabs(static_cast<double>(p.x) - static_cast<double>(q.x)) +
                        fabs(static_cast<double>(p.y) - static_cast<double>(q.y))) +
                       (fabs(static_cast<double>(p.z) - static_cast<double>(q.z)) +
                        fabs(static_cast<double>(p.w) - static_cast<double>(q.w)));
      sum += valid ? v : 0.0;
    });
    const double mean = wave_sum_f64(sum) / count;
    const double mx = 4 * sub < d ? mean : 0.0, my = 4 * sub + 1 < d ? mean : 0.0, mz = 4 * sub + 2 < d ? mean : 0.0,
                 mw = 4 * sub + 3 < d ? mean : 0.0;
    walk([&](const float4& p, const float4& q, bool valid) {
      const double vx = fabs(static_cast<double>(p.x) - static_cast<double>(q.x)) - mx,
                   vy = fabs(static_cast<double>(p.y) - static_cast<double>(q.y)) - my,
                   vz = fabs(static_cast<double>(p.z) - static_cast<double>(q.z)) - mz,
                   vw = fabs(static_cast<double>(p.w) - static_cast<double>(q.w)) - mw;
      const double v = (vx * vx + vy * vy) + (vz * vz + vw * vw);
      dev += valid ? v : 0.0;
    });
    total = merge(total, Moments{count, mean, 0.0});
  }
  total.dev += wave_sum_f64(dev);
  if (lane == 0) s_m[wib] = total;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < kWavesPerBlock; ++i) total = merge(total, s_m[i]);
    part[blockIdx.x] = total;
  }
}

// The variance of the blocks' moments (one block).
__global__ __launch_bounds__(kBlock) void k_vad_merge(const Moments* __restrict__ part, int nparts,
                                                      double* __restrict__ out) {
  __shared__ Moments s_m[kBlock];
  Moments m{0.0, 0.0, 0.0};
  for (int i = threadIdx.x; i < nparts; i += kBlock) m = merge(m, part[i]);
  s_m[threadIdx.x] = m;
  __syncthreads();
  for (int stride = kBlock / 2; stride > 0; stride >>= 1) {
    if (threadIdx.x < stride) s_m[threadIdx.x] = merge(s_m[threadIdx.x], s_m[threadIdx.x + stride]);
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = s_m[0].dev / s_m[0].count;
}

// Without room for an arranged grid the features are read where they are,
// every value of a pair at its own random place (1024^2 x 59: 6.2 ms against
// 0.3), in two passes (the mean, then the mean squared deviation).
template <typename SI>
__device__ __forceinline__ double feature(const SI* __restrict__ F, int64_t n, int d, int layout, int64_t i,
                                          int c) {
  const SI v = layout == 0 ? F[static_cast<int64_t>(c) * n + i] : F[i * d + c];
  return static_cast<double>(Storage<SI>::widen(v));
}

template <typename SI>
__global__ __launch_bounds__(kBlock) void k_vad_partial(const SI* __restrict__ F, const int32_t* __restrict__ perm,
                                                        int64_t n, int d, int w, int layout, int pass,
                                                        const double* __restrict__ mean_in,
                                                        double* __restrict__ part) {
  __shared__ double s_acc[kBlock];
  const double mean = pass == 0 ? 0.0 : mean_in[0];
  double acc = 0.0;
  for (int64_t p = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; p < n;
       p += static_cast<int64_t>(gridDim.x) * kBlock) {
    const int y = static_cast<int>(p / w), x = static_cast<int>(p - static_cast<int64_t>(y) * w);
    const int64_t a = perm != nullptr ? perm[p] : p;
    for (int dir = 0; dir < 2; ++dir) {
      const int yy = y + (dir == 1), xx = x + (dir == 0);
      if (yy >= w || xx >= w) continue;
      const int64_t q = static_cast<int64_t>(yy) * w + xx;
      const int64_t b = perm != nullptr ? perm[q] : q;
      for (int c = 0; c < d; ++c) {
        const double v = fabs(feature(F, n, d, layout, a, c) - feature(F, n, d, layout, b, c));
        acc += pass == 0 ? v : (v - mean) * (v - mean);
      }
    }
  }
  s_acc[threadIdx.x] = acc;
  __syncthreads();
  for (int stride = kBlock / 2; stride > 0; stride >>= 1) {
    if (threadIdx.x < stride) s_acc[threadIdx.x] += s_acc[threadIdx.x + stride];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = s_acc[0];
}

// out[0] = sum of part[0 .. nparts) / count (one block of kBlock threads).
__global__ __launch_bounds__(kBlock) void k_vad_finish(const double* __restrict__ part, int nparts, double count,
                                                       double* __restrict__ out) {
  __shared__ double s_acc[kBlock];
  double acc = 0.0;
  for (int i = threadIdx.x; i < nparts; i += kBlock) acc += part[i];
  s_acc[threadIdx.x] = acc;
  __syncthreads();
  for (int stride = kBlock / 2; stride > 0; stride >>= 1) {
    if (threadIdx.x < stride) s_acc[threadIdx.x] += s_acc[threadIdx.x + stride];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = s_acc[0] / count;
}

// -------------------------------------------------------------- controller

// The control step after each reorder (Sec. 3.1), applied to a state copy:
// E is compared with the previous energy; an improvement of at least
// ceil(E_prev / M) keeps the level and its block shift; the first stall
// draws a new shift; a stall right after a new shift ends the level
// (phi <- decay * phi, precomputed in `levels`). The block shift number
// st.j, the grouping keys of reorder st.k + 1 and the next level come
// prepared in st.next_* (none depends on E). E, moved: the reorder's sums.
// trace may be NULL.
__device__ void control_step(DevState& st, const LevelInfo* __restrict__ levels,
                             plas_level_out* __restrict__ trace, unsigned long long E, unsigned long long moved) {
  st.blocks_done = 0;
  st.k += 1;
  st.level_reorders += 1;
  st.level_moved += moved;
  st.energy_last = E;
  if (st.level_reorders == 1) st.levels_run += 1;
  const int L = st.level;
  if (trace != nullptr) {
    plas_level_out& tr = trace[L];
    tr.phi = levels[L].phi;
    tr.r = levels[L].r;
    tr.beta = levels[L].beta;
    tr.reorders = st.level_reorders;
    tr.energy_fixed = E;
    tr.moved = st.level_moved;
  }
  const uint64_t M = st.inv_threshold;
  const uint64_t prev = st.energy_prev;
  const bool improved = !st.has_prev || (E < prev && prev - E >= (prev + M - 1) / M);
  if (improved) {
    st.energy_prev = E;
    st.has_prev = 1;
    st.just_shifted = 0;
  } else if (st.just_shifted) {
    const int next = L + 1;
    if (next >= st.nlevels) {
      st.done = 1;
      st.ended = 1;
    } else {
      const LevelInfo lv = st.next_level;
      st.level = next;
      st.r = lv.r;
      st.beta = lv.beta;
      st.nb = lv.nb;
      st.groups_per_block = lv.groups_per_block;
      st.groups = lv.groups;
      st.singles = lv.singles;
      st.by_gpb = lv.by_gpb;
      st.by_nb = lv.by_nb;
      st.by_rest = lv.by_rest;
      st.dy = st.next_dy;
      st.dx = st.next_dx;
      st.j += 1;
      st.has_prev = 0;
      st.just_shifted = 0;
      st.level_reorders = 0;
      st.level_moved = 0;
    }
  } else {
    st.dy = st.next_dy;
    st.dx = st.next_dx;
    st.j += 1;
    st.just_shifted = 1;
    st.energy_prev = E;
  }
  if (st.max_reorders > 0 && st.k >= st.max_reorders) st.done = 1;
  if (!st.done)
    for (int i = 0; i < 4; ++i) st.keys[i] = st.next_keys[i];
}

// What the control step of the running reorder may need, prepared by the
// first wave of a block of the assignment launch that does nothing else (the
// draws take longer than a block's share of a small grid): block shift number
// j (lane 0), the grouping keys of reorder k + 1 (lane 1), the next level.
// Written with device-scope atomic exchanges, made where every block's
// atomics meet and complete (their results returned) before that wave takes
// its block's ticket, so the last block, which reads the state after every
// ticket, sees them.
__device__ void prepare_step(DevState* __restrict__ st, const LevelInfo* __restrict__ levels) {
  const int lane = threadIdx.x & 63;
  const Words4 u = draw(st->seed, lane == 0 ? kDrawShift : kDrawGrouping,
                        lane == 0 ? st->j : static_cast<uint64_t>(st->k + 1));
  uint64_t old = 0;  // what the exchanges return: waiting for it is waiting for them
  if (lane == 0) {
    int32_t dy, dx;
    scale_shift_words(u, st->w, &dy, &dx);
    old |= static_cast<uint32_t>(__hip_atomic_exchange(&st->next_dy, dy, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    old |= static_cast<uint32_t>(__hip_atomic_exchange(&st->next_dx, dx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  } else if (lane == 1) {
    for (int i = 0; i < 4; ++i)
      old |= __hip_atomic_exchange(&st->next_keys[i], u.v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const int next = st->level + 1;
  if (next < st->nlevels) {
    static_assert(sizeof(LevelInfo) % 4 == 0, "level copied as 32-bit words");
    constexpr int kWords = sizeof(LevelInfo) / 4;
    static_assert(kWords <= 64, "one word per lane");
    const uint32_t* src = reinterpret_cast<const uint32_t*>(levels + next);
    uint32_t* dst = reinterpret_cast<uint32_t*>(&st->next_level);
    if (lane < kWords)
      old |= __hip_atomic_exchange(dst + lane, src[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  asm volatile("s_waitcnt vmcnt(0)" : : "v"(old) : "memory");
}

// The end of a reorder's assignment launch, run by the first wave of every
// block after the block has added its sums to the state (nblocks blocks of
// this sort; the block's other waves have ended). Its first thread takes a
// ticket (an atomic increment, made after the sums were added); the wave
// that draws the last ticket sees every block's sums and runs the control
// step on the state in place: no block of the launch reads the state after
// taking its ticket, and the next launch of the sort starts after this one
// ends. Device-scope fences are not needed and would be costly here (each
// writes back the L2 of its chiplet): the sums, the tickets, the prepared
// values and the last wave's reads are all device-scope atomics.
__device__ void reorder_done(DevState* __restrict__ st, const LevelInfo* __restrict__ levels,
                             plas_level_out* __restrict__ trace, uint32_t nblocks) {
  static_assert(sizeof(DevState) % 4 == 0, "state is copied as 32-bit words");
  constexpr int kWords = sizeof(DevState) / 4;
  __shared__ DevState s_st;
  const int lane = threadIdx.x & 63;
  uint32_t last = 0;
  if (lane == 0)
    last = __hip_atomic_fetch_add(&st->blocks_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nblocks - 1
               ? 1u
               : 0u;
  if (__builtin_amdgcn_readfirstlane(last) == 0) return;
  uint32_t* words = reinterpret_cast<uint32_t*>(&s_st);
  uint32_t* gwords = reinterpret_cast<uint32_t*>(st);
  for (int i = lane; i < kWords; i += 64)
    words[i] = __hip_atomic_load(gwords + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  wave_lds_sync();
  // Energy slots by the lower half of the wave, moved counts by the upper.
  static_assert(kAccSlots == 32, "one slot per lane of a half");
  unsigned long long* acc = (lane < kAccSlots ? s_st.energy_acc : s_st.moved_acc) + lane % kAccSlots;
  unsigned long long sum = *acc;
  *acc = 0;
#pragma unroll
  for (int m = kAccSlots / 2; m >= 1; m >>= 1) sum += __shfl_xor(sum, m);
  const unsigned long long moved = __shfl(sum, kAccSlots);
  wave_lds_sync();
  if (lane == 0) control_step(s_st, levels, trace, sum, moved);
  wave_lds_sync();
  for (int i = lane; i < kWords; i += 64) gwords[i] = words[i];
}

// ------------------------------------------------------------------ batch
//
// Many independent sorts advance together, one reorder per launch sequence.
// grids[i] holds sort i's buffers and state pair; a launch covers several
// sorts, and its block map gives each block its sort and its index among
// that sort's blocks: map[b] = (grid index << 16) | block index. Every block
// then runs the device functions of single-sort launches. A sort's blur may
// take another kernel than it would alone (batch_ring, ring_rows); all of them
// do the same operations in the same order, so each sort's result does not
// depend on the batch it runs in.

// The kernels' view of BatchGrid: the same layout, with every pointer
// declared as device (global) memory. Pointers read from memory are
// otherwise generic to the compiler, which then emits flat instructions.
#define PLAS_GLOBAL __attribute__((address_space(1)))
struct BatchGridView {
  void PLAS_GLOBAL* G;
  void PLAS_GLOBAL* H;
  void PLAS_GLOBAL* T;
  int32_t PLAS_GLOBAL* P;
  int32_t PLAS_GLOBAL* table;
  const float PLAS_GLOBAL* inv;
  const LevelInfo PLAS_GLOBAL* levels;
  plas_level_out PLAS_GLOBAL* trace;
  DevState PLAS_GLOBAL* state;
  int32_t w;
  int32_t blur_blocks;
  int32_t assign_blocks;
  int32_t pad;
};
static_assert(sizeof(BatchGridView) == sizeof(BatchGrid), "descriptor view layout");
static_assert(offsetof(BatchGridView, w) == offsetof(BatchGrid, w), "descriptor view layout");

__device__ __forceinline__ const BatchGridView& batch_grid(const BatchGrid* __restrict__ grids,
                                                           const uint32_t* __restrict__ map, uint32_t& local) {
  const uint32_t e = map[blockIdx.x];
  local = e & 0xffffu;
  return reinterpret_cast<const BatchGridView*>(grids)[e >> 16];
}

// A global pointer of the view as a plain pointer of type T (the compiler
// keeps track of where it points).
template <typename T, typename U>
__device__ __forceinline__ T* global_ptr(U PLAS_GLOBAL* p) {
  return (T*)((T PLAS_GLOBAL*)p);
}

// A batch blur pass's route (see launch_blur_batch): its axis, source and
// destination grids (0 G, 1 H, 2 T) and whether it fills the grouping table
// afterwards (the first row pass of a reorder).
__host__ __device__ __forceinline__ int route_vertical(int route) { return route & 1; }
__device__ __forceinline__ bool route_table(int route) { return (route >> 5) & 1; }
template <typename S>
__device__ __forceinline__ S* route_grid(const BatchGridView& g, int sel) {
  return global_ptr<S>(sel == 0 ? g.G : sel == 1 ? g.H : g.T);
}

template <typename S, int DP, int GPB>
__global__ __launch_bounds__(GPB * kRelayWaves * 64) __attribute__((amdgpu_waves_per_eu(relay_waves_per_eu<S, GPB>())))
void k_blur_relay_batch(const BatchGrid* __restrict__ grids, const uint32_t* __restrict__ map, int route, int stream) {
  __shared__ RelayLds<S> s_lds[GPB];
  uint32_t local;
  const BatchGridView& g = batch_grid(grids, map, local);
  const DevState* st = global_ptr<const DevState>(g.state);
  int r;
  if (!pass_radius(st, 0, g.w, r)) return;
  const int vertical = route_vertical(route);
  const S* in = route_grid<S>(g, (route >> 1) & 3);
  S* out = route_grid<S>(g, (route >> 3) & 3);
  blur_relay_lines<S, DP, GPB, false>(in, out, g.w, r, vertical, stream != 0, local, g.blur_blocks, s_lds);
  if (route_table(route))
    fill_group_table<GPB * kRelayWaves * 64>(global_ptr<int32_t>(g.table), st->beta, st->keys, local, g.blur_blocks);
}

template <int DP, bool NT>
__global__ __launch_bounds__(kRingWavesPerBlock * 64) __attribute__((amdgpu_waves_per_eu(1)))
void k_blur_ring_batch(const BatchGrid* __restrict__ grids, const uint32_t* __restrict__ map, int route) {
  __shared__ RingLds<128> s_ring[kRingWavesPerBlock];
  uint32_t local;
  const BatchGridView& g = batch_grid(grids, map, local);
  const DevState* st = global_ptr<const DevState>(g.state);
  int r;
  if (!pass_radius(st, 0, g.w, r)) return;
  const int vertical = route_vertical(route);
  const float* in = route_grid<float>(g, (route >> 1) & 3);
  float* out = route_grid<float>(g, (route >> 3) & 3);
  blur_ring_lines<DP, 128, NT>(in, out, g.w, r, vertical, local, g.blur_blocks, s_ring);
  if (route_table(route))
    fill_group_table<kRingWavesPerBlock * 64>(global_ptr<int32_t>(g.table), st->beta, st->keys, local, g.blur_blocks);
}

template <int DP, typename S>
__global__ __launch_bounds__(kBlock) void k_blur_batch(const BatchGrid* __restrict__ grids,
                                                       const uint32_t* __restrict__ map, int route) {
  uint32_t local;
  const BatchGridView& g = batch_grid(grids, map, local);
  const DevState* st = global_ptr<const DevState>(g.state);
  int r;
  if (!pass_radius(st, 0, g.w, r)) return;
  const int vertical = route_vertical(route);
  const S* in = route_grid<S>(g, (route >> 1) & 3);
  S* out = route_grid<S>(g, (route >> 3) & 3);
  const int64_t wave = (static_cast<int64_t>(local) * kBlock + threadIdx.x) >> 6;
  blur_reg_lines<DP, S>(in, out, g.w, r, vertical, global_ptr<const float>(g.inv), wave, threadIdx.x & 63);
  if (route_table(route))
    fill_group_table<kBlock>(global_ptr<int32_t>(g.table), st->beta, st->keys, local, g.blur_blocks);
}

// Every block of a sort adds its sums; the last one of the sort runs its
// control step.
template <int DP, typename S>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kAssignWavesPerEu)))
void k_assign_batch(const BatchGrid* __restrict__ grids, const uint32_t* __restrict__ map) {
  uint32_t local;
  const BatchGridView& g = batch_grid(grids, map, local);
  DevState* st = global_ptr<DevState>(g.state);
  ItemGeometry geo;
  geo.init(st, global_ptr<const int32_t>(g.table));
  if (st->done) return;
  if (local > 0)
    assign_items<DP, S>(global_ptr<S>(g.G), global_ptr<const S>(g.T), global_ptr<int32_t>(g.P), geo, st,
                        static_cast<int64_t>(local) - 1, static_cast<int64_t>(g.assign_blocks) - 1);
  else if (threadIdx.x < 64)
    prepare_step(st, global_ptr<const LevelInfo>(g.levels));
  if (threadIdx.x < 64)
    reorder_done(st, global_ptr<const LevelInfo>(g.levels), global_ptr<plas_level_out>(g.trace),
                 static_cast<uint32_t>(g.assign_blocks));
}

// (done, r, k) of each listed sort's state, for the host's check between
// chunks.
__global__ __launch_bounds__(kBlock) void k_batch_status(const BatchGrid* __restrict__ grids,
                                                         const int32_t* __restrict__ list, int count,
                                                         HostStatus* __restrict__ out) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= count) return;
  const DevState* st = global_ptr<const DevState>(reinterpret_cast<const BatchGridView*>(grids)[list[i]].state);
  HostStatus hs;
  hs.done = st->done;
  hs.r = st->r;
  hs.k = st->k;
  out[i] = hs;
}

}  // namespace

// ------------------------------------------------- no-allocation scratch

// The device memory of plas_grid_energy_noalloc: its three grids, the range
// pass scratch, an accumulator and a flag, and the 1/c table. Host code
// must not pass `scratch` itself to a kernel (it names a host-side stand-in):
// noalloc_scratch gives its address on the current device.
static __device__ __align__(256) unsigned char scratch[NoAllocLayout::kBytes];
static_assert(NoAllocLayout::kOut + sizeof(QueryOut) <= NoAllocLayout::kInv, "query results");
static_assert((kNoAllocMaxSide + 1) * sizeof(float) <= 4096, "1/c table");

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_address[kMaxScratchDevices] = {};
}  // namespace

hipError_t noalloc_scratch(int device, void** out) {
  if (out == nullptr || device < 0 || device >= kMaxScratchDevices) return hipErrorInvalidValue;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_address[device] == nullptr) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_address[device] = ptr;
  }
  *out = g_scratch_address[device];
  return hipSuccess;
}

// --------------------------------------------------------------- launchers

#define PLAS_DISPATCH_DP(dp, CALL) \
  switch (dp) {                    \
    case 4: { constexpr int DPV = 4; CALL; } break;   \
    case 8: { constexpr int DPV = 8; CALL; } break;   \
    case 16: { constexpr int DPV = 16; CALL; } break; \
    case 32: { constexpr int DPV = 32; CALL; } break; \
    case 64: { constexpr int DPV = 64; CALL; } break; \
    default: return hipErrorInvalidValue;             \
  }

// The body sees SV = the storage element type (float, or uint16_t holding
// bfloat16 bits).
#define PLAS_DISPATCH_STORAGE(storage, ...)                \
  if ((storage) == kStorageF32) {                          \
    using SV = float;                                      \
    __VA_ARGS__;                                           \
  } else if ((storage) == kStorageBF16) {                  \
    using SV = uint16_t;                                   \
    __VA_ARGS__;                                           \
  } else {                                                 \
    return hipErrorInvalidValue;                           \
  }

hipError_t launch_begin(QueryOut* out, const int32_t* perm, int64_t n, int32_t* inv, float* counts, int w,
                        hipStream_t stream) {
  const int64_t work = std::max<int64_t>(perm != nullptr ? n : 1, counts != nullptr ? w + 1 : 1);
  k_begin<<<blocks_for(work), kBlock, 0, stream>>>(out, perm, n, inv, counts, w);
  return hipGetLastError();
}

hipError_t launch_start_perm(int32_t* P, int32_t* inv, int64_t n, const uint64_t keys[4], hipStream_t stream) {
  Words4 k;
  for (int i = 0; i < 4; ++i) k.v[i] = keys[i];
  k_start_perm<<<blocks_for(n), kBlock, 0, stream>>>(P, inv, n, k);
  return hipGetLastError();
}

hipError_t launch_check_perm(const int32_t* perm, int64_t n, int32_t* inv, QueryOut* out, hipStream_t stream) {
  const hipError_t e = launch_begin(out, perm, n, inv, nullptr, 0, stream);
  if (e != hipSuccess) return e;
  k_check_inverse<<<blocks_for(n), kBlock, 0, stream>>>(perm, inv, n, &out->bad_perm);
  return hipGetLastError();
}

namespace {
template <typename SI, typename SO, int DP>
void ingest_dp(const void* features, int64_t n, int d, int layout, const int32_t* inv, const int32_t* perm, void* G,
               float* part, QueryOut* out, hipStream_t stream) {
  constexpr int kTile = kIngestTile / DP;
  const int blocks = static_cast<int>(std::min<int64_t>((n + kTile - 1) / kTile, kIngestBlocks));
  const SI* F = static_cast<const SI*>(features);
  SO* dst = static_cast<SO*>(G);
  if (layout == 0)
    k_ingest<DP, SI, SO, 0><<<blocks, kBlock, 0, stream>>>(F, n, d, inv, perm, dst, part, out);
  else
    k_ingest<DP, SI, SO, 1><<<blocks, kBlock, 0, stream>>>(F, n, d, inv, perm, dst, part, out);
  k_ingest_finish<DP><<<1, kFinishBlock, 0, stream>>>(part, blocks, d, n, out);
}
}  // namespace

hipError_t launch_ingest(const void* features, int input_bf16, int64_t n, int d, int layout, int dp, int storage,
                         const int32_t* inv, const int32_t* perm, void* G, float* part, QueryOut* out,
                         hipStream_t stream) {
  if (n < 1 || d < 1 || d > dp) return hipErrorInvalidValue;
  PLAS_DISPATCH_STORAGE(storage, {
    if (input_bf16) {
      PLAS_DISPATCH_DP(dp, (ingest_dp<uint16_t, SV, DPV>(features, n, d, layout, inv, perm, G, part, out, stream)));
    } else {
      PLAS_DISPATCH_DP(dp, (ingest_dp<float, SV, DPV>(features, n, d, layout, inv, perm, G, part, out, stream)));
    }
  });
  return hipGetLastError();
}

constexpr int64_t kInfinityCacheBytes = int64_t(256) << 20;
// Above this the Infinity Cache does not hold a pass's input and output beside
// what the assignment reads next.
constexpr int64_t kLargeWorkingSetBytes = kInfinityCacheBytes / 2;

bool blur_large_working_set(int64_t working_bytes) { return working_bytes > kLargeWorkingSetBytes; }

// Ring rows of a float32 pass at radius r over `groups` line groups of cells of
// DP channels, in a grid of `bytes`; 0: the relay kernel.
//
// 128 rows, about one group per SIMD: where memory bounds the pass, the
// register slots spare the second read of leaving values that the relay ring
// does not hold (1024^2 x 64, row / column pass inside sorts: 97 / 90 us
// against 126 / 122 us at radii 32 to 192, 117 / 114 against 122 / 119 above,
// 92 / 86 both below). With fewer groups a wave that loads, sums and stores in
// turn is the bound (2091^2 x 16, 523 groups: 140 / 138 us against 117 / 129);
// with more than fit the chip at four per CU its waves run in two rounds.
//
// 64 rows, up to two groups per SIMD. Reorders of whole sorts, us, against the
// relay kernel:
//  - r = 32 to 64, where the slots hold the leaving values: 1040^2 x 64 342 and
//    354 at r = 32, 1150^2 400 and 453, 1448^2 583 and 706, 2020^2 1166 and
//    1405, 2600^2 x 32 1019 and 1231. Cells of 16 channels gain too little
//    from it (4200^2 x 16 1916 and 1752);
//  - r of 2/5 of a side and more, where lines take up to half as many steps
//    again and the relay's, four groups per CU, run in two rounds: 1150^2 x 64
//    483 and 489 at half a side, 1448^2 705 and 741, 2020^2 1358 and 1439,
//    4200^2 x 16 2370 and 2555 (at 3/10: 1448^2 735 and 712, 2020^2 1442 and
//    1385). Grids of little more than the cache stay (1040^2 398 and 387).
//    Between, and below r = 32, the relay pass is as fast or faster.
constexpr int64_t kRingMinGroups = 769, kRingMaxGroups = 1024, kSmallRingMaxGroups = 2048;
template <int DP>
inline int ring_rows(int w, int64_t groups, int64_t bytes, int r) {
  if (groups >= kRingMinGroups && groups <= kRingMaxGroups) return blur_large_working_set(bytes) ? 128 : 0;
  if (DP < 16 || groups <= kRingMaxGroups || groups > kSmallRingMaxGroups) return 0;
  if (DP >= 32 && r >= 32 && r <= 64) return bytes > kInfinityCacheBytes ? 64 : 0;
  return 5 * static_cast<int64_t>(r) >= 2 * static_cast<int64_t>(w) && 8 * bytes > 9 * kInfinityCacheBytes ? 64 : 0;
}

// Line groups per block of a relay column pass over a large working set:
// neighbouring groups walk down the same grid rows at the same time, and one
// CU reads them as longer runs. As many as keep every group of the pass on
// the chip at once: float32 blocks of two groups leave room for four groups
// per CU and blocks of three for three, bfloat16 blocks of three for six.
// Column passes inside sorts, one / two / three groups per block: 1448^2 x 64
// bfloat16 117 / 112 / 97 us (r <= 31) and 149 / 143 / 135 (above); 2091^2 x 16
// float32 126 / 132 / 125 and 171 / 199 / 159. Row passes read long runs with
// one (two: 97 -> 117 us), and grids the Infinity Cache holds are not bound
// by memory (723^2 x 64 float32: 47 us with one, 48 with two).
template <typename S>
inline int relay_column_groups(int64_t groups) {
  return sizeof(S) == 2 || groups <= 768 ? 3 : 2;
}

// Streaming stores of a float32 relay pass over more than kRingMaxGroups line
// groups (so of two groups per block along columns): what the next kernel reads
// back from the Infinity Cache is then worth less than the lines the stores
// push out. Below r = 32, where a pass reads once, that takes larger grids.
// Reorders of whole sorts, us, with plain and streaming stores: 1448^2 x 64 584
// and 592 (r = 3), 725 and 708 (65); 1800^2 948 and 927, 1158 and 1088; 2091^2
// 1299 and 1243, 1589 and 1495; 2100^2 x 32 664 and 658, 840 and 789; 1100^2 x
// 64 342 and 354, 430 and 436; with fewer groups (2091^2 x 16) the same within
// 1 %.
inline bool relay_streams_stores(int64_t groups, int64_t bytes, int r) {
  return groups > kRingMaxGroups && 2 * bytes > (r >= 32 ? 3 : 5) * kInfinityCacheBytes;
}

// One pass for storage S and DP channels: the relay or ring kernel when
// cells hold whole 16-byte pieces, else the register kernel.
template <typename S, int DP>
hipError_t blur_pass_dp(const void* in, void* out, int w, const DevState* st, int radius, int vertical,
                        const float* inv, hipStream_t stream, const TableArgs& ta) {
  // With the table, also enough blocks to fill it at about one entry per
  // thread (blocks beyond the lines only do that).
  auto with_table = [&](int64_t blocks, int threads) {
    if (ta.table == nullptr) return static_cast<int>(blocks);
    const int64_t need = std::min<int64_t>(1024, (ta.max_cells + threads - 1) / threads);
    return static_cast<int>(std::max<int64_t>(blocks, need));
  };
  const S* src = static_cast<const S*>(in);
  S* dst = static_cast<S*>(out);
  if constexpr (staged_cells<S, DP>()) {
    const int64_t groups = staged_groups<DP>(w);
    const int64_t bytes = static_cast<int64_t>(w) * w * DP * static_cast<int64_t>(sizeof(S));
    const bool large = blur_large_working_set(bytes);
    const int streams = large && vertical ? 1 : 0;
    if constexpr (sizeof(S) == 4) {
      const int rows = ring_rows<DP>(w, groups, bytes, radius);
      if (rows != 0) {
        constexpr int kThreads = kRingWavesPerBlock * 64;
        const int blocks = with_table((groups + kRingWavesPerBlock - 1) / kRingWavesPerBlock, kThreads);
        if (rows == 128 && streams)
          k_blur_ring<DP, 128, true><<<blocks, kThreads, 0, stream>>>(src, dst, w, st, radius, vertical, ta.table);
        else if (rows == 128)
          k_blur_ring<DP, 128, false><<<blocks, kThreads, 0, stream>>>(src, dst, w, st, radius, vertical, ta.table);
        else if constexpr (DP >= 16) {
          if (streams)
            k_blur_ring<DP, 64, true><<<blocks, kThreads, 0, stream>>>(src, dst, w, st, radius, vertical, ta.table);
          else
            k_blur_ring<DP, 64, false><<<blocks, kThreads, 0, stream>>>(src, dst, w, st, radius, vertical, ta.table);
        }
        return hipGetLastError();
      }
    }
    const int per_block = large && vertical ? relay_column_groups<S>(groups) : 1;
    const int blocks = with_table((groups + per_block - 1) / per_block, per_block * kRelayWaves * 64);
    constexpr int kThreads = kRelayWaves * 64;
    if constexpr (sizeof(S) == 4 && DP >= 16) {
      if (relay_streams_stores(groups, bytes, radius)) {
        if (per_block == 1)
          k_blur_relay<S, DP, 1, true><<<blocks, kThreads, 0, stream>>>(src, dst, w, st, radius, vertical, streams,
                                                                        ta.table);
        else
          k_blur_relay<S, DP, 2, true><<<blocks, 2 * kThreads, 0, stream>>>(src, dst, w, st, radius, vertical, streams,
                                                                            ta.table);
        return hipGetLastError();
      }
    }
    switch (per_block) {
      case 1:
        k_blur_relay<S, DP, 1, false><<<blocks, kThreads, 0, stream>>>(src, dst, w, st, radius, vertical, streams,
                                                                       ta.table);
        break;
      case 2:
        k_blur_relay<S, DP, 2, false><<<blocks, 2 * kThreads, 0, stream>>>(src, dst, w, st, radius, vertical, streams,
                                                                          ta.table);
        break;
      default:
        k_blur_relay<S, DP, 3, false><<<blocks, 3 * kThreads, 0, stream>>>(src, dst, w, st, radius, vertical, streams,
                                                                          ta.table);
    }
  } else {
    const int blocks = with_table((blur_reg_waves<DP>(w) + kWavesPerBlock - 1) / kWavesPerBlock, kBlock);
    k_blur<DP, S><<<blocks, kBlock, 0, stream>>>(src, dst, w, st, radius, vertical, inv, ta.table);
  }
  return hipGetLastError();
}

hipError_t launch_blur_pass(const void* in, void* out, int w, int dp, int storage, const DevState* st,
                            int radius, int vertical, const float* inv, hipStream_t stream, const TableArgs* table) {
  const TableArgs ta = table != nullptr ? *table : TableArgs{};
  PLAS_DISPATCH_STORAGE(storage, {
    PLAS_DISPATCH_DP(dp, return (blur_pass_dp<SV, DPV>(in, out, w, st, radius, vertical, inv, stream, ta)));
  });
  return hipSuccess;
}

hipError_t launch_group_table(int32_t* table, const DevState* st, int64_t max_cells,
                              hipStream_t stream) {
  k_group_table<<<blocks_for(max_cells), kBlock, 0, stream>>>(table, st);
  return hipGetLastError();
}

// Items per wave of the assignment kernel: 64 lanes over DP / C lanes per
// item (C from assign_channels).
inline int64_t assign_items_per_wave(int dp, int storage) {
  const int c = (storage == kStorageBF16 && dp >= 8) ? 8 : 4;
  return 64 / (dp / c);
}

hipError_t launch_assign(void* G, const void* T, int32_t* P, const int32_t* table, DevState* st, int dp,
                         int storage, int64_t max_items, hipStream_t stream, const ControlArgs* control) {
  const int64_t items_per_wave = assign_items_per_wave(dp, storage);
  const int64_t waves = (max_items + items_per_wave - 1) / items_per_wave;
  const ControlArgs ca = control != nullptr ? *control : ControlArgs{};
  const int with_control = control != nullptr ? 1 : 0;
  const int blocks = blocks_for(waves * 64, assign_blocks_cap(storage)) + with_control;
  PLAS_DISPATCH_STORAGE(storage, {
    PLAS_DISPATCH_DP(dp, (k_assign<DPV, SV><<<blocks, kBlock, 0, stream>>>(
                             static_cast<SV*>(G), static_cast<const SV*>(T), P, table, st, ca.levels, ca.trace,
                             with_control)));
  });
  return hipGetLastError();
}

hipError_t launch_energy(const void* G, const void* T, int64_t n, int dp, int storage, int s,
                         const int32_t* s_device, unsigned long long* energy_out, hipStream_t stream) {
  const int64_t cells_per_wave = kEnergyFlight * (64 / (dp / 4));
  const int64_t waves = (n + cells_per_wave - 1) / cells_per_wave;
  const int blocks = blocks_for(waves * 64, kEnergyBlocks);
  PLAS_DISPATCH_STORAGE(storage, {
    PLAS_DISPATCH_DP(dp, (k_energy<DPV, SV><<<blocks, kBlock, 0, stream>>>(
                             static_cast<const SV*>(G), static_cast<const SV*>(T), n, s, s_device, energy_out)));
  });
  return hipGetLastError();
}

// ---- VAD

size_t vad_partial_doubles() { return kMaxGridBlocks; }
static_assert(sizeof(Moments) * kVadBlocks <= kMaxGridBlocks * sizeof(double), "partials");

hipError_t launch_vad_grid(const void* G, int d, int w, int dp, int storage, double* part, double* out,
                           hipStream_t stream) {
  const int row_chunks = (w + kVadRows - 1) / kVadRows;
  const int columns = 64 / (dp / 4);
  const int chunks = (w + columns - 1) / columns * row_chunks;
  const int blocks = blocks_for(static_cast<int64_t>(chunks) * 64, kVadBlocks);
  Moments* moments = reinterpret_cast<Moments*>(part);
  PLAS_DISPATCH_STORAGE(storage, {
    PLAS_DISPATCH_DP(dp, (k_vad_grid<DPV, SV><<<blocks, kBlock, 0, stream>>>(static_cast<const SV*>(G), d, w,
                                                                            row_chunks, chunks, moments)));
  });
  k_vad_merge<<<1, kBlock, 0, stream>>>(moments, blocks, out);
  return hipGetLastError();
}

hipError_t launch_vad_in_place(const void* features, int input_bf16, const int32_t* perm, int64_t n, int d, int w,
                      int layout, double* part, double* out, hipStream_t stream) {
  const int blocks = blocks_for(n);
  const double count = static_cast<double>(d) * 2.0 * w * (w - 1);
  // out[0]: mean |a - b|; out[1]: the variance.
  for (int pass = 0; pass < 2; ++pass) {
    if (input_bf16)
      k_vad_partial<uint16_t><<<blocks, kBlock, 0, stream>>>(static_cast<const uint16_t*>(features), perm, n, d, w,
                                                             layout, pass, out, part);
    else
      k_vad_partial<float><<<blocks, kBlock, 0, stream>>>(static_cast<const float*>(features), perm, n, d, w,
                                                          layout, pass, out, part);
    k_vad_finish<<<1, kBlock, 0, stream>>>(part, blocks, count, out + pass);
  }
  return hipGetLastError();
}

// ---- batch

bool staged_blur(int dp, int storage) { return dp * (storage == kStorageBF16 ? 2 : 4) >= 16; }

int64_t blur_groups(int w, int dp) { return (static_cast<int64_t>(w) * dp + 63) / 64; }

// The ring kernel (128 rows) in batches. It reads leaving values once up to r =
// 192, the relay up to r = 31; but it waits for its own loads, sums and stores
// in turn, so many short lines run slower in it. Reorders, us, relay and ring
// for all grids:
//  - 32 <= r <= 192: four grids of 1024^2 x 64 1475 / 1210 at r = 40 and 1490 /
//    1264 at 190, two of 1448^2 1532 / 1256 and 1536 / 1313, six of 724^2 1118 /
//    975 and 1108 / 1091, two of 3600^2 x 16 2791 / 2232 and 3145 / 2573, eight
//    of 300^2 to 724^2 x 64 794 / 702 and (140) 801 / 788; not where windows
//    are a good part of the line (32 of 256^2 x 64 683 / 707 at r = 100);
//  - below, 1024^2 1240 / 1201 at r = 3, 1448^2 1280 / 1244, 900^2 967 / 958,
//    but 800^2 757 / 796, 300^2 to 724^2 663 / 683, 2091^2 x 16 814 / 952;
//  - above, little (1024^2 1471 / 1466 at r = 300, 1448^2 1537 / 1523).
// Two launches instead of one cost more than either (300^2 to 1024^2 at r =
// 40: ring for all 888, for the three largest 944, for none 1065), so a batch
// decides for all its grids of a width at once, by these gains (in percent of
// a reorder) times cells.
int64_t batch_ring_gain(int w, int dp, int r) {
  const int64_t groups = blur_groups(w, dp), cells = static_cast<int64_t>(w) * w;
  if (dp < 32 && groups < kRingMinGroups) return r < 32 ? -16 * cells : 0;
  if (r < 32) return groups > 896 ? 4 * cells : -4 * cells;
  return r <= 192 && 3 * r <= w ? 16 * cells : 0;
}

// Fewer than 769 groups leave SIMDs idle. The chip takes 1024 at once, and a
// last round that is partly idle costs its share of about a third of the time
// (one grid of n^2 x 64, relay and ring, us, r = 3 and r = 40: 1024 294 / 282
// and 354 / 288, 1280 490 / 547 and 599 / 552, 1448 627 / 652 and 754 / 656,
// 1800 1007 / 970 and 1219 / 986). Where the cache holds the relay's second
// read, only whole rounds are worth it (whole batches, ms: 900^2 and 400^2,
// 1300 groups, 112.5 / 115.5; two of 740^2 125.9 / 126.8; four of 512^2, 2048
// groups, 110.2 / 107.7).
bool batch_ring(int64_t groups, int64_t cells, int64_t bytes, int64_t gain) {
  if (groups < kRingMinGroups) return false;
  const int64_t slots = (groups + kRingMaxGroups - 1) / kRingMaxGroups * kRingMaxGroups;
  if (slots == 2 * kRingMaxGroups && groups < slots && 2 * bytes <= 3 * kInfinityCacheBytes) return false;
  return gain * slots > 32 * (slots - groups) * cells;
}

int batch_blur_blocks(int w, int dp, int storage, int groups_per_block, int64_t max_cells) {
  int64_t blocks = 0, threads = 0;
  const int64_t groups = blur_groups(w, dp);
  if (staged_blur(dp, storage) && groups_per_block == kBatchRing) {
    blocks = (groups + kRingWavesPerBlock - 1) / kRingWavesPerBlock;
    threads = kRingWavesPerBlock * 64;
  } else if (staged_blur(dp, storage)) {
    blocks = (groups + groups_per_block - 1) / groups_per_block;
    threads = kRelayWaves * 64 * groups_per_block;
  } else {
    blocks = (groups + kWavesPerBlock - 1) / kWavesPerBlock;
    threads = kBlock;
  }
  const int64_t need = std::min<int64_t>(1024, (max_cells + threads - 1) / threads);
  return static_cast<int>(std::max(blocks, need));
}

int batch_assign_blocks(int64_t max_items, int dp, int storage, int cap) {
  const int64_t items_per_wave = assign_items_per_wave(dp, storage);
  const int64_t waves = (max_items + items_per_wave - 1) / items_per_wave;
  return blocks_for(waves * 64, cap > 0 ? cap : assign_blocks_cap(storage)) + 1;
}

// Blocks of an assignment launch (its waves stride over the items). A block
// begins and ends with a chain of dependent memory accesses (state, table,
// sums, ticket) of several us, so few blocks that run all along beat many:
// two per CU in float32, three in bfloat16, whose waves hold half the bytes
// in flight. 512 / 768 / 1024 / 2048 / 4096 blocks, us per assignment inside
// sorts: 723^2 x 64 float32 53 / 54 / 53 / 58 / 71, 1024^2 x 64 98 / 101 / 101
// / 99 / 101, 1448^2 x 64 219 / 230 / 241 / 231 / 234 (256 / 384 blocks: 259 /
// 237), 1448^2 x 64 bfloat16 116 / 111 / 127 / 114 / 118.
int assign_blocks_cap(int storage) { return storage == kStorageBF16 ? 768 : 512; }

template <typename S, int DP>
hipError_t blur_batch_dp(const BatchGrid* grids, const uint32_t* map, int blocks, int groups_per_block,
                         int route, int large, hipStream_t stream) {
  if constexpr (staged_cells<S, DP>()) {
    const int streams = large && route_vertical(route) ? 1 : 0;
    if constexpr (sizeof(S) == 4 && DP >= 16) {
      if (groups_per_block == kBatchRing) {
        if (streams)
          k_blur_ring_batch<DP, true><<<blocks, kRingWavesPerBlock * 64, 0, stream>>>(grids, map, route);
        else
          k_blur_ring_batch<DP, false><<<blocks, kRingWavesPerBlock * 64, 0, stream>>>(grids, map, route);
        return hipGetLastError();
      }
    }
    constexpr int kThreads = kRelayWaves * 64;
    switch (groups_per_block) {
      case 1: k_blur_relay_batch<S, DP, 1><<<blocks, kThreads, 0, stream>>>(grids, map, route, streams); break;
      case 2: k_blur_relay_batch<S, DP, 2><<<blocks, 2 * kThreads, 0, stream>>>(grids, map, route, streams); break;
      case 4: k_blur_relay_batch<S, DP, 4><<<blocks, 4 * kThreads, 0, stream>>>(grids, map, route, streams); break;
      default: return hipErrorInvalidValue;
    }
  } else {
    k_blur_batch<DP, S><<<blocks, kBlock, 0, stream>>>(grids, map, route);
  }
  return hipGetLastError();
}

int blur_route(int vertical, int src, int dst, int with_table) {
  return (vertical & 1) | ((src & 3) << 1) | ((dst & 3) << 3) | ((with_table & 1) << 5);
}

hipError_t launch_blur_batch(const BatchGrid* grids, const uint32_t* map, int blocks, int dp, int storage,
                             int groups_per_block, int route, int large, hipStream_t stream) {
  const int src = (route >> 1) & 3, dst = (route >> 3) & 3;
  if (src > 2 || dst < 1 || dst > 2 || src == dst) return hipErrorInvalidValue;
  PLAS_DISPATCH_STORAGE(storage, {
    PLAS_DISPATCH_DP(dp, return (blur_batch_dp<SV, DPV>(grids, map, blocks, groups_per_block, route, large, stream)));
  });
  return hipSuccess;
}

hipError_t launch_assign_batch(const BatchGrid* grids, const uint32_t* map, int blocks, int dp, int storage,
                               hipStream_t stream) {
  PLAS_DISPATCH_STORAGE(storage, {
    PLAS_DISPATCH_DP(dp, (k_assign_batch<DPV, SV><<<blocks, kBlock, 0, stream>>>(grids, map)));
  });
  return hipGetLastError();
}

hipError_t launch_batch_status(const BatchGrid* grids, const int32_t* list, int count, HostStatus* out,
                               hipStream_t stream) {
  if (count <= 0) return hipSuccess;
  k_batch_status<<<(count + kBlock - 1) / kBlock, kBlock, 0, stream>>>(grids, list, count, out);
  return hipGetLastError();
}

#undef PLAS_DISPATCH_STORAGE
#undef PLAS_DISPATCH_DP

}  // namespace plas
