// Closed-form enumeration of one row of the block-sparse pattern, usable from
// host code and from kernels.  Algorithm 1 (Section 3.3) decides per token
// pair; lifted to blocks, query block i attends key block j <= i when
// i-j < W, or i-j has at most one bit set, or j < S.  The three sets are a
// prefix [0,S), isolated blocks i-2^k, and a suffix [i-W+1, i] of the row, so
// the ascending duplicate-free union can be emitted without sorting.
#pragma once
#include <stdint.h>
#include "../../include/powattn.h"

#if defined(__HIPCC__)
#define PA_HD __host__ __device__ __forceinline__
#else
#define PA_HD inline
#endif

// I: int64_t, or int32_t where positions fit (kernels: half the scalar instructions)
template <class I>
struct pa_row_shape_t {
  I sink_end;  // sink blocks not inside the window: [0, sink_end)
  I win_start; // window (suffix) blocks: [win_start, i]
  I pow_lo;    // power blocks are emitted only inside [pow_lo, win_start)
};
using pa_row_shape = pa_row_shape_t<int64_t>;

template <class I>
PA_HD pa_row_shape_t<I> pa_shape_of_row(int32_t W, int32_t S, uint32_t flags, I i) {
  // the power test admits distance 0, so the diagonal is attended even with W == 0
  const I weff = (flags & POWATTN_POWER) ? (W > 1 ? W : 1) : W;
  pa_row_shape_t<I> r;
  r.win_start = i - weff + 1;
  if (r.win_start < 0) r.win_start = 0;
  const I s_end = (I)S < i + 1 ? (I)S : i + 1;
  r.pow_lo = s_end;
  r.sink_end = s_end < r.win_start ? s_end : r.win_start;
  return r;
}

// The isolated blocks i - 2^k of a row lie inside [pow_lo, win_start) exactly for i - win_start < 2^k <= i - pow_lo:
// n_pow exponents k_max, k_max-1, ... (ascending blocks), found with two leading-zero counts instead of a loop.
struct pa_row_powers { int n_pow, k_max; };
PA_HD int pa_bits(int64_t x) { return 64 - __builtin_clzll((unsigned long long)x); }   // x > 0: its number of bits
PA_HD int pa_bits(int32_t x) { return 32 - __builtin_clz((unsigned)x); }
template <class I>
PA_HD pa_row_powers pa_powers_of_row(const pa_row_shape_t<I>& r, uint32_t flags, I i) {
  pa_row_powers w = {0, 0};
  if (flags & POWATTN_POWER) {
    const I below = i - r.win_start, upto = i - r.pow_lo;
    if (upto >= 1) {
      const int k_min = below > 0 ? pa_bits(below) : 0;
      w.k_max = pa_bits(upto) - 1;
      w.n_pow = w.k_max >= k_min ? w.k_max - k_min + 1 : 0;
    }
  }
  return w;
}

// Calls emit(j) for every attended key block of query block i in ascending
// order and returns how many there were.
template <class F>
PA_HD int64_t pa_for_each_block(int32_t W, int32_t S, uint32_t flags, int64_t i, F&& emit) {
  int64_t n = 0;
  if (flags & POWATTN_DENSE) {
    for (int64_t j = 0; j <= i; ++j) { emit(j); ++n; }
    return n;
  }
  pa_row_shape r = pa_shape_of_row<int64_t>(W, S, flags, i);
  for (int64_t j = 0; j < r.sink_end; ++j) { emit(j); ++n; }
  if (flags & POWATTN_POWER) {
    int64_t p = 1;
    while ((p << 1) <= i) p <<= 1;  // largest power of two <= i (i >= 1), else 1
    for (; p >= 1; p >>= 1) {
      int64_t j = i - p;
      if (j >= r.pow_lo && j < r.win_start) { emit(j); ++n; }
    }
  }
  for (int64_t j = r.win_start; j <= i; ++j) { emit(j); ++n; }
  return n;
}

PA_HD bool pa_block_attended(int32_t W, int32_t S, uint32_t flags, int64_t i, int64_t j) {
  if (j > i || j < 0) return false;
  if (flags & POWATTN_DENSE) return true;
  int64_t d = i - j;
  if (d < W || j < S) return true;
  return (flags & POWATTN_POWER) && ((d & (d - 1)) == 0);
}

// Backward pass: the column of a sink block (every later query block attends it) is cut into parts of this many query
// blocks; kv_heads counts those of all sequences, G the query heads of each.
//
// Short parts end early: a workgroup takes about 1.1 us for 64 queries of a head, and on a short sequence the longest part
// is all that is still running at the end; parts no longer than the longest ordinary column cost nothing there.  But
// every part adds B x head_dim sums of dK and of dV to the same addresses, at about 50 additions a ns on the whole card.
// Both times together are least at part^2 = 0.3 nb sinks kv_heads / G (block size and head_dim cancel); beyond 16 blocks
// nothing is gained.  Gradient pass, head_dim 128, one sink, window only, 32 heads on 8, us, parts as long as an
// ordinary column / of 16 blocks / by this rule: block 64, W = 1, N = 131072 8490 / 2300 / 2340, N = 4096 287 / 167 / 129;
// W = 4, N = 131072 4490 / 3620 / 3630, N = 1000 64 / 114 / 63; block 256, W = 5, 28 on 4, N = 32768 2460 / 2800 / 2470.
PA_HD int32_t pa_sink_part(int64_t nb, int32_t sinks, int32_t W, uint32_t flags, int64_t kv_heads, int32_t G, int32_t B) {
  int64_t longest = (flags & POWATTN_POWER) ? (W > 1 ? W : 1) : W;
  if (flags & POWATTN_POWER)
    for (int64_t pw = 1; pw < nb; pw <<= 1) longest += pw >= W ? 1 : 0;
  int64_t part = longest < 16 ? longest : 16;
  while (part < 16 && 10.0 * part * part * G < 3.0 * nb * sinks * kv_heads) ++part;
  // very many sink blocks of a very long sequence: longer parts, so that the launch has fewer than 2^32 threads (at most
  // 512 for 64 keys)
  while ((nb + sinks * ((nb + part - 1) / part)) * (B / 64) * 512 > 0xffffffffLL && part < nb) part *= 2;
  return (int32_t)part;
}
