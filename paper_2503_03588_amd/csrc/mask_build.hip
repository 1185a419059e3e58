// Block-index generation: the ascending list of attended key blocks of every
// query block (Algorithm 1 lifted to blocks); a second, optional kernel fills
// the nb x nb byte map.
#include "common.h"

// Bound by latency: a few hundred to a few ten thousand words are written, so what counts is the longest chain of
// one thread.  2^row_shift lanes share a row and entry c of it is formed in closed form (a thread per row, which walks
// the powers of two and stores its entries one after another, each to a cache line of its own: 2.1 -> 1.4 us at 16 blocks,
// 3.8 -> 2.4 us at 2048).
__global__ __launch_bounds__(256) void pa_mask_rows_kernel(int32_t W, int32_t S, uint32_t flags, int32_t nb, int row_shift,
                                                           int32_t* __restrict__ kv_cnt, int32_t* __restrict__ kv_idx, int32_t max_k) {
  const int64_t tid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t i = tid >> row_shift;
  if (i >= nb) return;
  const int c0 = (int)tid & ((1 << row_shift) - 1);
  int32_t* row = kv_idx + i * max_k;
  if (flags & POWATTN_DENSE) {
    if (c0 == 0) kv_cnt[i] = (int32_t)(i + 1 < max_k ? i + 1 : max_k);
    for (int64_t c = c0; c < max_k; c += 1 << row_shift) row[c] = c <= i ? (int32_t)c : -1;
    return;
  }
  const pa_row_shape r = pa_shape_of_row(W, S, flags, i);
  const pa_row_powers w = pa_powers_of_row(r, flags, i);
  const int64_t head = r.sink_end + w.n_pow, n = head + (i - r.win_start + 1);
  if (c0 == 0) kv_cnt[i] = (int32_t)(n < max_k ? n : max_k);   // capacity was checked on the host; never write past the row
  for (int64_t c = c0; c < max_k; c += 1 << row_shift) {
    int64_t j = c;                                            // sink blocks, powers (k descending), window, padding
    if (c >= r.sink_end) j = c < head ? i - ((int64_t)1 << (w.k_max - (int)(c - r.sink_end))) : r.win_start + (c - head);
    row[c] = c < n ? (int32_t)j : -1;
  }
}

__global__ void pa_mask_bytes_kernel(int32_t W, int32_t S, uint32_t flags, int32_t nb, uint8_t* __restrict__ bm) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t total = (int64_t)nb * nb;
  if (idx >= total) return;
  int64_t i = idx / nb, j = idx % nb;
  bm[idx] = pa_block_attended(W, S, flags, i, j) ? 1 : 0;
}

extern "C" int powattn_mask_build(const powattn_pattern* pattern, int64_t seq_len,
                                  int32_t* d_kv_cnt, int32_t* d_kv_idx, int32_t max_k,
                                  uint8_t* d_block_mask, void* hip_stream) {
  int st = pa_check_pattern(pattern);
  if (st != POWATTN_OK) return st;
  if (seq_len < 1 || !d_kv_cnt || !d_kv_idx || max_k < 1) return POWATTN_INVALID_ARG;
  int64_t nb64 = powattn_num_blocks(pattern, seq_len);
  if (nb64 < 0) return POWATTN_INVALID_ARG;
  int32_t need = powattn_max_k(pattern, seq_len);
  if (need < 0) return -need;
  if (max_k < need) return POWATTN_WORKSPACE_TOO_SMALL;
  const int32_t nb = (int32_t)nb64;
  hipStream_t stream = (hipStream_t)hip_stream;
  // lanes of a row: the power of two that covers it, 8 to 64
  int row_shift = 3;
  while (row_shift < 6 && (1 << row_shift) < max_k) ++row_shift;
  while (row_shift > 0 && ((int64_t)nb << row_shift) > (1LL << 31)) --row_shift;   // a launch has fewer than 2^32 threads
  const int64_t row_blocks = (((int64_t)nb << row_shift) + 255) / 256;
  hipLaunchKernelGGL(pa_mask_rows_kernel, dim3((uint32_t)row_blocks), dim3(256), 0, stream,
                     pattern->window, pattern->sink, pattern->flags, nb, row_shift, d_kv_cnt, d_kv_idx, max_k);
  st = pa_note_hip(hipGetLastError());
  if (st != POWATTN_OK) return st;
  if (d_block_mask) {
    int64_t total = (int64_t)nb * nb;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 0x7fffffff) return POWATTN_UNSUPPORTED;
    hipLaunchKernelGGL(pa_mask_bytes_kernel, dim3((uint32_t)blocks), dim3(256), 0, stream,
                       pattern->window, pattern->sink, pattern->flags, nb, d_block_mask);
    st = pa_note_hip(hipGetLastError());
  }
  return st;
}
