// Numbering of the bf16 prefill's work items, usable from host code and from kernels.
//
// The queries of a sequence (those of the call: qs .. n-1) lie in nblk blocks of B tokens from block `first` on.  For one
// KV head, a query block has G tasks (the query heads of the group) for each of its 32-query slices that holds a query of
// the call, and a work item is up to nw of them.  Items are counted from the last block down.
#pragma once
#include <stdint.h>
#include "pattern.h"

constexpr int PA_QW = 32;   // query tokens of a task (one wavefront)

// Work items of the last block, and of all blocks.  The first block of a piece that starts inside it and a ragged last
// one take fewer items than a whole one.  (Counted as whole ones, a piece of 2000 rows from position 30001, 28 query heads
// on 4, made 264 items on 256 compute units, a second round for eight of them: 47.9 -> 29.5 us.)
struct pa_seq_items { int c_last, n; };
PA_HD pa_seq_items pa_items_of_sequence(int n, int qs, int first, int nblk, int B, int G, int nw) {
  pa_seq_items s = {0, 0};
  if (nblk <= 0) return s;
  const int skipped = (qs - first * B) / PA_QW, last = (n - 1 - (first + nblk - 1) * B) / PA_QW;
  s.c_last = (G * (last + 1 - (nblk == 1 ? skipped : 0)) + nw - 1) / nw;
  s.n = s.c_last;
  if (nblk > 1) s.n += (nblk - 2) * ((G * (B / PA_QW) + nw - 1) / nw) + (G * (B / PA_QW - skipped) + nw - 1) / nw;
  return s;
}

// A sequence whose length and start come from a device array: keys, first query and its block, blocks, items of the last
// block and in all.  Values outside the context (N keys) or the slab of Q/O (q_rows rows) are clamped.  b_shift: log2 of B, or -1.
struct pa_seq { int n, qs, first, nblk, c_last, n_items; };
PA_HD int pa_block_of(int pos, int B, int b_shift) { return b_shift >= 0 ? pos >> b_shift : pos / B; }
PA_HD pa_seq pa_sequence(int len, int start, int64_t N, int64_t q_rows, int B, int b_shift, int G, int nw) {
  pa_seq s;
  s.qs = start < 0 ? 0 : (start > (int)N ? (int)N : start);
  int room = (int)N - s.qs;            // rows that fit the context, and the slab of Q/O
  if ((int64_t)room > q_rows) room = (int)q_rows;
  s.n = s.qs + (len < 0 ? 0 : (len > room ? room : len));
  s.first = pa_block_of(s.qs, B, b_shift);
  s.nblk = s.n > s.qs ? pa_block_of(s.n - 1, B, b_shift) - s.first + 1 : 0;
  const pa_seq_items it = pa_items_of_sequence(s.n, s.qs, s.first, s.nblk, B, G, nw);
  s.c_last = it.c_last; s.n_items = it.n;
  return s;
}
// Sequences are looked up more than once: items are counted, then found.  Should a caller change the arrays in between,
// item q need not exist any more, and a block number formed from it could lie outside the lists (blocks 0 .. i_max): then the
// sequence's last item takes its place, or, where the sequence has none, an item without a query.
PA_HD int pa_existing_item(pa_seq& s, int q, int B, int i_max) {
  if (q < s.n_items) return q;
  if (s.n_items > 0) return s.n_items - 1;
  s.first = s.first < i_max ? s.first : i_max;
  s.nblk = s.c_last = s.n_items = 1;
  s.qs = s.n = s.first * B + 1;
  return 0;
}

// counts of slices and items are powers of two but for ragged blocks of 128 keys or more and unusual head groups
PA_HD int pa_quot(unsigned x, unsigned y) { return (int)((y & (y - 1)) == 0 ? x >> __builtin_ctz(y) : x / y); }

// Where item q of a sequence lies: query block i, the item's number in it, and the block's slices that hold queries of the
// call (sl0, nsl); chunks: items of a whole block.
struct pa_item_place { int i, chunk, sl0, nsl; };
PA_HD pa_item_place pa_place_item(int q, const pa_seq& s, int chunks, int B) {
  pa_item_place a;
  int r = 0;                           // query blocks behind the item's
  a.chunk = q;
  if (q >= s.c_last) {
    const int rest = q - s.c_last, blocks = pa_quot(rest, chunks);
    r = 1 + blocks;
    a.chunk = rest - blocks * chunks;
  }
  a.i = s.first + s.nblk - 1 - r;
  const int before = s.qs - a.i * B, keys = s.n - a.i * B;
  a.sl0 = before > 0 ? before / PA_QW : 0;
  a.nsl = ((keys < B ? keys : B) + PA_QW - 1) / PA_QW - a.sl0;
  if (a.nsl < 1) a.nsl = 1;
  return a;
}
