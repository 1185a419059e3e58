"""The numbering of the bf16 prefill's work items (csrc/items.h, the code the kernel runs), compiled for the CPU and
compared with a plain enumeration of (query block, query head, slice): every task of a call belongs to exactly one item,
and an item looked up with lengths other than those it was counted with still names a block of the lists."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include "items.h"

static void fail(const char* what, const pa_seq& s, int B, int G, int nw, int q) {
  printf("%s: B %d G %d nw %d, queries %d .. %d, item %d of %d\n", what, B, G, nw, s.qs, s.n - 1, q, s.n_items);
  exit(1);
}

int main() {
  const int N = 2048;                            // keys of the context
  for (int B : {64, 128, 192, 256, 1024})
    for (int G : {1, 3, 4, 7})
      for (int nw : {4, 8}) {
        const int shift = (B & (B - 1)) == 0 ? __builtin_ctz((unsigned)B) : -1;
        const int whole = (G * (B / PA_QW) + nw - 1) / nw, i_max = (N - 1) / B;
        const int starts[] = {-5, 0, 1, 31, 32, 33, 63, 64, 100, 127, 128, 191, 192, 255, 256, 600, 1023, 1024, 2047, 2048, 5000};
        const int lens[] = {-1, 0, 1, 2, 31, 32, 33, 64, 65, 150, 192, 255, 256, 257, 513, 1025, 2047, 2048, 9999};
        for (int start : starts)
          for (int len : lens) {
            const pa_seq s = pa_sequence(len, start, N, 1500, B, shift, G, nw);
            const int qs = std::min(std::max(start, 0), N), n = qs + std::min(std::max(len, 0), std::min(N - qs, 1500));
            if (s.qs != qs || s.n != n) fail("clamped wrongly", s, B, G, nw, -1);
            std::map<long, int> seen;            // task -> how often
            int block = 1 << 30;
            for (int q = 0; q < s.n_items; ++q) {
              pa_seq t = s;
              if (pa_existing_item(t, q, B, i_max) != q || t.n_items != s.n_items) fail("not an item that exists", s, B, G, nw, q);
              const pa_item_place a = pa_place_item(q, s, whole, B);
              if (a.i > block) fail("not from the last block down", s, B, G, nw, q);
              block = a.i;
              if (a.chunk * nw >= G * a.nsl) fail("an item without a task", s, B, G, nw, q);
              for (int t = a.chunk * nw; t < std::min((a.chunk + 1) * nw, G * a.nsl); ++t)
                ++seen[((long)a.i * G + t / a.nsl) * (B / PA_QW) + a.sl0 + t % a.nsl];
            }
            long tasks = 0;
            for (int tok = qs - qs % PA_QW; tok < n; tok += PA_QW)
              for (int g = 0; g < G; ++g, ++tasks)
                if (n > qs && seen[((long)(tok / B) * G + g) * (B / PA_QW) + tok % B / PA_QW] != 1) fail("a task not done once", s, B, G, nw, tok);
            if (n > qs ? (long)seen.size() != tasks : s.n_items != 0) fail("tasks of no query", s, B, G, nw, -1);
            // items that the sequence does not have: counted with other lengths
            for (int q : {0, 1, s.n_items, s.n_items + 1, 3 * s.n_items + 7, 100000}) {
              pa_seq t = s;
              const int q1 = pa_existing_item(t, q, B, i_max);
              const pa_item_place a = pa_place_item(q1, t, whole, B);
              if (q1 >= t.n_items) fail("no end", s, B, G, nw, q);
              if (a.i < 0 || a.i > i_max || a.i * B >= t.n || t.n > N) fail("a block outside the lists", s, B, G, nw, q);
              if (a.sl0 < 0 || a.nsl < 1 || a.sl0 + a.nsl > B / PA_QW) fail("slices outside the block", s, B, G, nw, q);
              if (s.n_items == 0 && t.n > t.qs) fail("queries out of nothing", s, B, G, nw, q);
            }
          }
      }
  puts("ok");
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a C++ compiler")
def test_items_cover_every_task_once_and_stay_inside_the_lists(tmp_path):
    src, exe = tmp_path / "items.cpp", tmp_path / "items"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2503_03588_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
