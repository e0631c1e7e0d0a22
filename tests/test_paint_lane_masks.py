"""The paints' lane masks (paper_1805_02247_amd/csrc/chunk_masks.h), built with the host compiler,
on the chunks of the last row of a mesh of 2^32 cells in all, with lanes without a particle that
carry the keys of cells that hold some: every run must still end exactly once."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_1805_02247_amd", "csrc")

SRC = r"""
#include <cstdio>
#include "chunk_masks.h"
int main() {
  long wrong = 0, chunks = 0;
  const uint32_t row = 0xffffffffu - 63u;  // first cell of the last row of 64
  for (int lo = 0; lo < 64; ++lo)
    for (int hi = lo; hi < 64; ++hi)
      for (uint32_t iz = 0; iz < 64; ++iz)
        for (int c = 0; c < 9; ++c) {
          const int len = 1 + c % 3;  // the last run's length; one cell less before it
          const int empty = c / 3;    // empty lanes' keys: the nearest particle's, 2^32 - 1 - lane,
                                      // or the last cell's
          const uint64_t ok = (~0ull << lo) & (~0ull >> (63 - hi));
          uint32_t key[64];
          for (int l = 0; l < 64; ++l)
            key[l] = row + iz - (l <= hi - len && iz > 0 ? 1 : 0);
          for (int l = 0; l < 64; ++l)
            if (!((ok >> l) & 1))
              key[l] = empty == 0 ? key[l < lo ? lo : hi] : empty == 1 ? 0xffffffffu - l : 0xffffffffu;
          uint64_t same = 0, ends = 0, joins = 0;
          for (int l = 0; l < 64; ++l) {
            if (key[l] == (l ? key[l - 1] : 0u)) same |= 1ull << l;  // below lane 0: key 0
            if (l < lo || l > hi) continue;
            if (l == hi || key[l + 1] != key[l]) ends |= 1ull << l;
            if (l > lo && key[l - 1] == key[l]) joins |= 1ull << l;
          }
          ++chunks;
          const uint64_t j = pmr::run_joins(same, ok);
          wrong += j != joins || pmr::run_ends(j, ok) != ends;
        }
  std::printf("%ld %ld\n", chunks, wrong);
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_every_run_ends_once_where_empty_lanes_share_a_key(tmp_path):
    src, exe = tmp_path / "masks.cpp", tmp_path / "masks"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    chunks, wrong = map(int, subprocess.run([str(exe)], capture_output=True, text=True,
                                            check=True).stdout.split())
    assert chunks == 64 * 65 // 2 * 64 * 9
    assert wrong == 0
