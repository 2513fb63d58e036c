"""Node a lane loads in a sweep over a tile's Krylov basis: its own, and past the end of the tile one that its
own wave has written, for every tile size up to three nodes per thread and both workgroup sizes.

A dropped lane's value is multiplied by zero, so it has to be finite: a vector just written by another
wave may still read as whatever the memory held before.  Run on the host, from the library's header."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2103_17081_amd", "csrc")

MAIN = """
#include <cstdio>
#include "common.hpp"
int main() {
  for (int nt : {256, 512})
    for (int nj = 1; nj <= 3 * nt; ++nj)
      for (int tid = 0; tid < nt; ++tid) {
        if (tid / 64 * 64 >= nj) continue;   // the wave has no node
        for (int n = tid; n < nj + 2 * nt; n += nt) {
          const int got = ddh::sweep_node(n, tid, nj);
          const bool own = n < nj ? got == n : got >= 0 && got < nj && got % nt / 64 == tid / 64;
          if (!own) { std::printf("nt %d nj %d tid %d n %d: %d\\n", nt, nj, tid, n, got); return 1; }
        }
      }
  return 0;
}
"""


def test_dropped_lanes_load_what_their_wave_wrote(tmp_path):
    from paper_2103_17081_amd import build
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "sweep.cpp", tmp_path / "sweep"
    src.write_text(MAIN)
    subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", *build.COMMON, "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, capture_output=True, timeout=300)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
