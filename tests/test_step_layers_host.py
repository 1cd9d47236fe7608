"""Which layers of a decode step may be attended in any order (okv_host.h): the sweep over sorted buffers against every pair of
them, on random buffers.  No GPU: the header is compiled by the host compiler."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_11816_amd", "csrc")
PROGRAM = r"""
#define __host__
#define __device__
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include "okv_host.h"
int main() {
  int free_ones = 0, bound_ones = 0;
  for (int t = 0; t < 200000; ++t) {
    srand(t);
    const int n = 1 + rand() % 12, layers = 1 + rand() % 4, room = 8 + rand() % 90;
    std::vector<okv::Buffer> b;
    for (int i = 0; i < n; ++i) {
      const uintptr_t first = rand() % room;
      b.push_back({first, first + 1 + rand() % 12, rand() % layers, rand() % 3 == 0});
    }
    bool want = true;
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < i; ++j)
        if (b[i].layer != b[j].layer && (b[i].written || b[j].written) && b[i].first < b[j].last && b[j].first < b[i].last) want = false;
    if (okv::layers_independent(b) != want) return printf("wrong for seed %d\n", t), 1;
    (want ? free_ones : bound_ones) += 1;
  }
  printf("%d %d\n", free_ones, bound_ones);
  return 0;
}
"""


def test_layers_that_may_go_together(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    free_ones, bound_ones = map(int, out.stdout.split())
    assert free_ones > 20000 and bound_ones > 20000
