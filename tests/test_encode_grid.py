"""CPU check of the encoder's launch for small codebooks: `sph_encode_blocks()` from csrc/sph_host.h, built for the
host. A launch has fewer than 2^32 threads at every size the interface takes (n x k / 8 vectors, below 2^35), and
up to 2^30 vectors a wave for every 64 of them."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "%s/paper_2609_24875_amd/csrc/sph_host.h"
int main(int argc, char** argv) {
  for (int i = 1; i < argc; ++i) printf("%%u %%d\n", sph_encode_blocks(atoll(argv[i])), 64 * kEncodeWaves);
}
"""


def test_small_codebook_grid(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "grid.cpp", tmp_path / "grid"
    src.write_text(DRIVER % ROOT)
    res = subprocess.run([gxx, "-std=c++17", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    units = [1, 2, 3, 4, 5, 1000, (1 << 24) - 1, 1 << 24, (1 << 24) + 1, (1 << 26) - 1, 1 << 26, (1 << 26) + 1, (1 << 29) - 1]
    out = subprocess.run([str(exe), *map(str, units)], capture_output=True, text=True, timeout=60).stdout.split("\n")
    for u, line in zip(units, out):
        blocks, threads = map(int, line.split())
        assert 1 <= blocks and blocks * threads < 1 << 32, u
        waves = blocks * threads // 64
        assert u > waves - 4 and (waves >= u or u > 1 << 24), u
