"""CPU checks of the two-product prefill kernel's routing and work split, on a model that restates
`wide_plan()`, the kernel's tile and K-range bounds and its LDS sizes in
paper_2609_24875_amd/csrc/sph_kernels.hip, and of the pack-time flag that admits a matrix to it
(`sph_host_radius_split()` itself, from csrc/sph_pack.cpp built for the host).

- every row tile belongs to exactly one wave, every chunk to exactly one K range, for 12 and 16 tiles
  per workgroup;
- partial outputs fit the workspace the plan sizes;
- the modelled rounding error of the chosen plan is never above the three-product kernel's;
- no plan is chosen at up to 64 batch rows or without the flag;
- the flag is set exactly where its conditions hold, at their edges.
"""
from __future__ import annotations

import os
import random
import shutil
import subprocess

import numpy as np
import pytest

from test_prefill_plan_model import prefill_plan

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PW_MC, KS_MAX = 128, 16


def partial_bytes(n: int, m: int, ks: int) -> int:
    return ks * m * ((n + 15) // 16) * 16 * 4 if ks > 1 else 0


def wide_plan(n: int, k: int, m: int, cus: int = 256, flag: bool = True, third_stream: bool = False) -> dict | None:
    """``third_stream``: the 2^13 codebook with 4 radius bits."""
    if m <= 64 or not flag:
        return None
    nt, ng = (n + 15) // 16, k // 128
    old = prefill_plan(n, k, m, cus)

    def cost(wgs, ks, per_chunk):
        c = (wgs * ks + cus - 1) // cus * ((ng + ks - 1) // ks) * per_chunk
        return c + 4000 + partial_bytes(n, m, ks) // 1000 if ks > 1 else c

    least = cost(old["gx"] * old["gy"], old["ks"], 2600 if old["mc"] == 48 else 3200)
    old_err = 0.18 * ng / old["ks"] + (0.104 * old["ks"] if old["ks"] > 1 else 0.0)
    best = None
    for T in (16, 12):
        gx, gy = (nt + T - 1) // T, (m + PW_MC - 1) // PW_MC
        most = max(1, min(min(cus // (gx * gy), ng), KS_MAX))
        for ks in range(1, most + 1):
            err = 1.9 + 0.1 * ng / ks + (0.05 + 0.005 * ng / ks + 0.0075 * ng if ks > 1 else 0.0)
            if err > old_err:
                continue
            c = cost(gx * gy, ks, {(16, False): 4000, (12, False): 3200, (16, True): 5000, (12, True): 4000}[T, third_stream])
            if c < least:
                least = c
                best = dict(T=T, gx=gx, gy=gy, ks=ks, nt=nt, ng=ng, err=err, old_err=old_err, ws=partial_bytes(n, m, ks))
    return best


def check(n: int, k: int, m: int, cus: int = 256) -> bool:
    P = wide_plan(n, k, m, cus)
    if P is None:
        return False
    T, nt, ng, ks = P["T"], P["nt"], P["ng"], P["ks"]
    assert 1 <= ks <= min(KS_MAX, ng) and P["err"] <= P["old_err"]
    bounds = [(ng * z // ks, ng * (z + 1) // ks) for z in range(ks)]
    assert bounds[0][0] == 0 and bounds[-1][1] == ng and all(a[1] == b[0] for a, b in zip(bounds, bounds[1:]))
    assert all(c1 > c0 for c0, c1 in bounds)
    seen = []
    for bx in range(P["gx"]):
        for wave in range(8):
            if T == 16 or wave < 4:
                seen += [bx * T + 2 * wave, bx * T + 2 * wave + 1]
            else:
                seen.append(bx * T + 4 + wave)
    assert sorted(t for t in seen if t < nt) == list(range(nt)) and len(set(seen)) == len(seen)
    assert P["gy"] * PW_MC >= m > (P["gy"] - 1) * PW_MC
    if ks > 1:
        last = ((ks - 1) * m + m - 1) * (nt * 16) + nt * 16 - 1
        assert (last + 1) * 4 == P["ws"]
    return True


# shapes of the GPU tests (tests/test_gpu_prefill_wide.py): both tile counts, with and without a K split; then
# those whose batches run through the rows per workgroup
WIDE_SHAPES = {(10764, 3968, 66): (12, 4), (16627, 2304, 65): (16, 3), (21807, 3072, 129): (12, 1), (24629, 3072, 130): (16, 1)}
ROW_SHAPES = {**{(10753, 3968, m): (12, 4) for m in (80, 81, 96, 97, 112, 113, 128)},
              **{(7169, 3968, m): (16, 4) for m in (160, 161, 192, 193, 224, 225)}}


@pytest.mark.parametrize("n,k,m", [*WIDE_SHAPES, *ROW_SHAPES])
def test_gpu_test_shapes_take_the_wide_kernel(n, k, m):
    want = {**WIDE_SHAPES, **ROW_SHAPES}[n, k, m]
    assert check(n, k, m)
    P = wide_plan(n, k, m)
    assert (P["T"], P["ks"]) == want


def test_random_shapes():
    rng, taken = random.Random(3), 0
    for _ in range(400):
        n, k = rng.randint(1, 60000), 128 * rng.randint(1, 200)
        m = rng.choice([33, 64, 65, 100, 128, 129, 256, 700, 2048, 65536])
        taken += check(n, k, m, cus=rng.choice([256, 304, 80]))
        assert m > 64 or wide_plan(n, k, m) is None
        assert wide_plan(n, k, m, flag=False) is None
    assert taken > 50


def test_lds_fits():
    for table, kc in [(256 << 4, 128), (256 << 6, 128), (256 << 7, 128), (256 << 8, 128), (16 << 13, 64)]:
        assert table + 2 * PW_MC * kc * 2 <= 160 * 1024


DRIVER = r"""
#include <cstdio>
#include <vector>
#include "../../paper_2609_24875_amd/csrc/sph_host.h"
int main(int argc, char** argv) {
  FILE* f = argc == 2 ? fopen(argv[1], "rb") : nullptr;
  int32_t h[2];   // direction and radius bits, then rows and columns
  int64_t nk[2];
  while (f && fread(h, 4, 2, f) == 2 && fread(nk, 8, 2, f) == 2) {
    const size_t g = (size_t)(nk[0] * (nk[1] / 128)), c = (size_t)8 << h[0];
    std::vector<uint16_t> off(g), st(g), cb(c);
    if (fread(off.data(), 2, g, f) != g || fread(st.data(), 2, g, f) != g || fread(cb.data(), 2, c, f) != c) return 2;
    const sph_format fmt = {8, h[0], h[1], 128};
    printf("%d\n", sph_host_radius_split(&fmt, nk[0], nk[1], off.data(), st.data(), cb.data()) ? 1 : 0);
  }
  return f ? 0 : 1;
}
"""


@pytest.fixture(scope="module")
def host_flag(tmp_path_factory):
    """flag(cases): `sph_host_radius_split()` of (D, V, offsets, steps, codebook) in fp16 bits, offsets and
    steps [n][k/128]."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("flag")
    src, exe = d / "a" / "b" / "flag.cpp", str(d / "flag")
    src.parent.mkdir(parents=True)
    os.symlink(os.path.join(ROOT, "paper_2609_24875_amd"), d / "paper_2609_24875_amd")
    os.symlink(os.path.join(ROOT, "include"), d / "include")
    src.write_text(DRIVER)
    res = subprocess.run([gxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), str(src),
                          os.path.join(ROOT, "paper_2609_24875_amd", "csrc", "sph_pack.cpp"), "-o", exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr

    def flag(cases):
        path = d / "cases.bin"
        with open(path, "wb") as f:
            for D, V, off, st, cb in cases:
                f.write(np.array([D, V], np.int32).tobytes() + np.array([off.shape[0], off.shape[1] * 128], np.int64).tobytes())
                for a in (off, st, cb):
                    f.write(np.ascontiguousarray(a, np.uint16).tobytes())
        out = subprocess.run([exe, str(path)], capture_output=True, text=True, timeout=60)
        assert out.returncode == 0
        return [int(x) for x in out.stdout.split()]

    return flag


def split_flag(off, st, cb, V: int) -> int:
    """The flag's conditions on fp16 bits, in fp64 (exact)."""
    o, s = (np.asarray(a, np.uint16).view(np.float16).astype(np.float64).reshape(-1) for a in (off, st))
    c = np.asarray(cb, np.uint16).view(np.float16).astype(np.float64).max(axis=1)
    o = np.abs(o)
    one, both = int(((o == 0) != (s == 0)).sum()), int(((o != 0) & (s != 0)).sum())
    return int(np.all((o == 0) | (o * 4096 >= o + (2 ** V - 1) * s)) and np.all((c == 0) | (c >= 0.25)) and 16 * one <= 3 * (one + both))


def bits(a):
    return np.asarray(a, np.float64).astype(np.float16).view(np.uint16)


def test_flag_at_its_edges(host_flag):
    g = np.random.default_rng(11)
    cases, want = [], []

    def case(D, V, off, st, cb=None, flag=None):
        if cb is None:
            a = np.abs(g.standard_normal((1 << D, 8)))
            cb = bits(a / np.linalg.norm(a, axis=1, keepdims=True))
        cases.append((D, V, off, st, cb))
        want.append(split_flag(off, st, cb, V) if flag is None else flag)
        assert flag is None or split_flag(off, st, cb, V) == flag

    plain = lambda v: np.full((4, 8), v, np.uint16)
    for V, D in ((2, 6), (3, 6), (4, 6), (8, 8), (3, 13)):
        top = 2 ** V - 1
        # one group's offset on either side of 2^-12 of its largest radius, of either sign
        for step in (1.0, 0.0371, 2.0 ** -9):
            st = bits(step)
            edge = top * float(st.view(np.float16)) / 4095
            near = bits(edge)
            for k in range(-2, 3):
                for sign in (0, 0x8000):
                    off, steps = plain(0x3800), plain(int(st))
                    off[2, 3] = (int(near) + k) | sign
                    case(D, V, off, steps)
        # subnormal offsets and steps, zeros of either sign
        for o, s in ((0x0001, 0x0001), (0x0001, 0x0400), (0x03FF, 0x0001), (0x8001, 0x0003), (0x8000, 0x3C00), (0x0000, 0x3C00), (0x7BFF, 0x7BFF)):
            off, st = plain(0x3800), plain(0x2000)
            off[0, 0], st[0, 0] = o, s
            case(D, V, off, st)
        # zero offsets or steps in 3 and 4 of 16 groups; all-zero groups do not count
        for which in (0, 1):
            for bad, flag in ((6, 1), (7, 0)):
                p = [plain(0x3800), plain(0x2000)]
                p[which].reshape(-1)[:bad] = 0
                case(D, V, *p, flag=flag)
        off, st = plain(0x3800), plain(0x2000)
        off[:3], st[:3] = 0, 0
        case(D, V, off, st, flag=1)
        case(D, V, plain(0), plain(0), flag=1)
        case(D, V, plain(0), plain(0x2000), flag=0)
        case(D, V, plain(0x3800), plain(0), flag=0)
        # the largest coordinate of one entry just below and at 1/4, and an entry of zeros
        for top_bits, flag in ((0x33FF, 0), (0x3400, 1), (0x0000, 1), (0x0001, 0)):
            cb = np.full((1 << D, 8), 0x3500, np.uint16)
            cb[5] = 0
            cb[5, 3] = top_bits
            case(D, V, plain(0x3800), plain(0x2000), cb, flag=flag)
    for _ in range(200):
        V, D = int(g.choice([2, 3, 4, 8])), 6
        off = bits(g.choice([-1, 1], (3, 5)) * 2.0 ** g.uniform(-24, 15, (3, 5)))
        st = bits(2.0 ** g.uniform(-24, 15, (3, 5)))
        if g.random() < 0.7:   # near the edge
            st = bits(np.minimum(np.abs(off.view(np.float16).astype(np.float64)) * 4095 / (2 ** V - 1) * 2.0 ** g.uniform(-1, 0.002, (3, 5)), 6e4))
        off[g.random((3, 5)) < 0.1] = 0
        case(D, V, off, st)
    assert host_flag(cases) == want and 0.2 < sum(want) / len(want) < 0.9


def test_flag_bounds_the_operand_error():
    """rho * t as two fp16 words (the kernel's rt_split) against the exact product, at the edges of
    what the flag admits: the error stays within 2^-25 of the vector's length in units where the
    group's largest radius is 2^13..2^14, or 1.5 fp32 roundings of the product."""
    f16 = np.float16
    g = np.random.default_rng(5)
    for V in (2, 3, 4, 8):
        top = (1 << V) - 1
        for ratio in (2.0 ** -12, 2.0 ** -6, 0.3, 1.0):
            step = g.uniform(0.5, 1.0, 64).astype(f16).astype(np.float64)
            off = (ratio * top * step * 1.001).astype(f16).astype(np.float64) * g.choice([-1, 1], 64)
            cb = np.abs(g.standard_normal((64, 8)))
            cb = (cb / np.linalg.norm(cb, axis=1, keepdims=True)).astype(f16).astype(np.float64)
            assert split_flag(bits(off), bits(step), bits(cb), V)
            up = 2.0 ** (13 - np.floor(np.log2(np.abs(off) + top * step)))
            for q in {0, 1, top // 2, top}:
                rho = ((off + q * step) * up).astype(np.float32).astype(np.float64)
                rh = rho.astype(f16).astype(np.float64)
                rl = (rho - rh).astype(f16).astype(np.float64)
                t = cb
                a, b = rh[:, None], rl[:, None]
                tb = (t * b).astype(f16).astype(np.float64)
                hi = (t * a + tb).astype(f16).astype(np.float64)
                d = (t * a - hi).astype(f16).astype(np.float64)
                lo = (t * b + d).astype(f16).astype(np.float64)
                err = np.abs(hi + lo - t * (rho[:, None]))
                assert np.all(err <= np.maximum(2.0 ** -25, 1.5 * 2.0 ** -23 * np.abs(t * rho[:, None])) + 1e-12), (V, ratio, q)


def wide_rows(m: int, gy: int, codebook13: bool) -> int:
    """Batch rows per workgroup on the two-product kernel."""
    even = (m + gy - 1) // gy
    if codebook13:
        return 96 if even <= 96 else 128
    return max(80, (even + 15) // 16 * 16)


def test_batch_rows_per_workgroup_keep_the_grid():
    """Fewer rows per workgroup: the same number of workgroups covers the batch, none of them empty,
    and both staged X buffers (whole passes of 512 threads) fit beside the tables."""
    for m in range(33, 4097):
        mc = 48 if (m + 47) // 48 == (m + 63) // 64 else 64
        gy = (m + 63) // 64
        assert gy * mc >= m > (gy - 1) * mc
        if m <= 64:
            continue
        gy = (m + PW_MC - 1) // PW_MC
        for cb, table, kc in ((True, 16 << 13, 64), (False, 256 << 8, 128)):
            mc = wide_rows(m, gy, cb)
            assert mc in ((96, 128) if cb else (80, 96, 112, 128)) and gy * mc >= m > (gy - 1) * mc
            step = 512 // (kc // 8)
            assert table + 2 * ((mc + step - 1) // step * step) * kc * 2 <= 160 * 1024
