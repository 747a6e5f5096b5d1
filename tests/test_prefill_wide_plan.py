"""CPU checks of the two-product prefill kernel's routing and work split, on a model that restates
`wide_plan()`, the kernel's tile and K-range bounds and its LDS sizes in
paper_2609_24875_amd/csrc/sph_kernels.hip, and of the pack-time flag that admits a matrix to it
(`sph_host_radius_split()`, through the packer built for the host).

- every row tile belongs to exactly one wave, every chunk to exactly one K range, for 12 and 16 tiles
  per workgroup;
- partial outputs fit the workspace the plan sizes;
- the modelled rounding error of the chosen plan is never above the three-product kernel's;
- no plan is chosen at up to 64 batch rows or without the flag.
"""
from __future__ import annotations

import random

import pytest

from test_prefill_plan_model import prefill_plan

PW_MC, KS_MAX = 128, 16


def partial_bytes(n: int, m: int, ks: int) -> int:
    return ks * m * ((n + 15) // 16) * 16 * 4 if ks > 1 else 0


def wide_plan(n: int, k: int, m: int, cus: int = 256, flag: bool = True) -> dict | None:
    if m <= 64 or not flag:
        return None
    nt, ng = (n + 15) // 16, k // 128
    old = prefill_plan(n, k, m, cus)

    def cost(wgs, ks, per_chunk):
        c = (wgs * ks + cus - 1) // cus * ((ng + ks - 1) // ks) * per_chunk
        return c + 4000 + partial_bytes(n, m, ks) // 1000 if ks > 1 else c

    least = cost(old["gx"] * old["gy"], old["ks"], 3200)
    old_err = ng / old["ks"] + 6.0 + (old["ks"] / 2.0 if old["ks"] > 1 else 0.0)
    best = None
    for T in (16, 12):
        gx, gy = (nt + T - 1) // T, (m + PW_MC - 1) // PW_MC
        most = max(1, min(min(cus // (gx * gy), ng), KS_MAX))
        for ks in range(1, most + 1):
            if ng / (2.0 * ks) + 16.7 > old_err:
                continue
            c = cost(gx * gy, ks, 4000 if T == 16 else 3200)
            if c < least:
                least = c
                best = dict(T=T, gx=gx, gy=gy, ks=ks, nt=nt, ng=ng, err=ng / (2.0 * ks) + 16.7, old_err=old_err,
                            ws=partial_bytes(n, m, ks))
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


# shapes of the GPU test (tests/test_gpu_prefill_wide.py): both tile counts, with and without a K split
WIDE_SHAPES = {(1033, 12416, 65): (12, 15), (17462, 1664, 65): (16, 3), (21885, 2816, 129): (12, 1), (24686, 2816, 129): (16, 1)}


@pytest.mark.parametrize("n,k,m", WIDE_SHAPES)
def test_gpu_test_shapes_take_the_wide_kernel(n, k, m):
    P = wide_plan(n, k, m)
    assert check(n, k, m) and (P["T"], P["ks"]) == WIDE_SHAPES[(n, k, m)]


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


def split_flag(gmin, gstep, codebook, radius_bits: int) -> bool:
    """`sph_host_radius_split()` on values."""
    top = (1 << radius_bits) - 1
    return (all(o == 0 or abs(o) * 4096 >= abs(o) + top * s for o, s in zip(gmin, gstep))
            and all(max(c) == 0 or max(c) >= 0.25 for c in codebook))


def test_flag_bounds_the_operand_error():
    """rho * t as two fp16 words (the kernel's rt_split) against the exact product, at the edges of
    what the flag admits: the error stays within 2^-25 of the vector's length in units where the
    group's largest radius is 2^13..2^14, or 1.5 fp32 roundings of the product."""
    import numpy as np
    f16 = np.float16
    g = np.random.default_rng(5)
    for V in (2, 3, 4, 8):
        top = (1 << V) - 1
        for ratio in (2.0 ** -12, 2.0 ** -6, 0.3, 1.0):
            step = g.uniform(0.5, 1.0, 64).astype(f16).astype(np.float64)
            off = (ratio * top * step * 1.001).astype(f16).astype(np.float64) * g.choice([-1, 1], 64)
            cb = np.abs(g.standard_normal((64, 8)))
            cb = (cb / np.linalg.norm(cb, axis=1, keepdims=True)).astype(f16).astype(np.float64)
            assert split_flag(off, step, cb, V)
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
