"""GPU parity of the two-product prefill kernel (large batches): every output against a plain fp64
product of the decoded codes, formed with torch on the GPU, at shapes that the plan sends there (both
tile counts per workgroup, with and without a K split; ragged rows, odd batches). The bar is the one
of every path, |y - y*| <= k 2^-23 sum (|min| + q step) |c| |x|, which does not see one of the operand's two
words missing: that is held by unit activations, whose outputs are the rebuilt weights, and by the
root mean square of the error against the three-product kernel's."""
from __future__ import annotations

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2609_24875_amd as pkg  # noqa: E402
from test_prefill_wide_plan import ROW_SHAPES, WIDE_SHAPES  # noqa: E402

DEV = torch.device("cuda:0")
FMTS = ["W2", "W3", "W2_cfg", "W3_cfg", "W2_16", "W3_25", "W2_63", "W2_72", "W2_82"]
SHAPES = list(WIDE_SHAPES)
CASES = [(f, s) for f in FMTS for s in SHAPES[:2]] + [(f, s) for f in ("W2", "W3") for s in SHAPES[2:]]
FLAGS = 7   # index of the flags word in the private part of the descriptor


def half(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to(DEV).view(torch.float16)


def reference(codes, cb, x, magnitudes=False):
    """X W^T in fp64 from the codes (Eq. 4, 7), or the bound's sum of magnitudes."""
    n, nv = codes["q"].shape
    c = half(cb).double()
    xd = x.double().abs() if magnitudes else x.double()
    out = torch.empty((x.shape[0], n), dtype=torch.float64, device=DEV)
    bits = torch.arange(8, device=DEV, dtype=torch.uint8)
    for lo in range(0, n, 2048):
        blk = {k: v[lo:lo + 2048] for k, v in codes.items()}
        q = torch.from_numpy(blk["q"]).to(DEV).double().view(blk["q"].shape[0], -1, 16)
        off, st = half(blk["gmin"]).double()[..., None], half(blk["gstep"]).double()[..., None]
        r = ((off.abs() if magnitudes else off) + q * st).reshape(q.shape[0], nv, 1)
        w = r * c[torch.from_numpy(blk["dir"].astype(np.int64)).to(DEV)]
        if not magnitudes:
            w = torch.where(((torch.from_numpy(blk["signs"]).to(DEV)[..., None] >> bits) & 1).bool(), -w, w)
        out[:, lo:lo + 2048] = xd @ w.reshape(q.shape[0], -1).t().contiguous()
    return out


def make(fmt, n, k, m, seed=41):
    D, V = synth.FORMATS[fmt]
    g = synth.rng(seed, n, k, synth.STREAM_CODES)
    codes = synth.uniform_codes(n, k, D, V, g)
    codes["gmin"], codes["gstep"] = synth.varied_group_params(n, k, V, g)
    cb = synth.random_codebook(D, synth.rng(seed, synth.STREAM_CODEBOOK))
    x = torch.randn((m, k + 24), generator=torch.Generator(DEV).manual_seed(seed), device=DEV).half()[:, :k]
    return D, V, codes, cb, x


def check(y, codes, cb, x):
    k = x.shape[1]
    err = (y.double() - reference(codes, cb, x)).abs()
    assert bool(torch.isfinite(y).all()) and bool((err <= k * 2.0 ** -23 * reference(codes, cb, x, True)).all())


@pytest.mark.parametrize("fmt,shape", CASES)
def test_wide_prefill_every_output(fmt, shape):
    n, k, m = shape
    D, V, codes, cb, x = make(fmt, n, k, m)
    w = pkg.pack(D, V, codes, cb, device=DEV)
    assert w.desc.off[FLAGS] == 1
    buf = torch.full((m, n + 3), float("nan"), dtype=torch.float32, device=DEV)
    y = pkg.gemm(w, x, out=buf[:, :n])
    check(y, codes, cb, x)
    assert bool(torch.isnan(buf[:, n:]).all())                       # nothing written past n
    again = pkg.gemm(w, x)
    assert torch.equal(again, y) and torch.equal(pkg.gemm(w, x, out_dtype=torch.float16), y.half())
    for ws in w.workspaces.values():
        assert int(torch.count_nonzero(ws)) == 0


def ordinary_params(n, k, V, g):
    """Offsets and steps of groups of Gaussian weights, every group with both."""
    step = g.uniform(0.03, 0.075, (n, k // 128)) / (2 ** V - 1)
    return synth.f16_bits(g.uniform(0.02, 0.04, step.shape)), synth.f16_bits(step)


def kernels(fmt, n, k, m):
    """A packed matrix with ordinary parameters, the same without the flag, its codes and codebook."""
    D, V, codes, cb, _ = make(fmt, n, k, 1)
    codes["gmin"], codes["gstep"] = ordinary_params(n, k, V, synth.rng(5, n, k))
    w, plain = (pkg.pack(D, V, codes, cb, device=DEV) for _ in range(2))
    assert w.desc.off[FLAGS] == 1
    plain.desc.off[FLAGS] = 0
    return w, plain, codes, cb


@pytest.mark.parametrize("fmt,shape", CASES)
def test_wide_prefill_rebuilt_weights(fmt, shape):
    """Unit activations: each output is one weight r s c. One fp32 rounding of the radius (2^-24 of it), the
    split into two fp16 words (1.5 * 2^-23, or 2^-25 where the group's largest radius stands at 2^12 or more:
    test_flag_bounds_the_operand_error) and one fp32 sum of the two (2^-24) make 1.25 * 2^-22 of the
    weight and 2^-37 of the largest radius. One word alone would be 2^-12 off."""
    n, k, m = shape
    w, _, codes, cb = kernels(fmt, n, k, m)
    x = torch.zeros((m, k), dtype=torch.float16, device=DEV)
    col = (torch.arange(m, device=DEV) * 97 + torch.arange(m, device=DEV) // 8) % k
    x[torch.arange(m, device=DEV), col] = 1.0
    y = pkg.gemm(w, x)
    ref = reference(codes, cb, x)
    most = 0.04 + 0.075                                             # ordinary_params
    assert bool(((y.double() - ref).abs() <= 1.25 * 2.0 ** -22 * reference(codes, cb, x, True) + 2.0 ** -37 * most).all())
    assert int(torch.count_nonzero(y)) > 0.9 * y.numel()


@pytest.mark.parametrize("fmt,shape", CASES)
def test_wide_prefill_error_is_no_larger(fmt, shape):
    """Root mean square error of fp32 outputs: within 1% of the three-product kernel's on the same matrix
    (the estimate's own spread over 10^6 outputs is a tenth of that), and of the size of fp32 sums."""
    n, k, m = shape
    w, plain, codes, cb = kernels(fmt, n, k, m)
    x = torch.randn((m, k), generator=torch.Generator(DEV).manual_seed(17), device=DEV).half()
    ref = reference(codes, cb, x)
    new, old = pkg.gemm(w, x), pkg.gemm(plain, x)
    err = [float((y.double() - ref).norm() / ref.norm()) for y in (new, old)]
    # the 2^13 codebook with 4 radius bits takes three products where its third stream makes two the slower way
    assert fmt == "W3_25" or not torch.equal(new, old)
    assert err[0] <= 1.01 * err[1] and err[0] <= 3e-7, err


@pytest.mark.parametrize("kind", ["offset", "step"])
def test_matrices_without_offsets_or_steps_keep_three_products(kind):
    """Their three-product sums round once a chunk, which two products do not match."""
    n, k, m = SHAPES[2]
    D, V, codes, cb, x = make("W2", n, k, m)
    codes["gmin"], codes["gstep"] = ordinary_params(n, k, V, synth.rng(6, n, k))
    codes["gmin" if kind == "offset" else "gstep"][:, ::5] = 0             # a fifth of the groups
    w = pkg.pack(D, V, codes, cb, device=DEV)
    assert w.desc.off[FLAGS] == 0


@pytest.mark.parametrize("fmt", ["W2", "W3"])
def test_matrices_outside_the_flag_and_small_workspaces_keep_the_general_kernel(fmt):
    n, k, m = SHAPES[0]
    D, V, codes, cb, x = make(fmt, n, k, m)
    plain = pkg.pack(D, V, codes, cb, device=DEV)
    plain.desc.off[FLAGS] = 0                                        # a descriptor from before the flag
    y0 = pkg.gemm(plain, x)
    check(y0, codes, cb, x)
    codes["gmin"][7, 3], codes["gstep"][7, 3] = 0x0001, 0x4000       # offset 2^-24 beside steps of 2
    w = pkg.pack(D, V, codes, cb, device=DEV)
    assert w.desc.off[FLAGS] == 0
    y1 = pkg.gemm(w, x)
    check(y1, codes, cb, x)
    keep = torch.arange(n, device=DEV) != 7
    assert torch.equal(y0[:, keep], y1[:, keep])                     # the same kernel, row by row


def test_unknown_flags_are_refused():
    D, V, codes, cb, x = make("W2", 64, 256, 65)
    w = pkg.pack(D, V, codes, cb, device=DEV)
    w.desc.off[FLAGS] = 2
    with pytest.raises(pkg.SphError):
        pkg.gemm(w, x)


# batches at the edges of 48, 64, 80, 96, 112 and 128 batch rows per workgroup: (n, k) on the three-product
# kernel, then on the two-product kernel with 12 and 16 tiles
@pytest.mark.parametrize("fmt", ["W2", "W3", "W3_cfg", "W3_25"])
@pytest.mark.parametrize("n,k,m", [(261, 1024, m) for m in (33, 48, 49, 64, 65, 96, 97, 128, 129, 144, 145)] + list(ROW_SHAPES))
def test_batch_rows_per_workgroup(fmt, n, k, m):
    D, V, codes, cb, x = make(fmt, n, k, m)
    w = pkg.pack(D, V, codes, cb, device=DEV)
    buf = torch.full((m + 1, n + 3), float("nan"), dtype=torch.float32, device=DEV)
    y = pkg.gemm(w, x, out=buf[:m, :n])
    check(y, codes, cb, x)
    assert bool(torch.isnan(buf[:, n:]).all()) and bool(torch.isnan(buf[m]).all())
    for ws in w.workspaces.values():
        assert int(torch.count_nonzero(ws)) == 0
