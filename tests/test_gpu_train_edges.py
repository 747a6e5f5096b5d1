"""The fine-tuning kernels at the sizes where their launches change: one block and many, gradient sums kept
in the workspace and in the radius gradient's array, two and eight vectors per thread; and at inputs
where the fp32 screening of the levels has to hand over (radii on rounding boundaries, tiny steps, radius
parameters from -80 to 1e4), wide radii, gradients that are not finite. Against the fp64 oracle."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from oracle import sph as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2609_24875_amd import sph as B  # noqa: E402

DEV = torch.device("cuda:0")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def make(fmt, n, k, seed=1, skew=False):
    D, V = synth.FORMATS[fmt]
    g = np.random.default_rng([seed, n, k])
    rho = (0.3 * g.standard_normal((n, k // 8)) - 2.8).astype(np.float32)
    signs = g.integers(0, 256, (n, k // 8)).astype(np.uint8)
    z = g.integers(0, 1 << D, (n, k // 8)).astype(np.uint16)
    if skew:
        z[g.random(z.shape) < 0.9] = 3
    cb = O.f16_to_f64(synth.random_codebook(D, g)).astype(np.float32)
    return D, V, rho, signs, z, cb


def sign_of(signs):
    return 1.0 - 2.0 * ((signs[..., None] >> np.arange(8)) & 1)


def forward(D, V, rho, signs, z, cb):
    return B.fake_quant_forward(D, V, dev(rho), dev(signs), dev(z.view(np.int16)), dev(cb), want_codes=True)


def check_forward(D, V, rho, signs, z, cb):
    n, nv = rho.shape
    w, r_hat, codes = forward(D, V, rho, signs, z, cb)
    r, rh, q = O.fake_quant_radius(rho.astype(np.float64), V)
    rg = r.reshape(n, -1, 16)
    lo, st = O.group_offset_step(rg, V)
    assert np.array_equal(codes["gmin"].cpu().numpy().view(np.uint16), lo)
    assert np.array_equal(codes["gstep"].cpu().numpy().view(np.uint16), st)
    got = codes["q"].cpu().numpy()
    stv = O.f16_to_f64(st)[..., None]
    with np.errstate(divide="ignore", invalid="ignore"):
        x = np.where(stv > 0, (rg - O.f16_to_f64(lo)[..., None]) / stv, 0.0).reshape(n, nv)
    bad = got != q
    assert np.all(np.abs(np.abs(x - np.floor(x)) - 0.5)[bad] <= 1e-12 * np.maximum(1, np.abs(x[bad])))
    ref = np.repeat(O.f16_to_f64(lo), 16, axis=1) + got * np.repeat(O.f16_to_f64(st), 16, axis=1)
    assert np.array_equal(r_hat.cpu().numpy(), ref.astype(np.float32))
    want = (ref[..., None] * sign_of(signs) * cb[z].astype(np.float64)).reshape(n, -1)
    assert np.array_equal(w.cpu().numpy(), want.astype(np.float32))      # one rounding of each product
    return w, r_hat


@pytest.mark.parametrize("fmt", ["W2", "W3", "W3_cfg", "W2_cfg"])
@pytest.mark.parametrize("n,k", [(1, 128), (5, 384), (1031, 512), (2100, 8192)])
def test_forward_sizes(fmt, n, k):
    check_forward(*make(fmt, n, k))


@pytest.mark.parametrize("fmt", ["W2", "W3_cfg"])
def test_forward_hard_levels(fmt):
    """Levels on or beside rounding boundaries, zero and tiny steps, and every size of softplus."""
    D, V, rho, signs, z, cb = make(fmt, 64, 1024)
    top = (1 << V) - 1
    r = np.empty((64, 8, 16))
    g = np.random.default_rng(9)
    for row in range(64):
        lo, st = 0.03125, 2.0 ** -(6 + row % 12)                         # exact in fp16
        lev = g.integers(0, top, (8, 16)) + 0.5 * (g.random((8, 16)) < 0.7)   # half-way points
        lev[:, 0], lev[:, 1] = 0, top
        r[row] = lo + lev * st
    rho = np.log(np.expm1(r)).reshape(64, 128).astype(np.float32)
    rho[7] = rho[7, 0]                                                   # zero steps
    rho[8] = np.linspace(-80, 80, 128)
    rho[9] = 10.0 ** np.linspace(-30, 4, 128)
    rho[10] = -(10.0 ** np.linspace(-30, 2, 128))
    check_forward(D, V, rho, signs, z, cb)


@pytest.mark.parametrize("fmt", ["W2", "W3", "W3_cfg"])
def test_forward_parameters_that_are_no_numbers(fmt):
    """They count as 0 (radius log 2), for their own vector and in their group's offset and step, alone or in
    groups full of them."""
    D, V, rho, signs, z, cb = make(fmt, 40, 1024)
    rho.reshape(-1)[::37] = 0.0
    rho[3, 16:32] = 0.0
    want = forward(D, V, rho, signs, z, cb)
    rho.reshape(-1)[::37] = np.nan
    rho[3, 16:32] = np.nan
    got = forward(D, V, rho, signs, z, cb)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert all(torch.equal(got[2][key], want[2][key]) for key in want[2])


def check_backward(D, V, rho, signs, z, cb, skip=()):
    n, nv = rho.shape
    w, r_hat = forward(D, V, rho, signs, z, cb)[:2]
    gw = np.random.default_rng(4).standard_normal((n, nv * 8)).astype(np.float32)
    for v, value in skip:
        gw.reshape(-1, 8)[v] = value
    perm, off = B.direction_groups(D, z)
    args = (D, V, dev(rho), dev(signs), dev(z.view(np.int16)), dev(cb), r_hat, dev(gw), dev(perm), dev(off))
    gr, gc = B.fake_quant_backward(*args)
    s, g64, c64 = sign_of(signs), gw.reshape(n, nv, 8).astype(np.float64), cb[z].astype(np.float64)
    with np.errstate(invalid="ignore"):
        sig = 1 / (1 + np.exp(-rho.astype(np.float64)))
        ref_r = sig * (g64 * s * c64).sum(axis=2)
        scale = sig * np.abs(g64 * c64).sum(axis=2)
        fine = np.isfinite(ref_r)
        assert np.all(np.abs(gr.cpu().numpy() - ref_r)[fine] <= 8 * 2.0 ** -24 * scale[fine] + 1e-30)
        p = r_hat.cpu().numpy().astype(np.float64)[..., None] * s * g64
        ref_c, mag = np.zeros(cb.shape), np.zeros(cb.shape)
        np.add.at(ref_c, z.reshape(-1), p.reshape(-1, 8))
        np.add.at(mag, z.reshape(-1), np.abs(p).reshape(-1, 8))
    out = gc.cpu().numpy()
    ok = np.isfinite(ref_c)
    # products rounded once; sums of at most 2^13 terms per partial sum, each rounding at most 2^-24 of
    # the magnitudes added so far (their square root in practice: a wide margin)
    assert np.all(np.abs(out - ref_c)[ok] <= 64 * 2.0 ** -24 * mag[ok] + 1e-30)
    assert np.array_equal(np.isfinite(out), ok)                           # only the centres concerned
    again = B.fake_quant_backward(*args)
    assert torch.equal(again[0].nan_to_num(), gr.nan_to_num()) and torch.equal(again[1].nan_to_num(), gc.nan_to_num())
    return args, gr, gc


@pytest.mark.parametrize("fmt", ["W2", "W3", "W3_cfg", "W2_cfg", "W2_72"])
@pytest.mark.parametrize("n,k", [(1, 128), (5, 384), (64, 1024), (129, 4096), (1500, 4096)])
@pytest.mark.parametrize("skew", [False, True])
def test_backward_sizes(fmt, n, k, skew):
    check_backward(*make(fmt, n, k, skew=skew))


@pytest.mark.parametrize("fmt", ["W2", "W3_cfg", "W3"])
def test_backward_gradients_not_finite(fmt):
    D, V, rho, signs, z, cb = make(fmt, 130, 4096)
    check_backward(D, V, rho, signs, z, cb, skip=[(5, np.inf), (70000 % z.size, np.nan), (31, 1e37)])


@pytest.mark.parametrize("fmt", ["W2", "W2_cfg", "W3_cfg", "W3"])
@pytest.mark.parametrize("scale", [1e-36, 1e-34, 1e-32, 1.0, 1e20, 1e26, 1e34])
def test_backward_gradient_scales(fmt, scale):
    """Gradients of any size that fp32 holds, some rows a million times smaller or larger than the others."""
    n, k = 2048, 8192
    D, V, rho, signs, z, cb = make(fmt, n, k)
    r_hat = forward(D, V, rho, signs, z, cb)[1]
    gw = torch.randn((n, k), generator=torch.Generator(DEV).manual_seed(3), device=DEV)
    gw[::31] *= 1e-6
    gw[1::97] *= 30.0
    gw = (gw.double() * scale).float()
    perm, off = (dev(a) for a in B.direction_groups(D, z))
    gc = B.fake_quant_backward(D, V, dev(rho), dev(signs), dev(z.view(np.int16)), dev(cb), r_hat, gw, perm, off)[1].double()
    i = perm.long()
    p = r_hat.reshape(-1)[i].double()[:, None] * dev(sign_of(signs)).reshape(-1, 8)[i] * gw.reshape(-1, 8)[i].double() / scale
    run = torch.cat([torch.zeros((1, 8), dtype=torch.float64, device=DEV), p.cumsum(dim=0)])
    ref = run[off[1:]] - run[off[:-1]]
    # a rounding of each product and a few of the sums, each of at most 2^-24, over the norm
    assert float((gc / scale - ref).norm() / ref.norm()) <= 8 * 2.0 ** -24


def in_place(over, args, gr, gc):
    """The gradients again through the C entry point, one of them over an input: a callable and its outputs."""
    import ctypes
    D, V, rho_d, signs_d, z_d, cb_d, r_hat, gw, perm, off = args
    n, nv = rho_d.shape
    nb = ctypes.c_size_t(0)
    lib = B.load_library()
    assert lib.sph_fake_quant_backward_workspace_bytes(D, ctypes.byref(nb)) == 0
    ws = torch.empty(nb.value, dtype=torch.uint8, device=DEV)
    out_r = {"rho": rho_d, "r_hat": r_hat}.get(over, torch.empty_like(gr))
    out_c = cb_d if over == "codebook" else torch.empty_like(gc)

    def call():
        assert lib.sph_fake_quant_backward(ctypes.byref(B.make_format(D, V)), n, nv * 8, rho_d.data_ptr(), signs_d.data_ptr(),
                                           z_d.data_ptr(), cb_d.data_ptr(), r_hat.data_ptr(), gw.data_ptr(), nv * 8, perm.data_ptr(),
                                           off.data_ptr(), out_r.data_ptr(), out_c.data_ptr(), ws.data_ptr(), ws.numel(),
                                           torch.cuda.current_stream().cuda_stream) == 0

    call.keep = ws
    return call, out_r, out_c


@pytest.mark.parametrize("fmt", ["W2", "W3", "W3_cfg"])
@pytest.mark.parametrize("over", ["rho", "r_hat", "codebook"])
@pytest.mark.parametrize("skew", [False, True])
def test_backward_in_place_of_an_input(fmt, over, skew):
    """The radius gradient written over rho or r^ (no sums are kept there meanwhile), or the codebook's over
    the codebook (which the radius gradient reads first)."""
    args, gr, gc = check_backward(*make(fmt, 1500, 4096, skew=skew))
    call, out_r, out_c = in_place(over, args, gr, gc)
    call()
    torch.cuda.synchronize()
    assert torch.equal(out_r, gr)
    # the same terms in another split: fp32 partial sums, each rounding 2^-24 of the magnitudes added
    assert torch.allclose(out_c, gc, rtol=0, atol=float(gc.abs().max()) * 1e-5)


# either side of the sizes where one pass takes over from the lists (64 entries: 3 * 2^16 vectors, 128 and 256: 2^21),
# and 2^13 entries with the slices' sums in the workspace and in the radius gradient's array
@pytest.mark.parametrize("fmt,n,k", [("W2", 1535, 1024), ("W2", 1536, 1024), ("W2_72", 4095, 4096), ("W2_72", 4096, 4096),
                                     ("W3_cfg", 4095, 4096), ("W3_cfg", 4096, 4096), ("W3", 2047, 4096), ("W3", 2048, 4096)])
@pytest.mark.parametrize("skew", [False, True])
def test_backward_route_edges(fmt, n, k, skew):
    check_backward(*make(fmt, n, k, skew=skew))


def test_backward_time_in_place_and_with_a_crowded_centre():
    """Neither writing a gradient over an input nor nine vectors in ten of one direction may leave the gradients
    to a handful of workgroups (12 to 43 times and 780 times as long as plain calls where they did; now
    about 1 and 30)."""
    def us(fn):
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                fn()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 200)
        return best

    for fmt in ("W2", "W3_cfg"):
        args, gr, gc = check_backward(*make(fmt, 4096, 4096))
        plain = us(lambda: B.fake_quant_backward(*args))
        for over in ("rho", "codebook"):
            assert us(in_place(over, args, gr, gc)[0]) <= 4 * plain, (fmt, over)
    t = [us(lambda: B.fake_quant_backward(*a)) for a in (check_backward(*make("W3", 1024, 4096, skew=s))[0] for s in (False, True))]
    assert t[1] <= 120 * t[0], t
