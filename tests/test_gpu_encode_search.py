"""The screened direction search (Eq. 5) and the k-means on listed samples at the inputs where screening
could go wrong: codebooks full of near-ties (entries a few fp16 steps apart), duplicates, vectors whose
squares leave fp32's range, zero vectors, matrices of a few vectors and of rows shorter than a wave,
and samples that fall on a few centres. Directions are compared with the fp64 oracle exactly, except
where its two best cosines differ by less than 1e-14 (fp64 rounding)."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from oracle import sph as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2609_24875_amd as pkg  # noqa: E402

DEV = torch.device("cuda:0")


def near_tied_codebook(D, g):
    """2^D entries in clusters of up to 8: a direction and copies of it with single coordinates
    moved by 0 to 3 steps of fp16 (0: duplicates)."""
    base = synth.random_codebook(D, g)
    for z in range(1 << D):
        src = base[z & ~7].copy()
        src[g.integers(0, 8)] += g.integers(0, 4)
        base[z] = src
    return base


def expected(w, cb):
    d = np.abs(w.astype(np.float64)).reshape(-1, 8)
    d = d / np.maximum(np.linalg.norm(d, axis=1, keepdims=True), 1e-12)
    c = O.f16_to_f64(cb)
    best, second, at = [], [], []
    for lo in range(0, d.shape[0], 2048):
        s = d[lo:lo + 2048] @ c.T
        i = s.argmax(axis=1)
        b = s[np.arange(len(i)), i].copy()
        s[np.arange(len(i)), i] = -1
        at.append(i), best.append(b), second.append(s.max(axis=1))
    return np.concatenate(at), np.concatenate(best) - np.concatenate(second)


def check(fmt, w, cb):
    D, V = synth.FORMATS[fmt]
    out = pkg.encode(D, V, torch.from_numpy(w).to(DEV), torch.from_numpy(cb.view(np.int16)).to(DEV))
    got = out["dir"].cpu().numpy().view(np.uint16).reshape(-1).astype(np.int64)
    at, gap = expected(w, cb)
    zero = np.abs(w).reshape(-1, 8).max(axis=1) == 0
    clear = (gap > 1e-14) & ~zero
    assert np.array_equal(got[clear], at[clear])
    assert np.all(got[zero] == 0)
    assert clear.mean() > 0.3            # the rest: duplicates, whose lower index has to win
    c = O.f16_to_f64(cb)
    same = (~clear) & ~zero
    assert np.all((c[got[same]] == c[at[same]]).all(axis=1) <= (got[same] <= at[same]))


@pytest.mark.parametrize("fmt", ["W2_cfg", "W2", "W2_72", "W3_cfg", "W3"])
@pytest.mark.parametrize("n,k", [(1, 128), (3, 384), (40, 1024)])
def test_near_ties(fmt, n, k):
    D, _ = synth.FORMATS[fmt]
    g = np.random.default_rng([D, n, k])
    cb = near_tied_codebook(D, g)
    # vectors beside the entries, so that several entries of a cluster compete
    c = O.f16_to_f64(cb)[g.integers(0, 1 << D, n * k // 8)]
    w = (c * (1 + 1e-4 * g.standard_normal(c.shape)) * g.choice([-1.0, 1.0], c.shape)).astype(np.float32).reshape(n, k)
    w.reshape(-1, 8)[::7] = 0.0
    check(fmt, w, cb)


@pytest.mark.parametrize("fmt", ["W2", "W3"])
@pytest.mark.parametrize("scale", [1e-36, 1e-20, 1e-10, 1.0, 1e20, 1e36])
def test_scales(fmt, scale):
    D, _ = synth.FORMATS[fmt]
    g = np.random.default_rng(3)
    w = (g.standard_normal((7, 640)) * scale).astype(np.float32)
    if scale >= 1e-10:                   # below, Eq. 3's floor of the radius makes all cosines tiny
        check(fmt, w, synth.random_codebook(D, g))
    else:
        cb = synth.random_codebook(D, g)
        out = pkg.encode(*synth.FORMATS[fmt], torch.from_numpy(w).to(DEV), torch.from_numpy(cb.view(np.int16)).to(DEV))
        got = out["dir"].cpu().numpy().view(np.uint16).reshape(-1)
        d = np.abs(w.astype(np.float64)).reshape(-1, 8)
        assert np.array_equal(got, (d @ O.f16_to_f64(cb).T).argmax(axis=1))


@pytest.mark.parametrize("fmt", ["W2_cfg", "W2", "W2_72", "W3_cfg", "W3"])
@pytest.mark.parametrize("copies", [2, 4, 16])
@pytest.mark.parametrize("n,k", [(1, 128), (40, 1024)])
def test_equal_entries(fmt, copies, n, k):
    """Every entry several times over the codebook: the lowest index, for encoding and for k-means samples (few
    and many lanes of a wave at once, a part of a wave, more copies than blocks are kept)."""
    D, V = synth.FORMATS[fmt]
    g = np.random.default_rng([D, copies, n])
    one = synth.random_codebook(D, g)[: (1 << D) // copies]
    cb = np.tile(one, (copies, 1))
    w = g.standard_normal((n, k)).astype(np.float32)
    wd, cd = torch.from_numpy(w).to(DEV), torch.from_numpy(cb.view(np.int16)).to(DEV)
    got = pkg.encode(D, V, wd, cd)["dir"].cpu().numpy().view(np.uint16).reshape(-1)
    at, gap = expected(w, one)
    assert np.array_equal(got[gap > 1e-14], at[gap > 1e-14])
    u = g.random(1000)
    _, obj, idx = pkg.kmeans_codebook(D, V, wd, torch.from_numpy(u).to(DEV), cd, 1)
    d = np.abs(w.astype(np.float64)).reshape(-1, 8)[idx.cpu().numpy()]
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    c = O.f16_to_f64(cb)
    z = (d @ c[: len(one)].T).argmax(axis=1)
    ref = [(d * c[z]).sum()]
    acc = np.zeros_like(c)
    np.add.at(acc, z, d)
    norm = np.linalg.norm(acc, axis=1, keepdims=True)
    c = np.where(norm > 0, acc / np.maximum(norm, 1e-300), c)        # the copies, without samples, stay
    ref.append((d @ c.T).max(axis=1).sum())
    assert np.allclose(obj.cpu().numpy(), ref, rtol=1e-12)


def test_equal_entries_time():
    """A vector's entries that tie are compared by all lanes together: not one vector after the other, which
    took 5.6 times as long for 64 entries."""
    D, V = synth.FORMATS["W2"]
    g = np.random.default_rng(8)
    one = synth.random_codebook(D, g)
    w = torch.randn((4096, 1024), generator=torch.Generator(DEV).manual_seed(1), device=DEV)

    def us(cb):
        cd, best = torch.from_numpy(cb.view(np.int16)).to(DEV), float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                pkg.encode(D, V, w, cd)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 100)
        return best

    assert us(np.tile(one[:32], (2, 1))) <= 3 * us(one)


def entries_above_two(D, g):
    """Every other entry large (up to fp16's end) where the weights are tiny, so that both kinds compete, the
    large ones a few fp16 steps from each other."""
    cb = synth.random_codebook(D, g)
    far = cb[1::2]
    far[:] = synth.f16_bits(1e-3 * g.random(far.shape))
    at = g.integers(3, 6, len(far))
    far[np.arange(len(far)), at] = 0x7B00 + g.integers(0, 250, len(far))
    return cb


def weights_tiny_there(g, n, k):
    w = g.standard_normal((n, k)).astype(np.float32)
    w.reshape(-1, 8)[:, 3:6] *= 10.0 ** g.uniform(-6, -4.3, (n * k // 8, 1))
    return w


@pytest.mark.parametrize("fmt", ["W2_cfg", "W2", "W2_72", "W3_cfg", "W3"])
def test_entries_above_two(fmt):
    """Larger than a unit direction's coordinates, and than what the packer takes, but finite: the nearest entry."""
    D, V = synth.FORMATS[fmt]
    g = np.random.default_rng(D)
    cb, w = entries_above_two(D, g), weights_tiny_there(g, 40, 1024)
    check(fmt, w, cb)
    # the k-means samples against the same entries as centres
    ns = 3000
    u = g.random(ns)
    _, obj, idx = pkg.kmeans_codebook(D, V, torch.from_numpy(w).to(DEV), torch.from_numpy(u).to(DEV),
                                      torch.from_numpy(cb.view(np.int16)).to(DEV), 0)
    d = np.abs(w.astype(np.float64)).reshape(-1, 8)[idx.cpu().numpy()]
    best = (d / np.linalg.norm(d, axis=1, keepdims=True) @ O.f16_to_f64(cb).T).max(axis=1).sum()
    assert np.allclose(obj.cpu().numpy(), best, rtol=1e-12)


@pytest.mark.parametrize("fmt,ns", [("W2", 5000), ("W3", 5000), ("W3_cfg", 1023), ("W2", 64), ("W3", 70000),
                                    # sums by chunks: a chunk of one sample over, and the most chunks
                                    ("W2_cfg", 32769), ("W3_cfg", 257), ("W2_cfg", 70000)])
def test_kmeans_samples_on_few_centres(fmt, ns):
    """Half of the weight vectors lie beside one of three directions, so a few centres hold most
    samples: objective and codebook against the oracle's fp64 sums."""
    D, V = synth.FORMATS[fmt]
    g = np.random.default_rng(ns)
    w = (0.02 * g.standard_normal((64, 1024))).astype(np.float32)
    vec = w.reshape(-1, 8)
    axis = np.eye(8)[[0, 3, 6]][g.integers(0, 3, len(vec) // 2)]
    vec[: len(vec) // 2] = (0.3 * axis + 0.001 * g.standard_normal(axis.shape)).astype(np.float32)
    cb = synth.random_codebook(D, g)
    u = g.random(ns)
    iters = 3
    got, obj, idx = pkg.kmeans_codebook(D, V, torch.from_numpy(w).to(DEV), torch.from_numpy(u).to(DEV),
                                        torch.from_numpy(cb.view(np.int16)).to(DEV), iters)
    d = np.abs(vec.astype(np.float64))
    d /= np.maximum(np.linalg.norm(d, axis=1, keepdims=True), 1e-12)
    d = d[idx.cpu().numpy()]
    cen, ref = O.f16_to_f64(cb), []
    for it in range(iters + 1):
        s = d @ cen.T
        z = s.argmax(axis=1)
        ref.append(s[np.arange(ns), z].sum())
        if it < iters:
            acc = np.zeros_like(cen)
            np.add.at(acc, z, d)
            norm = np.linalg.norm(acc, axis=1, keepdims=True)
            cen = np.where(norm > 0, acc / np.maximum(norm, 1e-300), cen)
    assert np.bincount(z, minlength=1 << D).max() > min(ns // 16, 300)
    assert np.allclose(obj.cpu().numpy(), ref, rtol=1e-12)
    out = got.cpu().numpy().view(np.uint16)
    assert np.max(np.abs(O.f16_to_f64(out) - cen)) <= 2.0 ** -11 and (out != O.f64_to_f16(cen)).mean() < 1e-4
    again = pkg.kmeans_codebook(D, V, torch.from_numpy(w).to(DEV), torch.from_numpy(u).to(DEV),
                                torch.from_numpy(cb.view(np.int16)).to(DEV), iters)
    assert torch.equal(again[0], got) and torch.equal(again[1], obj)
