"""The binding's order of attempts for a decode call: a held workspace (or none, up to batch 32) goes
to the library at once, everything else asks for the size, allocates and raises as stated."""
from types import SimpleNamespace

import pytest
import torch

from paper_2609_24875_amd import sph as B

STREAM = SimpleNamespace(cuda_stream=77)


def _weights():
    return B.SphWeights(B.CWeights(), torch.empty(0, dtype=torch.uint8), 16, 128, 6, 4)


def _library(need, calls, final=0):
    """An entry that refuses a short workspace before it does anything else, like the library's."""
    def fn(desc, ptr, size, handle):
        assert handle == 77
        calls.append(size)
        if need > 0 and ptr is None:
            return 1
        return 6 if size < need else final
    return fn


@pytest.mark.parametrize("m,held,need,sizes", [
    (1, None, 0, [0]),              # no workspace needed: one call
    (1, None, 512, [0, 512]),       # refused without one, then allocated
    (32, 512, 512, [512]),          # the held one is enough
    (8, 256, 512, [256, 512]),      # held but short: replaced
    (33, None, 0, [0]),             # above 32 the size is asked for first
    (33, None, 512, [512]),
    (2048, 512, 512, [512]),
])
def test_launch_attempts(monkeypatch, m, held, need, sizes):
    asked = []
    monkeypatch.setattr(B, "workspace_bytes", lambda w, mm: asked.append(mm) or need)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    w, calls = _weights(), []
    if held:
        w.workspaces[(m, 77)] = torch.zeros(held, dtype=torch.uint8)
    w.workspaces[(m, 78)] = torch.zeros(4096, dtype=torch.uint8)      # another stream's: never used
    B._launch(_library(need, calls), "call", w, m, SimpleNamespace(device="cpu"), (), STREAM)
    assert calls == sizes
    assert asked == ([] if len(sizes) == 1 and (held or m <= 32) else [m])
    assert w.workspaces[(m, 78)].numel() == 4096
    if need:
        ws = w.workspaces[(m, 77)]
        assert ws.numel() == need and int(ws.count_nonzero()) == 0


def test_launch_errors(monkeypatch):
    """A HIP error is raised at once (the launch may have happened); a refused call is raised by the
    long way; an allocation under capture is refused."""
    monkeypatch.setattr(B, "workspace_bytes", lambda w, m: 0)
    for final, n in ((B.SPH_ERR_HIP, 1), (2, 2)):
        calls = []
        with pytest.raises(B.SphError) as e:
            B._launch(_library(0, calls, final), "call", _weights(), 1, SimpleNamespace(device="cpu"), (), STREAM)
        assert e.value.status == final and len(calls) == n
    monkeypatch.setattr(B, "workspace_bytes", lambda w, m: 512)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)
    with pytest.raises(RuntimeError, match="capturing a graph"):
        B._launch(_library(512, []), "call", _weights(), 1, SimpleNamespace(device="cpu"), (), STREAM)


@pytest.mark.parametrize("missing", [None, "_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_current_stream_handle(monkeypatch, missing):
    """The raw lookup where torch has it, the public one where it does not."""
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=55))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda dev: 40 + dev, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    if missing:
        monkeypatch.delattr(torch._C, missing)
    assert B._stream_handle() == (55 if missing else 43)
    assert B._stream_handle(STREAM) == 77
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: False)
    assert B._stream_handle() == 55
