"""A workspace that the binding allocates belongs to the stream the call runs on: the allocator may hand it out
again as soon as the binding returns.  Host only: stand-ins for device tensors and streams."""
from __future__ import annotations

import contextlib

import pytest
import torch

from paper_2412_19829_amd import binding as gb

CURRENT, OTHER = 0x1000, 0x2000


class OnDevice:
    """A CPU tensor that says it is a device tensor."""
    is_cuda = True

    def __init__(self, t):
        self.t = t

    def __getattr__(self, name):
        return getattr(self.t, name)


def call(entry, stream):
    B, H, N, d, H0 = 1, 2, 1100, 64, 0
    q, k, v, out = (OnDevice(torch.zeros(B, H, N, d)) for _ in range(4))
    if entry == "fwd":
        gb.gformer_attn_fwd(q, k, v, out, 8, H0, stream=stream)
    elif entry == "prefill":
        gb.gformer_attn_prefill(q, k, v, out, None, None, OnDevice(torch.zeros(B, H, d * d + d)), 8, H0, stream=stream)
    else:
        gb.gformer_attn_bwd(q, k, v, out, *(OnDevice(torch.zeros(B, H, N, d)) for _ in range(3)), 8, H0, stream=stream)


@pytest.mark.parametrize("entry", ["fwd", "prefill", "bwd"])
@pytest.mark.parametrize("stream", [None, CURRENT, OTHER, 0])
def test_workspace_is_allocated_on_the_calls_stream(monkeypatch, entry, stream):
    active = [CURRENT]
    allocated, launched = [], []
    empty = torch.empty

    def on(s):
        @contextlib.contextmanager
        def scope():
            active.append(s)
            yield
            active.pop()
        return scope()

    def raw(*args):
        launched.append(args[-1])
        return gb.GF_OK

    def record(*args, **kw):
        allocated.append(active[-1])
        return empty(*args, **kw)

    monkeypatch.setattr(gb, "_current_stream", lambda t: active[-1])
    monkeypatch.setattr(gb, f"gformer_attn_{entry}_raw", raw)
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda ptr, device=None: ptr)
    monkeypatch.setattr(torch.cuda, "default_stream", lambda device=None: 0)
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch, "empty", record)
    call(entry, stream)
    assert launched == [CURRENT if stream is None else stream]
    assert allocated == launched and active == [CURRENT]
