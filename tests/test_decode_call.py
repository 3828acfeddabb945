"""The native host side of a decode step: the same step as the binding's own code, which takes whatever is not a plain call
and refuses what it refused."""
from __future__ import annotations

import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2412_19829_amd import binding as gb


def _step(B, H, H0, d, w, dtype, device):
    gen = torch.Generator().manual_seed(7)
    def normal(*shape, dt=dtype):
        return torch.randn(*shape, generator=gen).to(dt).to(device)
    q, k, v = (normal(B, H, d) for _ in range(3))
    kc, vc = (normal(B, H0, w, d) if H0 else None for _ in range(2))
    st = normal(B, H - H0, d * d + d, dt=torch.float32).abs() if H0 < H else None
    return q, k, v, torch.empty_like(q), kc, vc, st


def test_host_tensors_are_left_to_the_binding():
    args = _step(1, 2, 1, 64, 8, torch.float32, "cpu")
    assert gb._decode_call()(gb.lib().decode_address, *args, 8, 1, 3, 0, 1.0, 0.0, None) is None
    assert gb._decode_call()(gb.lib().decode_address, 1, *args[1:], 8, 1, 3, 0, 1.0, 0.0, None) is None
    with pytest.raises(ValueError, match="no CPU path"):
        gb.gformer_attn_decode(*args, 8, 1, 3)
    with pytest.raises(TypeError):
        gb._decode_call()(gb.lib().decode_address, *args)


@pytest.mark.parametrize("what", ["gb.CALL_PATH = '/none/_decode_call.so'", "del torch._C._cuda_getCurrentRawStream"],
                         ids=["no module", "no raw stream"])
def test_without_the_module_or_the_raw_stream(what):
    """What the module lacks is no reason to refuse a call: host tensors get the binding's own message, not the loader's."""
    code = f"""
import warnings
import torch
from paper_2412_19829_amd import binding as gb
from tests.test_decode_call import _step
{what}
args = _step(1, 2, 1, 64, 8, torch.float32, "cpu")
with warnings.catch_warnings(record=True) as said:
    for _ in range(2):
        try:
            gb.gformer_attn_decode(*args, 8, 1, 3)
        except ValueError as e:
            print(e)
print(len([w for w in said if w.category is RuntimeWarning]))
"""
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True)
    lines = r.stdout.strip().splitlines()
    assert r.returncode == 0 and len(lines) == 3, r.stderr[-500:]
    assert "no CPU path" in lines[0] and "no CPU path" in lines[1] and lines[2] == ("1" if "none" in what else "0")


@pytest.mark.gpu
@pytest.mark.parametrize("what", ["gb.CALL_PATH = '/none/_decode_call.so'", "del torch._C._cuda_getCurrentRawStream"],
                         ids=["no module", "no raw stream"])
def test_the_same_step_without_them(what):
    code = f"""
import torch
from paper_2412_19829_amd import binding as gb
from tests.test_decode_call import _step
args = [_step(2, 3, 1, 64, 8, torch.bfloat16, "cuda") for _ in range(2)]
{what}
gb.gformer_attn_decode(*args[0], 8, 1, 3)
gb.gformer_attn_decode(*args[1], 8, 1, 3, stream=torch.cuda.current_stream().cuda_stream)
torch.cuda.synchronize()
assert all(torch.equal(a, b) for a, b in zip(*args))
print("same")
"""
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "same", r.stderr[-500:]


# Each in a process of its own, which an exception that leaves the module's C function would end.
@pytest.mark.parametrize("which", range(7))
def test_a_nested_tensor_is_left_to_the_binding(which):
    code = f"""
import torch
from paper_2412_19829_amd import binding as gb
from tests.test_decode_call import _step
args = list(_step(2, 3, 1, 64, 8, torch.float32, "cpu"))
args[{which}] = torch.nested.nested_tensor([x.clone() for x in args[{which}]])
assert gb._decode_call()(gb.lib().decode_address, *args, 8, 1, 3, 0, 1.0, 0.0, None) is None
try:
    gb.gformer_attn_decode(*args, 8, 1, 3)
except (RuntimeError, ValueError):
    print("refused")
"""
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "refused", r.stderr[-500:]


@pytest.mark.gpu
@pytest.mark.parametrize("case", [(1, 12, 2, 64, 128, 2048), (3, 4, 4, 128, 300, 17), (2, 3, 0, 64, 8, 0), (2, 3, 1, 128, 1, 5)],
                         ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
@pytest.mark.parametrize("kw", [{}, {"softmax_scale": 0.5, "eps": 0.25}, {"side": True}], ids=["plain", "options", "stream"])
def test_same_step_either_way(case, dtype, kw):
    B, H, H0, d, w, t = case
    kw = dict(kw)
    side = torch.cuda.Stream() if kw.pop("side", False) else None
    args = [_step(B, H, H0, d, w, dtype, "cuda") for _ in range(2)]
    torch.cuda.synchronize()
    if side is not None:
        kw["stream"] = side.cuda_stream
    full = (w, H0, t, 0, kw.get("softmax_scale", 1.0), kw.get("eps", 0.0), kw.get("stream"))
    assert gb._decode_call()(gb.lib().decode_address, *args[0], *full) == gb.GF_OK
    gb.gformer_attn_decode(*args[1], np.int64(w), H0, t, **kw)   # not a plain int: the binding's own code
    torch.cuda.synchronize()
    for a, b in zip(*args):
        assert a is None or torch.equal(a, b)


@pytest.mark.gpu
def test_refusals():
    q, k, v, out, kc, vc, st = _step(2, 3, 1, 64, 8, torch.bfloat16, "cuda")
    run = gb.gformer_attn_decode
    for bad in ((q, k[:1], v, out, kc, vc, st), (q, k, v, out, None, vc, st), (q, k, v, out, kc, vc, st.bfloat16()),
                (q, k, v, out, kc[:, :, :4], vc, st), (q.half(), k, v, out, kc, vc, st),
                (q.transpose(0, 1), k, v, out, kc, vc, st), (q.float(), k, v, out, kc, vc, st)):
        with pytest.raises(ValueError):
            run(*bad, 8, 1, 3)
    for kw in ({"t": -1}, {"t": 3, "phi": 9}, {"t": 3, "eps": -1.0}):
        with pytest.raises(gb.GformerError):
            run(q, k, v, out, kc, vc, st, 8, 1, **kw)
    with pytest.raises(gb.GformerError):
        run(q, k, v, q, kc, vc, st, 8, 1, 3)
    with torch.inference_mode():
        run(*(x.clone() for x in (q, k, v, out, kc, vc, st)), 8, 1, 3)
    for i in range(7):   # nested tensors are strided, contiguous, have storage, and no sizes
        args = [q, k, v, out, kc, vc, st]
        args[i] = torch.nested.nested_tensor([x.clone() for x in args[i]])
        with pytest.raises((RuntimeError, ValueError)):
            run(*args, 8, 1, 3)
    native = gb._decode_call()   # vmap's wrappers have no memory of their own to hand over
    def wrapped(x):
        assert native(gb.lib().decode_address, x, k, v, out, kc, vc, st, 8, 1, 3, 0, 1.0, 0.0, None) is None
        with pytest.raises(RuntimeError):
            run(x, k, v, out, kc, vc, st, 8, 1, 3)
        return x
    torch.func.vmap(wrapped)(torch.stack([q, q]))
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_parameters_and_views_are_plain():
    """What is a dense tensor by another name takes the same way, with the same result."""
    q, k, v, out, kc, vc, st = _step(2, 3, 1, 64, 8, torch.bfloat16, "cuda")
    again = [x.clone() for x in (out, kc, vc, st)]
    gb.gformer_attn_decode(q, k, v, out, kc, vc, st, 8, 1, 3)
    wide = torch.stack([k, v])   # a contiguous part of a larger buffer
    gb.gformer_attn_decode(torch.nn.Parameter(q), wide[0], wide[1], *again, 8, 1, 3)
    torch.cuda.synchronize()
    for a, b in zip((out, kc, vc, st), again):
        assert torch.equal(a, b)
