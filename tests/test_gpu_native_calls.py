"""The calls that the extension makes, and those it leaves to the Python code: the same results and the same refusals."""
import threading

import pytest

from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _layer(kind, dtype=B.BF16, shape=(2, 20, 23), c=32):
    torch = G.torch_mod()
    n, h, w = shape
    groups = {"conv": 1, "gconv": 4, "dwconv": c}[kind]
    x = G.to_dev(synth.activations((n, h, w, c), dtype, 31, 1), dtype)
    wt = synth.he_weights(c, 3, 3, c // groups, dtype, 31, 2)
    wt = G.to_dev(wt[..., 0] if kind == "dwconv" else wt, dtype)
    bias = torch.from_numpy(synth.bias(c, 31, 3)).to(G.dev())
    mask = G.mask_dev(synth.mask_objects(n, h, w, 0.45, 31, 4))
    desc = B.conv_desc(n, h, w, c, c, in_dtype=dtype, flags=B.RELU)
    call = {"conv": B.focused_conv2d, "dwconv": B.focused_dwconv2d,
            "gconv": lambda d, *a, **k: B.focused_gconv2d(d, groups, *a, **k)}[kind]
    return call, desc, x, wt, bias, mask


@pytest.mark.parametrize("kind,dtype", [("conv", B.BF16), ("conv", B.F32), ("conv", B.FP8), ("gconv", B.F16), ("dwconv", B.BF16)])
def test_the_extension_and_the_python_code_make_the_same_call(kind, dtype, monkeypatch):
    torch = G.torch_mod()
    call, desc, x, wt, bias, mask = _layer(kind, dtype)
    for kw in ({}, dict(mask_in=mask), dict(mask_in=mask, bias=bias), dict(bias=bias)):
        got = call(desc, x, wt, **kw)
        mine = torch.full_like(got.view(torch.uint8), 7).view(got.dtype)
        assert call(desc, x, wt, out=mine, **kw) is mine
        monkeypatch.setattr(B, "_call", lambda *a: None)
        want = call(desc, x, wt, **kw)
        monkeypatch.undo()
        assert got.dtype == want.dtype and got.shape == want.shape and got.device == want.device and not got.requires_grad
        assert torch.equal(got.view(torch.uint8), want.view(torch.uint8)) and torch.equal(mine.view(torch.uint8), want.view(torch.uint8))


def test_calls_that_are_not_plain_are_made_as_before():
    torch = G.torch_mod()
    call, desc, x, wt, bias, mask = _layer("conv")
    want = call(desc, x, wt, bias, mask_in=mask)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    on_side = call(desc, x, wt, bias, mask_in=mask, stream=side)
    side.synchronize()
    assert torch.equal(on_side, want)
    with torch.cuda.stream(side):                           # (the current stream, with a workspace of its own)
        again = call(desc, x, wt, bias, mask_in=mask)
    side.synchronize()
    assert torch.equal(again, want)
    assert torch.equal(call(desc, x, torch.nn.Parameter(wt, requires_grad=False), bias, mask_in=mask), want)
    got = []
    worker = threading.Thread(target=lambda: got.append(call(desc, x, wt, bias, mask_in=mask)))
    worker.start()
    worker.join()
    torch.cuda.synchronize()
    assert torch.equal(got[0], want)
    idx, count = B.active_index_compact(mask)
    prepared = B.PreparedConv(desc, x, wt, bias, mask_in=mask, mask_out=mask, idx=idx, count=count)
    assert torch.equal(prepared(), want) and torch.equal(prepared(torch.cuda.current_stream()), want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = call(desc, x, wt, bias, mask_in=mask)
    for _ in range(3):
        captured.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(captured, want)


def test_refusals():
    torch = G.torch_mod()
    call, desc, x, wt, bias, mask = _layer("conv")
    for bad in (x.cpu(), x.transpose(1, 2)):
        with pytest.raises(ValueError):
            call(desc, bad, wt)
    with pytest.raises(B.FcError) as e:
        call(desc, x, wt, out=x)                            # the output over the input
    assert e.value.status == -1
    with pytest.raises(B.FcError) as e:
        call(desc, x, wt, mask_in=mask, workspace=torch.empty((16,), dtype=torch.uint8, device=G.dev()))
    assert e.value.status == -5
    with pytest.raises(B.FcError) as e:
        call(B.conv_desc(2, 20, 23, 0, 32), x, wt)
    assert e.value.status == -2
    for groups in (0, -1, 5):
        with pytest.raises(B.FcError):
            B.focused_gconv2d(desc, groups, x, wt)
    with pytest.raises(AttributeError):
        call(desc, None, wt)
