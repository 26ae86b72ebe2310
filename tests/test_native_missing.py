"""The C library without the Python extension: all calls are made by the Python code, and the library builds where there is no PyTorch."""
import ctypes
import os
import sys

import pytest

from paper_2207_10741_amd import binding as B, build, synth


@pytest.fixture
def no_extension(monkeypatch):
    monkeypatch.setattr(B, "NATIVE_PATH", os.path.join(os.path.dirname(B.NATIVE_PATH), "not_built.so"))
    monkeypatch.setattr(B, "_native_module", None)
    monkeypatch.setattr(B, "_call", B._first_call)


def test_plain_and_prepared_calls_without_the_extension(no_extension):
    assert B._call(None, 0, *[None] * 9) is None
    desc = B.conv_desc(1, 4, 4, 8, 8)
    run = B._prepared(B._CONV, (ctypes.addressof(desc), *[None] * 9, 0))
    assert run(0) == -1                                     # FC_ERR_NULL: no tensors
    assert B._prepared(B._DWCONV, (ctypes.addressof(desc), *[None] * 5))(0) == -1
    steps = B._steps_array([((3, 3), (1, 1), (1, 1), (1, 1))])
    assert B._prepared(B._PYRAMID, (None, 1, 4, 4, 1, ctypes.addressof(steps), None, None, None, None, 0))(0) == -1
    assert B._prepared(B._PYRAMID_PACKED, (None, 0, 1, 4, 4, 1, ctypes.addressof(steps), None, None, None, None, 0))(0) == -1
    with pytest.raises(ValueError):
        B._prepared(B._CONV, (ctypes.addressof(desc),))


def test_the_library_is_built_without_pytorch(monkeypatch):
    assert build._native_command("out.so")
    monkeypatch.setitem(sys.modules, "torch", None)
    assert build._native_command("out.so") is None


@pytest.mark.gpu
def test_results_without_the_extension(no_extension):
    from tests import gpu_util as G
    torch = G.torch_mod()
    n, h, w, c = 2, 20, 23, 32
    x = G.to_dev(synth.activations((n, h, w, c), B.BF16, 31, 1), B.BF16)
    wt = G.to_dev(synth.he_weights(c, 3, 3, c, B.BF16, 31, 2), B.BF16)
    dw = G.to_dev(synth.he_weights(c, 3, 3, 1, B.BF16, 31, 3)[..., 0], B.BF16)
    mask = G.mask_dev(synth.mask_objects(n, h, w, 0.45, 31, 4))
    desc = B.conv_desc(n, h, w, c, c, in_dtype=B.BF16, flags=B.RELU)
    steps = [((3, 3), (1, 1), (1, 1), (1, 1)), ((3, 3), (2, 2), (1, 1), (1, 1))]

    def everything():
        prepared = B.PreparedConv(desc, x, wt, mask_in=mask, workspace=torch.empty((B.workspace_bytes(desc),), dtype=torch.uint8, device=G.dev()))
        levels = [[t.clone() for t in level] for packed in (False, True) for level in B.PreparedPyramid(mask, steps, packed=packed)()]
        lists = [t for m, idx, count in levels for t in (m, idx[:int(count)], count)]
        return [B.focused_conv2d(desc, x, wt, mask_in=mask), B.focused_dwconv2d(desc, x, dw, mask_in=mask), prepared().clone(),
                B.PreparedDwConv(desc, x, dw, mask_in=mask)().clone(), *lists]

    without = everything()
    B.NATIVE_PATH, B._call = os.path.join(os.path.dirname(B.__file__), "_native.so"), B._first_call
    assert B._native() is not None
    assert len(without) == 16
    for a, b in zip(without, everything()):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
