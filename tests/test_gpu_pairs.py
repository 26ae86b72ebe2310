"""Two 1x1 layers in one launch: the bits of the two calls one after the other (which the parity tests hold to the oracle), and
a middle that is never written."""
import ctypes

import numpy as np
import pytest

from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

CANARY = 0x5a


def _run(shape, channels, dtype, mask, relu=(True, True), compact_in=False, compact_mid=False, compact_out=False, skip=True,
         bias=(True, True), seed=5, x_over_out=False):
    """(outputs of the two calls one by one, outputs as a pair, was the middle of the pair left alone?)"""
    torch = G.torch_mod()
    n, h, w = shape
    c0, c1, c2 = channels
    xt = G.to_dev(synth.activations((n, h, w, c0), dtype, seed, 1), dtype)
    ws = [G.to_dev(synth.he_weights(co, 1, 1, ci, dtype, seed, k), dtype) for k, (ci, co) in enumerate(((c0, c1), (c1, c2)))]
    bs = [torch.from_numpy(synth.bias(c, seed, 7 + k)).to(G.dev()) if b else None for k, (c, b) in enumerate(zip((c1, c2), bias))]
    m = idx = count = None
    if mask is not None:
        m = G.mask_dev(mask)
        idx, count = B.active_index_compact(m)
    flags = [B.RELU * relu[0] | B.COMPACT_IN * compact_in | B.COMPACT_OUT * compact_mid | B.SKIP_ZERO_FILL,
             B.RELU * relu[1] | B.COMPACT_IN * compact_mid | B.COMPACT_OUT * compact_out | B.SKIP_ZERO_FILL * skip]
    calls = (B.Call * 2)()
    for k, (ci, co) in enumerate(((c0, c1), (c1, c2))):
        d = B.conv_desc(n, h, w, ci, co, (1, 1), (1, 1), (0, 0), (1, 1), dtype, dtype, flags[k])
        masked = (1, 2, 3, 4) if mask is not None else (-1, -1, -1, -1)
        calls[k] = B.Call(d, B.CALL_CONV, 0 if k == 0 else 9, masked[0], 5 + 2 * k, -1 if bs[k] is None else 6 + 2 * k, masked[1], masked[2],
                          masked[3], 9 + k)
    item = B.torch_dtype(dtype).itemsize
    got, left = [], None
    for unseen in (None, bytes([1, 0])):
        x = xt.clone()
        mid = torch.full((n * h * w * c1 * item,), CANARY, dtype=torch.uint8, device=G.dev())
        out = torch.full((n * h * w * c2 * item,), CANARY, dtype=torch.uint8, device=G.dev())
        to = x.data_ptr() if x_over_out else out.data_ptr()
        tensors = [x, m, m, idx, count, ws[0], bs[0], ws[1], bs[1], mid]
        slots = (ctypes.c_void_p * 11)(*[None if t is None else t.data_ptr() for t in tensors], to)
        B.run_calls(calls, slots, None, unseen=unseen)
        torch.cuda.synchronize()
        got.append((x.view(torch.uint8) if x_over_out else out).cpu())
        if unseen:
            left = bool((mid == CANARY).all())
    return got[0], got[1], left


PAIRS = [((64, 256, 64), B.BF16), ((64, 192, 40), B.F16), ((8, 72, 8), B.BF16), ((64, 256, 64), B.FP8), ((128, 256, 128), B.FP8),
         ((48, 80, 112), B.FP8), ((32, 16, 96), B.BF16), ((96, 24, 144), B.F16), ((192, 32, 192), B.BF16), ((192, 64, 384), B.BF16),
         ((384, 64, 384), B.F16), ((200, 40, 72), B.BF16)]
STREAMED = [((128, 512, 128), B.BF16), ((128, 512, 128), B.FP8), ((128, 320, 72), B.F16), ((128, 1152, 112), B.FP8)]      # (more weights than LDS holds)


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 5, 13), (2, 61, 83), (6, 130, 131)])
@pytest.mark.parametrize("channels,dtype", PAIRS)
def test_a_pair_makes_the_bits_of_its_layers(channels, dtype, shape):
    """One row, less than a unit, a few units a CU, several units a wave; all rows and the kept ones."""
    n, h, w = shape
    for mask in (None, synth.mask_objects(n, h, w, 0.45, 11, 3)):
        one, both, left = _run(shape, channels, dtype, mask)
        assert left and (one == both).all(), (mask is None, int((one != both).sum()))


@pytest.mark.parametrize("channels,dtype", [PAIRS[0], PAIRS[3], PAIRS[8], PAIRS[9]])
def test_pairs_of_rows_in_list_order(channels, dtype):
    shape = (3, 33, 47)
    mask = synth.mask_objects(*shape, 0.5, 4, 9)
    for cin in (False, True):
        for cmid in (False, True):
            for cout in (False, True):
                one, both, left = _run(shape, channels, dtype, mask, compact_in=cin, compact_mid=cmid, compact_out=cout)
                assert left and (one == both).all(), (cin, cmid, cout)


@pytest.mark.parametrize("channels,dtype", [PAIRS[0], PAIRS[3], PAIRS[9]])
def test_pairs_without_relu_or_bias_and_masks_that_keep_nothing(channels, dtype):
    shape = (2, 20, 31)
    mask = synth.mask_objects(*shape, 0.5, 4, 2)
    for relu in ((False, True), (True, False), (False, False)):
        one, both, left = _run(shape, channels, dtype, mask, relu=relu, bias=(relu[1], relu[0]))
        assert left and (one == both).all(), relu
    one, both, left = _run(shape, channels, dtype, mask * 0)
    assert left and (one == CANARY).all() and (both == CANARY).all()


@pytest.mark.parametrize("channels,dtype", STREAMED)
def test_pairs_whose_weights_pass_through_lds(channels, dtype):
    """No rows, one, a unit and one more, fewer units than workgroups and more, some in a second pass; rows in list order on either side."""
    n, h, w = shape = (1, 150, 161)
    for kept in (0, 1, 32, 33, 1000, 20000, n * h * w):
        mask = np.zeros(n * h * w, np.uint8)
        mask[np.random.default_rng(kept).permutation(n * h * w)[:kept]] = 1
        one, both, left = _run(shape, channels, dtype, mask.reshape(shape), compact_in=kept == 33, compact_out=kept in (33, 1000))
        assert left and (one == both).all(), kept
    for relu in ((False, True), (True, False)):
        one, both, left = _run((7, 120, 121), channels, dtype, None, relu=relu, bias=relu)
        assert left and (one == both).all(), relu


def test_layers_that_cannot_run_as_one_run_one_by_one():
    shape = (1, 30, 40)
    mask = synth.mask_objects(*shape, 0.5, 4, 2)
    # the second clears irrelevant rows; weights that do not fit, or are too many for the rows; an output over the input
    for channels, over in (((64, 256, 64), dict(skip=False)), ((256, 1024, 256), {}), ((128, 512, 128), {}), ((64, 256, 64), dict(x_over_out=True))):
        one, both, left = _run(shape, channels, B.BF16, mask, **over)
        assert not left and (one == both).all(), (channels, over)
