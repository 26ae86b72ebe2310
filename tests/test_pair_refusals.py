"""What fc_run_calls_unseen refuses: the same as its calls one by one.  Addresses are nobody's memory: every refusal comes before a launch."""
import ctypes

import pytest

from paper_2207_10741_amd import binding as B

ADDR = 0x1000000


def _rc(desc1, desc2, masked, unseen=bytes([1, 0]), labels=None):
    slots = (ctypes.c_void_p * 9)(*[ADDR * (k + 1) for k in range(9)])
    mask, idx, count = (5, 6, 7) if masked else (-1, -1, -1)
    calls = (B.Call * 2)(B.Call(desc1, B.CALL_CONV, 0, mask, 1, -1, mask if labels is None else labels, idx, count, 2),
                         B.Call(desc2, B.CALL_CONV, 2, mask, 3, -1, mask, idx, count, 4))
    return B.lib().fc_run_calls_unseen(calls, 2, unseen, slots, 9, None, 0, None)


@pytest.mark.parametrize("h,w", [(16385, 1), (1, 16385), (20000, 3)])
def test_images_past_the_matrix_cores_limits(h, w):
    """E4M3 layers and rows in list order exist on the matrix cores only."""
    one = [B.conv_desc(1, h, w, ci, co, (1, 1), (1, 1), (0, 0), (1, 1), B.FP8, B.FP8) for ci, co in ((64, 256), (256, 64))]
    assert _rc(*one, False) == _rc(*one, False, unseen=None) == -3
    rows = [B.conv_desc(1, h, w, ci, co, (1, 1), (1, 1), (0, 0), (1, 1), B.BF16, B.BF16, B.SKIP_ZERO_FILL | f)
            for ci, co, f in ((64, 256, B.COMPACT_OUT), (256, 64, B.COMPACT_IN))]
    assert _rc(*rows, True) == _rc(*rows, True, unseen=None) == -3


def test_labels_without_a_mask():
    one = [B.conv_desc(1, 20, 30, ci, co, (1, 1), (1, 1), (0, 0), (1, 1), B.BF16) for ci, co in ((64, 256), (256, 64))]
    assert _rc(*one, False, labels=5) == _rc(*one, False, unseen=None, labels=5) == -1


@pytest.mark.gpu
def test_images_past_the_matrix_cores_limits_run_one_by_one():
    from tests import test_gpu_pairs as P
    for channels in ((64, 256, 64), (32, 16, 96)):
        one, both, left = P._run((1, 1, 16385), channels, B.BF16, None)
        assert not left and (one == both).all()
