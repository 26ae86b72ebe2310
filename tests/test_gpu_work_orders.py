"""Orders in which workgroups take their work: every output is made once, whatever the number of units, for eighths and for shorter runs."""
import pytest

from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G, test_gpu_grouped as GR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layer", [
    # n, h, w, ci, co, k, s, p, groups; blocks of 64 channels, spans of 64 positions
    (1, 5, 5, 64, 64, 3, 1, 1, 16), (1, 33, 37, 64, 64, 3, 1, 1, 16),                       # one block; one span, 20
    (3, 17, 19, 128, 128, 3, 1, 1, 32), (7, 30, 31, 192, 192, 3, 1, 1, 48),                 # two and three, fewer images than XCDs
    (8, 13, 15, 128, 128, 3, 1, 1, 32), (9, 11, 7, 576, 576, 3, 1, 1, 36),                  # as many, and more, 9 blocks
    (1, 8, 9, 512, 512, 3, 1, 1, 32), (2, 27, 23, 512, 512, 3, 1, 1, 32), (1, 7, 7, 1024, 1024, 3, 1, 1, 32)])  # 8 and 16 blocks
@pytest.mark.parametrize("mask_kind,irr", [("objects", 0.48), ("bernoulli", 0.5), ("objects", 1.0), (None, 0.0)])
def test_grouped_windows(layer, mask_kind, irr):
    out, want, keep = GR._run(layer, synth.BF16, B.F32, mask_kind=mask_kind, irr=irr)
    assert G.rel_err(G.to_f64(out), want, keep) <= GR.TOL_F32_OUT
    assert not out.cpu().numpy()[~keep].any()
