"""Split reductions whose units are kept to one a CU, and those beside them that are not: against the oracle, the same bits whether the list is
brought or made inside the call."""
import numpy as np
import pytest

from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G, test_gpu_parity as P
from tests.test_gpu_fp8 import TOL_FP8

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layer,dtype", [
    # n, h, w, ci, co, k, s, p, d
    ((4, 15, 19, 488, 248, 3, 1, 1, 1), synth.F16),     # 128-row tiles
    ((2, 14, 14, 512, 512, 3, 1, 1, 1), synth.BF16),    # 64-row tiles, too many waves for the small-layer kernel
    ((1, 14, 14, 512, 512, 3, 1, 1, 1), synth.BF16),    # few enough: that kernel's splits
    ((2, 31, 40, 512, 64, 3, 1, 1, 1), synth.BF16),     # 72 stages on tiles that one unit a CU leaves more than 24
    ((1, 23, 21, 1024, 192, 1, 1, 0, 1), synth.F16),    # 1x1, 64-row tiles
    ((2, 32, 45, 208, 64, 5, 2, 2, 1), synth.FP8),
    ((2, 24, 30, 384, 128, 3, 1, 1, 1), synth.FP8),     # E4M3: 64-row tiles of their own
])
@pytest.mark.parametrize("mask_kind,irr", [("objects", 0.48), ("objects", 0.05), (None, 0.0)])
def test_split_units(layer, dtype, mask_kind, irr):
    torch = G.torch_mod()
    out, want, keep = P._run_layer(*layer, dtype, mask_kind=mask_kind, irr=irr, seed=261)
    got = G.to_f64(out)
    rms = float(np.sqrt(np.mean(np.square(want[keep]))))
    assert float(np.abs(got[keep] - want[keep]).max()) / rms <= (TOL_FP8 if dtype == synth.FP8 else P.TOL_F32_OUT)
    assert not got[~keep].any()
    if mask_kind:
        again, _, _ = P._run_layer(*layer, dtype, mask_kind=mask_kind, irr=irr, seed=261, precomputed=True)
        assert torch.equal(out, again)
    else:                                               # split only where there is room
        x, wt = (G.to_dev(f, dtype) for f in (synth.activations((layer[0], *layer[1:4]), dtype, 261, 1),
                                              synth.he_weights(layer[4], layer[5], layer[5], layer[3], dtype, 261, 2)))
        desc = B.conv_desc(*layer[:5], (layer[5],) * 2, (layer[6],) * 2, (layer[7],) * 2, (1, 1), dtype, B.F32, B.RELU)
        bias = torch.from_numpy(synth.bias(layer[4], 261, 3)).to(G.dev())
        room = torch.empty((B.workspace_bytes(desc),), dtype=torch.uint8, device=G.dev())
        split = G.to_f64(B.focused_conv2d(desc, x, wt, bias, workspace=room))
        assert float(np.abs(split - want).max()) / rms <= (TOL_FP8 if dtype == synth.FP8 else P.TOL_F32_OUT)
