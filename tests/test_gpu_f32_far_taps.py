"""fp32 3x3 layers whose taps lie a quarter of a gigabyte apart: the pieces past the last channel are zeros, whatever the first pixel holds."""
import numpy as np
import pytest

from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c,w,dil", [(197, 13102, 13), (67, 5163, 97), (197, 13102, 12)])
def test_the_first_pixel_reaches_its_own_outputs_only(c, w, dil):
    """Offsets of 2^28 bytes and some hundred more, the first two of them; one output row."""
    torch = G.torch_mod()
    h, co = 2 * dil + 1, 8
    gen = torch.Generator(device=G.dev()).manual_seed(3)
    x = torch.randn((1, h, w, c), generator=gen, device=G.dev())
    x[0, 0, 0] = 0
    wt = torch.from_numpy(synth.he_weights(co, 3, 3, c, B.F32, 31, 2)).to(G.dev())
    desc = B.conv_desc(1, h, w, c, co, pad=(0, 0), dil=(dil, 1), in_dtype=B.F32)
    got = G.to_f64(B.focused_conv2d(desc, x, wt))
    want = torch.nn.functional.conv2d(x[:, ::dil].cpu().double().permute(0, 3, 1, 2), wt.cpu().double().permute(0, 3, 1, 2)).permute(0, 2, 3, 1).numpy()
    assert G.rel_err(got, want, np.ones(want.shape[:3], bool)) <= 1e-5
    for bad in (float("nan"), float("inf")):
        x[0, 0, 0] = bad
        again = G.to_f64(B.focused_conv2d(desc, x, wt))
        assert (again[:, :, 1:] == got[:, :, 1:]).all()
