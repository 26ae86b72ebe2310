"""The tiled kernels deal their tiles out by groups of channel tiles: every kept row and channel is written once, whatever
the number of channel tiles, the group and the remainders, against the oracle on sampled positions."""
import numpy as np
import pytest

from oracle import fc_oracle as O
from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

LAYERS = [
    # n, h, w, ci, co, k, stride
    (1, 61, 53, 64, 1024, 1, 1),      # 16 channel tiles in groups of 8
    (1, 61, 53, 72, 192, 1, 1),       # 3 channel tiles, one by one
    (4, 121, 99, 64, 256, 3, 2),      # 4 in one group
    (3, 45, 41, 136, 384, 3, 1),      # 6 in pairs, the last pixel tile short
    (2, 97, 65, 64, 512, 3, 2),       # 8 in groups of 4
    (9, 73, 119, 256, 256, 3, 2),     # a tile per CU, its size by the kept count
    (32, 15, 20, 1024, 512, 1, 1),    # the same, 1x1
]


@pytest.mark.parametrize("irrelevant", [0.48, 0.1, 0.95, None])
@pytest.mark.parametrize("layer", LAYERS)
def test_every_row_and_channel_once(layer, irrelevant):
    torch = G.torch_mod()
    n, h, w, ci, co, k, s = layer
    geo = ((k, k), (s, s), (k // 2, k // 2), (1, 1))
    x, wt, bias = synth.activations((n, h, w, ci), synth.BF16, 77, 1), synth.he_weights(co, k, k, ci, synth.BF16, 77, 2), synth.bias(co, 77, 3)
    mask = None if irrelevant is None else synth.mask_objects(n, h, w, irrelevant, 77, 4)
    kw = {}
    if mask is not None:
        md = G.mask_dev(mask)
        m_out = B.mask_downsample(md, *geo)
        idx, count = B.active_index_compact(m_out)
        kw = dict(mask_in=md, mask_out=m_out, idx=idx, count=count)
    desc = B.conv_desc(n, h, w, ci, co, *geo, B.BF16, B.F32, B.RELU)
    ho, wo = B.out_dims(desc)
    out = torch.full((n, ho, wo, co), 7.0, device=G.dev())
    B.focused_conv2d(desc, G.to_dev(x, synth.BF16), G.to_dev(wt, synth.BF16), torch.from_numpy(bias).to(G.dev()), out=out, **kw)
    got = out.reshape(-1, co)
    keep = np.ones(n * ho * wo, bool) if mask is None else (O.mask_downsample(mask, k, k, (s, s), (k // 2,) * 2, (1, 1)) != 0).reshape(-1)
    kd = torch.from_numpy(keep).to(G.dev())
    assert not bool(got[~kd].view(torch.int32).any()) and not bool((got[kd] == 7.0).any())
    pos = np.sort(np.random.default_rng(77).choice(np.flatnonzero(keep), size=min(400, int(keep.sum())), replace=False))
    shape = O.ConvShape(n, h, w, ci, co, k, k, (s, s), (k // 2,) * 2, (1, 1), relu=True)
    want = O.focused_conv2d_at(shape, x, wt, pos, bias=bias, mask_in=mask, dtype=synth.BF16)
    err = np.abs(got[torch.from_numpy(pos).to(G.dev())].cpu().numpy().astype(np.float64) - want).max()
    assert err / np.sqrt(np.mean(np.square(want))) <= 1e-4    # sums of fp32 in another order (the parity tests' bound)
