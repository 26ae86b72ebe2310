"""3x3 layers on the kernel for wide tiles (256 x 256 and 384 x 128 outputs a CU; from 1 000 granules of a tile on): against the oracle on sampled positions,
16- and 8-bit outputs against the rounding of the fp32 ones, irrelevant rows zero to the byte, kept rows all written."""
import numpy as np
import pytest

from oracle import fc_oracle as O
from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

LAYERS = [
    # n, h, w, ci, co, dtype, sh, (ph, pw), dh
    (4, 130, 161, 128, 256, synth.BF16, 1, (1, 1), 1),      # 256-channel tiles: 1 309 granules of 64 rows
    (8, 131, 127, 192, 128, synth.F16, 1, (1, 1), 1),       # 128-channel tiles: 1 040 granules of 128 rows, three chunks
    (1, 260, 130, 128, 512, synth.BF16, 1, (1, 1), 1),      # two channel tiles
    (120, 17, 33, 128, 256, synth.BF16, 1, (1, 1), 1),      # short image rows
    (7, 201, 99, 128, 256, synth.BF16, 2, (3, 2), 2),       # vertical stride and dilation, wide padding
    (4, 130, 161, 256, 256, synth.FP8, 1, (1, 1), 1),
    (2, 300, 301, 256, 128, synth.FP8, 1, (0, 0), 1),       # no padding
]


def _mask(kind, n, h, w):
    if kind is None:
        return None
    if kind == "all":
        return np.ones((n, h, w), np.uint8)
    if kind == "sparse":                                     # few rows kept: cleared after the tiles
        return synth.mask_objects(n, h, w, 0.97, 300, 4)
    if kind == "bernoulli":                                  # two slots a row: smaller tiles
        return synth.mask_bernoulli(n, h, w, 0.5, 300, 4)
    if kind == "checker":                                    # three slots a row: the smallest tile
        yy, xx = np.mgrid[0:h, 0:w]
        return np.ascontiguousarray(np.broadcast_to(((yy + xx) % 2).astype(np.uint8), (n, h, w)))
    return synth.mask_objects(n, h, w, 0.48, 300, 4)


@pytest.mark.parametrize("layer", LAYERS)
@pytest.mark.parametrize("kind", ["objects", "bernoulli", "checker", "sparse", "all", None])
def test_wide_tiles(layer, kind):
    torch = G.torch_mod()
    n, h, w, ci, co, dtype, sh, (ph, pw), dh = layer
    x = synth.activations((n, h, w, ci), dtype, 301, 1)
    wt = synth.he_weights(co, 3, 3, ci, dtype, 301, 2)
    bias = synth.bias(co, 301, 3)
    mask = _mask(kind, n, h, w)
    geo = ((3, 3), (sh, 1), (ph, pw), (dh, 1))
    xd, wd, bd = G.to_dev(x, dtype), G.to_dev(wt, dtype), torch.from_numpy(bias).to(G.dev())
    if dtype != synth.FP8 and mask is not None:              # what lies under irrelevant pixels is not looked at
        xd = xd.clone()
        xd[torch.from_numpy(mask == 0).to(G.dev())] = float("nan")
    kw = {}
    if mask is not None:
        md = G.mask_dev(mask)
        m_out = B.mask_downsample(md, *geo)
        idx, count = B.active_index_compact(m_out)
        kw = dict(mask_in=md, mask_out=m_out, idx=idx, count=count)
    outs = {}
    for out_dtype in (B.F32, B.BF16 if dtype == synth.FP8 else dtype, B.FP8):
        desc = B.conv_desc(n, h, w, ci, co, *geo, dtype, out_dtype, B.RELU)
        ho, wo = B.out_dims(desc)
        out = torch.full((n, ho, wo, co), 7.0, dtype=torch.float32, device=G.dev()).to(B.torch_dtype(out_dtype))
        B.focused_conv2d(desc, xd, wd, bd, out=out, **kw)
        outs[out_dtype] = out
        if out_dtype == B.F32 and mask is not None:          # chained: irrelevant rows stay as they were
            desc = B.conv_desc(n, h, w, ci, co, *geo, dtype, out_dtype, B.RELU | B.SKIP_ZERO_FILL)
            chained = torch.full((n, ho, wo, co), 7.0, dtype=torch.float32, device=G.dev())
            B.focused_conv2d(desc, xd, wd, bd, out=chained, **kw)
    f32 = outs[B.F32]
    keep = np.ones((n, ho, wo), bool) if mask is None else O.mask_downsample(mask, 3, 3, (sh, 1), (ph, pw), (dh, 1)) != 0
    kd = torch.from_numpy(keep).to(G.dev())
    assert not bool(f32[~kd].view(torch.int32).any())
    assert not bool((f32[kd] == 7.0).all(dim=-1).any())
    if mask is not None:
        assert torch.equal(chained[kd], f32[kd]) and bool((chained[~kd] == 7.0).all())
    for out_dtype, out in outs.items():
        if out_dtype == B.FP8:
            assert torch.equal(out.float(), f32.clamp(max=448.0).to(out.dtype).float())
        elif out_dtype != B.F32:
            assert torch.equal(out, f32.to(out.dtype))
    kept = np.flatnonzero(keep.reshape(-1))
    pos = np.sort(np.random.default_rng(301).choice(kept, size=min(600, kept.size), replace=False))
    shape = O.ConvShape(n, h, w, ci, co, 3, 3, (sh, 1), (ph, pw), (dh, 1), relu=True)
    want = O.focused_conv2d_at(shape, x, wt, pos, bias=bias, mask_in=mask, dtype=dtype)
    got = f32.reshape(-1, co)[torch.from_numpy(pos).to(G.dev())].cpu().numpy().astype(np.float64)
    from tests.test_gpu_fp8 import TOL_FP8
    rms = float(np.sqrt(np.mean(np.square(want))))
    assert float(np.abs(got - want).max()) / rms <= (TOL_FP8 if dtype == synth.FP8 else 1e-4)
