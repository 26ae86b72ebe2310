"""1x1 layers that are given masks and no list, on the kernel that labels its rows itself: one, two and four splits, sizes around the
rule for them, rows, channels and stages off the tiles, against the oracle; values that are not finite lie under the irrelevant pixels."""
import numpy as np
import pytest

from oracle import fc_oracle as O
from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

LAYERS = [
    # n, h, w, ci, co, dtype, stride, pad
    (1, 1, 1, 16, 8, synth.BF16, (1, 1), (0, 0)),
    (2, 5, 7, 40, 24, synth.F16, (1, 1), (0, 0)),         # one stage that is not full
    (1, 33, 31, 64, 40, synth.BF16, (2, 1), (0, 0)),
    (1, 9, 11, 72, 72, synth.F16, (1, 2), (2, 1)),        # positions outside the image, a second stage of eight channels
    (2, 17, 16, 256, 64, synth.BF16, (1, 1), (0, 0)),
    (1, 14, 15, 328, 48, synth.BF16, (2, 2), (1, 1)),     # six stages
    (3, 7, 7, 2048, 136, synth.F16, (1, 1), (0, 0)),      # four
    (1, 13, 9, 1000, 160, synth.BF16, (1, 1), (0, 0)),    # two, of sixteen stages, the last not full
    (1, 61, 47, 512, 200, synth.BF16, (1, 1), (0, 0)),    # 630 tiles of eight
    (1, 64, 64, 128, 288, synth.BF16, (1, 1), (0, 0)),    # 1 152 tiles, the last that two stages may have
    (1, 64, 64, 128, 296, synth.BF16, (1, 1), (0, 0)),    # one step past it, where a launch makes the list
]


@pytest.mark.parametrize("how", ["mask", "labels", "chained"])
@pytest.mark.parametrize("kind", ["objects", "bernoulli", "all", "none"])
@pytest.mark.parametrize("packed", [0, B.PACKED_MASKS])
@pytest.mark.parametrize("layer", LAYERS)
def test_small_1x1(layer, packed, kind, how):
    torch = G.torch_mod()
    n, h, w, ci, co, dtype, s, p = layer
    geo = ((1, 1), s, p, (1, 1))
    x, wt, bias = synth.activations((n, h, w, ci), dtype, 47, 1), synth.he_weights(co, 1, 1, ci, dtype, 47, 2), synth.bias(co, 47, 3)
    if kind in ("all", "none"):
        mask = np.full((n, h, w), kind == "all", np.uint8)
    else:
        mask = (synth.mask_objects if kind == "objects" else synth.mask_bernoulli)(n, h, w, 0.48, 47, 4)
    xd = G.to_dev(x, dtype).clone()
    xd[torch.from_numpy(mask == 0).to(G.dev())] = float("nan")
    wd, bd = G.to_dev(wt, dtype), torch.from_numpy(bias).to(G.dev())
    flags = B.RELU | packed | (B.SKIP_ZERO_FILL if how == "chained" else 0)
    desc = B.conv_desc(n, h, w, ci, co, *geo, dtype, B.F32, flags)
    ho, wo = B.out_dims(desc)
    # every position's sum, with what the mask drops taken as zero; the labels decide which of them are written
    want = O.focused_conv2d(O.ConvShape(n, h, w, ci, co, 1, 1, s, p, relu=True), np.where((mask != 0)[..., None], x, x.dtype.type(0)), wt, bias=bias,
                            mask_in=None, dtype=dtype).reshape(-1, co)
    keep = O.mask_downsample(mask, 1, 1, s, p) != 0
    if how == "labels":                                   # the caller's own, fewer than the mask's
        keep &= synth.mask_bernoulli(n, ho, wo, 0.4, 47, 5) != 0
    form = (lambda m: B.mask_pack(G.mask_dev(m))) if packed else G.mask_dev
    kw = dict(mask_in=form(mask))
    if how == "labels":
        kw["mask_out"] = form(keep.reshape(n, ho, wo).astype(np.uint8))
    keep = keep.reshape(-1)
    out = torch.full((n, ho, wo, co), 7.0, device=G.dev())
    B.focused_conv2d(desc, xd, wd, bd, out=out, **kw)
    got = out.reshape(-1, co).cpu().numpy().astype(np.float64)
    if keep.any():
        rms = max(float(np.sqrt(np.mean(np.square(want[keep])))), 1e-3)
        assert np.abs(got[keep] - want[keep]).max() / rms <= 1e-4    # fp32 sums in another order (the parity tests' bound)
    assert np.all(got[~keep] == (7.0 if how == "chained" else 0.0))
    # 16-bit outputs are the rounding of these
    out16 = torch.full(out.shape, 7.0, device=G.dev()).to(B.torch_dtype(dtype))
    B.focused_conv2d(B.conv_desc(n, h, w, ci, co, *geo, dtype, None, flags), xd, wd, bd, out=out16, **kw)
    assert torch.equal(out16, out.to(out16.dtype))
    # and with the list made beforehand, on other kernels, the same sums bit for bit
    if how != "labels":
        m_out = B.mask_downsample(G.mask_dev(mask), *geo)
        idx, count = B.active_index_compact(m_out)
        listed = torch.full(out.shape, 7.0, device=G.dev())
        room = torch.empty((B.workspace_bytes(desc),), dtype=torch.uint8, device=G.dev())   # (without it nothing is split)
        B.focused_conv2d(desc, xd, wd, bd, out=listed, mask_out=B.mask_pack(m_out) if packed else m_out, idx=idx, count=count, workspace=room, **kw)
        assert torch.equal(listed, out)
