"""fp32 3x3 layers of whole 32-channel chunks whose reduction four waves share: rows and channels past the last tile, stages that fill the
ring once and several times, every way a call says what is kept, against the oracle."""
import numpy as np
import pytest

from oracle import fc_oracle as O
from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

LAYERS = [
    # n, h, w, ci, co, stride, pad, vertical dilation
    (2, 60, 80, 64, 64, (1, 1), (1, 1), 1),       # work for two workgroups a CU: three rounds in LDS
    (1, 14, 20, 32, 32, (1, 1), (1, 1), 1),       # nine stages
    (1, 1, 4, 32, 4, (1, 1), (1, 1), 1),          # four mask bytes
    (3, 37, 5, 96, 35, (1, 1), (0, 2), 2),        # channels by threes, wide padding, dilation
    (1, 31, 33, 224, 40, (2, 1), (3, 3), 1),      # 63 stages, taps wholly outside the image
    (8, 30, 40, 64, 66, (2, 2), (1, 1), 1),
    (4, 67, 90, 32, 128, (1, 1), (1, 1), 1),      # three workgroups a CU
]


@pytest.mark.parametrize("how", ["dense", "mask", "labels", "list", "chained", "no bias"])
@pytest.mark.parametrize("kind", ["objects", "bernoulli", "all", "none"])
@pytest.mark.parametrize("layer", LAYERS)
def test_f32_rounds(layer, kind, how):
    torch = G.torch_mod()
    n, h, w, ci, co, s, p, dh = layer
    if how == "dense" and kind != "all":
        pytest.skip("no mask: one kind")
    geo = ((3, 3), s, p, (dh, 1))
    x, wt, bias = synth.activations((n, h, w, ci), synth.F32, 43, 1), synth.he_weights(co, 3, 3, ci, synth.F32, 43, 2), synth.bias(co, 43, 3)
    mask = {"all": lambda: np.ones((n, h, w), np.uint8), "none": lambda: np.zeros((n, h, w), np.uint8),
            "objects": lambda: synth.mask_objects(n, h, w, 0.48, 43, 4), "bernoulli": lambda: synth.mask_bernoulli(n, h, w, 0.48, 43, 4)}[kind]()
    mask = mask * np.uint8(200)
    xd = G.to_dev(x, synth.F32)
    kw = {}
    if how != "dense":
        xd = xd.clone()
        xd[torch.from_numpy(mask == 0).to(G.dev())] = float("nan")
        md = G.mask_dev(mask)
        kw = dict(mask_in=md)
        if how in ("labels", "list"):
            kw.update(mask_out=B.mask_downsample(md, *geo))
        if how == "list":
            kw.update(zip(("idx", "count"), B.active_index_compact(kw["mask_out"])))
    bd = None if how == "no bias" else torch.from_numpy(bias).to(G.dev())
    desc = B.conv_desc(n, h, w, ci, co, *geo, B.F32, B.F32, B.RELU | (B.SKIP_ZERO_FILL if how == "chained" else 0))
    ho, wo = B.out_dims(desc)
    out = torch.full((n, ho, wo, co), 7.0, device=G.dev())
    B.focused_conv2d(desc, xd, G.to_dev(wt, synth.F32), bd, out=out, **kw)
    got = out.reshape(-1, co).cpu().numpy().astype(np.float64)
    keep = np.ones(n * ho * wo, bool) if how == "dense" else (O.mask_downsample(mask, 3, 3, s, p, (dh, 1)) != 0).reshape(-1)
    assert np.all(got[~keep] == (7.0 if how == "chained" else 0.0))
    if not keep.any():
        return
    pos = np.sort(np.random.default_rng(43).choice(np.flatnonzero(keep), size=min(500, int(keep.sum())), replace=False))
    want = O.focused_conv2d_at(O.ConvShape(n, h, w, ci, co, 3, 3, s, p, (dh, 1), relu=True), x, wt, pos, bias=None if bd is None else bias,
                               mask_in=None if how == "dense" else mask, dtype=synth.F32)
    # fp32 sums of up to 2 016 products in four parts: 504 roundings of 2^-24 in a row, of which the random walk's share is 1.4e-6 of the
    # sums' size; the largest of thousands lies within five times that
    assert np.abs(got[pos] - want).max() / np.sqrt(np.mean(np.square(want))) <= 1e-5
    assert not np.any(got[keep] == 7.0)


@pytest.mark.parametrize("how", ["mask", "labels", "list"])
@pytest.mark.parametrize("layer", LAYERS)
def test_same_sums_as_the_kernel_for_any_layer(layer, how):
    """Masks of bits send these layers to the kernel that serves every fp32 layer: the same products in the same order, so the same bits."""
    torch = G.torch_mod()
    n, h, w, ci, co, s, p, dh = layer
    geo = ((3, 3), s, p, (dh, 1))
    xd = G.to_dev(synth.activations((n, h, w, ci), synth.F32, 47, 1), synth.F32)
    wd, bd = G.to_dev(synth.he_weights(co, 3, 3, ci, synth.F32, 47, 2), synth.F32), torch.from_numpy(synth.bias(co, 47, 3)).to(G.dev())
    md = G.mask_dev(synth.mask_objects(n, h, w, 0.48, 47, 4))
    m_out = B.mask_downsample(md, *geo)
    idx, count = B.active_index_compact(m_out)
    outs = []
    for flag, form in ((0, lambda m: m), (B.PACKED_MASKS, B.mask_pack)):
        kw = dict(mask_in=form(md))
        if how != "mask":
            kw["mask_out"] = form(m_out)
        if how == "list":
            kw.update(idx=idx, count=count)
        desc = B.conv_desc(n, h, w, ci, co, *geo, B.F32, B.F32, B.RELU | flag)
        outs.append(B.focused_conv2d(desc, xd, wd, bd, **kw))
    assert float(outs[0].abs().max()) > 0 or int(count) == 0
    assert torch.equal(outs[0], outs[1])
