"""3x3 layers of a few hundred row blocks whose waves have at most nine stages: every way a call can say what is kept, at sizes off
the tiles, against the oracle; values that are not finite lie under the irrelevant pixels."""
import numpy as np
import pytest

from oracle import fc_oracle as O
from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

LAYERS = [
    # n, h, w, ci, co, dtype, stride, pad, vertical dilation
    (1, 56, 56, 64, 64, synth.BF16, (1, 1), (1, 1), 1),      # one wave a tile, nine stages
    (1, 1, 4, 64, 8, synth.BF16, (1, 1), (1, 1), 1),         # four mask bytes, one tile with rows and channels past its end
    (2, 37, 5, 64, 72, synth.F16, (1, 1), (0, 2), 2),        # channels past the last tile's quads, wide padding, dilation
    (1, 31, 33, 64, 40, synth.BF16, (2, 1), (3, 3), 1),      # taps wholly outside the image
    (3, 28, 27, 128, 128, synth.F16, (1, 1), (1, 1), 1),     # two waves
    (1, 29, 28, 128, 136, synth.BF16, (2, 2), (1, 1), 1),
    (1, 14, 14, 256, 256, synth.BF16, (1, 1), (1, 1), 1),    # four waves
    (1, 17, 19, 192, 64, synth.F16, (1, 1), (1, 1), 1),      # three waves
    (1, 9, 7, 320, 48, synth.BF16, (1, 1), (1, 1), 1),       # five splits: two workgroups, three waves without one
    (1, 7, 7, 512, 512, synth.BF16, (1, 1), (1, 1), 1),      # nine splits of eight stages
]


@pytest.mark.parametrize("how", ["dense", "mask", "labels", "list", "chained", "compact", "no workspace"])
@pytest.mark.parametrize("kind", ["objects", "bernoulli", "all", "none", "one"])
@pytest.mark.parametrize("layer", LAYERS)
def test_small_layers(layer, kind, how):
    torch = G.torch_mod()
    n, h, w, ci, co, dtype, s, p, dh = layer
    if how == "dense" and kind != "all":
        pytest.skip("no mask: one kind")
    geo = ((3, 3), s, p, (dh, 1))
    x, wt, bias = synth.activations((n, h, w, ci), dtype, 41, 1), synth.he_weights(co, 3, 3, ci, dtype, 41, 2), synth.bias(co, 41, 3)
    if kind == "all":
        mask = np.ones((n, h, w), np.uint8)
    elif kind in ("none", "one"):
        mask = np.zeros((n, h, w), np.uint8)
        if kind == "one":
            mask[-1, -1, -1] = 3                             # any nonzero byte
    else:
        mask = (synth.mask_objects if kind == "objects" else synth.mask_bernoulli)(n, h, w, 0.48, 41, 4)
    xd = G.to_dev(x, dtype)
    if how != "dense":
        xd = xd.clone()
        xd[torch.from_numpy(mask == 0).to(G.dev())] = float("nan")
    wd, bd = G.to_dev(wt, dtype), torch.from_numpy(bias).to(G.dev())
    flags = B.RELU | (B.SKIP_ZERO_FILL if how == "chained" else B.COMPACT_OUT if how == "compact" else 0)
    desc = B.conv_desc(n, h, w, ci, co, *geo, dtype, B.F32, flags)
    ho, wo = B.out_dims(desc)
    want = O.focused_conv2d(O.ConvShape(n, h, w, ci, co, 3, 3, s, p, (dh, 1), relu=True), x, wt, bias=bias,
                            mask_in=None if how == "dense" else mask, dtype=dtype).reshape(-1, co)
    keep = np.ones(n * ho * wo, bool) if how == "dense" else (O.mask_downsample(mask, 3, 3, s, p, (dh, 1)) != 0).reshape(-1)
    kw = {}
    if how != "dense":
        md = G.mask_dev(mask)
        kw = dict(mask_in=md)
        m_out = B.mask_downsample(md, *geo)
        if how == "labels":
            kw.update(mask_out=m_out)
        elif how not in ("mask", "no workspace"):
            idx, count = B.active_index_compact(m_out)
            kw.update(mask_out=m_out, idx=idx[:max(1, int(keep.sum()))].clone(), count=count)   # nothing past the count
    if how == "no workspace":
        kw.update(workspace=None)
    out = torch.full((n * ho * wo, co) if how == "compact" else (n, ho, wo, co), 7.0, device=G.dev())
    B.focused_conv2d(desc, xd, wd, bd, out=out, **kw)
    got = out.reshape(-1, co).cpu().numpy().astype(np.float64)
    rms = float(np.sqrt(np.mean(np.square(want[keep])))) if keep.any() else 1.0
    k = int(keep.sum())
    rows = got[:k] if how == "compact" else got[keep]
    rest = got[k:] if how == "compact" else got[~keep]
    assert k == 0 or np.abs(rows - want[keep]).max() / rms <= 1e-4    # fp32 sums in another order (the parity tests' bound)
    assert np.all(rest == (7.0 if how in ("chained", "compact") else 0.0))
    # 16-bit outputs are the rounding of these
    out16 = torch.full(out.shape, 7.0, device=G.dev()).to(B.torch_dtype(dtype))
    B.focused_conv2d(B.conv_desc(n, h, w, ci, co, *geo, dtype, None, flags), xd, wd, bd, out=out16, **kw)
    assert torch.equal(out16, out.to(out16.dtype))


@pytest.mark.parametrize("how", ["mask", "labels", "list"])
@pytest.mark.parametrize("layer", LAYERS)
def test_same_sums_as_the_looping_kernel(layer, how):
    """Masks of bits send these layers to the kernel that loops over its stages: the same products in the same order, so the same bits."""
    torch = G.torch_mod()
    n, h, w, ci, co, dtype, s, p, dh = layer
    geo = ((3, 3), s, p, (dh, 1))
    xd = G.to_dev(synth.activations((n, h, w, ci), dtype, 43, 1), dtype)
    wd, bd = G.to_dev(synth.he_weights(co, 3, 3, ci, dtype, 43, 2), dtype), torch.from_numpy(synth.bias(co, 43, 3)).to(G.dev())
    md = G.mask_dev(synth.mask_objects(n, h, w, 0.48, 43, 4))
    m_out = B.mask_downsample(md, *geo)
    idx, count = B.active_index_compact(m_out)
    outs = []
    for flag, form in ((0, lambda m: m), (B.PACKED_MASKS, B.mask_pack)):
        kw = dict(mask_in=form(md))
        if how != "mask":
            kw["mask_out"] = form(m_out)
        if how == "list":
            kw.update(idx=idx, count=count)
        desc = B.conv_desc(n, h, w, ci, co, *geo, dtype, B.F32, B.RELU | flag)
        outs.append(B.focused_conv2d(desc, xd, wd, bd, **kw))
    assert float(outs[0].abs().max()) > 0 or int(count) == 0
    assert torch.equal(outs[0], outs[1])
