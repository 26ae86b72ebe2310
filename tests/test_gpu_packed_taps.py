"""Layers whose channels are off the 128-byte stage take their reduction as one run of 16-byte pieces: pieces a tap fewer than, equal to and more than the
eight of a stage, kernels of 9 to 32 taps, every tile that goes tap by tap, every way a call can say what is kept, against the oracle; values
that are not finite lie under the irrelevant pixels."""
import numpy as np
import pytest

from oracle import fc_oracle as O
from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

LAYERS = [
    # n, h, w, ci, co, kernel, dtype, stride, pad, dilation
    (1, 13, 17, 8, 8, (3, 3), synth.BF16, (1, 1), (1, 1), (1, 1)),      # one piece a tap, two stages, the second nearly empty
    (2, 75, 59, 24, 72, (3, 3), synth.F16, (1, 1), (1, 1), (1, 1)),     # three pieces a tap; tiles that label their rows
    (3, 75, 101, 72, 200, (3, 3), synth.BF16, (2, 2), (1, 1), (1, 1)),  # nine pieces
    (1, 29, 31, 40, 16, (5, 5), synth.BF16, (1, 1), (2, 2), (1, 1)),
    (2, 61, 67, 16, 136, (5, 5), synth.F16, (2, 1), (4, 3), (2, 1)),    # padding and dilation; 25 taps
    (1, 40, 52, 8, 40, (4, 8), synth.BF16, (1, 1), (2, 4), (1, 1)),     # 32 taps, one piece each
    (4, 61, 70, 72, 40, (3, 3), synth.BF16, (1, 1), (1, 1), (1, 1)),    # 128 x 64 tiles
    (9, 97, 95, 16, 56, (3, 3), synth.F16, (1, 1), (0, 0), (1, 1)),     # narrow layer, three workgroups a CU
    (9, 91, 95, 24, 128, (3, 3), synth.BF16, (1, 1), (1, 1), (1, 1)),   # 128 x 128 tiles
    (3, 45, 53, 48, 80, (3, 3), synth.FP8, (1, 1), (1, 1), (1, 1)),     # 16 channels a piece
    (2, 41, 67, 16, 48, (5, 5), synth.FP8, (2, 2), (2, 2), (1, 1)),
]


@pytest.mark.parametrize("how", ["dense", "mask", "labels", "packed", "list", "chained", "compact"])
@pytest.mark.parametrize("kind", ["objects", "bernoulli", "one"])
@pytest.mark.parametrize("layer", LAYERS)
def test_packed_taps(layer, kind, how):
    torch = G.torch_mod()
    n, h, w, ci, co, k, dtype, s, p, d = layer
    if how == "dense" and kind != "objects":
        pytest.skip("no mask: one kind")
    geo = (k, s, p, d)
    x, wt, bias = synth.activations((n, h, w, ci), dtype, 43, 1), synth.he_weights(co, *k, ci, dtype, 43, 2), synth.bias(co, 43, 3)
    if kind == "one":
        mask = np.zeros((n, h, w), np.uint8)
        mask[-1, h // 2, w // 2] = 3                             # any nonzero byte
    else:
        mask = (synth.mask_objects if kind == "objects" else synth.mask_bernoulli)(n, h, w, 0.48, 43, 4)
    xd = G.to_dev(x, dtype)
    if how != "dense":
        xd = (xd.view(torch.uint8) if dtype == synth.FP8 else xd).clone()
        xd[torch.from_numpy(mask == 0).to(G.dev())] = 0x7f if dtype == synth.FP8 else float("nan")
        xd = xd.view(B.torch_dtype(dtype))
    wd, bd = G.to_dev(wt, dtype), torch.from_numpy(bias).to(G.dev())
    flags = B.RELU | {"chained": B.SKIP_ZERO_FILL, "compact": B.COMPACT_OUT, "packed": B.PACKED_MASKS}.get(how, 0)
    desc = B.conv_desc(n, h, w, ci, co, *geo, dtype, B.F32, flags)
    ho, wo = B.out_dims(desc)
    keep = np.ones(n * ho * wo, bool) if how == "dense" else (O.mask_downsample(mask, *k, s, p, d) != 0).reshape(-1)
    kw = {}
    if how != "dense":
        md = G.mask_dev(mask)
        kw = dict(mask_in=B.mask_pack(md) if how == "packed" else md)
        if how not in ("mask", "packed"):
            m_out = B.mask_downsample(md, *geo)
            kw.update(mask_out=m_out)
            if how != "labels":
                idx, count = B.active_index_compact(m_out)
                kw.update(idx=idx[:max(1, int(keep.sum()))].clone(), count=count)   # nothing past the count
    out = torch.full((n * ho * wo, co) if how == "compact" else (n, ho, wo, co), 7.0, device=G.dev())
    B.focused_conv2d(desc, xd, wd, bd, out=out, **kw)
    got = out.reshape(-1, co).cpu().numpy().astype(np.float64)
    nk = int(keep.sum())
    rows, rest = (got[:nk], got[nk:]) if how == "compact" else (got[keep], got[~keep])
    assert np.all(rest == (7.0 if how in ("chained", "compact") else 0.0))
    if nk:
        at = np.sort(np.random.default_rng(43).choice(nk, size=min(500, nk), replace=False))
        want = O.focused_conv2d_at(O.ConvShape(n, h, w, ci, co, *k, s, p, d, relu=True), x, wt, np.flatnonzero(keep)[at], bias=bias,
                                   mask_in=None if how == "dense" else mask, dtype=dtype)
        # sums of fp32 in another order; E4M3 products are added on the instruction's grid (the parity tests' bounds)
        rms = max(float(np.sqrt(np.mean(np.square(want)))), 1e-3)
        assert np.isfinite(rows).all() and np.abs(rows[at] - want).max() / rms <= (5e-4 if dtype == synth.FP8 else 1e-4)
    # the storage types' outputs are the rounding of these
    out16 = torch.full(out.shape, 7.0, device=G.dev()).to(torch.bfloat16 if dtype == synth.FP8 else B.torch_dtype(dtype))
    B.focused_conv2d(B.conv_desc(n, h, w, ci, co, *geo, dtype, None, flags), xd, wd, bd, out=out16, **kw)
    assert torch.equal(out16, out.to(out16.dtype))
