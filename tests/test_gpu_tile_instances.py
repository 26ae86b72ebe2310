"""The tiles that the tiled kernel chooses from, for 1x1, 3x3 and other kernels, channels whole stages and packed taps, rows in place and in list
order, at sizes that choose each of them: against the oracle at sampled positions, the narrower outputs against the rounding of the fp32 one;
values that are not finite lie under the irrelevant pixels."""
import numpy as np
import pytest

from oracle import fc_oracle as O
from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

# n, h, w, ci, co, kernel, dtype, stride, flags, workspace
LAYERS = {
    # 512 tiles of 128 x 128 and more
    "wide, 5x5": (2, 91, 91, 64, 512, (5, 5), synth.BF16, 1, 0, True),
    "wide, 5x5, packed": (2, 91, 91, 16, 512, (5, 5), synth.F16, 1, 0, True),
    "wide, 5x5, E4M3": (2, 91, 91, 128, 512, (5, 5), synth.FP8, 1, 0, True),
    "wide, 3x3 stride 2": (4, 131, 131, 128, 512, (3, 3), synth.F16, 2, 0, True),
    "wide, 1x1": (2, 80, 83, 1024, 512, (1, 1), synth.BF16, 1, 0, True),
    "line, 128 channels": (8, 65, 67, 128, 200, (3, 3), synth.BF16, 1, 0, True),
    # more than 64 tiles of 128 x 64: with a workspace, into up to 64 channels without one
    "tall, 5x5": (1, 181, 187, 64, 40, (5, 5), synth.F16, 1, 0, True),
    "tall, 5x5, packed": (1, 91, 95, 24, 200, (5, 5), synth.BF16, 1, 0, True),
    "tall, 4x7, packed, E4M3": (1, 91, 95, 48, 80, (4, 7), synth.FP8, 1, 0, True),
    "narrow, 5x5": (1, 181, 187, 64, 48, (5, 5), synth.BF16, 1, 0, False),
    "narrow, 5x5, packed": (1, 181, 187, 24, 48, (5, 5), synth.F16, 1, 0, False),
    "narrow, 3x3 stride 2": (2, 181, 187, 128, 48, (3, 3), synth.BF16, 2, 0, False),
    # at most 64 of them (16-bit layers of this size run on the small layers' kernel)
    "small, 5x5, E4M3": (1, 37, 41, 128, 64, (5, 5), synth.FP8, 1, 0, True),
    "resident 1x1, four chunks": (1, 65, 67, 256, 48, (1, 1), synth.F16, 1, B.RESIDENT_WEIGHTS, True),
}


@pytest.mark.parametrize("how", ["dense", "list", "chained", "compact"])
@pytest.mark.parametrize("layer", list(LAYERS))
def test_tile_instances(layer, how):
    torch = G.torch_mod()
    n, h, w, ci, co, k, dtype, s, extra, ws = LAYERS[layer]
    geo = (k, (s, s), (k[0] // 2, k[1] // 2), (1, 1))
    draw = synth.activations_large if n * h * w * ci > 1 << 22 else synth.activations
    x, wt, bias = draw((n, h, w, ci), dtype, 59, 1), synth.he_weights(co, *k, ci, dtype, 59, 2), synth.bias(co, 59, 3)
    mask = synth.mask_objects(n, h, w, 0.48, 59, 4)
    xd, wd, bd = G.to_dev(x, dtype), G.to_dev(wt, dtype), torch.from_numpy(bias).to(G.dev())
    flags = B.RELU | extra | {"chained": B.SKIP_ZERO_FILL, "compact": B.COMPACT_OUT}.get(how, 0)
    if how == "compact" and extra:
        pytest.skip("the flag's kernels store rows in place")
    desc = lambda out: B.conv_desc(n, h, w, ci, co, *geo, dtype, out, flags)
    ho, wo = B.out_dims(desc(B.F32))
    keep, kw = np.ones(n * ho * wo, bool), {}
    if how != "dense":
        xd = (xd.view(torch.uint8) if dtype == synth.FP8 else xd).clone()
        xd[torch.from_numpy(mask == 0).to(G.dev())] = 0x7f if dtype == synth.FP8 else float("nan")
        xd = xd.view(B.torch_dtype(dtype))
        md = G.mask_dev(mask)
        m_out = B.mask_downsample(md, *geo)
        idx, count = B.active_index_compact(m_out)
        kw = dict(mask_in=md, mask_out=m_out, idx=idx, count=count)
        keep = (O.mask_downsample(mask, *k, (s, s), geo[2], (1, 1)) != 0).reshape(-1)
    if not ws:
        kw["workspace"] = None
    nk = int(keep.sum())
    kd = torch.from_numpy(keep).to(G.dev())
    outs = {}
    storage = synth.BF16 if dtype == synth.FP8 else dtype
    for out_dtype in (B.F32, storage) + ((B.FP8,) if co % 16 == 0 else ()):
        out = torch.full((n * ho * wo, co), 7.0, device=G.dev()).to(B.torch_dtype(out_dtype))
        B.focused_conv2d(desc(out_dtype), xd, wd, bd, out=out, **kw)
        rows, rest = (out[:nk], out[nk:]) if how == "compact" else (out[kd], out[~kd])
        assert bool((rest.float() == (7.0 if how in ("chained", "compact") else 0.0)).all())
        outs[out_dtype] = rows
    rows = outs[B.F32]
    assert bool(torch.isfinite(rows).all())
    assert torch.equal(outs[storage], rows.to(outs[storage].dtype))
    at = np.sort(np.random.default_rng(59).choice(nk, size=200, replace=False))
    got = rows[torch.from_numpy(at).to(G.dev())].cpu().numpy().astype(np.float64)
    if B.FP8 in outs:
        codes = outs[B.FP8].view(torch.uint8)[torch.from_numpy(at).to(G.dev())].cpu().numpy()
        np.testing.assert_array_equal(codes, O.narrow_fp8(got))
    want = O.focused_conv2d_at(O.ConvShape(n, h, w, ci, co, *k, (s, s), geo[2], (1, 1), relu=True), x, wt, np.flatnonzero(keep)[at], bias=bias,
                               mask_in=None if how == "dense" else mask, dtype=dtype)
    # the parity tests' bounds: fp32 sums in another order; E4M3 products are added on the instruction's grid
    assert np.abs(got - want).max() / float(np.sqrt(np.mean(np.square(want)))) <= (5e-4 if dtype == synth.FP8 else 1e-4)
