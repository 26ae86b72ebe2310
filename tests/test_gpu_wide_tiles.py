"""3x3 layers on the kernel for wide tiles (256 x 256 and 384 x 128 outputs a CU): against the oracle on sampled positions,
16- and 8-bit outputs against the rounding of the fp32 ones, irrelevant rows zero to the byte, kept rows all written."""
import functools

import numpy as np
import pytest

from oracle import fc_oracle as O
from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

LAYERS = [
    # n, h, w, ci, co, dtype, sh, (ph, pw), dh; granules of a tile: 64 rows x 256 channels, 128 x 128.  With a mask the kernel serves 1 000 of
    # them; zero-filled 3 000 of fewer than 36 stages (a stage: a tap and 128 bytes of channels) and 4 000 with 128-channel tiles.
    (13, 130, 161, 128, 256, synth.BF16, 1, (1, 1), 1),     # 256-channel tiles: 4 251 granules of 18 stages
    (31, 131, 127, 128, 128, synth.F16, 1, (1, 1), 1),      # 128-channel tiles: 4 029
    (1, 1000, 130, 128, 512, synth.BF16, 1, (1, 1), 1),     # two channel tiles
    (184, 17, 33, 256, 256, synth.BF16, 1, (1, 1), 1),      # short image rows
    (10, 201, 99, 256, 256, synth.BF16, 2, (3, 2), 2),      # vertical stride and dilation, wide padding
    (1, 360, 361, 64, 512, synth.BF16, 1, (1, 1), 1),       # one chunk of channels: three groups of stages
    (3, 110, 101, 512, 512, synth.F16, 1, (1, 1), 1),       # eight chunks, 1 041 granules
    (13, 130, 161, 256, 256, synth.FP8, 1, (1, 1), 1),
    (6, 300, 301, 256, 128, synth.FP8, 1, (0, 0), 1),       # no padding
]


def _mask(kind, n, h, w):
    if kind is None:
        return None
    if kind == "all":
        return np.ones((n, h, w), np.uint8)
    if kind == "sparse":                                     # few rows kept: most workgroups only clear
        return synth.mask_objects(n, h, w, 0.97, 300, 4)
    if kind == "bernoulli":                                  # two slots a row: tall tiles go tap by tap
        return synth.mask_bernoulli(n, h, w, 0.5, 300, 4)
    if kind == "fifth":                                      # short tiles (one and two granules), tap by tap
        return synth.mask_bernoulli(n, h, w, 0.8, 300, 4)
    if kind == "tenth":                                      # short tiles, more to clear than their stages hold
        return synth.mask_objects(n, h, w, 0.9, 300, 4)
    if kind == "checker":                                    # three slots a row: every tile tap by tap
        yy, xx = np.mgrid[0:h, 0:w]
        return np.ascontiguousarray(np.broadcast_to(((yy + xx) % 2).astype(np.uint8), (n, h, w)))
    return synth.mask_objects(n, h, w, 0.48, 300, 4)


@functools.lru_cache(maxsize=1)
def _inputs(layer):
    n, h, w, ci, co, dtype = layer[:6]
    draw = synth.activations_large if n * h * w * ci > 1 << 23 else synth.activations
    return draw((n, h, w, ci), dtype, 301, 1), synth.he_weights(co, 3, 3, ci, dtype, 301, 2), synth.bias(co, 301, 3)


@pytest.mark.parametrize("kind", ["objects", "bernoulli", "fifth", "checker", "tenth", "sparse", "none", "all", None])
@pytest.mark.parametrize("layer", LAYERS)
def test_wide_tiles(layer, kind):
    torch = G.torch_mod()
    n, h, w, ci, co, dtype, sh, (ph, pw), dh = layer
    x, wt, bias = _inputs(layer)
    mask = np.zeros((n, h, w), np.uint8) if kind == "none" else _mask(kind, n, h, w)
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
        if mask is not None:                                 # chained: irrelevant rows stay as they were
            desc = B.conv_desc(n, h, w, ci, co, *geo, dtype, out_dtype, B.RELU | B.SKIP_ZERO_FILL)
            chained = torch.full((n, ho, wo, co), 7.0, dtype=torch.float32, device=G.dev()).to(B.torch_dtype(out_dtype))
            B.focused_conv2d(desc, xd, wd, bd, out=chained, **kw)
            kd = m_out != 0
            assert torch.equal(chained[kd].float(), out[kd].float()) and bool((chained[~kd].float() == 7.0).all())
    f32 = outs[B.F32]
    keep = np.ones((n, ho, wo), bool) if mask is None else O.mask_downsample(mask, 3, 3, (sh, 1), (ph, pw), (dh, 1)) != 0
    kd = torch.from_numpy(keep).to(G.dev())
    assert not bool(f32[~kd].view(torch.int32).any())
    assert not bool((f32[kd] == 7.0).all(dim=-1).any())
    for out_dtype, out in outs.items():
        if out_dtype == B.FP8:
            assert torch.equal(out.float(), f32.clamp(max=448.0).to(out.dtype).float())
        elif out_dtype != B.F32:
            assert torch.equal(out, f32.to(out.dtype))
    kept = np.flatnonzero(keep.reshape(-1))
    if kept.size == 0:
        return
    pos = np.sort(np.random.default_rng(301).choice(kept, size=min(600, kept.size), replace=False))
    shape = O.ConvShape(n, h, w, ci, co, 3, 3, (sh, 1), (ph, pw), (dh, 1), relu=True)
    want = O.focused_conv2d_at(shape, x, wt, pos, bias=bias, mask_in=mask, dtype=dtype)
    got = f32.reshape(-1, co)[torch.from_numpy(pos).to(G.dev())].cpu().numpy().astype(np.float64)
    from tests.test_gpu_fp8 import TOL_FP8
    rms = float(np.sqrt(np.mean(np.square(want))))
    assert float(np.abs(got - want).max()) / rms <= (TOL_FP8 if dtype == synth.FP8 else 1e-4)


@pytest.mark.parametrize("kind", ["objects", "bernoulli", "fifth", "tenth"])
@pytest.mark.parametrize("layer", [LAYERS[0], LAYERS[1], LAYERS[4], LAYERS[7]])
def test_forms_of_a_call_give_the_same_bits(layer, kind):
    """Packed masks, a list without labels, a list in tile order, no list at all, no bias, and launch after launch."""
    torch = G.torch_mod()
    n, h, w, ci, co, dtype, sh, (ph, pw), dh = layer
    x, wt, bias = _inputs(layer)
    geo = ((3, 3), (sh, 1), (ph, pw), (dh, 1))
    xd, wd, bd = G.to_dev(x, dtype), G.to_dev(wt, dtype), torch.from_numpy(bias).to(G.dev())
    md = G.mask_dev(_mask(kind, n, h, w))
    m_out = B.mask_downsample(md, *geo)
    idx, count = B.active_index_compact(m_out)
    out_dtype = B.BF16 if dtype == synth.FP8 else dtype

    def run(b=bd, flags=0, **kw):
        desc = B.conv_desc(n, h, w, ci, co, *geo, dtype, out_dtype, B.RELU | flags)
        out = torch.full((n, *B.out_dims(desc), co), 7.0, dtype=B.torch_dtype(out_dtype), device=G.dev())
        return B.focused_conv2d(desc, xd, wd, b, out=out, **kw)

    want = run(mask_in=md, mask_out=m_out, idx=idx, count=count)
    for it in range(10):
        assert torch.equal(run(mask_in=md, mask_out=m_out, idx=idx, count=count), want), it
    assert torch.equal(run(mask_in=md, idx=idx, count=count), want)
    assert torch.equal(run(mask_in=md), want)
    t_idx, t_count = B.active_index_compact_tiled(m_out, 4, 8)
    assert torch.equal(run(mask_in=md, mask_out=m_out, idx=t_idx, count=t_count), want)
    bits = B.mask_pack(md)
    b_out, (_, ho, wo) = B.mask_downsample_packed(bits, (n, h, w), *geo)
    p_idx, p_count = B.active_index_compact_packed(b_out, n * ho * wo)
    assert torch.equal(run(flags=B.PACKED_MASKS, mask_in=bits, mask_out=b_out, idx=p_idx, count=p_count), want)
    assert torch.equal(run(flags=B.PACKED_MASKS, mask_in=bits, idx=p_idx, count=p_count), want)
    no_bias = run(b=torch.zeros_like(bd), mask_in=md, mask_out=m_out, idx=idx, count=count)
    assert torch.equal(run(b=None, mask_in=md, mask_out=m_out, idx=idx, count=count), no_bias)
