"""Chained 3x3 layers at the sizes where the one-workgroup-per-CU kernel and the wide tiles take over from the tiled kernel, rows left in place and
rows in list order, against the oracle on sampled positions."""
import numpy as np
import pytest

from oracle import fc_oracle as O
from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

LAYERS = [
    # n, h, w, ci, co, dtype, stride
    (13, 59, 57, 128, 128, synth.BF16, 1),      # 43 719 positions: the tiled kernel
    (13, 59, 58, 128, 128, synth.BF16, 1),      # 44 486: a workgroup per CU
    (23, 31, 28, 128, 104, synth.F16, 1),       # short rows, 19 964: the tiled kernel
    (25, 27, 30, 128, 104, synth.F16, 1),       # 20 250: a workgroup per CU
    (16, 61, 67, 192, 96, synth.F16, 1),
    (60, 61, 63, 64, 104, synth.BF16, 2),       # 59 520: no pixel line
    (90, 31, 29, 64, 128, synth.BF16, 2),       # 21 600 with short rows
    (13, 100, 101, 128, 128, synth.BF16, 1),    # 1 025 granules of 128 x 128: wide tiles
    (7, 100, 101, 256, 256, synth.F16, 1),      # 1 104 of 64 x 256
    (7, 100, 101, 256, 256, synth.FP8, 1),
]


@pytest.mark.parametrize("kind", ["objects", "bernoulli", "few", "all"])
@pytest.mark.parametrize("layer", LAYERS)
def test_rows_in_place_and_in_list_order(layer, kind):
    torch = G.torch_mod()
    n, h, w, ci, co, dtype, s = layer
    geo = ((3, 3), (s, s), (1, 1), (1, 1))
    draw = synth.activations_large if n * h * w * ci > 1 << 23 else synth.activations
    x, wt, bias = draw((n, h, w, ci), dtype, 51, 1), synth.he_weights(co, 3, 3, ci, dtype, 51, 2), synth.bias(co, 51, 3)
    mask = (np.ones((n, h, w), np.uint8) if kind == "all" else synth.mask_bernoulli(n, h, w, 0.4, 51, 4) if kind == "bernoulli"
            else synth.mask_objects(n, h, w, 0.95 if kind == "few" else 0.48, 51, 4))
    xd, wd, bd = G.to_dev(x, dtype), G.to_dev(wt, dtype), torch.from_numpy(bias).to(G.dev())
    if dtype != synth.FP8:                                   # what lies under irrelevant pixels is not looked at
        xd = xd.clone()
        xd[torch.from_numpy(mask == 0).to(G.dev())] = float("nan")
    md = G.mask_dev(mask)
    m_out = B.mask_downsample(md, *geo)
    idx, count = B.active_index_compact(m_out)
    keep = (O.mask_downsample(mask, 3, 3, (s, s), (1, 1), (1, 1)) != 0).reshape(-1)
    nk = int(keep.sum())
    got = {}
    for flags in (B.SKIP_ZERO_FILL, B.COMPACT_OUT):
        desc = B.conv_desc(n, h, w, ci, co, *geo, dtype, B.F32, B.RELU | flags)
        out = torch.full((n * int(np.prod(B.out_dims(desc))), co), 7.0, device=G.dev())
        B.focused_conv2d(desc, xd, wd, bd, mask_in=md, mask_out=m_out, idx=idx, count=count, out=out)
        kd = torch.from_numpy(keep).to(G.dev())
        rows, rest = (out[:nk], out[nk:]) if flags == B.COMPACT_OUT else (out[kd], out[~kd])
        assert bool((rest == 7.0).all())
        got[flags] = rows
    at = np.sort(np.random.default_rng(51).choice(nk, size=min(300, nk), replace=False))
    want = O.focused_conv2d_at(O.ConvShape(n, h, w, ci, co, 3, 3, (s, s), (1, 1), (1, 1), relu=True), x, wt, np.flatnonzero(keep)[at],
                               bias=bias, mask_in=mask, dtype=dtype)
    rms = float(np.sqrt(np.mean(np.square(want))))
    bar = 5e-4 if dtype == synth.FP8 else 1e-4               # the parity tests' bounds
    for rows in got.values():
        assert bool(torch.isfinite(rows).all())
        assert np.abs(rows[torch.from_numpy(at).to(G.dev())].cpu().numpy().astype(np.float64) - want).max() / rms <= bar
    # rows nobody sampled: the two forms differ in the order of their sums only
    assert float((got[B.SKIP_ZERO_FILL] - got[B.COMPACT_OUT]).abs().max()) / rms <= 2 * bar


WORKGROUP_PER_CU = [
    # n, h, w, ci, co, dtype, stride, pad, dilation: from 44 000 positions on (short rows: 20 000), at most eight 32-row blocks a CU
    (8, 96, 64, 120, 128, synth.BF16, (1, 1), (1, 1), (1, 1)),     # a partial channel chunk
    (15, 51, 61, 56, 96, synth.F16, (1, 1), (1, 1), (1, 1)),       # channel tails on both sides, ragged rows
    (16, 64, 64, 64 * 3, 104, synth.BF16, (1, 1), (1, 1), (1, 1)),  # the most positions, three chunks
    (25, 61, 60, 128, 128, synth.BF16, (2, 1), (0, 2), (2, 1)),    # vertical stride and dilation, wide padding
    (21, 127, 65, 128, 72, synth.BF16, (2, 2), (1, 1), (1, 1)),    # stride 2: no shared line, tap by tap
    (10, 70, 70, 104, 128, synth.F16, (1, 1), (1, 1), (2, 2)),     # dilation 2: tap by tap
    (28, 27, 29, 128, 120, synth.BF16, (1, 1), (1, 1), (1, 1)),    # short rows
]


@pytest.mark.parametrize("kind,irr", [("objects", 0.48), ("bernoulli", 0.5), ("objects", 0.95), ("objects", 0.0), ("objects", 1.0)])
@pytest.mark.parametrize("layer", WORKGROUP_PER_CU)
def test_a_workgroup_per_cu(layer, kind, irr):
    torch = G.torch_mod()
    n, h, w, ci, co, dtype, s, p, d = layer
    geo = ((3, 3), s, p, d)
    x, wt, bias = synth.activations_large((n, h, w, ci), dtype, 53, 1), synth.he_weights(co, 3, 3, ci, dtype, 53, 2), synth.bias(co, 53, 3)
    mask = np.ones((n, h, w), np.uint8) if irr == 0 else np.zeros((n, h, w), np.uint8) if irr == 1 else \
        (synth.mask_bernoulli if kind == "bernoulli" else synth.mask_objects)(n, h, w, irr, 53, 4)
    xd, wd, bd = G.to_dev(x, dtype).clone(), G.to_dev(wt, dtype), torch.from_numpy(bias).to(G.dev())
    xd[torch.from_numpy(mask == 0).to(G.dev())] = float("nan")
    md = G.mask_dev(mask)
    m_out = B.mask_downsample(md, *geo)
    idx, count = B.active_index_compact(m_out)
    keep = (O.mask_downsample(mask, 3, 3, s, p, d) != 0).reshape(-1)
    positions = keep.size
    assert (44000 if B.out_dims(B.conv_desc(n, h, w, ci, co, *geo, dtype))[1] >= 32 else 20000) <= positions <= 65536
    outs = []
    for out_dtype in (B.F32, None):
        desc = B.conv_desc(n, h, w, ci, co, *geo, dtype, out_dtype, B.RELU | B.SKIP_ZERO_FILL)
        out = torch.full((positions, co), 7.0, device=G.dev(), dtype=B.torch_dtype(B.F32 if out_dtype is not None else dtype))
        B.focused_conv2d(desc, xd, wd, bd, mask_in=md, mask_out=m_out, idx=idx, count=count, out=out)
        outs.append(out)
    kd = torch.from_numpy(keep).to(G.dev())
    assert bool((outs[0][~kd] == 7.0).all()) and torch.equal(outs[1], outs[0].to(outs[1].dtype))
    if not keep.any():
        return
    assert bool(torch.isfinite(outs[0]).all())
    at = np.sort(np.random.default_rng(53).choice(np.flatnonzero(keep), size=min(400, int(keep.sum())), replace=False))
    want = O.focused_conv2d_at(O.ConvShape(n, h, w, ci, co, 3, 3, s, p, d, relu=True), x, wt, at, bias=bias, mask_in=mask, dtype=dtype)
    got = outs[0][torch.from_numpy(at).to(G.dev())].cpu().numpy().astype(np.float64)
    assert np.abs(got - want).max() / float(np.sqrt(np.mean(np.square(want)))) <= 1e-4     # the parity tests' bound
