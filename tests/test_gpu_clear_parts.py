"""Irrelevant rows cleared by several waves a block of positions: every one of them zero to the byte, kept rows the bits of a launch that clears
nothing, rows past the end untouched; blocks from one position to several, rows on both sides of the line for sharing."""
import pytest

from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["objects", "bernoulli", "all", "none"])
@pytest.mark.parametrize("layer,out_dtype", [
    # n, h, w, ci, co, k, dtype
    ((1, 1, 1, 64, 2048, 1, synth.BF16), None), ((1, 8, 8, 64, 1000, 1, synth.F16), None), ((1, 5, 13, 512, 2048, 1, synth.BF16), None),
    ((3, 7, 9, 72, 128, 1, synth.BF16), None), ((3, 7, 9, 72, 248, 1, synth.BF16), None), ((3, 7, 9, 72, 256, 1, synth.BF16), None),
    ((2, 31, 33, 40, 136, 1, synth.F16), B.F32), ((8, 22, 23, 256, 1024, 1, synth.BF16), None), ((2, 17, 16, 512, 520, 3, synth.BF16), None),
    ((2, 17, 16, 128, 1040, 1, synth.FP8), None), ((2, 17, 16, 128, 1040, 3, synth.FP8), B.F32),
])
def test_every_row_is_cleared_once(layer, out_dtype, kind):
    torch = G.torch_mod()
    n, h, w, ci, co, k, dtype = layer
    geo = ((k, k), (1, 1), (k // 2, k // 2))
    xd = G.to_dev(synth.activations((n, h, w, ci), dtype, 51, 1), dtype)
    wd, bd = G.to_dev(synth.he_weights(co, k, k, ci, dtype, 51, 2), dtype), torch.from_numpy(synth.bias(co, 51, 3)).to(G.dev())
    mask = torch.full((n, h, w), int(kind == "all"), dtype=torch.uint8, device=G.dev())
    if kind in ("objects", "bernoulli"):
        mask = G.mask_dev((synth.mask_objects if kind == "objects" else synth.mask_bernoulli)(n, h, w, 0.48, 51, 4))
    idx, count = B.active_index_compact(mask)
    keep = mask.reshape(-1) != 0
    outs = []
    for flag in (0, B.SKIP_ZERO_FILL):
        desc = B.conv_desc(n, h, w, ci, co, *geo, in_dtype=dtype, out_dtype=out_dtype, flags=B.RELU | flag)
        room = torch.empty((B.workspace_bytes(desc),), dtype=torch.uint8, device=G.dev())
        size = torch.empty((), dtype=B.torch_dtype(desc.out_dtype)).element_size()
        raw = torch.full(((n * h * w + 1) * co * size,), 0x3C, dtype=torch.uint8, device=G.dev())
        out = raw[:n * h * w * co * size].view(B.torch_dtype(desc.out_dtype)).reshape(n, h, w, co)
        B.focused_conv2d(desc, xd, wd, bd, mask_in=mask, mask_out=mask, idx=idx, count=count, out=out, workspace=room)
        outs.append(raw.reshape(n * h * w + 1, -1))
    filled, chained = outs
    assert not bool(filled[:-1][~keep].any()) and bool((chained[:-1][~keep] == 0x3C).all())
    assert torch.equal(filled[:-1][keep], chained[:-1][keep])
    assert bool((filled[-1] == 0x3C).all())
