"""Orders in which workgroups take their work: every output is made once, whatever the number of units, for eighths and for shorter runs."""
import pytest

from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G, test_gpu_grouped as GR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layer", [
    # n, h, w, ci, co, k, s, p, groups; blocks of 64 channels, spans of 64 positions
    (1, 5, 5, 64, 64, 3, 1, 1, 16), (1, 33, 37, 64, 64, 3, 1, 1, 16),                       # one block; one span, 20
    (3, 17, 19, 128, 128, 3, 1, 1, 32), (7, 30, 31, 192, 192, 3, 1, 1, 48),                 # two and three, fewer images than XCDs
    (8, 13, 15, 128, 128, 3, 1, 1, 32), (9, 11, 7, 576, 576, 3, 1, 1, 36),                  # as many, and more, 9 blocks
    (1, 8, 9, 512, 512, 3, 1, 1, 32), (2, 27, 23, 512, 512, 3, 1, 1, 32), (1, 7, 7, 1024, 1024, 3, 1, 1, 32)])  # 8 and 16 blocks
@pytest.mark.parametrize("mask_kind,irr", [("objects", 0.48), ("bernoulli", 0.5), ("objects", 1.0), (None, 0.0)])
def test_grouped_windows(layer, mask_kind, irr):
    out, want, keep = GR._run(layer, synth.BF16, B.F32, mask_kind=mask_kind, irr=irr)
    assert G.rel_err(G.to_f64(out), want, keep) <= GR.TOL_F32_OUT
    assert not out.cpu().numpy()[~keep].any()


@pytest.mark.parametrize("layer", [
    # n, h, w, c, stride; 64 MB and more: segments of 2^k workgroups, the last one short; images of one workgroup, and more than a segment has
    (67, 57, 61, 144, 1), (9, 121, 113, 272, 2), (4001, 9, 9, 104, 1), (2, 500, 499, 72, 1), (1, 601, 700, 96, 2), (11, 60, 60, 1040, 1)])
@pytest.mark.parametrize("masked", [True, False])
def test_depthwise_tiles(layer, masked):
    """The images of a batch give the bits that each gives alone."""
    torch = G.torch_mod()
    n, h, w, c, s = layer
    gen = torch.Generator(device=G.dev()).manual_seed(7)
    x = torch.randn((n, h, w, c), generator=gen, device=G.dev()).to(torch.bfloat16)
    wt = G.to_dev(synth.he_weights(c, 3, 3, 1, B.BF16, 53, 2)[..., 0], B.BF16)
    mask = (torch.rand((n, h, w), generator=gen, device=G.dev()) < 0.5).to(torch.uint8) if masked else None
    desc = lambda images: B.conv_desc(images, h, w, c, c, stride=(s, s), in_dtype=B.BF16, flags=B.RELU)
    ho, wo = B.out_dims(desc(n))
    assert n * (h * w + ho * wo) * c * 2 >= 64000000
    out = torch.full((n, ho, wo, c), 7.0, dtype=torch.bfloat16, device=G.dev())
    B.focused_dwconv2d(desc(n), x, wt, mask_in=mask, out=out)
    few = max(1, 30000000 // ((h * w + ho * wo) * c * 2))       # (as many images as stay below)
    for i in range(0, n, few):
        part = x[i:i + few]
        alone = B.focused_dwconv2d(desc(part.shape[0]), part, wt, mask_in=None if mask is None else mask[i:i + few])
        assert torch.equal(out[i:i + few], alone), i
    if masked:
        kept = mask[:, ::s, ::s].bool()
        assert not out[~kept].any() and out[kept].any()


@pytest.mark.parametrize("layer", [
    # n, h, w, co, k, s: about 198 MB of output (22 MB a tap), where more workgroups are started than are resident, and below
    (2, 601, 800, 128, 3, 1), (2, 380, 1001, 128, 3, 1), (1, 1081, 1920, 136, 5, 1), (4, 1080, 1919, 96, 3, 2)])
def test_rgb_rows_cleared_beside_tiles(layer):
    torch = G.torch_mod()
    n, h, w, co, k, s = layer
    gen = torch.Generator(device=G.dev()).manual_seed(9)
    x = torch.randn((n, h, w, 3), generator=gen, device=G.dev()).to(torch.bfloat16)
    wt = G.to_dev(synth.he_weights(co, k, k, 3, B.BF16, 57, 2), B.BF16)
    mask = G.mask_dev(synth.mask_objects(n, h, w, 0.48, 57, 4))
    outs = []
    for flag in (0, B.SKIP_ZERO_FILL):
        desc = B.conv_desc(n, h, w, 3, co, (k, k), (s, s), (k // 2, k // 2), in_dtype=B.BF16, flags=B.RELU | flag)
        ho, wo = B.out_dims(desc)
        raw = torch.full((n * ho * wo + 1, co), 7.0, dtype=torch.bfloat16, device=G.dev())
        B.focused_conv2d(desc, x, wt, mask_in=mask, out=raw[:-1].view(n, ho, wo, co))
        outs.append(raw)
    keep = torch.cat([B.mask_downsample(mask, (k, k), (s, s), (k // 2, k // 2)).reshape(-1).bool(), torch.zeros(1, dtype=torch.bool, device=G.dev())])
    filled, chained = outs
    assert torch.equal(filled[keep], chained[keep]) and filled[keep].any()
    assert bool((chained[~keep] == 7.0).all()) and bool((filled[-1] == 7.0).all())
    assert not filled[:-1][~keep[:-1]].any()
