"""Masks and kept lists of all levels from one launch: rows off the 16-byte pieces, steps of 1 to 16 pixels, workgroups that begin
anywhere in a row, the mask's last bytes, any nonzero byte; against the oracle, to the bit."""
import numpy as np
import pytest

from oracle import fc_oracle as O
from paper_2207_10741_amd import binding as B, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

S1, S2, S4 = ((3, 3), (1, 1), (1, 1), (1, 1)), ((3, 3), (2, 2), (1, 1), (1, 1)), ((1, 1), (4, 4), (0, 0), (1, 1))
PYRAMIDS = [
    # n, h, w, steps
    (1, 224, 224, (S1, S2, S2, S2)),
    (1, 65, 67, (S2, S2, S2, S2)),                               # steps of 2 .. 16, a level of 17 reads
    (3, 71, 93, (S2, S4, S2)),
    (1, 64, 16, (S2, S2, S2, S2)),                               # rows of fewer than four positions
    (2, 40, 1031, (S1, ((3, 5), (1, 2), (1, 2), (1, 1)), S2)),   # rows of more than a workgroup's positions
    (1, 200, 333, (((3, 3), (2, 1), (0, 0), (1, 1)), S2)),       # a step of 1 that starts off the first byte
    (1, 150, 210, (((3, 3), (1, 3), (1, 1), (1, 1)), S2)),       # a step of 3: position by position
    (1, 90, 100, (((5, 5), (2, 2), (4, 4), (2, 2)), S2)),        # centre taps clamped at the border
    (5, 126, 130, (S1, S2, S2)),                                 # 1 024 threads
    (8, 130, 131, (S1, S2, S2)),                                 # just inside one launch (through the stride, rows off the pieces)
    (9, 130, 131, (S1, S2, S2)),                                 # just outside
    (5, 208, 244, (S1, ((1, 1), (16, 16), (0, 0), (1, 1)))),     # just inside at the mask's resolution
    (7, 188, 199, (S1,)),
    (8, 181, 182, (S1, S2)),                                     # just outside
    (2, 120, 180, (S1, S2, S2, S2, S2)),                         # five levels
    (2, 120, 180, (S1, S2, S2, S2, S2, S2)),                     # six
]


@pytest.mark.parametrize("kind", ["objects", "bernoulli", "all", "none", "last"])
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("pyramid", PYRAMIDS)
def test_levels_of_one_mask(pyramid, offset, packed, kind):
    torch = G.torch_mod()
    n, h, w, steps = pyramid
    mask = {"objects": lambda: synth.mask_objects(n, h, w, 0.48, 9, 1), "bernoulli": lambda: synth.mask_bernoulli(n, h, w, 0.5, 9, 1),
            "all": lambda: np.ones((n, h, w), np.uint8), "none": lambda: np.zeros((n, h, w), np.uint8),
            "last": lambda: np.zeros((n, h, w), np.uint8)}[kind]()
    mask = mask * np.random.default_rng(9).integers(1, 256, mask.shape).astype(np.uint8)
    if kind == "last":
        mask[-1, -1, -1] = 128
    room = torch.zeros((mask.size + 16,), dtype=torch.uint8, device=G.dev())
    md = room[offset:offset + mask.size].view(n, h, w)           # (offset 1: no aligned loads)
    md.copy_(G.mask_dev(mask))
    room[offset + mask.size:] = 255                              # what follows the mask is not looked at
    pyr = B.PreparedPyramid(md, list(steps), packed=packed)
    for _ in range(2):
        for level, step in zip(pyr(), steps):
            pass
    want = mask
    for (m_out, idx, count), ((kh, kw), s, p, d), dims in zip(pyr.levels, steps, pyr.dims):
        want = O.mask_downsample(want, kh, kw, s, p, d)
        assert want.shape == tuple(dims)
        if packed:
            assert torch.equal(m_out[:B.packed_mask_words(want.size)], B.mask_pack(G.mask_dev(want))[:B.packed_mask_words(want.size)])
        else:
            np.testing.assert_array_equal(m_out.cpu().numpy(), want)
        kept = np.flatnonzero(want.reshape(-1))
        assert int(count) == kept.size
        np.testing.assert_array_equal(idx[:kept.size].cpu().numpy(), kept)
