"""RGB stems whose pieces reach past either end of the input (loaded inside it and shifted), against the oracle."""
import pytest

from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layer", [
    # n, h, w, ci, co, k, s, p, d: fewer than 8 elements in all (one by one), just 8 and 9, images smaller than the kernel, an image of one
    # row, rows that start and end inside a piece, padding that moves pieces a whole row past the ends, two channel blocks
    (1, 1, 2, 3, 8, 7, 1, 3, 1), (1, 2, 1, 4, 8, 7, 1, 3, 1), (1, 1, 3, 3, 8, 7, 1, 3, 1), (1, 5, 5, 3, 64, 7, 2, 3, 1), (1, 1, 40, 3, 16, 7, 2, 3, 1),
    (2, 8, 8, 2, 72, 7, 1, 3, 1), (1, 4, 41, 4, 136, 7, 1, 3, 1), (3, 13, 7, 3, 64, 7, 2, 6, 1), (1, 30, 31, 3, 64, 5, 1, 4, 1), (1, 3, 4, 4, 24, 2, 1, 1, 1)])
@pytest.mark.parametrize("mask_kind,precomputed", [("objects", False), ("bernoulli", True), (None, False)])
def test_pieces_past_the_ends(layer, mask_kind, precomputed):
    P.test_stem_kernel_rows(layer, mask_kind, precomputed)
