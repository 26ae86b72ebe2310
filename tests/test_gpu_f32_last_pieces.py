"""fp32 layers whose rows end one to three channels into a 32-channel chunk: the last piece of a row begins in the chunk before it, which
for the first output channel and the first pixel lies before the lane's own offset."""
import pytest

from tests import test_gpu_f32_rounds as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("how", ["dense", "mask", "list"])
@pytest.mark.parametrize("layer", [
    (1, 6, 5, 225, 40, (1, 1), (1, 1), 1),
    (1, 6, 5, 226, 33, (1, 1), (0, 0), 1),
    (2, 5, 4, 33, 8, (1, 1), (1, 1), 1),
    (1, 4, 4, 67, 8, (1, 1), (0, 0), 1),
    (1, 150, 230, 35, 64, (1, 1), (1, 1), 1),     # without a mask the kernel of 128-row tiles
])
def test_last_pieces(layer, how):
    R.test_f32_rounds(layer, "all", how)
