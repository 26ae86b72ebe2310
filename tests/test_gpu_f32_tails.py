"""fp32 3x3 layers whose input channels are no whole 32-channel chunks, on the kernel of rounds: last stages of one to thirty-one channels,
rows that are no whole 16-byte pieces, against the oracle and, bit for bit, against the kernel that masks of bits go to."""
import pytest

from tests import test_gpu_f32_rounds as R

pytestmark = pytest.mark.gpu

LAYERS = [
    (1, 1, 4, 4, 4, (1, 1), (1, 1), 1),           # one piece
    (1, 9, 7, 5, 3, (1, 1), (1, 1), 1),           # a second piece of one channel: three again
    (2, 17, 38, 21, 44, (1, 1), (1, 1), 1),
    (1, 14, 20, 31, 33, (1, 1), (0, 2), 2),
    (3, 37, 5, 33, 35, (1, 1), (1, 1), 1),        # a second chunk of one channel, loaded from the end of the first
    (1, 31, 33, 42, 24, (2, 1), (3, 3), 1),       # two again, taps wholly outside the image
    (2, 60, 80, 62, 64, (1, 1), (1, 1), 1),       # work for two workgroups a CU: three rounds in LDS
    (4, 67, 90, 16, 116, (1, 1), (1, 1), 1),      # half a stage, three workgroups a CU
    (1, 19, 21, 223, 40, (2, 2), (1, 1), 1),      # 63 stages
    (1, 19, 21, 225, 40, (1, 1), (1, 1), 1),      # one channel too many: the general kernel
]


@pytest.mark.parametrize("how", ["dense", "mask", "labels", "list", "chained", "no bias"])
@pytest.mark.parametrize("kind", ["objects", "bernoulli", "all", "none"])
@pytest.mark.parametrize("layer", LAYERS)
def test_f32_tails(layer, kind, how):
    R.test_f32_rounds(layer, kind, how)


@pytest.mark.parametrize("how", ["mask", "labels", "list"])
@pytest.mark.parametrize("layer", LAYERS)
def test_same_sums_as_the_general_kernel(layer, how):
    R.test_same_sums_as_the_kernel_for_any_layer(layer, how)
