"""Values that are not finite in a pair of 1x1 layers: they stay in the channels that the two calls put them in, also where the middle does
not fill its blocks of 32 channels (zero weights times an infinite pixel are NaN)."""
import numpy as np
import pytest

from paper_2207_10741_amd import binding as B, synth
from tests import test_gpu_pairs as P

pytestmark = pytest.mark.gpu

INF = {B.BF16: 0x7f80, B.F16: 0x7c00}
NAN = {B.BF16: 0x7fc0, B.F16: 0x7e00, B.FP8: 0x7f}
SIGN = {B.BF16: 0x8000, B.F16: 0x8000, B.FP8: 0x80}

NARROW = [((32, 8, 96), B.BF16), ((32, 16, 96), B.BF16), ((96, 24, 144), B.F16), ((200, 40, 72), B.BF16), ((192, 32, 192), B.BF16)]
WIDE = [((8, 72, 8), B.BF16), ((64, 80, 64), B.F16), ((64, 184, 40), B.BF16), ((64, 256, 64), B.F16)]
BYTES = [((48, 80, 112), B.FP8), ((64, 144, 64), B.FP8)]


@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 20, 31)])
@pytest.mark.parametrize("channels,dtype", NARROW + WIDE + BYTES)
def test_values_that_are_not_finite_stay_where_the_calls_put_them(channels, dtype, shape, monkeypatch):
    """Weights above zero: an infinite channel makes the row's outputs +Inf; a first layer that turns it to -Inf and has a ReLU leaves the
    bias.  E4M3 has no infinity: NaN.  NaN under every irrelevant pixel."""
    n, h, w = shape
    mask = synth.mask_objects(n, h, w, 0.45, 11, 3) if n > 1 else np.ones(shape, np.uint8)
    activations, he_weights = synth.activations, synth.he_weights
    for kept_only in (False, True):
        for relu1 in (False, True):
            def pixels(size, dt, seed, stream):
                x = activations(size, dt, seed, stream).copy()
                if kept_only:
                    x[mask == 0] = NAN[dt]
                rows = x.reshape(-1, size[-1])
                at = np.flatnonzero(mask)[::7]
                rows[at, 0] = INF.get(dt, NAN[dt])
                return x

            def weights(co, kh, kw, ci, dt, seed, stream):
                bits = np.maximum(he_weights(co, kh, kw, ci, dt, seed, stream) & (SIGN[dt] - 1), 0x0400 if dt != B.FP8 else 0x08).copy()
                if relu1 and stream == 0:       # of the first layer
                    bits[..., 0] |= SIGN[dt]
                return bits

            monkeypatch.setattr(synth, "activations", pixels)
            monkeypatch.setattr(synth, "he_weights", weights)
            one, both, left = P._run(shape, channels, dtype, mask if kept_only else None, relu=(relu1, True))
            monkeypatch.undo()
            assert left and (one == both).all(), (kept_only, relu1, int((one != both).sum()))
            if dtype != B.FP8:          # the calls themselves make no NaN of these
                bits = one.numpy().view(np.uint16).reshape(-1, channels[2])
                assert ((bits[np.flatnonzero(mask)] & 0x7fff) <= INF[dtype]).all()
