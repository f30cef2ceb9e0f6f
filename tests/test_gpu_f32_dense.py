"""The dense form of the convolution with fp32 activations at the edges of its blocks of 32 pixels, 32 output channels and
eight input channels, with its channels split over waves and not, against the oracle."""
import sys

import numpy as np
import pytest

from paper_2110_09195_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


# N, C_in, C_out, H, W, stride, K
@pytest.mark.parametrize("case", [
    (1, 1, 1, 1, 1, 1, 16),             # one pixel, one channel
    (40, 3, 5, 1, 1, 1, 512),           # 32 images in a block of pixels
    (3, 24, 33, 5, 7, 1, 32),           # the most channels that are not split; one output channel over a block
    (3, 25, 31, 5, 7, 2, 32),           # the fewest that are split, an odd number
    (2, 41, 64, 4, 8, 1, 64),           # waves of one and of two groups of channels, the last group with one channel
    (1, 513, 20, 6, 6, 1, 300),
    (2, 40, 512, 3, 11, 1, 4),          # few subset members: many output channels alone decide
    (2, 15, 256, 3, 11, 2, 15),
])
def test_f32_dense_form(oracle, case):
    N, C_in, C_out, H, W, stride, K = case
    print("f32 dense", case, file=sys.stderr, flush=True)
    g = np.random.default_rng(sum(case))
    x = g.standard_normal((N, C_in, H, W), dtype=np.float32)
    cb, idx, alpha = synth.codebook(g, K), synth.indices(g, C_out, C_in, K), synth.alpha(g, C_out)
    w9 = oracle.expand(cb, idx)
    _, Y = oracle.conv_f32(x, w9, alpha, stride)
    _, mag = oracle.conv_f32(np.abs(x), np.full_like(w9, 511), np.abs(alpha), stride)       # sums of magnitudes
    got = G.subbit_f32(x, cb, idx, alpha, stride)
    # at most a rounding per channel of a tap, thirteen joining the sums and one for alpha, each of 2^-24 of the magnitudes
    assert (np.abs(got.astype(np.float64) - Y) <= (C_in + 16) * 2.0 ** -24 * mag.astype(np.float64) * 1.01).all()
