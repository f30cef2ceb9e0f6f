"""The dense contraction on packed rows (the form the library picks for +-1 activations) against the oracle, bit for bit,
at the sizes where its tiles, channel blocks and packed words end: one below, at and above each multiple, for every
number of pixel blocks per wave, in the fp32 and the sign form."""
import sys

import numpy as np
import pytest

from paper_2110_09195_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

# N, C_in, C_out, H, W, stride, K
EDGES = [
    (2, 1, 1, 1, 1, 1, 2),              # one pixel, one channel: every border at once
    (3, 31, 33, 5, 31, 1, 32),          # one short of a channel block, one over; one-word rows of odd width
    (2, 32, 32, 4, 32, 1, 300),         # exactly one block each way; K past the one-hot forms
    (2, 33, 31, 6, 33, 2, 32),          # a second channel block with one channel; the row's second word holds one pixel
    (2, 64, 64, 7, 8, 1, 64),           # one pair of channel blocks
    (2, 65, 65, 7, 9, 1, 16),           # a pair and a single block of one channel
    (2, 97, 129, 3, 64, 2, 32),         # an odd number of blocks; five blocks of output channels
    (1, 20, 70, 4, 97, 1, 32),          # rows of four words, the last one with one pixel
    (1, 1030, 40, 3, 4, 1, 32),         # many pairs
    (5, 512, 40, 9, 9, 1, 32),          # channel blocks that come through LDS in two parts
    (300, 24, 20, 7, 7, 1, 32),         # two pixel blocks per wave, tiles that run over several images
    (40, 40, 200, 30, 30, 1, 32),       # two by two blocks, a pixel tail
    (70, 10, 70, 60, 60, 1, 8),         # four pixel blocks per wave
]


@pytest.mark.parametrize("case", EDGES)
def test_rows_form_at_the_edges_of_its_tiles(oracle, case):
    N, C_in, C_out, H, W, stride, K = case
    print("rows form", case, file=sys.stderr, flush=True)
    g = np.random.default_rng(sum(case))
    x = g.standard_normal((N, C_in, H, W), dtype=np.float32)
    x.flat[::9] = 0.0
    cb, idx, alpha = synth.codebook(g, K), synth.indices(g, C_out, C_in, K), synth.alpha(g, C_out)
    xs, codes = oracle.sign(x), oracle.expand(cb, idx)
    _, Y = oracle.conv_bin(xs, codes, alpha, stride)
    y = G.subbit_bin(x, cb, idx, alpha, stride)
    assert (y == Y).all(), np.argwhere(y != Y)[:5]
    if K > 64 or (C_in == 1 and K <= 32):
        return                                          # the sign calls refuse these
    # thresholds on attained values: where the two roundings of the definition matter
    alpha[::3] *= -1.0
    beta = -(alpha * np.median(Y, axis=(0, 2, 3))).astype(np.float32)
    want, _ = oracle.conv_sign(xs, codes, alpha, beta, stride)
    got = G.subbit_sign(oracle.pack_rows(x), x.shape, cb, idx, alpha, beta, stride)
    assert (got == want).all(), np.argwhere(got != want)[:5]
