"""The 1x1 layers' dense contraction against the oracle and against the one-hot form, bit for bit, on both sides of the line between its tiles:
odd numbers of words, channels that are no whole word, pixel and channel tails, tiles that run over images, both strides."""
import sys

import numpy as np
import pytest
import torch

from paper_2110_09195_amd import binding as B
from paper_2110_09195_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

# N, C_in, C_out, H, W, stride, K
CASES = [
    (1, 16, 1, 1, 1, 1, 32),            # one pixel, one channel
    (3, 24, 31, 5, 7, 1, 20),           # less than a word, less than a block
    (2, 32, 33, 4, 8, 1, 64),           # whole word and block of pixels, one channel over
    (7, 96, 64, 3, 3, 1, 32),           # an odd number of words; tiles over several images
    (2, 136, 65, 9, 11, 2, 32),         # five words, the last one with eight channels
    (1, 2048, 100, 7, 7, 1, 64),        # many pairs of words
    (37, 40, 70, 30, 31, 1, 32),        # two by two blocks, every tail
    (64, 8, 96, 32, 32, 1, 64),         # ... one group of channels
    (90, 328, 64, 29, 29, 2, 7),        # ... eleven words, stride 2
    (400, 64, 256, 7, 7, 1, 32),        # ... tiles over two images
    (25, 64, 256, 64, 64, 1, 32),       # ... output of more than 96 MB
    (62, 48, 41, 63, 64, 1, 32),        # ... planes of half lines
]


@pytest.mark.parametrize("case", CASES)
def test_dense_1x1(oracle, case, tune):
    N, C_in, C_out, H, W, stride, K = case
    print("dense 1x1", case, file=sys.stderr, flush=True)
    g = np.random.default_rng(7000 + sum(case))
    images = min(N, 3)
    x = np.resize(g.standard_normal((images, C_in, H, W), dtype=np.float32), (N, C_in, H, W))     # the batch repeats up to three images
    cb = g.permutation(256)[:K].astype(np.uint16)
    idx = g.integers(0, K, size=(C_out, C_in // 8)).astype(np.uint16)
    alpha = synth.alpha(g, C_out)
    _, Y = oracle.conv1x1_bin(oracle.sign(x[:images]), cb, idx, alpha, stride)
    d = B.make_desc(N, C_in, C_out, H, W, stride, K, B.SNN_ACT_BIN_CHANNELS)
    xp = B.snn_pack_activations(G.dev(x), B.SNN_ACT_BIN_CHANNELS)
    want = torch.from_numpy(Y).cuda()

    def run():
        ws, y = G.guarded_workspace(d, B.SNN_WS_CONV1X1), G.Guarded(Y[0].size * N, torch.float32, float("nan"))
        B.snn_subbit_conv1x1_prepare(d, G.dev(cb), G.dev(idx), G.dev(alpha), workspace=ws.t)
        B.snn_subbit_conv1x1_prepared(d, xp, ws.t, y.t)
        ws.check("the workspace")
        y.check("y")
        return y.t.view((N,) + Y.shape[1:])

    y = run()
    for i in range(images):
        assert bool((y[i::images] == want[i]).all()), i
    tune("MFMA_KS", 1)                   # asks for the one-hot form
    assert torch.equal(run(), y)
