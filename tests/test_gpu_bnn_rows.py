"""The 1-bit layer on packed channels as a matrix-core contraction against the oracle, bit for bit, where its tiles, channel
blocks and channel words end; the same for the popcount kernels, which a knob selects."""
import sys

import numpy as np
import pytest

from paper_2110_09195_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

# N, C_in, C_out, H, W, stride
EDGES = [
    (2, 1, 1, 1, 1, 1),              # one pixel, one channel
    (3, 1, 256, 5, 6, 1),            # the fewest kernels the matrix cores take, and one less
    (3, 255, 1, 5, 6, 2),
    (3, 31, 33, 5, 31, 1),           # one channel short of a word, one over a block
    (2, 32, 32, 4, 32, 2),
    (2, 33, 31, 6, 33, 1),           # a second word with one channel
    (2, 65, 65, 7, 9, 2),            # a pair of words and a single one
    (2, 97, 129, 3, 64, 1),
    (1, 1030, 40, 3, 4, 1),          # past the register-window kernel's range
    (5, 512, 40, 9, 9, 1),           # words that come through LDS in two parts
    (300, 24, 20, 7, 7, 1),          # tiles that run over several images
    (40, 40, 200, 30, 30, 1),
    (70, 10, 70, 60, 60, 1),         # four pixel blocks per wave
    # images of fewer words than the four that are loaded side by side, alone and as the last one of a batch
    (1, 32, 8, 1, 1, 1),
    (3, 20, 40, 1, 1, 2),
    (1, 64, 70, 1, 1, 1),
    (129, 33, 40, 1, 1, 1),
    (2, 160, 33, 1, 1, 1),           # five words: the second group of four has one
    (1, 30, 64, 1, 2, 2),
    # both sides of the line to the popcount kernels: output channels against expanded pixels, one word and many, wide rows
    (2, 40, 15, 56, 56, 1),
    (2, 40, 16, 56, 56, 1),
    (1, 24, 117, 3, 600, 1),
    (1, 24, 118, 3, 600, 1),
    (1, 70, 234, 3, 600, 2),
    (1, 520, 8, 3, 600, 1),
    (1, 520, 32, 3, 600, 1),
    (1, 520, 33, 3, 600, 1),
]


@pytest.mark.parametrize("regs", [None, 1, 0])
@pytest.mark.parametrize("case", EDGES)
def test_bnn_at_the_edges_of_its_tiles(oracle, tune, case, regs):
    import torch

    from paper_2110_09195_amd import binding as B
    if regs is not None:
        tune("BNN_REGS", regs)
    N, C_in, C_out, H, W, stride = case
    print("bnn", case, file=sys.stderr, flush=True)
    g = np.random.default_rng(sum(case))
    x = g.standard_normal((N, C_in, H, W), dtype=np.float32)
    x.flat[::9] = 0.0
    codes = g.integers(0, 512, (C_out, C_in)).astype(np.uint16)
    alpha = synth.alpha(g, C_out)
    _, Y = oracle.conv_bin(oracle.sign(x), codes, alpha, stride)
    d = B.make_desc(N, C_in, C_out, H, W, stride, 512, B.SNN_ACT_BIN_CHANNELS)
    xp = B.snn_pack_activations(torch.from_numpy(x).cuda(), B.SNN_ACT_BIN_CHANNELS)
    w9, al = torch.from_numpy(codes.view(np.int16)).cuda(), torch.from_numpy(alpha).cuda()
    y = B.snn_bnn_conv2d(d, xp, w9, al).cpu().numpy()
    assert (y == Y).all(), np.argwhere(y != Y)[:5]
    ws = B.alloc_workspace(d, B.SNN_WS_BNN)
    B.snn_bnn_prepare(d, w9, ws)
    y2 = torch.full((N, C_out) + B.out_hw(d), float("nan"), device="cuda")
    B.snn_bnn_conv2d_prepared(d, xp, al, ws, y2)
    assert (y2.cpu().numpy() == Y).all()
