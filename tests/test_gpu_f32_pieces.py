"""fp32 activations as three bf16 pieces: the edges of its steps of sixteen channels, of its blocks, and of the rules that choose the number of loads, blocks
and waves, against float64; values that pieces do not hold beside values that they do."""
import sys

import numpy as np
import pytest
import torch

from paper_2110_09195_amd import binding as B
from paper_2110_09195_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _run(oracle, case, x):
    N, C_in, C_out, H, W, stride, K = case
    g = np.random.default_rng(sum(case))
    cb, idx, alpha = synth.codebook(g, K), synth.indices(g, C_out, C_in, K), synth.alpha(g, C_out)
    d = B.make_desc(N, C_in, C_out, H, W, stride, K, B.SNN_ACT_F32)
    Ho, Wo = B.out_hw(d)
    y = G.Guarded(N * C_out * Ho * Wo, torch.float32, float("nan"))
    ws = G.guarded_workspace(d, B.SNN_WS_SUBBIT)
    B.snn_subbit_prepare(d, G.dev(cb), G.dev(idx), G.dev(alpha), workspace=ws.t)
    B.snn_subbit_conv2d_prepared(d, G.dev(x), G.dev(alpha), ws.t, y.t)
    ws.check("the workspace")
    y.check("y")
    one = B.snn_subbit_conv2d(d, G.dev(x), G.dev(cb), G.dev(idx), G.dev(alpha))
    assert torch.equal(one.flatten().view(torch.int32), y.t.view(torch.int32)), "the call that may look its codes up"
    w9 = oracle.expand(cb, idx)
    return y.t.cpu().numpy().reshape(N, C_out, Ho, Wo), w9, alpha


# N, C_in, C_out, H, W, stride, K
CASES = [
    (1, 9, 1, 1, 1, 1, 2),              # the fewest channels, one pixel
    (3, 16, 32, 5, 7, 1, 4),            # one step, one block; a subset that the two-stage form had
    (2, 17, 33, 8, 8, 1, 32),           # a second step with one channel, a second block with one
    (5, 40, 70, 7, 7, 2, 32),           # an odd number of quads: the last step's second half has no words
    (2, 48, 64, 13, 13, 1, 16),         # three steps: the waves have none or one
    (2, 49, 40, 14, 14, 1, 16),         # four steps, four loads
    (9, 65, 96, 28, 28, 1, 32),         # five steps, six loads; an odd number of blocks in pairs
    (130, 64, 64, 8, 8, 1, 32),         # two blocks a wave
    (33, 64, 129, 6, 9, 1, 300),        # ... the last pair half empty, tiles over two images
    (300, 20, 64, 16, 16, 2, 7),        # ... one wave to a block
    (700, 10, 36, 8, 8, 1, 512),        # ... of one step, the last workgroup not full
    (2, 512, 40, 4, 5, 1, 32),
]


@pytest.mark.parametrize("case", CASES)
def test_pieces(oracle, case):
    N, C_in, C_out, H, W, stride, K = case
    print("f32 pieces", case, file=sys.stderr, flush=True)
    x = np.random.default_rng(sum(case)).standard_normal((N, C_in, H, W), dtype=np.float32)
    got, w9, alpha = _run(oracle, case, x)
    _, Y = oracle.conv_f32(x, w9, alpha, stride)
    _, mag = oracle.conv_f32(np.abs(x), np.full_like(w9, 511), np.abs(alpha), stride)
    # nine roundings for sixteen channels of a wave, of a chain of its own for the small pieces, four joining the sums and one for alpha
    steps = 9 * ((C_in + 15) // 16)
    assert (np.abs(got.astype(np.float64) - Y) <= (steps * 1.1 + 6) * 2.0 ** -24 * mag.astype(np.float64)).all()


@pytest.mark.parametrize("case", [(2, 40, 40, 8, 8, 1, 32), (70, 64, 64, 8, 8, 1, 32), (300, 10, 64, 8, 8, 1, 32)])
@pytest.mark.parametrize("value", [np.inf, np.nan, 1e-40, 2.0 ** -110 * (1 + 2.0 ** -23)])
def test_values_that_pieces_do_not_hold(oracle, case, value):
    """One such value among zeros and numbers of its size or ordinary ones: it counts in full where its window reaches, and nowhere else."""
    N, C_in, C_out, H, W, stride, K = case
    g = np.random.default_rng(sum(case))
    small = np.isfinite(value)
    x = np.zeros((N, C_in, H, W), dtype=np.float32) if small else g.standard_normal((N, C_in, H, W), dtype=np.float32)
    n, c, h, w = N // 2, C_in - 2, 3, 4
    x[n, c, h, w] = value
    got, w9, alpha = _run(oracle, case, x)
    clean = x.copy()
    clean[n, c, h, w] = 0.0
    ref = _run(oracle, case, clean)[0]
    inside = np.zeros(got.shape, bool)
    inside[n, :, h - 1:h + 2, w - 1:w + 2] = True
    if not small:
        assert not np.isfinite(got[inside]).any() and (np.isnan(got[inside]).all() if np.isnan(value) else np.isinf(got[inside]).all())
        assert np.isfinite(got[~inside]).all() and np.allclose(got[~inside], ref[~inside], rtol=0, atol=1e-4)
    else:
        sign = np.where((w9[:, c, None] >> (8 - np.arange(9))) & 1, 1.0, -1.0).reshape(C_out, 3, 3)[:, ::-1, ::-1]
        want = np.zeros(got.shape)
        want[n, :, h - 1:h + 2, w - 1:w + 2] = sign * float(np.float32(value)) * alpha[:, None, None].astype(np.float64)
        assert (np.abs(got - want) <= 2.0 ** -24 * np.abs(want) + 2.0 ** -149).all()
