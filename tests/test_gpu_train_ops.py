"""The straight-through / subset gradients at the sizes where their blocks end and the block size changes, on tensors that
are not 16-byte aligned, and with values that are not finite."""
import numpy as np
import pytest
import torch

from paper_2110_09195_amd import binding as B

pytestmark = pytest.mark.gpu


def _inputs(n, K, shift):
    g = np.random.default_rng(n + 31 * K + shift)
    w = (1.2 * g.standard_normal((n, 9))).astype(np.float32)
    gw = g.standard_normal((n, 9)).astype(np.float32)
    idx = np.minimum(g.geometric(min(0.3, 8 / K), size=n) - 1, K - 1)           # skewed, as in trained networks

    def dev(a):
        buf = torch.empty(a.size + 8, dtype=torch.from_numpy(a).dtype, device="cuda")
        v = buf[shift:shift + a.size].view(a.shape)
        v.copy_(torch.from_numpy(a))
        return v
    return w, gw, idx, dev(w), dev(gw), dev(idx.astype(np.int16)), dev(np.zeros_like(w))


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n,K", [(1, 32), (3, 1), (111, 16), (112, 17), (113, 32), (112 * 320, 32), (112 * 320 + 1, 33), (112 * 1280, 64),
                                 (112 * 1280 + 5, 65), (5000, 128), (5000, 129), (150000, 256), (5000, 257), (40000, 512),
                                 (112 * 320, 128), (112 * 320 + 1, 128), (112 * 320, 65), (513, 129), (10240, 512), (10241, 512), (5 << 12, 256),
                                 (1 + (5 << 12), 256), (112 * 320 + 1, 129)])
def test_gradients_at_the_edges_of_the_blocks(oracle, n, K, shift):
    w, gw, idx, dw, dg, di, do = _inputs(n, K, shift)
    got_w, got_p = B.snn_project_backward(dw, dg, di, K, g_w=do)
    ref_w, ref_p = oracle.project_backward(w, gw, idx, K)
    assert (got_w.cpu().numpy() == ref_w).all()
    sum_abs = np.zeros((K, 9))
    np.add.at(sum_abs, idx, np.abs(gw).astype(np.float64))
    # a block adds at most 448 terms one after the other (256 where a wave has 512 kernels' sums to itself or with one other), a lane of the second pass at most blocks / 64 + 1 of the
    # partial sums, and six additions join the lanes: so many roundings of at most 2^-24 of the sum of magnitudes
    tol = (448 + n // 112 // 64 + 7) * 2.0 ** -24 * sum_abs + 1e-30
    assert (np.abs(got_p.cpu().numpy().astype(np.float64) - ref_p) <= tol).all()


@pytest.mark.parametrize("K, n", [(8, 300), (100, 300), (250, 300), (300, 300), (100, 112 * 320 + 1)])
def test_values_that_are_not_finite_stay_in_their_member(K, n):
    w = torch.zeros((n, 9), device="cuda")
    g = torch.ones((n, 9), device="cuda")
    idx = (torch.arange(n, device="cuda") % K).to(torch.int16)
    g[3, 2], g[12, 5], w[20, 1] = float("inf"), float("nan"), float("nan")
    g_w, g_p = B.snn_project_backward(w, g, idx, K)
    p = g_p.cpu().numpy()
    assert np.isinf(p[3, 2]) and np.isnan(p[12 % K, 5]) and np.isfinite(p).sum() == K * 9 - 2
    assert g_w[20, 1] == 0.0
