"""The gradients of layers of few kernels in one launch: the edges of its rounds of indices, on either side of the line to the two launches, subsets of
one member to all 512, values that are not finite, and in place."""
import numpy as np
import pytest
import torch

from paper_2110_09195_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _one_launch(n, K):
    return n <= (5120 if K < 8 else 8192)


def _inputs(n, K, skew):
    g = np.random.default_rng(n + 17 * K)
    w = (1.2 * g.standard_normal((n, 9))).astype(np.float32)
    gw = g.standard_normal((n, 9)).astype(np.float32)
    idx = np.zeros(n, np.int64) if skew == "one" else np.minimum(g.geometric(min(0.3, 8 / K), size=n) - 1, K - 1)
    return w, gw, idx


@pytest.mark.parametrize("n", [1, 7, 63, 64, 65, 113, 1023, 1024, 1025, 4096, 5120, 5121, 8191, 8192, 8193])
@pytest.mark.parametrize("K, skew", [(1, "one"), (2, "geometric"), (7, "geometric"), (8, "geometric"), (32, "geometric"), (32, "one"), (512, "geometric")])
def test_members(oracle, n, K, skew):
    w, gw, idx = _inputs(n, K, skew)
    ref_w, ref_p = oracle.project_backward(w, gw, idx, K)
    o_w, o_p = G.Guarded(n * 9, torch.float32, float("nan")), G.Guarded(K * 9, torch.float32, float("nan"))
    di = G.dev(idx.astype(np.uint16))
    B.snn_project_backward(G.dev(w), G.dev(gw), di, K, g_w=o_w.t.view(n, 9), g_p=o_p.t.view(K, 9))
    o_w.check("g_w")
    o_p.check("g_p")
    assert (o_w.t.cpu().numpy().reshape(n, 9) == ref_w).all()
    sum_abs = np.zeros((K, 9))
    np.add.at(sum_abs, idx, np.abs(gw).astype(np.float64))
    # a wave has at most 512 kernels of a member, seven at a time in four chains of pairs: 512 / 28 + 1 roundings in a row, three and seven more
    # join the chains, the entries and the waves (two launches: 112 of a block's in a row and three of the second pass)
    tol = (512 // 28 + 11 if _one_launch(n, K) else 122) * 2.0 ** -24 * sum_abs + 1e-30
    got = o_p.t.cpu().numpy().astype(np.float64).reshape(K, 9)
    assert (np.abs(got - ref_p) <= tol).all()
    again = B.snn_project_backward(G.dev(w), G.dev(gw), di, K)[1]
    if _one_launch(n, K):
        assert torch.equal(again.flatten(), o_p.t), "the order of the additions is fixed"


@pytest.mark.parametrize("n, K", [(300, 8), (8192, 40)])
def test_not_finite(n, K):
    g = torch.ones((n, 9), device="cuda")
    idx = (torch.arange(n, device="cuda") % K).to(torch.int16)
    g[3, 2], g[12, 5] = float("inf"), float("nan")
    p = B.snn_project_backward(torch.zeros((n, 9), device="cuda"), g, idx, K)[1].cpu().numpy()
    assert np.isinf(p[3, 2]) and np.isnan(p[12 % K, 5]) and np.isfinite(p).sum() == K * 9 - 2


@pytest.mark.parametrize("n", [200, 4096])
def test_in_place(oracle, n):
    w, gw, idx = _inputs(n, 32, "geometric")
    ref_w, ref_p = oracle.project_backward(w, gw, idx, 32)
    g = G.dev(gw)
    _, p = B.snn_project_backward(G.dev(w), g, G.dev(idx.astype(np.uint16)), 32, g_w=g)
    assert (g.cpu().numpy() == ref_w).all()
    assert np.abs(p.cpu().numpy() - ref_p).max() <= 1e-4 * np.abs(ref_p).max()


@pytest.mark.parametrize("over", ["w", "g_wbar"])
@pytest.mark.parametrize("n, K", [(200, 32), (4096, 512), (8192, 40)])
def test_sums_over_an_input(oracle, n, K, over):
    """g_p in the last rows of an input, which it may take over: every sum is of the values that were there."""
    w, gw, idx = _inputs(n, K, "geometric")
    ref_w, ref_p = oracle.project_backward(w, gw, idx, K)
    t = {"w": G.dev(w), "g_wbar": G.dev(gw)}
    rows = min(n, K)
    place = torch.empty((n + K - rows, 9), device="cuda")
    place[:n] = t[over]
    t[over] = place[:n]
    p = place[n - rows:n - rows + K]
    g_w, _ = B.snn_project_backward(t["w"], t["g_wbar"], G.dev(idx.astype(np.uint16)), K, g_p=p)
    assert (g_w.cpu().numpy() == ref_w).all()
    assert np.abs(p.cpu().numpy() - ref_p).max() <= 1e-4 * np.abs(ref_p).max()
