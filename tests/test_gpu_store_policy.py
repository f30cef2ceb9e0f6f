"""Outputs of the dense contraction are stored under one of three cache policies, chosen by the size and alignment of their planes: each side
of each line against the oracle, image by image (a batch repeats two images)."""
import sys

import numpy as np
import pytest
import torch

from paper_2110_09195_amd import binding as B
from paper_2110_09195_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def layer(g, oracle, N, C_in, C_out, H, W):
    """A prepared layer of N images, of which only two differ, and their outputs as the oracle has them."""
    x = g.standard_normal((2, C_in, H, W), dtype=np.float32)
    cb, idx, alpha = synth.codebook(g, 32), synth.indices(g, C_out, C_in, 32), synth.alpha(g, C_out)
    _, Y = oracle.conv_bin(oracle.sign(x), oracle.expand(cb, idx), alpha, 1)
    d = B.make_desc(N, C_in, C_out, H, W, 1, 32, B.SNN_ACT_BIN_ROWS)
    packed = torch.from_numpy(oracle.pack_rows(x).view(np.int32)).cuda().flatten(1)
    xp = packed.repeat((N + 1) // 2, 1)[:N].contiguous().flatten()
    ws = B.snn_subbit_prepare(d, G.dev(cb), G.dev(idx), G.dev(alpha))
    return {"desc": d, "x": xp, "workspace": ws, "alpha": G.dev(alpha), "want": torch.from_numpy(Y).cuda()}


def same(y, L):
    d = L["desc"]
    got = y.view((d.N, d.C_out) + B.out_hw(d))
    return bool((got[0::2] == L["want"][0]).all()) and bool((got[1::2] == L["want"][1]).all())


# planes of whole lines, half lines and neither; outputs of the first two on both sides of 96 and 144 MB
@pytest.mark.parametrize("case", [(2, 16, 40, 16, 16), (125, 32, 64, 56, 56), (129, 32, 64, 56, 56), (3, 16, 40, 28, 28), (377, 16, 128, 28, 28),
                                  (379, 16, 128, 28, 28), (5, 16, 40, 14, 14), (170, 16, 256, 14, 14), (174, 16, 256, 14, 14), (9, 16, 40, 13, 13),
                                  (65, 16, 40, 3, 5)])
@pytest.mark.parametrize("shift", [0, 1])
def test_policies_of_one_layer(oracle, case, shift):
    print("store policy", case, shift, file=sys.stderr, flush=True)
    L = layer(np.random.default_rng(sum(case)), oracle, *case)
    out = G.Guarded(L["want"][0].numel() * case[0] + shift, torch.float32)          # (shift: an output that is aligned to four bytes only)
    out.t.fill_(float("nan"))
    B.snn_subbit_conv2d_prepared(L["desc"], L["x"], L["alpha"], L["workspace"], out.t[shift:])
    out.check("y")
    assert same(out.t[shift:], L)


@pytest.mark.parametrize("N", [1, 64, 67, 260, 360])       # outputs of 0.7, 46, 49, 189 and 261 MB: all policies and orders of the launch of several layers
def test_policies_of_several_layers(oracle, N):
    g = np.random.default_rng(N)
    layers = [layer(g, oracle, N, *s) for s in ((32, 64, 28, 28), (32, 256, 14, 14), (64, 512, 13, 13), (16, 70, 7, 7))]
    outs = []
    for L in layers:
        outs.append(G.Guarded(L["want"][0].numel() * N, torch.float32, float("nan")))
        L["y"] = outs[-1].t
    B.snn_subbit_conv2d_prepared_many(B.layer_io_array(layers))
    for o, L in zip(outs, layers):
        o.check("y")
        assert same(o.t, L)
