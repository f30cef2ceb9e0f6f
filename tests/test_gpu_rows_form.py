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
    (150, 3, 2, 2, 900, 1, 8),          # wide rows that the one-hot form takes, ends in a sign or not
    (200, 3, 2, 2, 700, 1, 8),          # only if it ends in a sign
    (200, 3, 2, 2, 500, 1, 8),          # not at all
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


def test_weights_of_a_layer_whose_form_depends_on_its_ending(oracle):
    """The tables that one call writes for a layer with fp32 output and for the same layer ending in a sign are those its two
    convolutions read, where the two take different forms."""
    import torch

    from paper_2110_09195_amd import binding as B
    N, C_in, C_out, H, W, K = 200, 3, 2, 2, 700, 8
    g = np.random.default_rng(5)
    x = g.standard_normal((N, C_in, H, W), dtype=np.float32)
    cb, w, alpha = synth.codebook(g, K), synth.real_kernels(g, C_out * C_in), synth.alpha(g, C_out)
    beta = np.array([0.5, -1.5], dtype=np.float32)
    d = B.make_desc(N, C_in, C_out, H, W, 1, K, B.SNN_ACT_BIN_ROWS)
    layers = [{"desc": d, "w": G.dev(w), "codebook": G.dev(cb), "alpha": G.dev(alpha), "beta": b,
               "idx_out": torch.empty(C_out * C_in, dtype=torch.int16, device="cuda"), "workspace": B.alloc_workspace(d, B.SNN_WS_SUBBIT)}
              for b in (None, G.dev(beta))]
    B.snn_subbit_project_prepare_many(B.layer_weights_array(layers))
    xp = B.snn_pack_activations(G.dev(x), B.SNN_ACT_BIN_ROWS)
    codes = oracle.expand(cb, oracle.project(w, cb)[0].reshape(C_out, C_in))
    _, Y = oracle.conv_bin(oracle.sign(x), codes, alpha, 1)
    assert (B.snn_subbit_conv2d_prepared(d, xp, layers[0]["alpha"], layers[0]["workspace"]).cpu().numpy() == Y).all()
    y = torch.full((N, C_out, H, W), float("nan"), device="cuda")
    B.snn_subbit_conv2d_prepared_many(B.layer_io_array([{"desc": d, "x": xp, "y": y, "workspace": layers[0]["workspace"]}]))
    assert (y.cpu().numpy() == Y).all()
    want, _ = oracle.conv_sign(oracle.sign(x), codes, alpha, beta, 1)
    got = B.snn_subbit_conv2d_sign_prepared(d, xp, layers[1]["workspace"])
    assert (got.cpu().numpy().view(np.uint32).ravel() == np.asarray(want).view(np.uint32).ravel()).all()


@pytest.mark.parametrize("W", [500, 700, 900])
def test_one_call_forms_on_wide_rows(oracle, W):
    """The calls that project and convolve, and the tables from packed indices, on both sides of the line to the one-hot form."""
    import torch

    from paper_2110_09195_amd import binding as B
    N, C_in, C_out, H, K = 200, 3, 2, 2, 8
    g = np.random.default_rng(W)
    x = g.standard_normal((N, C_in, H, W), dtype=np.float32)
    cb, w, alpha = synth.codebook(g, K), synth.real_kernels(g, C_out * C_in), synth.alpha(g, C_out)
    beta = np.array([0.5, -1.5], dtype=np.float32)
    idx = oracle.project(w, cb)[0].reshape(C_out, C_in)
    xs, codes = oracle.sign(x), oracle.expand(cb, idx)
    _, Y = oracle.conv_bin(xs, codes, alpha, 1)
    y, got = G.subbit_forward(x, w, cb, alpha, C_out)
    assert (got.reshape(C_out, C_in) == idx).all() and (y == Y).all()
    want, _ = oracle.conv_sign(xs, codes, alpha, beta, 1)
    bits, got = G.subbit_forward_sign(oracle.pack_rows(x), x.shape, w, cb, alpha, beta, C_out)
    assert (got.reshape(C_out, C_in) == idx).all() and (bits == want).all()
    d = B.make_desc(N, C_in, C_out, H, W, 1, K, B.SNN_ACT_BIN_ROWS)
    xd = G.dev(x)
    arr = [{"desc": d, "x": xd, "w": G.dev(w), "codebook": G.dev(cb), "alpha": G.dev(alpha),
            "idx_out": torch.full((C_out * C_in,), -1, dtype=torch.int16, device="cuda"),
            "y": torch.full((N, C_out, H, W), float("nan"), device="cuda"), "workspace": B.alloc_workspace(d, B.SNN_WS_FORWARD)}]
    B.snn_subbit_forward_many(B.layer_forward_array(arr))
    assert (arr[0]["y"].cpu().numpy() == Y).all()
    ws = B.snn_subbit_prepare_packed(d, G.dev(cb), B.snn_pack_indices(G.dev(idx), 3), 3, G.dev(alpha))
    assert (B.snn_subbit_conv2d_prepared(d, B.snn_pack_activations(xd, B.SNN_ACT_BIN_ROWS), G.dev(alpha), ws).cpu().numpy() == Y).all()


@pytest.mark.parametrize("n_layers, N", [(3, 2), (34, 1), (36, 2), (3, 1700)])
def test_many_layers_in_one_call_equal_one_call_per_layer(n_layers, N):
    """The several-layers launch: fewer layers than one holds, exactly as many, a few more, and outputs past 256 MB (the layers
    come in another order there).  Integer sums and one multiplication: bit for bit."""
    import torch

    from paper_2110_09195_amd import binding as B
    print("many layers", n_layers, N, file=sys.stderr, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_layers + N)
    shapes = [(40, 70, 9, 33, 1), (65, 33, 5, 7, 2), (8, 128, 14, 25, 1), (200, 16, 6, 6, 1)]
    layers, want = [], []
    for i in range(n_layers):
        C_in, C_out, H, W, stride = shapes[i % len(shapes)]
        d = B.make_desc(N, C_in, C_out, H, W, stride, 16, B.SNN_ACT_BIN_ROWS)
        x = B.snn_pack_activations(torch.randn((N, C_in, H, W), generator=gen, device="cuda"), B.SNN_ACT_BIN_ROWS)
        cb = torch.randperm(512, generator=gen, device="cuda")[:16].to(torch.int16)
        idx = torch.randint(0, 16, (C_out, C_in), generator=gen, device="cuda").to(torch.int16)
        alpha = torch.rand(C_out, generator=gen, device="cuda") + 0.5
        y = torch.full((N, C_out) + B.out_hw(d), float("nan"), device="cuda")
        layers.append({"desc": d, "x": x, "y": y, "workspace": B.snn_subbit_prepare(d, cb, idx, alpha)})
        want.append(B.snn_subbit_conv2d(d, x, cb, idx, alpha))
    if N > 1000:
        assert sum(v.numel() * 4 for v in want) > 256 << 20
    B.snn_subbit_conv2d_prepared_many(B.layer_io_array(layers))
    torch.cuda.synchronize()
    for a, b in zip(layers, want):
        assert torch.equal(a["y"], b)


@pytest.mark.parametrize("n_layers, N", [(1, 1), (3, 70), (35, 2), (37, 1)])
def test_forward_of_many_layers_equals_forward_per_layer(n_layers, N):
    """Projection and packing of several layers in one launch: a grid of almost nothing but projections, one with packing
    workgroups between all of them, as many layers as a launch holds and a few more; rows that pack vectorised and not."""
    import torch

    from paper_2110_09195_amd import binding as B
    print("forward of many layers", n_layers, N, file=sys.stderr, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_layers * 1000 + N)
    shapes = [(40, 70, 9, 33, 1), (65, 33, 5, 7, 2), (64, 64, 28, 28, 1), (3, 16, 2, 2100, 2)]
    layers = []
    for i in range(n_layers):
        C_in, C_out, H, W, stride = shapes[i % len(shapes)]
        K = (16, 64, 5)[i % 3]
        d = B.make_desc(N, C_in, C_out, H, W, stride, K, B.SNN_ACT_BIN_ROWS)
        layers.append({"desc": d, "x": torch.randn((N, C_in, H, W), generator=gen, device="cuda"),
                       "w": torch.randn((C_out * C_in, 9), generator=gen, device="cuda"),
                       "codebook": torch.sort(torch.randperm(512, generator=gen, device="cuda")[:K]).values.to(torch.int16),
                       "alpha": torch.rand(C_out, generator=gen, device="cuda") + 0.5,
                       "idx_out": torch.full((C_out * C_in,), -1, dtype=torch.int16, device="cuda"),
                       "y": torch.full((N, C_out) + B.out_hw(d), float("nan"), device="cuda"), "workspace": B.alloc_workspace(d, B.SNN_WS_FORWARD)})
    B.snn_subbit_forward_many(B.layer_forward_array(layers))
    for L in layers:
        idx = B.snn_project_kernels(L["w"], L["codebook"])
        assert torch.equal(L["idx_out"], idx)
        d = L["desc"]
        y = B.snn_subbit_conv2d(d, B.snn_pack_activations(L["x"], B.SNN_ACT_BIN_ROWS), L["codebook"], idx.view(d.C_out, d.C_in), L["alpha"])
        assert torch.equal(L["y"], y)


# N, C_in, C_out, H, W, stride, K, launches: the convolution makes its weight words itself in one or two passes of 32 output x 64 input
# channels, and the layers past that line; rows of odd and even width with and without a last group of less than four pixels
ONE_LAUNCH = [(1, 1, 1, 5, 3, 1, 2, 1), (3, 31, 32, 7, 7, 1, 5, 1), (2, 33, 17, 9, 15, 2, 512, 1), (5, 64, 32, 16, 31, 1, 200, 1),
              (40, 16, 16, 64, 64, 1, 32, 2), (2, 65, 31, 14, 14, 1, 32, 1), (9, 128, 20, 7, 13, 2, 64, 1), (4, 64, 64, 8, 8, 1, 16, 1),
              (2, 40, 33, 33, 6, 1, 300, 1), (2, 129, 32, 8, 8, 1, 32, 2), (2, 64, 65, 9, 9, 1, 32, 2), (130, 16, 16, 33, 33, 1, 32, 2),
              (100, 16, 16, 32, 32, 1, 32, 1)]


@pytest.mark.parametrize("case", ONE_LAUNCH)
def test_words_made_by_the_convolution(oracle, case):
    """Which launches a call made shows in its workspace: the one that makes the words itself leaves it alone."""
    import torch
    from paper_2110_09195_amd import binding as B
    N, C_in, C_out, H, W, stride, K, launches = case
    print("one launch", case, file=sys.stderr, flush=True)
    g = np.random.default_rng(sum(case[:-1]))
    x = g.standard_normal((N, C_in, H, W), dtype=np.float32)
    cb, idx, alpha = synth.codebook(g, K), synth.indices(g, C_out, C_in, K), synth.alpha(g, C_out)
    _, Y = oracle.conv_bin(oracle.sign(x), oracle.expand(cb, idx), alpha, stride)
    d = B.make_desc(N, C_in, C_out, H, W, stride, K, B.SNN_ACT_BIN_ROWS)
    xp = B.snn_pack_activations(G.dev(x), B.SNN_ACT_BIN_ROWS)
    ws = B.alloc_workspace(d, B.SNN_WS_SUBBIT).fill_(0x5a)
    y = B.snn_subbit_conv2d(d, xp, G.dev(cb), G.dev(idx), G.dev(alpha), None, ws).cpu().numpy()
    assert (y == Y).all(), np.argwhere(y != Y)[:5]
    assert bool((ws == 0x5a).all()) == (launches == 1)
    ws = B.snn_subbit_prepare(d, G.dev(cb), G.dev(idx), G.dev(alpha))
    prepared = B.snn_subbit_conv2d_prepared(d, xp, G.dev(alpha), ws)
    torch.cuda.synchronize()
    assert (prepared.cpu().numpy() == Y).all()


@pytest.mark.parametrize("W", [5, 8, 16, 32, 33, 64])
def test_thresholds_of_the_sign_ending(oracle, W):
    """Scales and shifts of either sign, zero, infinite and not a number, and thresholds on attained sums."""
    g = np.random.default_rng(W)
    N, C_in, C_out, H, K = 3, 40, 96, 6, 32
    x = g.standard_normal((N, C_in, H, W), dtype=np.float32)
    cb, idx, alpha = synth.codebook(g, K), synth.indices(g, C_out, C_in, K), synth.alpha(g, C_out)
    xs, codes = oracle.sign(x), oracle.expand(cb, idx)
    alpha[::2] *= -1.0
    S, _ = oracle.conv_bin(xs, codes, np.ones_like(alpha), 1)
    beta = -(alpha * np.median(S, axis=(0, 2, 3))).astype(np.float32)
    inf, nan = np.float32(np.inf), np.float32(np.nan)
    for c, (a, b) in enumerate([(0, 0), (0, -1), (-0.0, 1), (nan, 0), (1, nan), (inf, 0), (-inf, 0), (inf, -inf), (1, inf), (-1, -inf), (1e-45, 0),
                                (1e-45, -1e-45), (3e38, 1), (-3e38, 3e38), (1, 1e9), (1, -1e9), (nan, nan), (0, nan)]):
        alpha[c], beta[c] = a, b
    with np.errstate(all="ignore"):
        want, _ = oracle.conv_sign(xs, codes, alpha, beta, 1)
    got = G.subbit_sign(oracle.pack_rows(x), x.shape, cb, idx, alpha, beta, 1)
    assert (got == want).all(), np.argwhere(got != want)[:5]
