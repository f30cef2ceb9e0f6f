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


# values: what the inputs hold beside ordinary numbers
@pytest.mark.parametrize("case", [(2, 3, 40, 5, 9, 1, 16), (2, 41, 70, 6, 7, 2, 32), (3, 64, 33, 8, 8, 1, 64), (2, 10, 20, 5, 6, 1, 4)])
@pytest.mark.parametrize("values", ["infinite", "nan", "subnormal", "huge"])
def test_f32_special_values(oracle, case, values):
    """Infinities and NaN reach the outputs whose windows hold them and no other (padding is no product with zero); subnormal
    inputs count in full.  The last case is the two-stage form's."""
    N, C_in, C_out, H, W, stride, K = case
    print("f32 special", case, values, file=sys.stderr, flush=True)
    g = np.random.default_rng(sum(case))
    x = g.standard_normal((N, C_in, H, W), dtype=np.float32)
    if values == "infinite":
        x.flat[::97], x.flat[50::131] = np.inf, -np.inf
    elif values == "nan":
        x.flat[::97] = np.nan
    elif values == "subnormal":
        x = (x * np.float32(1e-39)).astype(np.float32)
        assert (np.abs(x) < 2.0 ** -126).all() and x.any()
    else:                                               # sums of magnitudes up to 64 * 9 * 5e35 stay below 3.4e38
        x = np.clip(x, -5, 5) * np.float32(1e35)
    cb, idx = synth.codebook(g, K), synth.indices(g, C_out, C_in, K)
    alpha = np.ones(C_out, dtype=np.float32) if values != "subnormal" else np.full(C_out, 2.0 ** 20, dtype=np.float32)
    sg = np.where((oracle.expand(cb, idx)[:, :, None] >> (8 - np.arange(9))) & 1, 1.0, -1.0)        # [C_out][C_in][9]
    xp = np.pad(x.astype(np.float64), ((0, 0), (0, 0), (1, 1), (1, 1)))
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    win = np.stack([xp[:, :, t // 3:t // 3 + stride * (Ho - 1) + 1:stride, t % 3:t % 3 + stride * (Wo - 1) + 1:stride] for t in range(9)], 2)
    finite = np.where(np.isfinite(win), win, 0.0)
    want = np.einsum("oct,nctyx->noyx", sg, finite) * float(alpha[0])
    mag = np.abs(finite).sum((1, 2))[:, None] * float(alpha[0])
    plus = np.einsum("oct,nctyx->noyx", (sg > 0) * 1.0, (win == np.inf) * 1.0) + np.einsum("oct,nctyx->noyx", (sg < 0) * 1.0, (win == -np.inf) * 1.0)
    minus = np.einsum("oct,nctyx->noyx", (sg < 0) * 1.0, (win == np.inf) * 1.0) + np.einsum("oct,nctyx->noyx", (sg > 0) * 1.0, (win == -np.inf) * 1.0)
    nan = np.isnan(win).any((1, 2))[:, None] | ((plus > 0) & (minus > 0))
    got = G.subbit_f32(x, cb, idx, alpha, stride).astype(np.float64)
    assert (np.isnan(got) == nan).all()
    assert (got[~nan & (plus > 0)] == np.inf).all() and (got[~nan & (minus > 0)] == -np.inf).all()
    ok = ~nan & (plus == 0) & (minus == 0)
    assert np.isfinite(got[ok]).all()
    # sums as above; a subnormal's roundings are of an absolute size (2^-150, and those of up to 9 C_in terms scaled by alpha)
    tol = (C_in + 16) * 2.0 ** -24 * mag * 1.01
    assert (np.abs(got - want) <= np.broadcast_to(tol, got.shape))[ok].all(), np.abs(got - want)[ok].max()


# N, C_in, C_out, H, W, stride, K: rows that a wave brings to LDS in three, four and six loads, and rows too wide for that; one wave per
# block (up to 24 channels) and four; tiles over several images, one-row and one-column images, odd channel counts
STAGED = [(9, 40, 33, 7, 7, 1, 32), (5, 24, 40, 8, 8, 2, 16), (40, 33, 64, 3, 3, 1, 64), (3, 64, 32, 14, 14, 1, 32), (3, 7, 70, 9, 16, 2, 20),
          (2, 65, 32, 28, 28, 1, 32), (2, 16, 32, 5, 33, 2, 32), (2, 48, 32, 6, 60, 1, 32), (3, 8, 32, 4, 61, 1, 16), (33, 40, 16, 1, 5, 1, 32),
          (17, 9, 300, 6, 1, 1, 4), (2, 128, 32, 28, 28, 1, 32), (3, 40, 32, 8, 8, 2, 32), (30, 33, 64, 16, 16, 1, 16), (100, 40, 64, 13, 13, 1, 16)]


@pytest.mark.parametrize("case", STAGED)
def test_rows_through_lds(oracle, case):
    """Against float64, and the call that looks its codes up against the one on prepared words, bit for bit."""
    import torch
    from paper_2110_09195_amd import binding as B
    N, C_in, C_out, H, W, stride, K = case
    print("fp32 rows", case, flush=True)
    g = np.random.default_rng(sum(case))
    x = g.standard_normal((N, C_in, H, W), dtype=np.float32)
    cb, idx, alpha = synth.codebook(g, K), synth.indices(g, C_out, C_in, K), synth.alpha(g, C_out)
    ref = oracle.conv_f32(x, oracle.expand(cb, idx), alpha, stride)
    y = G.subbit_f32(x, cb, idx, alpha, stride)
    G.assert_f32_close(y, ref[1] if isinstance(ref, tuple) else ref)
    d = B.make_desc(N, C_in, C_out, H, W, stride, K, B.SNN_ACT_F32)
    ws = B.snn_subbit_prepare(d, G.dev(cb), G.dev(idx), G.dev(alpha))
    prepared = B.snn_subbit_conv2d_prepared(d, G.dev(x), G.dev(alpha), ws)
    torch.cuda.synchronize()
    assert (prepared.cpu().numpy() == y).all()


# N, C_in, C_out, H, W, stride, K, whether the call leaves the workspace alone: one launch where the convolution looks the codes up, two past
# the lines of that rule, from rows in LDS and straight from memory, one wave and four per block
ROUTES = [(8, 64, 64, 8, 8, 1, 32, True), (257, 64, 64, 8, 8, 1, 64, False), (8, 128, 128, 14, 14, 1, 32, True), (20, 128, 128, 13, 13, 1, 32, False),
          (9, 64, 64, 28, 28, 1, 32, True), (40, 64, 64, 28, 28, 1, 512, False), (3, 300, 40, 9, 9, 2, 32, False), (130, 3, 64, 28, 28, 1, 17, True),
          (170, 3, 64, 28, 28, 1, 32, False), (5, 70, 33, 8, 8, 2, 32, True)]


@pytest.mark.parametrize("case", ROUTES)
def test_call_looks_its_codes_up_or_prepares_them(case):
    """Which launches a call made shows in its workspace; the result is that of prepare and convolution, bit for bit."""
    import torch
    from paper_2110_09195_amd import binding as B
    *shape, alone = case
    N, C_in, C_out, H, W, stride, K = shape
    print("fp32 call", case, flush=True)
    g = np.random.default_rng(sum(shape))
    x = G.dev(g.standard_normal((N, C_in, H, W), dtype=np.float32))
    cb, idx, alpha = G.dev(synth.codebook(g, K)), G.dev(synth.indices(g, C_out, C_in, K)), G.dev(synth.alpha(g, C_out))
    d = B.make_desc(N, C_in, C_out, H, W, stride, K, B.SNN_ACT_F32)
    ws = B.alloc_workspace(d, B.SNN_WS_SUBBIT).fill_(0x5a)
    y = B.snn_subbit_conv2d(d, x, cb, idx, alpha, None, ws)
    assert bool((ws == 0x5a).all()) == alone
    prepared = B.snn_subbit_conv2d_prepared(d, x, alpha, B.snn_subbit_prepare(d, cb, idx, alpha))
    assert torch.equal(y, prepared)
