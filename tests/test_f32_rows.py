"""The places of the input values in the rows that a block of the fp32 dense form keeps in LDS (csrc/f32_rows.h), on the host: against
the definition of the convolution's window, also where the rows of the batch together are more than 2^31."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# Output pixels of block `blk` whose taps are not where the kernel looks for them, or -1 if one lies past the loads.
SOURCE = r"""
#include "f32_rows.h"
using namespace snn;
extern "C" long long bad_pixels(int N, int H, int W, int stride, long long blk)
{
    const Geom g = make_geom({N, 1, 1, H, W, stride, 32, SNN_ACT_F32});
    const SdRows rows = sd_rows(g);
    const SdBlock b = sd_block(g, (uint32_t)blk);
    long long bad = 0;
    for (int64_t p = blk * 32; p < blk * 32 + 32 && p < g.P; ++p) {
        const int64_t n = p / g.HoWo;
        const int ho = (int)(p % g.HoWo) / g.Wo, wo = (int)(p % g.HoWo) % g.Wo;
        const int64_t at = sd_window(g, rows, b, (uint32_t)n, ho, wo);
        bool ok = true;
        for (int t = 0; t < 9; ++t) {
            const int64_t q = at + (t / 3) * rows.pitch + t % 3;
            if (q < 0 || q >= 32 * sd_loads(g)) return -1;
            const SdPixel v = sd_pixel(g, rows, b, (int)q);
            const int h = ho * stride + t / 3 - 1, w = wo * stride + t % 3 - 1;
            const bool in = h >= 0 && h < H && w >= 0 && w < W;
            ok = ok && (in ? v.in && (int64_t)b.n0 + v.image == n && v.h == h && v.w == w : !v.in);
        }
        bad += !ok;
    }
    return bad;
}
// loads of the instance that runs, or -1 if the rows do not fit them; pieces: 100 more for each block of output channels of a wave, 1000 for four waves
extern "C" int loads(int N, int C_in, int C_out, int H, int W, int stride)
{
    const Geom g = make_geom({N, C_in, C_out, H, W, stride, 32, SNN_ACT_F32});
    const SdSplit s = sd_split_plan(g);
    const int n = sd_split(g) ? s.loads : sd_staged(g);
    if (n != 0 && n < sd_loads(g)) return -1;
    return sd_split(g) ? 1000 * s.four + 100 * s.CB + n : n;
}
extern "C" int looks_up(int N, int C_in, int C_out, int H, int W, int stride)
{
    const Geom g = make_geom({N, C_in, C_out, H, W, stride, 32, SNN_ACT_F32});
    if (sd_split(g)) return sd_pieces_look_up(g, sd_split_plan(g));
    const int quads = (C_in + 7) / 8;
    const int64_t n_blocks = (g.P + 31) / 32 * ((C_out + 31) / 32);
    return sd_looks_up(g, sd_staged(g), quads, quads < 4 ? (n_blocks + 3) / 4 : n_blocks);
}
extern "C" long long blocks(int N, int H, int W, int stride)
{
    return (make_geom({N, 1, 1, H, W, stride, 32, SNN_ACT_F32}).P + 31) / 32;
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("f32_rows")
    src, lib = str(d / "rows.hip"), str(d / "rows.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2110_09195_amd", "csrc"), src, "-o", lib], check=True)
    L = ctypes.CDLL(lib)
    for f in (L.bad_pixels, L.blocks):
        f.restype = ctypes.c_longlong
    L.bad_pixels.argtypes = [ctypes.c_int] * 4 + [ctypes.c_longlong]
    L.blocks.argtypes = [ctypes.c_int] * 4
    L.loads.argtypes = L.looks_up.argtypes = [ctypes.c_int] * 6
    return L


# N, H, W, stride: N (H + 1) on either side of 2^31 and of 2^32; tall and wide images; the ordinary ones
@pytest.mark.parametrize("case", [(2 ** 30 + 32768, 1, 1, 1), (2 ** 31 - 8192, 1, 1, 1), (7 * 10 ** 8, 3, 1, 1), (7 * 10 ** 8, 3, 1, 2), (2 ** 30 - 1, 1, 2, 1),
                                  (5 * 10 ** 8, 2, 2, 2), (1, 2 ** 28, 1, 1), (3, 10 ** 7, 5, 2), (256, 8, 8, 1), (33, 7, 7, 2), (5, 9, 19, 1),
                                  (100, 1, 31, 1), (40, 3, 3, 1)])
def test_every_tap_is_found(host, case):
    N, H, W, stride = case
    n = host.blocks(N, H, W, stride)
    # first and last blocks, and those around every eighth of the batch
    for blk in sorted({b for e in range(9) for b in range(n * e // 8 - 40, n * e // 8 + 40) if 0 <= b < n}):
        assert host.bad_pixels(N, H, W, stride, blk) == 0, (case, blk)


# which kernel, and its instance: either side of each line.  Eight channels and fewer: rows through LDS (3, 4, 6) or straight from memory (0); more: in
# pieces while the rows fit six loads, always through LDS
@pytest.mark.parametrize("case, loads", [((1, 3, 5, 3, 5, 1), 3), ((256, 8, 64, 8, 8, 1), 3), ((64, 8, 64, 16, 16, 1), 4), ((256, 1, 8, 14, 14, 1), 4),
                                         ((64, 8, 64, 28, 28, 1), 0), ((256, 8, 128, 8, 8, 2), 6), ((256, 8, 128, 7, 7, 2), 0), ((64, 8, 64, 1, 1, 1), 0),
                                         ((1, 512, 512, 56, 56, 1), 0), ((32, 16, 16, 56, 56, 1), 0), ((4, 64, 64, 8, 8, 2), 1106), ((4, 64, 64, 16, 16, 2), 0),
                                         ((9, 9, 32, 35, 35, 1), 106),
                                         ((9, 9, 32, 39, 39, 1), 0), ((256, 64, 64, 8, 8, 1), 1203), ((127, 64, 64, 8, 8, 1), 1103), ((128, 64, 64, 8, 8, 1), 1203),
                                         ((1, 16, 5, 3, 5, 1), 103), ((16, 64, 64, 16, 16, 1), 1104), ((256, 24, 64, 16, 16, 1), 204),
                                         ((64, 24, 64, 13, 13, 1), 1104), ((256, 128, 128, 8, 8, 2), 1206), ((1, 512, 64, 32, 32, 1), 1106)])
def test_kernel_and_loads(host, case, loads):
    assert host.loads(*case) == loads


@pytest.mark.parametrize("case, yes", [
    # pieces: workgroups and steps of a wave, one or two blocks of output channels, rows of indices of whole 32 bytes or others
    ((64, 64, 64, 8, 8, 1), 1), ((128, 64, 64, 8, 8, 1), 0), ((256, 64, 64, 8, 8, 1), 0), ((256, 32, 32, 8, 8, 1), 1), ((257, 32, 32, 8, 8, 1), 0),
    ((33, 96, 96, 8, 8, 1), 1), ((50, 128, 64, 8, 8, 1), 1), ((65, 128, 64, 8, 8, 1), 0), ((1, 256, 256, 8, 8, 1), 0),
    ((133, 40, 96, 8, 8, 1), 1), ((125, 100, 60, 8, 8, 1), 1), ((127, 100, 60, 8, 8, 1), 1), ((129, 100, 60, 8, 8, 1), 0), ((64, 200, 60, 8, 8, 1), 1),
    ((64, 300, 60, 8, 8, 1), 0), ((2048, 9, 32, 8, 8, 1), 1), ((2049, 9, 32, 8, 8, 1), 0), ((256, 60, 64, 8, 8, 1), 1), ((257, 60, 64, 8, 8, 1), 0),
    # the fp32 unit
    ((512, 8, 128, 8, 8, 1), 1), ((513, 8, 128, 8, 8, 1), 0), ((256, 8, 128, 16, 16, 2), 1), ((257, 8, 128, 16, 16, 2), 0), ((167, 3, 64, 28, 28, 1), 1),
    ((256, 3, 64, 28, 28, 1), 0), ((20, 16, 64, 56, 56, 1), 1), ((21, 16, 64, 56, 56, 1), 0), ((1, 128, 128, 37, 53, 1), 1), ((1, 512, 64, 56, 56, 1), 0),
    ((1, 256, 256, 37, 53, 1), 0)])
def test_codes_are_looked_up_only_where_that_is_faster(host, case, yes):
    assert host.looks_up(*case) == yes
