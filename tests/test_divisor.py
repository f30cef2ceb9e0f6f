"""Division by multiplication (csrc/snn_internal.h), on the host: exact for every divisor, one among them, up to 2^31 - 1."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "snn_internal.h"
using namespace snn;
// quotients that are wrong, of n around multiples of d over the whole range
extern "C" long long wrong(unsigned d)
{
    const Divisor D = make_divisor(d);
    const unsigned long long top = (1ull << 31) - 1, multiples = top / d;
    long long bad = 0;
    for (unsigned long long i = 0; i <= 600; ++i)
        for (const unsigned long long m : {i, multiples - (i < multiples ? i : multiples), multiples / 601 * i})
            for (const unsigned long long n : {m * d, m * d + d - 1, m * d + d / 2})
                if (n <= top && fast_div((unsigned)n, D) != n / d) ++bad;
    return bad + (fast_div((unsigned)top, D) != top / d);
}
extern "C" unsigned shift(unsigned d) { return make_divisor(d).shift; }
extern "C" unsigned by_none(unsigned n) { return fast_div(n, make_divisor(0)); }
"""


def test_quotients(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    src, lib = str(tmp_path / "divisor.hip"), str(tmp_path / "divisor.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2110_09195_amd", "csrc"), src, "-o", lib], check=True)
    L = ctypes.CDLL(lib)
    L.wrong.argtypes, L.wrong.restype = [ctypes.c_uint], ctypes.c_longlong
    for f in (L.shift, L.by_none):
        f.argtypes, f.restype = [ctypes.c_uint], ctypes.c_uint
    around = {v for s in range(31) for v in (2 ** s - 1, 2 ** s, 2 ** s + 1) if 1 <= v < 2 ** 31}
    for d in sorted(around | set(range(1, 2000)) | {3 ** i for i in range(19)}):
        assert L.wrong(d) == 0, d
        assert (L.shift(d) == 0) == (d == 1), d
    assert [L.by_none(n) for n in (0, 7, 2 ** 31 - 1)] == [0, 7, 2 ** 31 - 1]        # (a size that does not exist: through, and no trap)
