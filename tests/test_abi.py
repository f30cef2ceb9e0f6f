"""The C-ABI library loads and exports what include/snn.h declares (CPU only: no compute call)."""
import ctypes
import os
import re
import sys

import pytest

from paper_2110_09195_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "snn.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(snn_[a-z0-9_]+)\s*\(", text)))


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(binding.LIB_PATH):
        from paper_2110_09195_amd import build
        build.build()
    return binding.lib()


def test_header_declares_the_boundary():
    names = _declared()
    for required in ("snn_pack_activations", "snn_project_kernels", "snn_subbit_conv2d", "snn_bnn_conv2d"):
        assert required in names
    assert sorted(binding.EXPORTS) == names


def test_every_declared_symbol_is_exported(L):
    for name in _declared():
        assert hasattr(L, name), name
        assert ctypes.cast(getattr(L, name), ctypes.c_void_p).value


def test_status_strings(L):
    assert binding.status_string(0) == "SNN_OK"
    assert binding.status_string(-1) == "SNN_ERR_INVALID_ARG"
    assert binding.status_string(-2) == "SNN_ERR_UNSUPPORTED"
    assert binding.status_string(-3) == "SNN_ERR_WORKSPACE"
    assert binding.status_string(-4) == "SNN_ERR_LAUNCH"
    assert binding.status_string(-99) == "SNN_ERR_UNKNOWN"


def test_packed_bytes(L):
    assert binding.snn_packed_bytes(2, 3, 4, 33, binding.SNN_ACT_BIN_ROWS) == 2 * 3 * 4 * 2 * 4
    assert binding.snn_packed_bytes(2, 40, 4, 5, binding.SNN_ACT_BIN_CHANNELS) == 2 * 4 * 5 * 2 * 4
    assert binding.snn_packed_bytes(2, 3, 4, 5, binding.SNN_ACT_F32) == 2 * 3 * 4 * 5 * 4
    assert binding.snn_packed_bytes(0, 3, 4, 5, binding.SNN_ACT_BIN_ROWS) == 0
    assert binding.snn_packed_bytes(2, 3, 4, 5, 7) == 0


def test_workspace_bytes_and_rejections(L):
    d = binding.make_desc(128, 256, 256, 14, 14, 1, 32, binding.SNN_ACT_BIN_ROWS)
    assert binding.snn_workspace_bytes(d, binding.SNN_WS_SUBBIT) > 256 * 256 * 2
    assert binding.snn_workspace_bytes(d, binding.SNN_WS_BNN) == 0        # rows layout: not for the 1-bit kernel
    d.act = binding.SNN_ACT_BIN_CHANNELS
    assert binding.snn_workspace_bytes(d, binding.SNN_WS_BNN) >= 256 * 9 * 8 * 4
    assert binding.snn_workspace_bytes(d, binding.SNN_WS_SUBBIT) == 0
    for field, bad in (("stride", 3), ("K", 0), ("K", 513), ("N", 0), ("C_in", 0), ("act", 9)):
        d = binding.make_desc(1, 32, 32, 8, 8, 1, 32, binding.SNN_ACT_BIN_ROWS)
        setattr(d, field, bad)
        assert binding.snn_workspace_bytes(d, binding.SNN_WS_SUBBIT) == 0, field
    assert binding.snn_workspace_bytes(binding.make_desc(1, 32, 32, 8, 8), 5) == 0


def test_invalid_arguments_are_status_codes_not_crashes(L):
    d = binding.make_desc(1, 32, 32, 8, 8, 1, 32, binding.SNN_ACT_BIN_ROWS)
    null = ctypes.c_void_p(0)
    assert L.snn_subbit_conv2d(ctypes.byref(d), null, null, null, null, null, null, 0, null) == binding.SNN_ERR_INVALID_ARG
    assert L.snn_bnn_conv2d(ctypes.byref(d), null, null, null, null, null, 0, null) == binding.SNN_ERR_INVALID_ARG
    assert L.snn_bnn_prepare(ctypes.byref(d), null, null, 0, null) == binding.SNN_ERR_INVALID_ARG
    assert L.snn_bnn_conv2d_prepared(ctypes.byref(d), null, null, null, null, 0, null) == binding.SNN_ERR_INVALID_ARG
    assert L.snn_subbit_forward(ctypes.byref(d), null, null, null, null, null, null, null, 0, null) == binding.SNN_ERR_INVALID_ARG
    assert L.snn_pack_activations(null, null, 1, 1, 1, 1, 0, null) == binding.SNN_ERR_INVALID_ARG
    assert L.snn_project_kernels(null, 4, null, 32, null, null) == binding.SNN_ERR_INVALID_ARG
    assert L.snn_subbit_conv2d(None, null, null, null, null, null, null, 0, null) == binding.SNN_ERR_INVALID_ARG
    # layout / size checks happen before any device work
    one = ctypes.c_void_p(256)   # never dereferenced: the calls below are rejected first
    assert L.snn_pack_activations(one, one, 1, 1, 1, 1, binding.SNN_ACT_F32, null) == binding.SNN_ERR_INVALID_ARG
    assert L.snn_project_kernels(one, 4, one, 513, one, null) == binding.SNN_ERR_INVALID_ARG
    d.act = binding.SNN_ACT_BIN_CHANNELS
    assert L.snn_subbit_conv2d(ctypes.byref(d), one, one, one, one, one, one, 1 << 20, null) == binding.SNN_ERR_UNSUPPORTED
    d.act = binding.SNN_ACT_BIN_ROWS
    assert L.snn_bnn_conv2d(ctypes.byref(d), one, one, one, one, one, 1 << 20, null) == binding.SNN_ERR_UNSUPPORTED
    assert L.snn_subbit_conv2d(ctypes.byref(d), one, one, one, one, one, one, 16, null) == binding.SNN_ERR_WORKSPACE
    # a workspace of sufficient size at an address that is not a multiple of 256 is refused too
    odd = ctypes.c_void_p(256 + 16)
    assert L.snn_subbit_conv2d(ctypes.byref(d), one, one, one, one, one, odd, 1 << 30, null) == binding.SNN_ERR_WORKSPACE
    d.act = binding.SNN_ACT_BIN_CHANNELS
    assert L.snn_bnn_conv2d(ctypes.byref(d), one, one, one, one, odd, 1 << 30, null) == binding.SNN_ERR_WORKSPACE
    # the one-call forward pass: binary activations only, and its own workspace size
    assert L.snn_subbit_forward(ctypes.byref(d), one, one, one, one, one, one, one, 1 << 30, null) == binding.SNN_ERR_UNSUPPORTED
    d.act = binding.SNN_ACT_BIN_ROWS
    assert L.snn_subbit_forward(ctypes.byref(d), one, one, one, one, one, one, one, 16, null) == binding.SNN_ERR_WORKSPACE
    assert L.snn_subbit_forward(ctypes.byref(d), one, one, one, one, one, one, odd, 1 << 30, null) == binding.SNN_ERR_WORKSPACE
    ws_conv = binding.snn_workspace_bytes(d, binding.SNN_WS_SUBBIT)
    ws_fwd = binding.snn_workspace_bytes(d, binding.SNN_WS_FORWARD)
    assert ws_fwd >= ws_conv + binding.snn_packed_bytes(d.N, d.C_in, d.H, d.W, binding.SNN_ACT_BIN_ROWS)
    d.act = binding.SNN_ACT_F32
    assert binding.snn_workspace_bytes(d, binding.SNN_WS_FORWARD) == 0


def test_tuning_knobs_and_slots(L, tune):
    B = binding
    for knob in range(B.SNN_TUNE_COUNT):
        assert B.snn_get_tuning(knob) == B.SNN_TUNE_AUTO
    assert B.snn_get_tuning(99) == B.SNN_TUNE_AUTO
    assert L.snn_set_tuning(99, 1) == B.SNN_ERR_INVALID_ARG
    assert L.snn_set_tuning(B.SNN_TUNE_MFMA_TILE, 33) == B.SNN_ERR_INVALID_ARG
    assert L.snn_set_tuning(B.SNN_TUNE_MFMA_KS, 3) == B.SNN_ERR_INVALID_ARG
    assert L.snn_set_tuning(B.SNN_TUNE_STACK, 2) == B.SNN_ERR_INVALID_ARG
    # slots per channel of the form a layer is launched in (Sec. 4.5: the gather needs one)
    rows = B.SNN_ACT_BIN_ROWS
    assert B.snn_subbit_slots_per_channel(B.make_desc(64, 256, 256, 14, 14, 1, 32, rows)) == 32
    assert B.snn_subbit_slots_per_channel(B.make_desc(64, 256, 256, 14, 14, 1, 64, rows)) == 64
    assert B.snn_subbit_slots_per_channel(B.make_desc(64, 256, 256, 14, 14, 1, 512, rows)) == 0
    assert B.snn_subbit_slots_per_channel(B.make_desc(64, 1, 256, 14, 14, 1, 32, rows)) == 0
    assert B.snn_subbit_slots_per_channel(B.make_desc(64, 64, 64, 8, 8, 1, 32, B.SNN_ACT_F32)) == 0
    assert B.snn_subbit_slots_per_channel(B.make_desc(256, 512, 512, 7, 7, 1, 16, rows)) == 16   # long channel runs
    assert B.snn_subbit_slots_per_channel(B.make_desc(64, 64, 64, 56, 56, 1, 16, rows)) == 32
    tune("MFMA_QUAD", 0)
    assert B.snn_get_tuning(B.SNN_TUNE_MFMA_QUAD) == 0
    assert B.snn_subbit_slots_per_channel(B.make_desc(256, 512, 512, 7, 7, 1, 16, rows)) == 32
    tune("SUBBIT_MFMA", 0)
    assert B.snn_subbit_slots_per_channel(B.make_desc(64, 256, 256, 14, 14, 1, 32, rows)) == 0
    bad = B.make_desc(64, 256, 256, 14, 14, 1, 32, rows)
    bad.stride = 3
    assert L.snn_subbit_slots_per_channel(ctypes.byref(bad)) == B.SNN_ERR_INVALID_ARG


def test_workspace_covers_both_pixel_block_forms(L, tune):
    """The plain and the sign-epilogue calls cut the pixels differently and can pick different table layouts
    (four channels per step only in one of them): the reported size is the larger of the two.  Shapes on which
    the two differ, with the byte counts of the larger layout worked out by hand: selector rows of
    ceil(C_in / 4) * 4 * COP words + finishing table + table image + the stack kernel's tables."""
    B = binding
    for N, C_in in ((112, 386), (224, 258)):
        d = B.make_desc(N, C_in, 256, 14, 14, 1, 16, B.SNN_ACT_BIN_ROWS)
        COP = 256
        sel = (C_in + 3) // 4 * 4 * COP * 4
        assert B.snn_workspace_bytes(d, B.SNN_WS_SUBBIT) >= sel + COP * 16 * 8 + 512 * 48
        tune("MFMA_QUAD", 0)
        smaller = B.snn_workspace_bytes(d, B.SNN_WS_SUBBIT)
        tune("MFMA_QUAD", B.SNN_TUNE_AUTO)
        assert smaller < B.snn_workspace_bytes(d, B.SNN_WS_SUBBIT)


def test_layers_past_the_documented_limits_are_refused_before_device_work(L):
    """Packed inputs of 2^31 words and more, and outputs of more than 65535 channel blocks: UNSUPPORTED from every call, whichever
    kernel the library would pick for a smaller layer of that kind.  (The pointers are never used.)"""
    B = binding
    p, big = ctypes.c_void_p(256), 1 << 62
    rows, chans = B.SNN_ACT_BIN_ROWS, B.SNN_ACT_BIN_CHANNELS
    for N, C_in, C_out, H, W, K in ((1 << 20, 2048, 8, 1, 1, 512), (1 << 20, 2048, 8, 1, 1, 32), (1 << 16, 128, 300, 32, 257, 64),
                                    (1 << 20, 4096, 40, 1, 3, 200), (1, 32, 65536 * 256, 1, 1, 512)):
        d = B.make_desc(N, C_in, C_out, H, W, 1, K, rows)
        r = ctypes.byref(d)
        assert L.snn_subbit_conv2d(r, p, p, p, p, p, p, big, None) == B.SNN_ERR_UNSUPPORTED, (N, C_in, C_out, H, W, K)
        assert L.snn_subbit_prepare(r, p, p, p, p, big, None) == B.SNN_ERR_UNSUPPORTED
        assert L.snn_subbit_conv2d_prepared(r, p, p, p, p, big, None) == B.SNN_ERR_UNSUPPORTED
        assert L.snn_subbit_forward(r, p, p, p, p, p, p, p, big, None) == B.SNN_ERR_UNSUPPORTED
    # 2^31 words; 65536 blocks of 64 channels of the kernel with register-resident windows, and of 32 of the other one
    for N, C_in, C_out, H, W in ((1 << 20, 4096, 8, 4, 4), (1 << 24, 128, 40, 4, 8), (1, 32, 65536 * 64, 8, 8), (1, 600, 65536 * 32, 8, 8)):
        d = B.make_desc(N, C_in, C_out, H, W, 1, 512, chans)
        r = ctypes.byref(d)
        assert L.snn_bnn_conv2d(r, p, p, p, p, p, big, None) == B.SNN_ERR_UNSUPPORTED, (N, C_in, C_out, H, W)
        assert L.snn_bnn_prepare(r, p, p, big, None) == B.SNN_ERR_UNSUPPORTED
        assert L.snn_bnn_conv2d_prepared(r, p, p, p, p, big, None) == B.SNN_ERR_UNSUPPORTED


def test_gradient_workspace_of_a_larger_layer_serves_a_smaller_one(L):
    """Non-decreasing in the number of kernels (one workspace for a network's largest layer), across the sizes where the kernel's
    blocks change, and in the subset size."""
    size = binding.lib().snn_project_backward_workspace_bytes
    edges = [112 * 320, 112 * 1280]
    ns = sorted({0, 1, 112, 113, 128 * 256, 192 * 192, 512 * 512} | {e + i for e in edges for i in (-113, -1, 0, 1, 2, 113, 225, 40000)} |
                set(range(1, 400000, 997)))
    for K in (1, 32, 257, 512):
        sizes = [size(n, K) for n in ns]
        assert sizes == sorted(sizes), K
    assert all(size(n, 32) <= size(n, 33) for n in ns)
    assert size(128 * 256, 32) <= size(192 * 192, 32)


def test_a_workspace_holds_the_tables_of_one_form(L):
    """The size is that of the largest form's tables, not their sum (a network keeps a workspace per layer): the two-stage tables'
    by hand, and the limit of the call with the library's own buffer, which reports it before any device work."""
    B = binding
    rows = B.SNN_ACT_BIN_ROWS

    def up(n):
        return (n + 255) // 256 * 256
    # K > 64: 512 codes, uint16 offsets of ceil(C_in / 8) * 8 x 256-channel blocks, 16 border corrections per channel
    assert B.snn_workspace_bytes(B.make_desc(8, 512, 512, 7, 7, 1, 128, rows), B.SNN_WS_SUBBIT) == 2048 + up(512 * 512 * 2) + up(512 * 64)
    assert B.snn_workspace_bytes(B.make_desc(8, 100, 150, 37, 53, 2, 128, rows), B.SNN_WS_SUBBIT) == 2048 + up(104 * 256 * 2) + up(256 * 64)
    # K <= 32: a selector word per input and output channel (four bytes a kernel), and less than 128 KB of other tables
    for C in (128, 256, 512):
        assert 4 * C * C < B.snn_workspace_bytes(B.make_desc(64, C, C, 14, 14, 1, 32, rows), B.SNN_WS_SUBBIT) < 4 * C * C + (1 << 17)
    # the dense contraction's where they are the largest: 2304 bytes per 64 x 32 channels and the scales
    assert B.snn_workspace_bytes(B.make_desc(8, 264, 8, 7, 7, 1, 128, rows), B.SNN_WS_SUBBIT) == 5 * 2304 + 256
    p = ctypes.c_void_p(256)
    d = B.make_desc(1, 1024, 1024, 1, 1, 1, 32, rows)
    assert B.snn_workspace_bytes(d, B.SNN_WS_SUBBIT) > 4 << 20
    assert L.snn_subbit_conv2d_noalloc(ctypes.byref(d), p, p, p, p, p, None) == B.SNN_ERR_WORKSPACE


def test_the_binding_loads_without_its_native_part(L, monkeypatch):
    """Only a shortcut for the host: without it the library serves every call, and a warning says that it is missing."""
    with monkeypatch.context() as mp:
        mp.setitem(sys.modules, "paper_2110_09195_amd._marshal", None)
        mp.delattr("paper_2110_09195_amd._marshal", raising=False)
        mp.setattr(binding, "_lib", None)
        mp.setattr(binding, "_fast", binding._fast)
        with pytest.warns(RuntimeWarning, match="native part of the binding"):
            assert binding.status_string(0) == "SNN_OK"
        assert binding._fast is None
        with pytest.raises(TypeError):
            binding.snn_subset_update(None, None, 0.0)
    assert binding._fast is not None
