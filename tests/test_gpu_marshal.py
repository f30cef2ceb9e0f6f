"""The native part of the binding takes the ordinary case of a call and nothing else: it gives what the general part gives, on the current stream, and what
that part refuses is refused with the same error."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2110_09195_amd import binding as B
from paper_2110_09195_amd import synth

pytestmark = pytest.mark.gpu


def _layer(K=32, C_in=32, C_out=40):
    g = np.random.default_rng(5)
    d = B.make_desc(3, C_in, C_out, 9, 11, 2, K, B.SNN_ACT_BIN_ROWS)
    t = {"desc": d, "codebook": torch.from_numpy(synth.codebook(g, K).view(np.int16)).cuda(),
         "idx": torch.from_numpy(synth.indices(g, C_out, C_in, K).astype(np.int16)).cuda(), "alpha": torch.from_numpy(synth.alpha(g, C_out)).cuda(),
         "x4": torch.randn(3, C_in, 9, 11, device="cuda"), "y": torch.empty(3, C_out, 5, 6, device="cuda")}
    t["x"] = B.snn_pack_activations(t["x4"], B.SNN_ACT_BIN_ROWS)
    t["ws"] = B.alloc_workspace(d, B.SNN_WS_SUBBIT)
    return t


def _calls():
    """(name, arguments, position -> arguments that are refused there)"""
    t = _layer()
    d, f32, i32 = t["desc"], torch.zeros(8, device="cuda"), torch.zeros(8, dtype=torch.int32, device="cuda")
    bad_f = [f32.double(), t["alpha"].cpu(), torch.zeros(8, 8, device="cuda").t(), 3, None]
    small_y = [t["y"][:2].contiguous(), t["y"].double(), t["y"].cpu()]
    prepared = B.snn_subbit_prepare(d, t["codebook"], t["idx"], t["alpha"])
    sign = B.snn_subbit_prepare_sign(d, t["codebook"], t["idx"], t["alpha"], t["alpha"])
    out = torch.empty(3 * 40 * 5, dtype=torch.int32, device="cuda")
    yield "snn_subbit_conv2d", [d, t["x"], t["codebook"], t["idx"], t["alpha"], t["y"], t["ws"]], {2: bad_f, 3: bad_f, 4: bad_f, 5: small_y, 6: [t["ws"][:256]]}
    yield "snn_subbit_conv2d_prepared", [d, t["x"], t["alpha"], prepared, t["y"]], {2: bad_f, 3: [prepared[:256]], 4: small_y}
    yield "snn_subbit_conv2d_sign_prepared", [d, t["x"], sign, out], {1: [t["x4"], t["x"].cpu(), None], 2: [sign[:256]], 3: [out[:9].clone(), out.float()]}
    dc = B.make_desc(3, 32, 40, 9, 11, 2, 32, B.SNN_ACT_BIN_CHANNELS)
    xc, packed = B.snn_pack_activations(t["x4"], B.SNN_ACT_BIN_CHANNELS), torch.empty_like(t["x"])
    yield "snn_pack_activations", [t["x4"], B.SNN_ACT_BIN_ROWS, packed], {0: [t["x4"].double(), t["x4"].cpu(), t["x4"].transpose(2, 3)], 1: [7], 2: [packed[:9].clone(), packed.float()]}
    w1 = B.snn_subbit_conv1x1_prepare(dc, torch.arange(32, dtype=torch.int16, device="cuda"), t["idx"][:, :4].contiguous(), t["alpha"])
    yield "snn_subbit_conv1x1_prepared", [dc, xc, w1, t["y"]], {1: [t["x4"], xc.cpu()], 2: [w1[:256]], 3: small_y}
    wb = B.alloc_workspace(dc, B.SNN_WS_BNN)
    B.snn_bnn_prepare(dc, t["idx"], wb)
    yield "snn_bnn_conv2d_prepared", [dc, xc, t["alpha"], wb, t["y"]], {2: bad_f, 3: [wb[:256]], 4: small_y}
    w, g, k = torch.randn(200, 9, device="cuda"), torch.randn(200, 9, device="cuda"), torch.randint(0, 32, (200,), device="cuda").to(torch.int16)
    wp = torch.empty(int(B.lib().snn_project_backward_workspace_bytes(200, 32)), dtype=torch.uint8, device="cuda")
    yield ("snn_project_backward", [w, g, k, 32, torch.empty_like(w), torch.empty(32, 9, device="cuda"), wp],
           {0: [w.double(), w[:9].clone()], 1: [g.cpu(), g[:9].clone()], 2: [k.int(), k[:9].clone()], 3: [0, 513], 4: [w.double()], 5: [w.cpu()], 6: [wp[:256]]})
    p, m = torch.randn(32, 9, device="cuda"), torch.where(torch.randn(32, 9, device="cuda") >= 0, 1, -1).to(torch.int8)
    yield "snn_subset_update", [p, m, 0.3], {0: [p.double(), p.cpu(), p[:9].clone()], 1: [m.int(), m[:9].clone()], 2: [-1.0, float("nan")]}


def _flat(r):
    return [v.clone() for v in (r if isinstance(r, tuple) else (r,))]


def _general(monkeypatch, name, args):
    with monkeypatch.context() as mp:
        mp.setattr(B, "_fast", None)
        try:
            return _flat(getattr(B, name)(*args)), None
        except Exception as e:
            return None, e


def test_native_and_general_calls_agree(monkeypatch):
    for name, args, bad in _calls():
        assert getattr(B._fast, name[4:])(*args), name                  # (the ordinary case is taken)
        native = _flat(getattr(B, name)(*args))
        general, error = _general(monkeypatch, name, args)
        assert error is None and all(torch.equal(a, b) for a, b in zip(native, general)), name
        for at, values in bad.items():
            for v in values:
                wrong = list(args)
                wrong[at] = v
                _, error = _general(monkeypatch, name, wrong)
                assert error is not None, (name, at)
                with pytest.raises(type(error)) as e:
                    getattr(B, name)(*wrong)
                assert str(e.value) == str(error), (name, at)
        if isinstance(args[0], B.snn_conv_desc):                        # a descriptor that is none
            assert not getattr(B._fast, name[4:])(bytes(args[0]), *args[1:])


def test_outputs_that_are_not_given_and_parameters():
    t = _layer()
    y = B.snn_subbit_conv2d(t["desc"], t["x"], t["codebook"], t["idx"], t["alpha"])
    z = B.snn_subbit_conv2d(t["desc"], t["x"], codebook=t["codebook"], idx=t["idx"], alpha=torch.nn.Parameter(t["alpha"]), y=t["y"], workspace=t["ws"])
    assert z is t["y"] and torch.equal(y, z)


def test_the_current_stream():
    t = _layer()
    want = B.snn_subbit_conv2d(t["desc"], t["x"], t["codebook"], t["idx"], t["alpha"], t["y"], t["ws"]).clone()
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        big = torch.empty(1 << 26, device="cuda").fill_(1.0)           # the call is behind this on its stream
        t["x"].copy_(t["x"] ^ 0)
        t["y"].fill_(float("nan"))
        for _ in range(20):
            big.mul_(1.0)
        B.snn_subbit_conv2d(t["desc"], t["x"], t["codebook"], t["idx"], t["alpha"], t["y"], t["ws"])
        got = t["y"].clone()
    side.synchronize()
    assert torch.equal(got, want)


# position of the function's address in _marshal.use
NATIVE = ["snn_subbit_conv2d", "snn_subbit_conv2d_prepared", "snn_subbit_conv2d_sign_prepared", "snn_subbit_conv1x1_prepared",
          "snn_bnn_conv2d_prepared", "snn_pack_activations", "snn_packed_bytes", "snn_project_backward", "snn_subset_update"]


@pytest.mark.parametrize("status, again", [(-4, False), (-77, False), (B.SNN_ERR_INVALID_ARG, True)])
def test_a_failed_launch_is_reported_and_not_repeated(status, again):
    """A library whose functions only count and fail (nothing is launched): after a refusal of the arguments the general part has its say, and
    makes the call with the library proper; after anything else work may be on the stream already, and there is no second call."""
    made = []
    stub = ctypes.CFUNCTYPE(ctypes.c_int)(lambda: made.append(1) or status)          # (arguments it does not look at)
    address = ctypes.cast(stub, ctypes.c_void_p).value
    calls = list(_calls())
    real = [ctypes.cast(getattr(B.lib(), n), ctypes.c_void_p).value for n in NATIVE]
    try:
        for name, args, _ in calls:
            B._fast.use(B.snn_conv_desc, B.SnnError, tuple(address if n == name else r for n, r in zip(NATIVE, real)))
            made.clear()
            if again:
                getattr(B, name)(*args)
            else:
                with pytest.raises(B.SnnError) as e:
                    getattr(B, name)(*args)
                assert e.value.status == status and name in str(e.value)
            assert made == [1], name
    finally:
        B._use(B.lib())
    torch.cuda.synchronize()
