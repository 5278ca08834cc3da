"""Calls on one problem from several streams."""
import ctypes

import numpy as np
import pytest

import paper_2212_01110_amd as SP
import spock_gen as G
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_calls_without_waits_on_two_blocking_streams(prec, monkeypatch):
    # per-stage sweeps: T without statistics and prox_f return while their work
    # is queued. Two of them on two blocking streams, both held back until both
    # are queued or the library waits, share the problem's workspace: the second
    # runs after the first
    monkeypatch.setenv("SPOCK_TEAM", "8")
    inst = G.make_random_small(71, [1] * 80, 3, 2)
    gp = SP.Problem.from_instance(inst, precision=SP.FP64 if prec == "fp64" else SP.FP32)
    x0 = dev(inst.x0, torch.float64)
    rng = np.random.default_rng(71)
    v = [dev(rng.standard_normal(gp.n_v), gp.torch_dtype) for _ in range(2)]
    zin = v[1][:gp.n_z].contiguous()

    def first(out):
        gp.T(v[0], x0, out[0], want_stats=False)

    def second(out):
        gp.prox_f(zin, x0, out[1])
        gp.T(v[1], x0, out[2], want_stats=False)

    def buffers():
        return [torch.zeros(m, dtype=gp.torch_dtype, device="cuda") for m in (gp.n_v, gp.n_z, gp.n_v)]

    want = buffers()
    first(want)
    second(want)
    torch.cuda.synchronize()
    assert gp.mapping()["mapping"] == 8
    hip = ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))
    handles = [ctypes.c_void_p() for _ in range(2)]
    for h in handles:
        assert hip.hipStreamCreate(ctypes.byref(h)) == 0
    a, b = (torch.cuda.ExternalStream(h.value) for h in handles)
    gate = torch.cuda.Stream()
    for _ in range(3):
        got = buffers()
        torch.cuda.synchronize()
        with torch.cuda.stream(gate):
            torch.cuda._sleep(20_000_000)
            ready = gate.record_event()
        a.wait_event(ready)
        b.wait_event(ready)
        with torch.cuda.stream(a):
            first(got)
        with torch.cuda.stream(b):
            second(got)
        torch.cuda.synchronize()
        assert all(torch.equal(g, w) for g, w in zip(got, want))
    torch.cuda.synchronize()
    for h in handles:
        assert hip.hipStreamDestroy(h) == 0
