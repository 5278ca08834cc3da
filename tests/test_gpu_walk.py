"""GPU tests of the walk form of the sweeps (SPOCK_FLOW_WALK fixes it): which
calls run it, every kernel build, and its bounded waits."""
import numpy as np
import pytest

import oracle as O
import paper_2212_01110_amd as SP
import spock_gen as G
from tests.gpu_util import check, dev, host, relerr

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

PREC = {"fp64": (SP.FP64, 1e-12), "fp32": (SP.FP32, 5e-6)}  # the bounds of prox_f and T in the parity tests


@pytest.mark.parametrize("prec", list(PREC))
def test_reported_mapping_is_the_one_that_T_runs(prec, monkeypatch):
    # the resident grids of the two forms differ (four and five wavefronts a
    # SIMD at these dimensions), so the reported grid tells which one it is: in
    # FP32 T keeps the dataflow form, in FP64 it runs the walk form
    monkeypatch.setenv("SPOCK_TEAM", "512")
    inst = G.make_random_small(51, [3, 1, 2], 4, 3)
    x0 = dev(inst.x0, torch.float64)
    grids = {}
    for walk in (None, "51"):
        if walk:
            monkeypatch.setenv("SPOCK_FLOW_WALK", walk)
        gp = SP.Problem.from_instance(inst, precision=PREC[prec][0])
        v = torch.zeros(gp.n_v, dtype=gp.torch_dtype, device="cuda")
        gp.T(v, x0, torch.zeros_like(v))
        got = gp.mapping()
        assert got["mapping"] == 512 and not got["flow_failed"], got
        assert gp.solve(x0, v, SP.default_settings(max_iters=0))["mapping"] == 512
        grids[walk] = got["flow_grid"]
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    assert grids[None] == 5 * ncu
    assert grids["51"] == (4 * ncu if prec == "fp64" else 5 * ncu)
