"""Rounds of the shared-tree form: what a call evaluates."""
import time

import numpy as np
import pytest

import paper_2212_01110_amd as SP
import spock_gen as G
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_no_evaluation_after_the_last_instance_ended(prec):
    # the host queues one round past the end: its evaluation of T must not run.
    # A call of k CP iterations evaluates T k + 1 times. On a chain of 300
    # stages an evaluation is over a millisecond of dependent stages and the
    # rest of a call about a tenth of that, so a call of no iteration takes
    # little over one evaluation, and over two if the last round runs too
    inst = G.make_random_small(61, [1] * 300, 3, 2)
    gp = SP.Problem.from_instance(inst, precision=SP.FP64 if prec == "fp64" else SP.FP32)
    x0s = [dev(s * inst.x0 / max(1.0, np.max(np.abs(inst.x0))), torch.float64) for s in (0.5, -0.5)]
    vs = [torch.zeros(gp.n_v, dtype=gp.torch_dtype, device="cuda") for _ in x0s]

    def seconds(iters):
        s = SP.default_settings(eps_abs=1e-30, eps_rel=0.0, max_iters=iters, method="cp")
        got = []
        for _ in range(9):
            torch.cuda.synchronize()
            t = time.perf_counter()
            infos = SP.solve_batched([gp] * 2, x0s, vs, s)
            got.append(time.perf_counter() - t)
            assert [i["t_evals"] for i in infos] == [iters + 1] * 2
        return sorted(got)[len(got) // 2]

    seconds(0)
    t0, t10 = seconds(0), seconds(10)
    evaluation = (t10 - t0) / 10
    assert t0 < 1.6 * evaluation, (t0, evaluation)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,nu,br", [(4, 2, [1] * 9), (20, 10, [2, 2, 1]), (33, 17, [3]), (2, 1, [2, 1] * 2)])
def test_one_launch_of_both_sweeps_gives_the_bits_of_two(nx, nu, br, prec, monkeypatch):
    # a tree of one segment of stages runs both sweeps in one launch; cut in two
    # segments, every sweep is a launch each: the same sums in the same order
    inst = G.make_random_small(62 + nx, br, nx, nu)
    gp = SP.Problem.from_instance(inst, precision=SP.FP64 if prec == "fp64" else SP.FP32)
    x0s = [dev(s * inst.x0 / max(1.0, np.max(np.abs(inst.x0))), torch.float64) for s in np.linspace(-0.9, 0.9, 17)]
    out = {}
    for cut in ("0", "1"):
        monkeypatch.setenv("SPOCK_SH_CUT", cut)
        vs = [torch.full((gp.n_v,), 0.1, dtype=gp.torch_dtype, device="cuda") for _ in x0s]
        s = SP.default_settings(eps_abs=1e-30, eps_rel=0.0, max_iters=5)
        infos = SP.solve_batched([gp] * len(x0s), x0s, vs, s)
        out[cut] = (torch.stack(vs), [i["t_evals"] for i in infos])
    assert out["0"][1] == out["1"][1] and torch.equal(out["0"][0], out["1"][0])
