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


# the kernel builds that the other walk tests do not force: five rows a
# wavefront, 13 with two slots, 16 with one, 13 with one at its edge. A chain, a
# family of several chunks and path pieces in each; T and its statistics in
# both precisions as a solve of no iteration returns them
@pytest.mark.parametrize("prec", list(PREC))
@pytest.mark.parametrize("walk", ["160", "51"])
@pytest.mark.parametrize("nx,nu", [(20, 10), (13, 1), (50, 50), (33, 32), (60, 4), (52, 12)])
def test_walk_kernel_builds(nx, nu, walk, prec, monkeypatch):
    monkeypatch.setenv("SPOCK_TEAM", "512")
    monkeypatch.setenv("SPOCK_FLOW_WALK", walk)
    inst = G.make_random_small(1100 + nx, [1, 2, 9, 1, 1], nx, nu)
    inst.x0 = 0.9 * inst.x0 / max(1.0, np.max(np.abs(inst.x0)))
    op = O.Problem(inst)
    gp = SP.Problem.from_instance(inst, precision=PREC[prec][0], alpha=op.alpha)
    tol = PREC[prec][1]
    v = dev(np.random.default_rng([nx, nu]).standard_normal(gp.n_v), gp.torch_dtype)
    hv = host(v)
    x0 = dev(inst.x0, torch.float64)
    zo = torch.zeros(gp.n_z, dtype=gp.torch_dtype, device="cuda")
    gp.prox_f(v[:gp.n_z].contiguous(), x0, zo)
    check(f"walk_build_prox_f:{nx}:{nu}:{walk}:{prec}",
          relerr(host(zo), O.prox_f(op.lay, inst, op.fac, hv[:gp.n_z], op.alpha, inst.x0)), tol)
    Tv = v.clone()
    info = gp.solve(x0, Tv, SP.default_settings(max_iters=0))
    assert info["t_evals"] == 1 and info["mapping"] == 512 and not info["flow_fallback"], info
    ref = O.T_apply(op, hv, inst.x0)
    check(f"walk_build_T:{nx}:{nu}:{walk}:{prec}", relerr(host(Tv), ref), tol)
    rs = O.residual_stats(op, hv - ref)
    xi = max(float(np.max(np.abs(rs["xi_p"]))), float(np.max(np.abs(rs["xi_d"]))))
    # xi = r / alpha - L r of the residual: four times the bound of T
    check(f"walk_build_xi:{nx}:{nu}:{walk}:{prec}", abs(info["xi0"] - xi) / max(1.0, xi), 4 * tol)


@pytest.mark.parametrize("prec", list(PREC))
@pytest.mark.parametrize("walk,lds", [("51", None), ("0", "4096"), ("160", "16384")])
def test_walk_give_up_falls_back_to_per_stage_form(walk, lds, prec, monkeypatch):
    # SPOCK_FLOW_SPIN=0: every bounded wait gives up at once, its values zero and
    # the results finite, and every kernel ends normally. Each call has to find
    # the error word, switch the problem to the per-stage form and evaluate
    # again. Chains, path pieces, chunks whose last one waits for partial sums
    inst = G.make_random_small(64, [2, 1, 12, 1], 4, 3, a=0.3, box=50.0)
    inst.x0 = 0.9 * inst.x0 / max(1.0, np.max(np.abs(inst.x0)))
    op = O.Problem(inst)
    x0 = dev(inst.x0, torch.float64)
    pr, tol = PREC[prec]
    eps = 1e-11 if prec == "fp64" else 1e-6
    free = SP.Problem.from_instance(inst, precision=pr, alpha=op.alpha)
    vs = torch.zeros(free.n_v, dtype=free.torch_dtype, device="cuda")
    want = free.solve(x0, vs, SP.default_settings(eps_abs=eps, eps_rel=eps, max_iters=400000))
    aset = SP.default_settings(eps_abs=1e-12 if prec == "fp64" else 1e-7, max_iters=400000)
    want_g = free.backward(vs, x0, settings=aset)
    assert want["status"] == "converged" and want_g[3]["status"] == "converged"
    monkeypatch.setenv("SPOCK_TEAM", "512")
    monkeypatch.setenv("SPOCK_FLOW_WALK", walk)
    monkeypatch.setenv("SPOCK_FLOW_SPIN", "0")
    if lds:
        monkeypatch.setenv("SPOCK_FLOW_LDS", lds)

    def fresh():
        return SP.Problem.from_instance(inst, precision=pr, alpha=op.alpha)

    def gave_up(gp):
        got = gp.mapping()
        assert got == {"mapping": 256, "flow_grid": 0, "flow_failed": True}, got

    rng = np.random.default_rng(64)
    v = dev(rng.standard_normal(free.n_v), free.torch_dtype)
    hv = host(v)
    gp = fresh()
    zo = torch.zeros(gp.n_z, dtype=gp.torch_dtype, device="cuda")
    gp.prox_f(v[:gp.n_z].contiguous(), x0, zo)
    gave_up(gp)
    check(f"walk_giveup_prox_f:{walk}:{prec}",
          relerr(host(zo), O.prox_f(op.lay, inst, op.fac, hv[:gp.n_z], op.alpha, inst.x0)), tol)
    ref = O.T_apply(op, hv, inst.x0)
    for stats in (True, False):
        gp = fresh()
        Tv = torch.zeros_like(v)
        st = gp.T(v, x0, Tv, want_stats=stats)
        gave_up(gp)
        assert st is None or all(np.isfinite(list(st.values())))
        check(f"walk_giveup_T:{walk}:{prec}:{stats}", relerr(host(Tv), ref), tol)
    gp = fresh()
    got = torch.zeros_like(v)
    info = gp.solve(x0, got, SP.default_settings(eps_abs=eps, eps_rel=eps, max_iters=400000))
    gave_up(gp)
    assert info["flow_fallback"] == 1 and info["mapping"] == 256 and info["status"] == "converged", info
    # two solves of a convex problem to eps: the bound of the other give-up test
    check(f"walk_giveup_solve:{walk}:{prec}", abs(info["V_s0"] - want["V_s0"]) / max(1, abs(want["V_s0"])), 1e-4)
    gp = fresh()
    g = gp.backward(vs, x0, settings=aset)
    gave_up(gp)
    assert g[3]["flow_fallback"] == 1 and g[3]["status"] == "converged", g[3]
    for a, b in zip(g[:3], want_g[:3]):
        check(f"walk_giveup_backward:{walk}:{prec}", float((a - b).abs().max() / max(1.0, float(b.abs().max()))),
              1e-6 if prec == "fp64" else 1e-4)
