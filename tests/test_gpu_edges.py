"""GPU parity at the sizes where a kernel's split can go wrong: lane and tile
remainders, the smallest and the largest dimensions, odd families and batches.
References: the oracle on identical inputs, or the one-instance form of the
same call where that form has its own oracle tests."""
import numpy as np
import pytest

import oracle as O
import paper_2212_01110_amd as SP
import spock_gen as G
from tests.gpu_util import check, dev, host

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# one lane per state component: one, a partial, a full wavefront; inputs
# likewise; families of 1 to 5 children, and one wider than a wavefront (the
# separate kernels in place of the fused ones)
@pytest.mark.parametrize("nx,nu,br", [(1, 1, [5, 1]), (33, 7, [2, 3]), (64, 3, [1, 2]), (2, 1, [70])])
def test_adjoint_gradients_at_dimension_edges(nx, nu, br):
    # V's gradients by the batched adjoint (three instances, one of them with
    # no u^0 cotangent given) against the envelope formula at the same v*
    inst = G.make_random_small(300 + nx, br, nx, nu, a=0.5, box=50.0)
    op = O.Problem(inst)
    gp = SP.Problem.from_instance(inst, precision=SP.FP64, alpha=op.alpha)
    x0s = [dev(s * inst.x0 / np.max(np.abs(inst.x0)), torch.float64) for s in (1.0, 0.5, -0.7)]
    vs = []
    for x0 in x0s:
        v = torch.zeros(gp.n_v, dtype=torch.float64, device="cuda")
        info = gp.solve(x0, v, SP.default_settings(eps_abs=1e-11, eps_rel=1e-11, max_iters=400000))
        assert info["status"] == "converged", info
        vs.append(v)
    zero = torch.zeros(nu, dtype=torch.float64, device="cuda")
    got = SP.backward_batched(gp, vs, x0s, gV=1.0, gu0s=[zero, None, zero])
    lv = op.lay.leaves
    for k, (gx, gq, gqN, info) in enumerate(got):
        assert info["status"] == "converged", info
        g = O.envelope_gradients(op, host(vs[k]))
        # the bounds of the oracle comparison of the same gradients in FP64
        check(f"edge_Vx0:{nx}:{k}", np.max(np.abs(host(gx) - g["x0"])) / max(1.0, np.max(np.abs(g["x0"]))), 1e-6)
        check(f"edge_Vq:{nx}:{k}", np.max(np.abs(host(gq)[1:] - g["q"][1:])) / max(1.0, np.max(np.abs(g["q"]))), 1e-6)
        check(f"edge_VqN:{nx}:{k}", np.max(np.abs(host(gqN)[lv] - g["qN"][lv])) / max(1.0, np.max(np.abs(g["qN"]))),
              1e-6)
        assert np.all(host(gq)[0] == 0.0)
        assert np.all(np.delete(host(gqN), lv, axis=0) == 0.0)


# more rows than a wavefront has lanes, single rows, wide and narrow families,
# the largest dimensions; dense costs read the whole vector of a cone block
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,nu,br,nc,ncN,dense", [(64, 64, [2, 1], 70, 130, False), (1, 1, [3, 2], 1, 1, False),
                                                   (5, 2, [11, 1], 64, 65, False), (33, 17, [1, 3], 3, 2, True),
                                                   (64, 2, [2], None, None, True)])
def test_general_operators_at_dimension_edges(nx, nu, br, nc, ncN, dense, prec):
    inst = G.make_random_small(500 + nx + nu, br, nx, nu, a=0.5)
    rng = np.random.default_rng([nx, nu, 5])
    if nc is not None:
        inst.cons = G.random_constraints(rng, inst, nc, ncN, 1.0)
    inst.risk = G.mixture_risk(inst, 0.4)
    if dense:
        inst = G.dense_costs(inst, 3)
    op = O.Problem(inst)
    gp = SP.Problem.from_instance(inst, precision=SP.FP64 if prec == "fp64" else SP.FP32, alpha=op.alpha)
    # rounding of sums of up to n_x + n_u or n_c products: a few hundred units
    # in FP64, and the per-operator FP32 bound of the other parity tests
    tol = 1e-12 if prec == "fp64" else 5e-6
    v = dev(rng.standard_normal(gp.n_v), gp.torch_dtype)
    x0 = dev(inst.x0, torch.float64)
    hv = host(v)
    z, eta = hv[:gp.n_z], hv[gp.n_z:]
    dz, de = v[:gp.n_z].clone(), v[gp.n_z:].clone()
    Lz, Lte, pg, Tv = (torch.zeros(m, dtype=gp.torch_dtype, device="cuda") for m in (gp.n_eta, gp.n_z, gp.n_eta, gp.n_v))
    gp.apply_L(dz, Lz)
    gp.apply_Lt(de, Lte)
    gp.prox_gstar(de, pg)
    stats = gp.T(v, x0, Tv)
    ref_T = O.T_apply(op, hv, inst.x0)
    for tag, got, ref in (("L", Lz, O.L_apply(op.lay, inst, z)), ("Lt", Lte, O.Lt_apply(op.lay, inst, eta)),
                          ("prox", pg, O.prox_gstar(op.lay, inst, eta, op.alpha)), ("T", Tv, ref_T)):
        check(f"edge_gen_{tag}:{nx}:{nu}:{nc}:{prec}", np.max(np.abs(host(got) - ref)) / max(1.0, np.max(np.abs(ref))),
              tol)
    rs = O.residual_stats(op, hv - host(Tv))
    for k in ("xi_p", "xi_d"):
        ref = float(np.max(np.abs(rs[k])))
        check(f"edge_gen_{k}:{nx}:{nu}:{nc}:{prec}", abs(stats[k] - ref) / max(1.0, ref),
              1e-11 if prec == "fp64" else 2e-5)


# teams of 8, 16, 32 and 64 lanes (two components a lane above 64), families
# wider than a team, chains, a tree too large for the LDS form, N = 1; mixed
# with a small tree so that the instances of a launch differ
BLOCK = [(2, 1, [3, 3]), (6, 2, [11, 1]), (9, 7, [2, 2, 1, 1]), (20, 13, [2] * 4 + [1] * 2), (40, 30, [2, 1]),
         (64, 64, [2]), (13, 7, [2] * 9), (3, 3, [70])]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,nu,br", BLOCK)
def test_block_engine_matches_single_solves_at_edges(nx, nu, br, prec):
    insts = [G.make_random_small(700 + nx + len(br), br, nx, nu), G.make_random_small(701, [1, 2], nx, nu),
             G.make_random_small(702, [2], nx, nu)]
    pr = SP.FP64 if prec == "fp64" else SP.FP32
    probs = [SP.Problem.from_instance(i, precision=pr) for i in insts]
    x0s = [dev(0.9 * i.x0 / max(1.0, np.max(np.abs(i.x0))), torch.float64) for i in insts]
    for method, iters in (("cp", 10), ("spock", 4)):
        s = SP.default_settings(eps_abs=1e-30, eps_rel=0.0, max_iters=iters, method=method)
        vs = [torch.zeros(p.n_v, dtype=p.torch_dtype, device="cuda") for p in probs]
        infos = SP.solve_batched(probs, x0s, vs, s)
        for k, p in enumerate(probs):
            ref = torch.zeros(p.n_v, dtype=p.torch_dtype, device="cuda")
            one = p.solve(x0s[k], ref, s)
            assert [infos[k][f] for f in ("iters", "t_evals", "n_k0", "n_k1", "n_k2")] == \
                   [one[f] for f in ("iters", "t_evals", "n_k0", "n_k1", "n_k2")]
            # a few hundred roundings per evaluation of T, grown over the budget
            # of iterations (CP is nonexpansive; SPOCK divides by Gram pivots)
            a, b = host(vs[k]), host(ref)
            tol = {"cp": 1e-12, "spock": 1e-10}[method] if prec == "fp64" else {"cp": 2e-5, "spock": 2e-4}[method]
            check(f"edge_block:{nx}:{nu}:{prec}:{method}:{k}", np.max(np.abs(a - b)) / max(1.0, np.max(np.abs(b))), tol)


# shared-tree form: a batch that pads to two tiles of 16, segments of stages of
# every kind (wide, chains, one stage), teams of 8 to 64 lanes with one or two
# components a lane, a rejected start among the instances
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,nu,br,B", [(2, 1, [2] * 5, 17), (9, 5, [3, 1, 1, 2], 3), (17, 3, [2] * 6 + [1], 16),
                                        (33, 17, [2, 2], 2), (64, 64, [1, 2], 5), (3, 2, [40, 1], 2)])
def test_shared_form_matches_single_solves_at_edges(nx, nu, br, B, prec):
    inst = G.make_random_small(800 + nx, br, nx, nu)
    gp = SP.Problem.from_instance(inst, precision=SP.FP64 if prec == "fp64" else SP.FP32)
    rng = np.random.default_rng([nx, B])
    x0s = [dev(rng.uniform(-1.0, 1.0, nx), torch.float64) for _ in range(B)]
    x0s[B // 2] = dev(np.full(nx, 6.0), torch.float64)  # outside the box
    for method, iters in (("cp", 10), ("spock", 4)):
        s = SP.default_settings(eps_abs=1e-30, eps_rel=0.0, max_iters=iters, method=method)
        vs = [torch.full((gp.n_v,), 0.25, dtype=gp.torch_dtype, device="cuda") for _ in range(B)]
        infos = SP.solve_batched([gp] * B, x0s, vs, s)
        for k in range(B):
            if k == B // 2:
                assert infos[k]["status"] == "rejected" and bool((vs[k] == 0.25).all())
                continue
            ref = torch.full((gp.n_v,), 0.25, dtype=gp.torch_dtype, device="cuda")
            one = gp.solve(x0s[k], ref, s)
            assert [infos[k][f] for f in ("status", "iters", "t_evals", "n_k0", "n_k1", "n_k2", "n_km")] == \
                   [one[f] for f in ("status", "iters", "t_evals", "n_k0", "n_k1", "n_k2", "n_km")]
            a, b = host(vs[k]), host(ref)
            # as for the block engine above
            tol = {"cp": 1e-12, "spock": 1e-10}[method] if prec == "fp64" else {"cp": 2e-5, "spock": 2e-4}[method]
            check(f"edge_shared:{nx}:{nu}:{prec}:{method}:{k}", np.max(np.abs(a - b)) / max(1.0, np.max(np.abs(b))), tol)


# one wavefront per unit: dimensions of one lane, a partial and a full
# wavefront, wide families, in place and out of place
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,nu,br", [(1, 1, [2]), (64, 64, [1, 2]), (33, 5, [3, 1]), (4, 3, [70])])
def test_prox_gstar_at_dimension_edges(nx, nu, br, prec):
    inst = G.make_random_small(900 + nx, br, nx, nu)
    op = O.Problem(inst)
    gp = SP.Problem.from_instance(inst, precision=SP.FP64 if prec == "fp64" else SP.FP32, alpha=op.alpha)
    w = dev(2.0 * np.random.default_rng([nx, 9]).standard_normal(gp.n_eta), gp.torch_dtype)
    out = torch.zeros_like(w)
    ref = O.prox_gstar(op.lay, inst, host(w), op.alpha)
    gp.prox_gstar(w, out)
    tol = 1e-12 if prec == "fp64" else 5e-6  # the per-operator bounds of the parity tests
    check(f"edge_prox:{nx}:{nu}:{prec}", np.max(np.abs(host(out) - ref)) / max(1.0, np.max(np.abs(ref))), tol)
    gp.prox_gstar(w, w)
    assert torch.equal(w, out)


# walk variant of the dataflow sweeps: chains (from a family of one, two and
# several chunks), path pieces over all stages, over some with chunks below,
# several pieces one after the other, dimensions on both sides of the lane
# groups, and grids in which a workgroup runs items of every kind in turn
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("grid", ["1", "3", None])
@pytest.mark.parametrize("walk", [160, 8])
@pytest.mark.parametrize("nx,nu,br", [(3, 2, [2, 2, 2]), (9, 4, [2, 2, 1, 1, 3, 1, 1, 1]), (4, 3, [1, 1, 40, 1, 1]),
                                      (22, 21, [2, 1, 1, 2]), (7, 33, [3, 1, 1]), (64, 64, [1, 1, 2]),
                                      (5, 1, [2] * 9 + [1]), (2, 2, [1] * 30)])
def test_walk_variant_of_the_sweeps(nx, nu, br, walk, grid, prec, monkeypatch):
    monkeypatch.setenv("SPOCK_TEAM", "512")
    monkeypatch.setenv("SPOCK_FLOW_WALK", str(walk))
    if grid:
        monkeypatch.setenv("SPOCK_FLOW_GRID", grid)
    inst = G.make_random_small(1000 + nx, br, nx, nu)
    op = O.Problem(inst)
    gp = SP.Problem.from_instance(inst, precision=SP.FP64 if prec == "fp64" else SP.FP32, alpha=op.alpha)
    rng = np.random.default_rng([nx, nu, walk])
    tol = 1e-12 if prec == "fp64" else 5e-6  # the bounds of prox_f and T in the parity tests
    for k in range(2):
        v = dev(rng.standard_normal(gp.n_v), gp.torch_dtype)
        x0 = dev(inst.x0, torch.float64)
        zo = torch.zeros(op.lay.n_z, dtype=gp.torch_dtype, device="cuda")
        gp.prox_f(v[:op.lay.n_z].contiguous(), x0, zo)
        assert gp.mapping()["mapping"] == 512 and not gp.mapping()["flow_failed"]
        ref = O.prox_f(op.lay, op.inst, op.fac, host(v)[:op.lay.n_z], op.alpha, op.inst.x0)
        check(f"edge_walk:{nx}:{nu}:{walk}:{grid}:{prec}:{k}", np.max(np.abs(host(zo) - ref)) / max(1.0, np.max(np.abs(ref))), tol)
        if prec == "fp64":
            out = torch.zeros_like(v)
            gp.T(v, x0, out)
            ref = O.T_apply(op, host(v), inst.x0)
            check(f"edge_walk_T:{nx}:{nu}:{walk}:{grid}:{k}", np.max(np.abs(host(out) - ref)) / max(1.0, np.max(np.abs(ref))), tol)
