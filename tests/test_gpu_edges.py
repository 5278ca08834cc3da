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
# likewise; families of 1 to 5 children
@pytest.mark.parametrize("nx,nu,br", [(1, 1, [5, 1]), (33, 7, [2, 3]), (64, 3, [1, 2])])
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
