"""Where a combination is formed in FP64 from FP32 data and rounded once, the
GPU's bits against the same expression in numpy."""
import ctypes

import numpy as np
import pytest

import paper_2212_01110_amd as SP
import spock_gen as G
from tests.gpu_util import check, dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _f32(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("tiles", [False, True])
def test_adjoint_combinations_are_formed_in_fp64(tiles):
    # cz = w_z + 2 alpha tz and out = a v + s (la - alpha tz) + c g with the
    # unrounded alpha, rounded once: the launchers of the two halves of an
    # adjoint application on random FP32 data. The FP64 expressions differ from
    # numpy's by their own rounding at most (a fused multiply-add), 1e-16 of the
    # terms: an FP32 result differs only if that crosses a rounding boundary
    inst = G.make_random_small(31, [2, 3, 1], 5, 3, a=0.5)
    gp = SP.Problem.from_instance(inst, precision=SP.FP32)
    assert abs(float(np.float32(gp.alpha)) - gp.alpha) > 1e-9 * gp.alpha
    L = SP.lib()
    vp, ll, dbl, i32 = ctypes.c_void_p, ctypes.c_longlong, ctypes.c_double, ctypes.c_int
    front = L._ZN3spk16launch_adj_frontIfEE10hipError_tRKNS_7ProblemEPKT_S7_xPS5_S8_S8_S8_S8_S8_S8_xibP12ihipStream_t
    back = L._ZN3spk15launch_adj_backIfEE10hipError_tRKNS_7ProblemEdPKT_xdS7_S7_S7_dS7_PS5_xxiP12ihipStream_t
    front.argtypes = [vp, vp, vp, ll, vp, vp, vp, vp, vp, vp, vp, ll, i32, ctypes.c_bool, vp]
    back.argtypes = [vp, dbl, vp, ll, dbl, vp, vp, vp, dbl, vp, vp, ll, ll, i32, vp]
    rng = np.random.default_rng(31)
    B, nn = 2, gp.tree.num_nodes  # (a tile of the shared form holds 16 instances)
    vec = lambda: dev(rng.standard_normal((B, gp.n_v)), torch.float32)  # noqa: E731
    b, w, la, v, g = vec(), vec(), vec(), vec(), vec()
    lb, tz, cz, lo, out = (torch.zeros_like(b) for _ in range(5))
    xb, ub, q = (torch.zeros(16 * nn * m, dtype=torch.float32, device="cuda") for m in (gp.nx, gp.nu, gp.nx))
    p = lambda t: t.data_ptr()  # noqa: E731
    assert front(gp.handle, p(b), p(w), gp.n_v, p(lb), p(tz), p(cz), p(lo), p(xb), p(ub), p(q), gp.n_v, B, tiles, None) == 0
    z = slice(0, gp.n_z)
    hw, ht = _f32(w)[:, z].astype(np.float64), _f32(tz)[:, z].astype(np.float64)
    assert np.count_nonzero(ht) > 0.4 * ht.size
    assert np.array_equal(_f32(cz)[:, z], (hw + 2.0 * gp.alpha * ht).astype(np.float32))
    for a, s, c in ((0.0, 1.0, 1.0), (1.0, -1.0, 0.0)):
        assert back(gp.handle, a, p(v), gp.n_v, s, p(la), p(tz), p(lb), c, p(g), p(out), gp.n_v, gp.n_v, B, None) == 0
        hv, hl, hg = (_f32(t)[:, z].astype(np.float64) for t in (v, la, g))
        assert np.array_equal(_f32(out)[:, z], (a * hv + s * (hl - gp.alpha * ht) + c * hg).astype(np.float32))


@pytest.mark.parametrize("nx,nu,br", [(5, 3, [2, 2, 1]), (20, 10, [2, 1, 2]), (40, 30, [2, 1])])
def test_block_engine_direction_subtracts_its_columns_in_fp64(nx, nu, br):
    # d = -r - gamma (dV - dR) from the FP32 columns dV and dR, subtracted in
    # FP64. With c0 huge every step is K0 (v + d), so the second iterate follows
    # in numpy from the engine's own T(v^0) and T(v^1); T of it must be, bit for
    # bit, what the engine returns after two iterations. gamma's sums differ
    # from numpy's in their order: 1e-16 relative, far below a rounding of d
    inst = G.make_random_small(41, br, nx, nu, a=0.5)
    gp = SP.Problem.from_instance(inst, precision=SP.FP32)
    x0 = dev(0.9 * inst.x0 / max(1.0, np.max(np.abs(inst.x0))), torch.float64)

    def engine(v, iters):
        t = torch.as_tensor(v, device="cuda").clone()
        s = SP.default_settings(eps_abs=1e-30, eps_rel=0.0, max_iters=iters, c0=1e30)
        info, = SP.solve_batched([gp], [x0], [t], s)
        assert info["iters"] == iters and info["t_evals"] == iters + 1
        return _f32(t)

    v0 = np.random.default_rng(nx).standard_normal(gp.n_v).astype(np.float32)
    r0 = v0 - engine(v0, 0)
    v1 = v0 - r0
    T1 = engine(v1, 0)
    assert np.array_equal(T1, engine(v0, 1))
    r1 = v1 - T1
    dV, dR = (v1 - v0).astype(np.float64), (r1 - r0).astype(np.float64)
    gamma = (dR @ r1.astype(np.float64)) / (dR @ dR)
    d1 = (-r1.astype(np.float64) - gamma * (dV - dR)).astype(np.float32)
    v2 = (v1.astype(np.float64) + d1).astype(np.float32)
    assert np.array_equal(engine(v2, 0), engine(v0, 2))


@pytest.mark.parametrize("nx,nu,br", [(1, 1, [5, 1]), (33, 7, [2, 3]), (64, 3, [1, 2]), (2, 1, [70])])
def test_fp32_adjoint_against_fp64_at_dimension_edges(nx, nu, br):
    # the same point v*, cast to FP32, through the FP32 and the FP64 adjoint;
    # adjoint tolerance and bound are those of the FP32 gradients of the 95-node
    # workload (1e-7 and 1e-4)
    inst = G.make_random_small(300 + nx, br, nx, nu, a=0.5, box=50.0)
    g64 = SP.Problem.from_instance(inst, precision=SP.FP64)
    g32 = SP.Problem.from_instance(inst, precision=SP.FP32, alpha=g64.alpha)
    x0 = dev(inst.x0 / np.max(np.abs(inst.x0)), torch.float64)
    v = torch.zeros(g64.n_v, dtype=torch.float64, device="cuda")
    info = g64.solve(x0, v, SP.default_settings(eps_abs=1e-11, eps_rel=1e-11, max_iters=400000))
    assert info["status"] == "converged", info
    ref = g64.backward(v, x0)
    s = SP.default_settings(eps_abs=1e-7, max_iters=400000)
    one = g32.backward(v.float(), x0, settings=s)
    two = SP.backward_batched(g32, [v.float()] * 2, [x0] * 2, settings=s)
    for got in (one, *two):
        assert got[3]["status"] == "converged", got[3]
        for a, b in zip(got[:3], ref[:3]):
            check(f"edge_fp32_adjoint:{nx}", float((a - b).abs().max() / max(1.0, float(b.abs().max()))), 1e-4)
