"""Where a combination is formed in FP64 from FP32 data and rounded once, the
GPU's bits against the same expression in numpy."""
import ctypes

import numpy as np
import pytest

import paper_2212_01110_amd as SP
import spock_gen as G
from tests.gpu_util import dev

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
