"""Workloads of the SPOCK library as its users run them, with their inputs and reference values.

Eight kinds of call, over trees that branch b ways for `split` stages and then go on as chains to stage N:

  T                one evaluation of the Chambolle-Pock operator with its residual statistics
  operators        L, L*, prox_f and prox_g* one after another (a splitting method of the user's own)
  solve            a budget of iterations of the single-instance solver (CP or SPOCK)
  general          the same with a conic mixture risk and polyhedral constraint rows
  uneven           spock_solve_batched over trees of different shapes
  shared           spock_solve_batched over initial states of one problem
  adjoint          implicit-differentiation gradients of one instance, a budget of Krylov steps
  adjoint_batched  the same for many instances of one problem at once

Solves run a fixed budget of iterations: a converged solution of this problem class is not unique, the iterates are.
`plain` problems and their operators below are written in 64-bit torch from the definitions of z, eta, L, f and g alone.
"""
import math
import random
from types import SimpleNamespace

import numpy as np
import torch

import paper_2212_01110_amd as SP

DEV = "cuda"


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest call: the introductory 15-node tree, one operator evaluation, all latency
        dict(name="T_15n_fp64", kind="T", b=2, split=3, N=3, nx=2, nu=1, fp=64, data="rot"),
        # the largest: the 20 776-node tree (2187 scenarios) whose matrices exceed the caches, FP32 bulk
        dict(name="T_20776n_fp32", kind="T", b=3, split=7, N=15, nx=50, nu=20, fp=32, data="rot"),
        # the operators one by one on the data-centre tree of the closed loop (N 10, 2047 nodes)
        dict(name="operators_2047n_fp32", kind="operators", b=2, split=10, N=10, nx=20, nu=20, fp=32, data="dc"),
        # an ordinary single solve: 223 nodes, n_x 20, n_u 10, SPOCK in FP64
        dict(name="solve_223n_fp64", kind="solve", b=2, split=5, N=10, nx=20, nu=10, fp=64, data="spec", method="spock",
             iters=40),
        # the open-loop scaling series at n_x = n_u = 50 (N = 11, 4095 nodes), CP in FP32
        dict(name="solve_4095n_fp32", kind="solve", b=2, split=11, N=11, nx=50, nu=50, fp=32, data="dc", method="cp",
             iters=12),
        # general risk and polyhedral rows on an odd-sized tree, FP64
        dict(name="general_364n_fp64", kind="general", b=3, split=5, N=5, nx=13, nu=6, nc=9, ncN=7, fp=64, data="rot",
             method="cp", iters=20),
        # 512 uneven trees (n_x 10, n_u 5) in one launch, FP32
        dict(name="uneven_512_fp32", kind="uneven", batch=512, tree_seed=4, nx=10, nu=5, fp=32, method="spock", iters=6),
        # a smaller uneven batch with odd sizes, FP64: fewer instances than compute units
        dict(name="uneven_60_fp64", kind="uneven", batch=60, tree_seed=7, nx=13, nu=7, fp=64, method="spock", iters=8),
        # 64 initial states of one 95-node problem (the differentiation workload's forward), FP32
        dict(name="shared_64x95n_fp32", kind="shared", batch=64, b=2, split=4, N=8, nx=20, nu=10, fp=32, data="rot",
             method="spock", iters=6),
        # one step of the closed loop: 15 realisations of the data-centre model (2047 nodes), FP64
        dict(name="shared_15x2047n_fp64", kind="shared", batch=15, b=2, split=10, N=10, nx=20, nu=20, fp=64, data="dc",
             method="spock", iters=6),
        # the gradient of one 95-node instance (the autograd path), FP64
        dict(name="adjoint_95n_fp64", kind="adjoint", b=2, split=4, N=8, nx=20, nu=10, fp=64, data="rot", iters=32),
        # the gradients of 64 instances of the 95-node problem at once, FP64
        dict(name="adjoint_64x95n_fp64", kind="adjoint_batched", batch=64, b=2, split=4, N=8, nx=20, nu=10, fp=64,
             data="rot", iters=32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_tree(rng, most):
    """A branching, split and horizon with at most `most` nodes, spread over the logarithm of the node count."""
    goal = math.exp(rng.uniform(math.log(12), math.log(most)))
    for _ in range(1000):
        b, N = rng.choice([2, 2, 3, 4, 5]), rng.randint(2, 15)
        split = rng.randint(1, N)
        n = _nodes(b, split, N)
        if n <= most and 0.5 * goal <= n <= 1.5 * goal:
            return dict(b=b, split=split, N=N)
    return dict(b=2, split=3, N=4)


def _nodes(b, split, N):
    n = sum(b ** t for t in range(split + 1))
    return n + (N - split) * b ** split


def draw(rng):
    """A case of the ranges that the listed ones stand for: 12 to 20 776 nodes, n_x 2 to 50, both precisions."""
    kind = rng.choice(["T", "T", "operators", "solve", "general", "uneven", "shared", "adjoint", "adjoint_batched"])
    c = dict(kind=kind, fp=rng.choice([32, 64]))
    nx = _log(rng, 2, 50)
    nu = max(1, min(nx, _log(rng, 1, 32)))
    if kind in ("T", "operators"):
        top = min(20776, int((4.0e8 if kind == "T" else 6e7) / (c["fp"] // 8) / (2 * nx * (nx + nu) + nx)))
        c.update(_draw_tree(rng, max(20, top)), nx=nx, nu=nu, data="rot")
    elif kind in ("solve", "general"):
        nx, nu = min(nx, 30), min(nu, 20)
        c.update(_draw_tree(rng, 600), nx=nx, nu=nu, data="rot", iters=rng.randint(8, 20))
        c["method"] = "cp" if c["fp"] == 32 or kind == "general" else rng.choice(["cp", "spock"])
        if kind == "general":
            c.update(nc=rng.randint(1, 12), ncN=rng.randint(1, 12))
    elif kind == "uneven":
        nx, nu = min(nx, 16), min(nu, 8)
        c.update(batch=_log(rng, 2, 256), tree_seed=rng.randint(10, 10 ** 6), nx=nx, nu=nu, iters=rng.randint(3, 8))
        c["method"] = "cp" if c["fp"] == 32 else "spock"
    elif kind == "shared":
        nx, nu = min(nx, 24), min(nu, 20)
        c.update(_draw_tree(rng, 700), batch=_log(rng, 2, 64), nx=nx, nu=nu, data="rot", iters=rng.randint(4, 12))
        c["method"] = "cp" if c["fp"] == 32 else "spock"
    else:
        nx, nu = min(nx, 20), min(nu, 10)
        c.update(_draw_tree(rng, 220), nx=nx, nu=nu, fp=64, data="rot", iters=rng.randint(15, 30))
        if kind == "adjoint_batched":
            c["batch"] = _log(rng, 2, 40)
    return c


# ------------------------------------------------------------------ inputs
def _anc(b, split, N):
    anc, stage = [np.array([-1])], np.array([0])
    first = 1
    for t in range(N):
        k = b if t < split else 1
        anc.append(np.repeat(stage, k))
        stage = np.arange(first, first + len(anc[-1]))
        first += len(stage)
    return np.concatenate(anc).astype(np.int32)


def _uneven_shapes(case):
    """(split, N) of each tree of an uneven batch: horizons 5 to 12, 2 to 6 branching stages."""
    rng = random.Random(case["tree_seed"])
    out = []
    for _ in range(case["batch"]):
        N = rng.randint(5, 12)
        out.append((min(rng.randint(2, 6), N), N))
    return out


def _orthogonal(g, n, nx):
    """n matrices nx x nx: products of three random reflections."""
    A = torch.eye(nx, dtype=torch.float64, device=DEV).expand(n, nx, nx).contiguous()
    for _ in range(3):
        w = torch.randn(n, nx, 1, generator=g, dtype=torch.float64, device=DEV)
        w = w / w.norm(dim=1, keepdim=True)
        A = A - 2.0 * w * (A * w).sum(1, keepdim=True)
    return A


def _data(case, seed, anc):
    """Dynamics, costs, boxes and risk of the tree `anc`: torch tensors in 64 bits."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (seed + 1) + 17)
    f = dict(dtype=torch.float64, device=DEV)
    nn, nx, nu = len(anc), case["nx"], case["nu"]
    par = torch.as_tensor(anc, device=DEV).long()
    nch = torch.bincount(par[1:], minlength=nn)
    kind = case.get("data", "rot")
    if kind == "dc":  # the data-centre model: tridiagonal A(w), B = I, w the child's place among its siblings
        w = torch.zeros(nn, **f)
        w[1:] = (torch.arange(1, nn, device=DEV) - 1 - (torch.cumsum(nch, 0) - nch)[par[1:]]).double() + 1.0
        j = torch.arange(nx, device=DEV).double()
        A = torch.diag_embed(1.0 + (w[:, None] - 1.0) / 2.0 * (1.0 + j / nx))
        off = 0.01 * torch.ones(nx - 1, **f)
        A = A + torch.diag(off, 1) + torch.diag(off, -1)
        B = torch.eye(nx, **f).expand(nn, nx, nu).contiguous()
        q, r, qN = torch.ones(nn, nx, **f), torch.full((nn, nu), 10.0, **f), torch.ones(nn, nx, **f)
        xb, ub, a = 1.0, 1.5, torch.full((nn,), 0.95, **f)
        cond = torch.where(w == 1.0, 0.3, 0.7).double()
        x0 = 0.2 * torch.rand(case.get("batch", 1), nx, generator=g, **f) - 0.05
    else:
        rad = 0.9 + 0.2 * torch.rand(nn, 1, 1, generator=g, **f)
        A = rad * _orthogonal(g, nn, nx)
        B = torch.randn(nn, nx, nu, generator=g, **f) * (1.0 if kind == "rot" else 1.0 / math.sqrt(nu))
        q = torch.ones(nn, nx, **f) if kind == "rot" else 0.5 + 1.5 * torch.rand(nn, nx, generator=g, **f)
        r, qN = torch.full((nn, nu), 0.1, **f), torch.ones(nn, nx, **f)
        xb, ub = 5.0, 1.0
        a = 0.1 + 0.8 * torch.rand(nn, generator=g, **f)
        wgt = 0.2 + torch.rand(nn, generator=g, **f)
        tot = torch.zeros(nn, **f).index_put_((par[1:],), wgt[1:], accumulate=True).cpu().numpy()
        # the sums again in a fixed order, so that the same seed gives the same bits
        tot = torch.as_tensor(np.bincount(anc[1:], weights=wgt[1:].cpu().numpy(), minlength=nn) + 0.0 * tot, device=DEV)
        cond = wgt / tot[par.clamp(min=0)]
        x0 = 4.0 * torch.rand(case.get("batch", 1), nx, generator=g, **f) - 2.0
    cond[0] = 1.0
    A[0], B[0] = 0.0, 0.0
    prob = cond.cpu().numpy().copy()
    for i in range(1, nn):
        prob[i] *= prob[anc[i]]
    D = SimpleNamespace(anc=anc, prob=prob, nx=nx, nu=nu, A=A, B=B, q=q, r=r, qN=qN, xb=xb, ub=ub, a=a, x0=x0, gen=g,
                        cond=torch.as_tensor(np.where(anc >= 0, prob / prob[np.maximum(anc, 0)], 1.0), device=DEV),
                        kappa=None, cons=None)
    if case["kind"] == "general":
        D.kappa = 0.4
        nc, ncN = case["nc"], case["ncN"]
        G = torch.randn(nn, nc, nx + nu, generator=g, **f)
        G = G / G.norm(dim=2, keepdim=True)
        GN = torch.randn(nn, ncN, nx, generator=g, **f)
        GN = GN / GN.norm(dim=2, keepdim=True)
        bound = 0.5 + torch.rand(nn, 1, generator=g, **f)
        D.cons = SimpleNamespace(Gx=G[:, :, :nx].contiguous(), Gu=G[:, :, nx:].contiguous(), c=bound.expand(nn, nc),
                                 GN=GN, cN=bound.expand(nn, ncN))
    return D


def _handle(case, D, alpha=0.0, tree=None):
    """The factored problem a program keeps."""
    h = lambda t: np.ascontiguousarray(t.cpu().numpy())  # noqa: E731
    nn = len(D.anc)
    risk = cons = None
    if D.kappa is not None:
        fc, nch, _ = _shape(D.anc)
        E, F, b = [None] * nn, [None] * nn, [None] * nn
        kpos = np.zeros(nn, dtype=np.int64)
        p = h(D.cond)
        for i in np.nonzero(nch)[0]:
            n = int(nch[i])
            E[i], F[i] = (m.numpy() for m in _mixture(n, D.kappa))
            b[i] = np.concatenate([np.zeros(n), (1.0 - D.kappa) * p[fc[i]:fc[i] + n], [1.0]])
            kpos[i] = n
        risk = SimpleNamespace(E=E, F=F, b=b, kpos=kpos)
        c, cN = h(D.cons.c), h(D.cons.cN)
        cons = SimpleNamespace(Gx=h(D.cons.Gx), Gu=h(D.cons.Gu), cmin=-c, cmax=c, GN=h(D.cons.GN), cNmin=-cN, cNmax=cN)
    box = lambda m, v: np.full((nn, m), v)  # noqa: E731
    return SP.Problem(tree or SP.Tree(D.anc, D.prob), D.nx, D.nu, h(D.A), h(D.B), h(D.q), h(D.r), h(D.qN),
                      box(D.nx, -D.xb), box(D.nx, D.xb), box(D.nu, -D.ub), box(D.nu, D.ub), h(D.a),
                      SP.FP32 if case["fp"] == 32 else SP.FP64, alpha, risk, cons)


def _tuned(prob, D):
    """The state of a program that has solved before: the first solve of a problem picks its kernels."""
    v = torch.zeros(prob.n_v, dtype=prob.torch_dtype, device=DEV)
    prob.solve(D.x0[0].contiguous(), v, SP.default_settings(max_iters=0))


def _settings(case):
    # tolerances out of reach: the whole budget of iterations runs
    return SP.default_settings(eps_abs=1e-30, eps_rel=0.0, max_iters=case["iters"], method=case.get("method", "spock"))


def _has_exact(case):
    return case["kind"] in ("T", "operators") or case["kind"] in ("solve", "general") and case["method"] == "cp"


def prepare(case, seed):
    kind = case["kind"]
    dt = torch.float32 if case["fp"] == 32 else torch.float64
    if kind == "uneven":
        shapes = _uneven_shapes(case)
        ancs = [_anc(2, k, N) for k, N in shapes]
        # one draw for all trees, then each tree's rows
        off = np.concatenate([[0], np.cumsum([len(a) for a in ancs])])
        flat = np.concatenate([np.where(a < 0, -1, a) for a in ancs]).astype(np.int32)
        g = torch.Generator(device=DEV)
        g.manual_seed(7919 * (seed + 1) + 3)
        f = dict(dtype=torch.float64, device=DEV)
        nn, nx, nu = len(flat), case["nx"], case["nu"]
        rad = 0.9 + 0.2 * torch.rand(nn, 1, 1, generator=g, **f)
        A = (rad * _orthogonal(g, nn, nx)).cpu().numpy()
        B = torch.randn(nn, nx, nu, generator=g, **f).cpu().numpy()
        a = (0.1 + 0.8 * torch.rand(nn, generator=g, **f)).cpu().numpy()
        x0 = torch.randn(len(ancs), nx, generator=g, **f).clamp(-4, 4)
        x0s = [x0[k].clone() for k in range(len(ancs))]
        probs = []
        for k, anc in enumerate(ancs):
            s = slice(off[k], off[k + 1])
            m = len(anc)
            cond = 1.0 / np.bincount(anc[1:], minlength=m)[np.maximum(anc, 0)]
            prob = np.where(anc < 0, 1.0, cond)
            for i in range(1, m):
                prob[i] *= prob[anc[i]]
            box = lambda w, v: np.full((m, w), v)  # noqa: E731
            Ak, Bk = A[s].copy(), B[s].copy()
            Ak[0], Bk[0] = 0.0, 0.0
            probs.append(SP.Problem(SP.Tree(anc, prob), nx, nu, Ak, Bk, box(nx, 1.0), box(nu, 0.1), box(nx, 1.0),
                                    box(nx, -5.0), box(nx, 5.0), box(nu, -1.0), box(nu, 1.0), a[s].copy(),
                                    SP.FP32 if case["fp"] == 32 else SP.FP64))
        # all iterates in one tensor, each at an aligned start
        at = np.concatenate([[0], np.cumsum([-(-p.n_v // 64) * 64 for p in probs])])
        allv = torch.zeros(int(at[-1]), dtype=dt, device=DEV)
        vs = [allv[int(at[k]):int(at[k]) + p.n_v] for k, p in enumerate(probs)]
        return dict(case=case, probs=probs, x0s=x0s, allv=allv, vs=vs, s=_settings(case))
    anc = _anc(case["b"], case["split"], case["N"])
    D = _data(case, seed, anc)
    alpha = Plain(D).alpha if _has_exact(case) else 0.0
    prob = _handle(case, D, alpha)
    st = dict(case=case, prob=prob, x0=D.x0[0].contiguous())
    if kind in ("T", "operators"):
        v = (0.5 * torch.randn(prob.n_v, generator=D.gen, dtype=torch.float64, device=DEV)).to(dt)
        _tuned(prob, D)
        st.update(v=v, Tv=torch.zeros_like(v), z=v[:prob.n_z].clone(), eta=v[prob.n_z:].clone(),
                  Lz=torch.zeros(prob.n_eta, dtype=dt, device=DEV), Lte=torch.zeros(prob.n_z, dtype=dt, device=DEV),
                  pf=torch.zeros(prob.n_z, dtype=dt, device=DEV), pg=torch.zeros(prob.n_eta, dtype=dt, device=DEV))
    elif kind in ("solve", "general"):
        _tuned(prob, D)
        st.update(v=torch.zeros(prob.n_v, dtype=dt, device=DEV), s=_settings(case))
    elif kind == "shared":
        st.update(allv=torch.zeros(case["batch"], -(-prob.n_v // 64) * 64, dtype=dt, device=DEV), s=_settings(case),
                  x0s=[D.x0[k].clone() for k in range(case["batch"])])
        st["vs"] = [st["allv"][k, :prob.n_v] for k in range(case["batch"])]
    else:  # adjoints at the point that 60 plain CP iterations reach
        pl = Plain(D, prob.alpha, D.x0)
        v = torch.zeros(D.x0.shape[0], pl.nz + pl.neta, dtype=torch.float64, device=DEV)
        for _ in range(60):
            v = pl.T(v)
        gu = torch.randn(D.x0.shape[0], case["nu"], generator=D.gen, dtype=torch.float64, device=DEV)
        _tuned(prob, D)
        st.update(vs=[row.to(dt).clone() for row in v], x0s=[x.clone() for x in D.x0], gus=[x.clone() for x in gu],
                  s=SP.default_settings(eps_abs=1e-14, max_iters=case["iters"]))
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "T":
        stats = st["prob"].T(st["v"], st["x0"], st["Tv"])
        return {"Tv": st["Tv"], "stats": stats}
    if kind == "operators":
        p = st["prob"]
        p.apply_L(st["z"], st["Lz"])
        p.apply_Lt(st["eta"], st["Lte"])
        p.prox_f(st["z"], st["x0"], st["pf"])
        p.prox_gstar(st["eta"], st["pg"])
        return {k: st[k] for k in ("Lz", "Lte", "pf", "pg")}
    if kind in ("solve", "general"):  # a cold start, as a program that solves for a new state does
        st["v"].zero_()
        info = st["prob"].solve(st["x0"], st["v"], st["s"])
        return {"v": st["v"], "iters": info["iters"]}
    if kind in ("uneven", "shared"):
        st["allv"].zero_()
        probs = st["probs"] if kind == "uneven" else [st["prob"]] * case["batch"]
        infos = SP.solve_batched(probs, st["x0s"], st["vs"], st["s"])
        return {"v": st["allv"], "iters": np.array([i["iters"] for i in infos])}
    if kind == "adjoint":
        gx, gq, gqN, info = st["prob"].backward(st["vs"][0], st["x0s"][0], 1.0, st["gus"][0], settings=st["s"])
        return {"gx": gx, "gq": gq, "gqN": gqN, "applications": info["iters"]}
    got = SP.backward_batched(st["prob"], st["vs"], st["x0s"], 1.0, st["gus"], settings=st["s"])
    return {"gx": torch.stack([t[0] for t in got]), "gq": torch.stack([t[1] for t in got]),
            "gqN": torch.stack([t[2] for t in got]), "applications": np.array([t[3]["iters"] for t in got])}


# ------------------------------------------------------------------ what a pass cannot do without
def _sizes(anc, nx, nu, nc=None, ncN=None):
    nn = len(anc)
    nl = len(np.unique(anc[1:]))
    nc, ncN = nx + nu if nc is None else nc, nx if ncN is None else ncN
    nz = 1 + nn * nx + nl * nu + 4 * (nn - 1) + nl
    neta = 2 * (nn - 1) + nl * (2 + nc) + (nn - 1) * (nx + nu + 2) + (nn - nl) * (ncN + nx + 2)
    # both sweeps: the dynamics of every child in each, K in each, the inverse and W of every family
    mats = (nn - 1) * 2 * nx * (nx + nu) + nl * (3 * nu * nx + nu * nu)
    return nz, neta, mats


def work(case):
    """Bytes and operations of one pass: the sweeps' matrices once per evaluation of T, v read and T(v) written."""
    kind, e, it = case["kind"], case["fp"] // 8, case.get("iters", 0)
    nx, nu, B = case["nx"], case["nu"], case.get("batch", 1)
    if kind == "uneven":
        got = [_sizes(_anc(2, k, N), nx, nu) for k, N in _uneven_shapes(case)]
        nv, mats = sum(g[0] + g[1] for g in got), sum(g[2] for g in got)
        return {"bytes": float(e * (it + 1) * (mats + 2 * nv)), "flops": float(2 * (it + 1) * mats)}
    nz, neta, mats = _sizes(_anc(case["b"], case["split"], case["N"]), nx, nu, case.get("nc"), case.get("ncN"))
    nv = nz + neta
    if kind == "T":
        return {"bytes": float(e * (mats + 2 * nv)), "flops": float(2 * mats)}
    if kind == "operators":
        return {"bytes": float(e * (mats + 2 * (nz + neta) + 2 * nz + 2 * neta)), "flops": float(2 * mats + 10 * nv)}
    if kind in ("solve", "general", "shared"):
        return {"bytes": float(e * (it + 1) * (mats + 2 * nv * B)), "flops": float(2 * (it + 1) * mats * B)}
    # adjoints: one application of the transposed operator per step, and the Krylov basis of a Gram-Schmidt pass
    return {"bytes": float(e * it * (mats + (2 + it / 2) * nv * B)), "flops": float(it * (2 * mats + 2 * it * nv) * B)}


# ------------------------------------------------------------------ reference in 64 bits
def _shape(anc):
    nn = len(anc)
    nch = np.bincount(anc[1:], minlength=nn)
    fc = 1 + np.cumsum(nch) - nch
    return fc, nch, int((nch > 0).sum())


def _mixture(n, kappa):
    """E and F of the risk (1 - kappa) mean + kappa max."""
    eye, one = torch.eye(n, dtype=torch.float64), torch.ones(1, n, dtype=torch.float64)
    return torch.cat([0 * eye, eye, 0 * one]), torch.cat([-eye, -kappa * eye, one])


class Plain:
    """L, L*, the proximal maps and T of one problem from their definitions; rows of v are instances."""

    def __init__(self, D, alpha=None, x0=None):
        self.D, self.x0 = D, D.x0[:1] if x0 is None else x0
        nn, nx, nu = len(D.anc), D.nx, D.nu
        fc, nch, nl = _shape(D.anc)
        self.nn, self.nl, self.nx, self.nu = nn, nl, nx, nu
        self.nc = nx + nu if D.cons is None else D.cons.Gx.shape[1]
        self.ncN = nx if D.cons is None else D.cons.GN.shape[1]
        t = lambda m: torch.as_tensor(np.asarray(m), device=DEV).long()  # noqa: E731
        i = np.arange(nl)
        self.zU = 1 + nn * nx
        zb = self.zU + nl * nu + 4 * (fc[:nl] - 1) + i
        self.nz = 1 + nn * nx + nl * nu + 4 * (nn - 1) + nl
        e1 = 2 * (fc[:nl] - 1) + i * (2 + self.nc)
        self.eE2 = 2 * (nn - 1) + nl * (2 + self.nc)
        self.eE3 = self.eE2 + (nn - 1) * (nx + nu + 2)
        self.neta = self.eE3 + (nn - nl) * (self.ncN + nx + 2)
        c = np.arange(1, nn)
        par = D.anc[1:]
        k = c - fc[par]
        self.par = t(par)
        self.tau = t(zb[par] + 2 * nch[par] + 1 + k)
        self.s = t(np.concatenate([[0], zb[par] + 3 * nch[par] + 1 + k]))
        self.e1s = t(e1 + 2 * nch[:nl] + 1)
        self.e1c = t((e1 + 2 * nch[:nl] + 2)[:, None] + np.arange(self.nc))
        self.groups = []
        for n in np.unique(nch[:nl]):
            at = np.nonzero(nch[:nl] == n)[0]
            kid = t(fc[at][:, None] + np.arange(n))
            p, one = D.cond[kid], torch.ones(len(at), 1, dtype=torch.float64, device=DEV)
            eye = torch.eye(int(n), dtype=torch.float64, device=DEV).expand(len(at), n, n)
            if D.kappa is None:
                b, kpos = torch.cat([p, 0 * p, one], 1), 2 * n
                Et = torch.cat([D.a[t(at)][:, None, None] * eye, -eye, torch.ones(len(at), n, 1, device=DEV).double()], 2)
                G = torch.cat([Et, -eye, -eye], 2)
            else:
                b, kpos = torch.cat([0 * p, (1.0 - D.kappa) * p, one], 1), n
                E, F = (m.t().to(DEV).expand(len(at), *m.t().shape) for m in _mixture(int(n), D.kappa))
                G = torch.cat([torch.cat([E, -eye, -eye], 2), torch.cat([F, 0 * eye, 0 * eye], 2)], 1)
            Gt = G.transpose(1, 2).contiguous()
            proj = Gt @ torch.linalg.inv((G @ Gt).cpu()).to(DEV) @ G
            self.groups.append(SimpleNamespace(n=int(n), at=t(at), kid=kid, b=b, kpos=int(kpos), proj=proj,
                                               z2=t(zb[at][:, None] + np.arange(4 * n + 1)),
                                               e1=t(e1[at][:, None] + np.arange(2 * n + 1))))
        self.fac = None
        if alpha is None:  # just under 1 / ||L||, by power iteration
            z = torch.ones(1, self.nz, dtype=torch.float64, device=DEV)
            for _ in range(40):
                z = self.Lt(self.L(z))
                z = z / z.norm()
            alpha = round(0.9 / math.sqrt(float(self.Lt(self.L(z)).norm())), 3)
        self.alpha = alpha

    def parts(self, z):
        B = z.shape[0]
        return (z[:, 1:self.zU].reshape(B, self.nn, self.nx),
                z[:, self.zU:self.zU + self.nl * self.nu].reshape(B, self.nl, self.nu))

    def L(self, z):
        D, B, par = self.D, z.shape[0], self.par
        x, u = self.parts(z)
        eta = torch.zeros(B, self.neta, dtype=torch.float64, device=DEV)
        for g in self.groups:
            y = z[:, g.z2[:, :2 * g.n + 1]]
            eta[:, g.e1] = y
            eta[:, self.e1s[g.at]] = z[:, self.s[g.at]] - (g.b * y).sum(2)
        xl, ul = x[:, :self.nl], u
        if D.cons is None:
            eta[:, self.e1c] = torch.cat([xl, ul], 2)
            box = x[:, self.nl:]
        else:
            eta[:, self.e1c] = (D.cons.Gx[:self.nl] * xl[:, :, None]).sum(3) + (D.cons.Gu[:self.nl] * ul[:, :, None]).sum(3)
            box = (D.cons.GN[self.nl:] * x[:, self.nl:, None]).sum(3)
        half = 0.5 * z[:, self.tau][:, :, None]
        eta[:, self.eE2:self.eE3] = torch.cat([D.q[1:].sqrt() * x[:, par], D.r[1:].sqrt() * u[:, par], half, half],
                                              2).reshape(B, -1)
        half = 0.5 * z[:, self.s[self.nl:]][:, :, None]
        eta[:, self.eE3:] = torch.cat([box, D.qN[self.nl:].sqrt() * x[:, self.nl:], half, half], 2).reshape(B, -1)
        return eta

    def Lt(self, eta):
        D, B, nx, nu = self.D, eta.shape[0], self.nx, self.nu
        z = torch.zeros(B, self.nz, dtype=torch.float64, device=DEV)
        e2 = eta[:, self.eE2:self.eE3].reshape(B, self.nn - 1, nx + nu + 2)
        e3 = eta[:, self.eE3:].reshape(B, self.nn - self.nl, self.ncN + nx + 2)
        ec, es = eta[:, self.e1c], eta[:, self.e1s]
        x = torch.zeros(B, self.nn, nx, dtype=torch.float64, device=DEV)
        if D.cons is None:
            xl, ul, box = ec[:, :, :nx].clone(), ec[:, :, nx:].clone(), e3[:, :, :nx]
        else:
            xl, ul = ((m[:self.nl] * ec[:, :, :, None]).sum(2) for m in (D.cons.Gx, D.cons.Gu))
            box = (D.cons.GN[self.nl:] * e3[:, :, :self.ncN, None]).sum(2)
        wx, wu = D.q[1:].sqrt() * e2[:, :, :nx], D.r[1:].sqrt() * e2[:, :, nx:nx + nu]
        for g in self.groups:
            xl[:, g.at] += wx[:, g.kid - 1].sum(2)
            ul[:, g.at] += wu[:, g.kid - 1].sum(2)
            z[:, g.z2[:, :2 * g.n + 1]] = eta[:, g.e1] - g.b * es[:, g.at][:, :, None]
        x[:, :self.nl] = xl
        x[:, self.nl:] = box + D.qN[self.nl:].sqrt() * e3[:, :, self.ncN:self.ncN + nx]
        z[:, 1:self.zU] = x.reshape(B, -1)
        z[:, self.zU:self.zU + self.nl * nu] = ul.reshape(B, -1)
        z[:, self.tau] = 0.5 * (e2[:, :, nx + nu] + e2[:, :, nx + nu + 1])
        z[:, self.s[:self.nl]] = es
        z[:, self.s[self.nl:]] = 0.5 * (e3[:, :, -2] + e3[:, :, -1])
        return z

    def stages(self):
        fc, nch, _ = _shape(self.D.anc)
        out, lo, hi = [], 0, 1
        while lo < self.nl:
            n = int(nch[lo])
            out.append((lo, hi, n))
            lo, hi = hi, hi + (hi - lo) * n
        return out

    def factor(self):
        """K, the inverse of I + sum B'PB, and P of every node, from the leaves up."""
        D, nx = self.D, self.nx
        P = torch.eye(nx, dtype=torch.float64, device=DEV).repeat(self.nn, 1, 1)
        K = torch.zeros(self.nl, self.nu, nx, dtype=torch.float64, device=DEV)
        Ri = torch.zeros(self.nl, self.nu, self.nu, dtype=torch.float64, device=DEV)
        eye = torch.eye(self.nu, dtype=torch.float64, device=DEV)
        for lo, hi, n in reversed(self.stages()):
            m, kid = hi - lo, slice(hi, hi + (hi - lo) * n)
            A, B = D.A[kid], D.B[kid]
            Bt = B.transpose(1, 2).contiguous()
            BtP = Bt @ P[kid]
            R = eye + (BtP @ B).reshape(m, n, self.nu, self.nu).sum(1)
            Ri[lo:hi] = torch.linalg.inv(R.cpu()).to(DEV)
            K[lo:hi] = -(Ri[lo:hi] @ (BtP @ A).reshape(m, n, self.nu, nx).sum(1))
            Ab = A + B @ K[lo:hi].repeat_interleave(n, 0)
            Kt = K[lo:hi].transpose(1, 2).contiguous()
            P[lo:hi] += Kt @ K[lo:hi] + (Ab.transpose(1, 2).contiguous() @ (P[kid] @ Ab)).reshape(m, n, nx, nx).sum(1)
        self.fac = (K, Ri, P)

    def prox_f(self, zh):
        """The cost's shift of s^0, the dynamics' projection and the risk blocks' projection."""
        if self.fac is None:
            self.factor()
        D, B = self.D, zh.shape[0]
        K, Ri, P = self.fac
        xh, uh = self.parts(zh)
        mv = lambda M, v: (M @ v.unsqueeze(-1)).squeeze(-1)  # noqa: E731
        q = -xh.clone()
        d = torch.zeros_like(uh)
        At, Bt = D.A.transpose(1, 2).contiguous(), D.B.transpose(1, 2).contiguous()
        for lo, hi, n in reversed(self.stages()):
            m, kid = hi - lo, slice(hi, hi + (hi - lo) * n)
            d[:, lo:hi] = mv(Ri[lo:hi], uh[:, lo:hi] - mv(Bt[kid], q[:, kid]).reshape(B, m, n, -1).sum(2))
            dk = d[:, lo:hi].repeat_interleave(n, 1)
            q[:, lo:hi] += mv(At[kid], mv(P[kid], mv(D.B[kid], dk)) + q[:, kid]).reshape(B, m, n, -1).sum(2)
        x, u = torch.zeros_like(xh), torch.zeros_like(uh)
        x[:, 0] = self.x0
        for lo, hi, n in self.stages():
            kid = slice(hi, hi + (hi - lo) * n)
            u[:, lo:hi] = mv(K[lo:hi], x[:, lo:hi]) + d[:, lo:hi]
            x[:, kid] = mv(D.A[kid], x[:, lo:hi].repeat_interleave(n, 1)) + mv(D.B[kid], u[:, lo:hi].repeat_interleave(n, 1))
        z = zh.clone()
        z[:, 1:self.zU] = x.reshape(B, -1)
        z[:, self.zU:self.zU + self.nl * self.nu] = u.reshape(B, -1)
        for g in self.groups:
            w = zh[:, g.z2]
            z[:, g.z2] = w - mv(g.proj, w)
        z[:, 0] = zh[:, 0] - self.alpha
        return z

    def _soc(self, w):
        """w - alpha proj(w / alpha) on the cone |vector| <= t shifted by (0, 1/2, -1/2)."""
        al = self.alpha
        p = w / al
        p[:, :, -2] -= 0.5
        p[:, :, -1] += 0.5
        nrm, t = p[:, :, :-1].norm(dim=2, keepdim=True), p[:, :, -1:]
        c = 0.5 * (nrm + t)
        edge = torch.cat([p[:, :, :-1] * (c / nrm.clamp(min=1e-300)), c], 2)
        r = torch.where(nrm <= t, p, torch.where(nrm <= -t, 0 * p, edge))
        r[:, :, -2] += 0.5
        r[:, :, -1] -= 0.5
        return w - al * r

    def prox_gstar(self, w):
        D, B, al = self.D, w.shape[0], self.alpha
        out = torch.zeros_like(w)
        for g in self.groups:
            y = w[:, g.e1]
            out[:, g.e1[:, :g.kpos]] = y[:, :, :g.kpos].clamp(max=0.0)
        out[:, self.e1s] = w[:, self.e1s].clamp(max=0.0)
        if D.cons is None:
            hi = torch.cat([torch.full((self.nx,), D.xb), torch.full((self.nu,), D.ub)]).double().to(DEV)
            hiN = torch.full((self.nx,), D.xb, dtype=torch.float64, device=DEV)
        else:
            hi, hiN = D.cons.c[:self.nl], D.cons.cN[self.nl:]
        clip = lambda v, h: v - al * torch.minimum(torch.maximum(v / al, -h), h)  # noqa: E731
        out[:, self.e1c] = clip(w[:, self.e1c], hi)
        e2 = w[:, self.eE2:self.eE3].reshape(B, self.nn - 1, -1)
        e3 = w[:, self.eE3:].reshape(B, self.nn - self.nl, -1)
        out[:, self.eE2:self.eE3] = self._soc(e2).reshape(B, -1)
        out[:, self.eE3:] = torch.cat([clip(e3[:, :, :self.ncN], hiN), self._soc(e3[:, :, self.ncN:])], 2).reshape(B, -1)
        return out

    def T(self, v):
        z, eta = v[:, :self.nz], v[:, self.nz:]
        zp = self.prox_f(z - self.alpha * self.Lt(eta))
        return torch.cat([zp, self.prox_gstar(eta + self.alpha * self.L(2.0 * zp - z))], 1)

    def stats(self, v, Tv):
        r, al = v - Tv, self.alpha
        rz, re = r[:, :self.nz], r[:, self.nz:]
        Lrz = self.L(rz)
        rz2, re2, cross = float((rz * rz).sum()), float((re * re).sum()), float((re * Lrz).sum())
        return dict(xi_p=float((rz / al - self.Lt(re)).abs().max()), xi_d=float((re / al - Lrz).abs().max()),
                    omega2=rz2 + re2 - 2.0 * al * cross, rz2=rz2, re2=re2, cross=cross)


def exact(case, seed):
    """What run() returns, by the plain operators in 64 bits; None for the accelerated solves and the adjoints."""
    if not _has_exact(case):
        return None
    D = _data(case, seed, _anc(case["b"], case["split"], case["N"]))
    pl = Plain(D)
    dt = torch.float32 if case["fp"] == 32 else torch.float64
    if case["kind"] in ("T", "operators"):
        v = (0.5 * torch.randn(pl.nz + pl.neta, generator=D.gen, dtype=torch.float64, device=DEV)).to(dt).double()[None]
        z, eta = v[:, :pl.nz], v[:, pl.nz:]
        if case["kind"] == "T":
            Tv = pl.T(v)
            return {"Tv": Tv[0], "stats": pl.stats(v, Tv)}
        return {"Lz": pl.L(z)[0], "Lte": pl.Lt(eta)[0], "pf": pl.prox_f(z)[0], "pg": pl.prox_gstar(eta)[0]}
    v = torch.zeros(1, pl.nz + pl.neta, dtype=torch.float64, device=DEV)
    for _ in range(case["iters"] + 1):  # the solver returns T of its last iterate
        v = pl.T(v)
    return {"v": v[0], "iters": None}
