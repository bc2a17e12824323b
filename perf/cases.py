"""The framework's calls whose speed matters, as cases to be timed and compared.

A case is one pass through a public entry point of the real-valued path
(`binding.Context`: one cycle, one refinement step, a training step, a whole
solve, a serving round, flexible GMRES) or of the complex Helmholtz path
(`helmholtz.HelmholtzContext`: one cycle, flexible GMRES), at the sizes of the
repository's own workloads: the 33 x 33 Poisson problem, the block-diffusion
problems on 65 .. 1025 points per side that are served and trained on, and the
257 x 257 Helmholtz problem.  `exact` evaluates the same method in 64 bits
with plain torch gathers.
"""
from __future__ import annotations

import ctypes
import functools
import os

import numpy as np
import torch

import paper_2608_29082_amd
from paper_2608_29082_amd import binding
from paper_2608_29082_amd import helmholtz as hz

DEV = "cuda:0"
THETA = os.path.join(os.path.dirname(os.path.abspath(paper_2608_29082_amd.__file__)), "theta")
SERVED = (65, 129, 257, 513, 1025)      # sides with shipped parameters of the serving distribution
PI = float(np.pi)


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # one FP64 cycle on the smallest problem, one right-hand side: nothing but launches
        dict(name="vcycle_33_fp64", kind="vcycle", side=33, coarsest=3, nrhs=1, K=2, prec="fp64", agg="mean",
             basis="monomial", nu=2),
        # one outer iteration of the smallest served request
        dict(name="refine_65_b1", kind="refine", side=65, coarsest=3, nrhs=1, K=3, prec="fp32", agg="mean",
             basis="monomial", nu=2),
        # the headline workload's outer iteration: 64 right-hand sides of one operator
        dict(name="refine_513_b64", kind="refine", side=513, coarsest=3, nrhs=64, K=3, prec="fp32", agg="mean",
             basis="monomial", nu=2),
        # a preconditioner application on the largest served grid, BF16 intermediates
        dict(name="vcycle_1025_bf16_b16", kind="vcycle", side=1025, coarsest=3, nrhs=16, K=3, prec="bf16", agg="mean",
             basis="monomial", nu=2),
        # the ChebConv form in FP64 on a grid and a batch that are no powers of two, more smoothing steps
        dict(name="vcycle_385_sym_fp64_b7", kind="vcycle", side=385, coarsest=5, nrhs=7, K=3, prec="fp64", agg="sym",
             basis="chebyshev", nu=3),
        # training on the 257 workload: two unrolled steps, the loss and the whole reverse sweep
        dict(name="train_257_b32", kind="train", side=257, coarsest=3, nrhs=32, K=3, prec="fp32", agg="mean",
             basis="monomial", nu=2),
        # the same on a small grid with a ragged batch, as in a first search for parameters
        dict(name="train_81_b10", kind="train", side=81, coarsest=4, nrhs=10, K=3, prec="fp32", agg="mean",
             basis="monomial", nu=2),
        # one served request on its own: the whole solve to 1e-8 with the shipped parameters
        dict(name="solve_257_b1", kind="solve", side=257, coarsest=3, nrhs=1, K=3, prec="fp32", agg="mean",
             basis="monomial", nu=2),
        # a round of continuous batching: 32 requests, each with its own operator, eight cycles
        dict(name="round_257_b32", kind="round", side=257, coarsest=3, nrhs=32, K=3, prec="fp32", agg="mean",
             basis="monomial", nu=2),
        # flexible GMRES around the learned cycle to 1e-8
        dict(name="fgmres_129_b16", kind="fgmres", side=129, coarsest=3, nrhs=16, K=3, prec="fp32", agg="mean",
             basis="monomial", nu=2),
        # one Helmholtz cycle of the paper's 257 x 257 problem, 16 sources, trained parameters
        dict(name="helm_cycle_257_b16", kind="hcycle", side=257, k=16 * PI, levels=5, nrhs=16, K=1, prec="fp32"),
        # the Helmholtz solve by flexible GMRES at half the wave number, FP64 cycles, an odd batch
        dict(name="helm_fgmres_129_b5", kind="hfgmres", side=129, k=8 * PI, levels=5, nrhs=5, K=1, prec="fp64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _side(rng, lo, hi):
    """(side, coarsest) of a grid that coarsens to coarsest x coarsest interior points."""
    all_ = [((c + 1) * 2 ** k + 1, c) for c in (3, 4, 5, 6) for k in range(2, 9)]
    want = lo * (hi / lo) ** rng.random()
    return min((s for s in all_ if lo <= s[0] <= hi), key=lambda s: abs(np.log(s[0] / want)))


def draw(rng):
    kind = rng.choice(["vcycle", "refine", "refine", "train", "solve", "round", "fgmres", "hcycle", "hfgmres"])
    if kind in ("vcycle", "refine", "train"):
        side, c = _side(rng, 33, {"vcycle": 1025, "refine": 1025, "train": 257}[kind])
        top = {"vcycle": 1025 ** 2 * 16, "refine": 513 ** 2 * 64, "train": 257 ** 2 * 32}[kind]
        nrhs = _log_int(rng, 1, max(1, min(64, top // side ** 2)))
        if nrhs > 8 and rng.random() < 0.5:
            nrhs = nrhs // 16 * 16 or 16     # batches are mostly laid out in sixteens
            nrhs = min(nrhs, max(1, top // side ** 2))
        agg, basis = rng.choice([("mean", "monomial")] * 4 + [("weighted", "monomial"), ("sym", "chebyshev")])
        prec = "fp32" if kind != "vcycle" else rng.choice(["fp64", "fp32", "bf16"])
        return dict(kind=kind, side=side, coarsest=c, nrhs=nrhs, K=rng.choice([1, 2, 3, 3, 4]), prec=prec, agg=agg,
                    basis=basis, nu=rng.choice([1, 2, 2, 3]))
    base = dict(coarsest=3, K=3, prec="fp32", agg="mean", basis="monomial", nu=2)
    if kind == "solve":
        return dict(kind=kind, side=rng.choice([65, 129, 257]), nrhs=_log_int(rng, 1, 4), **base)
    if kind == "round":
        return dict(kind=kind, side=rng.choice([65, 129, 257]), nrhs=_log_int(rng, 4, 32), **base)
    if kind == "fgmres":
        return dict(kind=kind, side=rng.choice([65, 129]), nrhs=_log_int(rng, 1, 16), **base)
    side, k = rng.choice([(65, 4 * PI), (129, 8 * PI)] + ([(257, 16 * PI)] if kind == "hcycle" else []))
    nrhs = _log_int(rng, 1, 16 if kind == "hcycle" else 5)
    return dict(kind=kind, side=side, k=k, levels=5 if side > 65 else 4, nrhs=nrhs, K=1,
                prec=rng.choice(["fp32", "fp64"]) if kind == "hcycle" else "fp64")


# ------------------------------------------------------------------ inputs
def _blocks(rng):
    """Block coefficient of the served and trained-on problems: log10 a ~ U(-2, 2) on 16 x 16 blocks."""
    return 10.0 ** rng.uniform(-2.0, 2.0, (16, 16))


def _params(case, J, rng):
    """The shipped parameters where the case solves with them, else a draw near the identity initialisation."""
    K = case["K"]
    if case["kind"] in ("solve", "round", "fgmres"):
        return np.load(os.path.join(THETA, "k3_serving%d.npy" % case["side"])).ravel()
    p = np.zeros((J - 1, 2 + 3 * (K + 1)))
    p[:, 0] = rng.uniform(0.5, 0.7, J - 1)
    p[:, 1] = rng.uniform(0.9, 1.1, J - 1)
    for q in range(3):
        o = 2 + q * (K + 1)
        p[:, o] = rng.uniform(0.9, 1.1, J - 1)
        p[:, o + 1:o + K + 1] = rng.uniform(-0.15, 0.15, (J - 1, K))
    return p.ravel()


def _problem(case, seed):
    """The host side of a case: hierarchies (one, or one per column), parameters, right-hand sides, first iterate."""
    rng = np.random.default_rng([int(seed), case["side"], case["nrhs"]])
    many = case["nrhs"] if case["kind"] == "round" else 1
    hiers = [binding.SquareHierarchy(case["side"], _blocks(rng), case["coarsest"]) for _ in range(many)]
    n, B = hiers[0].sizes[0], case["nrhs"]
    prm = _params(case, hiers[0].nlevels, rng)
    f = rng.standard_normal((n, B))
    u0 = 0.1 * rng.standard_normal((n, B)) if case["kind"] in ("vcycle", "refine") else np.zeros((n, B))
    return hiers, prm, f, u0


@functools.lru_cache(maxsize=4)
def _helmholtz(side, k, levels):
    from mginputs import helmholtz as H
    h = H.hierarchy(side, k, levels)
    return h, H.smoother_plan(h), H.matrices(side)[1], H.mesh(side)[0]


def _helm_problem(case, seed):
    from mginputs import helmholtz as H
    h, plan, mass, pts = _helmholtz(case["side"], case["k"], case["levels"])
    rng = np.random.default_rng([int(seed), case["side"], case["nrhs"]])
    B, J, K = case["nrhs"], case["levels"], case["K"]
    cols = H.source_centres(B + 2, rng)[2:] if seed % 2 else H.source_centres(B, rng)
    cols = [[(x + 0.01 * rng.standard_normal(), y + 0.01 * rng.standard_normal()) for x, y in c] for c in cols]
    f = (mass @ np.stack([H.disk_source(pts, c) for c in cols], axis=1)).astype(np.complex128)
    if J == 5:
        prm = np.load(os.path.join(THETA, "hz_k1_helmholtz257.npy")).ravel()
        if case["kind"] == "hfgmres":
            prm = _helm_identity(J, K, plan)
    else:
        prm = _helm_identity(J, K, plan)
    return h, plan, prm, f


def _helm_identity(J, K, plan):
    per = 2 + 4 * (K + 1)
    lv = np.zeros((J - 1, per))
    lv[:, 0] = [2.0 / 3.0 if p[0] == "jacobi" else 0.0 for p in plan]
    lv[:, 1] = 1.0
    lv[:, 2] = lv[:, 5] = 1.0
    sh = np.zeros(4 * (K + 1))
    sh[0] = sh[3] = 1.0
    return np.concatenate([lv.ravel(), sh, sh])


def prepare(case, seed):
    if case["kind"] in ("hcycle", "hfgmres"):
        h, plan, prm, f = _helm_problem(case, seed)
        K = case["K"]
        ctx = hz.HelmholtzContext(h.A, h.P, prm, K, K, K, plan, precision=case["prec"], nrhs=case["nrhs"])
        dt = ctx.cycle_dtype if case["kind"] == "hcycle" else torch.complex128
        fd = torch.tensor(f, device=DEV).to(dt)
        return dict(kind=case["kind"], ctx=ctx, f=fd, u=torch.zeros_like(fd))
    hiers, prm, f, u0 = _problem(case, seed)
    K, kind = case["K"], case["kind"]
    ctx = binding.Context(None, None, prm, K, K, K, nu_pre=case["nu"], nu_post=case["nu"], precision=case["prec"],
                          nrhs=case["nrhs"], native=hiers[0], backward=kind == "train", aggregation=case["agg"],
                          basis=case["basis"], columns=hiers if kind == "round" else None,
                          max_outer=8 if kind == "round" else 10000, check_every=8 if kind == "round" else 10)
    dt = ctx.cycle_dtype if kind == "vcycle" else torch.float64
    fd, ud = torch.tensor(f, device=DEV).to(dt), torch.tensor(u0, device=DEV).to(dt)
    s = dict(kind=kind, ctx=ctx, f=fd, u0=ud, u=torch.empty_like(ud))
    if kind == "train":
        s["ck"] = [ctx.new_ckpt(), ctx.new_ckpt()]
    return s


def run(s):
    kind, ctx, f, u = s["kind"], s["ctx"], s["f"], s["u"]
    if kind == "vcycle":
        u.copy_(s["u0"])
        return ctx.vcycle(f, u)
    if kind == "refine":
        return ctx.refine_step(f, s["u0"], u)
    if kind == "train":
        u1 = ctx.refine_step(f, s["u0"], ckpt=s["ck"][0])
        u2 = ctx.refine_step(f, u1, u, ckpt=s["ck"][1])
        loss, g, _ = ctx.residual_loss(f, u2, want_gu=True)
        g1, gf1, gp1 = ctx.refine_step_backward(s["ck"][1], g)
        g0, gf0, gp0 = ctx.refine_step_backward(s["ck"][0], g1)
        return dict(u=u2, loss=loss, gu=g0, gf1=gf1, gf0=gf0, gp1=gp1, gp0=gp0)
    if kind in ("solve", "round"):
        u.zero_()
        info = ctx.solve(f, u)
        return dict(u=u, iters=info.iters, status=info.status)
    if kind == "fgmres":
        u.zero_()
        info = ctx.fgmres(f, u, restart=30)
        return dict(u=u, iters=info.iters, status=info.status)
    u.zero_()
    if kind == "hcycle":
        return ctx.vcycle(f, u)
    info = ctx.fgmres(f, u, restart=40)
    return dict(u=u, iters=info.iters, status=info.status)


# ------------------------------------------------------------------ the work that a pass cannot do without
# cycles (preconditioner calls) that a whole solve takes with the parameters it is given
_CYCLES = {"vcycle": 1, "refine": 1, "train": 2, "solve": 40, "round": 8, "fgmres": 14, "hcycle": 1, "hfgmres": 28}


def work(case):
    B, K, kind = case["nrhs"], case["K"], case["kind"]
    c = 8 if case["prec"] == "fp64" else 4
    helm = kind in ("hcycle", "hfgmres")
    m = case["side"] if helm else case["side"] - 2
    low = 0 if helm else case["coarsest"]
    per_op, flops, level = 0.0, 0.0, 0
    own = B if kind == "round" else 1                     # operators with values of their own
    while (m > low and not helm) or (helm and level < case["levels"]):
        n, w = m * m, (6 if level or helm else 4)
        per_op += n * (w * (4 + c * own * (1 + helm)) + c * own * (1 + helm)) + 2 * n * (4 + c)
        if not helm:
            sweeps = 2 * case["nu"]
            flops += n * B * ((sweeps + 1) * 2 * (w + 2) + (sweeps + 2) * K * (w + 3) + 12)
        else:
            jac = case["k"] / (case["side"] - 1) * 2 ** level <= 0.5
            flops += n * B * ((2 if jac else 15) * 8 * (w + 1) + 8 * (w + 1) + 4 * K * (2 * w + 10)
                              + (0 if jac else 3 * 4 * 40))
        m, level = (m - 1) // 2 if not helm else (m + 1) // 2, level + 1
    n0 = (case["side"] if helm else case["side"] - 2) ** 2
    vec = n0 * B * ((1 + helm) * (c if kind in ("vcycle", "hcycle") else 8))
    cycles = _CYCLES[kind]
    # each input once (operators, right-hand side, first iterate), each output once
    if kind == "train":
        return dict(bytes=per_op + 6.0 * vec, flops=cycles * 4 * flops)
    if kind in ("fgmres", "hfgmres"):
        flops += 8 * cycles * n0 * B                      # Gram-Schmidt against the basis so far
    return dict(bytes=per_op + 3.0 * vec, flops=cycles * flops)


# ------------------------------------------------------------------ the method in 64 bits
def _exact_dev():
    return DEV if torch.cuda.is_available() else "cpu"


def _csr_ell(rowptr, col, val, n):
    """Row-wise padded (n, w) columns and values (padding: column 0, value 0)."""
    rowptr, col, val = np.asarray(rowptr), np.asarray(col), np.asarray(val)
    lens = np.diff(rowptr)
    w = max(1, int(lens.max()))
    slot = np.arange(len(col)) - np.repeat(rowptr[:-1], lens)
    row = np.repeat(np.arange(n), lens)
    c, v = np.zeros((n, w), np.int64), np.zeros((n, w), val.dtype)
    c[row, slot], v[row, slot] = col, val
    return torch.tensor(c, device=_exact_dev()), torch.tensor(v, device=_exact_dev())


def _transpose(rowptr, col, val, ncols):
    n = len(rowptr) - 1
    row = np.repeat(np.arange(n), np.diff(rowptr))
    order = np.argsort(col, kind="stable")
    return np.concatenate([[0], np.cumsum(np.bincount(col, minlength=ncols))]), row[order], val[order]


def _mv(M, x):
    """M x for (n, w) columns and values; values (n, w, B) belong to the columns of x."""
    c, v = M
    y = 0
    for s in range(c.shape[1]):
        vs = v[:, s]
        y = y + (vs if vs.dim() == 2 else vs[:, None]) * x[c[:, s]]
    return y


def _view_csr(m):
    a = np.ctypeslib.as_array
    val = a(ctypes.cast(m.val, ctypes.POINTER(ctypes.c_double)), shape=(max(m.nnz, 1),))[:m.nnz].copy()
    return a(m.rowptr, shape=(m.nrows + 1,)).copy(), a(m.col, shape=(max(m.nnz, 1),))[:m.nnz].copy(), val


def _graph(rp, col, val, agg):
    """The aggregation operator of a level as (columns, values)."""
    n = len(rp) - 1
    row = np.repeat(np.arange(n), np.diff(rp))
    keep = (row != col) & (val != 0)
    row, c, v = row[keep], col[keep], np.abs(val[keep])
    grp = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))])
    deg = np.bincount(row, minlength=n).astype(float)
    if agg == "weighted":
        g = v / np.bincount(row, weights=v, minlength=n)[row]
    elif agg == "sym":
        g = 1.0 / np.sqrt(deg[row] * deg[c])
    else:
        g = 1.0 / deg[row]
    return _csr_ell(grp, c, g.astype(np.float64), n)


class _Exact:
    """The cycle of a real-valued case in 64 bits, differentiable in its parameters."""

    def __init__(self, case, seed):
        hiers, prm, f, u0 = _problem(case, seed)
        self.case, J = case, hiers[0].nlevels
        dev = _exact_dev()
        self.lv = []
        for l in range(J):
            rp, col, val = _view_csr(hiers[0].view.A[l])
            n = len(rp) - 1
            c, v = _csr_ell(rp, col, val, n)
            if len(hiers) > 1:
                v = torch.stack([_csr_ell(rp, col, _view_csr(h.view.A[l])[2], n)[1] for h in hiers], dim=2)
            own = (c == torch.arange(n, device=dev)[:, None])
            own = own[:, :, None] if v.dim() == 3 else own
            d = (v * own).sum(1)
            lev = dict(n=n, A=(c, v), D=d if d.dim() == 2 else d[:, None], G=_graph(rp, col, val, case["agg"]))
            if l + 1 < J:
                p = _view_csr(hiers[0].view.P[l])
                nc = hiers[0].sizes[l + 1]
                lev["P"] = _csr_ell(*p, n)
                lev["R"] = _csr_ell(*_transpose(*p, nc), nc)
            else:
                dense = torch.zeros((v.shape[2] if v.dim() == 3 else 1, n, n), dtype=torch.float64, device=dev)
                i = torch.arange(n, device=dev)[:, None].expand_as(c)
                for b in range(dense.shape[0]):
                    dense[b].index_put_((i, c), v[:, :, b] if v.dim() == 3 else v, accumulate=True)
                lev["inv"] = torch.linalg.inv(dense.cpu()).to(dev)
            self.lv.append(lev)
        self.prm = torch.tensor(prm, device=dev).reshape(J - 1, -1)
        self.f, self.u0 = torch.tensor(f, device=dev), torch.tensor(u0, device=dev)
        for h in hiers:
            h.close()

    def conv(self, l, c, x):
        G = self.lv[l]["G"]
        K = len(c) - 1
        if self.case["basis"] == "chebyshev":
            before, t = x, -_mv(G, x)
            y = c[0] * x + c[1] * t
            for k in range(2, K + 1):
                before, t = t, -2.0 * _mv(G, t) - before
                y = y + c[k] * t
            return y
        y = c[K] * x
        for k in range(K - 1, -1, -1):
            y = _mv(G, y) + c[k] * x
        return y

    def cycle(self, l, f, u, prm):
        lev = self.lv[l]
        if "inv" in lev:
            if lev["inv"].shape[0] == 1:
                return lev["inv"][0] @ f
            return (lev["inv"] * f.T[:, None, :]).sum(2).T
        p, K1 = prm[l], self.case["K"] + 1
        cB, cR, cP = p[2:2 + K1], p[2 + K1:2 + 2 * K1], p[2 + 2 * K1:]

        def smooth(v):
            return v + p[1] * self.conv(l, cB, p[0] * (f - _mv(lev["A"], v)) / lev["D"])
        for _ in range(self.case["nu"]):
            u = smooth(u)
        rc = _mv(lev["R"], self.conv(l, cR, f - _mv(lev["A"], u)))
        ec = self.cycle(l + 1, rc, torch.zeros_like(rc), prm)
        u = u + self.conv(l, cP, _mv(lev["P"], ec))
        for _ in range(self.case["nu"]):
            u = smooth(u)
        return u

    def step(self, f, u, prm):
        r = f - _mv(self.lv[0]["A"], u)
        return u + self.cycle(0, r, torch.zeros_like(r), prm)

    def train(self):
        u0, p = self.u0.clone().requires_grad_(), [self.prm.clone().requires_grad_() for _ in range(2)]
        f = [self.f.clone().requires_grad_() for _ in range(2)]
        u2 = self.step(f[1], self.step(f[0], u0, p[0]), p[1])
        r = self.f - _mv(self.lv[0]["A"], u2)
        loss = ((r * r).sum(0) / (self.f * self.f).sum(0)).mean()
        g = torch.autograd.grad(loss, [u0, f[1], f[0], p[1], p[0]])
        return dict(u=u2.detach(), loss=loss.detach().reshape(1), gu=g[0], gf1=g[1], gf0=g[2], gp1=g[3].reshape(-1),
                    gp0=g[4].reshape(-1))

    def solution(self, limit=4000):
        """A u = f to FP64 accuracy by the same iteration."""
        u, f = self.u0, self.f
        best = None
        for k in range(limit):
            r = f - _mv(self.lv[0]["A"], u)
            rel = float((r.norm(dim=0) / f.norm(dim=0)).max())
            if rel < 1e-13 or (best is not None and k % 20 == 0 and rel > 0.5 * best):
                break
            best = rel if k % 20 == 0 else best
            u = u + self.cycle(0, r, torch.zeros_like(r), self.prm)
        return u


class _HelmExact:
    """The Helmholtz cycle in 64 bits."""

    def __init__(self, case, seed):
        h, self.plan, prm, f = _helm_problem(case, seed)
        dev, K, J = _exact_dev(), case["K"], case["levels"]
        self.lv = []
        for l in range(J):
            a = h.A[l].tocsr()
            n = a.shape[0]
            c, v = _csr_ell(a.indptr, a.indices, a.data, n)
            d = (v * (c == torch.arange(n, device=dev)[:, None])).sum(1)
            lev = dict(A=(c, v), D=d[:, None], G=_graph(a.indptr, a.indices, a.data, "mean"))
            if l + 1 < J:
                p = h.P[l].tocsr()
                nc = h.A[l + 1].shape[0]
                lev["P"] = _csr_ell(p.indptr, p.indices, p.data, n)
                lev["R"] = _csr_ell(*_transpose(p.indptr, p.indices, p.data, nc), nc)
            else:
                lev["inv"] = torch.tensor(np.linalg.inv(a.toarray()), device=dev)
            self.lv.append(lev)
        per = 2 + 4 * (K + 1)
        self.lp = prm[:(J - 1) * per].reshape(J - 1, per)
        rest = prm[(J - 1) * per:].reshape(2, K + 1, 2, 2)
        self.WR, self.WP = rest
        self.f = torch.tensor(f, device=dev)

    @staticmethod
    def mix(W, x):
        return torch.complex(W[0, 0] * x.real + W[0, 1] * x.imag, W[1, 0] * x.real + W[1, 1] * x.imag)

    def conv(self, W, l, x):
        y = self.mix(W[-1], x)
        for k in range(len(W) - 2, -1, -1):
            y = _mv(self.lv[l]["G"], y) + self.mix(W[k], x)
        return y

    def gmres(self, A, r, x0, v):
        """v GMRES steps per column from x0 (Arnoldi with modified Gram-Schmidt, twice)."""
        r0 = r - _mv(A, x0)
        beta = r0.norm(dim=0)
        safe = torch.where(beta > 0, beta, torch.ones_like(beta))
        B = r.shape[1]
        V, H = [r0 / safe], torch.zeros((B, v + 1, v), dtype=torch.complex128, device=r.device)
        for j in range(v):
            w = _mv(A, V[j])
            for _ in range(2):
                for i in range(j + 1):
                    h = (V[i].conj() * w).sum(0)
                    H[:, i, j] += h
                    w = w - h * V[i]
            nw = w.norm(dim=0)
            H[:, j + 1, j] = nw.to(torch.complex128)
            V.append(w / torch.where(nw > 0, nw, torch.ones_like(nw)))
        rhs = torch.zeros((B, v + 1, 1), dtype=torch.complex128, device=r.device)
        rhs[:, 0, 0] = beta.to(torch.complex128)
        y = torch.tensor(np.stack([np.linalg.lstsq(h, g, rcond=None)[0] for h, g in zip(H.cpu().numpy(),
                                                                                       rhs.cpu().numpy())]),
                         device=r.device)[:, :, 0]
        x = x0
        for j in range(v):
            x = x + y[:, j] * V[j]
        return x

    def cycle(self, l, f, u):
        lev = self.lv[l]
        if "inv" in lev:
            return lev["inv"] @ f
        kind, pre, post = self.plan[l]
        th, et, WB = self.lp[l, 0], self.lp[l, 1], self.lp[l, 2:].reshape(-1, 2, 2)

        def smooth(u):
            r = f - _mv(lev["A"], u)
            if kind == "jacobi":
                return u + et * self.conv(WB, l, th * (r / lev["D"]))
            return u + et * self.gmres(lev["A"], r, th * self.conv(WB, l, r), 4)
        for _ in range(pre):
            u = smooth(u)
        rc = _mv(lev["R"], self.conv(self.WR, l, f - _mv(lev["A"], u)))
        u = u + self.conv(self.WP, l, _mv(lev["P"], self.cycle(l + 1, rc, torch.zeros_like(rc))))
        for _ in range(post):
            u = smooth(u)
        return u

    def solution(self, limit=300):
        """A u = f to FP64 accuracy by the stationary iteration; None where it does not converge."""
        u = torch.zeros_like(self.f)
        for _ in range(limit):
            r = self.f - _mv(self.lv[0]["A"], u)
            if float((r.norm(dim=0) / self.f.norm(dim=0)).max()) < 1e-12:
                return u
            u = self.cycle(0, self.f, u)
        return None


def exact(case, seed):
    kind = case["kind"]
    if kind in ("hcycle", "hfgmres"):
        h = _HelmExact(case, seed)
        if kind == "hcycle":
            return h.cycle(0, h.f, torch.zeros_like(h.f))
        u = h.solution()
        return None if u is None else dict(u=u, iters=None, status=None)
    e = _Exact(case, seed)
    if kind == "train":
        return e.train()
    with torch.no_grad():
        if kind == "vcycle":
            return e.cycle(0, e.f, e.u0, e.prm)
        if kind == "refine":
            return e.step(e.f, e.u0, e.prm)
        if kind == "round":
            u = e.u0
            for _ in range(8):
                u = e.step(e.f, u, e.prm)
            return dict(u=u, iters=None, status=None)
        return dict(u=e.solution(), iters=None, status=None)
