"""The coarse tail in LDS at the edges of its register variants.

One- to four-row variants (a level's rows per work-item of 1024), the
one-wavefront levels (at most 64 rows), four, six and eight slots per row, rows
too wide for a variant (generic sweeps), levels one row past a variant and a
graph that is not A's pattern.  A step that records a checkpoint sums in the
order of the per-level sweeps, so it is compared with them bit for bit, and so
is the reverse sweep; a cycle from a nonzero iterate is compared with the
oracle."""
import numpy as np
import pytest
import scipy.sparse as sp

from mginputs import configs as C
from oracle import lmg as O
from tests.gpu_util import elem_rel, to_dev, to_np

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 2e-5}


def _operator(n, width, g):
    """A ring of n nodes with chords (`width` neighbours a row), diagonally dominant."""
    i = np.arange(n)
    A = sp.csr_matrix((n, n))
    for d in range(1, width // 2 + 1):
        step = 1 if d == 1 else 5 * d + 2
        W = sp.coo_matrix((g.uniform(0.5, 1.5, n), (i, (i + step) % n)), shape=(n, n))
        A = A + W + W.T
    return sp.csr_matrix(sp.diags(np.asarray(A.sum(axis=1)).ravel() + 0.1) - A)


def _hierarchy(n, width, seed):
    """The fine operator and plain rings below it, with linear interpolation along the ring."""
    g = C.rng(11, 1, seed)
    As, Ps = [_operator(n, width, g)], []
    while n > 12:
        c = (n + 1) // 2
        even, odd = np.arange(0, n, 2), np.arange(1, n, 2)
        r = np.concatenate([even, odd, odd])
        k = np.concatenate([even // 2, odd // 2, ((odd + 1) // 2) % c])
        w = np.concatenate([np.ones(even.size), np.full(2 * odd.size, 0.5)])
        Ps.append(sp.coo_matrix((w, (r, k)), shape=(n, c)).tocsr())
        As.append(_operator(c, 2, g))
        n = c
    return As, Ps


def _ring_graph(A):
    n = A.shape[0]
    i = np.arange(n)
    return sp.csr_matrix((np.ones(2 * n), (np.r_[i, i], np.r_[(i + 1) % n, (i - 1) % n])), shape=(n, n))


@pytest.mark.parametrize("prec,n,width,graph", [
    ("fp32", 64, 6, False), ("fp32", 65, 6, False), ("fp32", 1024, 4, False), ("fp32", 1025, 8, False),
    ("fp32", 2049, 6, False), ("fp32", 3073, 4, False), ("fp32", 4096, 8, False), ("fp32", 4097, 6, False),
    ("fp32", 1300, 10, False), ("fp32", 1300, 6, True), ("fp32", 60, 6, True),
    ("fp64", 64, 8, False), ("fp64", 1025, 6, False), ("fp64", 2049, 8, False), ("fp64", 3070, 4, False)])
@pytest.mark.parametrize("agg", ["mean", "sym"])
def test_tail_variants(prec, n, width, graph, agg):
    import torch
    from paper_2608_29082_amd import binding as Bd
    A, P = _hierarchy(n, width, n)
    G = [_ring_graph(a) for a in A] if graph else None
    J, K, B = len(A), 2, 3
    flat = C.random_params(J, K, K, K, seed=n, spread=0.2)
    g = C.rng(11, 2, n)
    f, u = g.standard_normal((n, B)), g.standard_normal((n, B))
    outs = []
    for tail in (True, False):
        ctx = Bd.Context(A, P, flat, K, K, K, precision=prec, nrhs=B, tail=tail, G=G, aggregation=agg, backward=True)
        ck = ctx.new_ckpt()
        step = ctx.refine_step(to_dev(f, torch.float64), to_dev(u, torch.float64), ckpt=ck)
        gu = ctx.refine_step_backward(ck, to_dev(f, torch.float64))
        v = to_dev(u, ctx.cycle_dtype)
        ctx.vcycle(to_dev(f, ctx.cycle_dtype), v)
        outs.append((to_np(step), [to_np(t) for t in gu], to_np(v)))
        ctx.close()
    assert np.array_equal(outs[0][0], outs[1][0])
    # the reverse sweep (itself one launch on these levels) reads every level's checkpoint; its
    # parameter gradients are FP64 sums of n B ~ 1e4 products in another order (1e4 eps ~ 2e-12)
    assert all(np.array_equal(a, b) for a, b in zip(outs[0][1][:2], outs[1][1][:2]))
    gp = [o[1][2] for o in outs]
    assert np.linalg.norm(gp[0] - gp[1]) <= 1e-11 * np.linalg.norm(gp[1])
    want = O.lmg(O.make_levels(A, P, None, G, aggregation=agg), O.unpack(flat, J, K, K, K), 0, f, u)
    errs = [elem_rel(o[2], want) for o in outs]
    print(f"{prec} n={n} width={width} graph={graph} {agg}: cycle errors {errs[0]:.1e} {errs[1]:.1e}", flush=True)
    assert max(errs) <= TOL[prec]


@pytest.mark.parametrize("prec,n", [("fp32", 60), ("fp32", 900), ("fp32", 2100), ("fp32", 4000), ("fp64", 1500)])
def test_tail_without_convolutions(prec, n):
    """K = 0 (the classical cycle): no convolution's barriers lie between a residual's reads of the
    iterate and its update.  The cycle from zero against the oracle, and the same bits every time."""
    import torch
    from paper_2608_29082_amd import binding as Bd
    A, P = _hierarchy(n, 6, n)
    J, B = len(A), 3
    flat = C.identity_params(J, 0, 0, 0)
    f = C.rng(11, 3, n).standard_normal((n, B))
    ctx = Bd.Context(A, P, flat, 0, 0, 0, precision=prec, nrhs=B)
    fd = to_dev(f, torch.float64)
    outs = [to_np(ctx.refine_step(fd, torch.zeros_like(fd))) for _ in range(20)]
    want = O.lmg(O.make_levels(A, P), O.unpack(flat, J, 0, 0, 0), 0, f, np.zeros_like(f))
    assert elem_rel(outs[0], want) <= TOL[prec]
    assert all(np.array_equal(o, outs[0]) for o in outs)
    ctx.close()
