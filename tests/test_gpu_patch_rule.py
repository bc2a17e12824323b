"""Which levels run over patches.

A patch computes its halo anew for every four columns, so patches serve the graphs and widths whose
sweeps are bound by launches: long edges, three dimensions, full lanes and large levels stay with the
sweeps (there a step over patches took up to nine times as long)."""
import numpy as np
import pytest
import scipy.sparse as sp

from mginputs import configs as C, hierarchy as H
from tests.gpu_util import to_dev
from tests.test_gpu_tail import _hierarchy

pytestmark = pytest.mark.gpu


def _square(side):
    h = H.square_hierarchy(side, H.block_field(C.rng(7, 1, 1), 16, -2, 2))
    return h.A, h.P


def _cube(m):
    e, d = sp.identity(m), sp.diags([-1.0, 2.0, -1.0], [-1, 0, 1], shape=(m, m))
    A = [sp.csr_matrix(sp.kron(sp.kron(d, e), e) + sp.kron(sp.kron(e, d), e) + sp.kron(sp.kron(e, e), d))]
    P = []
    while m > 3:
        c, i = (m + 1) // 2, np.arange(m)
        p = sp.csr_matrix((np.ones(m), (i, i // 2)), shape=(m, c))
        P.append(sp.csr_matrix(sp.kron(sp.kron(p, p), p)))
        P[-1].sort_indices()
        A.append(sp.csr_matrix(P[-1].T @ A[-1] @ P[-1]))
        A[-1].sort_indices()
        m = c
    return A, P


def _mesh():
    h = H.lshape_hierarchy(C.rng(7, 4, 0), target_nodes=400, refinements=4)
    return h.A, h.P


MESH = {"square": lambda: _square(129), "square257": lambda: _square(257), "ring": lambda: _hierarchy(5000, 10, 3),
        "cube": lambda: _cube(20), "mesh": _mesh}


@pytest.mark.parametrize("mesh,K,prec,agg,B,patches", [
    ("square", 3, "fp32", "mean", 1, True), ("square", 3, "fp32", "mean", 4, True),
    ("square", 2, "fp64", "mean", 7, True), ("square", 3, "fp64", "sym", 16, True),
    ("square257", 3, "fp64", "weighted", 9, True), ("square257", 2, "fp32", "mean", 1, True),
    ("square", 3, "fp32", "mean", 40, False), ("square", 3, "fp64", "weighted", 64, False),
    ("square257", 3, "fp32", "mean", 5, False), ("square257", 3, "fp32", "weighted", 12, False),
    ("square257", 2, "fp64", "mean", 3, False),
    ("ring", 4, "fp32", "mean", 20, False), ("ring", 3, "fp64", "weighted", 64, False),
    ("cube", 3, "fp32", "mean", 4, False), ("cube", 3, "fp64", "sym", 20, False),
    ("mesh", 3, "fp64", "weighted", 4, False)])
def test_patches_where_they_pay(mesh, K, prec, agg, B, patches):
    import torch
    from paper_2608_29082_amd import binding as Bd
    A, P = MESH[mesh]()
    n, J = A[0].shape[0], len(A)
    ctx = Bd.Context(A, P, C.random_params(J, K, K, K, seed=3, spread=0.1), K, K, K, precision=prec, nrhs=B,
                     aggregation=agg, tail=False)
    f = to_dev(C.rng(11, 4, B).standard_normal((n, B)), torch.float64).to(ctx.cycle_dtype)
    u = torch.zeros_like(f)
    ctx.timing_start("conv", 0)
    ctx.vcycle(f, u)
    launches = ctx.timing_read()[0]
    ctx.timing_start(None)
    ctx.close()
    assert (launches > 0) == patches
