"""Steps of narrow batches as one launch over patches against the per-level sweeps.

Both round at the same places, so cycles from zero and from a nonzero iterate, full multigrid and the
reverse sweep's gradients carry the same bits.  Orders and step counts cover both parities of the
iterate's two vectors, prolongations of every kind and the step that stays in place; widths below, at
and past the four columns of a workgroup; rows of more than eight slots."""
import numpy as np
import pytest

from mginputs import configs as C, hierarchy as H
from tests.gpu_util import to_dev, to_np
from tests.test_gpu_tail import _hierarchy

pytestmark = pytest.mark.gpu

SQ = H.square_hierarchy(129, H.block_field(C.rng(7, 1, 1), 16, -3, 3))
LS = H.lshape_hierarchy(C.rng(7, 4, 0), target_nodes=120, refinements=4)
MESH = {"square": (SQ.A, SQ.P), "lshape": (LS.A, LS.P), "wide": _hierarchy(5000, 10, 3)}


def _run(A, P, flat, K, B, prec, nu, agg, tiles, bwd, f, u):
    import torch
    from paper_2608_29082_amd import binding as Bd
    ctx = Bd.Context(A, P, flat, *K, nu_pre=nu[0], nu_post=nu[1], precision=prec, nrhs=B, aggregation=agg,
                     tail=False, tiles=tiles, backward=bwd)
    fd, ud = to_dev(f, torch.float64), to_dev(u, torch.float64)
    cyc = lambda t: t.to(ctx.cycle_dtype).clone()
    v = cyc(ud)
    ctx.timing_start("conv", -1)
    ctx.vcycle(cyc(fd), v)
    n = ctx.timing_read()[0]
    ctx.timing_start(None)
    out = [v, ctx.refine_step(fd, torch.zeros_like(fd))]
    w = torch.zeros_like(v)
    ctx.fmg(cyc(fd), w)
    out.append(w)
    if bwd:
        ck = ctx.new_ckpt()
        out.append(ctx.refine_step(fd, ud, ckpt=ck))
        out += list(ctx.refine_step_backward(ck, fd))[:2]
    out = [to_np(t) for t in out]
    ctx.close()
    return n, out


@pytest.mark.parametrize("prec,B", [("fp32", 1), ("fp32", 3), ("fp32", 6), ("fp64", 1), ("fp64", 5), ("fp64", 16)])
@pytest.mark.parametrize("K,nu,agg", [((3, 3, 3), (2, 2), "mean"), ((2, 3, 4), (1, 2), "weighted"),
                                      ((4, 2, 1), (2, 1), "sym"), ((3, 1, 2), (0, 1), "mean"),
                                      ((2, 0, 0), (1, 2), "mean"), ((1, 2, 3), (1, 1), "sym")])
@pytest.mark.parametrize("mesh", ["square", "lshape", "wide"])
def test_patches_equal_sweeps(mesh, K, nu, agg, prec, B):
    A, P = MESH[mesh]
    n, J = A[0].shape[0], len(A)
    flat = C.random_params(J, *K, seed=109, spread=0.2)
    g = C.rng(11, 6, B)
    f, u = g.standard_normal((n, B)), g.standard_normal((n, B))
    bwd = K[1] >= 1 and prec == "fp32"
    (n1, on), (n0, off) = (_run(A, P, flat, K, B, prec, nu, agg, t, bwd, f, u) for t in (True, False))
    assert n1 > 0 and n0 == 0
    assert all(np.array_equal(a, b) for a, b in zip(on, off))
