"""Which levels the coarse tail holds."""
import pytest

from mginputs import configs as C
from tests.gpu_util import to_dev
from tests.test_gpu_tail import _hierarchy

pytestmark = pytest.mark.gpu


def _launches(family, level, prec, **kw):
    """Launches of one kernel family on one level of a cycle: 5000 rows with ten neighbours each, too wide
    for tiles, over 2500 rows with two."""
    from paper_2608_29082_amd import binding as Bd
    import torch
    A, P = _hierarchy(5000, 10, 3)
    J, K, B = len(A), 3, 16
    ctx = Bd.Context(A, P, C.random_params(J, K, K, K, seed=5, spread=0.1), K, K, K, precision=prec, nrhs=B, **kw)
    f = to_dev(C.rng(11, 7, 0).standard_normal((5000, B)), torch.float64)
    ctx.timing_start(family, level)
    ctx.refine_step(f, torch.zeros_like(f))
    n = ctx.timing_read()[0]
    ctx.close()
    return n


def test_tiled_level_below_an_untiled_one_stays_in_the_tail():
    """BF16 cycles hold FP32 vectors in the tail: it starts at the finest level without tiles that fits its LDS
    and holds every level below it, here the whole cycle, also the 2500 rows that have tiles."""
    assert _launches("hop", 0, "bf16", tail=False) > 0 and _launches("conv", 1, "bf16", tail=False) > 0
    assert _launches("conv", -1, "bf16") == 0 and _launches("resid", -1, "bf16") == 0


def test_fp32_tail_ends_below_a_wide_level():
    """FP32 cycles, whose vectors are the same either way, run the wide level above the tiled one by launches."""
    assert _launches("hop", 0, "fp32") > 0 and _launches("conv", 1, "fp32", tail=False) > 0


@pytest.mark.parametrize("n,width,B,inside", [(5000, 10, 5, False), (5000, 10, 64, False), (2100, 10, 3, False),
                                              (1300, 10, 3, True), (4000, 8, 3, True), (5000, 10, 70, True)])
def test_nonzero_iterate_over_a_level_of_generic_sweeps(n, width, B, inside):
    """Cycles from a nonzero iterate and those that record a checkpoint run a first level of the tail that has no
    register variant by launches where these are faster; a step that records carries the sweeps' bits."""
    import numpy as np
    import torch
    from oracle import lmg as O
    from paper_2608_29082_amd import binding as Bd
    from tests.gpu_util import elem_rel, to_np
    from tests.test_gpu_tail import TOL
    A, P = _hierarchy(n, width, n)
    J, K = len(A), 3
    flat = C.random_params(J, K, K, K, seed=n, spread=0.1)
    g = C.rng(11, 9, n)
    f, u = (g.standard_normal((n, B)).astype(np.float32).astype(np.float64) for _ in range(2))
    fd, ud = to_dev(f, torch.float64), to_dev(u, torch.float64)
    steps, launches = [], []
    for tail in (True, False):
        ctx = Bd.Context(A, P, flat, K, K, K, precision="fp32", nrhs=B, tail=tail, tiles=False, backward=True)
        v = ud.float()
        for call in (lambda: ctx.refine_step(fd, torch.zeros_like(fd)), lambda: ctx.vcycle(fd.float(), v),
                     lambda: steps.append(to_np(ctx.refine_step(fd, ud, ckpt=ctx.new_ckpt())))):
            ctx.timing_start("hop", 0)
            call()
            launches.append(ctx.timing_read()[0])
            ctx.timing_start(None)
        want = O.lmg(O.make_levels(A, P), O.unpack(flat, J, K, K, K), 0, f, u)
        assert elem_rel(to_np(v), want) <= TOL["fp32"]
        ctx.close()
    assert launches[0] == 0 and [k == 0 for k in launches[1:3]] == [inside, inside] and min(launches[3:]) > 0
    assert np.array_equal(*steps)


@pytest.mark.parametrize("prec,n,width", [("fp32", 60, 6), ("fp32", 900, 6), ("fp32", 1300, 10), ("fp32", 4000, 8),
                                          ("fp64", 900, 6), ("fp64", 2100, 4)])
def test_restriction_in_the_tail_rounds_as_the_sweeps(prec, n, width):
    """With restriction weights whose products are rounded (0.9 P^T), a step that records a checkpoint still
    carries the bits of the per-level sweeps, and so do its gradients."""
    import numpy as np
    import scipy.sparse as sp
    import torch
    from paper_2608_29082_amd import binding as Bd
    from tests.gpu_util import to_np
    A, P = _hierarchy(n, width, n)
    J, K, B = len(A), 2, 3
    flat = C.random_params(J, K, K, K, seed=n, spread=0.2)
    g = C.rng(11, 8, n)
    f, u = (to_dev(g.standard_normal((n, B)), torch.float64) for _ in range(2))
    outs = []
    for tail in (True, False):
        ctx = Bd.Context(A, P, flat, K, K, K, precision=prec, nrhs=B, tail=tail, tiles=False, backward=True,
                         R=[sp.csr_matrix(0.9 * p.T) for p in P])
        ck = ctx.new_ckpt()
        step = ctx.refine_step(f, u, ckpt=ck)
        outs.append([to_np(step)] + [to_np(t) for t in ctx.refine_step_backward(ck, f)[:2]])
        ctx.close()
    assert all(np.array_equal(a, b) for a, b in zip(*outs))
