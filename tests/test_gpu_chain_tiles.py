"""Transposed convolutions over tiles against the chain of per-hop sweeps.

Both multiply and add in the same order per node and column, so the gradients with respect to the
iterate and the right-hand side carry the same bits.  The parameter gradients sum products that FP64
holds exactly as unevaluated pairs and round once: they may differ by that rounding only."""
import numpy as np
import pytest

from mginputs import configs as C, hierarchy as H
from tests.gpu_util import ctx_for, to_dev, to_np

pytestmark = pytest.mark.gpu

HIER = {"square": H.square_hierarchy(129, H.block_field(C.rng(7, 1, 1), 16, -3, 3)),
        "lshape": H.lshape_hierarchy(C.rng(7, 4, 0), target_nodes=120, refinements=4)}


@pytest.mark.parametrize("agg", ["mean", "weighted", "sym"])
@pytest.mark.parametrize("K,nu", [((2, 3, 4), (1, 2)), ((4, 2, 2), (2, 1)), ((3, 1, 3), (0, 1))])
@pytest.mark.parametrize("mesh,B", [("square", 16), ("square", 48), ("lshape", 16)])
def test_chain_over_tiles_equals_hop_sweeps(agg, K, nu, mesh, B):
    import torch
    hier = HIER[mesh]
    flat = C.random_params(hier.nlevels, *K, seed=107, spread=0.2)
    g = C.rng(11, 5, B)
    f, u, w = (g.standard_normal((hier.sizes[0], B)) for _ in range(3))
    outs = []
    for tiles in (True, False):
        ctx = ctx_for(hier, flat, K, B, "fp32", tiles=tiles, tail=False, backward=True, nu=nu, aggregation=agg)
        ck = ctx.new_ckpt()
        ctx.refine_step(to_dev(f, torch.float64), to_dev(u, torch.float64), ckpt=ck)
        outs.append([to_np(t) for t in ctx.refine_step_backward(ck, to_dev(w, torch.float64))])
        ctx.close()
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
    gp = [o[2] for o in outs]
    # one rounding a slot, about ten slots a parameter
    assert np.linalg.norm(gp[0] - gp[1]) <= 16 * np.finfo(float).eps * np.linalg.norm(gp[1])
