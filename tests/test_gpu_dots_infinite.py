"""Parameter gradients that overflow are infinite, not NaN.

One post-smoothing step on a zero iterate with no coarse correction: its dot products are
<(G^T)^k g, D^{-1} f> with every factor positive, so a cotangent g with infinite entries (or, in FP64,
products past the largest double) makes each of them +inf."""
import numpy as np
import pytest

from mginputs import configs as C, hierarchy as H
from tests.gpu_util import ctx_for, to_dev, to_np

pytestmark = pytest.mark.gpu

HIER = {s: H.square_hierarchy(s) for s in (33, 65, 129)}


@pytest.mark.parametrize("side,prec,B,kw", [
    (65, "fp32", 3, {}), (65, "fp64", 3, {}), (33, "fp64", 2, {}),              # reverse tail
    (129, "fp32", 16, {}), (129, "bf16", 16, {}),                               # over tiles
    (129, "fp32", 5, dict(tail=False, tiles=False)), (65, "bf16", 3, {})])      # per-hop sweeps
@pytest.mark.parametrize("K", [1, 3])
def test_infinite_dot_products(side, prec, B, kw, K):
    import torch
    hier = HIER[side]
    J, n = hier.nlevels, hier.sizes[0]
    p = C.identity_params(J, K, K, K).reshape(J - 1, -1)
    p[:, 2:2 + K + 1] = 0.5
    p[:, 2 + 2 * (K + 1):] = 0.0                       # no correction from the coarse levels
    ctx = ctx_for(hier, p.ravel(), K, B, prec, nu=(0, 1), backward=True, **kw)
    g = C.rng(11, 9, side)
    f, w = (g.uniform(0.5, 1.5, (n, B)) for _ in range(2))
    cases = []
    hot = w.copy()
    hot[::97, B // 2] = np.inf
    cases.append((f, hot))
    if prec == "fp64":
        cases.append((1e180 * f, 1e180 * w))
    for fc, wc in cases:
        ck = ctx.new_ckpt()
        ud = to_dev(np.zeros_like(f), ctx.cycle_dtype)
        ctx.vcycle(to_dev(fc, ctx.cycle_dtype), ud, ckpt=ck)
        gp = to_np(ctx.vcycle_backward(ck, to_dev(wc, ctx.cycle_dtype))[2]).reshape(J - 1, -1)
        assert np.all(gp[0, 2:2 + K + 1] == np.inf), gp[0]
    ctx.close()
