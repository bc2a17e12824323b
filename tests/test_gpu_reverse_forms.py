"""Reverse sweeps without steps on one side or both, and with BF16 intermediates over tiles.

A parameter's gradient is a sum of a few dot products, each an unevaluated pair rounded once in either
path: 16 roundings of the gradients' norm is the bound between two paths over the same vectors."""
import numpy as np
import pytest

from mginputs import configs as C, hierarchy as H
from oracle import adjoint as AD
from oracle import lmg as O
from tests.gpu_util import ctx_for, elem_rel, to_dev, to_np
from tests.test_gpu_tail import _hierarchy

pytestmark = pytest.mark.gpu

EPS = 16 * np.finfo(float).eps


@pytest.mark.parametrize("prec,n", [("fp32", 60), ("fp32", 900), ("fp32", 2100), ("fp32", 4000), ("fp64", 60),
                                    ("fp64", 1500)])
@pytest.mark.parametrize("nu", [(2, 0), (0, 2), (1, 0), (0, 0), (2, 2)])
@pytest.mark.parametrize("K", [(2, 2, 2), (0, 1, 0), (1, 0, 3)])
def test_reverse_tail_with_any_steps(prec, n, nu, K):
    """The reverse sweep in one launch against the per-level sweeps, from the same checkpoint, and in FP64
    against the oracle's vector-Jacobian product."""
    import torch
    from paper_2608_29082_amd import binding as Bd
    A, P = _hierarchy(n, 6, n)
    J, B = len(A), 2
    flat = C.random_params(J, *K, seed=n, spread=0.2)
    g = C.rng(11, 11, n)
    f, u, w = (g.standard_normal((n, B)) for _ in range(3))
    outs, ck0 = [], None
    for tail in (True, False):
        ctx = Bd.Context(A, P, flat, *K, nu_pre=nu[0], nu_post=nu[1], precision=prec, nrhs=B, tail=tail, tiles=False,
                         backward=True)
        ck = ctx.new_ckpt()
        ctx.vcycle(to_dev(f, ctx.cycle_dtype), to_dev(u, ctx.cycle_dtype), ckpt=ck)
        ck0 = ck if ck0 is None else ck0
        outs.append([to_np(t) for t in ctx.vcycle_backward(ck0, to_dev(w, ctx.cycle_dtype))])
        torch.cuda.synchronize()
        ctx.close()
    assert all(np.array_equal(a, b) for a, b in zip(outs[0][:2], outs[1][:2]))
    gp = [o[2] for o in outs]
    assert np.linalg.norm(gp[0] - gp[1]) <= EPS * np.linalg.norm(gp[1])
    if prec == "fp64":
        lv, prm = O.make_levels(A, P), O.unpack(flat, J, *K, *nu)
        fbar, ubar, grads = AD.cycle_vjp(lv, prm, f, u, w)
        e = [elem_rel(a, b) for a, b in zip(outs[0], (ubar, fbar, O.pack(grads)))]
        print(f"n={n} nu={nu} K={K}: {e}", flush=True)
        assert max(e) <= 1e-10


@pytest.mark.parametrize("agg", ["mean", "weighted"])
@pytest.mark.parametrize("nu", [(0, 0), (0, 1)])
@pytest.mark.parametrize("B", [16, 48])
def test_chain_over_tiles_with_bf16_intermediates(agg, nu, B):
    """Transposed convolutions over tiles against the per-hop sweeps where the dot products' other vectors
    are stored in BF16.  From one checkpoint, and with no smoothing step on a corrected iterate (no steps,
    or one on an iterate whose correction has zero coefficients), both contexts hold the same vectors."""
    hier = H.square_hierarchy(129, H.block_field(C.rng(7, 1, 1), 16, -3, 3))
    J, K = hier.nlevels, 3
    p = C.random_params(J, K, K, K, seed=41, spread=0.2).reshape(J - 1, -1)
    if nu[1]:
        p[:, 2 + 2 * (K + 1):] = 0.0
    g = C.rng(11, 12, B)
    f, w = (g.standard_normal((hier.sizes[0], B)) for _ in range(2))
    outs, ck = [], None
    for tiles in (True, False):
        ctx = ctx_for(hier, p.ravel(), K, B, "bf16", nu=nu, backward=True, aggregation=agg, tail=False, tiles=tiles)
        if ck is None:
            ck = ctx.new_ckpt()
            ctx.vcycle(to_dev(f, ctx.cycle_dtype), to_dev(np.zeros_like(f), ctx.cycle_dtype), ckpt=ck)
        outs.append([to_np(t) for t in ctx.vcycle_backward(ck, to_dev(w, ctx.cycle_dtype))])
        ctx.close()
    assert all(np.array_equal(a, b) for a, b in zip(outs[0][:2], outs[1][:2]))
    gp = [o[2] for o in outs]
    assert np.linalg.norm(gp[1]) > 0 and np.linalg.norm(gp[0] - gp[1]) <= EPS * np.linalg.norm(gp[1])
