"""Vectors at addresses that are aligned for one element only, through the C entry points."""
import numpy as np
import pytest

from mginputs import configs as C, hierarchy as H
from tests.gpu_util import ctx_for

pytestmark = pytest.mark.gpu

HIER = H.square_hierarchy(129, H.block_field(C.rng(7, 1, 1), 16, -3, 3))


@pytest.mark.parametrize("B", [16, 5])
@pytest.mark.parametrize("shift", [1, 2, 3])
def test_cycle_and_reverse_sweep_at_odd_addresses(B, shift):
    """A cycle and its reverse sweep with every caller's vector `shift` floats past a 16-byte boundary give
    the bits of the aligned call (with B = 16 the level is computed over tiles, in 16-byte units), and
    nothing outside the vectors changes."""
    import torch
    from paper_2608_29082_amd import binding as Bd
    n, J, K = HIER.sizes[0], HIER.nlevels, 3
    flat = C.random_params(J, K, K, K, seed=31, spread=0.2)
    g = C.rng(11, 10, B)
    f, u, w = (torch.tensor(g.standard_normal(n * B), dtype=torch.float32, device="cuda") for _ in range(3))
    ctx = ctx_for(HIER, flat, K, B, "fp32", backward=True)
    lib, s = ctx.lib, ctx._s()
    outs = []
    for sh in (0, shift):
        def at(x=None):
            buf = torch.full((n * B + 16,), 7.0, dtype=torch.float32, device="cuda")
            v = buf[4 + sh:4 + sh + n * B]
            if x is not None:
                v.copy_(x)
            return buf, v
        (fb, fv), (ub, uv), (wb, wv), (gub, gu), (gfb, gf) = at(f), at(u), at(w), at(), at()
        gp = torch.empty(ctx.nparams, dtype=torch.float64, device="cuda")
        ck = ctx.new_ckpt()
        Bd._check(lib.mg_vcycle(ctx._h, fv.data_ptr(), uv.data_ptr(), ck.data_ptr(), s))
        Bd._check(lib.mg_vcycle_backward(ctx._h, ck.data_ptr(), wv.data_ptr(), gu.data_ptr(), gf.data_ptr(),
                                         gp.data_ptr(), s))
        torch.cuda.synchronize()
        for b in (fb, ub, wb, gub, gfb):
            assert float((b[:4 + sh] - 7.0).abs().max()) == 0.0 and float((b[4 + sh + n * B:] - 7.0).abs().max()) == 0.0
        outs.append([t.cpu().numpy() for t in (uv, gu, gf, gp)])
    ctx.close()
    assert all(np.array_equal(a, b) for a, b in zip(*outs))
