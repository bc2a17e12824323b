"""The GMRES smoothing step with its rows in registers, at the edges of its
forms: fewer rows than a wavefront, one and three rows per work-item of 512, the
last sizes of both, one size past them (the sweep form), 1 .. 4 steps and more
(the sweep form), convolution orders 0 .. 3."""
import numpy as np
import pytest

from mginputs import configs as C
from mginputs import helmholtz as HZ
from oracle import helmholtz as OH
from tests.gpu_util import elem_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,v,K", [(5, 2, 1), (9, 4, 2), (21, 4, 0), (23, 4, 1), (23, 1, 3), (39, 4, 1), (39, 3, 2),
                                      (41, 4, 1), (23, 5, 1)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_gmres_step_matches_oracle(side, v, K, prec):
    _check(side, v, K, prec, 2)


@pytest.mark.parametrize("side,v,K", [(53, 4, 1), (57, 4, 2), (65, 2, 1), (65, 4, 0), (69, 4, 1)])
def test_gmres_step_with_nine_rows_matches_oracle(side, v, K):
    """Single precision, rows of A read for each product: below, at the first and a late size of that
    form, and past it."""
    _check(side, v, K, "fp32", 3)


def _check(side, v, K, prec, levels):
    import torch
    from paper_2608_29082_amd import helmholtz as HB
    B, plan = 3, [("gmres", 1, 1)] * (levels - 1)
    h = HZ.hierarchy(side, 0.9 * (side - 1), levels)
    flat = C.hz_random_params(levels, K, 1, 1, plan, seed=side)
    g = C.rng(10, 12, side)
    f = HZ.load_vectors(side, HZ.source_centres(B, g)) + 1e-3 * (g.standard_normal((side * side, B)) + 0j)
    f[:, 2] = 0.0                                   # a zero column keeps a zero iterate
    u0 = 0.01 * (g.standard_normal(f.shape) + 1j * g.standard_normal(f.shape))
    u0[:, 2] = 0.0
    want = OH.lmg(OH.make_levels(h.A, h.P, h.R), OH.unpack(flat, levels, K, 1, 1, plan, v), 0, f, u0)
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    c = HB.HelmholtzContext(h.A, h.P, flat, K, 1, 1, plan, v=v, precision=prec, nrhs=B)
    u = torch.tensor(u0, device="cuda").to(dt)
    c.vcycle(torch.tensor(f, device="cuda").to(dt), u)
    got = u.cpu().numpy().astype(np.complex128)
    err = elem_rel(got[:, :2], want[:, :2])
    print(f"{prec} side={side} v={v} K={K}: rel {err:.2e}", flush=True)
    assert err <= (1e-11 if prec == "fp64" else 5e-5)
    assert np.all(got[:, 2] == 0)
    c.close()
