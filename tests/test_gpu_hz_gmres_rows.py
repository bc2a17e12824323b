"""The GMRES smoothing step with its rows in registers on rows of five, eight and nine entries (the mesh's
own have seven): slots past the operator's width, the forms of eight slots, and rows too wide for them
(the sweep form)."""
import numpy as np
import pytest
import scipy.sparse as sp

from mginputs import configs as C
from mginputs import helmholtz as HZ
from oracle import helmholtz as OH
from tests.gpu_util import elem_rel

pytestmark = pytest.mark.gpu


def _with_width(A, width):
    """A with `width` entries in its widest rows: the couplings along the mesh's diagonals taken out, or
    one or two symmetric couplings a row added."""
    A = sp.csr_matrix(A)
    n = A.shape[0]
    side = int(round(np.sqrt(n)))
    if width < 7:
        a = A.tocoo()
        keep = np.isin(np.abs(a.row - a.col), (0, 1, side))
        A = sp.csr_matrix((a.data[keep], (a.row[keep], a.col[keep])), shape=A.shape)
    for step in (2, 4)[:max(0, width - 7)]:
        i = np.arange(n)
        i = i[(i // step) % 2 == 0]
        i = i[i + step < n]
        w = sp.csr_matrix((np.full(i.size, 0.05 * abs(A.diagonal()).mean()), (i, i + step)), shape=A.shape)
        A = A + w + w.T
    A = sp.csr_matrix(A)
    A.sort_indices()
    assert np.diff(A.indptr).max() == width
    return A


@pytest.mark.parametrize("side,width,prec", [
    (s, w, p) for s in (21, 39) for w in (5, 8, 9) for p in ("fp64", "fp32")] + [(65, 5, "fp32"), (65, 8, "fp32")])
def test_gmres_step_on_other_row_widths(side, width, prec):
    import torch
    from paper_2608_29082_amd import helmholtz as HB
    levels, K, B, plan = 2, 1, 3, [("gmres", 1, 1)]
    h = HZ.hierarchy(side, 0.9 * (side - 1), levels)
    A = [_with_width(h.A[0], width)] + h.A[1:]
    flat = C.hz_random_params(levels, K, 1, 1, plan, seed=side)
    g = C.rng(10, 13, side)
    n = side * side
    f = g.standard_normal((n, B)) + 1j * g.standard_normal((n, B))
    u0 = 0.1 * (g.standard_normal((n, B)) + 1j * g.standard_normal((n, B)))
    want = OH.lmg(OH.make_levels(A, h.P, h.R), OH.unpack(flat, levels, K, 1, 1, plan, 4), 0, f, u0)
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    c = HB.HelmholtzContext(A, h.P, flat, K, 1, 1, plan, v=4, precision=prec, nrhs=B)
    u = torch.tensor(u0, device="cuda").to(dt)
    c.vcycle(torch.tensor(f, device="cuda").to(dt), u)
    err = elem_rel(u.cpu().numpy().astype(np.complex128), want)
    c.close()
    print(f"{prec} side={side} width={width}: rel {err:.2e}", flush=True)
    # the tolerances of the step on the mesh's own rows
    assert err <= (1e-11 if prec == "fp64" else 5e-5)
