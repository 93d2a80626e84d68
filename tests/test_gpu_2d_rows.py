"""The 2D wavefront-per-tile kernel at the edges of its tiles, against the
oracle: one column short of, at and past a 62-column strip, several strips,
row counts that leave a remainder with 1, 2 and 4 rows per wavefront, and
Dirichlet and natural faces.  Every kind with its compile-time and generic
exponents.  F in FP64 to 1e-12 and in FP32 to 1e-4 (FP32 levels take the node
kernels), J v against the exact derivative to 1e-5 (the bars of the other parity
tests), and a smoother of
degree 3 against the node-centric kernel of the same library (kernel_path 1)
to 1e-10: two roundings apart, amplified by the polynomial.
"""
import numpy as np
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

from _common import make_ctx, oracle_grid, oracle_problem, rel, to_dev, to_np
from oracle import derivatives as OD
from oracle import problems as OP
from paper_2103_13890_amd import api
from paper_2103_13890_amd import workloads as W

LO = [(0, 0), (1, 0)]


@pytest.mark.parametrize('kind,params', [('bratu', (5.0,)), ('plap', (1.0, 1.0)), ('plap', (3.0, 0.1)),
                                         ('plap', (2.5, 0.1)), ('plap_gauss', (3.0, 0.1)), ('invcoef', ())])
@pytest.mark.parametrize('n,faces', [((60, 40), W.ALL2), ((61, 43), LO), ((62, 8), W.ALL2), ((124, 150), LO),
                                     ((186, 260), W.ALL2), ((252, 602), LO), ((252, 1032), LO), ((2, 2), W.ALL2)])
def test_rows(kind, params, n, faces):
    w = dict(W.WORKLOADS['bratu2d-32'])
    nlevels = 3 if n[0] % 4 == 0 and n[1] % 4 == 0 and n[0] > 100 else 2 if n[0] % 2 == 0 and n[1] % 2 == 0 else 1
    w.update(kind=kind, params=params, n=n, h=1.0 / max(n), faces=faces, nlevels=nlevels,
             options=dict(vcycle_prec=0, coarse_rtol=1e-6, power_fixed=1, power_maxit=3))
    ctx = make_ctx(w)
    L = nlevels - 1
    g, pb = oracle_grid(w), oracle_problem(w)
    xs = g.node_coords()
    u = 0.4 * np.sin(3.0 * xs[0]) * np.cos(2.0 * xs[1]) + 1e-2 * w['h'] * W.rough_state(n, [], 41)
    v = W.normal_vector(n, faces, 42)
    b = 0.1 * W.normal_vector(n, faces, 43)
    m = 0.3 * np.cos(2.0 * xs[0] + xs[1]) if kind == 'invcoef' else None
    md = None if m is None else to_dev(m)
    F = OP.residual(pb, g, u, b, m)
    assert rel(to_np(api.jfnk_residual(ctx, L, to_dev(u), md, to_dev(b))), F) < 1e-12
    F32 = api.jfnk_residual(ctx, L, to_dev(u, torch.float32), md, to_dev(b, torch.float32))
    assert rel(to_np(F32), F) < 1e-4
    # (the oracle's derivative of the inverse coefficient is written for 3D cells)
    Jv = OD.jvp(pb, g, u, v, m) if kind != 'invcoef' else None
    for form in (1, 2) if Jv is not None else ():
        c2 = make_ctx(w, fd_form=form)
        assert rel(to_np(api.jfnk_jv(c2, L, to_dev(u), to_dev(v), md)), Jv) < 1e-5
    if nlevels > 1:
        out = []
        for path in (0, 1):
            c2 = make_ctx(w, kernel_path=path)
            api.mg_setup(c2, to_dev(u), md)
            out.append(to_np(api.mg_smooth(c2, L, to_dev(v), torch.zeros_like(to_dev(v)), 3, True)))
        assert rel(out[0], out[1]) < 1e-10
