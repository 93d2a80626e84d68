"""Exact VJPs on the wave (3D) and row (2D) kernels at ragged sizes, against
the oracle and, for kinds or sizes that the oracle's 3D formulas do not cover,
against the node-centric kernel of the same library: row lengths at, below
and past whole wavefronts, natural faces (the coefficient product has values
on every node, Dirichlet ones too), the smallest levels.  1e-12, the bar of
the other VJP tests.
"""
import numpy as np
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

from _common import make_ctx, oracle_grid, oracle_problem, rel, to_dev, to_np
from oracle import derivatives as OD
from paper_2103_13890_amd import api
from paper_2103_13890_amd import workloads as W


@pytest.mark.parametrize('kind,params', [('bratu', (2.0,)), ('plap', (3.0, 0.1)), ('plap', (2.5, 0.1)),
                                         ('plap', (1.0, 1.0)), ('plap_gauss', (3.0, 0.1)), ('invcoef', ())])
@pytest.mark.parametrize('n', [(64, 9, 10), (65, 8, 8), (33, 17, 12), (128, 11, 7), (32, 8, 3), (3, 2, 2), (130, 67),
                               (20, 9)])
def test_vjp_shapes(kind, params, n):
    w = dict(W.WORKLOADS['plap3d-128' if len(n) == 3 else 'bratu2d-32'])
    faces = [(0, 0), (1, 1)]
    w.update(kind=kind, params=params, n=n, h=1.0 / max(n), faces=faces, nlevels=1,
             options=dict(vcycle_prec=0, coarse_rtol=1e-6))
    g, pb = oracle_grid(w), oracle_problem(w)
    xs = g.node_coords()
    u = 0.4 * np.sin(3.0 * xs[0]) * np.cos(2.0 * xs[1]) + 1e-2 * w['h'] * W.rough_state(n, [], 51)
    lam = W.normal_vector(n, faces, 52)
    m = 0.3 * np.cos(2.0 * xs[0] + xs[1]) if kind == 'invcoef' else None
    md = None if m is None else to_dev(m)
    ctx, node = make_ctx(w), make_ctx(w, kernel_path=1)
    out = api.jfnk_vjp(ctx, 0, 0, to_dev(u), to_dev(lam), md)
    assert rel(to_np(out), to_np(api.jfnk_vjp(node, 0, 0, to_dev(u), to_dev(lam), md))) < 1e-12
    if kind != 'invcoef' or len(n) == 3:
        assert rel(to_np(out), OD.vjp(pb, g, u, lam, m)) < 1e-12
    if kind == 'invcoef':
        gm = api.jfnk_vjp(ctx, 0, 1, to_dev(u), to_dev(lam), md)
        assert rel(to_np(gm), to_np(api.jfnk_vjp(node, 0, 1, to_dev(u), to_dev(lam), md))) < 1e-12
        if len(n) == 3:
            assert rel(to_np(gm), OD.vjp_coef(pb, g, u, lam, m)) < 1e-12
        assert torch.equal(api.jfnk_coef_gradient(ctx, to_dev(u), md, to_dev(lam)), -gm)
