"""NaN and infinities stay with the elements they belong to in the 3D wave
kernel: a bad value at one node of the state or of the direction makes
exactly those entries non-finite that the node-centric kernel (kernel_path 1,
which evaluates the elements of a node alone) makes so.  The node is at x = 0
in the first, middle or last row (the lane left of it holds the far end of an
earlier row), at the far end, and inside; sizes with one and several columns
of waves and with rows past the last group.  All modes: F, J v in both forms
and both precisions, the exact VJPs.
"""
import numpy as np
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

from _common import make_ctx, to_dev
from paper_2103_13890_amd import api
from paper_2103_13890_amd import workloads as W


@pytest.mark.parametrize('kind,params', [('bratu', (2.0,)), ('plap', (3.0, 0.1)), ('plap', (2.5, 0.1)),
                                         ('plap_gauss', (3.0, 0.1)), ('invcoef', ())])
@pytest.mark.parametrize('n', [(30, 12, 6), (20, 9, 7), (64, 30, 20)])
@pytest.mark.parametrize('bad', [float('nan'), float('inf')])
def test_bad_values_stay(kind, params, n, bad):
    w = dict(W.WORKLOADS['plap3d-128'])
    faces = [(1, 0)]
    w.update(kind=kind, params=params, n=n, h=1.0 / max(n), faces=faces, nlevels=1,
             options=dict(vcycle_prec=0, coarse_rtol=1e-6))
    x, y, z = np.meshgrid(*[np.arange(k + 1) * w['h'] for k in n], indexing='ij')
    u = (0.4 * np.sin(3.0 * x) * np.cos(2.0 * y + z)).T + 1e-2 * w['h'] * W.rough_state(n, [], 91)
    v = W.normal_vector(n, faces, 92)
    md = to_dev(0.3 * np.cos(2.0 * x + y).T) if kind == 'invcoef' else None
    wave = {f: make_ctx(w, kernel_path=2, fd_form=f) for f in (1, 2)}
    node = {f: make_ctx(w, kernel_path=1, fd_form=f) for f in (1, 2)}
    for at in ((n[2] // 2, n[1] // 2, 0), (n[2] // 2, n[1], 0), (0, 1, 0), (n[2], n[1] // 2, n[0]),
               (n[2] // 2, n[1] // 2, n[0] // 2)):
        ub, vb = u.copy(), v.copy()
        ub[at] = vb[at] = bad

        def same(call):
            a, b = torch.isfinite(call(wave)), torch.isfinite(call(node))
            assert torch.equal(a, b), (at, int((~a).sum()), int((~b).sum()))
        for dt in (torch.float64, torch.float32):
            U, V, UB, VB = (to_dev(t, dt) for t in (u, v, ub, vb))
            same(lambda c: api.jfnk_residual(c[2], 0, UB, md))
            for f in (1, 2):
                same(lambda c: api.jfnk_jv(c[f], 0, UB, V, md, None, 1e-4))
                same(lambda c: api.jfnk_jv(c[f], 0, U, VB, md, None, 1e-4))
        U, V, UB, VB = (to_dev(t) for t in (u, v, ub, vb))
        same(lambda c: api.jfnk_vjp(c[2], 0, 0, UB, V, md))
        same(lambda c: api.jfnk_vjp(c[2], 0, 0, U, VB, md))
        if kind == 'invcoef':
            same(lambda c: api.jfnk_coef_gradient(c[2], UB, md, V))
