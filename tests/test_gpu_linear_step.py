"""J v of the linear Gauss-point kind (p = 2) by the difference form: no FD step
enters it.  A state whose norm overflows makes the step infinite, one with a NaN
makes it NaN; J v is that of any other state all the same, bit for bit, but at
the nodes of the elements that hold the NaN or the infinity.
Few lanes per node, waves (3D) and rows (2D).
"""
import numpy as np
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

from _common import make_ctx, to_dev
from paper_2103_13890_amd import api
from paper_2103_13890_amd import workloads as W


@pytest.mark.parametrize('n', [(10, 8, 6), (34, 22, 14), (20, 12), (150, 140)])
@pytest.mark.parametrize('prec', [torch.float64, torch.float32])
def test_any_step(n, prec):
    w = dict(W.WORKLOADS['plap3d-128' if len(n) == 3 else 'bratu2d-32'])
    faces = [(1, 0)]
    w.update(kind='plap_gauss', params=(2.0, 0.1), n=n, h=1.0 / max(n), faces=faces, nlevels=1,
             options=dict(vcycle_prec=0, coarse_rtol=1e-6, fd_form=2))
    ctx = make_ctx(w)
    u = 0.4 * W.rough_state(n, [], 391)
    v = to_dev(W.normal_vector(n, faces, 392), prec)
    ref = api.jfnk_jv(ctx, 0, to_dev(u, prec), v).cpu().numpy()
    at = tuple(k // 2 for k in reversed(n))
    near = np.max([abs(i - k) for i, k in zip(np.indices(u.shape), at)], axis=0) <= 1
    for bad in (np.nan, np.inf, 1e200) if prec == torch.float64 else (np.nan, np.inf):
        ub = u.copy()
        ub[at] = bad
        out = api.jfnk_jv(ctx, 0, to_dev(ub, prec), v).cpu().numpy()
        hit = near if not np.isfinite(bad) else np.zeros_like(near)
        assert np.array_equal(~np.isfinite(out), hit), bad
        assert np.array_equal(out[~hit], ref[~hit]), bad
