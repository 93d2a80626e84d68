"""A Bratu state of minus infinity at a node: its exponential is 0 at every Gauss
point around, as for any state far below 0, and not a NaN.  J v in the
difference form and J^T lam hold the state in the exponential alone, so they are
those of a large negative value there, bit for bit; so are F, and J v of such a
direction, at the nodes whose stiffness row has no entry for the bad node (in 3D
its edge neighbours and everything past its elements); the others are not finite.
All kernels: few lanes per node, node-centric, rows (2D), waves (3D).
"""
import numpy as np
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

from _common import make_ctx, to_dev
from paper_2103_13890_amd import api
from paper_2103_13890_amd import workloads as W


@pytest.mark.parametrize('n,path', [((10, 9, 8), 0), ((30, 12, 6), 1), ((30, 12, 6), 2), ((64, 30, 20), 0),
                                    ((20, 9), 0), ((150, 140), 0), ((150, 140), 1)])
@pytest.mark.parametrize('dt,large', [(torch.float64, 1e300), (torch.float32, 1e30)])
def test_minus_infinity(n, path, dt, large):
    dim = len(n)
    w = dict(W.WORKLOADS['plap3d-128' if dim == 3 else 'bratu2d-32'])
    faces = [(1, 0)]
    w.update(kind='bratu', params=(2.0,), n=n, h=1.0 / max(n), faces=faces, nlevels=1,
             options=dict(vcycle_prec=0, coarse_rtol=1e-6, kernel_path=path, fd_form=2))
    ctx = make_ctx(w)
    u = 0.4 * W.rough_state(n, [], 191)
    v = to_dev(W.normal_vector(n, faces, 192))
    at = tuple(k // 2 for k in reversed(n))
    ui, ul = u.copy(), u.copy()
    ui[at], ul[at] = -np.inf, -large
    UI, UL, V = to_dev(ui, dt), to_dev(ul, dt), v.to(dt)
    a, b = (api.jfnk_jv(ctx, 0, x, V, None, None, 1e-4) for x in (UI, UL))
    assert bool(torch.isfinite(b).all()) and torch.equal(a, b)
    if dt == torch.float64:
        a, b = (api.jfnk_vjp(ctx, 0, 0, x, V) for x in (UI, UL))
        assert bool(torch.isfinite(b).all()) and torch.equal(a, b)
    off = sum(abs(i - k) for i, k in zip(np.indices(u.shape), at))
    near = np.max([abs(i - k) for i, k in zip(np.indices(u.shape), at)], axis=0) <= 1
    hit = near & (off != 1) if dim == 3 else near
    for call in (lambda x: api.jfnk_residual(ctx, 0, x),
                 lambda x: api.jfnk_jv(ctx, 0, to_dev(0 * u, dt), x, None, None, 1e-4)):
        a, b = (call(x).cpu().numpy() for x in (UI, UL))
        assert np.array_equal(~np.isfinite(a), hit)
        assert np.array_equal(a[~hit], b[~hit])
