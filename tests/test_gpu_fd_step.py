"""The FD step of a single J v, summed in one pass over u and v: eps against
root (1 + ||u||) / ||v|| (or the mean form) over the DoFs of u and every entry
of v, on grids of less than one block, of remainders and of several trips of
the grid-stride loop.  A sum of positive terms in a tree rounds by at most
~30 x 1.1e-16; the bar is 1e-13.  With and without a given A(u) the result is
the same bit for bit in both FD forms.
"""
import numpy as np
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

from _common import make_ctx, oracle_grid, to_dev, to_np
from paper_2103_13890_amd import api
from paper_2103_13890_amd import workloads as W


@pytest.mark.parametrize('prec', ['f64', 'f32'])
@pytest.mark.parametrize('n,faces,mode', [((3, 2), W.ALL2, 0), ((17, 31), [(0, 0)], 1), ((896, 704), W.ALL2, 0),
                                          ((20, 9, 11), [(0, 0), (1, 0)], 0), ((6, 5, 4), [(0, 0)], 1)])
def test_step(prec, n, faces, mode):
    beam = len(n) == 3 and n[0] == 6
    w = dict(W.WORKLOADS['bratu2d-32'])
    w.update(kind='neohooke' if beam else 'plap', params=(1.0, 0.3) if beam else (3.0, 0.1), n=n, h=1.0 / max(n),
             faces=faces, nlevels=5 if n[0] > 100 else 1)
    L = w['nlevels'] - 1
    dt = torch.float64 if prec == 'f64' else torch.float32
    rng = np.random.default_rng(7)
    shape = ((3,) if beam else ()) + oracle_grid(w).dof_mask().shape
    u, v = 0.01 * rng.standard_normal(shape), rng.standard_normal(shape)
    ud, vd = to_dev(u, dt), to_dev(v, dt)
    dof = oracle_grid(w).dof_mask()
    x = to_np(ud)[..., dof]
    root = 1e-6
    num = root * (1.0 + np.sqrt(np.sum(x * x))) if mode == 0 else root * np.mean(1.0 + np.abs(x))
    eps = num / np.sqrt(np.sum(to_np(vd) ** 2))
    for form in (1, 2):
        ctx = make_ctx(w, fd_form=form, fd_root=root, eps_mode=mode)
        Jv, got = api.jfnk_jv(ctx, L, ud, vd, want_eps=True)
        assert abs(got - eps) < 1e-13 * eps
        Au = api.jfnk_residual(ctx, L, ud)
        assert torch.equal(api.jfnk_jv(ctx, L, ud, vd, Au=Au), Jv)
