"""Neo-Hookean element kernels at the edges of their shapes, against the
oracle: rows that fill a block (256 elements), leave lanes idle (20, 36) and
are split over blocks with a seam (257, 300), levels on both sides of the
lines between the wavefront-per-node, split and whole-element kernels, and
natural and Dirichlet faces.  F and J^T lam in FP64 to 1e-12 relative (sums of
some 100 products with rounding 1e-16 each), J v at the step
1e-2 (1 + ||u||)/||v|| likewise, the FP32 residual to 1e-5 (100 roundings of
6e-8).  The residual without a context gives the same bits.
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


@pytest.mark.parametrize('n,faces', [((5, 4, 4), [(0, 0)]), ((20, 10, 10), [(0, 0), (1, 1)]), ((36, 30, 31), [(0, 0)]),
                                     ((256, 12, 12), [(0, 0), (0, 1)]), ((257, 12, 12), [(0, 0)]),
                                     ((300, 12, 9), [(2, 0)]), ((520, 9, 8), [(0, 0)])])
def test_nh_shapes(n, faces):
    w = dict(W.WORKLOADS['neohooke-256x64'])
    w.update(n=n, h=1.0 / n[1], faces=faces, nlevels=1, options=dict(vcycle_prec=0, coarse_rtol=1e-6, fd_form=2))
    ctx = make_ctx(w)
    g, pb = oracle_grid(w), oracle_problem(w)
    xs = g.node_coords()
    bump = np.sin(0.7 * xs[0]) * np.cos(xs[1]) * (1.0 + xs[2])
    u = np.stack([0.03 * bump, -0.02 * bump, 0.025 * bump]) + 2e-3 * w['h'] * W.rough_state(n, [], 31, ncomp=3)
    v = W.normal_vector(n, faces, 32, ncomp=3)
    b = 0.1 * W.normal_vector(n, faces, 33, ncomp=3)
    F = OP.residual(pb, g, u, b)
    Fd = api.jfnk_residual(ctx, 0, to_dev(u), b=to_dev(b))
    assert rel(to_np(Fd), F) < 1e-12
    assert torch.equal(api.jfnk_residual_static(ctx.problem, 0, to_dev(u), to_dev(b)), Fd)
    F32 = api.jfnk_residual(ctx, 0, to_dev(u, torch.float32), b=to_dev(b, torch.float32))
    assert rel(to_np(F32), F) < 1e-5
    assert rel(to_np(api.jfnk_vjp(ctx, 0, 0, to_dev(u), to_dev(v))), OD.vjp(pb, g, u, v)) < 1e-12
    eps = 1e-2 * (1.0 + np.linalg.norm(u)) / np.linalg.norm(v)
    Jv = (OP.residual(pb, g, u + eps * v, None) - OP.residual(pb, g, u, None)) / eps
    assert rel(to_np(api.jfnk_jv(ctx, 0, to_dev(u), to_dev(v), eps_override=eps)), Jv) < 1e-12
