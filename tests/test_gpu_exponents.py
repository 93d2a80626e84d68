"""The p-Laplacians' exponents, each of which has kernels of its own: 3, 2, 1 and
the general one (2.5, 4, and 1.5 beside them), at both quadratures.

Coarse solves on grids past the small solver's size, where the element
quotient is compiled per exponent.  The stop is ||b - J s|| <= rtol ||b||, and
the residual is formed afterwards from one product J s of the library.  The two
differ by the curvature along the FD steps, which move the state by
sqrt(eps) (1 + ||x||) / sqrt(nodes) or 1e-4 (FP32) and 1e-8 (FP64) per node:
under 1e-2 and 1e-6 of its gradients at this h.  Twice rtol = 1e-4 in FP64 and
five times 1e-2 in FP32 hold both with room; another exponent's quotient is off
by its whole size.
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

EXPONENTS = [(3.0, 0.1), (2.0, 0.1), (1.0, 1.0), (2.5, 0.1), (4.0, 0.1), (1.5, 0.1)]


def _workload(kind, params, n, faces, nlevels, **options):
    w = dict(W.WORKLOADS['plap3d-128' if len(n) == 3 else 'bratu2d-32'])
    w.update(kind=kind, params=params, n=n, h=1.0 / max(n), faces=faces, nlevels=nlevels,
             options=dict(vcycle_prec=0, coarse_rtol=1e-6, power_fixed=1, power_maxit=3, **options))
    ax = [np.arange(k + 1) * w['h'] for k in n]
    x = np.meshgrid(*ax, indexing='ij')
    u = (0.4 * np.sin(3.0 * x[0]) * np.cos(2.0 * x[1])).T + 1e-2 * w['h'] * W.rough_state(n, [], 141)
    return w, u, W.normal_vector(n, faces, 142)


@pytest.mark.parametrize('params', EXPONENTS)
@pytest.mark.parametrize('n', [(48, 44), (14, 13, 12)])
@pytest.mark.parametrize('prec', [0, 1])
def test_coarse_solves(params, n, prec):
    faces = [(a, s) for a in range(len(n)) for s in range(2)]
    rtol, bar = (1e-4, 2e-4) if prec == 0 else (1e-2, 5e-2)
    w, u, v = _workload('plap_gauss', params, tuple(2 * k for k in n), faces, 2)
    w['options'].update(vcycle_prec=prec, coarse_rtol=rtol, fd_form=2)
    ctx = make_ctx(w)
    dt = torch.float64 if prec == 0 else torch.float32
    api.mg_setup(ctx, to_dev(u))
    b = api.mg_restrict(ctx, 1, to_dev(v, dt))
    s, shift, its, rounds = api.mg_coarse_solve(ctx, b)
    assert shift == 0.0 and rounds == 0 and its > 1
    Js = api.jfnk_jv(ctx, 0, api.mg_get_level(ctx, 0, 'x'), s)
    r = (b - Js).double()
    assert float(r.norm()) <= bar * float(b.double().norm())


@pytest.mark.parametrize('kind', ['plap', 'plap_gauss'])
@pytest.mark.parametrize('params', EXPONENTS)
@pytest.mark.parametrize('n', [(30, 12, 6), (62, 10, 8), (96, 92, 64)])
def test_wave_kernels(kind, params, n):
    """The 3D wave kernel's instances against the node-centric kernel, which reads
    the exponent: F, J v in both forms and the VJP to 1e-12 in FP64 (the same
    element values summed in another order; the black-box quotient divides a
    difference of two such sums by a step of 1e-4, so 1e-8), a smoother of degree 4 to
    1e-10, FP32 to 1e-4 (J v by the difference form)."""
    nlevels = 3 if n[0] == 96 else 2      # the coarsest grid has at most 65,536 nodes
    top = nlevels - 1
    w, u, v = _workload(kind, params, n, [(0, 0), (1, 0), (2, 1)], nlevels)
    U, V = to_dev(u), to_dev(v)

    def diff(call):
        a, b = call(2), call(1)
        return float((a - b).norm() / b.norm())

    def jv(path, form, x, d):
        return api.jfnk_jv(make_ctx(w, kernel_path=path, fd_form=form), top, x, d, None, None, 1e-4)

    def smooth(path):
        c = make_ctx(w, kernel_path=path)
        api.mg_setup(c, U)
        return api.mg_smooth(c, top, V, torch.zeros_like(V), 4, True)
    assert diff(lambda p: api.jfnk_residual(make_ctx(w, kernel_path=p), top, U)) < 1e-12
    assert diff(lambda p: api.jfnk_vjp(make_ctx(w, kernel_path=p), top, 0, U, V)) < 1e-12
    assert diff(lambda p: jv(p, 2, U, V)) < 1e-12
    assert diff(lambda p: jv(p, 1, U, V)) < 1e-8
    assert diff(smooth) < 1e-10
    assert diff(lambda p: api.jfnk_residual(make_ctx(w, kernel_path=p), top, U.float())) < 1e-4
    assert diff(lambda p: jv(p, 2, U.float(), V.float())) < 1e-4


@pytest.mark.parametrize('params', EXPONENTS)
@pytest.mark.parametrize('n', [(140, 131), (700, 41)])
def test_2d_fp32_gauss(params, n):
    """The node kernel's instances on 2D FP32 levels of the Gauss-point kind, against
    the oracle at the same FP32 state and direction.  The fluxes come from
    differences of neighbours, which FP32 holds to a rounding: about 4 x 6e-8 of a
    flux, h / h^2 of which stays in F and J v: 1.7e-4 / 10 at h = 1/700 with
    second derivatives near 10; 1e-4, the bar of the other FP32 parity tests."""
    w, u, v = _workload('plap_gauss', params, n, [(0, 0), (1, 1)], 1, fd_form=2)
    g, pb = oracle_grid(w), oracle_problem(w)
    ctx = make_ctx(w)
    U, V = to_dev(u, torch.float32), to_dev(v, torch.float32)
    u, v = to_np(U), to_np(V)
    assert rel(to_np(api.jfnk_residual(ctx, 0, U)), OP.residual(pb, g, u, None)) < 1e-4
    assert rel(to_np(api.jfnk_jv(ctx, 0, U, V)), OD.jvp(pb, g, u, v)) < 1e-4
