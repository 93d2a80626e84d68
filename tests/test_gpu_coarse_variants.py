"""The one-workgroup coarse solver's variants: every kind with its exponents, both
FD forms, both precisions, 1, 2 and 4 nodes per thread, plain CG and CG-QN with
the pairs in registers and in global memory (a recording solve and one with
the pairs).

At u = 0 with delta = 1 the Jacobian is the Laplacian (weighted by e^m, less
lam times the mass for Bratu) and the residual is linear in the FD steps up to
their squares (Bratu: up to half a step): a node moves by less than eps = 1.5e-8
or 3.5e-4, a gradient by eps / h < 1.6e-2.  A(0) = 0, so that the black-box quotient
cancels nothing (but for Bratu, which takes the difference form here).  The
solver stops at ||r|| <= rtol ||b|| by its recursion; the residual checked is
b - J s in FP64.  They part by at most iterations x rounding x condition number
(60, 0.5 (n + 1)^2 < 1100): 7e-12 in FP64, 4e-3 in FP32, and by the steps' squares,
2.6e-4 of J s, which is b there.  Twice rtol = 1e-6 and 1e-2 hold that.
"""
import numpy as np
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

from _common import make_ctx, to_dev
from paper_2103_13890_amd import api
from paper_2103_13890_amd import workloads as W


@pytest.mark.parametrize('kind,params', [('bratu', (2.0,)), ('plap', (3.0, 1.0)), ('plap', (2.5, 1.0)),
                                         ('plap', (2.0, 1.0)), ('plap', (1.0, 1.0)), ('plap_gauss', (3.0, 1.0)),
                                         ('plap_gauss', (1.5, 1.0)), ('invcoef', ())])
@pytest.mark.parametrize('coarse,qn', [((20, 20), 0), ((7, 7, 7), 0), ((31, 30), 0), ((9, 9, 8), 0), ((44, 44), 0),
                                       ((11, 11, 13), 0), ((25, 25), 20), ((8, 8, 8), 20), ((31, 30), 20),
                                       ((44, 44), 24)])
@pytest.mark.parametrize('prec', [0, 1])
def test_coarse_variants(kind, params, coarse, qn, prec):
    n = tuple(2 * k for k in coarse)
    w = dict(W.WORKLOADS['plap3d-128' if len(n) == 3 else 'bratu2d-32'])
    faces = [(a, s) for a in range(len(n)) for s in range(2)]
    rtol = 1e-6 if prec == 0 else 1e-2
    w.update(kind=kind, params=params, n=n, h=1.0 / max(n), faces=faces, nlevels=2,
             options=dict(vcycle_prec=prec, coarse_rtol=rtol, power_fixed=1, power_maxit=2, coarse_qn=qn))
    m = None
    if kind == 'invcoef':
        x = np.meshgrid(*[np.arange(k + 1) * w['h'] for k in n], indexing='ij')
        m = to_dev((0.3 * np.cos(2.0 * x[0] + x[1])).T)
    for form in (1, 2) if kind != 'bratu' else (2,):
        ctx = make_ctx(w, fd_form=form)
        api.mg_setup(ctx, ctx.empty(1), m)
        m0 = None if m is None else api.mg_get_level(ctx, 0, 'kap').double().log()
        dt = torch.float64 if prec == 0 else torch.float32
        for seed in (301, 302):
            b = api.mg_restrict(ctx, 1, to_dev(W.normal_vector(n, faces, seed), dt))
            s, shift, its, rounds = api.mg_coarse_solve(ctx, b)
            assert shift == 0.0 and rounds == 0 and its > 1
            Js = api.jfnk_jv(ctx, 0, ctx.empty(0), s.double(), m0)
            r = float((b.double() - Js).norm() / b.double().norm())
            assert r <= 2 * rtol, (form, seed, its, r)
