"""The one-workgroup coarse solver at the edges of its shapes, against the
oracle: 512, 529, 1024 and 1056 nodes (one, two and four nodes per thread),
2025 and 2116 (the last small level and the first generic one), and with
CG-QN the pairs in registers (up to 40 columns on 768 nodes) and in global
memory (784 nodes; 24 and 32 pairs).

The problem is linear (p-Laplacian with p = 2, delta = 0: the Q1 Laplacian),
so the FD quotient is exact up to rounding and both sides solve the same
system to ||r|| <= 1e-10 ||b||.  The corrections then differ by at most
2e-10 times the condition number, below 0.5 (n + 1)^2 < 1100 for the unit
square's n x n Laplacian: 1e-6 leaves a factor of five.
"""
import numpy as np
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

from _common import make_ctx, oracle_grid, oracle_mg_options, oracle_problem, rel, to_dev, to_np
from oracle import mg as OM
from paper_2103_13890_amd import api
from paper_2103_13890_amd import workloads as W


@pytest.mark.parametrize('coarse,qn', [((7, 7, 7), 0), ((22, 22), 0), ((31, 31), 0), ((31, 32), 0), ((44, 44), 0),
                                       ((45, 45), 0), ((3, 2), 4), ((25, 25), 20), ((26, 27), 20), ((27, 27), 20),
                                       ((25, 25), 24), ((31, 32), 20), ((25, 25), 32)])
def test_coarse_shapes(coarse, qn):
    w = W.scaled('bratu2d-32' if len(coarse) == 2 else 'plap3d-128', tuple(2 * k for k in coarse), nlevels=2,
                 vcycle_prec=0)
    w.update(kind='plap', params=(2.0, 0.0))
    g = oracle_grid(w)
    grids = OM.make_grids(g, 2)
    opts = oracle_mg_options(w, fd_root=1e-2, coarse_rtol=1e-10, power_fixed=True, power_maxit=2, coarse_qn=qn)
    ctx = make_ctx(w, fd_root=1e-2, coarse_rtol=1e-10, power_fixed=1, power_maxit=2, coarse_qn=qn)
    u = np.zeros(g.node_shape)
    api.mg_setup(ctx, to_dev(u))
    pb = oracle_problem(w)
    state = {}
    levels = OM.mg_setup(pb, grids, u, None, opts, None, None, state)
    rng = np.random.default_rng(77)
    for _ in range(2 if qn else 1):
        r = rng.normal(size=grids[0].node_shape)
        r[grids[0].dirichlet_mask()] = 0
        s, shift, its, rounds = api.mg_coarse_solve(ctx, to_dev(r))
        ref, shift_o, iters_o = OM.coarse_solve(lambda x: OM.level_jv(pb, levels[0], x), r, grids[0].n_dof(), opts,
                                                None, state)
        assert rounds == 0 and shift == 0.0
        assert rel(to_np(s), ref) < 1e-6, (its, iters_o)
