"""Transfers at the edges of their kernels, against the oracle: grids of two
elements, coarse rows shorter than, equal to and longer than a wavefront (the
left neighbour of a pair crosses lanes), several trips of the grid-stride loop,
one and three components, Dirichlet and natural faces.  A node takes at most 27
rounded multiply-adds: 1e-14 in FP64 and 1e-6 in FP32, in norm.
"""
import numpy as np
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

from _common import make_ctx, rel, to_dev, to_np
from oracle import transfer as OT
from oracle.fe import Grid
from paper_2103_13890_amd import api
from paper_2103_13890_amd import workloads as W

X0 = [(0, 0)]


SCALAR = [((2, 2), 2, W.ALL2), ((62, 4), 2, X0), ((124, 128), 3, W.ALL2), ((128, 252), 3, [(1, 1)]),
          ((256, 256, 80), 5, W.ALL3)]
BOTH = [((2, 2, 2), 2, X0), ((126, 4, 6), 2, W.ALL3), ((128, 8, 12), 2, X0), ((124, 60, 20), 3, [(0, 1), (2, 0)])]


@pytest.mark.parametrize('kind,n,nl,faces', [('plap', *a) for a in SCALAR + BOTH] + [('neohooke', *a) for a in BOTH])
def test_transfers(kind, n, nl, faces):
    w = dict(W.WORKLOADS['bratu2d-32'])
    w.update(kind=kind, params=(1.0, 0.3) if kind == 'neohooke' else (3.0, 0.1), n=n, h=1.0 / max(n), faces=faces,
             nlevels=nl)
    ctx = make_ctx(w)
    fine, coarse = Grid(n, 1.0 / max(n), faces), Grid([k // 2 for k in n], 2.0 / max(n), faces)
    rng = np.random.default_rng(3)
    lead = (3,) if kind == 'neohooke' else ()
    r, c, s = (rng.standard_normal(lead + g.node_shape) for g in (fine, coarse, fine))
    for dt, tol in ((torch.float64, 1e-14), (torch.float32, 1e-6)):
        rd, cd, sd = (to_dev(t, dt) for t in (r, c, s))
        R, S = OT.restrict(coarse, fine, to_np(rd)), to_np(sd)
        S = np.where(fine.dirichlet_mask(), 0.0, S + OT.prolong(coarse, fine, to_np(cd)))
        assert rel(to_np(api.mg_restrict(ctx, nl - 1, rd)), R) < tol
        api.mg_prolong_add(ctx, nl - 1, cd, sd)
        assert rel(to_np(sd), S) < tol
