"""The 3D residual's walk of a wave over several tiles (more tiles than
WAVE_BLOCKS_MAX blocks hold: 4,096 x 4,096 x 1 elements, 67,733 tiles of 4 rows or
more of fewer), through the residual without a context, against the same
element sums in plain FP64 PyTorch.  F to 1e-12, ||F||^2 to 1e-13 of the sum of
its squares, the bars of the other residual tests.
"""
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

from paper_2103_13890_amd import api


def test_walk():
    n, h, p, delta = (4096, 4096, 1), 1.0 / 4096, 3.0, 0.1
    prob = api.make_problem('plap', n, h, [(0, 0), (1, 1)], (p, delta), 1)
    g = torch.Generator(device='cuda').manual_seed(401)
    sh = tuple(k + 1 for k in reversed(n))
    u = h * torch.randn(sh, generator=g, device='cuda', dtype=torch.float64)
    b = torch.randn(sh, generator=g, device='cuda', dtype=torch.float64) * h * h
    n2 = torch.zeros(1, device='cuda', dtype=torch.float64)
    F = api.jfnk_residual_static(prob, 0, u, b, None, n2)
    # corner a: a_x + 2 a_y + 4 a_z; K u = h (u_a / 3 - (the four corners two or three axes away) / 12)
    part = [tuple(slice((a >> k) & 1, sh[2 - k] - 1 + ((a >> k) & 1)) for k in (2, 1, 0)) for a in range(8)]
    c = [u[s] for s in part]
    Ku = [h * (c[a] / 3 - (c[a ^ 3] + c[a ^ 5] + c[a ^ 6] + c[a ^ 7]) / 12) for a in range(8)]
    q = (delta ** 2 + sum(c[a] * Ku[a] for a in range(8)) / h ** 3) ** ((p - 2) / 2)
    ref = -b
    for a in range(8):
        ref[part[a]] += q * Ku[a]
    ref[:, :, 0] = 0
    ref[:, n[1], :] = 0
    assert float((F - ref).norm() / ref.norm()) < 1e-12
    s2 = float((F * F).sum())
    assert abs(float(n2[0]) - s2) <= 1e-13 * s2
