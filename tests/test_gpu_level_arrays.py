"""The size check of a level's arrays holds on every call, also after calls
with arrays of the right size, for each level and for closed contexts."""
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

from _common import make_ctx
from paper_2103_13890_amd import api
from paper_2103_13890_amd import workloads as W


@pytest.mark.parametrize('name', ['bratu2d-32', 'plap3d-128'])
def test_sizes(name):
    ctx = make_ctx(W.WORKLOADS[name])
    for level in range(ctx.nlevels):
        u = ctx.empty(level)
        api.jfnk_residual(ctx, level, u)
        api.jfnk_residual(ctx, level, u)
        with pytest.raises(ValueError):
            api.jfnk_residual(ctx, level, ctx.empty((level + 1) % ctx.nlevels))
    with pytest.raises(api.JfnkError):
        api.jfnk_residual(ctx, ctx.nlevels, u, F=u)
    ctx.close()
    with pytest.raises(api.JfnkError):
        api.jfnk_residual(ctx, level, u, F=u)
