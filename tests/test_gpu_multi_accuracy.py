"""GPU: the float32 sweeps of a batch are no further from float64 than the single-geometry float32
sweep on the same geometry. With one refinement around an inner solve of a fixed number of steps,
more than it needs, the residual that a solve reports is the error of its float32 operator (2e-8 to
1e-7). Geometries above the size of the one-launch float64 apply; the errors are root mean squares
over thousands of nodes, equal up to 2% for two sweeps of the same accuracy. (Laplace items of fewer
than 32 nodes per body stay in float64.)"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


def errors(kind, bodies, nodes, groups):
    """Residuals after one refinement: [batch], [single geometry], one entry per group of inputs."""
    rng = np.random.default_rng(bodies)
    g = bie2d.Geometry.from_curves(wl.mixed_grid(rng, bodies, np.full(bodies, nodes)))
    X = torch.as_tensor(rng.standard_normal((57, bodies * (3 if kind else 1))), device="cuda")
    o = bie2d.default_opts(precision=bie2d.BIE_MIXED, mixed_strategy=bie2d.BIE_MIXED_REFINE,
                           precond=bie2d.BIE_PRECOND_BLOCK, inner_tol=1e-15, tol=1e-16, max_refine=1,
                           restart=80, max_iter=80)
    solve = bie2d.bie_mobility_solve if kind else bie2d.bie_elastance_solve
    b = bie2d.Batch()
    off, ref = [], []
    for r0, r1 in groups:
        x = X[r0:r1].contiguous()
        off.append(bie2d.bie_batch_solve(b, [(g, kind, x)], o, allow_noconv=True)[2][0])
        ref.append(solve(g, x, o, allow_noconv=True)[1]["rel_residual"])
    assert max(ref) < 1e-6  # (the inner solves are done)
    return off, ref


@pytest.mark.parametrize("kind,bodies,nodes", [(0, 520, 8)] + [
    (kind, *size) for kind in (0, 1) for size in ((290, 16), (160, 32), (70, 64), (45, 96), (17, 256))])
def test_batch_float32_error(kind, bodies, nodes):
    off, ref = errors(kind, bodies, nodes, ((0, 32), (32, 57)))  # full groups of 16, and nine in one
    assert np.mean(off) < 1.02 * np.mean(ref), (off, ref)


@pytest.mark.parametrize("bodies,nodes", [(64, 195), (390, 32)])
def test_large_item_float32_error(bodies, nodes):
    off, ref = errors(1, bodies, nodes, ((0, 1), (1, 8), (8, 19)))  # the vector sweep's groups of 4
    assert np.mean(off) < 1.02 * np.mean(ref), (off, ref)
