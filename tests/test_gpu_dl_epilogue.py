"""GPU: the double-layer epilogue's eight lanes per node: bodies below, at and above eight, node
totals that leave 1 to 7 nodes in the last workgroup, one and several splits, against the oracle's
dense operators (the tolerance of the applies' parity tests: sums of at most M float64 terms)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import dirichlet as dr  # noqa: E402
from oracle import nystrom as ny  # noqa: E402
from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("bodies,nodes", [(1, 65), (7, 53), (8, 64), (9, 75), (17, 62)])
@pytest.mark.parametrize("kind", [0, 1])
def test_dl_epilogue_lanes(bodies, nodes, kind):
    rng = np.random.default_rng(bodies)
    curves = wl.mixed_grid(rng, bodies, np.full(bodies, nodes))
    geo = ny.geometry_of(curves)
    g = bie2d.Geometry.from_curves(curves)
    n = (1 + kind) * geo["M"]
    mu = rng.standard_normal((2, n))
    D = dr.laplace_D(geo) if kind == 0 else dr.stokes_D(geo)
    A = dr.capacitance_operator(geo) if kind == 0 else dr.resistance_operator(geo)
    f = bie2d.bie_laplace_dl_apply if kind == 0 else bie2d.bie_stokes_dl_apply
    x = torch.as_tensor(mu, device="cuda")
    for op, full in ((A, True), (0.5 * np.eye(n) + D, False)):
        ref = mu @ op.T
        got = f(g, x, with_completion=full).cpu().numpy()
        assert np.abs(got - ref).max() < 1e-12 * np.abs(ref).max(), full
