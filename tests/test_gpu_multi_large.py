"""GPU: batches of one large item, at sizes on both sides of the lines where its source splits change
(8,192 nodes, one workgroup per compute unit) and right-hand side counts on both sides of each sweep's
(float64, float32 vector, matrix cores), against float64 single solves. Both sides solve to 1e-11; the
limit 1e-9 is the amplification of 1e2 that the preconditioner's tests allow."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("kind,bodies,nodes", [(0, 43, 192), (0, 57, 192), (0, 91, 191), (1, 43, 192),
                                               (1, 91, 191)])
def test_large_items(kind, bodies, nodes):
    rng = np.random.default_rng(bodies)
    g = bie2d.Geometry.from_curves(wl.mixed_grid(rng, bodies, np.full(bodies, nodes)))
    X = torch.as_tensor(rng.standard_normal((25, bodies * (3 if kind else 1))), device="cuda")
    solve = bie2d.bie_mobility_solve if kind else bie2d.bie_elastance_solve
    ref = solve(g, X, bie2d.default_opts(tol=1e-11, restart=100))[0]
    b = bie2d.Batch()
    for n in (1, 7, 8, 11, 12, 17, 24, 25):
        o = bie2d.default_opts(tol=1e-11, restart=100, precision=bie2d.BIE_MIXED)
        out = bie2d.bie_batch_solve(b, [(g, kind, X[:n].contiguous())], o)[0][0]
        assert float((out - ref[:n]).abs().max() / ref.abs().max()) < 1e-9, n
