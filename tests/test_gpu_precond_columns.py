"""GPU: the block preconditioner over coarse sizes whose column ranges leave 0 to 7 columns past the
blocks of eight, in single solves (512 and 1,024 threads per body) and batches (256): the solution is
the unpreconditioned one's to the tolerance both are solved to (1e-12, amplified by at most the
1e2 the preconditioner's other tests allow)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("nodes", [41, 47, 53, 58, 63, 64, 126])
@pytest.mark.parametrize("kind", [0, 1])
def test_column_remainders(kind, nodes):
    rng = np.random.default_rng(nodes)
    c = wl.mobility_ellipses(nbodies=4, n=nodes)[0]
    g = bie2d.Geometry.from_curves(c)
    X = torch.as_tensor(rng.standard_normal((2, 4 * (3 if kind else 1))), device="cuda")
    solve = bie2d.bie_mobility_solve if kind else bie2d.bie_elastance_solve
    ref = solve(g, X, bie2d.default_opts(tol=1e-12, restart=100))[0]
    o = bie2d.default_opts(tol=1e-12, restart=100, precond=bie2d.BIE_PRECOND_BLOCK)
    out = solve(g, X, o)[0]
    assert float((out - ref).abs().max() / ref.abs().max()) < 1e-10
    b = bie2d.bie_batch_solve(bie2d.Batch(), [(g, kind, X)], o)[0][0]
    assert float((b - ref).abs().max() / ref.abs().max()) < 1e-10
