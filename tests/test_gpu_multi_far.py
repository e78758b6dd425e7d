"""GPU: the float32 vector sweep of large Stokes items (12,288 nodes and more): batches of 1, 3, 4, 5
and 7 right-hand sides (every group size and its remainder), bodies that are no multiple of a
wave, and requests merged by the server, against float64 single solves. Both solve to 1e-11; the
limit 1e-9 is the amplification of 1e2 that the preconditioner's tests allow."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("bodies", [63, 64])  # 12,285 and 12,480 nodes: below and above the line
def test_large_stokes_items(bodies):
    rng = np.random.default_rng(bodies)
    c = wl.mixed_grid(rng, bodies, np.full(bodies, 195))
    g = bie2d.Geometry.from_curves(c)
    X = rng.standard_normal((7, 3 * bodies))
    ref = bie2d.bie_mobility_solve(g, torch.as_tensor(X, device="cuda"),
                                   bie2d.default_opts(tol=1e-11, restart=100))[0].cpu().numpy()
    ref = ref.reshape(7, -1)
    o = bie2d.default_opts(tol=1e-11, restart=100, precision=bie2d.BIE_MIXED)
    b = bie2d.Batch()
    for n in (1, 3, 4, 5, 7):
        out = bie2d.bie_batch_solve(b, [(g, 1, torch.as_tensor(X[:n], device="cuda"))], o)[0][0]
        out = out.cpu().numpy().reshape(n, -1)
        assert np.abs(out - ref[:n]).max() < 1e-9 * np.abs(ref).max(), n
    srv = bie2d.Server(bie2d.default_opts(tol=1e-11, restart=30, precision=bie2d.BIE_MIXED))
    tickets = [srv.submit(g, 1, X[i]) for i in range(7)]
    for i, t in enumerate(tickets):
        out, info = srv.wait(t, timeout=100)
        assert info["status"] == 0, info
        assert np.abs(out.reshape(-1) - ref[i]).max() < 1e-9 * np.abs(ref).max(), i
    srv.close()
