"""GPU: the direct read-off where its source splits begin: 510 to 1,282 nodes (one, four and five splits, with
and without a remainder), against the oracle's solves (the 1e-9 of the step tests, which solve
the same two discs)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import nystrom as ny  # noqa: E402
from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("n", [255, 511, 512, 513, 640, 641])
def test_read_off_splits(n):
    c = wl.two_discs(0.05, n)
    geo = ny.geometry_of(c)
    g = bie2d.Geometry.from_curves(c)
    rng = np.random.default_rng(n)
    o = bie2d.default_opts(tol=1e-12, restart=100)
    Q, FT = rng.standard_normal((2, 2)), rng.standard_normal((2, 6))
    phi = bie2d.bie_elastance_solve(g, torch.as_tensor(Q, device="cuda"), o)[0].cpu().numpy()
    VW = bie2d.bie_mobility_solve(g, torch.as_tensor(FT, device="cuda"), o)[0].cpu().numpy()
    for r in range(2):
        ref = ny.elastance_solve(geo, Q[r])["phi"].reshape(-1)
        assert np.abs(phi[r].reshape(-1) - ref).max() < 1e-9 * np.abs(ref).max()
        ref = ny.mobility_solve(geo, FT[r])["VW"].reshape(-1)
        assert np.abs(VW[r].reshape(-1) - ref).max() < 1e-9 * np.abs(ref).max()
