"""GPU: the batched apply's right-hand side groups. A column of an item with any number of right-hand
sides (every group size and remainder) matches the oracle and the column alone: for mobility to
the last bit, for elastance up to the right-hand side's rounding (the single-geometry apply that
forms it has a form of its own for one charge vector)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import nystrom as ny  # noqa: E402
from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("kind,nodes", [(0, [3, 127, 130]), (0, [300, 257, 64]), (1, [3, 65]),
                                        (1, [256, 200, 130])])
def test_columns_do_not_depend_on_their_group(kind, nodes):
    rng = np.random.default_rng(len(nodes) + kind)
    c = wl.mixed_grid(rng, len(nodes), np.array(nodes))
    geo = ny.geometry_of(c)
    g = bie2d.Geometry.from_curves(c)
    width = g.N * (3 if kind else 1)
    data = torch.as_tensor(rng.standard_normal((17, width)), device="cuda")
    o = bie2d.default_opts(tol=1e-12, restart=60, max_iter=2000)
    b = bie2d.Batch()
    alone = [bie2d.bie_batch_solve(b, [(g, kind, data[r:r + 1].contiguous())], o)[0][0] for r in range(17)]
    solve, key = (ny.mobility_solve, "VW") if kind else (ny.elastance_solve, "phi")
    for r in (0, 16):
        ref = solve(geo, data[r].cpu().numpy())[key].reshape(-1)
        assert np.abs(alone[r].cpu().numpy()[0] - ref).max() < 1e-10 * np.abs(ref).max()
    for n in (2, 3, 4, 5, 7, 8, 9, 15, 17):
        out = bie2d.bie_batch_solve(b, [(g, kind, data[:n].contiguous())], o)[0][0]
        for r in range(n):
            off = float((out[r] - alone[r][0]).abs().max() / alone[r][0].abs().max())
            assert off == 0.0 if kind else off < 1e-12, (n, r, off)
