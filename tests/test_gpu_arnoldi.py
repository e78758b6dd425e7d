"""GPU: the Arnoldi steps at the sizes where their kernels change: one chunk of 1,024 unknowns per
system (one launch per step), up to eight chunks (the small kernel adds the chunk sums), more; and
cycles past 48 vectors. Solves against the oracle, and the same bits whichever kernels a batch's
longest system selects."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import nystrom as ny  # noqa: E402
from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")


@pytest.mark.parametrize("n", [3, 255, 256, 257])  # 4 n unknowns around 1,024
@pytest.mark.parametrize("strategy", [None, bie2d.BIE_MIXED_RELAXED, bie2d.BIE_MIXED_REFINE])
def test_mobility_steps_vs_oracle(n, strategy):
    c = wl.two_discs(0.05, n)  # about 66 steps once resolved
    geo = ny.geometry_of(c)
    g = bie2d.Geometry.from_curves(c)
    FT = wl.random_forces(np.random.default_rng(n), 2, 2)
    o = bie2d.default_opts(tol=1e-12, restart=100)
    if strategy is not None:
        o.precision, o.mixed_strategy = bie2d.BIE_MIXED, strategy
    VW, info = bie2d.bie_mobility_solve(g, dev(FT), o)
    for r in range(2):
        ref = ny.mobility_solve(geo, FT[r])["VW"].reshape(-1)
        assert np.abs(VW[r].cpu().numpy() - ref).max() < 1e-9 * np.abs(ref).max(), info


@pytest.mark.parametrize("strategy", [None, bie2d.BIE_MIXED_RELAXED, bie2d.BIE_MIXED_REFINE])
def test_step_kernels_give_the_same_bits(strategy):
    """Systems of 512, 1,024 and 1,300 unknowns alone and beside one of 8,192 or 8,320."""
    rng = np.random.default_rng(9)
    o = bie2d.default_opts(tol=1e-12, restart=60, max_iter=2000)
    if strategy is not None:
        o.precision, o.mixed_strategy = bie2d.BIE_MIXED, strategy
    small = [(wl.mixed_grid(rng, 4, np.full(4, 128)), 0), (wl.two_discs(0.05, 256), 1),
             (wl.mixed_grid(rng, 5, np.full(5, 130)), 1)]
    large = [wl.mixed_grid(rng, 64, np.full(64, 128)), wl.mixed_grid(rng, 65, np.full(65, 128))]
    items = [(bie2d.Geometry.from_curves(c), k, dev(rng.standard_normal((2, c.nbodies * (3 if k else 1)))))
             for c, k in small]
    b = bie2d.Batch()
    alone = [bie2d.bie_batch_solve(b, [it], o)[0][0] for it in items]
    for c in large:
        big = (bie2d.Geometry.from_curves(c), 0, dev(rng.standard_normal((1, c.nbodies))))
        mix, _, _ = bie2d.bie_batch_solve(b, items + [big], o)
        for a, m in zip(alone, mix):
            assert torch.equal(a, m)
