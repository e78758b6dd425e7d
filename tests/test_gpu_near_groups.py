"""GPU: the FMM apply's near field over every grouping of right-hand sides, both precisions, leaves
with small and large neighbourhoods, and lengths far from 1, against the direct apply."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("leaf,scale", [(16, 1.0), (64, 1.0), (400, 1.0), (64, 2.0 ** -80), (64, 2.0 ** 60)])
def test_near_field_groups(kind, leaf, scale):
    rng = np.random.default_rng(leaf + kind)
    c = wl.mixed_grid(rng, 24, rng.integers(40, 700, size=24))
    for a in ("x", "y", "dx", "dy", "ddx", "ddy"):
        setattr(c, a, getattr(c, a) * scale)
    g = bie2d.Geometry.from_curves(c)
    g.set_fmm(48, leaf)
    f = bie2d.bie_laplace_apply if kind == 0 else bie2d.bie_stokes_apply
    mu = torch.as_tensor(rng.standard_normal((13, c.M * (1 + kind))), device="cuda")
    ref = f(g, mu, bie2d.BIE_FP64, bie2d.BIE_DIRECT, with_L=False)
    norm = ref.abs().max()
    for n in (1, 2, 3, 4, 5, 8, 13):
        for prec, tol in ((bie2d.BIE_FP64, 1e-12), (bie2d.BIE_MIXED, 5e-6)):
            out = f(g, mu[:n].contiguous(), prec, bie2d.BIE_FMM, with_L=False)
            assert float((out - ref[:n]).abs().max() / norm) < tol, (n, prec)
