"""GPU: an FMM apply reserves no memory for the direct sweep's partial sums: 12 bytes per unknown and
right-hand side (strengths) and one partial sum per unknown for up to 8 (Laplace) or 4 (Stokes), plus
the eighth that every buffer has to spare."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("kind", [0, 1])
def test_fmm_apply_reserves_its_own_workspace_only(kind):
    rng = np.random.default_rng(2)
    g = bie2d.Geometry.from_curves(wl.mixed_grid(rng, 200, np.full(200, 200)))
    n = g.M * (1 + kind)
    mu = torch.as_tensor(rng.standard_normal((1, n)), device="cuda")
    before = g.device_bytes()
    (bie2d.bie_stokes_apply if kind else bie2d.bie_laplace_apply)(g, mu, bie2d.BIE_FP64, bie2d.BIE_FMM)
    need = 12 * n + 8 * (4 if kind else 8) * n
    assert g.device_bytes() - before <= need + need // 8 + 8192
