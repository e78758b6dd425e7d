"""GPU: batches of more items than have precisions of their own (1,024) take the float32 sweeps like
smaller ones: launches of the float32 pair sweeps of each kind, and the same answers as a batch of a
few items (to 1e-10 of tolerance times the amplification of 1e2 of the preconditioner's tests)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("items", [1024, 1025, 1100])
def test_float32_sweeps_of_many_items(kind, items):
    rng = np.random.default_rng(kind)
    g = bie2d.Geometry.from_curves(wl.mixed_grid(rng, 3, np.full(3, 64)))
    X = torch.as_tensor(rng.standard_normal((8 if kind else 25, g.N * (3 if kind else 1))), device="cuda")
    o = bie2d.default_opts(tol=1e-10, restart=30, precision=bie2d.BIE_MIXED)
    b = bie2d.Batch()
    ref = bie2d.bie_batch_solve(b, [(g, kind, X)], o)[0][0]
    k = bie2d.BIE_K_FAR_STOKES_F32 if kind else bie2d.BIE_K_FAR_LAPLACE_F32
    bie2d.bie_profile_select([k])
    bie2d.bie_profile_enable(True)
    out = bie2d.bie_batch_solve(b, [(g, kind, X)] * items, o)[0]
    launches = bie2d.bie_profile_read(k)["launches"]
    bie2d.bie_profile_enable(False)
    bie2d.bie_profile_select()
    assert launches > 0
    for i in range(items):
        assert float((out[i] - ref).abs().max() / ref.abs().max()) < 1e-8, i
