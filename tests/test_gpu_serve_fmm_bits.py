"""GPU: requests on one FMM geometry that the server merges into one item give the bits of the same
request alone, in both kinds and precisions (the near field takes four, two or one right-hand side per
workgroup, and one alone has a form of its own outside the server)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("precision", [bie2d.BIE_FP64, bie2d.BIE_MIXED])
def test_merged_fmm_requests_have_the_bits_of_lone_ones(kind, precision):
    rng = np.random.default_rng(12 + kind)
    g = bie2d.Geometry.from_curves(wl.mixed_grid(rng, 12, np.full(12, 96)))
    opts = bie2d.default_opts(precision=precision, method=bie2d.BIE_FMM, tol=1e-11, restart=40,
                              fmm_order=32, fmm_leaf=32)
    data = [rng.standard_normal((1 + i % 2, g.N * (3 if kind else 1))) for i in range(8)]
    srv = bie2d.Server(opts)
    alone = [srv.wait(srv.submit(g, kind, q), timeout=100)[0] for q in data]
    tickets = [srv.submit(g, kind, q) for q in data]
    got = [srv.wait(t, timeout=100) for t in tickets]
    srv.close()
    assert max(info["inflight"] for _, info in got) > 2  # some were merged
    for i, ((out, info), ref) in enumerate(zip(got, alone)):
        assert info["status"] == 0, info
        assert np.array_equal(out, ref), i
