"""GPU: requests that share the server with others in every stage of convergence (lengths of one to
several chunks, tolerances reached in different cycles, some systems converged while the rest of a
merged item go on) give the bits of the same request alone."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


@pytest.mark.parametrize("precision", [bie2d.BIE_FP64, bie2d.BIE_MIXED])
@pytest.mark.parametrize("restart", [12, 30])
def test_crowded_requests_have_the_bits_of_lone_ones(precision, restart):
    rng = np.random.default_rng(3)
    geoms = [bie2d.Geometry.from_curves(wl.mixed_grid(rng, n, np.full(n, 48 + 16 * n)))
             for n in (1, 2, 5)]
    reqs = []
    for i in range(48):
        k, kind = i % 3, (i // 3) % 2
        reqs.append((geoms[k], kind, rng.standard_normal((1 + i % 2, geoms[k].N * (3 if kind else 1)))))
    srv = bie2d.Server(bie2d.default_opts(precision=precision, tol=1e-11, restart=restart))
    alone = [srv.wait(srv.submit(*r), timeout=100)[0] for r in reqs]
    tickets = [srv.submit(*r) for r in reqs]
    got = [srv.wait(t, timeout=100) for t in tickets]
    srv.close()
    assert max(info["inflight"] for _, info in got) > 16
    for i, ((out, info), ref) in enumerate(zip(got, alone)):
        assert info["status"] == 0, info
        assert np.array_equal(out, ref), (i, float(np.abs(out - ref).max()))


@pytest.mark.parametrize("kind", [0, 1])
def test_refined_items_have_the_bits_of_lone_ones(kind):
    """Batches refine in cycles too: an item beside one that is exact after its first cycle (a
    lone disc has no pairs of different bodies)."""
    rng = np.random.default_rng(7)
    c = wl.mixed_grid(rng, 9, np.full(9, 128))
    g, disc = bie2d.Geometry.from_curves(c), bie2d.Geometry.from_curves(wl.single_disc(64))
    X = torch.as_tensor(rng.standard_normal((9, g.N * (3 if kind else 1))), device="cuda")
    Y = torch.as_tensor(rng.standard_normal((1, 3 if kind else 1)), device="cuda")
    o = bie2d.default_opts(tol=1e-12, precision=bie2d.BIE_MIXED, mixed_strategy=bie2d.BIE_MIXED_REFINE)
    b = bie2d.Batch()
    alone, info, _ = bie2d.bie_batch_solve(b, [(g, kind, X)], o)
    assert info["refinements"] > 1
    both = bie2d.bie_batch_solve(b, [(g, kind, X), (disc, kind, Y)], o)[0]
    assert torch.equal(both[0], alone[0])
