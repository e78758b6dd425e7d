"""GPU: more requests in flight than one launch of range copies takes (64 ranges, two per request),
of uneven lengths, against the oracle, with the options and the limit of the serving loop's
oracle test. (Bits of a crowd on one geometry are not compared with those of a request alone: the
server merges such requests into one item, and some mobility answers differ by a unit in the
last place.)"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import nystrom as ny  # noqa: E402
from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


def test_many_requests_match_oracle():
    rng = np.random.default_rng(3)
    curves = [wl.mixed_grid(rng, n, np.full(n, 48 + 16 * n)) for n in (1, 2, 5)]
    geoms = [bie2d.Geometry.from_curves(c) for c in curves]
    geos = [ny.geometry_of(c) for c in curves]
    reqs = []
    for i in range(75):
        k, kind = i % 3, (i // 3) % 2
        width = geoms[k].N * (3 if kind else 1)
        reqs.append((k, kind, rng.standard_normal((1 + i % 2, width))))
    srv = bie2d.Server(bie2d.default_opts(tol=1e-12, restart=30))
    tickets = [srv.submit(geoms[k], kind, q) for k, kind, q in reqs]
    got = [srv.wait(t, timeout=100) for t in tickets]
    srv.close()
    assert max(info["inflight"] for _, info in got) > 32
    for (k, kind, q), (out, info) in zip(reqs, got):
        ref = (ny.mobility_solve(geos[k], q)["VW"] if kind else ny.elastance_solve(geos[k], q)["phi"])
        ref = np.asarray(ref).reshape(out.shape)
        assert info["status"] == 0 and info["rel_residual"] <= 1e-12, info
        assert float(np.abs(out - ref).max() / np.abs(ref).max()) < 1e-10, (k, kind)
