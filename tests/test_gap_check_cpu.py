"""The resolution warning's closest pair (body boxes first, then nodes) against all pairs in numpy:
separated, touching, nested and interleaved bodies, and long node lists (the grid)."""
import re

import numpy as np
import pytest

from paper_1507_05925_amd import bie2d
from paper_1507_05925_amd import workloads as wl


def brute(c):
    npb = np.asarray(c.nodes_per_body)
    body = np.repeat(np.arange(len(npb)), npb)
    w = 2 * np.pi / npb[body] * np.hypot(c.dx, c.dy)
    best = (3.0, -1, -1)
    for b in range(len(npb)):
        i, k = np.where(body == b)[0], np.where(body != b)[0]
        r = np.hypot(c.x[i][:, None] - c.x[k], c.y[i][:, None] - c.y[k]) / w[k]
        if r.min() < best[0]:
            at = np.unravel_index(r.argmin(), r.shape)
            best = (r.min(), b, body[k[at[1]]])
    return best


def ellipses(rng, n, spread, nodes):
    s, cen = [], rng.uniform(-spread, spread, size=(n, 2))
    for i in range(n):
        s.append(wl.ellipse_samples(int(rng.integers(*nodes)), cen[i, 0], cen[i, 1],
                                    *rng.uniform(0.3, 0.6, size=2), rng.uniform(0, 6)))
    return wl.assemble(s, cen, np.ones(n))


def cases():
    rng = np.random.default_rng(4)
    out = [ellipses(rng, int(rng.integers(2, 14)), float(rng.uniform(1.0, 8.0)), (100, 200))
           for _ in range(40)]
    ring = wl.assemble([wl.disc_samples(3000, 0, 0, 2.0), wl.disc_samples(2000, 0.1, 0, 1.897)],
                       [[0, 0], [0.1, 0]], [2.0, 1.897])  # nested, long lists (curves resolved, so that the warning is about the gap)
    return out + [ring, wl.two_discs(0.5, 64)]


@pytest.mark.parametrize("n", range(42))
def test_closest_pair(n):
    c = cases()[n]
    code, msg = bie2d.bie_curves_check(c)
    ratio, b, k = brute(c)
    if b < 0:
        assert code == bie2d.BIE_OK, msg
        return
    assert code == bie2d.BIE_ERESOLVE
    found = re.search(r"bodies (\d+) and (\d+) are closer than .* \(([\d.]+) spacings", msg)
    assert found and abs(float(found[3]) - ratio) < 1e-6 * max(1.0, ratio), (msg, ratio)
    if n != 41:  # (symmetric bodies: either order)
        assert {int(found[1]), int(found[2])} == {b, k}
