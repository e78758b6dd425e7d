"""The resolution warning's closest pair where one body's box holds many others (a container, a wall
beside discs, nested rings, crowds of overlapping boxes), against all pairs in numpy, at lengths whose
squares leave the range of a float64 too; and the growth of the time that a container takes."""
import re
import time

import numpy as np
import pytest

from paper_1507_05925_amd import bie2d
from paper_1507_05925_amd import workloads as wl


def closest(c):
    npb = np.asarray(c.nodes_per_body)
    body = np.repeat(np.arange(len(npb)), npb)
    w = 2 * np.pi / npb[body] * np.hypot(c.dx, c.dy)
    best = 3.0
    for b in range(len(npb)):
        i, k = np.where(body == b)[0], np.where(body != b)[0]
        r = np.hypot(c.x[i][:, None] - c.x[k], c.y[i][:, None] - c.y[k]) / w[k]
        best = min(best, r.min())
    return best


def discs(n, radius, nodes=16, pitch=1.0):
    k = int(np.ceil(np.sqrt(n)))
    return [wl.disc_samples(nodes, pitch * (i % k), pitch * (i // k), radius) for i in range(n)], k


def pack(samples):
    return wl.assemble(samples, np.zeros((len(samples), 2)), np.ones(len(samples)))


def container(n, nodes, radius=0.2, gap=0.0):
    s, k = discs(n, radius)
    mid = (k - 1) / 2
    return pack(s + [wl.disc_samples(nodes, mid, mid, np.sqrt(2) * mid + radius + gap)])


def crowd(rng, n):
    return pack([wl.ellipse_samples(120, *rng.uniform(-1, 1, 2), *rng.uniform(0.3, 2.0, 2),
                                    rng.uniform(0, 6)) for _ in range(n)])


def geometries():
    rng = np.random.default_rng(8)
    out = [container(40, 400, gap=g) for g in (0.05, 0.3, 1.0)]
    out += [pack(discs(12, 0.3)[0] + [wl.ellipse_samples(600, 2, h, 9, 0.4, 0)]) for h in (-1.0, -0.8, 9.0)]
    out += [pack([wl.disc_samples(300, 0, 0, r) for r in (1.0, 1.05, 1.5, 2.5)])]
    out += [crowd(rng, n) for n in (2, 9, 14, 24)]
    return out


@pytest.mark.parametrize("scale", [1.0, 1e-150, 1e150])
@pytest.mark.parametrize("n", range(11))
def test_closest_pair(n, scale):
    c = geometries()[n]
    want = closest(c)
    for a in ("x", "y", "dx", "dy", "ddx", "ddy"):
        setattr(c, a, getattr(c, a) * scale)
    code, msg = bie2d.bie_curves_check(c)
    if want >= 3.0:
        assert code == bie2d.BIE_OK, msg
        return
    found = re.search(r"\(([\d.]+) spacings", msg)
    assert code == bie2d.BIE_ERESOLVE and found, msg
    assert abs(float(found[1]) - want) < 1e-6, (msg, want)


def test_container_cost_grows_with_its_size():
    """Eight times the bodies and nodes: 8 times the work if it grows as they do, 64 times if as
    their square; the line is half-way (in the logarithm)."""
    def seconds(c):
        best = 1e9
        for _ in range(5):
            t = time.perf_counter()
            assert bie2d.bie_curves_check(c)[0] == bie2d.BIE_OK
            best = min(best, time.perf_counter() - t)
        return best

    assert seconds(container(16000, 16000, gap=1.0)) < 22.6 * seconds(container(2000, 2000, gap=1.0))
