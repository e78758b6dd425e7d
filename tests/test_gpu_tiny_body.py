"""GPU: geometries with one body many orders of magnitude smaller than the rest (at the origin, where
float64 coordinates resolve it): applies by the direct float64 pair sweeps (one launch, split, double
layer) against the sums in numpy, which take one reciprocal per pair, relative to each body's largest
value; 1e-11 allows for some hundreds of roundings in sums of a few thousand terms. And a batched
mobility solve against a single one. (FMM coordinates are relative to the tree's centre, where such a
body is one point.)"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


def curves(radius, bodies):
    s = [wl.disc_samples(48, 0.0, 0.0, radius)]
    k = int(np.ceil(np.sqrt(bodies)))
    s += [wl.ellipse_samples(64, 3.0 + 2 * (i % k), 2 * (i // k), 0.6, 0.4, i) for i in range(bodies)]
    return wl.assemble(s, np.zeros((bodies + 1, 2)), np.ones(bodies + 1))


def dense(c, mu, kind, source_normal):
    n = np.repeat(c.nodes_per_body, c.nodes_per_body)
    sp = np.hypot(c.dx, c.dy)
    w, nx, ny = 2 * np.pi / n * sp, c.dy / sp, -c.dx / sp
    kappa = (c.dx / sp * (c.ddy / sp) - c.dy / sp * (c.ddx / sp)) / sp
    dx, dy = c.x[:, None] - c.x, c.y[:, None] - c.y
    np.fill_diagonal(dx, 1.0)
    r = np.hypot(dx, dy)
    ux, uy = dx / r, dy / r
    np.fill_diagonal(ux, 0.0)
    np.fill_diagonal(uy, 0.0)
    rn = (ux * nx + uy * ny if source_normal else ux * nx[:, None] + uy * ny[:, None]) / r
    sign = 1.0 if source_normal else -1.0
    if kind == 0:
        return 0.5 * mu - w * mu * kappa / (4 * np.pi) + sign / (2 * np.pi) * (rn @ (w * mu))
    m = mu.reshape(-1, 2)
    s = w[:, None] * m
    rs = ux * s[:, 0] + uy * s[:, 1]
    tx, ty = -ny, nx
    d = -kappa / (2 * np.pi) * (tx * s[:, 0] + ty * s[:, 1])
    out = 0.5 * m + np.stack([d * tx, d * ty], 1)
    return (out + sign / np.pi * np.stack([(rn * rs * ux).sum(1), (rn * rs * uy).sum(1)], 1)).reshape(-1)


def check(c, out, ref, comps, tol):
    bp = c.body_ptr * comps
    for b in (0, 1, c.nbodies - 1):
        o, r = out[bp[b]:bp[b + 1]], ref[bp[b]:bp[b + 1]]
        assert np.abs(o - r).max() < tol * np.abs(r).max(), b


@pytest.mark.parametrize("radius", [1e-20, 1e-42, 1e-60])
@pytest.mark.parametrize("bodies", [5, 70])
@pytest.mark.parametrize("kind", [0, 1])
def test_applies(radius, bodies, kind):
    c = curves(radius, bodies)
    g = bie2d.Geometry.from_curves(c)
    mu = np.random.default_rng(bodies).standard_normal((2, c.M * (1 + kind)))
    t = torch.as_tensor(mu, device="cuda")
    ref = [dense(c, mu[r], kind, False) for r in range(2)]
    apply = bie2d.bie_stokes_apply if kind else bie2d.bie_laplace_apply
    for n in (1, 2):
        out = apply(g, t[:n].contiguous(), bie2d.BIE_FP64, bie2d.BIE_DIRECT, with_L=False).cpu().numpy()
        for r in range(n):
            check(c, out[r], ref[r], 1 + kind, 1e-11)
        dl = bie2d.bie_stokes_dl_apply if kind else bie2d.bie_laplace_dl_apply
        out = dl(g, t[:n].contiguous(), False).cpu().numpy()
        for r in range(n):
            check(c, out[r], dense(c, mu[r], kind, True), 1 + kind, 1e-11)


def test_batch_gives_the_single_solves_answer():
    c = curves(1e-42, 5)
    g = bie2d.Geometry.from_curves(c)
    X = torch.as_tensor(np.random.default_rng(1).standard_normal((3, 18)), device="cuda")
    X[:, :3] = 0.0  # (the tiny body moves with the flow)
    o = bie2d.default_opts(tol=1e-11, restart=100)
    one = bie2d.bie_mobility_solve(g, X, o)[0][:, 3:]
    many = bie2d.bie_batch_solve(bie2d.Batch(), [(g, 1, X)], o)[0][0][:, 3:]
    assert float((one - many).abs().max() / one.abs().max()) < 1e-9
