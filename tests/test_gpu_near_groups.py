"""GPU: the FMM apply's near field over every grouping of right-hand sides, both precisions, leaves
with small and large neighbourhoods, and lengths far from 1. Float64 against the direct apply;
float32 groups against the apply of one right-hand side, which reads the same rounded coordinates
(its distance to the direct apply, set by those coordinates, is test_fmm_mixed_apply_accuracy)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]


def absolute_sums(c, mu, kind):
    """Per right-hand side and unknown: sum over k != i of w_k |mu_k| / (2 pi r) (Stokes: |mu_k| the
    vector's length, over pi r), in float64."""
    w = 2.0 * np.pi / np.repeat(c.nodes_per_body, c.nodes_per_body) * np.hypot(c.dx, c.dy)
    w, x, y = (torch.as_tensor(a, device="cuda") for a in (w, c.x, c.y))
    m = mu.abs() if kind == 0 else mu.reshape(len(mu), -1, 2).norm(dim=2)
    inv = 1.0 / torch.hypot(x[:, None] - x, y[:, None] - y)
    inv.fill_diagonal_(0.0)
    s = (m * w) @ inv / (2.0 * np.pi if kind == 0 else np.pi)
    return s if kind == 0 else s.repeat_interleave(2, dim=1)


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
        out = f(g, mu[:n].contiguous(), bie2d.BIE_FP64, bie2d.BIE_FMM, with_L=False)
        assert float((out - ref[:n]).abs().max() / norm) < 1e-12, n
    # A pair term takes at most 8 float32 roundings and joins a sum of 8: 16 eps32/2 of its size in
    # either grouping, and as much again for the expansions: 64 roundings of eps32/2, times the sum
    # of the terms' sizes |strength| / r over all sources.
    size = absolute_sums(c, mu, kind)
    one = torch.cat([f(g, mu[k:k + 1].contiguous(), bie2d.BIE_MIXED, bie2d.BIE_FMM, with_L=False)
                     for k in range(mu.shape[0])])
    for n in (1, 2, 3, 4, 5, 8, 13):
        out = f(g, mu[:n].contiguous(), bie2d.BIE_MIXED, bie2d.BIE_FMM, with_L=False)
        assert bool(((out - one[:n]).abs() <= 64 * 2.0 ** -24 * size[:n]).all()), n


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("factor", [2.0 ** -60, 2.0 ** 40, 2.0 ** 80])
def test_near_field_large_densities(kind, factor):
    """Powers of two pass through the float32 near field: no strength may meet the reciprocal of a
    target's pair with itself (1e30). Bits agree, the apply being linear with only exponents moved."""
    rng = np.random.default_rng(7)
    c = wl.mixed_grid(rng, 9, np.full(9, 96))
    g = bie2d.Geometry.from_curves(c)
    g.set_fmm(32, 48)
    f = bie2d.bie_laplace_apply if kind == 0 else bie2d.bie_stokes_apply
    mu = torch.as_tensor(rng.standard_normal((3, c.M * (1 + kind))), device="cuda")
    for n in (1, 3):
        a = f(g, mu[:n].contiguous(), bie2d.BIE_MIXED, bie2d.BIE_FMM, with_L=False)
        b = f(g, (factor * mu[:n]).contiguous(), bie2d.BIE_MIXED, bie2d.BIE_FMM, with_L=False)
        assert bool(torch.isfinite(b).all()), (n, factor)
        assert torch.equal(factor * a, b), (n, factor)


@pytest.mark.parametrize("kind", [0, 1])
def test_fmm_apply_completion(kind):
    """The evaluation adds the completion from per-body sums: bodies of fewer, exactly and more
    nodes than the 256 threads that sum one, against the direct apply (float64 sums of at most M
    terms and expansions of 48: the 1e-12 of the groups' test)."""
    rng = np.random.default_rng(11)
    c = wl.mixed_grid(rng, 7, np.array([64, 255, 256, 257, 511, 512, 700]))
    g = bie2d.Geometry.from_curves(c)
    g.set_fmm(48, 64)
    f = bie2d.bie_laplace_apply if kind == 0 else bie2d.bie_stokes_apply
    mu = torch.as_tensor(1.0 + rng.standard_normal((9, c.M * (1 + kind))), device="cuda")
    for with_L in (True, False):
        ref = f(g, mu, bie2d.BIE_FP64, bie2d.BIE_DIRECT, with_L=with_L)
        for n in (1, 4, 9):
            out = f(g, mu[:n].contiguous(), bie2d.BIE_FP64, bie2d.BIE_FMM, with_L=with_L)
            assert float((out - ref[:n]).abs().max() / ref.abs().max()) < 1e-12, (n, with_L)
