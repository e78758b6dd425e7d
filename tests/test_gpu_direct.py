"""GPU: the float64 direct apply (one launch for small geometries, split sweep and finishing launch
for larger ones) against the oracle, at the edges of its tiles: bodies of 3 nodes, node counts
around 16, 64, 128 and 256, geometries with 256 and 257 small tiles, every right-hand side
grouping, with and without the completion, and lengths scaled far from 1."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import dirichlet as di  # noqa: E402
from oracle import nystrom as ny  # noqa: E402
from paper_1507_05925_amd import bie2d  # noqa: E402
from paper_1507_05925_amd import workloads as wl  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs the GPU")]

NODES = {"three": [3], "sixteen": [16, 15, 17], "stage": [255, 257, 127, 129],
         "small_most": [256] * 16, "split_least": [256] * 16 + [5], "ragged": [513, 64, 67, 300, 1999]}


@pytest.mark.parametrize("name,scale", [(k, 1.0) for k in NODES] +
                         [("stage", 2.0 ** -60), ("stage", 2.0 ** 100)])
def test_direct_apply_edges(name, scale):
    rng = np.random.default_rng(len(name))
    c = wl.mixed_grid(rng, len(NODES[name]), np.array(NODES[name]))
    geo = ny.geometry_of(c)
    K = {0: ny.laplace_K(geo), 1: ny.stokes_K(geo)}
    for a in ("x", "y", "dx", "dy", "ddx", "ddy"):
        setattr(c, a, getattr(c, a) * scale)
    g = bie2d.Geometry.from_curves(c)
    for kind, rhs in ((0, (1, 2, 3, 7, 8, 13)), (1, (1, 2, 3, 4, 5))):
        f = bie2d.bie_laplace_apply if kind == 0 else bie2d.bie_stokes_apply
        for R in rhs:
            mu = rng.standard_normal((R, g.M * (1 + kind)))
            # K does not depend on the unit of length (w / |r|)
            ref = 0.5 * mu + mu @ K[kind].T
            tol = 64 * np.finfo(float).eps * (np.abs(K[kind]) @ np.abs(mu).T).max()
            out = f(g, torch.as_tensor(mu, device="cuda"), with_L=False).cpu().numpy()
            assert np.abs(out - ref).max() <= tol, (kind, R)
    if scale == 1.0:  # the completion
        for kind, A in ((0, ny.laplace_operator(geo)), (1, ny.stokes_operator(geo))):
            f = bie2d.bie_laplace_apply if kind == 0 else bie2d.bie_stokes_apply
            mu = rng.standard_normal((3, g.M * (1 + kind)))
            tol = 64 * np.finfo(float).eps * (np.abs(A) @ np.abs(mu).T).max()
            out = f(g, torch.as_tensor(mu, device="cuda")).cpu().numpy()
            assert np.abs(out - mu @ A.T).max() <= tol, kind


@pytest.mark.parametrize("nodes", [[3], [64, 65], [127, 129, 5], [500, 500], [257, 511, 900]])
def test_double_layer_apply_edges(nodes):
    """The double-layer applies at the edges of their tiles and splits, every grouping of
    densities, against the dense oracle."""
    rng = np.random.default_rng(len(nodes))
    c = wl.mixed_grid(rng, len(nodes), np.array(nodes))
    geo = ny.geometry_of(c)
    g = bie2d.Geometry.from_curves(c)
    for kind, rhs in ((0, (1, 2, 3, 6, 8, 11)), (1, (1, 2, 3, 4, 7))):
        A = di.capacitance_operator(geo) if kind == 0 else di.resistance_operator(geo)
        f = bie2d.bie_laplace_dl_apply if kind == 0 else bie2d.bie_stokes_dl_apply
        for R in rhs:
            mu = rng.standard_normal((R, g.M * (1 + kind)))
            tol = 64 * np.finfo(float).eps * (np.abs(A) @ np.abs(mu).T).max()
            out = f(g, torch.as_tensor(mu, device="cuda")).cpu().numpy()
            assert np.abs(out - mu @ A.T).max() <= tol, (kind, R)
