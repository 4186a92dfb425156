"""Scenes that a bin of the neighbour search cannot hold (15 spheres): the
automatic DEM choice against the one-workgroup kernel, which searches all
pairs."""
import numpy as np
import pytest

from paper_2003_01490_amd import workloads as W

from harness import gpu_domain

pytestmark = pytest.mark.gpu


def _grid(n, pitch, low):
    m = int(np.ceil(n ** (1 / 3)))
    k = np.arange(n)
    return np.asarray(low, dtype=float) + pitch * np.stack([k % m, k // m % m, k // (m * m)], 1)


def _scene(name):
    rng = np.random.default_rng(5)
    if name in ("cluster-65", "cluster-100", "cluster-256"):
        # a settled heap in a wide box, where bins are few and wide
        n, count = 160, int(name.split("-")[1])
        x, R, max_radius = _grid(count, 3.6, (5.0, 6.0, 7.0)), np.full(count, 1.5), 1.5
    elif name == "loose-bound":
        # small spheres under a max_radius that leaves one bin per axis
        n, x, R, max_radius = 48, _grid(70, 4.4, (6.0, 6.0, 6.0)), np.full(70, 2.0), 12.0
    else:
        # one large sphere among small ones
        n, max_radius = 64, 8.0
        x = np.concatenate([[[24.2, 24.2, 24.2]], _grid(100, 3.6, (4.0, 4.0, 4.0))])
        R = np.r_[8.0, np.full(100, 1.5)]
    P = len(R)
    u = rng.normal(0.0, 0.04, (P, 3))
    p = W.base_params(nx=n, ny=n, nz=n, nu=0.02, max_spheres=P)
    return W.Workload(name, p, x, R, np.full(P, 2.0), u, rng.normal(0.0, 1e-3, (P, 3)), 6), max_radius


@pytest.mark.parametrize("name", ["cluster-65", "cluster-100", "cluster-256", "loose-bound", "one-large"])
def test_crowded_bins(name):
    """64 < P <= 256 spheres, more than 15 of them in one bin: the automatic
    choice runs and gives the bits of the one-workgroup kernel."""
    wl, max_radius = _scene(name)
    print(f"[case] {name}: {len(wl.R)} spheres in {wl.params['nx']}^3, max_radius {max_radius}, FP32", flush=True)
    a, b = [gpu_domain(wl, storage=1, dem_kernel=k, map_kernel=1, max_radius=max_radius) for k in (0, 1)]
    for g in (a, b):
        g.step(6)
        g.sync()
    sa, sb = a.spheres(), b.spheres()
    assert all(np.array_equal(sa[k], sb[k]) for k in sa)
    assert np.array_equal(a.field("flags"), b.field("flags"))
    assert np.array_equal(a.field("vel"), b.field("vel"))
    lub = [np.abs(b.sphere(i)["F_lub"]).max() > 0 for i in range(len(wl.R))]
    assert sum(lub) > 20, "no crowd"
    a.close()
    b.close()
