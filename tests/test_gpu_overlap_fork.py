"""The DEM beside the sweep through a ramp, a release, wall contact and
collisions, on lattices whose sweep is estimated (its bytes at 5.5 TB/s) at twice
the 80 us from which a step forks: the bits of the sequential step, by direct
launches (which fork with 30 spheres and not with 40) and by a step graph."""
import numpy as np
import pytest

from paper_2003_01490_amd import workloads as W

from harness import gpu_domain

pytestmark = pytest.mark.gpu

N = (160, 160, 256)


def _workload(kind):
    count = {"ramp": 1, "few": 30, "lanes": 40, "chain": 70}[kind]
    rng = np.random.default_rng(11)
    wl = W.dense(6, nxyz=N, count=count, D=10.0, min_gap=2.0, u_rms=0.05, nu=0.02)
    # sphere 0 is ramped to the lower wall, released 3 above it and touches it;
    # the others (if any) stay clear of it, some of them in pairs about to collide
    x, u = wl.x.copy(), wl.u.copy()
    x[0] = (40.0, 40.0, 14.0)
    if count > 1:
        k = np.arange(count - 1)
        x[1:] = np.stack([15.0 + 13.0 * (k % 10), np.full(count - 1, 100.0), 50.0 + 20.0 * (k // 10)], 1)
        x[2::2, 0] -= 2.4  # gap 0.6 to the one before
        u[1::2, 0], u[2::2, 0] = 0.04, -0.04
    p = dict(wl.params, lub_mask=0, tc=8.0, gravity=(0.0, 0.0, -1e-4))
    ramp = dict(u_target=(0.0, 0.0, -0.1), c_acc=10.0, t_st=20.0, release_gap=3.0)
    return W.Workload(kind, p, x, np.full(count, 5.0), np.full(count, 2.0), u, rng.normal(0.0, 1e-3, (count, 3)), 0,
                      ramp=ramp)


@pytest.mark.parametrize("kind", ["ramp", "few", "lanes", "chain"])
def test_forked_step_equals_sequential(kind):
    import torch

    from paper_2003_01490_amd import lbmdem as L

    wl = _workload(kind)
    print(f"[case] {N}, {len(wl.R)} spheres, FP32: overlap, sequential, overlap in a graph", flush=True)
    stream = torch.cuda.Stream()
    gs = [gpu_domain(wl, storage=L.STORE_F32, stream=stream, overlap=o) for o in (1, 0, 1)]
    gs[2].set_graph(True)
    assert gs[0].sweep_bytes() / 5.5e6 > 2 * 80.0
    released = touched = collided = False
    for _ in range(40):
        for g in gs:
            g.step(4)
        ref = gs[1].spheres()
        for g in (gs[0], gs[2]):
            s = g.spheres()
            assert all(np.array_equal(s[k], ref[k]) for k in s)
        s0 = gs[1].sphere(0)
        released = released or s0["mode"] == L.FREE
        touched = touched or s0["F_col"].any()
        collided = collided or any(gs[1].sphere(i)["F_col"].any() for i in range(1, len(wl.R)))
    assert released and touched and (collided or len(wl.R) == 1)
    for g in (gs[0], gs[2]):
        assert np.array_equal(g.field("flags"), gs[1].field("flags"))
        assert np.array_equal(g.field("vel"), gs[1].field("vel"))
    for g in gs:
        g.sync()
        g.close()
