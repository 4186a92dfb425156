"""The three DEM kernels against each other at sphere counts where the automatic
choice is the chain, with the same boundary pass."""
import numpy as np
import pytest

from paper_2003_01490_amd import workloads as W

from harness import gpu_domain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,n,map_kernel", [(65, 48, 1), (156, 96, 0), (156, 96, 3), (256, 72, 1), (257, 72, 1),
                                                (257, 72, 2)])
def test_automatic_choice_equals_the_others(count, n, map_kernel):
    D = 12.0 if n == 96 else 6.0
    wl = W.dense(8, n=n, count=count, D=D, min_gap=0.1, u_rms=0.06, nu=0.02)
    print(f"[case] {count} spheres D={D} in {n}^3, FP32, map kernel {map_kernel}, DEM kernels 0, 1, 2", flush=True)
    gs = [gpu_domain(wl, storage=1, dem_kernel=k, map_kernel=map_kernel) for k in (1, 0, 2)]
    for _ in range(3):
        for g in gs:
            g.step(10)
        ref = gs[0].spheres()
        for g in gs[1:]:
            s = g.spheres()
            assert all(np.array_equal(s[k], ref[k]) for k in s)
    for g in gs:
        g.sync()
    assert any(gs[0].sphere(i)["F_col"].any() for i in range(count)) or n == 96
    for g in gs[1:]:
        assert np.array_equal(g.field("pdf"), gs[0].field("pdf"))
    for g in gs:
        g.close()
