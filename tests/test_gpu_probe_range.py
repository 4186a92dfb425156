"""Density probes at coordinates that no lattice index can hold."""
import numpy as np
import pytest

from paper_2003_01490_amd import workloads as W

from harness import gpu_domain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", [0, 1, 2])
def test_probe_far_outside_a_walled_axis(storage):
    print(f"[case] probes far outside z walls, storage {storage}", flush=True)
    wl = W.dense(1, n=24, count=1, D=6.0)
    g = gpu_domain(wl, storage=storage)
    g.step(2)
    far = [24.0, 30.0, 2147483647.0, 2147483648.5, 3e9, 1e18, 1e300, np.inf, np.nan]
    z = np.array(far + [-v for v in far])
    pts = np.stack([np.full(len(z), 2.5), np.full(len(z), 2.5), z], 1)
    assert np.isnan(g.probe_density(pts)).all()
    # a periodic axis wraps
    x = np.array([2.5, 26.5, -21.5, 2.5 + 24 * 1000, np.inf, np.nan])
    r = g.probe_density(np.stack([x, np.full(6, 2.5), np.full(6, 2.5)], 1))
    assert np.isfinite(r[0]) and (r[:4] == r[0]).all() and np.isnan(r[4:]).all()
    g.close()
