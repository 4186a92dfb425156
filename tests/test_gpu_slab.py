"""Boundary pass of few spheres: the row and column chunks of a block, from
spheres of less than a cell to ones of several chunks, moved a little and
across the whole lattice (a mapping update then covers old and new place in one
box), against the oracle's mapping, populations and spheres."""
import numpy as np
import pytest

from paper_2003_01490_amd import workloads as W

from harness import fp64_bounds, check_all, gpu_domain, oracle_domain, random_pdf, sphere_errs
from test_gpu_parity import _compare_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("walls", [(0, 0, 0), (1, 1, 0)])
@pytest.mark.parametrize("R", [0.6, 2.0, 3.5, 6.0, 9.7])
def test_chunks_of_one_slab(R, walls):
    n = (46, 41, 33)
    print(f"[case] slab chunks R {R} walls {walls}", flush=True)
    r2 = 0.5 * R + 0.2
    x = np.array([[12.3, 13.1, 15.7], [12.3 + R + r2 + 0.02, 13.1, 15.7]])
    p = W.base_params(nx=n[0], ny=n[1], nz=n[2], walls=walls, nu=0.04, max_spheres=2)
    wl = W.Workload("slab", p, x, np.array([R, r2]), np.array([2.0, 3.0]),
                    np.array([[0.03, 0.02, 0.01], [-0.02, 0.0, 0.01]]), np.array([[0.0, 0.0, 0.01], [0.0, 0.002, 0.0]]), 0)
    f = random_pdf(n, seed=4, u0=(0.02, 0.0, 0.0))
    o, g = oracle_domain(wl), gpu_domain(wl)
    for dom in (o, g):
        dom.set_pdf(f)
        dom.step(3)
    _compare_fields(g, o)
    # far along x, y and both: boxes of several column and row chunks
    for to in ([33.4, 13.2, 15.9], [33.4, 28.6, 15.9], [12.1, 13.3, 16.2]):
        o.update_sphere(0, x=to)
        g.update_spheres([0], x=np.array([to]))
        _compare_fields(g, o)
        o.step(2)
        g.step(2)
        _compare_fields(g, o)
        F = max(float(np.abs(o.sphere(i)["F_tot"]).max()) for i in range(2))
        for i in range(2):
            check_all(sphere_errs(g.sphere(i), o.sphere(i), 2 * R, {"u": 0.03, "F": F}),
                      fp64_bounds(**{k: 1e-10 for k in ("u", "w", "F_fp", "F_raw", "F_tot", "F_lub", "F_col",
                                                        "T_fp", "T_raw")}), f"sphere {i}")
