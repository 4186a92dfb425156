"""A large sphere whose box more spheres' shells meet than the mapping's gathered
set holds (48): its cells are evaluated from the mapping bins."""
import numpy as np
import pytest

from paper_2003_01490_amd import workloads as W

from harness import check_all, fp64_bounds, gpu_domain, oracle_domain, sphere_errs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("few,map_kernel", [(40, 2), (60, 2), (60, 3)])
def test_crowd_around_a_large_sphere(few, map_kernel):
    R, r, c = 10.0, 1.5, np.array([24.3, 23.8, 24.1])
    k = np.arange(few) + 0.5
    th, ph = np.arccos(1 - 2 * k / few), np.pi * (1 + 5 ** 0.5) * k
    dirs = np.stack([np.cos(ph) * np.sin(th), np.sin(ph) * np.sin(th), np.cos(th)], 1)
    x = np.concatenate([c[None], c + dirs * (R + r + 2.2)])
    u = np.concatenate([[[0.05, -0.03, 0.04]], 0.03 * np.cross(dirs, [0.3, -0.5, 0.8])])
    P = few + 1
    # shells (r + 2) that meet the box of the mapped ball and its neighbour cells
    lo, hi = np.floor(c - R) - 1.5, np.floor(c + R) + 2.5
    away = np.linalg.norm(np.maximum(np.maximum(lo - x[1:], x[1:] - hi), 0.0), axis=1)
    near = 1 + int((away <= r + 2.0).sum())
    assert (near > 48) == (few == 60), f"{near} spheres in reach"
    p = W.base_params(nx=48, ny=48, nz=48, nu=0.05, max_spheres=P)
    wl = W.Workload("crowd", p, x, np.array([R] + [r] * few), np.full(P, 3.0), u, np.zeros((P, 3)), 6)
    print(f"[case] one sphere R=10 with {few} of R=1.5 around it, FP64, map kernel {map_kernel}", flush=True)
    o, g = oracle_domain(wl), gpu_domain(wl, map_kernel=map_kernel)
    for _ in range(3):
        o.step(2)
        g.step(2)
        co, oo = o.flags()
        cg, og = g.flags()
        assert np.array_equal(cg, co)
        assert np.array_equal(og[co == 2], oo[co == 2])
    g.sync()
    F = max(float(np.abs(o.sphere(i)["F_fp"]).max()) for i in range(P))
    # FP64 rounding of sums of up to 10,000 links of size 2 w_q is ~1e-12 of the
    # largest force of the run; six steps leave an order of magnitude
    for i in range(P):
        check_all(sphere_errs(g.sphere(i), o.sphere(i), 2 * wl.R[i], {"u": 0.05, "F": F}),
                  fp64_bounds(**{q: 1e-11 for q in ("x", "u", "w", "F_fp", "F_raw", "F_tot", "F_lub", "F_col", "T_fp",
                                                    "T_raw")}), f"sphere {i}")
    g.close()
