"""A sphere whose 24 contact-history slots are all taken: contacts that end
free their slots and new ones take them in the order of the partner list, in
every DEM kernel."""
import numpy as np
import pytest

from paper_2003_01490_amd import workloads as W

from harness import gpu_domain

pytestmark = pytest.mark.gpu


def _slots_case(far):
    """A sphere of R = 8 (id 0) with 25 of R = 1.5 around it (ids 1 to 25) and
    `far` more out of reach; everything keeps its place."""
    c, k = np.array([20.3, 19.8, 20.1]), np.arange(25) + 0.5
    th, ph = np.arccos(1 - 2 * k / 25), np.pi * (1 + 5 ** 0.5) * k
    dirs = np.stack([np.cos(ph) * np.sin(th), np.sin(ph) * np.sin(th), np.cos(th)], 1)
    q = np.arange(far)
    rest = np.stack([4.0 + 7.0 * (q % 8), 4.0 + 11.0 * (q // 8), np.full(far, 52.0)], 1)
    x = np.concatenate([c[None], c + dirs * 10.0, rest])
    # sliding partners, so that the springs grow
    t = np.cross(dirs, [0.3, -0.5, 0.8])
    u = np.concatenate([np.zeros((1, 3)), 0.02 * t, np.zeros((far, 3))])
    P = 26 + far
    p = W.base_params(nx=64, ny=64, nz=64, nu=0.05, tc=8.0, max_spheres=P, lub_mask=0, n_sub=1)
    wl = W.Workload("slots", p, x, np.array([8.0] + [1.5] * (P - 1)), np.full(P, 3.0), u, np.zeros((P, 3)), 8)
    return wl, c, dirs


# end, start: partners whose contacts end and start in the same sub-cycle, in
# one round of eight partners or in two.  In list order a contact that ends
# first makes room; one that starts first finds no slot.
@pytest.mark.parametrize("end,start,fits", [(3, 5, True), (1, 8, True), (3, 20, True), (5, 3, False), (20, 3, False)])
def test_full_history(end, start, fits):
    from paper_2003_01490_amd import lbmdem as L

    for far, kernels in ((0, (0, 2)), (40, (1, 0, 2))):
        wl, c, dirs = _slots_case(far)
        res = []
        for k in kernels:
            print(f"[case] 24 of 25 partners in contact, {end} ends as {start} starts, {len(wl.R)} spheres, "
                  f"DEM kernel {k}", flush=True)
            g = gpu_domain(wl, storage=1, dem_kernel=k, map_kernel=1)
            for i in range(len(wl.R)):
                g.set_mode(i, L.FIXED)
            gap = np.full(25, -0.05)
            gap[start - 1] = 0.5
            g.update_spheres(np.arange(1, 26), x=c + dirs * (9.5 + gap)[:, None], u=wl.u[1:26])
            g.step(3)
            g.sync()
            assert np.abs(g.sphere(end)["F_col"]).max() > 0 and not g.sphere(start)["F_col"].any()
            gap[end - 1], gap[start - 1] = 0.5, -0.05
            g.update_spheres(np.arange(1, 26), x=c + dirs * (9.5 + gap)[:, None])
            if fits:
                g.step(3)
                g.sync()
                assert np.abs(g.sphere(start)["F_col"]).max() > 0
                res.append(np.array([g.sphere(i)[q] for i in range(26) for q in ("F_tot", "T_tot", "F_col", "T_col")]))
            else:
                g.step(1)
                with pytest.raises(L.LbmdemError) as e:
                    g.sync()
                assert e.value.code == L.ECAPACITY
            g.close()
        assert all(np.array_equal(r, res[0]) for r in res), "the kernels differ"
