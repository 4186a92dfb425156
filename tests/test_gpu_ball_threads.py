"""The per-sphere kernels of the ball pass at the sphere counts where their
block sizes change: flags and owners equal to the slab pass's, spheres and
populations to FP64 rounding over a short run (sums of one sphere's links are
taken in another order)."""
import numpy as np
import pytest

from paper_2003_01490_amd import workloads as W

from harness import check, gpu_domain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,n", [(130, 40), (512, 60), (513, 60), (4096, 120), (4097, 120)])
def test_block_sizes(count, n):
    wl = W.dense(count, n=n, count=count, D=5.0, min_gap=0.1, u_rms=0.1, nu=0.03)
    print(f"[case] ball pass, {count} spheres in {n}^3", flush=True)
    a, b = gpu_domain(wl, map_kernel=2), gpu_domain(wl, map_kernel=1)
    for _ in range(2):
        a.step(3)
        b.step(3)
        (ca, oa), (cb, ob) = a.flags(), b.flags()
        assert np.array_equal(ca, cb)
        assert np.array_equal(oa[ca == 2], ob[ca == 2])
    sa, sb = a.spheres(), b.spheres()
    for k, scale in (("x", 5.0), ("u", 0.1), ("F_fp", None), ("T_fp", None)):
        ref = scale or float(np.abs(sb[k]).max())
        check(k, float(np.abs(sa[k] - sb[k]).max()) / ref, 1e-10, k)
    fluid = ca <= 1
    fa, fb = a.field("pdf"), b.field("pdf")
    check("pdf", float(np.abs(fa - fb)[:, fluid].max()) / float(np.abs(fb).max()), 1e-10)
