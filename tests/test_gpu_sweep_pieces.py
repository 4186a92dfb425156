"""Rows cut into an odd number of pieces of whole cache lines, and the runs of
tiles that large lattices are handed to the XCDs in."""
import numpy as np
import pytest

from paper_2003_01490_amd import workloads as W

from harness import check, gpu_domain, oracle_domain, random_pdf, rel_field_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [136, 192, 256, 264, 272, 288, 384, 512, 544, 656, 768, 1024, 2048, 3072])
def test_row_pieces(nx):
    """3 steps of a random field: FP64 against the oracle; the reduced storages
    to one rounding of the largest deviation (~0.02) per value and step, and a
    few more in the moments.  The batch's tiles give the bits of the single sweep."""
    import torch

    from paper_2003_01490_amd import lbmdem as L

    print(f"[case] {nx}x5x4 fluid, three storages, alone and in a batch", flush=True)
    p = W.base_params(nx=nx, ny=5, nz=4, walls=(0, 0, 1), wall_u_hi=(0.03, 0.01, 0.0), nu=0.03, max_spheres=1)
    e = np.zeros((0, 3))
    wl, f = W.Workload("fluid", p, e, np.zeros(0), np.zeros(0), e, e, 3), random_pdf((nx, 5, 4), nx)
    o = oracle_domain(wl)
    o.set_pdf(f)
    o.step(3)
    ref = o.field("pdf")
    stream = torch.cuda.Stream()
    for storage, bound in ((0, 1e-13), (1, 20 * 2.0 ** -24), (2, 20 * 2.0 ** -11)):
        a, m = [gpu_domain(wl, storage=storage, stream=stream) for _ in range(2)]
        b = L.Batch(stream, pool_bytes=1 << 40)
        b.admit(m)
        for g in (a, m):
            g.set_pdf(f)
        a.step(3)
        b.step(3)
        check(f"pdf storage {storage}", rel_field_err(a.field("pdf"), ref), bound, f"nx {nx}")
        assert np.array_equal(a.field("pdf"), m.field("pdf"))
        b.close()


@pytest.mark.parametrize("n,storage", [((544, 250, 200), 1), ((128, 512, 421), 1), ((544, 500, 200), 2),
                                       ((272, 260, 200), 0)])
def test_large_lattice(n, storage):
    """More than 2 GB a buffer (the batch's sweep takes the tiles in order): a
    forced shear flow, whose every cell changes in every step."""
    import torch

    from paper_2003_01490_amd import lbmdem as L

    print(f"[case] {n} storage {storage}, single against batched sweep", flush=True)
    p = W.base_params(nx=n[0], ny=n[1], nz=n[2], walls=(0, 0, 1), wall_u_hi=(0.03, 0.01, 0.0), nu=0.03, max_spheres=1,
                      body_force=(2e-3, -1e-3, 3e-3))
    e = np.zeros((0, 3))
    wl = W.Workload("fluid", p, e, np.zeros(0), np.zeros(0), e, e, 3)
    stream = torch.cuda.Stream()
    out = []
    for batched in (False, True):
        g = gpu_domain(wl, storage=storage, stream=stream)
        b = L.Batch(stream, pool_bytes=1 << 40)
        if batched:
            b.admit(g)
        for _ in range(3):
            (b if batched else g).step(1)
        vel = torch.empty(3 * g.N, dtype=torch.float64, device="cuda:0")
        g.field_into("vel", vel)
        out.append(vel)
        b.close()
        g.close()
    assert torch.equal(out[0], out[1])
    assert bool((out[0].view(3, n[2], -1)[0, 1:-1] != 0).all())
