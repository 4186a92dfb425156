"""Fluid with a body force on rows that do and do not start on 64-byte pieces
(the sweep's store kinds), alone and in a batch beside unforced fluid."""
import numpy as np
import pytest

from paper_2003_01490_amd import workloads as W

from harness import check, gpu_domain, oracle_domain, random_pdf, rel_field_err

pytestmark = pytest.mark.gpu

WIDTHS = [15, 16, 32, 65, 129, 256, 257, 320, 513]


def _fluid(nx, force):
    p = W.base_params(nx=nx, ny=5, nz=6, walls=(0, 0, 1), nu=0.03, max_spheres=1, body_force=force)
    e = np.zeros((0, 3))
    return W.Workload("forced", p, e, np.zeros(0), np.zeros(0), e, e, 3), random_pdf((nx, 5, 6), nx)


@pytest.mark.parametrize("nx", WIDTHS)
def test_forced_row_widths(nx):
    """3 steps of a random field: FP64 against the oracle; the reduced storages
    to one rounding of the largest deviation (~0.02) per value and step, and a
    few more in the moments."""
    wl, f = _fluid(nx, (2e-5, -1e-5, 3e-5))
    print(f"[case] {nx}x5x6 fluid with a body force, three storages", flush=True)
    o = oracle_domain(wl)
    o.set_pdf(f)
    o.step(3)
    ref = o.field("pdf")
    for storage, bound in ((0, 1e-13), (1, 20 * 2.0 ** -24), (2, 20 * 2.0 ** -11)):
        g = gpu_domain(wl, storage=storage)
        g.set_pdf(f)
        g.step(3)
        check(f"pdf storage {storage}", rel_field_err(g.field("pdf"), ref), bound, f"nx {nx}")


@pytest.mark.parametrize("storage", [0, 1, 2])
def test_forced_and_unforced_domains_in_a_batch(storage):
    import torch

    from paper_2003_01490_amd import lbmdem as L

    stream = torch.cuda.Stream()
    print(f"[case] batches without and with forced domains, storage {storage}", flush=True)
    for forces in (((0, 0, 0),), ((0, 0, 0), (2e-5, -1e-5, 3e-5)), ((2e-5, -1e-5, 3e-5),)):
        alone, mixed = [], []
        for k, nx in enumerate(WIDTHS):
            wl, f = _fluid(nx, forces[k % len(forces)])
            for group in (alone, mixed):
                group.append(gpu_domain(wl, storage=storage, stream=stream))
                group[-1].set_pdf(f)
        b = L.Batch(stream, pool_bytes=1 << 40)
        for g in mixed:
            b.admit(g)
        b.step(3)
        for nx, a, m in zip(WIDTHS, alone, mixed):
            a.step(3)
            assert np.array_equal(a.field("pdf"), m.field("pdf")), f"nx {nx}"
        b.close()
