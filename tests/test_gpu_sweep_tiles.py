"""Row widths at the edges of the sweep's tile rules (whole rows, pieces, rows
that do and do not start on a 64-byte piece, in the single and the batched
sweep), and the checkpoint's own population format."""
import numpy as np
import pytest

from paper_2003_01490_amd import workloads as W

from harness import check, gpu_domain, oracle_domain, random_pdf, rel_field_err

pytestmark = pytest.mark.gpu

WIDTHS = [4, 15, 16, 31, 64, 65, 127, 129, 160, 255, 257, 320, 429, 480, 511, 513, 640, 1001]


def _fluid(nx, seed):
    n = (nx, 5, 6)
    p = W.base_params(nx=n[0], ny=n[1], nz=n[2], walls=(0, 0, 1), wall_u_hi=(0.03, 0.01, 0.0), nu=0.03, max_spheres=1)
    e = np.zeros((0, 3))
    return W.Workload("fluid", p, e, np.zeros(0), np.zeros(0), e, e, 3), random_pdf(n, seed)


@pytest.mark.parametrize("nx", WIDTHS)
def test_row_widths(nx):
    """3 steps of a random field: FP64 against the oracle; the reduced storages
    against FP64 (one rounding of the largest deviation ~0.02 per value and
    step: 2^-24 and 2^-11 of it, and a few more in the moments)."""
    wl, f = _fluid(nx, nx)
    print(f"[case] {nx}x5x6 fluid, z walls, three storages", flush=True)
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
def test_batched_sweep_equals_single(storage):
    import torch

    from paper_2003_01490_amd import lbmdem as L

    stream = torch.cuda.Stream()
    wls = [_fluid(nx, nx) for nx in WIDTHS]
    print(f"[case] batch of {len(wls)} widths, storage {storage}", flush=True)
    alone, mixed = [], []
    for wl, f in wls:
        for group in (alone, mixed):
            group.append(gpu_domain(wl, storage=storage, stream=stream))
            group[-1].set_pdf(f)
    b = L.Batch(stream, pool_bytes=1 << 40)
    for g in mixed:
        b.admit(g)
    b.step(3)
    for (wl, _), a, m in zip(wls, alone, mixed):
        a.step(3)
        assert np.array_equal(a.field("pdf"), m.field("pdf")), f"nx {wl.params['nx']}"
    b.close()


def test_checkpoint_population_format():
    """The populations of a checkpoint are 19 planes of N stored deviations,
    x fastest, whatever the layout on the device; they restore to the same
    field."""
    wl, f = _fluid(21, 3)
    w = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
    g = gpu_domain(wl, storage=0)
    g.set_pdf(f)
    blob = g.save()
    assert blob.find((f - w[:, None, None, None]).tobytes()) > 0
    h = gpu_domain(wl, storage=0)
    h.restore(blob)
    assert np.array_equal(g.field("pdf_raw"), h.field("pdf_raw"))
    assert h.save() == blob
