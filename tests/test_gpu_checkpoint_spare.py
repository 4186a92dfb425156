"""A checkpoint is laid out in the spare population buffer: the run it is taken
from, and the one it is restored into, go on as if nothing had been there."""
import numpy as np
import pytest

from paper_2003_01490_amd import workloads as W

from harness import gpu_domain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("map_kernel", [1, 2, 3])
@pytest.mark.parametrize("storage", [0, 1, 2])
def test_checkpoints_leave_the_run_alone(storage, map_kernel):
    print(f"[case] checkpoints after odd and even steps, 37x32x30, storage {storage}, map kernel {map_kernel}", flush=True)
    wl = W.dense(4, nxyz=(37, 32, 30), count=14, D=6.0, min_gap=0.2, u_rms=0.05, nu=0.02)
    ref, run = [gpu_domain(wl, storage=storage, map_kernel=map_kernel) for _ in range(2)]
    other = gpu_domain(wl, storage=storage, map_kernel=map_kernel)
    ref.step(7)
    for k in (1, 1, 2):  # the current buffer alternates
        run.step(k)
        blob = run.save()
        assert run.save() == blob
        other.step(1)  # leaves other populations in both of its buffers
        other.restore(blob)
        assert np.array_equal(other.field("pdf_raw"), run.field("pdf_raw"))
    for g in (run, other):
        g.step(3)
        a, b = ref.spheres(), g.spheres()
        assert all(np.array_equal(a[q], b[q]) for q in a)
        assert np.array_equal(ref.field("pdf"), g.field("pdf"))
        assert np.array_equal(ref.field("flags"), g.field("flags"))
        g.sync()
        g.close()
    ref.close()
