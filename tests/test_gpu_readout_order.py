"""Flag and owner read-outs into a device tensor that work on the null stream
has still to write: the read-out comes after it."""
import numpy as np
import pytest

from paper_2003_01490_amd import workloads as W

from harness import gpu_domain

pytestmark = pytest.mark.gpu


def test_map_readout_follows_the_null_stream():
    import torch

    print("[case] flags and owners into tensors with pending null-stream work, 48^3", flush=True)
    wl = W.dense(2, n=48, count=20, D=8.0, min_gap=0.5)
    g = gpu_domain(wl, storage=1, stream=torch.cuda.Stream())
    g.step(2)
    g.sync()
    cells, owner = g.flags()
    for k, ref, dtype in (("flags", cells, torch.uint8), ("owner", owner, torch.int32)):
        out = torch.empty(g.N, dtype=dtype, device="cuda:0")
        torch.cuda.synchronize()
        with torch.cuda.stream(torch.cuda.default_stream()):
            torch.cuda._sleep(20_000_000)  # about 10 ms
            out.fill_(77)
        g.field_into(k, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().reshape(ref.shape), ref), k
    g.close()
