"""Device-descriptor batches of one run (up to 64 items) keep no state: the
library allocates nothing for them and binds nothing to their stream, so the
first one may run while another stream is being captured.  Larger batches
take the queue kernel.  Bit-exact against the CPU oracle."""
import os
import subprocess
import sys
from pathlib import Path

import numpy as np
import pytest

import gpu_util as gu
import pins

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
ROOT = Path(__file__).resolve().parents[1]


@pytest.fixture(scope="module")
def xr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2510_20171_amd as xr
    xr.load()
    return xr


def _batch(xr, sizes, nsrc, seed):
    rng = np.random.default_rng(seed)
    host, outs, keep, rows = [], [], [], np.zeros(len(sizes), xr.ITEM_DTYPE)
    for k, n in enumerate(sizes):
        srcs = [pins.random_column_values(rng, "bf16", n) for _ in range(nsrc)]
        dev = [gu.to_dev(s, "bf16") for s in srcs]
        out = torch.zeros(n, dtype=torch.bfloat16, device="cuda")
        pa = torch.tensor([d.data_ptr() for d in dev], dtype=torch.int64, device="cuda")
        rows[k] = (pa.data_ptr(), out.data_ptr(), n, nsrc, 0)
        host.append(srcs)
        outs.append(out)
        keep += dev + [pa]
    return host, outs, keep, torch.from_numpy(rows.view(np.uint8).copy()).to("cuda")


def _check(orc, host, outs, what):
    for k, (srcs, out) in enumerate(zip(host, outs)):
        gu.assert_parity(out, orc.allreduce_local(srcs, "bf16", "sum"), "bf16", "sum",
                         f"{what}: item {k}")


@pytest.mark.parametrize("K", [1, 2, 63, 64])
def test_first_small_batch_during_a_capture(xr, orc, K):
    """After xred_release the library holds nothing; a small batch on one
    stream while another is being captured neither fails nor ends the capture."""
    sizes = [1 + (k * 3371) % 40000 for k in range(K)]
    host, outs, keep, items = _batch(xr, sizes, 3, K)
    chost, couts, ckeep, citems = _batch(xr, [5000, 70001], 2, 100 + K)
    xr.batched_reduce(items, dtype="bf16")      # the kernel is loaded
    torch.cuda.synchronize()
    for o in outs:
        o.zero_()
    xr.release()
    # named, since torch hands out a pool's streams in turn: two in a row differ
    capture, work = torch.cuda.Stream(), torch.cuda.Stream()
    assert capture.cuda_stream != work.cuda_stream
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=capture):
        xr.batched_reduce(citems, dtype="bf16")
        xr.batched_reduce(items, dtype="bf16", stream=work)
    torch.cuda.synchronize()
    _check(orc, host, outs, f"K={K} during the capture")
    for r in range(3):
        for o in couts:
            o.zero_()
        torch.cuda.synchronize()
        graph.replay()
        xr.batched_reduce(items, dtype="bf16", stream=work)
        torch.cuda.synchronize()
        _check(orc, chost, couts, f"K={K} replay {r}")
    _check(orc, host, outs, f"K={K} after replays")


CHILD = """
import numpy as np, torch
import paper_2510_20171_amd as xr
src = torch.ones(8, 64, dtype=torch.float32, device="cuda")
out = torch.zeros(80, 64, dtype=torch.float32, device="cuda")
ptrs = torch.tensor([s.data_ptr() for s in src], dtype=torch.int64, device="cuda")
for n in (64, 65):
    rows = np.zeros(n, xr.ITEM_DTYPE)
    for k in range(n):
        rows[k] = (ptrs.data_ptr(), out[k].data_ptr(), 64, 8, 0)
    xr.batched_reduce(torch.from_numpy(rows.view(np.uint8).copy()).to("cuda"), dtype="f32")
    torch.cuda.synchronize()
    assert bool((out[:n] == 8).all())
"""


def test_routes(xr):
    """64 items run on the stateless kernel, 65 on the queue kernel."""
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT,
                       env=dict(os.environ, XRED_TRACE="1"), capture_output=True, text=True,
                       timeout=110)
    assert r.returncode == 0, r.stderr
    launches = [l for l in r.stderr.splitlines() if l.startswith("[xred] launch ")]
    assert len(launches) == 2, launches
    assert "batched_runs_kernel" in launches[0] and "batched_queue_kernel" in launches[1], launches
