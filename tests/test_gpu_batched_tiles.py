"""Batched items through every tile path of the batched kernels -- up to 8 and
more sources at one offset, sources at different offsets, items too short for
a vector, outputs on and off the sources' grid, items to be skipped -- for the
table kernel (host descriptors), the queue kernel (device descriptors, eager
and allocation-free; one unit of tiles per workgroup, several units with and
without claims) and the runs kernel (graph replay).  Bit-exact against the CPU
oracle, guard bands around every output."""
import numpy as np
import pytest

import gpu_util as gu
import pins

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
PAD = 32
ES = {"bf16": 2, "f32": 4, "e4m3": 1, "i64": 8}


@pytest.fixture(scope="module")
def xr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2510_20171_amd as xr
    xr.load()
    yield xr
    xr.set_max_workgroups(0)


class Batch:
    """Items (nsrc, count, source offsets, output offset) of random elements."""

    def __init__(self, rng, dtype, specs):
        self.dtype, self.specs = dtype, specs
        pool = pins.random_column_values(rng, dtype, max(n for _, n, _, _ in specs) + 64)
        self.np_srcs, self.srcs, self.raw, self.out = [], [], [], []
        for k, (nsrc, n, offs, doff) in enumerate(specs):
            vals = [np.roll(pool, 7 * p + k)[:n].copy() for p in range(nsrc)]
            self.np_srcs.append(vals)
            dev = []
            for p, v in enumerate(vals):
                buf = np.zeros(offs[p] + n + PAD, v.dtype)
                buf[offs[p]:offs[p] + n] = v
                dev.append(gu.to_dev(buf, dtype)[offs[p]:offs[p] + n])
            self.srcs.append(dev)
            es = ES[dtype]
            raw = torch.empty((doff + n + PAD) * es, dtype=torch.uint8, device="cuda")
            self.raw.append((raw, doff * es, (doff + n) * es))
            self.out.append(raw[doff * es:(doff + n) * es].view(gu.torch_dtype(dtype)))
        self.reset()

    def reset(self):
        for raw, _, _ in self.raw:
            raw.fill_(0xA5)

    def host_items(self):
        return list(zip(self.srcs, self.out))

    def device_items(self, xr, skip=()):
        self.keep = [torch.tensor([s.data_ptr() for s in ss] if k not in skip
                                  else [0] * len(ss), dtype=torch.int64, device="cuda")
                     for k, ss in enumerate(self.srcs)]
        rows = np.zeros(len(self.specs), xr.ITEM_DTYPE)
        for k, (nsrc, n, _, _) in enumerate(self.specs):
            rows[k] = (self.keep[k].data_ptr(), self.out[k].data_ptr(), n, nsrc, 0)
        return torch.from_numpy(rows.view(np.uint8).copy()).to("cuda")

    def expect(self, orc, op):
        self.exp = [orc.allreduce_local(v, self.dtype, op) for v in self.np_srcs]

    def check(self, op, what, skip=()):
        torch.cuda.synchronize()
        for k, (raw, lo, hi) in enumerate(self.raw):
            r = raw.cpu().numpy()
            assert (r[:lo] == 0xA5).all() and (r[hi:] == 0xA5).all(), f"{what} item {k}: guard"
            if k in skip:
                assert (r == 0xA5).all(), f"{what} item {k}: skipped item written"
            else:
                gu.assert_parity(self.out[k], self.exp[k], self.dtype, op,
                                 f"{what} item {k} {self.specs[k][:2]}")


def _specs(rng, dtype, K):
    vec = 16 // ES[dtype]
    tile = 512 * vec
    lengths = [1, vec - 1 or 1, vec, vec + 1, 3 * vec + 1, tile - 1, tile, tile + 1, 2 * tile + 1,
               3 * tile + vec + 1]
    out = []
    for k in range(K):
        nsrc = [1, 2, 3, 5, 8, 9, 16, 17, 33][k % 9]
        n = lengths[(k // 2) % len(lengths)]
        kind = k % 5
        if kind == 0:                       # one offset for all, the output included
            offs, doff = [k % vec] * nsrc, k % vec
        elif kind == 1:                     # the output at another
            offs, doff = [k % vec] * nsrc, (k + 1) % vec
        elif kind == 2:                     # every source at its own
            offs, doff = [int(x) for x in rng.integers(0, vec, nsrc)], int(rng.integers(0, vec))
        else:
            offs, doff = [0] * nsrc, 0
        out.append((nsrc, n, offs, doff))
    return out


@pytest.mark.parametrize("dtype", ["bf16", "f32", "e4m3", "i64"])
@pytest.mark.parametrize("K", [1, 7, 64, 65, 130])
def test_tile_paths(xr, orc, dtype, K):
    rng = np.random.default_rng(1000 + K)
    b = Batch(rng, dtype, _specs(rng, dtype, K))
    op = "avg" if dtype == "f32" else "sum"
    b.expect(orc, op)
    xr.batched_reduce(b.host_items(), op, dtype=dtype)
    b.check(op, "host")
    skip = (2,) if K > 2 else ()
    items = b.device_items(xr, skip)
    for budget in (0, 3, 40):               # 40: several units per workgroup, claims
        prev = xr.set_max_workgroups(budget)
        try:
            for call in (xr.batched_reduce, xr.batched_reduce_noalloc, xr.batched_reduce):
                b.reset()
                call(items, op, dtype=dtype)
                b.check(op, f"{call.__name__} budget {budget}", skip)
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                xr.batched_reduce(items, op, dtype=dtype)
            for _ in range(3):
                b.reset()
                g.replay()
                b.check(op, f"graph budget {budget}", skip)
        finally:
            xr.set_max_workgroups(prev)


def test_queue_units(xr, orc):
    """Many small items: units of several tiles, fewer claims than tiles."""
    rng = np.random.default_rng(3)
    sizes = [int(x) for x in rng.integers(1, 3000, 1500)]
    sizes[700] = 8192 * 40 + 5              # one item of many whole tiles among them
    b = Batch(rng, "bf16", [(2, n, [0, 0], 0) for n in sizes])
    b.expect(orc, "sum")
    items = b.device_items(xr)
    for call in (xr.batched_reduce, xr.batched_reduce, xr.batched_reduce_noalloc,
                 xr.batched_reduce_noalloc):
        b.reset()
        call(items, "sum", dtype="bf16")
        b.check("sum", call.__name__)
