"""Step-wise calls split by accumulator vectors: every type at the edges of a
tile (512 vectors) and of a vector, the chunk, the accumulator and the output
each at element offsets of their own, with guard bands around what is written.
Bit-exact against the CPU oracle."""
import numpy as np
import pytest

import gpu_util as gu
import pins

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ACC = {"f64": "f64", "i64": "u64", "u64": "u64", "f32": "f32", "bf16": "f32", "f16": "f32",
       "e4m3": "f32", "e5m2": "f32"}   # the others: u32
DTYPES = ("f32", "bf16", "f16", "e4m3", "e5m2", "f64", "i8", "u8", "i32", "i64")
PAD = 32


@pytest.fixture(scope="module")
def xr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2510_20171_amd as xr
    xr.load()
    return xr


def _at(values, dtype, offset):
    """values on the device, `offset` elements past an aligned address."""
    buf = np.zeros(offset + values.size + PAD, values.dtype)
    buf[offset:offset + values.size] = values
    return gu.to_dev(buf, dtype)[offset:offset + values.size]


class Guarded:
    """n elements at an element offset, a known byte all around them."""

    def __init__(self, n, dtype, offset):
        es = np.dtype(gu.NP_BITS[dtype]).itemsize
        self.raw = torch.full(((offset + n + PAD) * es,), 0xA5, dtype=torch.uint8, device="cuda")
        self.lo, self.hi = offset * es, (offset + n) * es
        self.t = self.raw[self.lo:self.hi].view(gu.torch_dtype(dtype))

    def check(self, what):
        r = self.raw.cpu().numpy()
        assert (r[:self.lo] == 0xA5).all() and (r[self.hi:] == 0xA5).all(), f"{what}: guard written"


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("offsets", [(0, 0, 0), (1, 0, 0), (0, 1, 3), (3, 2, 1), (5, 3, 0)])
def test_step_parts(xr, orc, dtype, offsets):
    rng = np.random.default_rng(71)
    o_in, o_acc, o_out = offsets
    accd = ACC.get(dtype, "u32")
    pv = 2 if accd in ("f64", "u64") else 4     # values per accumulator vector
    tile = 512 * pv
    for n in (1, pv - 1, pv, pv + 1, 64 * pv - 1, tile - 1, tile, tile + 1, 3 * tile + 2 * pv + 1):
        for op in ("sum", "max"):
            what = f"{dtype} {op} n={n} offsets={offsets}"
            chunks = [pins.random_column_values(rng, dtype, n) for _ in range(3)]
            dev = [_at(c, dtype, o_in) for c in chunks]
            acc, out, cast, one = (Guarded(n, accd, o_acc), Guarded(n, dtype, o_out),
                                   Guarded(n, dtype, o_out), Guarded(n, dtype, o_out))
            xr.reduce_copy_step(dev[0], acc.t, None, op, init=True, dtype=dtype)
            xr.reduce_copy_step(dev[1], acc.t, None, op, dtype=dtype)
            xr.reduce_copy_step(dev[2], acc.t, out.t, op, final=True, dtype=dtype)
            xr.acc_cast(acc.t, cast.t, dtype=dtype)
            xr.reduce_copy_step(dev[0], None, one.t, op, init=True, final=True, dtype=dtype)
            torch.cuda.synchronize()
            for g in (acc, out, cast, one):
                g.check(what)
            oacc = orc.reduce_copy_step(chunks[0], None, dtype, op, init=True)
            oacc = orc.reduce_copy_step(chunks[1], oacc, dtype, op)
            gu.assert_parity(acc.t, oacc, accd, op, what + " acc")
            gu.assert_parity(cast.t, orc.acc_cast(oacc, dtype), dtype, op, what + " cast")
            gu.assert_parity(out.t, orc.reduce_copy_step(chunks[2], oacc.copy(), dtype, op,
                                                         final=True), dtype, op, what + " final")
            gu.assert_parity(one.t, orc.reduce_copy_step(chunks[0], None, dtype, op, init=True,
                                                         final=True), dtype, op, what + " init|final")
            # in place: the last step's output over its own chunk
            xr.reduce_copy_step(dev[2], acc.t, dev[2], op, final=True, dtype=dtype)
            torch.cuda.synchronize()
            assert np.array_equal(gu.bits(dev[2], dtype), gu.bits(out.t, dtype)), what + " in place"
