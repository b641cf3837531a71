"""Fused reduces whose sources and output sit at different offsets within 16
bytes: vectors read where they lie (whole dwords, or off the dword grid), one
and several groups of 8 sources, lengths at the edges of the lead, of a
vector, of a 128-vector tile and of the runs of 32 tiles per XCD, in place and
out of place, with guard bands around the output.  Bit-exact against the CPU
oracle."""
import numpy as np
import pytest

import gpu_util as gu
import pins

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
PAD = 64


@pytest.fixture(scope="module")
def xr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2510_20171_amd as xr
    xr.load()
    return xr


def _run(xr, orc, dtype, op, P, n, src_off, dst_off, seed, in_place=False):
    rng = np.random.default_rng(seed)
    base = [pins.random_column_values(rng, dtype, n) for _ in range(min(P, 9))]
    srcs = [np.roll(base[p % len(base)], p // len(base)) for p in range(P)]
    dev = []
    for p, v in enumerate(srcs):
        buf = np.full(src_off[p] + n + PAD, v[0], v.dtype)
        buf[src_off[p]:src_off[p] + n] = v
        dev.append(gu.to_dev(buf, dtype)[src_off[p]:src_off[p] + n])
    es = np.dtype(gu.NP_BITS[dtype]).itemsize
    what = f"{dtype} {op} P={P} n={n} src={src_off[:9]} dst={dst_off} in_place={in_place}"
    if in_place:
        out, raw = dev[P // 2], None
    else:
        raw = torch.full(((dst_off + n + PAD) * es,), 0xA5, dtype=torch.uint8, device="cuda")
        out = raw[dst_off * es:(dst_off + n) * es].view(gu.torch_dtype(dtype))
    xr.allreduce_local(dev, out, op, dtype=dtype)
    torch.cuda.synchronize()
    gu.assert_parity(out, orc.allreduce_local(srcs, dtype, op), dtype, op, what)
    if raw is not None:
        r = raw.cpu().numpy()
        assert (r[:dst_off * es] == 0xA5).all() and (r[(dst_off + n) * es:] == 0xA5).all(), what


@pytest.mark.parametrize("dtype", ["bf16", "f16", "e4m3", "i8", "f32", "f64"])
@pytest.mark.parametrize("P", [1, 2, 8, 9, 16, 17, 33, 64])
def test_offsets(xr, orc, dtype, P):
    es = np.dtype(gu.NP_BITS[dtype]).itemsize
    vec = 16 // es
    op = "avg" if dtype in ("f16", "f64") and P > 1 else "sum"
    whole = [4 * ((p * 3 + 1) % 4) // es if es < 4 else (p * 3 + 1) % vec for p in range(P)]
    odd = [(p * 5 + 1) % vec for p in range(P)]
    same = [1] * P                      # one offset for all sources, another for the output
    for src_off, dst_off in ((whole, 0), (odd, 0), (odd, 3 % vec), (same, 0), (same, 2 % vec)):
        for n in (1, 2 * vec - 1, 3 * vec, 5 * vec + 1, 128 * vec + 2, 1000 * vec + 5):
            _run(xr, orc, dtype, op, P, n, src_off, dst_off, 100 * P + n)
        _run(xr, orc, dtype, "max", P, 777 * vec + 3, src_off, dst_off, P, in_place=True)


@pytest.mark.parametrize("extra", [-1, 0, 1, 129])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_offsets_xcd_runs(xr, orc, dtype, extra):
    vec = 16 // np.dtype(gu.NP_BITS[dtype]).itemsize
    for blocks in (1, 3):               # 256 tiles of 128 vectors are one block of runs
        n = (blocks * 256 * 128 + extra) * vec + 3
        _run(xr, orc, dtype, "sum", 3, n, [1, 0, 3], 0, n)
        prev = xr.set_max_workgroups(37)
        try:
            _run(xr, orc, dtype, "sum", 3, n, [1, 0, 3], 2, n)
        finally:
            xr.set_max_workgroups(prev)


@pytest.mark.parametrize("P,nbytes", [(8, (128 << 20) // 9), (8, 9 << 20), (2, 16 << 20),
                                      (9, 1 << 20), (16, (128 << 20) // 17), (1, 17 << 20)])
def test_cached_shapes(xr, orc, P, nbytes):
    """Sizes at the edges of the shapes for calls of at most 128 MiB (one and
    two vectors per thread, more than 8 sources past 1 MiB), on and off the
    sources' grid."""
    for n in (nbytes // 16 * 8, nbytes // 16 * 8 + 9):
        for src, dst in ((0, 0), (1, 0)):
            _run(xr, orc, "bf16", "sum", P, n, [src] * P, dst, n)


@pytest.mark.parametrize("dtype", ["bf16", "e4m3"])
@pytest.mark.parametrize("P", [9, 15, 17, 24, 25])
def test_runtime_counts(xr, orc, dtype, P):
    """Source counts without a kernel of their own, on both sides of 1 MiB a
    source (the next group of 8 in flight, then one group at a time) and, past
    128 MiB in all, in the wave-capped shape; whole and partial last groups."""
    es = np.dtype(gu.NP_BITS[dtype]).itemsize
    for nbytes in (1 << 20, (1 << 20) + 16, (128 << 20) // (P + 1) + 32):
        for src, dst in ((0, 0), (1, 0)):
            _run(xr, orc, dtype, "sum", P, nbytes // es + src, [src] * P, dst, P)


@pytest.mark.parametrize("dtype,op", [("bf16", "sum"), ("e4m3", "sum"), ("i8", "max")])
@pytest.mark.parametrize("P", [7, 8])
def test_two_vector_limit(xr, orc, dtype, op, P):
    """Up to 8 sources at the size up to which a thread takes two vectors:
    108 MiB of sources and output (128 MiB off the sources' grid)."""
    es = np.dtype(gu.NP_BITS[dtype]).itemsize
    for src, limit in ((0, 108 << 20), (1, 128 << 20)):
        for extra in (0, 16):
            n = (limit // (P + 1) + extra) // es
            _run(xr, orc, dtype, op, P, n, [src] * P, 0, n)
