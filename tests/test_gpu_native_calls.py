"""The binding's compiled marshalling against its Python code: tensor
subclasses are left to the Python code, plain tensors are not; both must run
the same call and raise the same errors."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


class Sub(torch.Tensor):
    pass


@pytest.fixture(scope="module")
def xr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2510_20171_amd as xr
    xr.load()
    return xr


def _calls(xr, wrap, stream):
    g = torch.Generator(device="cuda").manual_seed(5)
    n = 5003
    src = [wrap(torch.randn(n, device="cuda", generator=g).bfloat16()) for _ in range(5)]
    big = [wrap(torch.randn(4 * n, device="cuda", generator=g).bfloat16()) for _ in range(4)]
    new = lambda t=torch.bfloat16: torch.full((n,), 7, dtype=t, device="cuda")  # noqa: E731
    outs = []

    def out(t=torch.bfloat16):
        outs.append(new(t))
        return wrap(outs[-1])

    torch.cuda.synchronize()
    kw = {"stream": stream}
    xr.allreduce_local(src, out(), "avg", **kw)
    xr.allreduce_local(tuple(src), out(), "max", dtype="bf16", **kw)
    xr.reduce_scatter_local(big, 2, out(), **kw)
    acc = out(torch.float32)
    xr.reduce_copy_step(src[0], acc, None, init=True, **kw)
    xr.reduce_copy_step(src[1], acc, out(), final=True, **kw)
    xr.acc_cast(acc, out(), **kw)
    xr.batched_reduce([(src[:2], out()), (src[2:], out())], "min", dtype="bf16", **kw)
    ready = torch.ones(5, dtype=torch.int32, pin_memory=True)
    status = torch.zeros(1, dtype=torch.int32, pin_memory=True)
    xr.ring_reduce(src, out(), ready=ready, epoch=1, status=status, **kw)
    xr.allreduce_sim(src[:3], [out(), out(), out()], schedule="ring1", **kw)
    torch.cuda.synchronize()
    assert int(status[0]) == 0
    return outs


@pytest.mark.parametrize("which", ["current", "object", "handle"])
def test_same_results(xr, which):
    s = torch.cuda.Stream()
    stream = {"current": None, "object": s, "handle": s.cuda_stream}[which]
    with torch.cuda.stream(s):
        fast = _calls(xr, lambda t: t, stream)
        slow = _calls(xr, lambda t: t.as_subclass(Sub), stream)
    for k, (a, b) in enumerate(zip(fast, slow)):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), k


def test_plain_tensors_are_taken(xr):
    nat = xr.native()
    a = [torch.ones(64, device="cuda") for _ in range(3)]
    out = torch.empty(64, device="cuda")
    assert nat.allreduce(a, out, "sum", None, None) == xr.SUCCESS
    torch.cuda.synchronize()
    assert (out == 3).all()
    for srcs in ([a[0], a[1][:63]], [a[0], torch.ones(128, device="cuda")[::2]],
                 [a[0], torch.ones(64)], [a[0], a[1].as_subclass(Sub)], [], iter(a)):
        assert nat.allreduce(srcs, out, "sum", None, None) is None
    assert nat.allreduce(a, out, "nope", None, None) is None
    assert nat.allreduce(a, out, "sum", "bf16", None) is None


def test_same_errors(xr):
    a = torch.ones(64, device="cuda")
    out = torch.empty(64, device="cuda")
    for bad in ([a, a[:63]], [a, torch.ones(64)], [a, torch.ones(128, device="cuda")[::2]],
                [a, a.bfloat16()], [a] * 65):
        with pytest.raises(xr.XredError) as e:
            xr.allreduce_local(bad, out)
        assert e.value.status == xr.INVALID_ARGUMENT
    with pytest.raises(xr.XredError) as e:      # refused by the library itself
        xr.allreduce_local([torch.ones(128, device="cuda")[:64]], out[1:].new_empty(64), "avg",
                           dtype="i32")
    assert e.value.status == xr.UNSUPPORTED
    with pytest.raises(KeyError):
        xr.allreduce_local([a], out, "nope")


def test_same_results_without_the_module(xr, monkeypatch):
    """Every call gives the same bytes through the Python code alone."""
    fast = _calls(xr, lambda t: t, None)
    assert not isinstance(xr._lib.native(), xr._lib._Declines)
    monkeypatch.setattr(xr._lib, "_native", xr._lib._Declines())
    slow = _calls(xr, lambda t: t, None)
    for k, (a, b) in enumerate(zip(fast, slow)):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), k
