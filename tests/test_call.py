"""The native part of the binding: the same results as the path through ctypes, on the caller's stream, and every
call that is not plain is left to that path, which raises what it always raised."""
import pytest

torch = pytest.importorskip("torch")
rsr = pytest.importorskip("paper_2603_27462_amd")
from paper_2603_27462_amd import binding  # noqa: E402


def _product():
    rsr.load_library()
    assert binding._product is not None, "not built"
    return binding._product


def test_leaves_what_is_not_plain():
    product = _product()
    x = torch.zeros(4)
    for args in ((1, 4, 4, x, 1.0), (1, 4, 4, None, 1.0), (1, 4, 4, [0.0] * 4, 1.0), ("h", 4, 4, x, 1.0),
                 (1, 4, 4, x, "one"), (1, 4, 4, x), (1, 4, 4, torch.nn.Parameter(x), 1.0), ()):
        assert product(*args) is None


def test_not_used_with_another_torch(monkeypatch):
    """Compiled against one torch's tensor classes: under another the path through ctypes is taken."""
    product = _product()
    monkeypatch.setattr(binding, "_product", product)
    monkeypatch.setattr(binding._build, "torch_tag", lambda: "another torch", raising=False)
    with pytest.warns(UserWarning, match="another torch"):
        binding._load_call(rsr.load_library())
    assert binding._product is None


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_same_as_through_ctypes(dtype):
    rows, cols = 300, 517
    M = torch.randint(-1, 2, (rows, cols), dtype=torch.int8, device="cuda:0")
    h = rsr.rsr_preprocess(M, 4, rsr.RSR_TERNARY_FUSED)
    x = torch.randn((7, cols + 3), device="cuda:0").to(dtype)
    for v in (x[0, :cols], x[:1, :cols], x[:, :cols], x[::2, 3:]):
        out = torch.empty((*v.shape[:-1], rows), device="cuda:0")
        rsr.rsr_matvec_ex(h, v, scale=0.5, out=out)
        got = _product()(h.ptr, h.rows, h.cols, v, 0.5)
        assert got.shape == out.shape and got.dtype == torch.float32 and torch.equal(got, out)
        assert torch.equal(rsr.rsr_matvec_ex(h, v, scale=0.5), out)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        v = torch.zeros(cols, device="cuda:0", dtype=dtype)
        for _ in range(200):
            v += 1                                  # the product sees all of it only on the same stream
        got = rsr.rsr_matvec_ex(h, v)
    side.synchronize()
    assert torch.equal(got, 200.0 * M.sum(dim=1, dtype=torch.float32))


@pytest.mark.gpu
def test_refusals_stay():
    M = torch.randint(-1, 2, (40, 64), dtype=torch.int8, device="cuda:0")
    h = rsr.rsr_preprocess(M, 4, rsr.RSR_TERNARY_FUSED)
    x = torch.ones((64, 64), device="cuda:0")
    for v in (x[0].cpu(), x[0, :63], x[0].half(), x[:, 0], x.t(), x[None], x[0, 0]):
        with pytest.raises(TypeError):
            rsr.rsr_matvec_ex(h, v)
    with pytest.raises(rsr.RsrError):
        rsr.rsr_matvec_ex(h, x[:0])
    with pytest.raises(RuntimeError):               # no storage to take a pointer of
        torch.vmap(lambda v: rsr.rsr_matvec_ex(h, v))(x)
    rsr.rsr_destroy(h)
    with pytest.raises(rsr.RsrError):
        rsr.rsr_matvec_ex(h, x[0])


@pytest.mark.gpu
def test_errors_of_a_dispatch_mode():
    """The result is allocated under the caller's dispatch modes, and what those raise reaches the caller."""
    from torch.utils._python_dispatch import TorchDispatchMode

    class Refuses(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            raise LookupError("no tensors here")

    M = torch.randint(-1, 2, (40, 64), dtype=torch.int8, device="cuda:0")
    h = rsr.rsr_preprocess(M, 4, rsr.RSR_TERNARY_FUSED)
    x = torch.ones(64, device="cuda:0")
    with Refuses(), pytest.raises(LookupError, match="no tensors here"):
        rsr.rsr_matvec_ex(h, x)
    assert torch.equal(rsr.rsr_matvec_ex(h, x), M.sum(dim=1, dtype=torch.float32))
