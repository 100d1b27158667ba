"""The layer's direct call: the same bits as the operator, and whoever can see
the operator's call still sees it (modes, tracing, transforms, gradients,
profilers); the size arithmetic of ops.gemm equals the library's."""
import pytest

torch = pytest.importorskip("torch")

import paper_2408_11743_amd as mk
import synth
from paper_2408_11743_amd import ops


@pytest.mark.parametrize("sparse", [False, True])
def test_packed_bytes_equal_the_library(sparse):
    weight_bytes = mk.marlin_packed_sparse_weight_bytes if sparse else mk.marlin_packed_weight_bytes
    for K in (0, 64, 100, 128, 384, 4096, 1 << 20, (1 << 20) + 128):
        for N in (0, 32, 64, 192, 4096, 8192, 1 << 20, (1 << 20) + 64):
            for g in (-1, 0, -2, 64, 128, 200, 256, 384, 4096, K):
                wb, sb = ops._packed_bytes(K, N, g, sparse)
                want = (weight_bytes(K, N), mk.marlin_packed_scale_bytes(K, N, g))
                assert (wb, sb) == (want if all(want) else (0, 0)), (K, N, g)


@pytest.fixture
def layer():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    K, N = 512, 192
    q, s = synth.weights(41, K, N, 128)
    wp, sp = mk.pack(torch.from_numpy(q).cuda(), torch.from_numpy(s).cuda())
    return mk.MarlinLinear(wp, sp, K, N, 128)


def operator(layer, x):
    return torch.ops.marlin_mi355x.gemm(x.reshape(-1, 512), layer.w_packed, layer.s_packed, 512, 192, 128,
                                        False).reshape(*x.shape[:-1], 192)


@pytest.mark.gpu
def test_direct_call_equals_the_operator(layer):
    for shape in ((1, 512), (2, 3, 512), (1, 1, 5, 512), (0, 512), (512,)):
        x = torch.randn(*shape, device="cuda").half()
        y = layer(x)
        assert y.shape == (*shape[:-1], 192) and torch.equal(y, operator(layer, x))
    x = torch.randn(4, 1024, device="cuda").half()[:, ::2]  # not contiguous
    assert torch.equal(layer(x), operator(layer, x))
    x = torch.randn(6, 2, 512, device="cuda").half().transpose(0, 1)
    assert torch.equal(layer(x), operator(layer, x))
    with pytest.raises(TypeError):
        layer(torch.zeros(2, 512, device="cuda"))


@pytest.mark.gpu
def test_the_operator_is_seen(layer):
    from torch.utils._python_dispatch import TorchDispatchMode
    from torch.overrides import TorchFunctionMode
    x = torch.randn(2, 512, device="cuda").half()
    want = layer(x)
    seen = []

    class Dispatch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            seen.append(str(func))
            return func(*args, **(kwargs or {}))

    class Function(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(str(func))
            return func(*args, **(kwargs or {}))

    for mode in (Dispatch, Function):
        seen.clear()
        with mode():
            assert torch.equal(layer(x), want)
        assert any("marlin_mi355x" in f for f in seen), mode
    from torch.fx.experimental.proxy_tensor import make_fx
    assert "marlin_mi355x.gemm" in make_fx(layer)(x).code
    with torch.profiler.profile() as prof:
        layer(x)
    assert any("marlin_mi355x" in e.key for e in prof.key_averages())
    # no autograd formula: refused in backward, as the operator refuses it
    y = layer(x.clone().requires_grad_())
    assert y.requires_grad
    with pytest.raises(RuntimeError):
        y.float().sum().backward()
    with torch.no_grad():
        assert torch.equal(layer(x.clone().requires_grad_()), want)


@pytest.mark.gpu
def test_the_buffers_are_looked_at_too(layer):
    x = torch.randn(2, 512, device="cuda").half()
    want = layer(x)
    # scales that want a gradient: refused in backward, as the operator refuses it
    layer.s_packed.requires_grad_()
    y = layer(x)
    assert y.requires_grad and torch.equal(y, want)
    with pytest.raises(RuntimeError):
        y.float().sum().backward()
    with torch.no_grad():
        assert not layer(x).requires_grad
    layer.s_packed.requires_grad_(False)

    # a buffer that is a tensor subclass sees the operator
    seen = []

    class Watched(torch.Tensor):
        @classmethod
        def __torch_function__(cls, func, types, args=(), kwargs=None):
            seen.append(str(func))
            return super().__torch_function__(func, types, args, kwargs or {})

    for name in ("w_packed", "s_packed"):
        seen.clear()
        plain = getattr(layer, name)
        setattr(layer, name, plain.as_subclass(Watched))
        assert torch.equal(layer(x).as_subclass(torch.Tensor), want)
        assert any("marlin_mi355x" in f for f in seen), name
        setattr(layer, name, plain)


@pytest.mark.gpu
def test_a_lazily_negated_view_is_read_as_its_values(layer):
    x = torch.randn(3, 512, device="cuda").half()
    neg = torch._neg_view(x)  # as the imaginary part of a conjugate is
    assert neg.is_neg() and torch.equal(layer(neg), layer(-x))
    layer.s_packed = layer.s_packed.neg()
    want = layer(x)
    layer.s_packed = torch._neg_view(layer.s_packed.neg())
    assert layer.s_packed.is_neg() and torch.equal(layer(x), want)


@pytest.mark.gpu
def test_default_workspace_is_made_once_per_stream(layer):
    x = torch.randn(300, 512, device="cuda").half()
    y = layer(x)
    count = len(ops._default_ws)
    assert torch.equal(layer(x), y) and len(ops._default_ws) == count
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        z = layer(x)
    st.synchronize()
    assert torch.equal(z, y) and len(ops._default_ws) == count + 1
