"""Loading a linear layer's weight [N, K] in one launch gives the bits of the
three steps it replaces (transposed copy, marlin_quantize, marlin_pack_weights,
each checked against its oracle elsewhere), whatever the weight's layout; and
pack and unpack take codes at any byte alignment."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth

pytestmark = pytest.mark.gpu

CLIP = tuple(1.0 - 0.05 * i for i in range(10))


@pytest.fixture(scope="module")
def mk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_11743_amd as m
    return m


def three_steps(mk, weight, g, ratios):
    q, s = mk.quantize(weight.t().contiguous(), group=g, ratios=ratios)
    return mk.pack(q, s, group=g)


def same(a, b):
    return torch.equal(a[0], b[0]) and torch.equal(a[1].view(torch.int16), b[1].view(torch.int16))


@pytest.mark.parametrize("ratios", [(1.0,), CLIP, tuple(1.0 - i / 128.0 for i in range(64))])
@pytest.mark.parametrize("K,N,g", [(128, 64, -1), (256, 320, 128), (512, 192, 256), (1408, 576, -1), (768, 64, 384)])
def test_one_launch_equals_three_steps(mk, K, N, g, ratios):
    W = synth.fp16_weights(31, K, N).T.copy()
    W[0] = 0                                  # a zero column, a zero group, a scale that flushes to zero
    W[1, :128] = 0
    W[2] = 1e-8
    W[3] = -65504.0
    W[4, 5], W[5, 7] = np.inf, np.nan         # out of contract, but the same bits as before
    w = torch.from_numpy(W).cuda()
    want = three_steps(mk, w, g, ratios)
    layer = mk.MarlinLinear.from_float(w, group=g, ratios=ratios)
    assert same((layer.w_packed, layer.s_packed), want)


def test_any_layout_of_the_weight(mk):
    K, N = 256, 192
    w = torch.from_numpy(synth.fp16_weights(32, K, N).T.copy()).cuda()
    want = three_steps(mk, w, 128, CLIP)
    shifted = torch.zeros(N * K + 1, dtype=torch.float16, device="cuda")[1:].view(N, K)
    shifted.copy_(w)                          # two bytes off any 16-byte boundary
    wide = torch.zeros(N, 2 * K, dtype=torch.float16, device="cuda")
    wide[:, ::2] = w
    transposed = w.t().contiguous().t()
    negated = torch._neg_view(-w)             # as the imaginary part of a conjugate is
    for v in (shifted, wide[:, ::2], transposed, torch.nn.Parameter(w), negated):
        layer = mk.MarlinLinear.from_float(v)
        assert same((layer.w_packed, layer.s_packed), want)
    with pytest.raises(TypeError):
        mk.MarlinLinear.from_float(w.float())
    for bad, g in ((w[:, :200].contiguous(), 128), (w, 64)):
        with pytest.raises(mk.MarlinError):
            mk.MarlinLinear.from_float(bad, group=g)
    with pytest.raises(mk.MarlinError):
        mk.MarlinLinear.from_float(w, ratios=(1.5,))


@pytest.mark.parametrize("shift", [0, 1, 2, 7])
@pytest.mark.parametrize("K,N", [(128, 64), (384, 320)])
def test_codes_at_any_alignment(mk, shift, K, N):
    q, s = synth.weights(33, K, N, 128)
    buf = torch.full((K * N + 16,), 0xAB, dtype=torch.uint8, device="cuda")
    view = buf[shift:shift + K * N].view(K, N)
    high = torch.from_numpy(q | 0xA0).cuda()  # only the low nibble counts
    view.copy_(high)
    sd = torch.from_numpy(s).cuda()
    wp, sp = mk.pack(view, sd)
    assert same((wp, sp), mk.pack(torch.from_numpy(q).cuda(), sd))
    buf.fill_(0xAB)
    mk.marlin_unpack_weights(wp, sp, K, N, 128, view, torch.empty_like(sd), torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert np.array_equal(view.cpu().numpy(), q)
    assert bool((buf[:shift] == 0xAB).all()) and bool((buf[shift + K * N:] == 0xAB).all())
