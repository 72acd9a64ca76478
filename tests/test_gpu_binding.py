"""The short way from Python into a planned layer: the same results, errors and weight updates as the general path."""
import pytest
import torch

from conv_workloads import ConvLayer

pytestmark = pytest.mark.gpu
LAYER = ConvLayer("small", 2, 12, 9, 10, 20, 3, 3, 1, 1)


@pytest.fixture
def mnn():
    import paper_2002_12418_amd as m
    yield m
    m.cache_clear()


@pytest.fixture(params=["short", "general"])
def way(request, monkeypatch):
    """The short way, and the general one alone, as where the native module is not built."""
    from paper_2002_12418_amd import binding
    binding._find_current_stream()
    assert binding._fast_call is not None
    if request.param == "general":
        monkeypatch.setattr(binding, "_fast_call", None)
    return request.param


def tensors(seed=0):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(*s, generator=g).cuda() for s in ((2, 12, 9, 10), (20, 12, 3, 3), (20,))]


def close(y, x, w, b):
    ref = torch.nn.functional.conv2d(x.cpu().double(), w.detach().cpu().double(), b.cpu().double() if b is not None else None, padding=1)
    return float((y.cpu().double() - ref).abs().max() / ref.abs().max()) < 2e-6


def test_weights_followed(mnn, way):
    """The weight tensor of the call before, changed in place, replaced by an equal one elsewhere, by a parameter, by a view, set by hand."""
    x, w, b = tensors()
    y = torch.empty(2, 20, 9, 10, device="cuda")
    with mnn.ConvPlan.for_layer(LAYER, options=mnn.Options(force_kind=mnn.SCHEME_DIRECT)) as p:
        for _ in range(3):
            assert p.run(x, w, b, y) is y and close(y, x, w, b)
        w.mul_(2)
        p.run(x, w, b, y)
        assert close(y, x, w, b)
        other = w * 3
        p.run(x, other, None, y)
        assert close(y, x, other, None)
        p.run(x, w, b, y)
        assert close(y, x, w, b)
        third = other * 2
        p.set_weights(third)
        p.run(x, w, b, y)                               # not what was set
        assert close(y, x, w, b)
        with torch.no_grad():
            w.add_(1)
        p.run(x, w, b, y)
        assert close(y, x, w, b)
        par = torch.nn.Parameter(w.clone())
        for _ in range(2):
            p.run(x, par, b, y)
            assert close(y, x, par, b)
        part = torch.cat([w, w * 5])[20:]               # a storage offset
        for _ in range(2):
            p.run(x, part, b, y)
            assert close(y, x, part, b)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            p.run(x, part, None, y)
        s.synchronize()
        assert close(y, x, part, None)
        assert close(p.run(x, part, b), x, part, b) and close(p.run(x, part, b, y, stream=s), x, part, b)


def test_errors_worded_by_the_general_path(mnn, way):
    x, w, b = tensors(1)
    y = torch.empty(2, 20, 9, 10, device="cuda")
    p = mnn.ConvPlan.for_layer(LAYER, options=mnn.Options(force_kind=mnn.SCHEME_DIRECT))
    for _ in range(2):
        p.run(x, w, b, y)
        for args, what in (((x[:1], w, b, y), "input"), ((x.double(), w, b, y), "input"), ((x.transpose(2, 3).contiguous().transpose(2, 3), w, b, y), "input"),
                           ((x.cpu(), w, b, y), "input"), ((x, w[:, :6], b, y), "weight"), ((x, w, b, y.half()), "output"), ((x, w, b[:3], y), "bias"),
                           ((x, w, torch.cat([b, b])[::2], y), "bias")):
            with pytest.raises(ValueError, match=what):
                p.run(*args)
        assert close(p.run(x, w, b, y), x, w, b)
    p.close()
    with pytest.raises(mnn.MnnError):
        p.run(x, w, b, y)


def test_call_without_allocation(mnn, way):
    """Strides and paddings as numbers, pairs and lists; an unknown layer object or a wrong tile is reported as before."""
    x, w, b = tensors(2)
    y = torch.empty(2, 20, 9, 10, device="cuda")
    for pad in (1, (1, 1), [1, 1]):
        layer = ConvLayer("static", 2, 12, 9, 10, 20, 3, 3, 1, pad)
        for tile in (0, 2):
            y.fill_(float("nan"))
            assert mnn.conv_run_static(layer, tile, x, w, b, y) is y and close(y, x, w, b)
    with pytest.raises(mnn.MnnError) as e:
        mnn.conv_run_static(layer, -1, x, w, b, y)
    assert e.value.code == -1
    with pytest.raises(AttributeError):
        mnn.conv_run_static(object(), 2, x, w, b, y)


def test_the_short_way_is_taken(mnn):
    """By the usual call and no other: 0 from the library, or None."""
    from paper_2002_12418_amd import binding
    x, w, b = tensors(3)
    y = torch.empty(2, 20, 9, 10, device="cuda")
    p = mnn.ConvPlan.for_layer(LAYER, options=mnn.Options(force_kind=mnn.SCHEME_DIRECT))
    assert p._fast(x, w, b, y) is None                  # no weight tensor yet
    p.run(x, w, b, y)
    for bias in (b, None):
        y.fill_(float("nan"))
        assert p._fast(x, w, bias, y) == 0 and close(y, x, w, bias)
    y.fill_(7.0)
    for args in ((x, w.clone(), b, y), (x, w.view_as(w), b, y), (x[:1], w, b, y), (x.double(), w, b, y), (x.cpu(), w, b, y), (x, w, b[:3], y), (x, w, b, y.half()),
                 (x.transpose(2, 3).contiguous().transpose(2, 3), w, b, y), (x, w, torch.cat([b, b])[::2], y), (None, w, b, y), (x, w, b, None)):
        assert p._fast(*args) is None
    assert bool((y == 7.0).all())
    w.mul_(2)
    assert p._fast(x, w, b, y) is None                  # other values
    p.run(x, w, b, y)
    assert p._fast(x, w, b, y) == 0 and close(y, x, w, b)
    other = w * 3
    p.set_weights(other)
    assert p._fast(x, w, b, y) is None and p._fast(x, other, b, y) == 0 and close(y, x, other, b)
    p.close()
    assert p._fast(x, other, b, y) is None

    def static(layer, tile, *args):
        return binding._fast_call.run_static(binding._address["mnn_conv_run_static"], layer, tile, *args)

    for tile in (0, 2):
        y.fill_(float("nan"))
        assert static(LAYER, tile, x, w, b, y) == 0 and close(y, x, w, b)
    assert static(ConvLayer("pair", 2, 12, 9, 10, 20, 3, 3, 1, (1, 1)), 2, x, w, None, y) == 0 and close(y, x, w, None)
    assert static(ConvLayer("list", 2, 12, 9, 10, 20, 3, 3, 1, [1, 1]), 2, x, w, b, y) is None
    assert static(LAYER, 2, x.double(), w, b, y) is None and static(object(), 2, x, w, b, y) is None and static(LAYER, -1, x, w, b, y) == -1


def test_a_chain_without_the_short_way(mnn, way):
    x, w, b = tensors(4)
    chain = mnn.ConvChain([LAYER])
    chain.set_weights(0, w, b)
    y = chain.run(x)
    # whatever scheme is chosen: 1e-4 of the largest result bounds the error of every one
    ref = torch.nn.functional.conv2d(x.cpu().double(), w.cpu().double(), b.cpu().double(), padding=1)
    assert float((y.cpu().double() - ref).abs().max() / ref.abs().max()) < 1e-4
    chain.close()
