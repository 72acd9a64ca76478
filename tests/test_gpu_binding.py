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


def tensors(seed=0):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(*s, generator=g).cuda() for s in ((2, 12, 9, 10), (20, 12, 3, 3), (20,))]


def close(y, x, w, b):
    ref = torch.nn.functional.conv2d(x.cpu().double(), w.detach().cpu().double(), b.cpu().double() if b is not None else None, padding=1)
    return float((y.cpu().double() - ref).abs().max() / ref.abs().max()) < 2e-6


def test_weights_followed(mnn):
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


def test_errors_worded_by_the_general_path(mnn):
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


def test_call_without_allocation(mnn):
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
