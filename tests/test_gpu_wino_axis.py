"""Winograd one axis at a time: every built F(n,k) against float64 at the edges of its tiles, blocks and chunks; values that parts do not hold."""
import pytest
import torch

from conv_workloads import ConvLayer

pytestmark = pytest.mark.gpu

BUILT = [(n, k) for k in (5, 6, 7) for n in range(2, 9) if 7 <= n + k - 1 <= 10]


def plan(m, layer, n, variant):
    return m.ConvPlan.for_layer(layer, options=m.Options(force_kind=m.SCHEME_WINOGRAD, force_tile_n=n, force_variant=variant))


def mnn():
    import paper_2002_12418_amd
    return paper_2002_12418_amd


def inputs(layer, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.rand(layer.n, layer.c_in, layer.h, layer.w, generator=g) * 2 - 1
    w = torch.randn(layer.c_out, layer.c_in, layer.kh, layer.kw, generator=g)
    return x, w, torch.rand(layer.c_out, generator=g)


def conv64(layer, x, w, b):
    return torch.nn.functional.conv2d(x.double(), w.double(), b.double() if b is not None else None, padding=layer.pad)


def error(y, ref):
    return float((y.cpu().double() - ref).abs().max() / ref.abs().max())


@pytest.mark.parametrize("nk", BUILT, ids=lambda t: f"F({t[0]},{t[1]})")
@pytest.mark.parametrize("shape", [
    (1, 16, 9, 9, 32, 2), (3, 33, 20, 21, 130, 3),        # one chunk; a chunk of one channel, blocks of 64 and 128 output channels not full
    (2, 5, 7, 8, 9, 0), (1, 20, 40, 7, 65, 3),            # no padding, fewer channels than a chunk; a narrow image
    (4, 64, 24, 28, 64, 1),                               # whole chunks and blocks
])
def test_against_float64(nk, shape):
    m = mnn()
    (n, k), (N, C, H, W, K, pad) = nk, shape
    layer = ConvLayer("axis", N, C, H, W, K, k, k, 1, pad)
    x, w, b = inputs(layer, 7 * n + k)
    ref = conv64(layer, x, w, b)
    xd, wd, bd = x.cuda(), w.cuda(), b.cuda()
    with plan(m, layer, n, m.WINO_UNFUSED) as p:
        unfused = error(p.run(xd, wd, bd), ref)
    with plan(m, layer, n, m.WINO_BY_AXIS) as p:
        assert "by axes" in p.describe()
        guard = torch.full((ref.numel() + 256,), 7.0, device="cuda")
        y = guard[128:128 + ref.numel()].view(ref.shape)
        p.run(xd, wd, bd, y)
        torch.cuda.synchronize()
        assert bool((guard[:128] == 7.0).all()) and bool((guard[128 + ref.numel():] == 7.0).all())
        # the same transforms in the same precision: the maximum over a few thousand outputs scatters by less than a factor of two
        assert error(y, ref) <= 2 * unfused + 1e-6
        assert error(y, ref) < 1e-3
        off = torch.full((ref.numel() + 1,), 7.0, device="cuda")[1:].view(ref.shape)      # 4-byte aligned: single stores
        assert torch.equal(p.run(xd, wd, bd, off), y)
        assert error(p.run(xd, wd, None), conv64(layer, x, w, None)) < 1e-3


@pytest.mark.parametrize("nk", [(4, 5), (2, 7), (4, 7)])
def test_values_that_parts_do_not_hold(nk):
    """Tiny images and weights beside ordinary ones, and non-finite ones: as accurate as the separate kernels, and only where they reach."""
    m = mnn()
    n, k = nk
    layer = ConvLayer("tiny", 3, 24, 20, 20, 70, k, k, 1, k // 2)
    x, w, _ = inputs(layer, n)
    x[0] *= 2.0 ** -116
    w[5] *= 2.0 ** -114
    w[6] *= 2.0 ** 60
    ref = conv64(layer, x, w, None)
    err = {}
    for variant in (m.WINO_UNFUSED, m.WINO_BY_AXIS):
        with plan(m, layer, n, variant) as p:
            y = p.run(x.cuda(), w.cuda(), None).cpu().double()
            # per image and channel; what lies below 2^-126 keeps multiples of 2^-149, times what the transforms amplify (below 2^12)
            size = ref.abs().amax(dim=(2, 3), keepdim=True)
            err[variant] = (((y - ref).abs() - 2.0 ** -137).clamp(min=0) / size.clamp(min=2.0 ** -126)).amax(dim=(2, 3))
            bad = x.clone()
            bad[1, 23, 10, 10], bad[1, 0, 0, 0] = float("nan"), float("inf")
            out = p.run(bad.cuda(), w.cuda(), None).cpu().double()
            reach = torch.isnan(conv64(layer, bad, w, None)[1])
            assert torch.isnan(out[1])[reach].all() and torch.equal(out[2], y[2])
    assert bool((err[m.WINO_BY_AXIS] <= 4 * err[m.WINO_UNFUSED] + 1e-6).all())


def test_chain_and_saved_choice(tmp_path):
    m = mnn()
    layer = ConvLayer("saved", 2, 32, 24, 24, 64, 5, 5, 1, 2)
    x, w, b = (t.cuda() for t in inputs(layer, 1))
    opt = m.Options(force_kind=m.SCHEME_WINOGRAD, force_tile_n=4, force_variant=m.WINO_BY_AXIS)
    with m.ConvPlan.for_layer(layer, options=opt) as p:
        y = p.run(x, w, b).clone()
    with m.ConvChain([layer, layer.__class__("next", 2, 64, 24, 24, 64, 5, 5, 1, 2)], options=opt) as chain:
        w2 = torch.randn(64, 64, 5, 5, device="cuda")
        chain.set_weights(0, w, b)
        chain.set_weights(1, w2, None)
        eager = chain.run(x).clone()
        assert torch.equal(torch.from_numpy(chain.activation_to_numpy(0)).reshape(y.shape), y.cpu())
        out = torch.empty_like(eager)
        chain.capture(x, out)
        for _ in range(3):
            out.zero_()
            chain.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, eager)
            x.mul_(1.0)
