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


def planned_unfused(m, layer, n, name, path):
    """The separate kernels with the tile configuration `name`: left to timings, the configuration of products this short changes from run to run, and with it
    the rounding."""
    v = m.gemm_variants().index(name)
    product = [str(layer.c_out), None, str(layer.c_in), str((n + layer.kh - 1) ** 2)]          # rows, columns, depth, batch

    def pinned(line):
        key = line.split("|")[0].split()
        ours = key[:1] == ["G"] and key[-1] == "0" and all(a == b for a, b in zip(product, key[3:]) if a is not None)
        return f"{line.split('|')[0]}| {v} 1" if ours else line

    plan(m, layer, n, m.WINO_UNFUSED).close()
    m.cache_save(str(path))
    path.write_text("".join(pinned(l) + "\n" for l in path.read_text().splitlines()))
    m.cache_load(str(path))
    p = plan(m, layer, n, m.WINO_UNFUSED)
    assert f"gemm={name}" in p.describe()
    return p


@pytest.mark.parametrize("nk", BUILT, ids=lambda t: f"F({t[0]},{t[1]})")
@pytest.mark.parametrize("shape", [
    (1, 16, 9, 9, 32, 2), (3, 33, 20, 21, 130, 3),        # one chunk; a chunk of one channel, blocks of 64 and 128 output channels not full
    (2, 5, 7, 8, 9, 0), (1, 20, 40, 7, 65, 3),            # no padding, fewer channels than a chunk; a narrow image
    (4, 64, 24, 28, 64, 1),                               # whole chunks and blocks
])
def test_against_float64(nk, shape, tmp_path):
    m = mnn()
    (n, k), (N, C, H, W, K, pad) = nk, shape
    layer = ConvLayer("axis", N, C, H, W, K, k, k, 1, pad)
    x, w, b = inputs(layer, 7 * n + k)
    ref = conv64(layer, x, w, b)
    xd, wd, bd = x.cuda(), w.cuda(), b.cuda()
    with planned_unfused(m, layer, n, "64x64x16_w2x2", tmp_path / "cache") as p:           # one sum per result, on the fp32 instructions
        unfused = error(p.run(xd, wd, bd), ref)
    with plan(m, layer, n, m.WINO_BY_AXIS) as p:
        assert "by axes" in p.describe()
        guard = torch.full((ref.numel() + 256,), 7.0, device="cuda")
        y = guard[128:128 + ref.numel()].view(ref.shape)
        p.run(xd, wd, bd, y)
        torch.cuda.synchronize()
        assert bool((guard[:128] == 7.0).all()) and bool((guard[128 + ref.numel():] == 7.0).all())
        # the same transforms and sums in the same precision: the maximum over a few thousand outputs scatters by less than a factor of two
        # (tiles that cut the sum in eight pieces round less: their maximum is lower by up to 2.7)
        assert error(y, ref) <= 2 * unfused + 1e-6
        assert error(y, ref) < 1e-3
        off = torch.full((ref.numel() + 1,), 7.0, device="cuda")[1:].view(ref.shape)      # 4-byte aligned: single stores
        assert torch.equal(p.run(xd, wd, bd, off), y)
        assert error(p.run(xd, wd, None), conv64(layer, x, w, None)) < 1e-3


@pytest.mark.parametrize("nk", [(4, 5), (2, 7), (4, 7)])
def test_values_that_parts_do_not_hold(nk, tmp_path):
    """Tiny images and weights beside ordinary ones, and non-finite ones: as accurate as the separate kernels, and only where they reach.

    An image beside a non-finite one keeps its accuracy, not its bits: tiles run on from image to image, and a block of them that meets a value
    which parts do not hold, or a sum that is not finite, is formed on the fp32 instructions as a whole."""
    m = mnn()
    n, k = nk
    layer = ConvLayer("tiny", 3, 24, 20, 20, 70, k, k, 1, k // 2)
    x, w, _ = inputs(layer, n)
    x[0] *= 2.0 ** -116
    w[5] *= 2.0 ** -114
    w[6] *= 2.0 ** 60
    ref = conv64(layer, x, w, None)
    bad = x.clone()
    bad[1, 23, 10, 10], bad[1, 0, 0, 0] = float("nan"), float("inf")
    reach = torch.isnan(conv64(layer, bad, w, None)[1])

    def errors(y):
        # per image and channel; what lies below 2^-126 keeps multiples of 2^-149, times what the transforms amplify (below 2^12)
        size = ref.abs().amax(dim=(2, 3), keepdim=True)
        return (((y - ref).abs() - 2.0 ** -137).clamp(min=0) / size.clamp(min=2.0 ** -126)).amax(dim=(2, 3))

    separate = None
    # 32-column tiles without a tiny channel and across two images: the clean call multiplies them in parts, the other one repeats them
    for name in ("x6_32x32_k8", "x6_64x64_k8", None):
        with planned_unfused(m, layer, n, name, tmp_path / "cache") if name else plan(m, layer, n, m.WINO_BY_AXIS) as p:
            clean = errors(p.run(x.cuda(), w.cuda(), None).cpu().double())
            out = p.run(bad.cuda(), w.cuda(), None).cpu().double()
            beside = errors(out)[[0, 2]]
        # the same sums in parts or in fp32: the maximum over the 400 outputs of an image and channel scatters by less than a factor of four
        separate = clean if separate is None else separate
        assert bool((clean <= 4 * separate + 1e-6).all()), name
        assert torch.isnan(out[1])[reach].all(), name
        assert bool(torch.isfinite(out[[0, 2]]).all()) and bool((beside <= 4 * separate[[0, 2]] + 1e-6).all()), name


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
