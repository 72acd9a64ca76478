"""Pointwise layers with prepared weights: every configuration against float64, at the edges of its tiles, steps and wavefronts."""
import pytest
import torch

from conv_workloads import ConvLayer
from test_gpu_conv_patch import conv64, inputs

pytestmark = pytest.mark.gpu

NAMES = ["x6_prepared_128x128x32_w2x2", "x6_prepared_128x64x64_w2x2", "x6_prepared_64x128x32_w2x2", "x6_prepared_64x64x64_w2x2",
         "x6_prepared_32x32_k8", "x6_prepared_64x64_k8"]

# n, c_in, h, w, c_out
LAYERS = [
    (1, 16, 1, 2, 1),                # one step, one pair of columns
    (1, 17, 2, 2, 3),
    (3, 23, 5, 6, 33),               # columns that pairs, but not groups of four, divide
    (2, 40, 8, 16, 64),              # whole tiles
    (2, 129, 8, 17, 130),            # one past the tiles, a reduction one past its chunks
    (3, 255, 7, 7, 127),             # an odd plane
    (1, 1000, 3, 3, 70),
    (2, 72, 16, 16, 300),
]


@pytest.fixture
def mnn():
    import paper_2002_12418_amd as m
    yield m
    m.cache_clear()


def layer_of(shape):
    n, c, h, w, k = shape
    return ConvLayer("x".join(map(str, shape)), n, c, h, w, k, 1, 1, 1, 0)


def prepared_variants(m):
    """(number, name): they follow the last configuration with a public name and the four of the sliding window on short grids."""
    v = len(m.gemm_variants())
    while m.gemm_variant_name(v):
        v += 1
    return [(v + 4 + i, name) for i, name in enumerate(NAMES)]


def planned(m, layer, variant, path, kind):
    """A plan whose remembered configuration is `variant`."""
    opt = m.Options(force_kind=kind)
    m.cache_clear()
    m.ConvPlan.for_layer(layer, options=opt).close()
    m.cache_save(str(path))
    lines = [l.split("|")[0] + f"| {variant} 1" if l.startswith("G ") and l.split("|")[0].split()[-1] == "0" else l      # fp32 entries
             for l in path.read_text().splitlines()]
    path.write_text("\n".join(lines) + "\n")
    m.cache_clear()
    m.cache_load(str(path))
    return m.ConvPlan.for_layer(layer, options=opt)


def check(plan, name, x, w, b, ref):
    xd, wd, bd = x.cuda(), w.cuda(), b.cuda()
    # sums of R terms of magnitude below 5, each rounded once at 2^-24 of the running sum, against the largest result
    for shift in (0, 1, 2):                               # from 16-byte aligned to 4-byte aligned tensors
        xs = torch.empty(xd.numel() + 8, device="cuda")[shift:shift + xd.numel()].view(xd.shape).copy_(xd)
        guard = torch.full((ref.numel() + 256,), 7.0, device="cuda")         # writes outside the output would show
        y = guard[128 + shift:128 + shift + ref.numel()].view(ref.shape)
        y.fill_(float("nan"))
        plan.run(xs, wd, bd, y)
        torch.cuda.synchronize()
        assert bool((guard[:128 + shift] == 7.0).all()) and bool((guard[128 + shift + ref.numel():] == 7.0).all()), name
        assert float((y.cpu().double() - ref).abs().max() / ref.abs().max()) < 2e-6, (name, shift)
    plain = plan.run(xd, wd, None)
    assert float((plain.cpu().double() - (ref - b.double()[None, :, None, None])).abs().max() / ref.abs().max()) < 2e-6, name
    assert torch.equal(plain, plan.run(xd, wd, None)), name                  # the same bits every run


@pytest.mark.parametrize("shape", LAYERS, ids=str)
def test_every_configuration_against_float64(mnn, shape, tmp_path):
    layer = layer_of(shape)
    x, w, b = inputs(layer, layer.c_in)
    ref = conv64(layer, x, w, b)
    for v, name in prepared_variants(mnn):
        with planned(mnn, layer, v, tmp_path / "cache", mnn.SCHEME_GEMM1X1) as plan:
            assert name in plan.describe()
            assert plan.workspace_bytes == (layer.c_out + 127) // 128 * 128 * ((layer.c_in + 15) // 16 * 16) * 6
            check(plan, name, x, w, b, ref)
            plan.set_weights((w * 3).cuda())
            check(plan, name, x, w, b, ref)               # prepared again: another pointer


@pytest.mark.parametrize("layer, kind", [
    (ConvLayer("fifteen_channels", 2, 15, 8, 8, 40, 1, 1, 1, 0), "SCHEME_GEMM1X1"),
    (ConvLayer("sliding", 2, 24, 9, 9, 40, 3, 3, 1, 1), "SCHEME_DIRECT"),
    (ConvLayer("strided", 2, 24, 9, 9, 40, 1, 1, 2, 0), "SCHEME_DIRECT"),
    (ConvLayer("products", 2, 24, 9, 9, 40, 3, 3, 1, 1), "SCHEME_WINOGRAD"),
], ids=lambda v: getattr(v, "name", v))
def test_remembered_where_it_does_not_apply(mnn, layer, kind, tmp_path):
    x, w, b = inputs(layer, 3)
    ref = conv64(layer, x, w, b)
    for v, name in prepared_variants(mnn):
        with planned(mnn, layer, v, tmp_path / "cache", getattr(mnn, kind)) as plan:
            y = plan.run(x.cuda(), w.cuda(), b.cuda()).cpu().double()
            # a transform may be chosen: its error is bounded by the largest tile's, 1e-4 of the largest result
            assert float((y - ref).abs().max() / ref.abs().max()) < (1e-4 if kind == "SCHEME_WINOGRAD" else 2e-6), name


def test_values_that_parts_do_not_hold(mnn, tmp_path):
    """Tiny and non-finite inputs and weights: what fp32 gives, and only where they reach, past the last channel and image included."""
    layer = ConvLayer("edge", 2, 180, 6, 6, 40, 1, 1, 1, 0)
    x, w, b = inputs(layer, 5)
    x[0] *= 2.0 ** -115                                   # image 0: tiny times weights up to 2^60
    w[3] *= 2.0 ** 60
    w[5] *= 2.0 ** -118                                   # a tiny output channel
    b[:] = 0
    x[1, 178, 5, 5] = 3.4e38                              # rounds to an infinite bf16
    w[7] *= 2.0 ** -20
    ref = conv64(layer, x, w, b)
    scale = conv64(layer, x.abs(), w.abs(), b)            # sum of magnitudes
    xd, wd, bd = x.cuda(), w.cuda(), b.cuda()
    for v, name in prepared_variants(mnn):
        with planned(mnn, layer, v, tmp_path / "cache", mnn.SCHEME_GEMM1X1) as plan:
            y = plan.run(xd, wd, bd).cpu().double()
            finite = scale < 3.0e38
            # 180 products and sums at 2^-24 each; results below 2^-126 keep multiples of 2^-149
            assert bool(((y - ref).abs()[finite] <= 180 * 2.0 ** -24 * scale[finite] + 180 * 2.0 ** -149).all()), name
            for img in (0, 1):
                bad = xd.clone()
                bad[img, 179, 3, 3], bad[img, 0, 0, 0] = float("nan"), float("inf")
                out = plan.run(bad, wd, bd).cpu()
                assert torch.equal(out[1 - img], y[1 - img].float()), name
                want = torch.nn.functional.conv2d(bad.cpu().double(), w.double(), b.double()).float()
                assert torch.equal(torch.isnan(out[img]), torch.isnan(want[img])) and torch.equal(torch.isinf(out[img]), torch.isinf(want[img])), name
