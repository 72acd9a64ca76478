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


def numbers(first, plan_of):
    """(number, name) of NAMES, as plans describe them that were made by plan_of(number): these have no public names."""
    found, v = {}, first
    while len(found) < len(NAMES):
        with plan_of(v) as plan:                          # a number beyond the last is refused, and ends the search with an error
            found.update({n: v for n in NAMES if f"gemm={n}" in plan.describe()})
        v += 1
    return [(found[n], n) for n in NAMES]


@pytest.fixture(scope="module")
def prepared_variants(tmp_path_factory):
    import paper_2002_12418_amd as m
    path = tmp_path_factory.mktemp("numbers") / "cache"
    return numbers(len(m.gemm_variants()), lambda v: planned(m, layer_of((2, 40, 8, 16, 64)), v, path, m.SCHEME_GEMM1X1))


@pytest.fixture(scope="module")
def wino_variants(tmp_path_factory, prepared_variants):
    """By precision; in fp32 they are those of pointwise layers."""
    import paper_2002_12418_amd as m
    path, shape = tmp_path_factory.mktemp("numbers") / "cache", (2, 40, 12, 12, 40, 3, 3, 4)
    return {0: prepared_variants, 2: numbers(1, lambda v: wino_planned(m, wino_layer(shape), 4, v, path, 2))}


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
def test_every_configuration_against_float64(mnn, prepared_variants, shape, tmp_path):
    layer = layer_of(shape)
    x, w, b = inputs(layer, layer.c_in)
    ref = conv64(layer, x, w, b)
    for v, name in prepared_variants:
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
    (ConvLayer("products", 2, 12, 9, 9, 40, 3, 3, 1, 1), "SCHEME_WINOGRAD"),             # a reduction below one step
], ids=lambda v: getattr(v, "name", v))
def test_remembered_where_it_does_not_apply(mnn, prepared_variants, layer, kind, tmp_path):
    x, w, b = inputs(layer, 3)
    ref = conv64(layer, x, w, b)
    for v, name in prepared_variants:
        make = wino_planned(mnn, layer, 4, v, tmp_path / "cache", 0) if kind == "SCHEME_WINOGRAD" else planned(mnn, layer, v, tmp_path / "cache", getattr(mnn, kind))
        with make as plan:
            assert name not in plan.describe()
            y = plan.run(x.cuda(), w.cuda(), b.cuda()).cpu().double()
            # F(4,3): its error is bounded by 1e-4 of the largest result
            assert float((y - ref).abs().max() / ref.abs().max()) < (1e-4 if kind == "SCHEME_WINOGRAD" else 2e-6), name


def test_values_that_parts_do_not_hold(mnn, prepared_variants, tmp_path):
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
    for v, name in prepared_variants:
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


# ---------------------------------------------------------------- Winograd products
# n, c_in, h, w, c_out, kh, kw, tile
PRODUCTS = [
    (1, 16, 6, 6, 16, 3, 3, 4),            # one step, four columns
    (3, 17, 14, 9, 33, 3, 3, 4),
    (2, 130, 10, 11, 129, 3, 3, 2),        # one past the tiles and the chunks
    (5, 24, 60, 62, 70, 3, 3, 4),          # runs of 64 columns, the last one ragged
    (2, 300, 9, 8, 65, 5, 5, 2),
    (2, 40, 17, 17, 100, 1, 7, 2),         # a kernel with one row
]


def wino_layer(shape):
    n, c, h, w, k, kh, kw, tile = shape
    return ConvLayer("x".join(map(str, shape)), n, c, h, w, k, kh, kw, 1, (kh // 2, kw // 2))


def wino_planned(m, layer, tile, variant, path, prec, make=None):
    opt = m.Options(force_kind=m.SCHEME_WINOGRAD, force_tile_n=tile, force_prec=prec, force_variant=m.WINO_UNFUSED)
    m.cache_clear()
    m.ConvPlan.for_layer(layer, options=opt).close()
    m.cache_save(str(path))
    lines = [l.split("|")[0] + f"| {variant} 1" if l.startswith("G ") and l.split("|")[0].split()[-1] == str(prec) else l
             for l in path.read_text().splitlines()]
    path.write_text("\n".join(lines) + "\n")
    m.cache_clear()
    m.cache_load(str(path))
    return (make or (lambda o: m.ConvPlan.for_layer(layer, options=o)))(opt)


@pytest.mark.parametrize("prec", [0, 2], ids=["fp32", "bf16x3"])
@pytest.mark.parametrize("shape", PRODUCTS, ids=str)
def test_winograd_products(mnn, wino_variants, shape, prec, tmp_path):
    """M against the float64 product of the plan's own U and V: R sums, each rounded at 2^-24; two bf16 parts hold an operand to 2^-17, and the
    product of the two second parts is left out."""
    layer = wino_layer(shape)
    x, w, b = inputs(layer, layer.c_in)
    xd, wd, bd = x.cuda(), w.cuda(), b.cuda()
    for v, name in wino_variants[prec]:
        with wino_planned(mnn, layer, shape[-1], v, tmp_path / "cache", prec) as plan:
            assert name in plan.describe()
            info = plan.info
            for weights in (wd, wd * 3):                  # prepared again: another pointer
                y = plan.run(xd, weights, bd)
                torch.cuda.synchronize()
                U, V, M = (torch.from_numpy(plan.buffer_to_numpy(i)) for i in (mnn.BUF_U, mnn.BUF_V, mnn.BUF_M))
                a2, C, K = U.numel() // (layer.c_in * info["ldk"]), layer.c_in, layer.c_out
                U = U.view(a2, C, info["ldk"])[:, :, :K].double()
                if info["tiled"]:
                    V, M = V.view(C, -1, a2, 64).permute(2, 0, 1, 3), M.view(K, -1, a2, 64).permute(2, 0, 1, 3)
                V, M = V.reshape(a2, C, -1).double(), M.reshape(a2, K, -1).double()
                Ut = U.transpose(1, 2).contiguous()
                bound = ((C + 6) * 2.0 ** -24 + (3 * 2.0 ** -17 if prec else 0)) * torch.bmm(Ut.abs(), V.abs())
                assert bool(((M - torch.bmm(Ut, V)).abs() <= bound).all()), name
                assert torch.equal(y, plan.run(xd, weights, bd)), name       # the same bits every run


def test_winograd_products_of_values_that_parts_do_not_hold(mnn, prepared_variants, tmp_path):
    layer = wino_layer((2, 40, 12, 12, 40, 3, 3, 4))
    x, w, b = inputs(layer, 9)
    x[0] *= 2.0 ** -115
    w[3] *= 2.0 ** 60
    w[5] *= 2.0 ** -118
    bad = x.clone()
    bad[1, 39, 5, 5], bad[1, 0, 0, 0] = float("nan"), float("inf")
    bd = torch.zeros(layer.c_out).cuda()
    runs = []
    for v, name in [(next(i for i, n in enumerate(mnn.gemm_variants()) if n == "128x128x16_w2x2"), "128x128x16")] + prepared_variants:
        with wino_planned(mnn, layer, 4, v, tmp_path / "cache", 0) as plan:
            assert name in plan.describe()
            runs.append((name, plan.run(x.cuda(), w.cuda(), bd).cpu().double(), plan.run(bad.cuda(), w.cuda(), bd).cpu()))
    _, want, want_bad = runs[0]                           # the fp32 instructions
    scale = want.abs().amax(dim=(2, 3), keepdim=True)     # per image and channel; sums of 40 products and a transform that amplifies 2^-24 some 30 times
    for name, y, y_bad in runs[1:]:
        assert bool(((y - want).abs() <= 1e-4 * scale + 2.0 ** -140).all()), name
        assert torch.equal(torch.isfinite(y_bad), torch.isfinite(want_bad)), name
        assert torch.equal(y_bad[0], y[0].float()), name


def test_winograd_products_in_a_chain(mnn, prepared_variants, tmp_path):
    layer = wino_layer((2, 40, 12, 12, 40, 3, 3, 4))
    x, w, b = inputs(layer, 4)
    ref = conv64(layer, x, w, b)
    for v, name in prepared_variants:
        chain = wino_planned(mnn, layer, 4, v, tmp_path / "cache", 0, make=lambda o: mnn.ConvChain([layer], options=o))
        assert name in chain.describe(0)
        chain.set_weights(0, w.cuda(), b.cuda())
        y = chain.run(x.cuda(), torch.empty(layer.out_shape, device="cuda"))
        assert float((y.cpu().double() - ref).abs().max() / ref.abs().max()) < 1e-4, name
        chain.close()
