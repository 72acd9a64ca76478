"""Sliding window on staged patches: every configuration against float64, at the edges of its rectangles, patches and chunks of channels."""
import pytest
import torch

from conv_workloads import ConvLayer

pytestmark = pytest.mark.gpu

LAYERS = [
    ConvLayer("one_chunk", 1, 16, 9, 9, 32, 3, 3, 1, 1),
    ConvLayer("short_last_chunk", 2, 41, 13, 17, 70, 3, 3, 1, 1),            # 2 chunks of 16 channels and 9 channels
    ConvLayer("second_group_empty", 1, 24, 30, 33, 93, 3, 3, 1, 2, 2),       # dilated
    ConvLayer("stride2_rows", 3, 64, 56, 56, 128, 3, 3, 2, 1),               # whole rows, 16-byte stores
    ConvLayer("stride2_odd", 2, 20, 37, 29, 65, 5, 5, 2, 2),
    ConvLayer("stride3", 2, 8, 40, 41, 33, 3, 3, 3, 0),                      # taps no wider than the stride, all of them needed
    ConvLayer("stride5_of_2", 2, 9, 30, 31, 17, 2, 2, 5, 0),                 # a stride beyond the kernel
    ConvLayer("images_share_a_rectangle", 9, 33, 5, 5, 40, 3, 3, 1, 1),      # 25 pixels: 2 or 5 images per workgroup, the last short
    ConvLayer("wide", 1, 16, 3, 300, 16, 3, 3, 1, 1),
    ConvLayer("tall", 1, 16, 300, 2, 16, 3, 2, 1, 1),
    ConvLayer("one_column", 1, 12, 70, 1, 8, 3, 1, 1, (1, 0)),
    ConvLayer("row_kernel", 2, 32, 17, 17, 48, 1, 7, 1, (0, 3)),
    ConvLayer("two_taps", 2, 17, 12, 12, 130, 2, 1, 1, 0),
    ConvLayer("mostly_padding", 1, 16, 4, 4, 64, 5, 5, 1, 4),
    ConvLayer("wide_dilation", 1, 16, 30, 30, 16, 3, 3, 1, 6, 6),            # patches of 64 columns too large: the most columns that fit
]


@pytest.fixture
def mnn():
    import paper_2002_12418_amd as m
    yield m
    m.cache_clear()


def patch_variants(m):
    """(number, name): what planned layers take beyond the configurations of products."""
    out, v = [], len(m.gemm_variants())
    while m.gemm_variant_name(v):
        out.append((v, m.gemm_variant_name(v)))
        v += 1
    assert len(out) == 5 and all(n.startswith("x6_patch_") for _, n in out)
    return out


def planned(m, layer, variant, path):
    """A plan whose remembered configuration is `variant`."""
    opt = m.Options(force_kind=m.SCHEME_DIRECT)
    m.cache_clear()
    m.ConvPlan.for_layer(layer, options=opt).close()
    m.cache_save(str(path))
    lines = [l.split("|")[0] + f"| {variant} 1" if l.startswith("G ") and l.split("|")[0].split()[-1] == "0" else l      # fp32 entries
             for l in path.read_text().splitlines()]
    path.write_text("\n".join(lines) + "\n")
    m.cache_clear()
    m.cache_load(str(path))
    return m.ConvPlan.for_layer(layer, options=opt)


def inputs(layer, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.rand(layer.n, layer.c_in, layer.h, layer.w, generator=g) * 2 - 1
    w = torch.randn(layer.c_out, layer.c_in, layer.kh, layer.kw, generator=g)
    return x, w, torch.rand(layer.c_out, generator=g)


def conv64(layer, x, w, b):
    return torch.nn.functional.conv2d(x.double(), w.double(), b.double() if b is not None else None, stride=layer.stride, padding=layer.pad,
                                      dilation=layer.dil)


@pytest.mark.parametrize("layer", LAYERS, ids=lambda l: l.name)
def test_every_configuration_against_float64(mnn, layer, tmp_path):
    x, w, b = inputs(layer, layer.c_in)
    ref = conv64(layer, x, w, b)
    xd, wd, bd = x.cuda(), w.cuda(), b.cuda()
    for v, name in patch_variants(mnn):
        with planned(mnn, layer, v, tmp_path / "cache") as plan:
            assert name in plan.describe()
            shape = tuple(ref.shape)
            guard = torch.full((ref.numel() + 256,), 7.0, device="cuda")     # writes outside the output would show
            y = guard[128:128 + ref.numel()].view(shape)
            plan.run(xd, wd, bd, y)
            torch.cuda.synchronize()
            assert bool((guard[:128] == 7.0).all()) and bool((guard[128 + ref.numel():] == 7.0).all())
            # fp32 sums: R terms of magnitude below 5, each rounded once at 2^-24 of the running sum
            assert float((y.cpu().double() - ref).abs().max() / ref.abs().max()) < 2e-6, name
            off = torch.full((ref.numel() + 1,), 7.0, device="cuda")[1:].view(shape)      # 4-byte aligned: single stores
            plan.run(xd, wd, bd, off)
            assert torch.equal(off, y), name
            plain = plan.run(xd, wd, None)
            assert float((plain.cpu().double() - conv64(layer, x, w, None)).abs().max() / ref.abs().max()) < 2e-6, name


def test_values_that_parts_do_not_hold(mnn, tmp_path):
    """Inputs and weights below 2^-109, infinities, NaN and values that round to an infinite bf16: what fp32 gives, and only where they reach."""
    layer = ConvLayer("edge", 2, 24, 20, 20, 40, 3, 3, 2, 1)
    x, w, b = inputs(layer, 5)
    x[0] *= 2.0 ** -115                                   # image 0: tiny times weights up to 2^60
    w[3] *= 2.0 ** 60
    w[5] *= 2.0 ** -118                                   # a tiny output channel
    b[:] = 0
    x[1, 20, 19, 19] = 3.4e38                             # image 1, last pixel: rounds to an infinite bf16
    w[7] *= 2.0 ** -20
    ref = conv64(layer, x, w, b)
    scale = conv64(layer, x.abs(), w.abs(), b)            # sum of magnitudes
    xd, wd, bd = x.cuda(), w.cuda(), b.cuda()
    for v, name in patch_variants(mnn):
        with planned(mnn, layer, v, tmp_path / "cache") as plan:
            y = plan.run(xd, wd, bd).cpu().double()
            finite = scale < 3.0e38
            # 216 products and sums at 2^-24 each; results below 2^-126 keep multiples of 2^-149
            assert bool(((y - ref).abs()[finite] <= 216 * 2.0 ** -24 * scale[finite] + 216 * 2.0 ** -149).all()), name
            bad = xd.clone()
            bad[0, 23, 7, 7], bad[0, 0, 0, 0] = float("nan"), float("inf")
            out = plan.run(bad, wd, bd).cpu()
            assert torch.equal(out[1], y[1].float()), name
            want = torch.nn.functional.conv2d(bad.cpu().double(), w.double(), b.double(), stride=2, padding=1)
            assert torch.equal(torch.isnan(out[0]), torch.isnan(want[0])) and torch.equal(torch.isinf(out[0]), torch.isinf(want[0])), name


def test_first_pass_and_new_weights(mnn, tmp_path):
    """Weights rewritten behind one pointer are prepared again; a chain takes the same kernels."""
    layer = ConvLayer("again", 4, 32, 28, 28, 64, 3, 3, 2, 1)
    x, w, b = (t.cuda() for t in inputs(layer, 9))
    v, name = patch_variants(mnn)[0]
    with planned(mnn, layer, v, tmp_path / "cache") as plan:
        first = plan.run(x, w, b).clone()
        w2 = (w * -2).contiguous()
        plan.set_weights(w2)
        again = plan.run(x, w2, torch.zeros_like(b)).clone()
        assert torch.equal(again, plan.run(x, w2, torch.zeros_like(b)))
        ref = conv64(layer, x.cpu(), w2.cpu(), None)
        assert float((again.cpu().double() - ref).abs().max() / ref.abs().max()) < 2e-6
    with mnn.ConvChain([layer], options=mnn.Options(force_kind=mnn.SCHEME_DIRECT)) as chain:
        assert name in chain.describe(0)
        chain.set_weights(0, w, b)
        assert torch.equal(chain.run(x), first)


@pytest.mark.parametrize("layer", [
    ConvLayer("rgb", 2, 3, 40, 40, 64, 7, 7, 2, 3),                          # too few channels for the patch kernels
    ConvLayer("one_tap", 2, 16, 20, 20, 16, 1, 1, 2, 0),
    ConvLayer("wider_dilation", 1, 16, 30, 30, 16, 3, 3, 1, 9, 9),           # no patch fits
    ConvLayer("either", 2, 16, 20, 20, 16, 3, 3, 1, 1),
], ids=lambda l: l.name)
def test_weights_take_the_room_of_their_form(mnn, layer, tmp_path):
    """A plan owns the prepared weights in the form that its kernel reads, and no more."""
    x, w, b = (t.cuda() for t in inputs(layer, 3))
    taps = layer.kh * layer.kw
    plain = layer.c_in * taps * -(-layer.c_out // 4) * 4 * 4
    parts = -(-layer.c_out // 128) * 128 * -(-layer.c_in // 16) * 16 * taps * 6
    plain_tile = (mnn.gemm_variants().index("64x64x16_w2x2"), "64x64x16_w2x2")
    for v, name in [plain_tile] + patch_variants(mnn):
        patch = name.startswith("x6_patch_") and layer.name == "either"
        with planned(mnn, layer, v, tmp_path / "cache") as plan:
            assert ("x6_patch_" in plan.describe()) == patch
            assert plan.workspace_bytes == (parts if patch else plain), name
            y = plan.run(x, w, b)
            ref = conv64(layer, x.cpu(), w.cpu(), b.cpu())
            assert float((y.cpu().double() - ref).abs().max() / ref.abs().max()) < 2e-6, name
