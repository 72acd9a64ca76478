"""Sliding window on staged patches for short grids: every configuration against float64, at the edges of its rectangles, rounds and wavefronts."""
import pytest
import torch

from conv_workloads import ConvLayer
from test_gpu_conv_patch import LAYERS, conv64, inputs, planned

pytestmark = pytest.mark.gpu

NAMES = ["f32_patch_16x16_k8", "x6_patch_32x32_k8", "x6_patch_64x32_k8", "x6_patch_32x64_k8"]

MORE = [
    ConvLayer("one_step", 1, 8, 5, 5, 16, 1, 1, 2, 0),                       # fewer steps than wavefronts
    ConvLayer("one_tap", 2, 96, 20, 20, 48, 1, 1, 2, 0),
    ConvLayer("two_rounds", 1, 520, 9, 9, 20, 3, 3, 2, 1),                   # more channels than LDS holds, the last round short
    ConvLayer("many_rounds", 1, 264, 40, 40, 17, 7, 7, 3, 3),
    ConvLayer("sixty_four_taps", 1, 40, 19, 19, 33, 8, 8, 1, 0),
]
BEYOND = [
    ConvLayer("sixty_six_taps", 1, 40, 19, 30, 33, 6, 11, 1, 0),             # not offered: the other kernels
    ConvLayer("large_patch", 1, 16, 60, 60, 16, 3, 3, 1, 12, 12),
    ConvLayer("seven_channels", 1, 7, 12, 12, 16, 3, 3, 1, 1),
]


@pytest.fixture
def mnn():
    import paper_2002_12418_amd as m
    yield m
    m.cache_clear()


@pytest.fixture(scope="module")
def short_variants(tmp_path_factory):
    """(number, name), as plans describe them: these have no public names."""
    import paper_2002_12418_amd as m
    path, found, v = tmp_path_factory.mktemp("numbers") / "cache", {}, len(m.gemm_variants())
    while len(found) < len(NAMES):
        with planned(m, LAYERS[0], v, path) as plan:      # a number beyond the last is refused, and ends the search with an error
            found.update({n: v for n in NAMES if f"gemm={n}" in plan.describe()})
        v += 1
    return [(found[n], n) for n in NAMES]


def check(m, layer, plan, name, x, w, b, ref):
    xd, wd, bd = x.cuda(), w.cuda(), b.cuda()
    guard = torch.full((ref.numel() + 256,), 7.0, device="cuda")             # writes outside the output would show
    y = guard[128:128 + ref.numel()].view(ref.shape)
    y.fill_(float("nan"))
    plan.run(xd, wd, bd, y)
    torch.cuda.synchronize()
    assert bool((guard[:128] == 7.0).all()) and bool((guard[128 + ref.numel():] == 7.0).all()), name
    # fp32 sums: R terms of magnitude below 5, each rounded once at 2^-24 of the running sum
    assert float((y.cpu().double() - ref).abs().max() / ref.abs().max()) < 2e-6, name
    plain = plan.run(xd, wd, None)
    assert float((plain.cpu().double() - conv64(layer, x, w, None)).abs().max() / ref.abs().max()) < 2e-6, name
    assert torch.equal(plain, plan.run(xd, wd, None)), name                  # the same bits every run


@pytest.mark.parametrize("layer", LAYERS + MORE, ids=lambda l: l.name)
def test_every_configuration_against_float64(mnn, short_variants, layer, tmp_path):
    x, w, b = inputs(layer, layer.c_in)
    ref = conv64(layer, x, w, b)
    for v, name in short_variants:
        with planned(mnn, layer, v, tmp_path / "cache") as plan:
            assert name in plan.describe()
            check(mnn, layer, plan, name, x, w, b, ref)


@pytest.mark.parametrize("layer", BEYOND, ids=lambda l: l.name)
def test_remembered_where_it_does_not_apply(mnn, short_variants, layer, tmp_path):
    x, w, b = inputs(layer, 3)
    ref = conv64(layer, x, w, b)
    for v, name in short_variants:
        with planned(mnn, layer, v, tmp_path / "cache") as plan:
            assert name not in plan.describe()
            check(mnn, layer, plan, name, x, w, b, ref)


def test_values_that_parts_do_not_hold(mnn, short_variants, tmp_path):
    """Tiny and non-finite inputs and weights: what fp32 gives, and only where they reach, past the last channel and image included."""
    layer = ConvLayer("edge", 2, 20, 20, 20, 40, 3, 3, 2, 1)
    x, w, b = inputs(layer, 5)
    x[0] *= 2.0 ** -115                                   # image 0: tiny times weights up to 2^60
    w[3] *= 2.0 ** 60
    w[5] *= 2.0 ** -118                                   # a tiny output channel
    b[:] = 0
    x[1, 18, 19, 19] = 3.4e38                             # rounds to an infinite bf16
    w[7] *= 2.0 ** -20
    ref = conv64(layer, x, w, b)
    scale = conv64(layer, x.abs(), w.abs(), b)            # sum of magnitudes
    xd, wd, bd = x.cuda(), w.cuda(), b.cuda()
    for v, name in short_variants:
        with planned(mnn, layer, v, tmp_path / "cache") as plan:
            y = plan.run(xd, wd, bd).cpu().double()
            finite = scale < 3.0e38
            # 180 products and sums at 2^-24 each; results below 2^-126 keep multiples of 2^-149
            assert bool(((y - ref).abs()[finite] <= 180 * 2.0 ** -24 * scale[finite] + 180 * 2.0 ** -149).all()), name
            for img in (0, 1):
                bad = xd.clone()
                bad[img, 19, 7, 7], bad[img, 0, 0, 0] = float("nan"), float("inf")
                out = plan.run(bad, wd, bd).cpu()
                assert torch.equal(out[1 - img], y[1 - img].float()), name
                want = torch.nn.functional.conv2d(bad.cpu().double(), w.double(), b.double(), stride=2, padding=1).float()
                assert torch.equal(torch.isnan(out[img]), torch.isnan(want[img])) and torch.equal(torch.isinf(out[img]), torch.isinf(want[img])), name


def test_weights_take_the_room_of_their_form(mnn, short_variants, tmp_path):
    layer = ConvLayer("room", 2, 40, 20, 20, 70, 3, 3, 1, 1)
    parts, octets = 128 * 48 * 9 * 6, 80 * 64 * 9 * 4
    x, w, b = inputs(layer, 4)
    ref = conv64(layer, x, w, b)
    for v, name in short_variants:
        with planned(mnn, layer, v, tmp_path / "cache") as plan:
            assert plan.workspace_bytes == (octets if name.startswith("f32") else parts), name
            plan.set_weights((w * 3).cuda())
            check(mnn, layer, plan, name, x, w, b, ref)   # prepared again: another pointer
