"""The transforms of short grids: every built F(n,k) on both sides of the rules that choose them, and together with the weights' transform in
the call that allocates nothing."""
import pytest
import torch

from conv_workloads import ConvLayer

pytestmark = pytest.mark.gpu

BUILT = [(n, k) for k in range(2, 8) for n in range(2, 9) if n + k - 1 <= 10]


def mnn():
    import paper_2002_12418_amd
    return paper_2002_12418_amd


def inputs(layer, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.rand(layer.n, layer.c_in, layer.h, layer.w, generator=g) * 2 - 1
    w = torch.randn(layer.c_out, layer.c_in, layer.kh, layer.kw, generator=g)
    return x, w, torch.rand(layer.c_out, generator=g)


def conv64(layer, x, w, b):
    return torch.nn.functional.conv2d(x.double(), w.double(), b.double(), padding=layer.pad)


def error(y, ref):
    return float((y.cpu().double() - ref).abs().max() / ref.abs().max())


def bound(n, k):
    return 1e-4 if n + k - 1 <= 6 else 1e-3


@pytest.mark.parametrize("nk", BUILT, ids=lambda t: f"F({t[0]},{t[1]})")
def test_planned_and_allocation_free(nk):
    m = mnn()
    n, k = nk
    # K and P no multiples of 4 (padding of U and V is written), a single tile, an image narrower than a tile, whole tiles
    for N, C, H, W, K, pad in [(3, 9, 13, 17, 7, k // 2), (1, 5, k, k, 6, 0), (2, 16, 2 * k, 3, 20, k - 1), (2, 8, 4 * n, 4 * n, 12, k // 2)]:
        if W + 2 * pad < k:
            continue
        layer = ConvLayer("short", N, C, H, W, K, k, k, 1, pad)
        x, w, b = inputs(layer, 11 * n + k + H)
        ref = conv64(layer, x, w, b)
        xd, wd, bd = x.cuda(), w.cuda(), b.cuda()
        with m.ConvPlan.for_layer(layer, options=m.Options(force_kind=m.SCHEME_WINOGRAD, force_tile_n=n, force_variant=m.WINO_UNFUSED)) as p:
            guard = torch.full((ref.numel() + 256,), 7.0, device="cuda")
            y = guard[128:128 + ref.numel()].view(ref.shape)
            p.run(xd, wd, bd, y)
            torch.cuda.synchronize()
            assert bool((guard[:128] == 7.0).all()) and bool((guard[128 + ref.numel():] == 7.0).all())
            assert error(y, ref) < bound(n, k)
            off = torch.full((ref.numel() + 1,), 7.0, device="cuda")[1:].view(ref.shape)
            assert torch.equal(p.run(xd, wd, bd, off), y)
        # the scratch array holds what the last call left, here infinities: padding that were not written would show
        inf = torch.full_like(xd, float("inf"))
        s1, s2 = torch.empty_like(y), torch.empty_like(y)
        m.conv_run_static(layer, n, xd, wd, bd, s1)
        m.conv_run_static(layer, n, inf, wd, bd, s2)
        m.conv_run_static(layer, n, xd, wd, bd, s2)
        assert torch.equal(s1, s2) and error(s1, ref) < bound(n, k)


def test_no_cap_on_wavefronts_where_the_short_kernel_runs(tmp_path):
    """The cap on resident wavefronts is one of the other kernel: on a grid long enough for it, none is timed, kept or described."""
    m = mnn()
    options = m.Options(force_kind=m.SCHEME_WINOGRAD, force_tile_n=4, force_variant=m.WINO_UNFUSED)
    # 622592 pairs of channel and tile; alpha 8: a lane per row of a tile, alpha 6: a lane per tile
    for k, capped in ((5, False), (3, True)):
        layer = ConvLayer("cap", 19, 128, 64, 64, 32, k, k, 1, k // 2)
        with m.ConvPlan.for_layer(layer, options=options) as p:
            assert capped or "input-waves/cu" not in p.describe()
        m.cache_save(str(tmp_path / "cache"))
        sizes = ["19", "128", "64", "64", "32", "4", str(k)]
        kept = [l for l in (tmp_path / "cache").read_text().splitlines() if l.startswith("I ") and l.split()[3:10] == sizes]
        assert len(kept) == capped


@pytest.mark.parametrize("nk,shape", [
    ((2, 3), (4, 64, 32, 32, 64)), ((2, 3), (4, 64, 33, 32, 65)),            # C P and K P at 65536, and past it
    ((4, 3), (9, 74, 60, 60, 20)), ((4, 3), (9, 75, 60, 60, 20)),            # alpha 6: 149850 and 151875 pairs
    ((4, 3), (9, 98, 60, 60, 256)), ((4, 3), (9, 98, 60, 60, 257)), ((3, 5), (9, 98, 45, 45, 20)),      # up to 200000 with few output channels
    ((6, 3), (21, 64, 126, 126, 9)), ((4, 5), (24, 64, 80, 82, 20)),         # alpha 8: 592704 pairs and 645120
    ((6, 3), (3, 9, 120, 120, 166)), ((6, 3), (3, 9, 120, 120, 167)),        # its output: 199200 and 200400
    ((5, 5), (4, 64, 80, 80, 64)), ((5, 5), (4, 65, 80, 81, 65)),            # alpha 9: 65536, and past it
    ((8, 3), (4, 244, 128, 128, 40)), ((8, 3), (4, 245, 128, 128, 40)),      # alpha 10: 249856 and 250880
])
def test_both_sides_of_the_rules(nk, shape):
    m = mnn()
    (n, k), (N, C, H, W, K) = nk, shape
    layer = ConvLayer("rules", N, C, H, W, K, k, k, 1, k // 2)
    x, w, b = inputs(layer, n + H)
    with m.ConvPlan.for_layer(layer, options=m.Options(force_kind=m.SCHEME_WINOGRAD, force_tile_n=n, force_variant=m.WINO_UNFUSED)) as p:
        y = p.run(x.cuda(), w.cuda(), b.cuda()).clone()
        assert torch.equal(p.run(x.cuda(), w.cuda(), b.cuda()), y)
    pick = [0, N - 1]                                                         # whole images: the first and the last
    assert error(y[pick], conv64(layer, x[pick], w, b)) < bound(n, k)
