"""Allocation-free call, products and inverse transform in one kernel: around the sizes at which it is taken, at the edges of its tiles and steps."""
import pytest
import torch

from conv_workloads import ConvLayer

pytestmark = pytest.mark.gpu

# (n, k), the most channels of the one kernel; one more takes two
TAKEN = [((2, 2), 128), ((2, 3), 64), ((3, 2), 64), ((2, 4), 32), ((3, 3), 32), ((4, 2), 32), ((2, 5), 32), ((3, 4), 32), ((4, 3), 32), ((5, 2), 32)]


@pytest.mark.parametrize("tile,most", TAKEN, ids=lambda v: str(v).replace(" ", ""))
def test_against_float64(tile, most):
    import paper_2002_12418_amd as m
    n, k = tile
    g = torch.Generator().manual_seed(n * 10 + k)
    for images, c, h, w, k_out in ((1, most, 11, 9, 33), (1, most + 1, 11, 9, 33), (3, 5, 8, 8, 16), (2, 8, 5, 23, 1), (1, min(most, 31), 4 * n + k - 1, 4 * n + k - 1, 17), (4, 16, 30, 29, 40)):
        layer = ConvLayer("static", images, c, h, w, k_out, k, k, 1, k // 2)
        x, wt = torch.rand(images, c, h, w, generator=g) * 2 - 1, torch.randn(k_out, c, k, k, generator=g)
        b = torch.rand(k_out, generator=g)
        for bias in (b, None):
            ref = torch.nn.functional.conv2d(x.double(), wt.double(), bias.double() if bias is not None else None, padding=k // 2)
            guard = torch.full((ref.numel() + 257,), 7.0, device="cuda")
            for off in (128, 129):                              # wide stores, single ones
                y = guard[off:off + ref.numel()].view(ref.shape)
                y.fill_(float("nan"))
                m.conv_run_static(layer, n, x.cuda(), wt.cuda(), bias.cuda() if bias is not None else None, y)
                # the bound that Winograd with alpha <= 6 is held to everywhere is 1e-4; its fp32 transforms give some 1e-6
                assert float((y.cpu().double() - ref).abs().max() / ref.abs().max()) < 1e-5, (layer, off)
                assert bool((guard[:off] == 7.0).all()) and bool((guard[off + ref.numel():] == 7.0).all())
                guard.fill_(7.0)


def test_what_lies_behind_the_last_channel_does_not_matter():
    """Infinities and NaN of one image, and in the scratch memory of the call before, stay out of the others."""
    import paper_2002_12418_amd as m
    g = torch.Generator().manual_seed(1)
    layer = ConvLayer("static", 2, 13, 10, 10, 20, 3, 3, 1, 1)
    x, w = (torch.rand(2, 13, 10, 10, generator=g) * 2 - 1).cuda(), torch.randn(20, 13, 3, 3, generator=g).cuda()
    clean = m.conv_run_static(layer, 2, x, w, None, torch.empty(2, 20, 10, 10, device="cuda"))
    bad = x.clone()
    bad[0] = float("inf")
    bad[0, 12] = float("nan")
    out = m.conv_run_static(layer, 2, bad, w, None, torch.empty_like(clean))
    assert torch.equal(out[1], clean[1]) and not bool(torch.isfinite(out[0]).any())
    again = m.conv_run_static(layer, 2, x, w, None, torch.empty_like(clean))
    assert torch.equal(again, clean)
