"""fp32-grade products on the bf16 matrix cores (`x6_...` configurations): accuracy, ranges, non-finite operands, the gather of the
sliding window in every configuration, empty slices of a remembered split."""
import numpy as np
import pytest
import torch

from conv_workloads import ConvLayer

pytestmark = pytest.mark.gpu


def mnn():
    import paper_2002_12418_amd
    return paper_2002_12418_amd


def x6_variants(m):
    return [(i, name) for i, name in enumerate(m.gemm_variants()) if name.startswith(("x6_", "f32_"))]


def product(m, A, B, variant):
    batch, R, M = A.shape
    P = B.shape[2]
    D = torch.full((batch, M, P), 7.0, device="cuda")
    m.gemm_f32(A, B, D, M=M, ncols=P, R=R, batch=batch, variant=variant, strideA_batch=R * M, strideB_batch=R * P, strideD_batch=M * P)
    torch.cuda.synchronize()
    return D


@pytest.mark.parametrize("shape", [(128, 32, 128, 2), (132, 33, 260, 1), (64, 600, 72, 3), (512, 256, 512, 2), (4, 1, 4, 1)])
def test_error_no_larger_than_the_fp32_kernel(shape):
    """Relative 2-norm error against float64, next to the fp32 tile with one accumulator per output."""
    m = mnn()
    M, R, P, batch = shape
    g = torch.Generator().manual_seed(sum(shape))
    A = torch.randn(batch, R, M, generator=g)
    B = torch.randn(batch, R, P, generator=g)
    ref = A.double().transpose(1, 2) @ B.double()
    A, B = A.cuda(), B.cuda()
    fp32 = next(i for i, n in enumerate(m.gemm_variants()) if n == "64x64x16_w2x2")
    err = lambda v: float((product(m, A, B, v).cpu().double() - ref).norm() / ref.norm())
    base = err(fp32)
    for v, name in x6_variants(m):
        e = err(v)
        print(f"[case] {shape} {name}: {e:.2e}, fp32 kernel {base:.2e}", flush=True)
        # one rounding of the result (2^-24) is the floor where the fp32 kernel happens to be exact
        assert e <= max(1.1 * base, 2.0 ** -24), name


def test_operands_of_any_magnitude():
    """Every value keeps its own 24 bits: scales that vary over 2^80 within a reduction cost nothing (bound: 2^-21 of sum |a||b|)."""
    m = mnn()
    M, R, P = 68, 96, 132
    g = torch.Generator().manual_seed(3)
    e = torch.randint(-40, 41, (1, R, 1), generator=g).double()
    A = (torch.randn(1, R, M, generator=g).double() * 2.0 ** e).float()
    B = (torch.randn(1, R, P, generator=g).double() * 2.0 ** -e).float()
    ref = A.double().transpose(1, 2) @ B.double()
    scale = A.double().abs().transpose(1, 2) @ B.double().abs()
    for v, name in x6_variants(m):
        got = product(m, A.cuda(), B.cuda(), v).cpu().double()
        assert float(((got - ref).abs() / scale).max()) < 2.0 ** -21, name


@pytest.mark.parametrize("exponent", [-80, -112, -118, -124])
def test_tiny_operands_as_accurate_as_the_fp32_kernel(exponent):
    """Below 2^-109 a bf16 has no room for the last parts; tiles that hold such operands come from the fp32 instructions.  Either operand, and
    a matrix whose other half is zero."""
    m = mnn()
    M, R, P = 132, 96, 136
    g = torch.Generator().manual_seed(5)
    A = torch.randn(1, R, M, generator=g)
    B = torch.randn(1, R, P, generator=g)
    B[:, :, 70:] = 0.0
    fp32 = next(i for i, n in enumerate(m.gemm_variants()) if n == "64x64x16_w2x2")
    for a, b in ((A * 2.0 ** exponent, B), (A, B * 2.0 ** exponent)):
        ref = a.double().transpose(1, 2) @ b.double()
        ad, bd = a.cuda(), b.cuda()
        err = lambda v: float((product(m, ad, bd, v).cpu().double() - ref).norm() / ref.norm())
        base = err(fp32)
        for v, name in x6_variants(m):
            assert err(v) <= max(1.1 * base, 2.0 ** -24), name


def test_non_finite_operands_as_the_fp32_kernel_has_them():
    """Infinities, NaN, values that round to an infinite bf16 and sums that overflow give what the fp32 kernel gives, and touch
    no other row or column."""
    m = mnn()
    M, R, P = 132, 70, 196
    g = torch.Generator().manual_seed(4)
    A = torch.randn(1, R, M, generator=g)
    B = torch.randn(1, R, P, generator=g)
    A[0, 5, 3] = float("inf")
    A[0, 69, 131] = float("nan")
    A[0, 7, 40] = 3.4e38
    B[0, 11, 100] = float("-inf")
    B[0, 12, 100] = 0.5
    B[0, 7, 77] = 3.3e38
    B[0, 64, 195] = torch.finfo(torch.float32).max
    # no output gets an infinity and an overflowing finite product: whether that product overflows on its own depends on the order
    A[0, 64, 3] = A[0, 64, 40] = A[0, 7, 3] = B[0, 7, 100] = 0.0
    A, B = A.cuda(), B.cuda()
    fp32 = next(i for i, n in enumerate(m.gemm_variants()) if n == "64x64x16_w2x2")
    want = product(m, A, B, fp32).cpu()
    fine = torch.isfinite(want)
    assert (~fine).sum() > 300 and fine.sum() > 20000
    for v, name in x6_variants(m):
        got = product(m, A, B, v).cpu()
        assert torch.equal(torch.isnan(got), torch.isnan(want)), name
        assert torch.equal(got[torch.isinf(want)], want[torch.isinf(want)]), name
        assert torch.equal(torch.isfinite(got), fine), name
        assert torch.allclose(got[fine].double(), want[fine].double(), rtol=1e-4, atol=1e-4), name


# strides, dilation, padding beyond the kernel, channel counts around the groups of 8, one output pixel
GATHER = [
    ConvLayer("s2", 3, 16, 15, 13, 33, 3, 3, 2, 1),
    ConvLayer("c3", 2, 3, 17, 19, 20, 7, 7, 2, 3),
    ConvLayer("c9_d2", 1, 9, 14, 12, 70, 3, 3, 1, 2, 2),
    ConvLayer("c1_k2", 2, 1, 9, 9, 5, 2, 2, 1, 0),
    ConvLayer("c40_1px", 5, 40, 3, 3, 12, 3, 3, 1, 0),
    ConvLayer("c64_wide_pad", 1, 64, 6, 7, 130, 3, 5, 1, (3, 4)),
]


def rewrite_choices(m, path, prec, pick):
    """Replaces the remembered GEMM configuration of every entry of this precision (the last key value) and loads the file."""
    m.cache_save(str(path))
    out = []
    for line in path.read_text().splitlines():
        if line.startswith("G "):
            head, _ = line.split("|")
            if int(head.split()[-1]) == prec:
                line = f"{head}| {pick[0]} {pick[1]}"
        out.append(line)
    path.write_text("\n".join(out) + "\n")
    m.cache_clear()
    m.cache_load(str(path))


@pytest.mark.parametrize("layer", GATHER, ids=lambda l: l.name)
def test_sliding_window_in_every_configuration(layer, tmp_path):
    m = mnn()
    g = torch.Generator().manual_seed(layer.c_in)
    x = torch.rand(layer.n, layer.c_in, layer.h, layer.w, generator=g) * 2 - 1
    w = torch.randn(layer.c_out, layer.c_in, layer.kh, layer.kw, generator=g)
    b = torch.rand(layer.c_out, generator=g)
    ref = torch.nn.functional.conv2d(x.double(), w.double(), b.double(), stride=layer.stride, padding=layer.pad, dilation=layer.dil)
    x, w, b = x.cuda(), w.cuda(), b.cuda()
    for prec, tol in ((m.GEMM_FP32, 2e-6), (m.GEMM_BF16X3, 3e-5), (m.GEMM_BF16, 1e-2)):
        opt = m.Options(force_kind=m.SCHEME_DIRECT, force_prec=prec)
        names = m.gemm_variants(prec)
        for v in range(1, len(names)):
            if prec == m.GEMM_FP32 and not names[v].startswith(("x6_", "f32_")):
                continue
            for split in (1, 3, 64):                # 64: most slices are empty
                m.cache_clear()
                m.ConvPlan.for_layer(layer, options=opt).close()
                rewrite_choices(m, tmp_path / "cache", prec, (v, split))
                with m.ConvPlan.for_layer(layer, options=opt) as plan:
                    assert names[v] in plan.describe(), plan.describe()
                    y = plan.run(x, w, b)
                    torch.cuda.synchronize()
                    err = float((y.cpu().double() - ref).abs().max() / ref.abs().max())
                    assert err < tol, (names[v], split, err)
    m.cache_clear()


@pytest.mark.parametrize("c", [9, 67, 260])
@pytest.mark.parametrize("pointwise", [True, False])
def test_non_finite_image_stays_in_its_image(c, pointwise, tmp_path):
    """Channel counts that are no multiple of the groups of 8: the rows past the end of the reduction lie in the next image, whose infinities
    and NaN must not reach this one.  Tiles on the fp32 instructions give the very bits they give without them; of the others a block that
    holds a non-finite column is formed on the fp32 instructions as a whole."""
    m = mnn()
    k = 1 if pointwise else 3
    layer = ConvLayer("nf", 3, c, 3, 5, 20, k, k, 1, 0 if pointwise else 1)
    g = torch.Generator().manual_seed(c)
    x = torch.rand(layer.n, c, layer.h, layer.w, generator=g) * 2 - 1
    w = torch.randn(layer.c_out, c, k, k, generator=g)
    ref = torch.nn.functional.conv2d(x.double(), w.double(), padding=layer.pad)
    bad = x.clone()
    bad[1, :8, :, :] = torch.tensor([float("inf"), float("nan")] * 4)[:, None, None]
    x, bad, w = x.cuda(), bad.cuda(), w.cuda()
    opt = m.Options(force_kind=m.SCHEME_GEMM1X1 if pointwise else m.SCHEME_DIRECT)
    names = m.gemm_variants()
    failed = []
    for v in range(1, len(names)):
        for split in (1, 2):
            m.cache_clear()
            m.ConvPlan.for_layer(layer, options=opt).close()
            rewrite_choices(m, tmp_path / "cache", m.GEMM_FP32, (v, split))
            with m.ConvPlan.for_layer(layer, options=opt) as plan:
                try:
                    clean = plan.run(x, w, None).cpu()
                    got = plan.run(bad, w, None).cpu()
                except m.MnnError:          # the older tiles refuse a split with an empty slice
                    assert split > 1 and not names[v].startswith(("x6_", "f32_")), names[v]
                    continue
            for i in (0, 2):
                err = float((got[i].double() - ref[i]).abs().max() / ref.abs().max())
                if not err < 2e-6 or (not names[v].startswith("x6_") and not torch.equal(got[i], clean[i])):
                    failed.append((names[v], split, i, err))
            assert torch.isnan(got[1, :, 0, 0]).all(), names[v]
    m.cache_clear()
    assert not failed, failed


def test_few_columns_without_timing_keep_images_apart():
    """Variant 0 at 16 columns and fewer: a fully connected layer on a few samples."""
    m = mnn()
    M, R, P = 40, 300, 7
    g = torch.Generator().manual_seed(1)
    A, B = torch.randn(R, M, generator=g), torch.randn(P, R, generator=g)
    ref = (A.double().T @ B.double().T)
    B[3, :6] = float("nan")
    D = torch.zeros(P, M, device="cuda")
    m.gemm_f32(A.cuda(), B.cuda(), D, M=M, ncols=P, R=R, L=1, strideB_img=R, strideB_row=1, strideD_img=M, strideD_row=1)
    got = D.cpu().double().T
    others = [i for i in range(P) if i != 3]
    assert torch.isnan(got[:, 3]).all()
    assert float((got[:, others] - ref[:, others]).abs().max() / ref.abs().max()) < 2e-6


def tiny_error(m, A, B, v, absolute=0.0):
    """Largest error of an output in units of sum |a||b| (+ the spacing of the smallest fp32 values, where results come near it)."""
    ref = A.double().transpose(1, 2) @ B.double()
    scale = A.double().abs().transpose(1, 2) @ B.double().abs()
    got = product(m, A.cuda(), B.cuda(), v).cpu().double()
    return float((((got - ref).abs() - absolute).clamp_min(0) / scale.clamp_min(1e-300)).max())


@pytest.mark.parametrize("exponent,factor", [(-118, 0), (-126, 0), (-126, 40), (-140, 0), (-140, 30), (-147, 60)])
@pytest.mark.parametrize("where", ["column", "row", "column_of_all", "one_row_of_reduction"])
def test_tiny_operands_beside_ordinary_ones(exponent, factor, where):
    """One column (row) of tiny values in a tile of ordinary ones, and tiny values times large ones: each output keeps what the fp32
    instructions give it.  Bound: R roundings of 2^-24 of sum |a||b|, and of the spacing 2^-149 where products fall below the normal range."""
    m = mnn()
    M, R, P = 68, 48, 132
    g = torch.Generator().manual_seed(6)
    A = torch.randn(1, R, M, generator=g)
    B = torch.randn(1, R, P, generator=g)
    t = 2.0 ** exponent
    if where == "column":
        B[:, :, 5] *= t
        A *= 2.0 ** factor
    elif where == "row":
        A[:, :, 37] *= t
        B *= 2.0 ** factor
    elif where == "column_of_all":
        B *= t
        A *= 2.0 ** factor
    else:                                     # outputs of column 9 see the tiny row of B only
        B[:, 20] *= t
        B[:, :20, 9] = 0
        B[:, 21:, 9] = 0
        A *= 2.0 ** factor
    bound, absolute = R * 2.0 ** -24, R * 2.0 ** -149
    fp32 = next(i for i, n in enumerate(m.gemm_variants()) if n == "64x64x16_w2x2")
    assert tiny_error(m, A, B, fp32, absolute) <= bound
    errs = {name: tiny_error(m, A, B, v, absolute) for v, name in x6_variants(m)}
    assert all(e <= bound for e in errs.values()), errs


@pytest.mark.parametrize("exponents", [(-60, -50), (-60, -66), (-60, -70), (-70, -72), (-80, -72)])
def test_products_at_the_end_of_the_range(exponents):
    """Operands that three parts hold, products that are subnormal or below: the matrix cores keep subnormal values, so every configuration is
    as far off as the fp32 tile, R spacings of 2^-149 at the most beside its R roundings."""
    m = mnn()
    M, R, P = 68, 48, 132
    g = torch.Generator().manual_seed(7)
    A = torch.randn(1, R, M, generator=g) * 2.0 ** exponents[0]
    B = torch.randn(1, R, P, generator=g) * 2.0 ** exponents[1]
    for v, name in x6_variants(m):
        assert tiny_error(m, A, B, v, R * 2.0 ** -149) <= R * 2.0 ** -24, name


def test_equal_parts_in_every_term():
    """Operands whose lower parts are as large as they get and of one sign, so that the part products left out all add up: still no more than
    the rounding of a product, 2^-24."""
    m = mnn()
    M, R, P = 64, 512, 64
    x = 1.0 + 2.0 ** -8 - 2.0 ** -10 + 2.0 ** -17 - 2.0 ** -19
    A, B = torch.full((1, R, M), x), torch.full((1, R, P), x)
    ref = R * float(A[0, 0, 0].double()) ** 2
    for v, name in x6_variants(m):
        got = product(m, A.cuda(), B.cuda(), v).cpu().double()
        # 2^-24 for the terms, 2^-24 for each of the R / 16 steps of the sum at the most
        assert float((got - ref).abs().max()) / ref <= (1 + R / 16) * 2.0 ** -24, name


def test_bf16_operands_past_the_range_checked_loader(tmp_path):
    """Rows of 2^18 weights, more than the 32-bit offsets of the range-checked loader are used for: every bf16 configuration and its split of
    the reduction, plain and gathered."""
    m = mnn()
    K, c = 1 << 18, 8
    g = torch.Generator().manual_seed(2)
    layer = ConvLayer("wide", 1, c, 3, 2, K, 3, 3, 1, 1)
    x = torch.rand(1, c, 3, 2, generator=g) * 2 - 1
    w = torch.randn(K, c, 3, 3, generator=g)
    ref = torch.nn.functional.conv2d(x.double(), w.double(), padding=1)
    A, B = torch.randn(1, 70, 200, generator=g), torch.randn(1, 70, 36, generator=g)
    pref = A.double().transpose(1, 2) @ B.double()
    Aw = torch.zeros(70, K)
    Aw[:, :200] = A[0]
    x, w, Aw, B = x.cuda(), w.cuda(), Aw.cuda(), B.cuda()
    for prec, tol in ((m.GEMM_BF16X3, 3e-5), (m.GEMM_BF16, 1e-2)):
        opt = m.Options(force_kind=m.SCHEME_DIRECT, force_prec=prec)
        names = m.gemm_variants(prec)
        for v in range(1, len(names)):
            for ncols in (36, 35):                              # 16-byte loads and single ones
                D = torch.zeros(200, ncols, device="cuda")
                m.gemm_f32(Aw, B[:, :, :ncols].contiguous(), D, M=200, ncols=ncols, R=70, lda=K, variant=v, prec=prec)
                err = float((D.cpu().double() - pref[0, :, :ncols]).abs().max() / pref.abs().max())
                assert err < tol, (names[v], ncols, err)
            for split in (1, 2):
                m.cache_clear()
                m.ConvPlan.for_layer(layer, options=opt).close()
                rewrite_choices(m, tmp_path / "cache", prec, (v, split))
                with m.ConvPlan.for_layer(layer, options=opt) as plan:
                    assert names[v] in plan.describe() and ("splitk=2" in plan.describe()) == (split == 2)
                    y = plan.run(x, w, None)
                    err = float((y.cpu().double() - ref).abs().max() / ref.abs().max())
                    assert err < tol, (names[v], split, err)
    m.cache_clear()


@pytest.mark.parametrize("shape", [(103, 130, 326, 1), (64, 64, 32768, 1), (64, 64, 32704, 1), (64, 64, 49152, 1), (130, 70, 260, 72), (130, 70, 257, 72), (130, 128, 257, 72), (33, 9, 3, 36)])
def test_products_without_a_named_configuration(shape):
    """Variant 0 on both sides of the number of tiles, and of the alignment, at which it takes another one: the bits of the configuration it
    stands for."""
    m = mnn()
    M, R, P, batch = shape
    lda = (M + 3) // 4 * 4
    g = torch.Generator().manual_seed(sum(shape))
    A, B = torch.randn(batch, R, lda, generator=g), torch.randn(batch, R, P, generator=g)
    ref = A[:, :, :M].double().transpose(1, 2) @ B.double()
    A, B = A.cuda(), B.cuda()
    tiles = -(-M // 64) * -(-P // 64) * batch
    few = R > 32 and (tiles < 512 or P % 4 != 0)
    stands_for = "bf16_64x64x64_w2x2" if few else "bf16_64x128x32_w1x4" if M <= 64 else "bf16_128x128x32_w2x2"
    fills = -(-R // 64) * 64 * 4 <= R * 5
    many = ("x6_64x64x64_w2x2" if (fills if P % 4 else tiles < 768) else "x6_64x128x32_w1x4" if M <= 64
            else "x6_128x64x32_w2x2" if P % 4 else "x6_128x128x32_w2x2")
    for prec, name, tol in ((m.GEMM_BF16X3, stands_for, 3e-5), (m.GEMM_BF16, stands_for, 1e-2), (m.GEMM_FP32, many, 2e-6)):
        if prec == m.GEMM_FP32 and (R < 64 or tiles < 512):
            continue                                     # the rule for fewer tiles: other tests
        out = []
        for v in (0, m.gemm_variants(prec).index(name)):
            D = torch.zeros(batch, M, P, device="cuda")
            m.gemm_f32(A, B, D, M=M, ncols=P, R=R, batch=batch, lda=lda, variant=v, prec=prec, strideA_batch=R * lda, strideB_batch=R * P, strideD_batch=M * P)
            out.append(D.cpu())
        assert torch.equal(*out)
        assert float((out[0].double() - ref).abs().max() / ref.abs().max()) < tol


@pytest.mark.parametrize("c", [1, 3, 4, 9])
@pytest.mark.parametrize("prec", ["fp32", "bf16x3", "bf16"])
def test_sliding_windows_over_few_channels(c, prec):
    """1 to 3 channels take other kernels than 4 do (in large grids 4 and 9, others than 5): planned in every precision, and the call without
    timing, at 64 and 65 output channels."""
    m = mnn()
    p = {"fp32": m.GEMM_FP32, "bf16x3": m.GEMM_BF16X3, "bf16": m.GEMM_BF16}[prec]
    tol = {"fp32": 2e-6, "bf16x3": 3e-5, "bf16": 1e-2}[prec]
    g = torch.Generator().manual_seed(c)
    for k_out, n, h in ((64, 1, 27), (65, 1, 27), (65, 9, 63), (65, 8, 120)):
        layer = ConvLayer("few", n, c, h, h + 1, k_out, 7, 7, 2, 3)
        x, w = torch.rand(n, c, h, h + 1, generator=g) * 2 - 1, torch.randn(k_out, c, 7, 7, generator=g)
        ref = torch.nn.functional.conv2d(x.double(), w.double(), stride=2, padding=3)
        x, w = x.cuda(), w.cuda()
        with m.ConvPlan.for_layer(layer, options=m.Options(force_kind=m.SCHEME_DIRECT, force_prec=p)) as plan:
            got = [plan.run(x, w, None)]
        if prec == "fp32":
            got.append(m.conv_run_static(layer, 0, x, w, None, torch.full(ref.shape, float("nan"), device="cuda")))
        for y in got:
            assert float((y.cpu().double() - ref).abs().max() / ref.abs().max()) < tol, (k_out, n)
