"""Windowed searches (FP16 hi + lo, and FP32 DFT): blocks of several patterns, with remainders, give the bits of blocks
of one, and a few patterns do not cost what many do."""

import pytest

pytestmark = pytest.mark.gpu

FORMS = {"fp16x2": (2, 1), "fp32": (3, 0)}


def _spectra(n, p, l):
    import torch
    import paper_1807_11313_amd as tm

    g = torch.Generator(device="cuda:0").manual_seed(n + p)
    base = torch.randn((64, 1, n // 8, n // 8), generator=g, device="cuda:0")
    up = torch.nn.functional.interpolate(base, size=(n, n), mode="bicubic")[:, 0].contiguous()
    sl = tm.pattern_spectra(up + 0.5 * torch.randn(up.shape, generator=g, device="cuda:0"))
    sp = tm.pattern_spectra(up + 0.5 * torch.randn(up.shape, generator=g, device="cuda:0"))
    at = torch.arange(max(p, l), device="cuda:0")
    return tm, sp[at[:p] % 64].contiguous(), sl[at[:l] * 5 % 64].contiguous()


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("n, s", [(64, 0), (64, 15), (96, 7), (128, 15), (160, 3), (256, 15), (64, 16), (96, 31), (128, 16),
                                  (256, 31)])
def test_blocks_of_patterns_equal_single_ones(form, n, s):
    import torch

    f, prec = FORMS[form]
    # blocks of four from 193 on, of three from 513 on (193 at 256), with remainders on both sides
    for p, l in ((2, 1539), (3, 1545), (5, 1540), (2, 4101), (5, 2060), (9, 1551)):
        tm, sp, sl = _spectra(n, p, l)
        prm = tm.params_default(max_shift=s, form=f, precision=prec)
        out = tm.xcf_scores(sp, sl, n, prm)
        for i in range(p):
            assert torch.equal(out[i:i + 1], tm.xcf_scores(sp[i:i + 1].contiguous(), sl, n, prm)), (p, i)


@pytest.mark.parametrize("n", [128, 256])
def test_few_patterns_cost_little(n):
    import torch

    tm, sp, sl = _spectra(n, 100, 200)
    prm = tm.params_default(max_shift=7, form=3)

    def cost(p):
        best = float("inf")
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                tm.xcf_scores(sp[:p], sl, n, prm)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    cost(4)
    # a block of one pattern against the blocks of four that 100 patterns fill the chip with: measured 29 of 172 us at
    # 128 and 66 of 511 at 256 (63 and 176 where four patterns take a block of four)
    assert cost(4) < 0.25 * cost(100)


@pytest.mark.parametrize("n", [96, 128])
def test_small_windows_cost_what_the_bf16_halves_do(n):
    import torch

    tm, sp, sl = _spectra(n, 600, 1500)

    def cost(precision):
        best = float("inf")
        prm = tm.params_default(max_shift=7, form=2, precision=precision)
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(3):
                tm.xcf_scores(sp, sl, n, prm)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    cost(2)
    fp16, bf16 = cost(1), cost(2)
    print("[gpu]   n=%d: fp16x2 %.3f ms, bf16x2 %.3f ms" % (n, fp16 / 3, bf16 / 3), flush=True)
    # the same products on whole operands: measured 0.94 and 0.96 (1.08 and 1.10 with chunks of 32 rows only)
    assert fp16 < 1.03 * bf16


@pytest.mark.parametrize("n, s", [(64, 15), (96, 15), (128, 7), (160, 15), (256, 15)])
def test_split_blocks_of_two_and_three_equal_single_ones(n, s):
    import torch

    # the blocks that take the fewest rounds of the chip: of two (15 x 500 and 31 x 1,000, 2 x 1,539), of three (the
    # others), with remainders of one and of two patterns
    for p, l in ((2, 1539), (15, 500), (31, 1000), (61, 1000), (62, 1003)):
        tm, sp, sl = _spectra(n, p, l)
        prm = tm.params_default(max_shift=s, form=2, precision=1)
        out = tm.xcf_scores(sp, sl, n, prm)
        for i in {0, 1, p // 2, p - 2, p - 1}:
            assert torch.equal(out[i:i + 1], tm.xcf_scores(sp[i:i + 1].contiguous(), sl, n, prm)), (p, i)


def test_sixteen_patterns_fill_the_chip():
    import torch

    tm, sp, sl = _spectra(256, 48, 500)
    prm = tm.params_default(max_shift=15, form=2, precision=1)

    def cost(p):
        best = float("inf")
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                tm.xcf_scores(sp[:p], sl, 256, prm)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    cost(48)
    # 48 x 500: four full rounds of blocks of three, 222 us; 16 x 500 two of blocks of two, 91 us, but 113 of three
    few, many = cost(16), cost(48)
    print("[gpu]   16 x 500 %.0f us, 48 x 500 %.0f us" % (200 * few, 200 * many), flush=True)
    assert few < 0.46 * many
