"""Sub-pixel peak against the full grid in 64 bits, over sizes and upsampling factors (coarse strides of
1, 2 and 5 and a last coarse cell that reaches past the grid), for clear peaks, for peaks at the grid's edge,
for pairs without a peak, and for spectra where nothing can be excluded."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# FP32 sums of nk + nv terms with sum |Z| <= 1: (193 + 97 + 16) 2^-24 at the largest size is 1.9e-5 in the worst
# order of roundings; heights agree to a tenth of that here
TOL = 5e-6


def _grid(z, n, s, kappa):
    m = -(-3 * kappa // 4)
    b = 3 * n // 8
    u = np.concatenate([np.arange(b + 1), np.arange(-b, 0)])
    v = np.arange(b + 1)
    off = np.arange(-m, m + 1) / kappa
    wy = np.exp(2j * np.pi * np.outer(s[1] + off, u) / n)
    wx = np.exp(2j * np.pi * np.outer(v, s[0] + off) / n) * np.where(v > 0, 2.0, 1.0)[:, None]
    return np.real(wy @ z @ wx), m


@pytest.mark.parametrize("n", [64, 96, 128, 160, 256])
@pytest.mark.parametrize("kappa", [1, 7, 16, 50, 100])
def test_subpixel_winner(n, kappa):
    import torch
    import paper_1807_11313_amd as tm

    g = torch.Generator(device="cuda:0").manual_seed(n * 1000 + kappa)
    base = torch.randn((6, n // 8, n // 8), generator=g, device="cuda:0")
    imgs = torch.nn.functional.interpolate(base[:, None], size=(n, n), mode="bicubic")[:, 0].contiguous()
    noisy = imgs + 0.2 * torch.randn(imgs.shape, generator=g, device="cuda:0")
    sl, sp = tm.pattern_spectra(imgs), tm.pattern_spectra(noisy.contiguous())
    sp[5] = 0.0
    pi = torch.tensor([0, 1, 2, 3, 4, 5], dtype=torch.int32, device="cuda:0")
    li = torch.tensor([0, 1, 2, 4, 3, 5], dtype=torch.int32, device="cuda:0")     # 3 and 4: no common peak
    s = torch.tensor([[0, 0], [1, 0], [0, -1], [7, -9], [-n // 2, n // 2 - 1], [3, 4]], dtype=torch.int32,
                     device="cuda:0")
    h, sub = tm.xcf_subpixel(sp, sl, pi, li, s, n, tm.params_default(upsample=kappa))
    h, sub = h.cpu().numpy(), sub.cpu().numpy()
    b = 3 * n // 8
    band = lambda x: x.double().cpu().numpy().reshape(-1, 2 * b + 1, b + 1, 2) @ np.array([1.0, 1j])  # noqa: E731
    e, t = band(sp), band(sl)
    for k in range(6):
        c = s[k].cpu().numpy()
        rho, m = _grid(e[int(pi[k])] * np.conj(t[int(li[k])]), n, c, kappa)
        at = np.rint((sub[k] - c) * kappa).astype(int) + m
        assert abs(h[k] - rho.max()) < TOL
        assert rho[at[1], at[0]] > rho.max() - TOL
        if k == 5:                       # all equal: the first point
            assert h[k] == 0.0 and at[0] == 0 and at[1] == 0
