"""The rotation measurement over log-polar grids: every row-transform length, other lengths (the direct
form), one and several samples per lane with a remainder, upsampling factors down to 1, and images of the size
that is read from global memory, against the oracle's interpolant."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_rho,n_eta", [(64, 32, 128), (64, 7, 100), (96, 48, 192), (128, 64, 256), (128, 33, 130),
                                           (160, 80, 320), (160, 9, 512), (256, 40, 512)])
@pytest.mark.parametrize("kappa", [1, 7, 100])
def test_rotation_grid(n, n_rho, n_eta, kappa):
    import torch
    import paper_1807_11313_amd as tm
    from oracle import refine, spectra

    g = torch.Generator(device="cuda:0").manual_seed(n + n_eta)
    base = torch.randn((3, 10, 10), generator=g, device="cuda:0")
    t = torch.nn.functional.interpolate(base[:, None], size=(n, n), mode="bicubic", align_corners=True)[:, 0]
    p = t + 0.1 * torch.randn(t.shape, generator=g, device="cuda:0")
    p[1] = torch.rot90(t[1], 1)          # a quarter turn
    p[2] = t[0]                          # unrelated
    gam = tm.measure_rotation(p.contiguous(), t.contiguous(),
                              tm.params_default(upsample=kappa, n_rho=n_rho, n_eta=n_eta)).cpu().numpy()
    for k in range(3):
        le = refine.logpolar(spectra.normalise(p[k].cpu().numpy()), n_rho, n_eta)
        lt = refine.logpolar(spectra.normalise(t[k].cpu().numpy()), n_rho, n_eta)
        c = refine.eta_correlation(le, lt)
        best, _ = refine.eta_peak(c, kappa)
        d = gam[k] * n_eta / (2 * np.pi)
        assert abs(d * kappa - round(d * kappa)) < 1e-6
        # the interpolant at the measured shift is the largest within the FP32 rounding of n_eta / 2 + n_rho n_eta
        # terms of sum at most 1 (statistically: sqrt of their number times 6e-8, times 10)
        assert refine.eta_value(c, d)[0] > best - 6e-7 * np.sqrt(n_rho * n_eta) ** 0.5
