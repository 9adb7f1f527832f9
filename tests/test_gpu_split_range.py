"""FP16 hi + lo products of spectra that are not of unit energy: finite and as accurate, relative to the product of
the norms, up to a product of 60, for patterns against templates and for the spectra with the largest sums (all
energy in one column)."""

import numpy as np
import pytest

from .test_gpu_even import TOL, _band, _exact

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 96, 128, 160, 256])
@pytest.mark.parametrize("s", [7, 16])
def test_scaled_spectra(n, s):
    import torch
    import paper_1807_11313_amd as tm

    g = torch.Generator(device="cuda:0").manual_seed(n)
    b = 3 * n // 8
    base = torch.randn((3, n // 8, n // 8), generator=g, device="cuda:0")
    up = torch.nn.functional.interpolate(base[:, None], size=(n, n), mode="bicubic")[:, 0].contiguous()
    sl = tm.pattern_spectra(up)
    col = torch.zeros((1, 2 * b + 1, b + 1, 2), device="cuda:0")
    col[0, 1, 0, 0] = col[0, 2 * b, 0, 0] = 0.5 ** 0.5                  # X(+-1, 0): A(1) = |E| |T|
    sl = torch.cat([sl, col.reshape(1, -1)]).contiguous()
    ref = _exact(_band(sl, n), _band(sl, n), n, s)
    prm = tm.params_default(max_shift=s, form=2, precision=1)
    for scale in (1.0, 31.0, 60.0):
        for ks, kl in ((scale, 1.0), (1.0, scale), (scale ** 0.5, scale ** 0.5)):
            out = tm.xcf_scores((sl * ks).contiguous(), (sl * kl).contiguous(), n, prm).cpu().numpy()
            assert np.max(np.abs(out / scale - ref)) < TOL, (scale, ks)
