"""The integer peak's forms (with the map, with a window, with neither) agree: the largest map value, ties to the first
row and column, and its signed shift."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 96, 128, 160])
@pytest.mark.parametrize("k", [1, 9])
def test_peak_is_the_first_largest_of_the_map(n, k):
    import torch
    import paper_1807_11313_amd as tm

    g = torch.Generator(device="cuda:0").manual_seed(n + k)
    x = torch.randn((k, n, n), generator=g, device="cuda:0")
    y = torch.roll(x, shifts=(3, -2), dims=(1, 2)) + torch.randn(x.shape, generator=g, device="cuda:0")
    y[k - 1] = 1.0                                                       # no energy: all values tie
    sp, sl = tm.pattern_spectra(x), tm.pattern_spectra(y)
    pi = torch.arange(k, dtype=torch.int32, device="cuda:0")
    for window in (-1, 0, 4, n // 2 - 1):
        prm = tm.params_default(max_shift=window)
        h, s = tm.xcf_peak(sp, sl, pi, pi, n, prm=prm)[:2]
        hm, sm, m = tm.xcf_peak(sp, sl, pi, pi, n, prm=prm, want_map=True)
        assert torch.equal(h, hm) and torch.equal(s, sm)
        m = m.cpu().numpy()
        sh = (np.arange(n) + n // 2) % n - n // 2
        inside = np.abs(sh) <= window if window >= 0 else np.ones(n, bool)
        m = np.where(inside[:, None] & inside[None], m, -np.inf).reshape(k, -1)
        at = m.argmax(1)
        assert np.array_equal(h.cpu().numpy(), m[np.arange(k), at])
        assert np.array_equal(s.cpu().numpy(), np.stack([sh[at % n], sh[at // n]], 1))
