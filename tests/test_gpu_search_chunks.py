"""Small searches, whose blocks take shorter runs of templates: the scores are those of the same pairs in a large
search, bit for bit, at template counts around the runs' lengths."""

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 96, 128, 160])
@pytest.mark.parametrize("window", [-1, 5])
def test_scores_do_not_depend_on_the_call(n, window):
    import torch
    import paper_1807_11313_amd as tm

    g = torch.Generator(device="cuda:0").manual_seed(n)
    f = tm.spectrum_floats(n)
    sp = 1e-2 * torch.randn((90, f), generator=g, device="cuda:0")
    sl = 1e-2 * torch.randn((3000, f), generator=g, device="cuda:0")
    prm = tm.params_default(max_shift=window)
    full = tm.xcf_scores(sp, sl, n, prm)
    for p, l in ((1, 1), (1, 3), (2, 5), (1, 31), (3, 33), (17, 65), (1, 2047), (33, 127), (64, 513)):
        part = tm.xcf_scores(sp[:p].contiguous(), sl[:l].contiguous(), n, prm)
        assert torch.equal(part, full[:p, :l]), (p, l)
