"""Bound-pruned searches over libraries that give patterns long lists: slices of a row, the second bound's sample, lists
of 16-entry chunks, whole rows; and patterns that match nothing cost about what the full search does."""

import numpy as np
import pytest

from .test_gpu_prune import PC, _picks, _setup

pytestmark = pytest.mark.gpu


def _patterns(tm, g, master, q, n, p):
    import torch

    l = len(q)
    img = tm.project_templates(master, q[torch.arange(p, device="cuda:0") * 7 % l].contiguous(), n, PC)
    # from matching patterns over ones that keep a part of the library to noise
    noise = torch.randn(img.shape, generator=g, device="cuda:0") * img.std()
    x = img + torch.logspace(-1, 1.5, p, device="cuda:0")[:, None, None] * noise
    x[p // 2] = 3.0                                                      # keeps every template: all scores equal
    x[p // 3, 1, 1] = float("nan")
    x[p // 4] = noise[0]
    return x.contiguous()


# (p, l): rows of one slice of up to 4,096 templates, of several, of slices with few templates
@pytest.mark.parametrize("n, p, l", [(64, 40, 5000), (64, 520, 4100), (96, 12, 4097), (96, 520, 1030), (128, 14, 2500),
                                     (128, 513, 4100), (160, 10, 2500), (160, 300, 257)])
@pytest.mark.parametrize("window", [-1, 15])
def test_long_lists(n, p, l, window):
    tm, g, master, q = _setup(n, p, l)
    q[l // 2:l // 2 + l // 4] = q[:l // 4]
    x = _patterns(tm, g, master, q, n, p)
    plan = tm.LibraryPlan(master, PC, q, n, prm=tm.params_default(max_shift=window))
    want = _picks(plan.index(x, scores=True)["scores"])
    assert np.array_equal(plan.index(x)["best_idx"].cpu().numpy(), want)


@pytest.mark.parametrize("n, p, l", [(64, 66, 1000), (64, 20, 4200), (96, 34, 1000), (96, 12, 4200), (128, 66, 1000),
                                     (128, 20, 4200), (160, 66, 1000), (160, 300, 900), (256, 17, 1000), (256, 8, 4200)])
@pytest.mark.parametrize("form, precision", [(2, 1), (3, 0)])
@pytest.mark.parametrize("window", [5, 31])
def test_long_windowed_lists(n, p, l, form, precision, window):
    import torch

    tm, g, master, q = _setup(n, p, l)
    q[l // 2:l // 2 + l // 4] = q[:l // 4]
    x = _patterns(tm, g, master, q, n, p)
    prm = tm.params_default(form=form, precision=precision, max_shift=window)
    plan = tm.LibraryPlan(master, PC, q, n, prm=prm)
    want, got = plan.index(x, scores=True), plan.index(x)
    assert np.array_equal(got["best_idx"].cpu().numpy(), _picks(want["scores"]))
    for k in got:
        assert torch.equal(torch.nan_to_num(got[k].double()), torch.nan_to_num(want[k].double())), k


@pytest.mark.parametrize("n, p, l, form, precision", [(64, 33, 1000, 1, 0), (64, 11, 3000, 1, 0), (96, 200, 4000, 1, 0),
                                                      (160, 8, 1100, 1, 0), (128, 33, 1000, 2, 1), (160, 17, 1000, 3, 0)])
def test_noise_costs_what_the_full_search_does(n, p, l, form, precision):
    import torch

    tm, g, master, q = _setup(n, p, l)
    prm = tm.params_default(form=form, precision=precision, max_shift=-1 if form == 1 else 15)
    plan = tm.LibraryPlan(master, PC, q, n, prm=prm)
    x = torch.randn((p, n, n), generator=g, device="cuda:0")

    def cost(scores):
        best = float("inf")
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                plan.index(x, scores=scores)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    cost(True)
    pruned, full = cost(False), cost(True)
    print("[gpu]   n=%d %d x %d form %d: noise %.0f us, every pair %.0f" % (n, p, l, form, 200 * pruned, 200 * full),
          flush=True)
    assert pruned < 1.25 * full
