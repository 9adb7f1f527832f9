"""Searches that keep no score matrix drop templates by a bound: their picks are the largest of the whole score
matrix, ties to the smallest index, for patterns that match, that match nothing, and that are not finite."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PC = (0.48, 0.55, 0.62)


def _setup(n, p, l):
    import torch
    import paper_1807_11313_amd as tm

    g = torch.Generator(device="cuda:0").manual_seed(n + p + l)
    coarse = torch.rand((1, 1, 24, 24), generator=g, device="cuda:0")
    master = torch.nn.functional.interpolate(coarse, size=(129, 129), mode="bicubic", align_corners=True)
    master = master[0, 0].contiguous()
    q = torch.randn((l, 4), generator=g, device="cuda:0", dtype=torch.float64)
    q = torch.nn.functional.normalize(q, dim=1)
    q = torch.where(q[:, :1] < 0, -q, q).contiguous()
    return tm, g, master, q


def _picks(scores):
    s = scores.cpu().numpy()
    s = np.where(np.isnan(s), -np.inf, s)
    return s.argmax(1)


@pytest.mark.parametrize("n, p, l", [(64, 37, 901), (64, 131, 255), (96, 17, 964), (96, 128, 128), (128, 9, 911), (128, 70, 129), (160, 8, 1024),
                                     (160, 8192, 1), (160, 33, 257)])
def test_picks_are_the_largest_scores(n, p, l):
    import torch

    tm, g, master, q = _setup(n, p, l)
    q[l // 2:l // 2 + l // 4] = q[:l // 4]                               # exact ties
    img = tm.project_templates(master, q, n, PC)
    x = img[torch.arange(p, device="cuda:0") * 7 % l].clone()
    x += (0.1 + torch.arange(p, device="cuda:0") % 5)[:, None, None] * x.std() * torch.randn(x.shape, generator=g,
                                                                                            device="cuda:0")
    x[1] = torch.randn((n, n), generator=g, device="cuda:0")             # matches nothing
    x[2] = 3.0                                                           # constant
    x[3, 1, 1] = float("nan")
    x[4, 0, 0] = float("inf")
    x[5] = -x[5]
    x[6] *= 1e18
    plans = {}
    for window in (-1, 0, 7, n // 3):
        prm = tm.params_default(max_shift=window)
        want = _picks(tm.index_patterns(x, master, PC, q, prm=prm, scores=True)["scores"])
        got = tm.index_patterns(x, master, PC, q, prm=prm)
        assert np.array_equal(got["best_idx"].cpu().numpy(), want), window
        plans[window] = tm.LibraryPlan(master, PC, q, n, prm=prm)
        again = plans[window].index(x)
        for k in got:
            assert torch.equal(torch.nan_to_num(got[k].double()), torch.nan_to_num(again[k].double())), (window, k)


@pytest.mark.parametrize("n, p, l", [(64, 33, 1000), (96, 17, 1024), (128, 16, 1031), (160, 67, 250), (256, 9, 911)])
@pytest.mark.parametrize("form, precision", [(2, 1), (3, 0)])             # split FP16 products, exact FP32 products
@pytest.mark.parametrize("window", [4, 20])
def test_windowed_picks(n, p, l, form, precision, window):
    import torch

    tm, g, master, q = _setup(n, p, l)
    q[l // 2:l // 2 + l // 4] = q[:l // 4]
    img = tm.project_templates(master, q, n, PC)
    x = img[torch.arange(p, device="cuda:0") * 7 % l].clone()
    x += 0.3 * x.std() * torch.randn(x.shape, generator=g, device="cuda:0")
    x[1:5] = torch.randn((4, n, n), generator=g, device="cuda:0")         # whole rows, one block and a part
    x[5] = 3.0
    x[6, 1, 1] = float("nan")
    x[7] = -x[7]
    prm = tm.params_default(form=form, precision=precision, max_shift=window)
    want = tm.index_patterns(x, master, PC, q, prm=prm, scores=True)
    got = tm.index_patterns(x, master, PC, q, prm=prm)
    again = tm.LibraryPlan(master, PC, q, n, prm=prm).index(x)
    assert np.array_equal(got["best_idx"].cpu().numpy(), _picks(want["scores"]))
    for k in got:
        for other in (want, again):
            assert torch.equal(torch.nan_to_num(got[k].double()), torch.nan_to_num(other[k].double())), k


def test_more_pairs_than_a_slab():
    import torch

    tm, g, master, q = _setup(96, 1700, 40000)
    x = tm.project_templates(master, q[::24][:1700 - 33].contiguous(), 96, PC)
    x = torch.cat([x, torch.randn((33, 96, 96), generator=g, device="cuda:0")]).contiguous()
    plan = tm.LibraryPlan(master, PC, q, 96)
    assert np.array_equal(plan.index(x)["best_idx"].cpu().numpy(), _picks(plan.index(x, scores=True)["scores"]))


@pytest.mark.parametrize("eager", [False, True])
def test_ragged_picks(eager):
    import torch

    l, per = 830, 40                                                     # 33,200 pairs of each size
    data, ns, offs, want, at = [], [], [], [], 0
    for n in (160, 96, 64, 128):
        tm, g, master, q = _setup(64, 1, l)
        x = tm.project_templates(master, q[5:5 + 3 * per:3].contiguous(), n, PC)
        x[-1] = torch.randn((n, n), generator=g, device="cuda:0")
        want += _picks(tm.index_patterns(x, master, PC, q, scores=True)["scores"]).tolist()
        ns += [n] * per
        offs += [at + i * n * n for i in range(per)]
        at += per * n * n
        data.append(x.reshape(-1))
    order = np.random.default_rng(3).permutation(len(ns))
    ns, offs, want = np.array(ns)[order], np.array(offs)[order], np.array(want)[order]
    plan = tm.RaggedPlan(ns, offs, l, stencil=False, eager=eager)
    data = torch.cat(data)
    out = plan.run(data, master, PC, q)
    for rep in range(3):                                                 # replays, with other work between
        torch.cuda.synchronize()
        assert np.array_equal(out["best_idx"].cpu().numpy(), want), rep
        out["best_idx"].fill_(-1)
        data.mul_(1.0)
        plan.run_into(data, master, PC, q, out)
    plan.close()


@pytest.mark.parametrize("p, l, k, tau", [(520, 64, 64, -1.0), (500, 70, 70, -1.0), (40, 900, 5, 2.0), (9, 911, 8, 2.0)])
def test_proposed_picks(p, l, k, tau):
    import torch

    # every template a candidate, or every pattern in the fallback: the pick is that of the whole search
    tm, g, master, q = _setup(128, p, l)
    q[l // 2:l // 2 + l // 4] = q[:l // 4]
    img = tm.project_templates(master, q, 128, PC)
    x = img[torch.arange(p, device="cuda:0") * 7 % l].clone()
    x += 0.5 * x.std() * torch.randn(x.shape, generator=g, device="cuda:0")
    x[1] = torch.randn((128, 128), generator=g, device="cuda:0")
    x[2] = 3.0
    x[3, 1, 1] = float("nan")
    net = tm.Cnn(l, seed=1)
    got = tm.index_proposed(x, master, PC, q, net, top_k=k, fallback_tau=tau)
    want = tm.index_patterns(x, master, PC, q, scores=True)
    ok = torch.arange(p, device="cuda:0") != 3                           # its proposals are of NaN logits
    assert torch.equal(got["best_idx"][ok], want["best_idx"][ok])
    assert torch.equal(got["peak_h"][ok], want["peak_h"][ok])
