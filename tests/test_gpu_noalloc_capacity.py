"""The largest batches that the static scratch of the allocation-free refinement holds at the default parameters
(256 MiB for the patterns' buffers, the tables beside them): accepted, and equal to the allocating call."""

import pytest
import torch

from .gpu_util import tm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, p", [(64, 3901), (96, 1744), (128, 983), (160, 630), (256, 208)])
def test_largest_batch(n, p):
    t = tm()
    g = torch.Generator(device="cuda:0").manual_seed(n)
    master = torch.rand((65, 129), generator=g, device="cuda:0")
    q = torch.nn.functional.normalize(torch.randn((p, 4), generator=g, device="cuda:0", dtype=torch.float64), dim=1)
    q = torch.where(q[:, :1] < 0, -q, q).contiguous()
    x = torch.randn((p, n, n), generator=g, device="cuda:0")
    prm = t.params_default(n_iter=1, max_shift=15 if n == 256 else -1)
    want = t.refine_orientations(x, master, (0.5, 0.5, 0.6), q, prm=prm)
    got = t.refine_orientations(x, master, (0.5, 0.5, 0.6), q, prm=prm, noalloc=True)
    for k in ("q", "peak_h", "shift"):
        assert torch.equal(got[k], want[k]), k
