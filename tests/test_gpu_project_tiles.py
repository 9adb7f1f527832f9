"""Template projection at the edges of its 32 x 32 px tiles and of the master's azimuth seam."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4, 31, 33, 64, 100])
@pytest.mark.parametrize("shape", [(4, 4), (5, 7), (64, 130), (256, 256)])
def test_project_tiles_and_seam(n, shape):
    import torch
    import paper_1807_11313_amd as tm
    from oracle import geometry, rotations
    from fixtures.orient import random_quats

    rng = np.random.default_rng(n)
    # a smooth master: the lookup's sensitivity to the FP32 direction is bounded by its slope
    h, w = shape
    th, ph = (np.arange(h) + 0.5) * np.pi / h, 2 * np.pi * np.arange(w) / w
    master = (1.0 + 0.5 * np.cos(th)[:, None] + 0.25 * np.sin(th)[:, None] * np.cos(ph + 0.3)[None, :]).astype(np.float32)
    q = random_quats(rng, 4)
    q[0] = (1.0, 0.0, 0.0, 0.0)        # looks along the pole: every azimuth, the seam included
    pcs = np.array([[0.5, 0.5, 0.6], [0.45, 0.55, 0.62], [0.6, 0.4, 0.5], [0.5, 0.2, 0.7]])
    dev = torch.device("cuda:0")
    out = tm.project_templates(torch.as_tensor(master, device=dev), torch.as_tensor(q, device=dev), n,
                               (0.5, 0.5, 0.6), torch.as_tensor(pcs, device=dev)).cpu().numpy()
    for k in range(4):
        r = rotations.quat_to_matrix(q[k:k + 1])[0]
        ref = geometry.project(master, r, n, pcs[k])
        # the azimuth is ill-conditioned within a few pixels of the pole on a coarse master; the FP32 direction
        # error (about 4e-7 rad) over the polar distance times the largest azimuth slope bounds it everywhere else
        c = geometry.crystal_directions(r, n, pcs[k])
        sin_t = np.sqrt(c[..., 0] ** 2 + c[..., 1] ** 2)
        tol = 2e-5 + 4e-7 / np.maximum(sin_t, 1e-9)
        assert np.all(np.abs(out[k] - ref) <= tol), (k, np.max(np.abs(out[k] - ref) - tol))
