"""Shadow marches on grids whose spacing is a power of two (the division by it is a multiplication), is not, and is one
outside the range whose inverse is used: the oracle's visibility bit for bit."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


SPACINGS = [1 / 32, 1 / 30, 0.05, 0.25, 1.0, 3.0, 2.0 ** 30, 1 / 32 + 2.0 ** -28]


# the smallest ones without the triangulated penumbra, whose squares underflow there
@pytest.mark.parametrize("h,penumbra", [(h, p) for h in SPACINGS for p in (0, 1)] +
                         [(2.0 ** -118, 0), (2.0 ** -121, 0)])
def test_shadow_spacing(h, penumbra):
    import torch
    import paper_2210_04449_amd.rtsdf as R
    h = float(np.float32(h))
    n, lo = 24, np.array([-3 * h, 0.5 * h, 0.0], np.float32)
    rng = np.random.default_rng(9)
    c = np.stack(np.meshgrid(*[np.arange(n) + 0.5] * 3, indexing="ij"), -1) - n / 2  # a ball in the middle
    sdf = ((np.linalg.norm(c, axis=-1) - 5.0) * h).astype(np.float32)
    pts = (lo + rng.uniform(-1, n + 1, (5003, 3)) * h).astype(np.float32)
    light = np.array([0.3, 0.9, 0.2], np.float32)
    light /= np.linalg.norm(light)
    g = R.Grid.make(n, h, lo)
    vis = torch.empty(len(pts), device="cuda")
    R.rtsdf_shadow_ex(g, torch.from_numpy(sdf).cuda().reshape(-1), torch.from_numpy(pts).cuda(), light, 8.0, h, 96,
                      2 * h, 30 * h, vis, penumbra=penumbra)
    want = oracle.shadow(n, lo, np.float32(h), sdf, pts, light, 8.0, h, 96, 2 * h, 30 * h, penumbra=penumbra)
    assert np.array_equal(vis.cpu().numpy().view(np.int32), want.view(np.int32))
    assert (want == 0).any() and (want == 1).any()
