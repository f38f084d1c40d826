"""Voxelization of triangles none of whose projections a lane takes: full workgroups leave 512 x 3 projections to their
wavefronts, or to the workgroup, and sparse ones theirs to wavefronts without triangles; the oracle's voxels, bit for
bit.  The triangles lie along one diagonal plane, so most of the grid stays empty."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nt,size,side", [(32, 530000, 0.2, 1.0), (32, 1500, 0.2, 0.9), (64, 530000, 0.1, 1.0),
                                            (64, 20000, 0.1, 1.0), (128, 6000, 0.3, 1.0), (256, 3000, 0.07, 1.3),
                                            (256, 700, 0.6, 1.0)])
def test_projections_left_by_lanes(n, nt, size, side):
    import torch
    import paper_2210_04449_amd.rtsdf as R
    rng = np.random.default_rng(n + nt)
    a, b = np.array([1, -1, 0]) / np.sqrt(2), np.array([1, 1, -2]) / np.sqrt(6)
    c = rng.uniform(-0.4, 0.4, (nt, 1, 2))
    angle = rng.uniform(0, 6.3, (nt, 1)) + np.array([0, 2.1, 4.2]) + rng.uniform(-0.5, 0.5, (nt, 3))
    q = c + size * rng.uniform(0.6, 1.0, (nt, 3, 1)) * np.stack([np.cos(angle), np.sin(angle)], -1)
    v = 0.5 + q[..., :1] * a + q[..., 1:] * b + rng.uniform(-0.02, 0.02, (nt, 1, 3))
    v = (np.clip(v, -0.9, 1.9) * side).reshape(-1, 3).astype(np.float32)
    f = np.arange(3 * nt, dtype=np.int32).reshape(-1, 3)
    g = R.Grid.make(n, side / n)
    want = oracle.voxelize(v, f, np.zeros(3, np.float32), np.float32(side / n), n)
    assert 0.01 < (want >= 0).mean() < 0.5
    seeds = torch.empty(n ** 3, dtype=torch.int32, device="cuda")
    R.rtsdf_voxelize(torch.from_numpy(v).cuda(), torch.from_numpy(f).cuda(), g, seeds)
    assert np.array_equal(seeds.cpu().numpy(), want)
    assert R.rtsdf_sync_status() == 0
