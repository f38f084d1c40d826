"""Voxelization by lanes, wavefronts and workgroups against the oracle, bit for bit: triangles of every size class and
at the classes' edges (16 and 512 columns, 32-voxel edges), slivers, degenerate and lattice-aligned ones, vertices outside
the grid, more triangles than a workgroup holds, voxel sizes that are and are not a power of two, shifted grids."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _triangles(rng, nt, size, lattice):
    c = rng.uniform(-0.6, 1.6, (nt, 1, 3))
    v = c + rng.uniform(-1, 1, (nt, 3, 3)) * size
    if lattice:  # vertices on voxel corners and column centres: every edge case of "inside or on the boundary"
        v = np.round(v * lattice) / lattice
    k = nt // 6
    v[:k, :, rng.integers(0, 3)] = v[:k, :1, rng.integers(0, 3)]  # axis-aligned
    v[k:2 * k, 2] = v[k:2 * k, 0] + (v[k:2 * k, 1] - v[k:2 * k, 0]) * rng.uniform(0, 1, (k, 1))  # slivers
    v[2 * k:2 * k + 5, 1] = v[2 * k:2 * k + 5, 0]  # degenerate
    return np.clip(v, -0.95, 1.95)


@pytest.mark.parametrize("n,nt,size,lattice,side,lo", [
    (8, 700, 0.5, 16, 1.0, 0.0), (32, 3001, 0.06, 64, 1.0, 0.0), (64, 5000, 0.03, 0, 1.0, 0.0),
    (64, 1500, 0.06, 128, 3.0, -1.7), (128, 1025, 0.13, 0, 1.7, 0.3), (256, 900, 0.5, 0, 1.0, 0.0),
    (256, 20000, 0.01, 512, 0.7, 5.1), (128, 64, 0.9, 256, 1.0, 0.0), (32, 1, 0.3, 0, 1.0, 0.0)])
def test_every_size_class(n, nt, size, lattice, side, lo):
    import torch
    import paper_2210_04449_amd.rtsdf as R
    rng = np.random.default_rng(n + nt)
    v = (_triangles(rng, nt, size, lattice) * side + lo).reshape(-1, 3).astype(np.float32)
    f = np.arange(3 * nt, dtype=np.int32).reshape(-1, 3)
    g = R.Grid.make(n, side / n, (lo,) * 3)
    want = oracle.voxelize(v, f, np.full(3, lo, np.float32), np.float32(side / n), n)
    seeds = torch.empty(n ** 3, dtype=torch.int32, device="cuda")
    R.rtsdf_voxelize(torch.from_numpy(v).cuda(), torch.from_numpy(f).cuda(), g, seeds)
    assert np.array_equal(seeds.cpu().numpy(), want)
    assert R.rtsdf_sync_status() == 0
