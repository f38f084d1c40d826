"""Selection and trilinear sampling on grids of 64^3 and more (16 bytes per lane, Morton blocks listed in LDS) against
the oracle, bit for bit: every texel ratio the kernels branch on, one and two levels of the block scan, fields with
infinities, NaN and the threshold itself, empty and full selections, full queues, arrays off 16-byte alignment."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _off(t, shift):
    """A copy of t whose storage starts `shift` elements past a 16-byte boundary."""
    import torch
    buf = torch.empty(t.numel() + 4, dtype=t.dtype, device="cuda")
    v = buf[shift:shift + t.numel()]
    v.copy_(t)
    return v


@pytest.mark.parametrize("n,r,fill,cap,shift", [(64, 1, 0.3, None, 0), (64, 2, 0.3, None, 0), (64, 4, 0.05, None, 0),
                                                (64, 8, 0.01, 1001, 0), (128, 2, 0.2, None, 0), (256, 1, 0.1, None, 0),
                                                (256, 2, 0.02, 70001, 0), (64, 2, 0.0, None, 0), (64, 2, 1.0, None, 0),
                                                (64, 2, 0.3, None, 1)])
def test_point_selection(n, r, fill, cap, shift):
    import torch
    import paper_2210_04449_amd.rtsdf as R
    rng = np.random.default_rng(n + r)
    d2 = rng.integers(0, 100, n ** 3).astype(np.int32)
    K = int(100 * fill) - 1
    d = float(np.float32(np.sqrt(max(K, 0) + 0.5) / n)) if fill else -1.0
    assert oracle.select_threshold(np.float32(1 / n), 0.0, d) == K
    want_mask, want = oracle.select(n, d2, n * r, K)
    mask = torch.full(((n * r) ** 3,), 7, dtype=torch.uint8, device="cuda")
    queue = torch.full((len(want) + 1 if cap is None else cap,), -5, dtype=torch.int32, device="cuda")
    count = torch.empty(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(R.rtsdf_select_workspace_size(n), dtype=torch.uint8, device="cuda")
    R.rtsdf_select(R.Grid.make(n), _off(torch.from_numpy(d2), shift), R.Grid.make(n * r), 0.0, d, mask, queue, count, ws)
    full = R.rtsdf_sync_status() == R.ERR_QUEUE_FULL
    assert full == (cap is not None and len(want) > cap) and int(count.item()) == len(want)
    assert np.array_equal(mask.cpu().numpy(), want_mask)
    got = queue.cpu().numpy()
    k = min(len(want), len(got))
    assert np.array_equal(got[:k], want[:k]) and (got[k:] == -5).all()


@pytest.mark.parametrize("n,d,shift", [(64, 0.25, 0), (128, 0.1, 0), (256, 0.5, 0), (64, -1.0, 0), (64, 2.0, 0),
                                       (64, 0.25, 3)])
def test_field_selection(n, d, shift):
    import torch
    import paper_2210_04449_amd.rtsdf as R
    rng = np.random.default_rng(n)
    f = rng.random(n ** 3, dtype=np.float32)
    f[rng.integers(0, n ** 3, 500)] = np.float32(d)
    f[rng.integers(0, n ** 3, 500)] = np.inf
    f[rng.integers(0, n ** 3, 500)] = np.nan
    want_mask, want = oracle.select_field(n, f, d)
    mask = torch.empty(n ** 3, dtype=torch.uint8, device="cuda")
    queue = torch.full((n ** 3,), -5, dtype=torch.int32, device="cuda")
    count = torch.empty(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(R.rtsdf_select_workspace_size(n), dtype=torch.uint8, device="cuda")
    R.rtsdf_select_field(R.Grid.make(n), _off(torch.from_numpy(f), shift), d, mask, queue, count, ws)
    assert int(count.item()) == len(want) and np.array_equal(mask.cpu().numpy(), want_mask)
    got = queue.cpu().numpy()
    assert np.array_equal(got[:len(want)], want) and (got[len(want):] == -5).all()


@pytest.mark.parametrize("nc,r,shift", [(8, 2, 0), (16, 2, 0), (32, 4, 0), (8, 8, 0), (8, 16, 0), (4, 2, 0), (2, 8, 0),
                                        (1, 16, 0), (16, 1, 0), (64, 2, 0), (16, 2, 2)])
def test_trilinear_rows(nc, r, shift):
    import torch
    import paper_2210_04449_amd.rtsdf as R
    rng = np.random.default_rng(nc + r)
    for holes in (0, 1, nc):
        c = rng.normal(size=nc ** 3).astype(np.float32)
        c[rng.integers(0, nc ** 3, holes)] = np.inf
        want = oracle.coarse_trilinear(nc, c, nc * r)
        out = _off(torch.full(((nc * r) ** 3,), 7.0), shift)
        R.rtsdf_coarse_trilinear(R.Grid.make(nc), torch.from_numpy(c).cuda(), R.Grid.make(nc * r), out)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), (nc, r, holes)
