"""Triangles so large and far that the watertight test's area times distance is past the largest float: rays near their
edges have no finite distance to report and miss; all other rays hit, and every traversal agrees."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _wall(x, width, cells=8):
    """A square across the x axis of 2 cells^2 triangles."""
    a = np.linspace(-width / 2, width / 2, cells + 1)
    v = np.array([(x, y, z) for y in a for z in a], np.float32)
    c = np.arange(cells)
    at = (c[:, None] * (cells + 1) + c).reshape(-1, 1)
    quad = at + np.array([0, 1, cells + 1, cells + 1, 1, cells + 2])
    return v, quad.reshape(-1, 3).astype(np.int32)


@pytest.mark.parametrize("far", [2.0 ** 20, 2.0 ** 65])
def test_closest_hits_of_far_triangles(far):
    import torch
    import paper_2210_04449_amd.rtsdf as R
    v, f = _wall(-far, far / 2)
    rng = np.random.default_rng(5)
    n = 20000
    t = f[rng.integers(0, len(f), n)]
    w = rng.dirichlet((1, 1, 1), n)
    w[::2, 2] = 0.0  # on an edge
    p = np.einsum("nk,nka->na", w / w.sum(1, keepdims=True), v[t].astype(np.float64))
    d = (p / np.linalg.norm(p, axis=1, keepdims=True)).astype(np.float32)
    s = R.Scene(torch.from_numpy(v).cuda(), torch.from_numpy(f).cuda())
    out = [torch.empty(n, device="cuda")] + [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2)]
    R.rtsdf_closest_hits(s, torch.full((n, 3), 0.5, device="cuda"), torch.from_numpy(d).cuda(), *out)
    dist, tri, front = (x.cpu().numpy() for x in out)
    s.close()
    hit = tri >= 0
    assert np.array_equal(np.isfinite(dist), hit) and not (front[~hit] != 0).any()
    assert hit[1::2].mean() > 0.98  # the fast test takes all but the rays next to an edge
    assert far > 2.0 ** 60 or hit.mean() > 0.98
    assert np.abs(dist[hit] / np.linalg.norm(p[hit], axis=1) - 1).max() < 1e-4


@pytest.mark.parametrize("far", [2.0 ** 20, 2.0 ** 65])
def test_traversals_agree_on_far_triangles(far):
    import torch
    from paper_2210_04449_amd.pipeline import Pipeline
    v, f = _wall(-far, far / 2)
    out = []
    for tuning in (dict(loop=0), dict(loop=1), dict(loop=2), dict(loop=3), dict(loop=3, bvh_width=4), dict(loop=4)):
        p = Pipeline(torch.from_numpy(v).cuda(), torch.from_numpy(f).cuda(), 16, 32, 0.5 / 16, 1.0, 16, seed=3)
        p.scene.set_tuning(**tuning)
        p.coarse_sdf.fill_(1.0)
        p.mask.fill_(1)
        p.queue.copy_(torch.arange(32 ** 3, dtype=torch.int32))
        p.count.fill_(32 ** 3)
        p.trace(0)
        torch.cuda.synchronize()
        out.append({k: t.cpu().numpy() for k, t in {**p.state.tensors(), "fine": p.fine_sdf}.items()})
        p.close()
    assert (out[0]["arg_tri"] >= 0).mean() > 0.1
    for o in out[1:]:
        for k in o:
            assert np.array_equal(o[k], out[0][k], equal_nan=True), k
