"""Closest hits and point distances of many queries, which go through a short traversal stack first and through the full
one where that overflows: each query's result equals, bit for bit, what it gets in a call of few queries (the full
stack).  Built and rebuilt hierarchies (32 and 64 stack entries), sizes on both sides of the line, points in a sphere's
centre and rays along its shell (stacks that overflow), infinities and NaN."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scenes():
    import torch
    import paper_2210_04449_amd.rtsdf as R
    from synth.scenes import icosphere, room_scene
    ball, room = icosphere(6, 0.3, (0.5, 0.5, 0.5)), room_scene(2, 60, "mid")
    out = {}
    for name, m in (("ball", ball), ("room", room)):
        for rebuilt in (False, True):
            v, f = torch.from_numpy(m.vertices).cuda(), torch.from_numpy(m.faces).cuda()
            s = R.Scene(v, f)
            if rebuilt:
                s.enable_rebuild()
                s.rebuild(v)
            out[name, rebuilt] = s
    yield R, out
    for s in out.values():
        s.close()


def _points(n, seed):
    import torch
    rng = np.random.default_rng(seed)
    p = rng.uniform(-0.1, 1.1, (n, 3)).astype(np.float32)
    p[::7] = 0.5 + rng.normal(scale=1e-3, size=p[::7].shape)  # the ball's centre: all triangles equally near
    p[5], p[70], p[n - 1] = np.inf, np.nan, (np.nan, 0.5, 0.5)
    return torch.from_numpy(p).cuda()


@pytest.mark.parametrize("name,rebuilt", [("ball", False), ("ball", True), ("room", False), ("room", True)])
@pytest.mark.parametrize("over", [0, 1, 64, 5003])
def test_distance_of_many_points(scenes, name, rebuilt, over):
    import torch
    R, S = scenes
    sc = S[name, rebuilt]
    n = (196608 if rebuilt else 393216) + over  # the last size of the full stack alone, and above
    p = _points(n, 3 + over)
    d, t = torch.empty(n, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
    d1, t1 = torch.empty_like(d), torch.empty_like(t)
    R.rtsdf_point_distance(sc, p, d, t)
    for a in range(0, n, 50000):
        b = min(n, a + 50000)
        R.rtsdf_point_distance(sc, p[a:b].contiguous(), d1[a:b], t1[a:b])
    assert torch.equal(d.view(torch.int32), d1.view(torch.int32)) and torch.equal(t, t1)
    d2 = torch.empty_like(d)
    R.rtsdf_point_distance(sc, p, d2)  # without the triangles
    assert torch.equal(d.view(torch.int32), d2.view(torch.int32))


@pytest.mark.parametrize("name,rebuilt", [("ball", False), ("ball", True), ("room", True)])
def test_distance_of_many_texels(scenes, name, rebuilt):
    import torch
    R, S = scenes
    sc, g = S[name, rebuilt], R.Grid.make(80)
    n = 80 ** 3
    d, t = torch.empty(n, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
    R.rtsdf_texel_distance(sc, g, None, d, t)
    q = torch.randperm(n, generator=torch.Generator().manual_seed(4)).int().cuda()
    d1, t1 = torch.empty_like(d), torch.empty_like(t)
    R.rtsdf_texel_distance(sc, g, q, d1, t1)
    assert torch.equal(d[q.long()], d1) and torch.equal(t[q.long()], t1)
    for a in range(0, n, 64000):
        c = q[a:a + 64000].contiguous()
        R.rtsdf_texel_distance(sc, g, c, d1[:len(c)], t1[:len(c)])
        assert torch.equal(d[c.long()], d1[:len(c)]) and torch.equal(t[c.long()], t1[:len(c)])


@pytest.mark.parametrize("name,rebuilt", [("ball", False), ("ball", True), ("room", False), ("room", True)])
@pytest.mark.parametrize("over", [0, 1, 64, 5003])
def test_closest_hits_of_many_rays(scenes, name, rebuilt, over):
    import torch
    R, S = scenes
    sc = S[name, rebuilt]
    n = (131072 if rebuilt else 262144) + over
    rng = np.random.default_rng(8 + over)
    o = rng.uniform(-0.1, 1.1, (n, 3)).astype(np.float32)
    w = rng.normal(size=(n, 3)).astype(np.float32)
    k = rng.normal(size=o[::5].shape)  # along the ball's shell, inside it
    k /= np.linalg.norm(k, axis=1, keepdims=True)
    o[::5] = 0.5 + 0.2999 * k
    w[::5] = np.cross(k, rng.normal(size=k.shape))
    w[1::9, 1] = 0.0
    w[3], o[12], w[n - 1] = 0.0, np.nan, (np.nan, 0.0, 1.0)
    o, w = torch.from_numpy(o).cuda(), torch.from_numpy(w).cuda()

    def out(m):
        return [torch.empty(m, device="cuda")] + [torch.empty(m, dtype=torch.int32, device="cuda") for _ in range(2)]
    many = out(n)
    R.rtsdf_closest_hits(sc, o, w, *many)
    for a in range(0, n, 50000):
        oo, ww = o[a:a + 50000].contiguous(), w[a:a + 50000].contiguous()
        few = out(len(oo))
        R.rtsdf_closest_hits(sc, oo, ww, *few)
        for x, y in zip(many, few):
            assert torch.equal(x[a:a + 50000].view(torch.int32), y.view(torch.int32))
    assert int((many[1] >= 0).sum()) > n // 20
