"""Entry points of full-size tiles: up to 62 of them (two mask words), in batches, whose tiles are as large as the ray
count and the tuning allow, and in a single scene on few wavefronts.  The traced state equals the one-fetch loop's, whose
rays start at the root, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS = ("fine_sdf", "u", "hits", "arg_tri", "arg_ray")
RAYS_PER_TILE = 768


def _meshes():
    from synth.scenes import ground_quad, icosphere, random_soup, room_scene
    tri = np.array([[0.2, 0.4, 0.3], [0.7, 0.45, 0.35], [0.4, 0.5, 0.8]], np.float32)
    m = {
        "one": (tri, np.array([[0, 1, 2]], np.int32)),
        "two": ground_quad(0.4),
        "sphere": icosphere(2, 0.3, (0.5, 0.5, 0.5)),
        "corner": icosphere(1, 0.05, (0.06, 0.06, 0.06)),
        "soup": random_soup(5, 3000, 0.0, 1.0, 0.08),
        "overlap": random_soup(6, 1500, 0.0, 1.0, 0.4),  # boxes that nearly all meet: stacks past their LDS part
        "room": room_scene(3, 24, "low"),
    }
    return {k: x if isinstance(x, tuple) else (x.vertices, x.faces) for k, x in m.items()}


def _entries(v, f, leaf, cap):
    """Entry points of a block of 4^3 texels at 32^3 in the middle of the unit cube, by the kernel's rule: nodes whose
    half area over squared distance exceeds 4 are opened from the root on, until `cap` subtrees are open."""
    import torch
    import paper_2210_04449_amd.rtsdf as R
    s = R.Scene(torch.from_numpy(v).cuda(), torch.from_numpy(f).cuda(), leaf_size=leaf)
    boxes, links, _ = s.hierarchy()
    s.close()
    lo, hi = np.full(3, (14 + 0.5) / 32), np.full(3, (17 + 0.5) / 32)
    s2 = 0.25 * 3 * (4 / 32) ** 2
    n, todo = 1, [0]
    while todo:
        node = todo.pop()
        n += 1
        for slot in range(2):
            b, (code, second) = boxes[node, slot].astype(np.float64), links[node, slot]
            if code < 0:
                n -= int(second) == 0  # the empty leaf of a scene of one leaf
                continue
            w = b[3:] - b[:3]
            d = np.maximum(np.maximum(b[:3] - hi, lo - b[3:]), 0.0)
            if (w[0] * w[1] + w[1] * w[2] + w[2] * w[0]) / (d @ d + s2) > 4.0:
                todo.append(int(code))
    return min(cap, n)


@pytest.mark.parametrize("rays,tile,leaf", [(3, 64, 1), (12, 64, 1), (12, 64, 4), (48, 16, 1), (64, 64, 8)])
def test_batches_of_full_tiles(rays, tile, leaf):
    import torch
    import paper_2210_04449_amd.rtsdf as R
    size = min(tile, RAYS_PER_TILE // rays) * rays  # a batch's tiles
    cap = min(62, 14 + size // 16)
    assert size == {3: 192, 12: 768, 48: 768, 64: 768}[rays]
    meshes = _meshes()
    count = {k: _entries(v, f, leaf, cap) for k, (v, f) in meshes.items()}
    if cap == 62 and leaf == 1:
        assert 1 < count["one"] < 32  # (a large triangle's pieces)
        assert count["soup"] == count["overlap"] == 62, count
    descs = [dict(vertices=torch.from_numpy(v).cuda(), faces=torch.from_numpy(f).cuda(), coarse_n=16, fine_n=32,
                  beta=0.5 / 16, d=30.0, rays=rays, alpha=0.9, scene_id=i) for i, (v, f) in enumerate(meshes.values())]
    out = {}
    for loop, depth in ((3, 12), (4, 12), (4, 24)):
        b = R.Batch(descs, seed=11, leaf_size=leaf)
        b.set_tuning(loop=loop, tile_texels=tile, stack_lds=depth)
        for frame in range(2):
            b.step(frame)
        torch.cuda.synchronize()
        out[loop, depth] = [{k: t.cpu().numpy() for k, t in b.tensors(i).items()} for i in range(b.n)]
        b.close()
    for (loop, depth), scenes in out.items():
        for name, got, ref in zip(meshes, scenes, out[3, 12]):
            assert int(got["count"][0]) == 32 ** 3, name  # whole tiles of neighbouring texels, near and far
            for k in KEYS:
                assert np.array_equal(got[k], ref[k], equal_nan=True), (name, loop, depth, k)


@pytest.mark.parametrize("mesh", ["soup", "overlap", "room"])
def test_single_scene_of_full_tiles(mesh):
    import torch
    from paper_2210_04449_amd.pipeline import Pipeline
    v, f = _meshes()[mesh]
    out = {}
    for loop in (3, 4):
        p = Pipeline(torch.from_numpy(v).cuda(), torch.from_numpy(f).cuda(), 32, 64, 0.5 / 32, 30.0, 24, seed=11,
                     alpha=0.9, leaf_size=1)
        p.scene.set_tuning(loop=loop, blocks_per_cu=1, stats=1)
        p.step(0)
        torch.cuda.synchronize()
        ctr = p.trace_ws[8:88].view(torch.int64).cpu().tolist()
        assert ctr[2] == 64 ** 3 * 24 and ctr[6] // 64 == 64 ** 3 * 24 // RAYS_PER_TILE  # rays, tiles
        out[loop] = {k: t.cpu().numpy() for k, t in {**p.state.tensors(), "fine": p.fine_sdf}.items()}
        p.close()
    for k in out[3]:
        assert np.array_equal(out[3][k], out[4][k], equal_nan=True), k
