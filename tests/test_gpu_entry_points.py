"""The queued loop's entry points: rays that start at the subtrees their tile's block can meet trace exactly what rays
that start at the root do (the one-fetch loop), where the choice of subtrees is at its limits: no triangle, one, two,
fewer nodes than entry points, many; tiles of one ray, of partial records, of 768; a block inside, beside and far from
the mesh."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _meshes():
    from synth.scenes import ground_quad, icosphere, random_soup, room_scene
    tri = np.array([[0.2, 0.4, 0.3], [0.7, 0.45, 0.35], [0.4, 0.5, 0.8]], np.float32)
    return {
        "none": (np.zeros((1, 3), np.float32), np.zeros((0, 3), np.int32)),
        "one": (tri, np.array([[0, 1, 2]], np.int32)),
        "two": (lambda m: (m.vertices, m.faces))(ground_quad(0.4)),
        "sphere": (lambda m: (m.vertices, m.faces))(icosphere(2, 0.3, (0.5, 0.5, 0.5))),
        "corner": (lambda m: (m.vertices, m.faces))(icosphere(1, 0.05, (0.06, 0.06, 0.06))),
        "soup": (lambda m: (m.vertices, m.faces))(random_soup(5, 900, 0.0, 1.0, 0.08)),
        "room": (lambda m: (m.vertices, m.faces))(room_scene(3, 24, "low")),
    }


@pytest.mark.parametrize("mesh", ["none", "one", "two", "sphere", "corner", "soup", "room"])
@pytest.mark.parametrize("rays,tile,leaf", [(1, 16, 1), (7, 64, 4), (64, 32, 8)])
def test_entry_points_trace_like_the_root(mesh, rays, tile, leaf):
    import torch
    from paper_2210_04449_amd.pipeline import Pipeline
    v, f = _meshes()[mesh]
    out = {}
    for loop in (3, 4):
        for rebuild in ((False, True) if len(f) > 1 else (False,)):
            d = 30.0 if mesh in ("corner", "two") else 2.0  # nearly every texel selected: blocks far from the mesh
            p = Pipeline(torch.from_numpy(v).cuda(), torch.from_numpy(f).cuda(), 16, 32, 0.5 / 16, d / 16, rays, seed=11,
                         scene_id=2, alpha=0.9, leaf_size=leaf, rebuild=rebuild)
            p.scene.set_tuning(loop=loop, tile_texels=tile)
            for frame in range(2):
                p.step(frame)
            torch.cuda.synchronize()
            out[loop, rebuild] = {k: t.cpu().numpy() for k, t in {**p.state.tensors(), "fine": p.fine_sdf}.items()}
            p.close()
    for (loop, rebuild), got in out.items():
        ref = out[3, rebuild]
        for k in ref:
            assert np.array_equal(got[k], ref[k], equal_nan=True), (mesh, rays, loop, rebuild, k)
