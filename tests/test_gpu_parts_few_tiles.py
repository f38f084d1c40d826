"""Two-level scenes start a wavefront's next tile early only in launches of enough tiles: few tiles, and tiles of one
wavefront of rays of which there are not two per wavefront, are traced one after another.  The state does not depend on
it, nor on the tile size."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rays", [1, 2, 5])
def test_parts_of_few_tiles(rays):
    import torch
    from paper_2210_04449_amd.pipeline import Pipeline
    from synth.scenes import rigid_parts
    v, f, offs, T = rigid_parts()

    def cu(a):
        return torch.from_numpy(np.ascontiguousarray(a)).cuda()
    out, started = [], []
    for nf, tuning in ((64, dict()), (64, dict(tile_texels=16)), (64, dict(tile_texels=16, blocks_per_cu=1))):
        nc = nf // 2
        p = Pipeline(cu(v), cu(f), nc, nf, 0.5 / nc, 2.0 / nc, rays, seed=5, scene_id=3, alpha=0.9, parts=(offs, cu(T)))
        p.scene.set_tuning(stats=1, **tuning)
        p.step(0)
        torch.cuda.synchronize()
        ctr = p.trace_ws[8:88].view(torch.int64).cpu().tolist()
        assert ctr[2] == p.selected() * rays
        tiles, early = ctr[6] // 64, ctr[8] // 64
        waves = torch.cuda.get_device_properties(0).multi_processor_count * 4 * tuning.get("blocks_per_cu", 6)
        rays_per_tile = -(-p.selected() // tiles) * rays
        started.append(early > 0)
        assert started[-1] == (tiles > waves * (2 if rays_per_tile <= 64 else 1)), (tiles, early, waves)
        out.append({k: t.cpu().numpy() for k, t in {**p.state.tensors(), "fine": p.fine_sdf}.items()})
        p.close()
    assert not started[0] and started[2]
    for o in out[1:]:
        for k in o:
            assert np.array_equal(o[k], out[0][k], equal_nan=True), k
