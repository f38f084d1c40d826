"""Boxes of rebuilt and refitted hierarchies where the passes over 1,024 references meet their borders: a box too small
loses hits, so the closest hits must be, bit for bit, those of a hierarchy built on the host."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt", [2, 3, 63, 1023, 1024, 1025, 2047, 2049, 5000, 70000])
@pytest.mark.parametrize("leaf", [1, 4, 8])
def test_boxes_at_chunk_borders(nt, leaf):
    import torch
    import paper_2210_04449_amd.rtsdf as R
    from synth.scenes import random_soup
    m = random_soup(9, nt, 0.0, 1.0, 0.3 / nt ** 0.4)
    rng = np.random.default_rng(nt)
    n = 20000
    c = m.vertices[m.faces[rng.integers(0, nt, n)]].mean(1)  # towards the triangles
    o = rng.uniform(-0.2, 1.2, (n, 3)).astype(np.float32)
    w = (c - o).astype(np.float32)
    o, w = torch.from_numpy(o).cuda(), torch.from_numpy(w).cuda()
    v, f = torch.from_numpy(m.vertices).cuda(), torch.from_numpy(m.faces).cuda()
    moved = (v * 0.9 + 0.05 * torch.sin(7.0 * v.flip(1))).contiguous()

    def hits(s):
        out = [torch.empty(n, device="cuda")] + [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2)]
        R.rtsdf_closest_hits(s, o, w, *out)
        torch.cuda.synchronize()
        return out
    s = R.Scene(v.clone(), f, leaf_size=leaf)
    s.enable_rebuild()
    for verts, update in ((v, s.rebuild), (moved, s.rebuild), (v, s.refit), (moved, s.refit)):
        update(verts)
        got = hits(s)
        ref = R.Scene(verts, f, leaf_size=leaf)
        want = hits(ref)
        for x, y in zip(got, want):
            assert torch.equal(x.view(torch.int32), y.view(torch.int32))
        ref.close()
        if verts is v:
            assert int((want[1] >= 0).sum()) > n // 2
    s.close()
