"""Performance cases of the library: what a user's program has it do, through its public entry points.

``listed()`` names the cases, ``draw(rng)`` gives further ones of the same ranges, ``prepare`` makes what a program
holds before the call (meshes, pipelines, query points), ``run`` is one pass, ``work`` the bytes and operations a
pass cannot do without, and ``exact`` the same outputs from plain torch / numpy in 64 bits where that is feasible.

A case's ``op``:

update    one SDF update of a scene (voxelize, jump flooding, selection, tracing with temporal accumulation), the
          frame index advancing from pass to pass; ``motion``: "static", "vertices" (a new vertex set every update),
          "parts" (rigid parts moved by transforms); ``graph``: replayed as one captured graph
batch     one update of many scenes at once
diff      the differentiable SDF: forward over some frames, a loss, backward to the vertex positions
coarse    the coarse field alone: voxelization and jump flooding
select    the texels to trace from a coarse field, point-sampled or trilinear
shadow    soft-shadow visibility of shading points from a fine SDF
pick      closest hits of arbitrary rays against moved geometry (device rebuild, then the rays)
distance  exact distance from the selected texels to the mesh
"""
from __future__ import annotations

import functools
import math
import random

import numpy as np
import torch

import paper_2210_04449_amd.rtsdf as R
from paper_2210_04449_amd.autograd import fine_sdf
from paper_2210_04449_amd.pipeline import Pipeline

DEV = "cuda"


def listed():
    return [
        # the smallest call: a few hundred triangles, every launch and its latency counts
        dict(name="tiny_update", op="update", scene="sphere", level=2, prims=1, nc=32, nf=64, beta=0.5, d=2.0, rays=4,
             alpha=1.0, sampling="point", sign="vote", motion="static", graph=False),
        # an ordinary scene in a real-time loop: one captured graph replayed per frame, thin surfaces as shells
        dict(name="graph_update", op="update", scene="room", level=2, prims=60, nc=64, nf=128, beta=0.5, d=2.0, rays=7,
             alpha=0.9, sampling="trilinear", sign="shell", motion="static", graph=True),
        # the room-scale scene of the benchmark
        dict(name="room_update", op="update", scene="room", level=3, prims=300, nc=128, nf=256, beta=0.5, d=3.0,
             rays=16, alpha=1.0, sampling="point", sign="vote", motion="static", graph=False),
        # the largest: about a million triangles, a fifth of them moving, a new vertex set every update
        dict(name="moving_update", op="update", scene="room", level=4, prims=366, nc=256, nf=512, beta=0.5, d=3.0,
             rays=8, alpha=0.9, sampling="point", sign="vote", motion="vertices", graph=False),
        # rigid parts moved by transforms (two-level scene)
        dict(name="parts_update", op="update", scene="room", level=3, prims=120, nc=128, nf=256, beta=0.5, d=2.0,
             rays=5, alpha=0.9, sampling="point", sign="vote", motion="parts", graph=False),
        # many scenes of uneven size per launch
        dict(name="batch_step", op="batch", scenes=12, tmin=1000, tmax=60000, ncmax=128, beta=0.5, d=2.0, rays=8,
             alpha=1.0),
        # fitting a mesh: forward over frames and backward to the vertices
        dict(name="diff_step", op="diff", freq=22, nc=64, nf=128, beta=0.5, d=2.0, rays=32, frames=6),
        # the coarse field of the largest grid
        dict(name="coarse_field", op="coarse", prims=366, level=4, nc=256, beta=0.5, variant="jfa"),
        # choosing the texels to trace from an interpolated coarse field, at the moving scene's size
        dict(name="select_texels", op="select", mode="trilinear", balls=60, nc=256, nf=512, beta=0.5, d=2.0),
        # the consumer: one 1080p frame of shading points, triangulated penumbra, jittered starts
        dict(name="shadow_frame", op="shadow", balls=120, nf=256, points=1920 * 1080, steps=96, penumbra=1,
             jitter=True),
        # picking rays and visibility queries against geometry that moves every frame
        dict(name="pick_rays", op="pick", prims=300, level=3, rays=300007),
        # how far the traced values are from the mesh: exact distances at the selected texels
        dict(name="distance_texels", op="distance", prims=300, level=3, nc=128, nf=256, beta=0.5, d=2.0, most=2000003),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    op = rng.choice(["update", "update", "update", "batch", "diff", "coarse", "select", "shadow", "pick", "distance"])
    if op == "update":
        nc = rng.choice([16, 32, 64, 128])
        nf = min(256, nc * rng.choice([1, 2, 2, 4]))
        most = max(1, min(64, int(1.2e8 / nf ** 3)))  # at most about the room's rays
        motion = rng.choice(["static", "static", "vertices", "parts"])
        return dict(op=op, scene="room", level=rng.choice([1, 2, 3]), prims=_log_int(rng, 3, 300), nc=nc, nf=nf,
                    beta=rng.choice([0.0, 0.5, 1.0]), d=rng.choice([1.0, 1.7, 2.0, 3.0]),
                    rays=_log_int(rng, 1, most), alpha=rng.choice([1.0, 0.9, 0.75]),
                    sampling=rng.choice(["point", "point", "trilinear"]), sign=rng.choice(["vote", "vote", "shell"]),
                    motion=motion, graph=rng.choice([False, False, True]))
    if op == "batch":
        return dict(op=op, scenes=rng.randint(2, 16), tmin=rng.choice([200, 1000]), tmax=_log_int(rng, 3000, 60000),
                    ncmax=rng.choice([32, 64, 128]), beta=0.5, d=rng.choice([1.5, 2.0]), rays=rng.randint(3, 12),
                    alpha=rng.choice([1.0, 0.9]))
    if op == "diff":
        nc = rng.choice([32, 64])
        return dict(op=op, freq=rng.randint(5, 30), nc=nc, nf=2 * nc, beta=0.5, d=2.0, rays=rng.randint(5, 48),
                    frames=rng.randint(2, 6))
    if op == "coarse":
        return dict(op=op, prims=_log_int(rng, 3, 366), level=rng.choice([1, 2, 3, 4]),
                    nc=rng.choice([32, 64, 128, 256]), beta=rng.choice([0.0, 0.5]),
                    variant=rng.choice(["jfa", "jfa", "jfa+1", "jfa+2", "1+jfa"]))
    if op == "select":
        nc = rng.choice([32, 64, 128, 256])
        return dict(op=op, mode=rng.choice(["point", "trilinear"]), balls=_log_int(rng, 2, 100), nc=nc,
                    nf=min(512, nc * rng.choice([1, 2, 4])), beta=rng.choice([0.0, 0.5]), d=rng.choice([1.0, 2.0, 3.3]))
    if op == "shadow":
        return dict(op=op, balls=_log_int(rng, 2, 150), nf=rng.choice([64, 128, 256]),
                    points=_log_int(rng, 1001, 2100000), steps=rng.choice([32, 64, 96]), penumbra=rng.choice([0, 1]),
                    jitter=rng.choice([False, True]))
    if op == "pick":
        return dict(op=op, prims=_log_int(rng, 3, 300), level=rng.choice([1, 2, 3]), rays=_log_int(rng, 501, 500000))
    nc = rng.choice([32, 64, 128])
    return dict(op=op, prims=_log_int(rng, 3, 300), level=rng.choice([1, 2, 3]), nc=nc, nf=2 * nc, beta=0.5,
                d=rng.choice([1.0, 2.0]), most=_log_int(rng, 5001, 2000003))


# ------------------------------------------------------------------ meshes


@functools.lru_cache(maxsize=None)
def _icosphere(level):
    phi = (1.0 + math.sqrt(5.0)) / 2.0
    v = np.array([[-1, phi, 0], [1, phi, 0], [-1, -phi, 0], [1, -phi, 0], [0, -1, phi], [0, 1, phi], [0, -1, -phi],
                  [0, 1, -phi], [phi, 0, -1], [phi, 0, 1], [-phi, 0, -1], [-phi, 0, 1]], np.float64)
    f = np.array([[0, 11, 5], [0, 5, 1], [0, 1, 7], [0, 7, 10], [0, 10, 11], [1, 5, 9], [5, 11, 4], [11, 10, 2],
                  [10, 7, 6], [7, 1, 8], [3, 9, 4], [3, 4, 2], [3, 2, 6], [3, 6, 8], [3, 8, 9], [4, 9, 5], [2, 4, 11],
                  [6, 2, 10], [8, 6, 7], [9, 8, 1]], np.int64)
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    for _ in range(level):
        e = np.sort(np.concatenate([f[:, [0, 1]], f[:, [1, 2]], f[:, [2, 0]]]), axis=1)
        pairs, which = np.unique(e, axis=0, return_inverse=True)
        mid = v[pairs[:, 0]] + v[pairs[:, 1]]
        m = len(v) + which.reshape(3, -1)
        v = np.concatenate([v, mid / np.linalg.norm(mid, axis=1, keepdims=True)])
        ab, bc, ca = m
        f = np.concatenate([np.stack(t, 1) for t in ((f[:, 0], ab, ca), (f[:, 1], bc, ab), (f[:, 2], ca, bc),
                                                     (ab, bc, ca))])
    return v, f


@functools.lru_cache(maxsize=None)
def _box():
    v = np.array([[x, y, z] for z in (-1, 1) for y in (-1, 1) for x in (-1, 1)], np.float64)
    q = [[0, 2, 3, 1], [4, 5, 7, 6], [0, 1, 5, 4], [2, 6, 7, 3], [0, 4, 6, 2], [1, 3, 7, 5]]
    return v, np.array([t for a, b, c, d in q for t in ([a, b, c], [a, c, d])], np.int64)


@functools.lru_cache(maxsize=None)
def _torus(nu, nv):
    u, w = np.meshgrid(2 * np.pi * np.arange(nu) / nu, 2 * np.pi * np.arange(nv) / nv, indexing="ij")
    r = 1.0 + 0.3 * np.cos(w)
    v = np.stack([r * np.cos(u), 0.3 * np.sin(w), r * np.sin(u)], -1).reshape(-1, 3) / 1.3
    i, j = np.meshgrid(np.arange(nu), np.arange(nv), indexing="ij")
    a, b = i * nv + j, (i + 1) % nu * nv + j
    c, d = (i + 1) % nu * nv + (j + 1) % nv, i * nv + (j + 1) % nv
    return v, np.concatenate([np.stack([a, c, b], -1).reshape(-1, 3), np.stack([a, d, c], -1).reshape(-1, 3)])


def _primitive(kind, level):
    if kind == 0:
        return _box()[0] / math.sqrt(3.0), _box()[1]
    return _icosphere(level) if kind == 1 else _torus(16 << (level > 2) << (level > 3), 8 + 4 * (level > 2) + 12 * (level > 3))


def _rotation(rng):
    q = rng.normal(size=4)
    a, b, c, d = q / np.linalg.norm(q)
    return np.array([[a * a + b * b - c * c - d * d, 2 * (b * c - a * d), 2 * (b * d + a * c)],
                     [2 * (b * c + a * d), a * a - b * b + c * c - d * d, 2 * (c * d - a * b)],
                     [2 * (b * d - a * c), 2 * (c * d + a * b), a * a - b * b - c * c + d * d]])


def _turn(axis, angle):
    x, y, z = axis / np.linalg.norm(axis)
    k = np.array([[0, -z, y], [z, 0, -x], [-y, x, 0]])
    return np.eye(3) + math.sin(angle) * k + (1 - math.cos(angle)) * (k @ k)


class _Scene:
    """The unit room's walls and `prims` random boxes, spheres and tori, a fifth of which move rigidly (the last
    ones, so that they are parts of their own); or one sphere over a ground quad."""

    def __init__(self, scene, prims, level, seed):
        rng = np.random.default_rng(seed)
        if scene == "sphere":
            v, f = _icosphere(level)
            g = np.array([[0, 0.15, 0], [1, 0.15, 0], [1, 0.15, 1], [0, 0.15, 1]])
            v = v * rng.uniform(0.28, 0.3) + rng.uniform(0.48, 0.52, 3)
            self.parts = [(np.concatenate([v, g]), np.concatenate([f, np.array([[0, 2, 1], [0, 3, 2]]) + len(v)]))]
            self.moving = []
            return
        wall, wf = _box()
        self.parts, self.moving = [((wall + 1) / 2, wf[:, ::-1])], []
        for i in range(prims):
            s = math.exp(rng.uniform(math.log(0.02), math.log(0.2)))
            v, f = _primitive(int(rng.integers(0, 3)), level)
            c = rng.uniform(s + 0.05, 0.95 - s, 3) if s < 0.44 else np.full(3, 0.5)
            part = ((v * s) @ _rotation(rng).T + c, f)
            how = (c, rng.normal(size=3), rng.uniform(0.02, 0.1), rng.uniform(0, 0.05), rng.uniform(0, 2 * math.pi))
            if i >= prims - max(1, prims // 5):
                self.moving.append((part, how))
            else:
                self.parts.append(part)

    @staticmethod
    def _at(how, frame):
        """Rotation and translation of a moving part at `frame`; the identity at frame 0."""
        c, axis, rate, radius, phase = how
        rot = _turn(axis, rate * frame)
        ring = lambda p: radius * np.array([math.cos(p), 0.0, math.sin(p)])  # noqa: E731
        return rot, c - rot @ c + ring(phase + 0.05 * frame) - ring(phase)

    def mesh(self):
        vs, fs, off = [], [], 0
        for v, f in self.parts + [m[0] for m in self.moving]:
            vs.append(v)
            fs.append(f + off)
            off += len(v)
        return (torch.from_numpy(np.concatenate(vs).astype(np.float32)).to(DEV),
                torch.from_numpy(np.concatenate(fs).astype(np.int32)).to(DEV))

    def vertices(self, frame):
        v = [p[0] for p in self.parts]
        for (x, _), how in self.moving:
            rot, t = self._at(how, frame)
            v.append(x @ rot.T + t)
        return torch.from_numpy(np.concatenate(v).astype(np.float32)).to(DEV)

    def offsets(self):
        offs = [0, sum(len(f) for _, f in self.parts)]
        for (_, f), _ in self.moving:
            offs.append(offs[-1] + len(f))
        return offs

    def transforms(self, frame):
        rows = [np.eye(3, 4)]
        for _, how in self.moving:
            rot, t = self._at(how, frame)
            rows.append(np.concatenate([rot, t[:, None]], 1))
        return torch.from_numpy(np.stack(rows).reshape(len(rows), 12).astype(np.float32)).to(DEV)


def _star(freq, seed):
    """A latitude-longitude sphere of about 20 freq^2 triangles with a smooth radial perturbation."""
    rng = np.random.default_rng(seed)
    nu, nv = max(4, int(freq * 4.5)), max(3, int(freq * 2.2))
    th = np.pi * np.arange(1, nv) / nv
    ph = 2 * np.pi * np.arange(nu) / nu
    ring = np.stack([np.sin(th)[:, None] * np.cos(ph), np.cos(th)[:, None] + 0 * ph, np.sin(th)[:, None] * np.sin(ph)],
                    -1).reshape(-1, 3)
    v = np.concatenate([[[0, 1, 0]], ring, [[0, -1, 0]]])
    f, last = [], len(v) - 1
    for j in range(nu):
        k = (j + 1) % nu
        f += [[0, 1 + k, 1 + j], [last, last - nu + j, last - nu + k]]
        for i in range(nv - 2):
            a, b = 1 + i * nu + j, 1 + i * nu + k
            f += [[a, b, a + nu], [b, b + nu, a + nu]]
    w = rng.normal(size=(5, 3))
    bump = np.sin((v @ w.T) * 2.5 + rng.uniform(0, 2 * np.pi, 5)).sum(1)
    r = 0.3 * (1 + 0.05 * bump / np.abs(bump).max())
    return (torch.from_numpy((v * r[:, None] + 0.5).astype(np.float32)).to(DEV),
            torch.from_numpy(np.array(f, np.int32)).to(DEV))


def _balls(n, k, seed):
    """[k^3] float64 distance at the cell centres of a k^3 grid to `n` random spheres and the room's walls (x runs
    fastest)."""
    rng = np.random.default_rng(seed)
    a = (torch.arange(k, dtype=torch.float32, device=DEV) + 0.5) / k
    wall = torch.minimum(a, 1 - a)
    out = torch.minimum(torch.minimum(wall[:, None, None], wall[None, :, None]), wall[None, None, :]).clone()
    for _ in range(n):
        s = math.exp(rng.uniform(math.log(0.02), math.log(0.15)))
        x, y, z = rng.uniform(s, 1 - s, 3)
        d = ((a - z) ** 2)[:, None, None] + ((a - y) ** 2)[None, :, None] + ((a - x) ** 2)[None, None, :]
        out = torch.minimum(out, d.sqrt_().sub_(s))
    return out.reshape(-1)


# ----------------------------------------------------------------- prepare


def _beta_d(case):
    return float(np.float32(case["beta"] / case["nc"])), float(np.float32(case["d"] / case["nc"]))


def prepare(case, seed):
    op = case["op"]
    s = {"case": case, "frame": 0}
    if op == "update":
        sc = _Scene(case["scene"], case["prims"], case["level"], seed)
        v, f = sc.mesh()
        beta, d = _beta_d(case)
        kw = dict(seed=seed & 0xFFFF, scene_id=seed & 7, alpha=case["alpha"], sampling=case["sampling"],
                  sign_policy=case["sign"], shell=0.5 / case["nf"] if case["sign"] == "shell" else 0.0)
        if case["motion"] == "parts":
            kw["parts"] = (sc.offsets(), sc.transforms(0))
        p = s["p"] = Pipeline(v, f, case["nc"], case["nf"], beta, d, case["rays"], **kw)
        if case["motion"] == "vertices":
            s["moves"] = [sc.vertices(k + 1) for k in range(4)]
        elif case["motion"] == "parts":
            s["moves"] = [sc.transforms(k + 1) for k in range(4)]
        if case["graph"]:
            s["graph"] = p.make_graph(first_frame=0, refit=case["motion"] != "static")
    elif op == "batch":
        sizes = np.random.default_rng(case["scenes"])  # grids and triangle budgets are the case's, meshes the seed's
        scenes = []
        for i in range(case["scenes"]):
            target = math.exp(sizes.uniform(math.log(case["tmin"]), math.log(case["tmax"])))
            nc = int(sizes.choice([n for n in (32, 64, 128) if n <= case["ncmax"]]))
            level = 2 if target < 10000 else 3
            v, f = _Scene("room", max(1, int(target / (170 if level == 2 else 680))), level, [seed, i]).mesh()
            scenes.append(dict(vertices=v, faces=f, coarse_n=nc, fine_n=2 * nc, beta=case["beta"] / nc,
                               d=case["d"] / nc, rays=case["rays"], alpha=case["alpha"], scene_id=i))
        s["b"] = R.Batch(scenes, seed=seed & 0xFFFF)
        s["out"] = [{k: torch.empty(x["fine_n"] ** 3, dtype=t, device=DEV)
                     for k, t in (("fine_sdf", torch.float32), ("hits", torch.int32), ("arg_tri", torch.int32))}
                    for x in scenes]
    elif op == "diff":
        v, f = _star(case["freq"], seed)
        beta, d = _beta_d(case)
        s["v"] = v
        s["p"] = Pipeline(v, f, case["nc"], case["nf"], beta, d, case["rays"], seed=seed & 0xFFFF)
        nf = case["nf"]
        a = (torch.arange(nf, device=DEV) + 0.5) / nf - 0.5
        s["target"] = ((a ** 2)[:, None, None] + (a ** 2)[None, :, None] + (a ** 2)).sqrt().reshape(-1) - 0.3
    elif op == "coarse":
        s["v"], s["f"] = _Scene("room", case["prims"], case["level"], seed).mesh()
        n = case["nc"]
        for k in ("seeds", "scratch", "dist2"):
            s[k] = torch.empty(n ** 3, dtype=torch.int32, device=DEV)
        s["sdf"] = torch.empty(n ** 3, dtype=torch.float32, device=DEV)
    elif op == "select":
        nc, nf = case["nc"], case["nf"]
        dist = _balls(case["balls"], nc, seed).abs_().mul_(nc).round_()  # whole voxels: an unsigned coarse field
        s["dist2"] = (dist * dist).to(torch.int32)
        s["c"] = (dist / nc - case["beta"] / nc).contiguous()
        s["fine_c"] = torch.empty(nf ** 3, dtype=torch.float32, device=DEV)
        s["mask"] = torch.empty(nf ** 3, dtype=torch.uint8, device=DEV)
        s["queue"] = torch.zeros(nf ** 3, dtype=torch.int32, device=DEV)
        s["count"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        s["ws"] = torch.empty(R.rtsdf_select_workspace_size(nf), dtype=torch.uint8, device=DEV)
    elif op == "shadow":
        nf, g = case["nf"], torch.Generator(device=DEV).manual_seed(seed)
        s["sdf"] = _balls(case["balls"], nf, seed)
        near = torch.nonzero((s["sdf"] >= 1 / nf) & (s["sdf"] <= 3 / nf)).flatten()
        # in texel order, as the shading points of one frame are coherent
        pick = near[torch.randint(0, near.numel(), (case["points"],), device=DEV, generator=g)].sort().values
        ijk = torch.stack([pick % nf, pick // nf % nf, pick // (nf * nf)], 1).float()
        s["pts"] = ((ijk + torch.rand(ijk.shape, device=DEV, generator=g)) / nf).contiguous()
        s["jitter"] = torch.rand(case["points"], device=DEV, generator=g) if case["jitter"] else None
        s["vis"] = torch.empty(case["points"], dtype=torch.float32, device=DEV)
    elif op == "pick":
        sc = _Scene("room", case["prims"], case["level"], seed)
        v, f = sc.mesh()
        s["f"], s["moves"] = f, [sc.vertices(k + 1) for k in range(2)]
        s["scene"] = R.Scene(v, f)
        s["scene"].enable_rebuild()
        n, g = case["rays"], torch.Generator(device=DEV).manual_seed(seed)
        s["o"] = torch.rand(n, 3, device=DEV, generator=g) * 0.98 + 0.01
        s["w"] = torch.nn.functional.normalize(torch.randn(n, 3, device=DEV, generator=g), dim=1)
        s["t"] = torch.empty(n, dtype=torch.float32, device=DEV)
        s["tri"], s["front"] = (torch.empty(n, dtype=torch.int32, device=DEV) for _ in range(2))
    elif op == "distance":
        v, f = _Scene("room", case["prims"], case["level"], seed).mesh()
        beta, d = _beta_d(case)
        s["p"] = p = Pipeline(v, f, case["nc"], case["nf"], beta, d, 1)
        p.voxelize()
        p.jfa()
        p.select()
        n = p.selected()
        s["q"] = p.queue[:min(n, case["most"])].clone()
        s["dist"] = torch.empty(s["q"].numel(), dtype=torch.float32, device=DEV)
        s["tri"] = torch.empty(s["q"].numel(), dtype=torch.int32, device=DEV)
    else:
        raise ValueError(op)
    return s


# --------------------------------------------------------------------- run


def _state(p):
    out = dict(u=p.state.u, hits=p.state.hits, arg_tri=p.state.arg_tri, arg_ray=p.state.arg_ray, fine_sdf=p.fine_sdf,
               mask=p.mask, count=p.count, coarse_sdf=p.coarse_sdf, seeds=p.seeds)
    return out if p.fine_c is None else dict(out, fine_c=p.fine_c)


_LIGHT = tuple(x / math.sqrt(0.3 ** 2 + 0.9 ** 2 + 0.2 ** 2) for x in (0.3, 0.9, 0.2))


def run(s):
    case = s["case"]
    op = case["op"]
    k = s["frame"]
    s["frame"] = k + 1
    if op == "update":
        p = s["p"]
        move = s["moves"][k % 4] if "moves" in s else None
        if case["graph"]:
            if move is not None:
                (p.transforms if p.parts else p.vertices).copy_(move)
            s["graph"].launch()
        else:
            if move is not None:
                (p.set_transforms if p.parts else p.set_vertices)(move)
            p.step(k)
        return _state(p)
    if op == "batch":
        b = s["b"]
        b.step(k)
        stream = torch.cuda.current_stream().cuda_stream
        for i, out in enumerate(s["out"]):
            view = b.view(i)
            for key, src in (("fine_sdf", view.fine_sdf), ("hits", view.state.hits), ("arg_tri", view.state.arg_tri)):
                R.lib().rtsdf_copy(out[key].data_ptr(), src, out[key].numel() * 4, stream)
        return s["out"]
    if op == "diff":
        v = s["v"].detach().requires_grad_(True)
        fine = fine_sdf(v, s["p"], range(case["frames"]))
        loss = torch.where(torch.isfinite(fine), fine - s["target"], torch.zeros_like(fine)).square().sum()
        loss.backward()
        return dict(fine=fine.detach(), loss=loss.detach(), grad=v.grad)
    if op == "coarse":
        n = case["nc"]
        g = R.Grid.make(n)
        R.rtsdf_voxelize(s["v"], s["f"], g, s["seeds"])
        if case["variant"] == "jfa":
            R.rtsdf_jfa(g, s["seeds"], s["scratch"], case["beta"] / n, s["dist2"], s["sdf"])
        else:
            R.rtsdf_jfa_steps(g, s["seeds"], s["scratch"], R.jfa_schedule(n, case["variant"]), case["beta"] / n,
                              s["dist2"], s["sdf"])
        return dict(seeds=s["seeds"], dist2=s["dist2"], sdf=s["sdf"])
    if op == "select":
        cg, fg = R.Grid.make(case["nc"]), R.Grid.make(case["nf"])
        d = case["d"] / case["nc"]
        if case["mode"] == "point":
            R.rtsdf_select(cg, s["dist2"], fg, case["beta"] / case["nc"], d, s["mask"], s["queue"], s["count"],
                           s["ws"])
            return dict(mask=s["mask"], queue=s["queue"], count=s["count"])
        R.rtsdf_coarse_trilinear(cg, s["c"], fg, s["fine_c"])
        R.rtsdf_select_field(fg, s["fine_c"], d, s["mask"], s["queue"], s["count"], s["ws"])
        return dict(fine_c=s["fine_c"], mask=s["mask"], queue=s["queue"], count=s["count"])
    if op == "shadow":
        h = 1.0 / case["nf"]
        R.rtsdf_shadow_ex(R.Grid.make(case["nf"]), s["sdf"], s["pts"], _LIGHT, 8.0, h, case["steps"], 2 * h, 0.3,
                          s["vis"], penumbra=case["penumbra"], jitter=s["jitter"], jitter_scale=2 * h)
        return s["vis"]
    if op == "pick":
        s["scene"].rebuild(s["moves"][k % 2])
        R.rtsdf_closest_hits(s["scene"], s["o"], s["w"], s["t"], s["tri"], s["front"])
        return dict(t=s["t"], tri=s["tri"], front=s["front"])
    R.rtsdf_texel_distance(s["p"].scene, s["p"].fine, s["q"], s["dist"], s["tri"])
    return dict(dist=s["dist"], tri=s["tri"])


# -------------------------------------------------------------------- work


def _triangles(prims, level):
    _, t = _primitive(2, level)
    return 12 + prims * (12 + 20 * 4 ** level + len(t)) / 3


def _selected(case):
    """Share of the fine texels within the band, roughly: walls and primitives of log-uniform size."""
    prims = case.get("prims", 1)
    band = (case["d"] + case["beta"]) / case["nc"]
    return min(1.0, 6 * band + prims * 0.06 * band) if case.get("scene") != "sphere" else min(1.0, 4 * band)


def _ray_flops(tris):
    # one ray: drawing it (Philox and the sphere map), one descent of a two-wide hierarchy, one leaf
    return 360 + 39 * math.log2(max(2.0, tris)) + 4 * 33


def work(case):
    op = case["op"]
    if op == "update":
        tris = _triangles(case["prims"], case["level"]) if case["scene"] != "sphere" else 322
        nc3, nf3 = case["nc"] ** 3, case["nf"] ** 3
        tex = _selected(case) * nf3
        return dict(bytes=tris * (12 + 6) + 8 * nc3 + nf3 * 5 + tex * 32, flops=tex * case["rays"] * _ray_flops(tris))
    if op == "batch":
        tris = math.sqrt(case["tmin"] * case["tmax"])
        tex = 0.35 * (2 * case["ncmax"] * 0.6) ** 3
        return dict(bytes=case["scenes"] * (tex * 40 + tris * 18),
                    flops=case["scenes"] * tex * case["rays"] * _ray_flops(tris))
    if op == "diff":
        tex = 0.05 * case["nf"] ** 3
        tris = 20 * case["freq"] ** 2
        return dict(bytes=case["frames"] * tex * 32 + case["nf"] ** 3 * 16 + tris * 18,
                    flops=case["frames"] * tex * case["rays"] * _ray_flops(tris))
    if op == "coarse":
        n3 = case["nc"] ** 3
        tris = _triangles(case["prims"], case["level"])
        return dict(bytes=12 * n3 + tris * 18, flops=tris * 3 * 60 + n3 * math.log2(case["nc"]) * 27 * 4)
    if op == "select":
        nf3, nc3 = case["nf"] ** 3, case["nc"] ** 3
        tex = min(1.0, 8 * case["d"] / case["nc"] * (1 + case["balls"] / 30)) * nf3
        return dict(bytes=4 * nc3 + nf3 * (5 if case["mode"] == "trilinear" else 1) + 4 * tex,
                    flops=nf3 * (21 if case["mode"] == "trilinear" else 1))
    if op == "shadow":
        return dict(bytes=4 * case["nf"] ** 3 + 20 * case["points"], flops=case["points"] * 20 * 60)
    if op == "pick":
        tris = _triangles(case["prims"], case["level"])
        return dict(bytes=36 * case["rays"] + tris * 18, flops=case["rays"] * _ray_flops(tris))
    tris = _triangles(case["prims"], case["level"])
    n = min(case["most"], _selected(case) * case["nf"] ** 3)
    return dict(bytes=12 * n + tris * 18, flops=n * (20 * math.log2(tris) + 4 * 60))


# ------------------------------------------------------------------- exact
#
# The traced state of an update, a batch or a differentiable step has no value here beyond the small cases: every
# ray would be tested against every triangle.  (A small update's `u` is computed so, for its first frame.)

_BRUTE = 6e9  # ray / triangle or point / triangle pairs that are worth the time


def _brute_hits(o, w, v, f):
    """Smallest t > 0 per ray over all triangles (Moller-Trumbore in float64); +inf on a miss."""
    a, b, c = (v.double()[f.long()[:, i]] for i in range(3))
    e1, e2 = b - a, c - a
    out = torch.full((len(o),), math.inf, dtype=torch.float64, device=o.device)
    step = max(1, int(2e7 / max(1, len(f))))
    for i in range(0, len(o), step):
        ww, oo = w[i:i + step].double()[:, None], o[i:i + step].double()[:, None]
        pv = torch.linalg.cross(ww.expand(-1, len(f), 3), e2[None].expand(ww.shape[0], -1, 3))
        det = (e1 * pv).sum(-1)
        s = oo - a
        bu = (s * pv).sum(-1) / det
        q = torch.linalg.cross(s, e1[None].expand(s.shape[0], -1, 3))
        bv = (ww * q).sum(-1) / det
        t = (e2 * q).sum(-1) / det
        ok = (det != 0) & (bu >= 0) & (bv >= 0) & (bu + bv <= 1) & (t > 0)
        out[i:i + step] = torch.where(ok, t, torch.full_like(t, math.inf)).min(1).values
    return out


def _philox_directions(seed, texel, rays, scene, frame=0):
    """Unit directions [len(texel), rays, 3]: Philox4x64-10 words to Marsaglia's sphere points, in float32 steps."""
    m32 = np.uint64(0xFFFFFFFF)

    def mul(a, b):
        al, ah, bl, bh = a & m32, a >> np.uint64(32), b & m32, b >> np.uint64(32)
        ll, lh, hl = al * bl, al * bh, ah * bl
        mid = (ll >> np.uint64(32)) + (lh & m32) + (hl & m32)
        return ah * bh + (lh >> np.uint64(32)) + (hl >> np.uint64(32)) + (mid >> np.uint64(32)), a * b

    n = len(texel) * rays
    tx = np.repeat(texel.astype(np.uint64), rays)
    ry = np.tile(np.arange(rays, dtype=np.uint64), len(texel)) | np.uint64(frame << 32)
    out = np.zeros((n, 3), np.float32)
    out[:, 2] = 1
    todo = np.arange(n)
    f32 = np.float32
    with np.errstate(over="ignore"):
        for attempt in range(8):
            c = [tx[todo], ry[todo], np.full(len(todo), scene, np.uint64), np.full(len(todo), attempt, np.uint64)]
            k0, k1 = np.uint64(seed), np.uint64(0)
            for r in range(10):
                if r:
                    k0, k1 = k0 + np.uint64(0x9E3779B97F4A7C15), k1 + np.uint64(0xBB67AE8584CAA73B)
                h0, l0 = mul(np.uint64(0xD2E7470EE14C6C93), c[0])
                h1, l1 = mul(np.uint64(0xCA5A826395121157), c[2])
                c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
            found = np.zeros(len(todo), bool)
            for p in range(4):
                x1, x2 = ((((h >> np.uint64(9)) << np.uint64(1)).astype(np.int64) + 1 - 8388608).astype(f32)
                          * f32(2.0 ** -23) for h in (c[p] & m32, c[p] >> np.uint64(32)))
                s = x1 * x1 + x2 * x2
                take = ~found & (s < 1)
                q = np.sqrt(f32(1) - s[take])
                out[todo[take]] = np.stack([f32(2) * x1[take] * q, f32(2) * x2[take] * q, f32(1) - f32(2) * s[take]], 1)
                found |= take
            todo = todo[~found]
            if not len(todo):
                break
    return out.reshape(len(texel), rays, 3)


def _exact_voxels(v, f, n):
    """Own index of every voxel the mesh marks, else -1 (int64 [n^3]): vertices snapped to 1/256 voxel, a column is
    covered where its centre is in or on the projected triangle, the voxel at the triangle's depth there is marked."""
    X = torch.round(v.double() * (n * 256.0)).long()[f.long()]  # [nt, 3, 3]
    out = torch.full((n ** 3,), -1, dtype=torch.int64, device=v.device)
    for axis in range(3):
        e1, e2 = (axis + 1) % 3, (axis + 2) % 3
        px, py, pz = X[:, :, e1], X[:, :, e2], X[:, :, axis]
        area = (px[:, 1] - px[:, 0]) * (py[:, 2] - py[:, 0]) - (py[:, 1] - py[:, 0]) * (px[:, 2] - px[:, 0])
        flip = (area < 0)[:, None]
        px, py, pz = (torch.where(flip, t[:, [0, 2, 1]], t) for t in (px, py, pz))
        area = area.abs()
        lo = lambda t: torch.div(t.min(1).values + 127, 256, rounding_mode="floor").clamp(min=0)  # noqa: E731
        hi = lambda t: torch.div(t.max(1).values - 128, 256, rounding_mode="floor").clamp(max=n - 1)  # noqa: E731
        i0, i1, j0, j1 = lo(px), hi(px), lo(py), hi(py)
        w, h = (i1 - i0 + 1).clamp(min=0), (j1 - j0 + 1).clamp(min=0)
        cnt = torch.where(area > 0, w * h, torch.zeros_like(w))
        t = torch.repeat_interleave(torch.arange(len(cnt), device=v.device), cnt)
        k = torch.arange(len(t), device=v.device) - (torch.cumsum(cnt, 0) - cnt)[t]
        i, j = i0[t] + k % w[t].clamp(min=1), j0[t] + k // w[t].clamp(min=1)
        cx, cy = 256 * i + 128, 256 * j + 128
        px, py, pz = px[t], py[t], pz[t]
        e = [(px[:, (a + 2) % 3] - px[:, (a + 1) % 3]) * (cy - py[:, (a + 1) % 3])
             - (py[:, (a + 2) % 3] - py[:, (a + 1) % 3]) * (cx - px[:, (a + 1) % 3]) for a in range(3)]
        num = e[0] * pz[:, 0] + e[1] * pz[:, 1] + e[2] * pz[:, 2]
        den = area[t] * 256
        L = torch.div(num, den, rounding_mode="floor")
        L = torch.where(num == n * den, torch.full_like(L, n - 1), L)
        ok = (e[0] >= 0) & (e[1] >= 0) & (e[2] >= 0) & (L >= 0) & (L < n)
        q = [None] * 3
        q[axis], q[e1], q[e2] = L[ok], i[ok], j[ok]
        at = q[0] + n * (q[1] + n * q[2])
        out[at] = at
    return out


def _exact_jfa(seed, n, steps):
    """(seeds, squared distances) of jump flooding with these steps, int64 [n^3]."""
    a = torch.arange(n, device=seed.device, dtype=torch.int32)
    Z, Y, X = a[:, None, None], a[None, :, None], a[None, None, :]
    none = (1 << 62)

    def key(sd):
        x, y, z = sd % n, sd // n % n, sd // (n * n)
        d = (x - X) ** 2 + (y - Y) ** 2 + (z - Z) ** 2
        return torch.where(sd >= 0, (d.long() << 32) | sd.long(), torch.full_like(d, 0).long() + none)

    cur = seed.to(torch.int32).reshape(n, n, n)
    for k in steps:
        best = key(cur)
        for dz in (-k, 0, k):
            for dy in (-k, 0, k):
                for dx in (-k, 0, k):
                    if not (dx or dy or dz):
                        continue
                    sh = torch.full_like(cur, -1)
                    dst, src = [], []
                    for o in (dz, dy, dx):
                        dst.append(slice(max(0, -o), n - max(0, o)))
                        src.append(slice(max(0, o), n - max(0, -o)))
                    sh[tuple(dst)] = cur[tuple(src)]
                    best = torch.minimum(best, key(sh))
        cur = torch.where(best < none, best & 0xFFFFFFFF, torch.full_like(best, -1)).to(torch.int32)
    best = key(cur)
    return cur.reshape(-1), torch.where(best < none, best >> 32, torch.full_like(best, -1)).reshape(-1)


def _exact_point_distance(p, v, f):
    a, b, c = (v.double()[f.long()[:, i]] for i in range(3))
    out = torch.empty(len(p), dtype=torch.float64, device=p.device)
    step = max(1, int(1e7 / len(f)))

    def seg(q, a, e):
        t = (((q - a) * e).sum(-1) / (e * e).sum(-1)).clamp(0, 1)
        return (a + t[..., None] * e - q).square().sum(-1)

    n = torch.linalg.cross(b - a, c - a)
    nn = (n * n).sum(-1)
    for i in range(0, len(p), step):
        q = p[i:i + step].double()[:, None]
        d = torch.minimum(torch.minimum(seg(q, a, b - a), seg(q, b, c - b)), seg(q, c, a - c))
        s = q - a
        h = (s * n).sum(-1)
        inside = torch.ones_like(h, dtype=torch.bool)
        for x, y in ((a, b), (b, c), (c, a)):
            inside &= (torch.linalg.cross((y - x)[None].expand(q.shape[0], -1, 3), q - x) * n).sum(-1) >= 0
        out[i:i + step] = torch.where(inside, h * h / nn, d).min(1).values.sqrt()
    return out


def _exact_shadow(s):
    case = s["case"]
    n, sdf = case["nf"], s["sdf"].double()
    h, k, P = 1.0 / n, 8.0, s["pts"].double()
    light = torch.tensor(_LIGHT, dtype=torch.float32).double().to(P.device)
    t = torch.full((len(P),), h, dtype=torch.float64, device=P.device)
    if s["jitter"] is not None:
        t = t + s["jitter"].double() * float(np.float32(2 * h))
    top = float(np.float32(0.3))
    vis, live = torch.ones_like(t), torch.ones_like(t, dtype=torch.bool)
    tp, sp = torch.zeros_like(t), torch.zeros_like(t)
    for step in range(case["steps"]):
        g = (P + t[:, None] * light) * n - 0.5
        live = live & (t <= top) & ((g >= -0.5) & (g <= n - 0.5)).all(1)
        gc = g.clamp(0, n - 1)
        i = gc.floor().clamp(max=n - 2).long()
        fr = gc - i
        at = lambda dx, dy, dz: sdf[(i[:, 0] + dx) + n * ((i[:, 1] + dy) + n * (i[:, 2] + dz))]  # noqa: E731
        mix = lambda x, y, w: x + w * (y - x)  # noqa: E731
        i = torch.minimum(torch.maximum(i, torch.zeros_like(i)), torch.full_like(i, n - 2))
        c = [[mix(at(0, y, z), at(1, y, z), fr[:, 0]) for y in (0, 1)] for z in (0, 1)]
        v = mix(mix(c[0][0], c[0][1], fr[:, 1]), mix(c[1][0], c[1][1], fr[:, 1]), fr[:, 2])
        dark = live & (v < h)
        vis = torch.where(dark, torch.zeros_like(vis), vis)
        live = live & ~dark
        cone = k * v / t
        if case["penumbra"] and step:
            D = t - tp
            y = torch.minimum(((D * D + v * v - sp * sp) / (2 * D)).clamp(min=0), v)
            w = t - y
            cone = torch.where(w > 0, k * (v * v - y * y).clamp(min=0).sqrt() / w, torch.full_like(w, math.inf))
        vis = torch.where(live, torch.minimum(vis, cone), vis)
        tp, sp = torch.where(live, t, tp), torch.where(live, v, sp)
        t = torch.where(live, t + v.clamp(max=2 * h).clamp(min=h), t)
        if not bool(live.any()):
            break
    return vis.clamp(min=0)


def exact(case, seed):
    op = case["op"]
    if op == "update":
        sc = _Scene(case["scene"], case["prims"], case["level"], seed)
        small = case["motion"] == "static" and not case["graph"] and case["sampling"] == "point"
        tris = sum(len(f) for _, f in sc.parts + [m[0] for m in sc.moving])
        if not small or _selected(case) * case["nf"] ** 3 * case["rays"] * tris > _BRUTE / 10:
            return None
        v, f = sc.mesh()
        n, nf, r = case["nc"], case["nf"], case["nf"] // case["nc"]
        beta, d = _beta_d(case)
        _, d2 = _exact_jfa(_exact_voxels(v, f, n), n, R.jfa_schedule(n))
        a = torch.arange(nf, device=v.device) // r
        up = lambda t: t.reshape(n, n, n)[a][:, a][:, :, a].reshape(-1)  # noqa: E731
        thr = math.floor(((d + beta) * n) ** 2)
        tex = torch.nonzero((up(d2) <= thr) & (up(d2) >= 0)).flatten()
        w = torch.from_numpy(_philox_directions(seed & 0xFFFF, tex.cpu().numpy(), case["rays"], seed & 7)).to(v.device)
        ijk = torch.stack([tex % nf, tex // nf % nf, tex // (nf * nf)], 1).double()
        o = ((ijk + 0.5) / nf)[:, None].expand(-1, case["rays"], 3).reshape(-1, 3)
        t = _brute_hits(o, w.reshape(-1, 3), v, f).reshape(-1, case["rays"]) * w.double().norm(dim=2)
        rt = t.min(1).values
        c = torch.where(d2 >= 0, d2.double().sqrt() / n - beta, torch.full((), math.inf, device=v.device).double())
        u = torch.full((nf ** 3,), math.inf, dtype=torch.float64, device=v.device)
        if case["alpha"] == 1.0 or case["alpha"] > 0:  # no history before the first frame: alpha inf stays inf
            u[tex] = rt
        keys = ("hits", "arg_tri", "arg_ray", "fine_sdf", "mask", "count", "seeds")
        return dict({k: None for k in keys}, u=u, coarse_sdf=c)
    if op == "coarse":
        n = case["nc"]
        v, f = _Scene("room", case["prims"], case["level"], seed).mesh()
        _, d2 = _exact_jfa(_exact_voxels(v, f, n), n, R.jfa_schedule(n, case["variant"]))
        return dict(seeds=None, dist2=None, sdf=d2.double().sqrt() / n - float(np.float32(case["beta"] / n)))
    if op == "select":
        if case["mode"] == "point":
            return None
        s = prepare(case, seed)
        n, nf = case["nc"], case["nf"]
        u = ((torch.arange(nf, device=DEV).double() + 0.5) * (n / nf) - 0.5).clamp(0, n - 1)
        i0 = u.floor().long()
        i1, t = (i0 + 1).clamp(max=n - 1), u - i0
        c = s["c"].double().reshape(n, n, n)
        s.clear()
        c = c[:, :, i0] + t * (c[:, :, i1] - c[:, :, i0])
        c = c[:, i0] + t[:, None] * (c[:, i1] - c[:, i0])
        c = c[i0] + t[:, None, None] * (c[i1] - c[i0])
        return dict(fine_c=c.reshape(-1), mask=None, queue=None, count=None)
    if op == "shadow":
        return _exact_shadow(prepare(case, seed))
    if op == "pick":
        if case["rays"] * _triangles(case["prims"], case["level"]) > _BRUTE:
            return None
        s = prepare(case, seed)
        return dict(t=_brute_hits(s["o"], s["w"], s["moves"][0], s["f"]), tri=None, front=None)
    if op == "distance":
        tris = _triangles(case["prims"], case["level"])
        if min(case["most"], _selected(case) * case["nf"] ** 3) * tris > _BRUTE:
            return None
        s = prepare(case, seed)
        q, nf = s["q"].long(), case["nf"]
        ijk = torch.stack([q % nf, q // nf % nf, q // (nf * nf)], 1).double()
        return dict(dist=_exact_point_distance((ijk + 0.5) / nf, s["p"].vertices, s["p"].faces), tri=None)
    return None
