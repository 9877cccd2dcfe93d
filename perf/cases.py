"""Performance cases of the dynamic ray tracer, from its smallest calls to its
largest, through the public entry points of paper_2112_07115_amd.dcem.

A case is a plain dict; `prepare` builds what a program holds before the frames
it measures (scene uploaded into a context, object transforms on the device,
for coherent work the first full trace done), `run` makes one pass and returns
its results, `work` counts what the pass cannot do without, and `exact` gives
the results in 64 bits from plain torch.  `kind` says how the entry points are
called:

  frame  one frame traced in full: place the objects, update (or rebuild) the
         tree, trace, read the powers (and the paths)
  drive  consecutive coherent frames, the next frame's geometry enqueued before
         a frame's powers are read; the objects drive `steps` / 2 frames out and
         back again, so a pass ends where it began
  step   one step of a material fit: per frame a new material table, a coherent
         trace, powers and their gradients
  batch  one batched frame of several cities of different sizes

and `scene` names the generator of paper_2112_07115_amd.scenes the geometry
comes from (its seed is the case's).  Powers are FP64 host arrays, as the entry
points return them.
"""
from __future__ import annotations

import dataclasses
import itertools
import math

import numpy as np
import torch

from paper_2112_07115_amd import dcem, scenes

# fields a case may leave out
DEFAULTS = dict(n_rays=4096, max_reflections=2, n_rx=64, n_tx=1, bands=1, tris=0, rebuild=False, visited=False,
                backward=False, max_transmissions=0, paths=False, steps=0, frames=0, cities=0, vehicles=0,
                grid_blocks=0, facade_cells=0, corridor_m=0, capacity=1 << 22)
PATH_ROWS = 4096   # rows of a program's path table (more paths are cut off)
BANDS = (28e9, 60e9, 3.5e9, 5.9e9)


def listed():
    return [
        # A planning tool's interactive query: one frame of a small static
        # scene, 16 receivers.  Launches and round trips are what counts.
        dict(name="toy_frame", kind="frame", scene="toy", n_rays=4096, max_reflections=2),
        # Channel sounding of a small site with turning objects: the powers
        # and every path with its length, delay, directions and field.
        dict(name="site_paths", kind="frame", scene="oblique", n_rays=1 << 16, max_reflections=3, paths=True),
        # The same site followed frame by frame (10 Hz), 3 bands, odd ray count.
        dict(name="site_drive", kind="drive", scene="oblique", n_rays=50021, max_reflections=3, bands=3, steps=8),
        # The urban street grid followed frame by frame at its full size: 32,002
        # triangles, 40 vehicles, 256 receivers, 2^20 rays, 4 reflections.
        dict(name="urban_drive", kind="drive", scene="urban", n_rays=1 << 20, max_reflections=4, n_rx=256, steps=8),
        # One frame of it from scratch: the tree rebuilt, every ray traced.
        dict(name="urban_full", kind="frame", scene="urban", n_rays=1 << 20, max_reflections=4, n_rx=256,
             rebuild=True),
        # The paper's visited-series tables on the same frame, tree refitted.
        dict(name="urban_visited", kind="frame", scene="urban", n_rays=1 << 20, max_reflections=4, n_rx=256,
             visited=True),
        # Backward tracing: 4,096 rays from each of the 256 receivers.
        dict(name="urban_backward", kind="frame", scene="urban", n_rays=4096, max_reflections=4, n_rx=256,
             visited=True, backward=True),
        # Indoor coverage through walls and glass (11 branches per ray).
        dict(name="office_capture", kind="frame", scene="office", n_rays=1 << 18, max_reflections=2,
             max_transmissions=2),
        dict(name="office_visited", kind="frame", scene="office", n_rays=1 << 18, max_reflections=2,
             max_transmissions=2, visited=True),
        # A step of the eight-class material fit: 1,024 receivers, 3 frames.
        dict(name="fit_step", kind="step", scene="urban8", n_rays=1 << 18, max_reflections=4, n_rx=1024, frames=3),
        # Eight ragged cities in one batched frame (10k-120k triangles,
        # 256k-1M rays, 1-8 transmitters, 2-6 reflections).
        dict(name="city_batch", kind="batch", scene="city", cities=8, tris=120000, n_rays=1 << 20, n_rx=512),
        # The large dynamic scene: 2.04M triangles, 4,096 receivers on the
        # vehicles, 4 transmitters x 2^22 rays, 6 reflections, two bands.
        dict(name="highway_drive", kind="drive", scene="highway", n_rays=1 << 22, max_reflections=6, n_rx=4096,
             n_tx=4, bands=2, vehicles=200, grid_blocks=16, facade_cells=19, corridor_m=6000, capacity=1 << 24,
             steps=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["toy", "site", "office", "city_frame", "city_frame", "city_drive", "city_visited",
                       "city_backward", "highway_drive", "highway_frame", "fit", "batch"])
    if what == "toy":
        return dict(kind="frame", scene="toy", n_rays=_log(rng, 1000, 1 << 17), max_reflections=rng.randint(0, 6),
                    bands=rng.randint(1, 4), visited=rng.random() < 0.3, paths=rng.random() < 0.3)
    if what == "site":
        c = dict(scene="oblique", n_rays=_log(rng, 3000, 1 << 18), max_reflections=rng.randint(1, 5),
                 bands=rng.randint(1, 4))
        if rng.random() < 0.5:
            return dict(kind="drive", steps=2 * rng.randint(1, 4), **c)
        return dict(kind="frame", rebuild=rng.random() < 0.3, paths=rng.random() < 0.3, **c)
    if what == "office":
        return dict(kind="frame", scene="office", n_rays=_log(rng, 1 << 11, 1 << 18),
                    max_reflections=rng.randint(1, 3), max_transmissions=rng.randint(0, 2),
                    visited=rng.random() < 0.5, bands=rng.randint(1, 3))
    if what == "fit":
        return dict(kind="step", scene="urban8", n_rays=_log(rng, 1 << 14, 1 << 19), max_reflections=rng.randint(2, 5),
                    n_rx=_log(rng, 64, 1024), bands=rng.randint(1, 2), frames=rng.randint(1, 4))
    if what == "batch":
        return dict(kind="batch", scene="city", cities=rng.randint(2, 8), tris=_log(rng, 12000, 160000),
                    n_rays=_log(rng, 300000, 1 << 20), n_rx=_log(rng, 70, 1024))
    if what.startswith("highway"):
        c = dict(scene="highway", n_rays=_log(rng, 1 << 16, 1 << 20), max_reflections=rng.randint(2, 6),
                 n_rx=_log(rng, 256, 4096), n_tx=rng.randint(1, 4), bands=rng.randint(1, 2),
                 vehicles=rng.randint(20, 200), grid_blocks=rng.randint(4, 16), facade_cells=rng.randint(4, 19),
                 corridor_m=200 * rng.randint(5, 30), capacity=1 << 24)
        if what == "highway_drive":
            return dict(kind="drive", steps=2 * rng.randint(1, 2), **c)
        return dict(kind="frame", rebuild=rng.random() < 0.5, **c)
    c = dict(scene="city", tris=_log(rng, 3000, 300000), max_reflections=rng.randint(1, 6), n_tx=rng.randint(1, 4),
             n_rx=_log(rng, 16, 1024), bands=rng.randint(1, 3))
    if what == "city_frame":
        return dict(kind="frame", n_rays=_log(rng, 1 << 13, 1 << 20), rebuild=rng.random() < 0.5,
                    paths=rng.random() < 0.2, **c)
    if what == "city_drive":
        return dict(kind="drive", n_rays=_log(rng, 1 << 13, 1 << 20), steps=2 * rng.randint(1, 4), **c)
    c.update(max_reflections=rng.randint(1, 4), n_rx=_log(rng, 16, 256), visited=True)
    if what == "city_backward":
        return dict(kind="frame", n_rays=_log(rng, 256, 4096), backward=True, **c)
    return dict(kind="frame", n_rays=_log(rng, 1 << 13, 1 << 18), **c)


# ---- what a program holds before the call


def _full(case):
    return {**DEFAULTS, **case}


def _make_scene(c, seed):
    """The case's scene, its geometry and positions drawn from `seed`."""
    freqs = list(BANDS[:c["bands"]])
    seed = int(seed) % (1 << 31)
    if c["scene"] == "toy":
        s = scenes.static_toy(seed)
    elif c["scene"] == "oblique":
        s = scenes.oblique_town(seed)
    elif c["scene"] in ("urban", "urban8"):
        s = scenes.dynamic_urban(seed, n_rx=c["n_rx"], material_classes=8 if c["scene"] == "urban8" else 3)
    elif c["scene"] == "office":
        # the floor plan is fixed; the transmitter stands anywhere in the
        # corridor and the receiver grid is shifted within a quarter metre
        s = scenes.indoor_office(max_transmissions=c["max_transmissions"])
        r = np.random.default_rng(seed)
        tx = np.array([[r.uniform(1.0, 23.0), r.uniform(6.4, 7.6), r.uniform(1.6, 2.4)]], np.float32)
        s = dataclasses.replace(s, tx=tx, rx=s.rx + np.append(r.uniform(-0.25, 0.25, 2), 0.0).astype(np.float32))
        freqs = [30e9, 60e9, 5.9e9][:c["bands"]]
    elif c["scene"] == "highway":
        s = scenes.highway_city(seed, grid_blocks=c["grid_blocks"], facade_cells=c["facade_cells"],
                                corridor_m=float(c["corridor_m"]), warehouses=c["corridor_m"] // 100,
                                n_vehicles=c["vehicles"], n_rx=c["n_rx"], n_tx=c["n_tx"])
    else:
        s = scenes.ragged_city(seed, c["tris"], n_tx=c["n_tx"], n_rx=c["n_rx"])
    return dataclasses.replace(s, n_rays=c["n_rays"], max_reflections=c["max_reflections"], freqs_hz=freqs,
                               max_transmissions=c["max_transmissions"])


def _city_sizes(c):
    """A batch's cities: triangles, rays, receivers, transmitters, reflections
    and bands each step through their ranges, in orders of their own."""
    n = c["cities"]

    def between(lo, hi, k):
        return int(lo * (hi / lo) ** (k / max(n - 1, 1)))
    return [dict(target_tris=between(10000, c["tris"], j), n_tx=1 + (5 * j) % 8, n_rx=between(64, c["n_rx"], (3 * j) % n),
                 n_rays=between(1 << 18, c["n_rays"], n - 1 - j) // (1 + (5 * j) % 8), max_reflections=2 + j % 5,
                 freqs_hz=BANDS[j % 2:j % 2 + 1]) for j in range(n)]


def _first_frame(s, seed):
    """The frame a pass starts at (a few frames into the motion)."""
    return 1 + int(seed) % max(1, min(s.n_frames - 6, 12)) if s.n_objects else 0


def _route(c, f0):
    """Frames of a drive's pass: steps / 2 out from f0 and back to it."""
    h = c["steps"] // 2
    return [f0 + k for k in range(1, h + 1)] + [f0 + k for k in range(h - 1, -1, -1)]


def _args(s, c, f, **kw):
    return dcem.scene_frame_args(s, f, trace_from_rx=c["backward"],
                                 discovery=dcem.DISCOVER_VISITED if c["visited"] else dcem.DISCOVER_CAPTURE, **kw)


class _State:
    pass


def prepare(case, seed):
    c = _full(case)
    st = _State()
    st.c = c
    st.rows = {}
    if c["kind"] == "batch":
        st.stream = torch.cuda.Stream()
        st.scenes = [scenes.ragged_city((int(seed) + 7919 * j) % (1 << 31), **size)
                     for j, size in enumerate(_city_sizes(c))]
        st.ctxs = []
        with torch.cuda.stream(st.stream):
            st.xfs = [torch.tensor(s.transforms(2), device="cuda") for s in st.scenes]
            for s in st.scenes:
                ctx = dcem.Context(0, stream=st.stream.cuda_stream)
                ctx.scene_upload(s)
                st.ctxs.append(ctx)
            st.frames = [dcem.scene_frame_args(s) for s in st.scenes]
            st.batch = dcem.Batch(st.ctxs)
        return st
    s = st.scene = _make_scene(c, seed)
    st.ctx = dcem.Context(0)
    if c["capacity"] != DEFAULTS["capacity"]:
        st.ctx.set_capture_capacity(c["capacity"])
    st.ctx.scene_upload(s)
    st.f0 = _first_frame(s, seed)
    if c["kind"] == "frame":
        st.frames = [st.f0]
    elif c["kind"] == "drive":
        st.frames = _route(c, st.f0)
    else:
        st.frames = [st.f0 + k for k in range(c["frames"])]
        r = np.random.default_rng(int(seed))
        st.tables = []
        for _ in st.frames:
            m = s.materials.copy()
            m[:, 0] = r.uniform(2.0, 20.0, m.shape[0])
            m[:, 1] = 10.0 ** r.uniform(-3.0, 0.0, m.shape[0])
            st.tables.append(m)
    # object transforms on the device, and each frame's call
    st.xf = {f: torch.tensor(s.transforms(f), device="cuda") for f in set(st.frames) | {st.f0}} if s.n_objects else {}
    mode = dcem.MODE_FULL if c["kind"] == "frame" else dcem.MODE_COHERENT
    st.args = {f: _args(s, c, f, mode=mode) for f in set(st.frames) | {st.f0}}
    if c["kind"] != "frame":
        _place(st, st.frames[-1])
        st.ctx.trace_frame(**st.args[st.frames[-1]])
        st.ctx.received_power()
    if c["kind"] == "drive":
        _place(st, st.frames[0])
    return st


def _place(st, f):
    if st.xf:
        st.ctx.set_object_transforms(st.xf[f])
        st.ctx.refit_bvh(force_rebuild=st.c["rebuild"])


def run(st):
    c = st.c
    if c["kind"] == "frame":
        f = st.frames[0]
        _place(st, f)
        st.ctx.trace_frame(**st.args[f])
        p_coh, p_inc = st.ctx.received_power()
        out = {"p_coh": p_coh, "p_inc": p_inc}
        if c["paths"]:
            # into the channel model's fixed number of rows
            for k, v in st.ctx.paths().items():
                rows = st.rows.setdefault(k, np.zeros((PATH_ROWS,) + v.shape[1:], v.dtype))
                n = min(len(v), PATH_ROWS)
                rows[:n] = v[:n]
                rows[n:] = 0
            out["paths"] = st.rows
        return out
    if c["kind"] == "drive":
        out = []
        for k, f in enumerate(st.frames):
            st.ctx.trace_frame(**st.args[f])
            _place(st, st.frames[(k + 1) % len(st.frames)])
            out.append(st.ctx.received_power())
        return out
    if c["kind"] == "step":
        out = []
        for f, table in zip(st.frames, st.tables):
            st.ctx.set_materials(table)
            _place(st, f)
            st.ctx.trace_frame(**st.args[f])
            out.append(st.ctx.received_power() + st.ctx.power_gradients())
        return out
    with torch.cuda.stream(st.stream):
        for ctx, xf in zip(st.ctxs, st.xfs):
            ctx.set_object_transforms(xf)
            ctx.refit_bvh()
        st.batch.trace(st.frames)
        return [ctx.received_power() for ctx in st.ctxs]


# ---- what a pass cannot do without


def _frame_work(s, c, n_tx, n_rx, rays, coherent):
    """Bytes: the geometry and the rays' directions read once, the powers
    written once.  A coherent frame traces about one ray in a hundred and
    checks the others' cached segments (a 16-byte origin per segment, two
    segments a ray).  Flops: two segments a ray, each with one four-box node
    per level of a four-wide tree and two triangle tests."""
    items = rays * dcem.n_branches(c["max_reflections"], c["max_transmissions"])
    tris = s["tris"]
    geometry = 4.0 * 3 * (0.6 * tris) + 4.0 * 4 * tris
    levels = max(1.0, math.log(max(tris, 4), 4))
    flops = 2.0 * items * (levels * 4 * 18 + 2 * 60)
    byts = geometry + 12.0 * rays + 16.0 * n_tx * n_rx * c["bands"]
    if coherent:
        flops, byts = 0.01 * flops + 2.0 * items * 40, geometry + 33.0 * items + 16.0 * n_tx * n_rx * c["bands"]
    return byts, flops


def _size(c):
    if c["scene"] in ("toy", "oblique", "office", "urban", "urban8"):
        return {"toy": (50, 1, 16), "oblique": (534, 1, 64), "office": (396, 1, 336),
                "urban": (32002, 1, c["n_rx"]), "urban8": (32002, 1, c["n_rx"])}[c["scene"]]
    if c["scene"] == "highway":
        t = 20 * c["grid_blocks"] ** 2 * c["facade_cells"] ** 2 + 512 * c["vehicles"] + 4 * c["corridor_m"]
        return t, c["n_tx"], c["n_rx"]
    return c["tris"], c["n_tx"], c["n_rx"]


def work(case):
    c = _full(case)
    if c["kind"] == "batch":
        each = [_frame_work({"tris": z["target_tris"]}, dict(c, max_reflections=z["max_reflections"]), z["n_tx"],
                            z["n_rx"], z["n_rays"] * z["n_tx"], False) for z in _city_sizes(c)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    tris, n_tx, n_rx = _size(c)
    rays = c["n_rays"] * (n_rx if c["backward"] else n_tx)
    b, f = _frame_work({"tris": tris}, c, n_tx, n_rx, rays, c["kind"] != "frame")
    n = c["steps"] if c["kind"] == "drive" else (c["frames"] if c["kind"] == "step" else 1)
    return {"bytes": b * n, "flops": f * n}


# ---- the results in 64 bits, from plain torch
#
# Brute force: every ray segment against every triangle, every candidate path
# by the image method and against every triangle.  Beyond EXACT_TESTS
# ray-triangle tests it takes too long, and there is no value.

EXACT_TESTS = 1.2e10
C0, EPS0 = 299792458.0, 8.8541878128e-12
T_MIN = 1e-4


def _dot(a, b):
    return (a * b).sum(-1)


def _unit(a):
    return a / a.norm(dim=-1, keepdim=True)


class _Exact:
    """The frame algorithm on one pose of a scene: forward tracing from the
    transmitters, candidates from capture spheres or visited series."""

    def __init__(self, s, c, f, device):
        self.s, self.c, self.dev = s, c, device
        t64 = lambda a: torch.tensor(np.asarray(a), dtype=torch.float64, device=device)  # noqa: E731
        v = np.asarray(s.vertices, np.float64).copy()
        ref = v.copy()
        for o, (a, b) in enumerate(s.object_vertex_range):
            m = np.asarray(s.transforms(f)[o], np.float64)
            v[a:b] = (ref[a:b] @ m[:, :3].T + m[:, 3]).astype(np.float32)
        self.V = t64(v)[torch.tensor(s.tris.astype(np.int64), device=device)]     # [T, 3, 3]
        self.face = torch.tensor(s.tri_face.astype(np.int64), device=device)
        # a face's plane: its largest triangle of the upload pose
        r = ref[s.tris]
        area = np.linalg.norm(np.cross(r[:, 1] - r[:, 0], r[:, 2] - r[:, 0]), axis=1)
        first = np.lexsort((np.arange(len(area)), -area, s.tri_face))
        _, at = np.unique(s.tri_face[first], return_index=True)
        rt = torch.tensor(first[at], device=device)
        q = self.V[rt]
        self.n = _unit(torch.linalg.cross(q[:, 1] - q[:, 0], q[:, 2] - q[:, 0]))
        self.w = _dot(self.n, q[:, 0])
        self.tx, self.rx = t64(s.tx), t64(s.rx_at(f))
        self.r2 = float(np.float32(s.rx_radius)) ** 2
        loss = np.full(len(s.materials), np.inf) if s.penetration_db is None else np.asarray(s.penetration_db)
        self.pen = t64(np.where(np.isfinite(loss), 10.0 ** (-np.where(np.isfinite(loss), loss, 0.0) / 20.0), 0.0))
        self.fmat = torch.tensor(s.face_material.astype(np.int64), device=device)
        self.mats = t64(s.materials)
        self.K, self.T = s.max_reflections, s.max_transmissions
        self.slots = self.K + self.T

    def directions(self):
        n = self.s.n_rays
        i = np.arange(n, dtype=np.float64)
        z = 1.0 - (2.0 * i + 1.0) / n
        rho = np.sqrt(1.0 - z * z)
        phi = i * (math.pi * (3.0 - math.sqrt(5.0)))
        d = np.stack([rho * np.cos(phi), rho * np.sin(phi), z], 1).astype(np.float32)
        return torch.tensor(d.astype(np.float64), device=self.dev)

    def nearest(self, o, d, last):
        """(t, triangle) of the closest hit off face `last`; t infinite on a miss."""
        e1, e2 = self.V[:, 1] - self.V[:, 0], self.V[:, 2] - self.V[:, 0]
        ts, ids = [], []
        step = max(1, int(8e6) // max(1, len(self.V)))
        for b in range(0, len(o), step):
            D, O = d[b:b + step, None], o[b:b + step, None]
            p = torch.linalg.cross(D.expand(-1, len(e2), -1), e2.expand(len(D), -1, -1))
            det = _dot(p, e1)
            tv = O - self.V[:, 0]
            u = _dot(tv, p) / det
            q = torch.linalg.cross(tv, e1.expand(len(D), -1, -1))
            v = _dot(q, D) / det
            t = _dot(q, e2) / det
            e = 1e-12
            ok = (det != 0) & (u >= -e) & (v >= -e) & (u + v <= 1 + e) & (t > T_MIN)
            ok &= self.face != last[b:b + step, None]
            t, i = torch.where(ok, t, torch.full_like(t, math.inf)).min(1)
            ts.append(t)
            ids.append(i)
        return torch.cat(ts), torch.cat(ids)

    def discover(self):
        """Candidate rows (tx, rx, order, entries), an entry 2 * face + transmits."""
        sets = [m for t in range(self.T + 1) for m in itertools.combinations(range(self.slots), t)]
        rows = [self.row(t, r, ()) for t in range(len(self.tx)) for r in range(len(self.rx))]
        got = [torch.tensor(rows, dtype=torch.int64, device=self.dev)]
        dirs = self.directions()
        for t in range(len(self.tx)):
            for through in sets:
                o, d = self.tx[t].expand(len(dirs), 3).clone(), dirs.clone()
                last = torch.full((len(d),), -1, dtype=torch.int64, device=self.dev)
                seq = torch.full((len(d), self.slots), -1, dtype=torch.int64, device=self.dev)
                reflected = 0
                for k in range(self.slots + 1):
                    if not len(d):
                        break
                    th, tri = self.nearest(o, d, last)
                    if not self.c["visited"] and k > (max(through) if through else -1):
                        got.append(self.captured(o, d, th, t, k, seq))
                    if k == self.slots:
                        break
                    goes = torch.isfinite(th)
                    f = self.face[tri]
                    if k in through:
                        goes &= self.pen[self.fmat[f]] > 0
                    elif reflected == self.K:
                        break
                    o, d, f, th, seq = o[goes], d[goes], f[goes], th[goes], seq[goes]
                    v = self.V[tri[goes]]
                    o = o + th[:, None] * d
                    if k not in through:
                        n = _unit(torch.linalg.cross(v[:, 1] - v[:, 0], v[:, 2] - v[:, 0]))
                        d = d - 2 * _dot(d, n)[:, None] * n
                        reflected += 1
                    seq[:, k] = 2 * f + (1 if k in through else 0)
                    last = f
                    if self.c["visited"] and len(seq) and k >= (max(through) if through else 0):
                        u = torch.unique(seq, dim=0)
                        r = torch.arange(len(self.rx), device=self.dev)
                        head = torch.tensor([t, 0, k + 1], device=self.dev).expand(len(u) * len(r), 3).clone()
                        head[:, 1] = r.repeat(len(u))
                        got.append(torch.cat([head, u.repeat_interleave(len(r), 0)], 1))
        return torch.unique(torch.cat(got), dim=0)

    def row(self, t, r, seq):
        return [t, r, len(seq)] + list(seq) + [-1] * (self.slots - len(seq))

    def captured(self, o, d, th, t, k, seq):
        out = []
        for b in range(0, len(o), 1 << 15):
            O, D = o[b:b + (1 << 15), None], d[b:b + (1 << 15), None]
            w = self.rx - O
            s = (_dot(w, D) / _dot(D, D)).clamp(min=0.0)
            s = torch.minimum(s, th[b:b + (1 << 15), None])
            i, r = torch.nonzero(((s[..., None] * D - w) ** 2).sum(-1) <= self.r2, as_tuple=True)
            head = torch.stack([torch.full_like(r, t), r, torch.full_like(r, k)], 1)
            out.append(torch.cat([head, seq[i + b]], 1))
        return torch.unique(torch.cat(out), dim=0)

    def inside(self, f, p, live):
        """Is p in a triangle of face f (edges inclusive)?  Dominant axis dropped."""
        drop = self.n[f].abs().argmax(1)
        keep = torch.tensor([[1, 2], [2, 0], [0, 1]], device=self.dev)[drop]
        out = torch.zeros(len(p), dtype=torch.bool, device=self.dev)
        at = torch.nonzero(live).flatten()
        step = max(1, int(8e6) // max(1, len(self.V)))
        for b in range(0, len(at), step):
            i = at[b:b + step]
            P = torch.gather(p[i], 1, keep[i])[:, None]
            Q = torch.gather(self.V[None].expand(len(i), -1, -1, -1), 3,
                             keep[i][:, None, None].expand(-1, len(self.V), 3, -1))
            e = []
            for a in range(3):
                A, B = Q[:, :, a], Q[:, :, (a + 1) % 3]
                e.append((B[..., 0] - A[..., 0]) * (P[..., 1] - A[..., 1]) - (B[..., 1] - A[..., 1]) * (P[..., 0] - A[..., 0]))
            e = torch.stack(e)
            ok = (e >= 0).all(0) | (e <= 0).all(0)
            out[i] = (ok & (self.face == f[i][:, None])).any(1)
        return out

    def blocked(self, p, q, fa, fb, live):
        """Does a triangle off faces fa and fb cross p..q, T_MIN away from both ends?"""
        out = torch.zeros(len(p), dtype=torch.bool, device=self.dev)
        at = torch.nonzero(live).flatten()
        A, B, Cc = self.V[:, 0], self.V[:, 1], self.V[:, 2]

        def vol(a, b, c, d):
            return _dot(b - a, torch.linalg.cross(c - a, d - a))
        step = max(1, int(4e6) // max(1, len(self.V)))
        for b in range(0, len(at), step):
            i = at[b:b + step]
            P, Q = p[i][:, None].expand(-1, len(A), -1), q[i][:, None].expand(-1, len(A), -1)
            a, bb, cc = (x.expand(len(i), -1, -1) for x in (A, B, Cc))
            op, oq = vol(a, bb, cc, P), vol(a, bb, cc, Q)
            t = op / (op - oq)
            lim = (T_MIN / (q[i] - p[i]).norm(dim=1))[:, None]
            s = torch.stack([vol(P, Q, a, bb), vol(P, Q, bb, cc), vol(P, Q, cc, a)])
            hit = (op != oq) & (t > lim) & (t < 1 - lim) & ((s >= 0).all(0) | (s <= 0).all(0))
            hit &= (self.face != fa[i][:, None]) & (self.face != fb[i][:, None])
            out[i] = hit.any(1)
        return out

    def refine(self, rows):
        """Image method on every candidate row: valid, points, length."""
        order, ent = rows[:, 2], rows[:, 3:]
        f, thr = torch.clamp(ent, min=0) // 2, (ent >= 0) & (ent % 2 == 1)
        T, R = self.tx[rows[:, 0]], self.rx[rows[:, 1]]
        K = self.slots
        images = [T]
        for j in range(K):
            n, im = self.n[f[:, j]], images[-1]
            mirror = im - 2 * (_dot(im, n) - self.w[f[:, j]])[:, None] * n
            images.append(torch.where(((j < order) & ~thr[:, j])[:, None], mirror, im))
        ok = torch.ones(len(rows), dtype=torch.bool, device=self.dev)
        d = (R - images[K]).norm(dim=1)
        P = torch.zeros((len(rows), K + 2, 3), dtype=torch.float64, device=self.dev)
        P[:, 0] = T
        P.scatter_(1, (order + 1)[:, None, None].expand(-1, 1, 3), R[:, None])
        Q = R
        for j in range(K, 0, -1):
            live = j <= order
            n = self.n[f[:, j - 1]]
            D = images[j] - Q
            s = (self.w[f[:, j - 1]] - _dot(Q, n)) / _dot(D, n)
            ok &= ~live | ((s > 0) & (s < 1))
            ok &= ~(live & thr[:, j - 1]) | (self.pen[self.fmat[f[:, j - 1]]] > 0)
            Q = torch.where(live[:, None], Q + s[:, None] * D, Q)
            P[:, j] = torch.where(live[:, None], Q, P[:, j])
        for j in range(1, K + 1):
            live = ok & (j <= order)
            ok &= ~live | self.inside(f[:, j - 1], P[:, j], live)
        none = torch.full_like(order, -1)
        for j in range(K + 1):
            live = ok & (j <= order)
            fa = f[:, j - 1] if j else none
            fb = torch.where(j < order, f[:, min(j, K - 1)], none) if K else none
            ok &= ~self.blocked(P[:, j], P[:, j + 1], fa, fb, live)
        return ok, P, d, f, thr

    def solve(self):
        rows = self.discover()
        ok, P, d, f, thr = self.refine(rows)
        rows, P, d, f, thr = rows[ok], P[ok], d[ok], f[ok], thr[ok]
        order, K = rows[:, 2], self.slots
        amps = []
        aod = _unit(P[:, 1] - P[:, 0])
        rho = (aod[:, :2] ** 2).sum(1).sqrt()
        e0 = torch.stack([aod[:, 2] * aod[:, 0] / rho, aod[:, 2] * aod[:, 1] / rho, -rho], 1)
        for fr in self.s.freqs_hz:
            E = e0.to(torch.complex128)
            for j in range(K):
                live = (j < order)[:, None]
                m = self.fmat[f[:, j]]
                straight = E * self.pen[m][:, None]
                ki, kr = _unit(P[:, j + 1] - P[:, j]), _unit(P[:, j + 2] - P[:, j + 1])
                n = self.n[f[:, j]]
                cos = _dot(ki, n).abs()
                s = _unit(torch.linalg.cross(ki, n))
                pin, pout = torch.linalg.cross(s, ki), torch.linalg.cross(s, kr)
                ec = torch.complex(self.mats[m, 0], -self.mats[m, 1] / (2 * math.pi * fr * EPS0))
                root = torch.sqrt(ec - (1 - cos * cos))
                te, tm = (cos - root) / (cos + root), (ec * cos - root) / (ec * cos + root)
                g = self.mats[m, 2]
                te = torch.where(torch.isnan(g), te, (-g).to(te.dtype))
                tm = torch.where(torch.isnan(g), tm, g.to(tm.dtype))
                bounced = (te * _dot(E, s.to(E.dtype)))[:, None] * s + (tm * _dot(E, pin.to(E.dtype)))[:, None] * pout
                E = torch.where(live, torch.where(thr[:, j, None], straight, bounced), E)
            lam = C0 / fr
            amps.append(math.sqrt(self.s.tx_power_w) * lam / (4 * math.pi * d[:, None]) *
                        torch.exp(-2j * math.pi * fr / C0 * d)[:, None] * E)
        nt, nr = len(self.tx), len(self.rx)
        pair = rows[:, 0] * nr + rows[:, 1]
        coh, inc = [], []
        for a in amps:
            A = torch.zeros((nt * nr, 3), dtype=torch.complex128, device=self.dev).index_add_(0, pair, a)
            coh.append((A.abs() ** 2).sum(1).reshape(nt, nr))
            inc.append(torch.zeros(nt * nr, dtype=torch.float64, device=self.dev)
                       .index_add_(0, pair, (a.abs() ** 2).sum(1)).reshape(nt, nr))
        return torch.stack(coh).cpu().numpy(), torch.stack(inc).cpu().numpy()


def exact(case, seed):
    c = _full(case)
    if c["kind"] not in ("frame", "drive") or c["backward"]:
        return None
    tris, n_tx, _ = _size(c)
    frames = max(1, c["steps"] // 2 + 1 if c["kind"] == "drive" else 1)
    items = c["n_rays"] * n_tx * dcem.n_branches(c["max_reflections"], c["max_transmissions"])
    if frames * items * tris * min(c["max_reflections"] + c["max_transmissions"] + 1, 4) > EXACT_TESTS:
        return None
    s = _make_scene(c, seed)
    device = "cuda" if torch.cuda.is_available() else "cpu"
    f0 = _first_frame(s, seed)
    if c["kind"] == "drive":
        route = _route(c, f0)
        got = {f: _Exact(s, c, f, device).solve() for f in set(route)}
        return [got[f] for f in route]
    coh, inc = _Exact(s, c, f0, device).solve()
    # the path list has one row per candidate, valid or not: no value
    return {"p_coh": coh, "p_inc": inc, **({"paths": None} if c["paths"] else {})}
