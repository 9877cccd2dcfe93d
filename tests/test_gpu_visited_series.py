"""GPU: visited discovery loses no series, from the trace log by brute force: every
series of faces some ray's hits run over is tried against every receiver on the
host (FP64 images, points strictly inside their segments and faces, away from the
edges), what passes is a candidate, and every candidate's first ray is the lowest
ray of its series.  Lists sorted by one workgroup and in launches per pass, one
source and two, and few rays in a corner whose neighbours differ in face 0."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes

pytestmark = pytest.mark.gpu


def lowest_rays(face, K):
    """(source, faces) -> lowest ray, from the hit faces [n_src][n_rays][K] (-1: none)."""
    first = {}
    n = face.shape[1]
    for src in range(len(face)):
        for d in range(1, K + 1):
            hit = np.flatnonzero((face[src, :, :d] >= 0).all(axis=1))
            seq, at = np.unique(face[src, hit, :d], axis=0, return_index=True)
            for q, i in zip(seq.tolist(), at):   # return_index: the lowest
                first[(src,) + tuple(q)] = src * n + int(hit[i])
    return first


def list_length(face, dirs, K):
    """Items the series are sorted from, up to rounding in the order of the rays: a
    run of neighbouring directions with one series enters it once in a wavefront."""
    d = dirs / np.abs(dirs).sum(axis=1, keepdims=True)
    fold = (1.0 - np.abs(d[:, [1, 0]])) * np.where(d[:, :2] >= 0, 1.0, -1.0)
    uv = np.where(d[:, 2:] >= 0, d[:, :2], fold)
    q = ((uv * 0.5 + 0.5) * 65535.0).astype(np.uint64)
    bits = np.arange(16, dtype=np.uint64)
    spread = ((q[:, :, None] >> bits & np.uint64(1)) << (np.uint64(2) * bits)).sum(axis=2)
    face = face[:, np.argsort(spread[:, 0] * np.uint64(2) + spread[:, 1], kind="stable")].reshape(-1, K)
    head = np.arange(len(face)) % 64 == 0
    n = 0
    for k in range(1, K + 1):
        has = (face[:, :k] >= 0).all(axis=1)
        new = np.r_[True, (face[1:, :k] != face[:-1, :k]).any(axis=1)]
        n += int((has & (head | new)).sum())
    return n


def cross2(a, b):
    return a[..., 0] * b[..., 1] - a[..., 1] * b[..., 0]


class Walk:
    """Image-method walks of series over the scene's faces, all receivers at once."""

    def __init__(self, s, verts, eps=1e-6):
        self.rx, self.eps, self.faces = np.asarray(s.rx, np.float64), eps, {}
        self.corner = np.asarray(verts, np.float64)[np.asarray(s.tris)]
        self.of_face = np.argsort(s.tri_face, kind="stable")
        self.start = np.searchsorted(np.asarray(s.tri_face)[self.of_face], np.arange(s.n_faces + 1))

    def face(self, f):
        """Unit normal, offset and triangles (on the two axes kept) of face f."""
        if f not in self.faces:
            t = self.corner[self.of_face[self.start[f]:self.start[f + 1]]]
            nrm = np.cross(t[:, 1] - t[:, 0], t[:, 2] - t[:, 0])
            best = np.argmax(np.linalg.norm(nrm, axis=1))
            n = nrm[best] / np.linalg.norm(nrm[best])
            keep = [a for a in range(3) if a != np.argmax(np.abs(n))]
            self.faces[f] = (n, float(n @ t[best, 0]), t[:, :, keep], keep)
        return self.faces[f]

    def survivors(self, T, series):
        """The receivers whose points of the series lie well inside."""
        im = [np.asarray(T, np.float64)]
        for f in series:
            n, w = self.face(f)[:2]
            im.append(im[-1] - 2.0 * (im[-1] @ n - w) * n)
        Q, ok = self.rx, np.ones(len(self.rx), bool)
        for j in range(len(series), 0, -1):
            n, w, tri, keep = self.face(series[j - 1])
            D = im[j] - Q
            with np.errstate(divide="ignore", invalid="ignore"):
                u = (w - Q @ n) / (D @ n)
                Q = Q + u[:, None] * D
                ok &= (u > self.eps) & (u < 1.0 - self.eps)
                p = Q[:, keep]
                inside = np.zeros(len(Q), bool)
                for t in tri:
                    area = cross2(t[1] - t[0], t[2] - t[0])
                    if area != 0.0:
                        e = [cross2(t[(k + 1) % 3] - t[k], p - t[k]) / area for k in range(3)]
                        inside |= np.min(e, axis=0) > self.eps
            ok &= inside
        return np.flatnonzero(ok)


def check(s, K, frame=0, dirs=None, n=None):
    tx = np.asarray(s.tx, np.float32)
    s = scenes.Scene(**{**s.__dict__, "max_reflections": K, **({"n_rays": n} if n else {})})
    n = n if dirs is None else len(dirs)
    ctx = dcem.Context(0)
    ctx.scene_upload(s)
    dcem.trace_scene_frame(ctx, s, frame=frame, ray_dirs=dirs, record_trace_log=True,
                           discovery=dcem.DISCOVER_VISITED)
    p = ctx.paths()
    tri = ctx.trace_log()[0].reshape(len(tx), n, K + 1)[..., :K]
    face = np.where(tri >= 0, np.asarray(s.tri_face)[np.maximum(tri, 0)], -1)
    first, items = lowest_rays(face, K), list_length(face, ctx.ray_dirs(), K)
    found = set()
    for key, ray in zip(p["keys"].tolist(), p["first_ray"].tolist()):
        if key[2]:
            series = (key[0],) + tuple(key[3:3 + key[2]])
            assert ray == first[series], (key, ray, first[series])
            found.add(series + (key[1],))
        else:
            assert ray == -1
    walk = Walk(s, ctx.vertices())
    must = {series + (int(r),) for series in first for r in walk.survivors(tx[series[0]], series[1:])}
    print(s.name, n, K, "items", items, "series", len(first), "candidates", len(found), "of them away from edges", len(must), flush=True)
    ctx.close()
    assert must <= found, sorted(must - found)[:5]
    assert len(must) >= 0.9 * len(found)
    return items, len(must)


@pytest.mark.parametrize("frame,n,two", [(0, 60_000, True), (1, 1 << 14, False), (1, 1 << 15, False)])
def test_urban(frame, n, two):
    s = scenes.dynamic_urban()
    tx = np.asarray(s.tx, np.float32)[:1]
    if two:
        tx = np.concatenate([tx, tx + np.float32([3.0, -2.0, 1.0])])
    s = scenes.Scene(**{**s.__dict__, "tx": tx})
    items, n_must = check(s, 4, frame, n=n)
    # one workgroup sorts 16384 items
    assert n_must > 1000 and (items > 17000 if two else items < 16000 or n > 1 << 14)


@pytest.mark.parametrize("n", [2, 3, 64, 65, 130])
def test_corner(n):
    """Each wavefront's first lane and the lanes after it, whatever face they hit."""
    s = scenes.corner([[5.0, 4.0, 3.0]], np.float32([[20.0, 3.0, 1.5], [4.0, 30.0, 2.0], [9.0, 9.0, 4.0]]))
    assert sum(check(s, 3, dirs=scenes.random_sphere_dirs(n, seed=q))[0] for q in range(700, 712)) > 12
