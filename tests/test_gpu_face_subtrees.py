"""GPU: in a tree with the objects apart, faces whose centres share a Morton cell
stay in one run of leaves each, however many they are: coincident sheets, details of a
site on a ground far wider, moving objects beside them, a finely tessellated face; and
after the subtrees are ordered again."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes
from tests.bvh_check import check_bvh

pytestmark = pytest.mark.gpu


def build(n_boxes=0, n_sheets=0, ground=60.0, objects=0, grid=0):
    rng = np.random.default_rng(5)
    mb = scenes._MeshBuilder()
    mb.add_ground(ground, material=0)
    for k in range(n_sheets):
        x = 10.0 + 1e-3 * k
        mb.add_polygon_face([[x, -5, 0], [x, 5, 0], [x, 5, 8], [x, -5, 8]], [[0, 1, 2], [0, 2, 3]], material=0)
    for _ in range(n_boxes):
        c, w = rng.uniform(-50, 50, 2), rng.uniform(1, 4, 3)
        mb.add_box([c[0] - w[0], c[1] - w[1], 0.01], [c[0] + w[0], c[1] + w[1], w[2]], (1, 1, 1), 0)
    if grid:
        mb.add_polygon_face(*scenes._quad_grid([-30, -30, 20], [30, -30, 20], [-30, 30, 20], grid, grid), 0)
    for o in range(objects):
        mb.add_box([-20.0 + 3 * o, -40, 0.2], [-18.0 + 3 * o, -36, 1.8], (2, 2, 2), 0, o)
    return mb.finish("faces", [scenes.CONCRETE], [[0.0, 0.0, 9.0]], [[-20.0, 3.0, 1.5], [5.0, -4.0, 2.0]],
                     rx_radius=1.0, n_rays=3000, max_reflections=2)


CASES = {"sheets_16": dict(n_sheets=16), "sheets_40": dict(n_sheets=40), "site": dict(n_boxes=60, ground=20_000.0),
         "site_objects": dict(n_boxes=60, ground=20_000.0, objects=5),
         "site_grid": dict(n_boxes=40, ground=20_000.0, objects=2, grid=50)}


@pytest.mark.parametrize("name", list(CASES))
def test_one_run_per_face(name):
    s = build(**CASES[name])
    ctx = dcem.Context(0)
    ctx.scene_upload(s)
    pad = np.float32(4e-6 * (2.0 * float(np.abs(s.vertices).max()) + 1.0))
    for again in range(1 + (s.n_objects > 0)):
        if again:
            ctx.refit_bvh(subtrees=True)
        child, box, leaf_tri = ctx.bvh()
        assert check_bvh(child, box, leaf_tri, ctx.vertices(), s.tris, pad=pad, exact=True) == []
        face = s.tri_face[leaf_tri]
        runs = 1 + int((face[1:] != face[:-1]).sum())
        print(name, again, s.n_tris, "triangles", s.n_faces, "faces", runs, "runs", flush=True)
        assert runs == s.n_faces
    got = []
    for rebuild in (False, True):
        if rebuild:
            ctx.refit_bvh(force_rebuild=True)
        ctx.trace_frame(**dcem.scene_frame_args(s))
        got.append(ctx.received_power() + tuple(v for _, v in sorted(ctx.paths().items())))
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    ctx.close()
