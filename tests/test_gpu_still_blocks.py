"""GPU: refits that leave out blocks of leaves none of which can move: nothing
moves, a few objects among many blocks, every block moving, objects on block
edges, static faces that use a moving object's vertices.  After each refit the
tree's boxes hold exactly and the frame equals that of a rebuilt tree bitwise;
the SAH ratio is that of a tree refitted whole."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes
from tests.bvh_check import check_bvh

pytestmark = pytest.mark.gpu

CASES = {"no_objects": lambda: scenes.box_field(200, 0, n_rays=2000),
         "one_among_many": lambda: scenes.box_field(900, 1, n_rays=2000),
         "few": lambda: scenes.box_field(700, 5, n_rays=2000),
         "all": lambda: scenes.box_field(0, 300, n_rays=2000),
         "one_block": lambda: scenes.box_field(20, 3, half=30.0, n_rays=2000),
         "static_shares_vertices": lambda: scenes.box_field(400, 4, n_rays=2000)}


@pytest.mark.parametrize("name", list(CASES))
def test_refits(name):
    s = CASES[name]()
    if name == "static_shares_vertices":
        # the first object's faces belong to the static geometry, its vertices still move
        fo = np.asarray(s.face_object).copy()
        fo[fo == 0] = -1
        s = scenes.Scene(**{**s.__dict__, "face_object": fo})
    pad = np.float32(4e-6 * (2.0 * float(np.abs(s.vertices).max()) + 1.0))
    a, b = dcem.Context(0), dcem.Context(0)
    for c in (a, b):
        c.scene_upload(s)
        c.refit_bvh()
    for frame in range(3):
        a.set_object_transforms(s.transforms(frame))
        a.refit_bvh(threshold=float("inf"))
        b.set_object_transforms(s.transforms(frame))
        b.refit_bvh(force_rebuild=True)
        assert check_bvh(*a.bvh(), a.vertices(), s.tris, pad=pad, exact=True) == []
        got = []
        for c in (a, b):
            c.trace_frame(**dcem.scene_frame_args(s))
            got.append(c.received_power() + tuple(v for _, v in sorted(c.paths().items())))
        for x, y in zip(*got):
            assert np.array_equal(x, y)
        # the surface areas of the refitted tree, from its boxes
        child, box, _ = a.bvh()
        d = box[..., 3:].astype(np.float64) - box[..., :3]
        area = 2.0 * (d[..., 0] * d[..., 1] + d[..., 1] * d[..., 2] + d[..., 2] * d[..., 0])
        lo, hi = box[0, :, :3].min(axis=0).astype(np.float64), box[0, :, 3:].max(axis=0).astype(np.float64)
        e = hi - lo
        root = 2.0 * (e[0] * e[1] + e[1] * e[2] + e[2] * e[0])
        sah = (area[child >= 0].sum() + root) / root
        if frame == 0:
            first = sah
        want = sah / first
        have = a.stats()["sah_ratio"]
        print(name, "frame", frame, "sah", have, want, flush=True)
        if frame == 0:
            first_have = have
        assert abs(have / first_have - want) < 1e-9
    for c in (a, b):
        c.close()
