"""GPU: which faces can move is told by the span of the objects' vertex ranges and a
flag for each vertex in it: static vertices before, between and after the ranges, an
object without vertices, static faces on moving vertices in either of two objects.
Refitted frames equal those of a rebuilt tree bitwise, the tree's boxes hold exactly."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes
from tests.bvh_check import check_bvh

pytestmark = pytest.mark.gpu


def build(shared):
    mb = scenes._MeshBuilder()
    mb.add_ground(80.0, material=0)
    for k in range(40):
        mb.add_box([-60 + 3 * k, 20, 0], [-58 + 3 * k, 24, 6], (2, 2, 2), 0)
    for o in range(3):
        mb.add_box([-9 + 8 * o, -8, 1], [-6 + 8 * o, -5, 4], (2, 2, 2), 0, o)
        if o == 1:
            mb.object_ranges[1] = (mb.object_ranges[1][0],) * 2   # no vertices: its faces stay
        for k in range(20):
            mb.add_box([-60 + 6 * k, -30 - 5 * o, 0], [-57 + 6 * k, -28 - 5 * o, 5], (1, 1, 1), 0)

    def move(frame):
        xf = scenes.identity_transforms(3)
        xf[:, 1, 3] = 2.5 * frame
        xf[:, 2, 3] = 0.5 * frame
        return xf

    s = mb.finish("spans", [scenes.CONCRETE], [[0.0, 2.0, 9.0]], [[-20.0, 3.0, 1.5], [5.0, -4.0, 2.0]], rx_radius=2.0,
                  n_rays=4000, max_reflections=2, transforms_fn=move)
    fo = np.asarray(s.face_object).copy()
    if shared is not None:
        fo[np.flatnonzero(fo == shared)[:1]] = -1   # one face of the object is static geometry
    return scenes.Scene(**{**s.__dict__, "face_object": fo})


@pytest.mark.parametrize("shared", [None, 0, 2])
def test_refits(shared):
    s = build(shared)
    pad = np.float32(4e-6 * (2.0 * float(np.abs(s.vertices).max()) + 1.0))
    a, b = dcem.Context(0), dcem.Context(0)
    for c in (a, b):
        c.scene_upload(s)
    for frame in range(3):
        got = []
        for c in (a, b):
            c.set_object_transforms(s.transforms(frame))
            c.refit_bvh(force_rebuild=c is b, threshold=float("inf"))
            c.trace_frame(**dcem.scene_frame_args(s))
            got.append(c.received_power() + tuple(v for _, v in sorted(c.paths().items())))
        assert check_bvh(*a.bvh(), a.vertices(), s.tris, pad=pad, exact=True) == []
        for x, y in zip(*got):
            assert np.array_equal(x, y)
        print(shared, frame, "paths", len(got[0][2]), flush=True)
    for c in (a, b):
        c.close()
