"""GPU: trees built from the face-coded keys, at the edges of their layout:
one face, more coincident faces than the code tells apart, no moving objects,
one object and many.  The tree's invariants hold exactly, and a frame's powers
and paths equal those on the one-curve tree of a forced rebuild bitwise."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes
from tests.bvh_check import check_bvh

pytestmark = pytest.mark.gpu


def _sheets(n):
    """n facing quads pairwise 1 mm apart, all centred on one Morton cell."""
    mb = scenes._MeshBuilder()
    mb.add_ground(60.0, material=0)
    for k in range(n):
        x = 10.0 + 1e-3 * k
        mb.add_polygon_face([[x, -5, 0], [x, 5, 0], [x, 5, 8], [x, -5, 8]], [[0, 1, 2], [0, 2, 3]], material=0)
    return mb.finish("sheets", [scenes.CONCRETE], [[0.0, 0.0, 5.0]], [[-20.0, 3.0, 1.5], [5.0, -4.0, 2.0]],
                     rx_radius=1.0, n_rays=3000, max_reflections=2)


CASES = {"one_face": lambda: scenes.single_wall([[0.0, 0.0, 1.0]], [[3.0, 4.0, 2.0]], n_rays=3000),
         "coincident_15": lambda: _sheets(15), "coincident_16": lambda: _sheets(16),
         "coincident_40": lambda: _sheets(40), "office": lambda: scenes.indoor_office(n_rays=3000),
         "one_object": lambda: scenes.box_field(5, 1, n_rays=3000),
         "objects_257": lambda: scenes.box_field(30, 257, n_rays=3000)}


@pytest.mark.parametrize("name", list(CASES))
def test_tree_and_frame(name):
    s = CASES[name]()
    ctx = dcem.Context(0)
    ctx.scene_upload(s)
    pad = np.float32(4e-6 * (2.0 * float(np.abs(s.vertices).max()) + 1.0))
    assert check_bvh(*ctx.bvh(), ctx.vertices(), s.tris, pad=pad, exact=True) == []
    got = []
    for rebuild in (False, True):
        if rebuild:
            rb, _ = ctx.refit_bvh(force_rebuild=True)
            assert rb == dcem.REBUILT_FULL
            assert check_bvh(*ctx.bvh(), ctx.vertices(), s.tris, pad=pad, exact=True) == []
        ctx.trace_frame(**dcem.scene_frame_args(s))
        got.append(ctx.received_power() + tuple(v for _, v in sorted(ctx.paths().items())))
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    ctx.close()
