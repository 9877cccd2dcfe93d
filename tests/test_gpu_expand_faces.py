"""GPU: the visited series' expansion shares the triangles of a face among 16
lanes: faces of 2 triangles to more than the lanes, ragged and whole multiples,
walls with a notch that only the triangle test sees, against the oracle."""
import numpy as np
import pytest

from paper_2112_07115_amd import scenes
from tests.gpu_frames import assert_comparable, run_pair

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def O():
    from oracle import oracle
    oracle.build()
    return oracle


def _street(cells):
    """Two facing blocks tessellated into `cells`, and a notched wall (an L of
    2 (cells + 2) triangles: points in its bounds may lie outside it)."""
    mb = scenes._MeshBuilder()
    mb.add_ground(60.0, material=0)
    mb.add_box((-20, 10, 0), (20, 14, 9), cells, 0)
    mb.add_box((-20, -14, 0), (20, -10, 9), cells, 0)
    n = sum(cells)
    z = np.linspace(0.0, 9.0, n + 1)
    pts, tris = [], []
    for i in range(n):
        y1 = 8.0 if z[i] < 4.0 else 1.0
        b = len(pts)
        pts += [[25.0, -8.0, z[i]], [25.0, y1, z[i]], [25.0, y1, z[i + 1]], [25.0, -8.0, z[i + 1]]]
        tris += [[b, b + 1, b + 2], [b, b + 2, b + 3]]
    mb.add_polygon_face(pts, tris, material=0)
    rx = [[x, y, 1.5] for x in (-15.0, -4.0, 9.0, 18.0) for y in (-6.0, 0.5, 7.0)]
    return mb.finish("street", [scenes.CONCRETE], [[3.0, 1.0, 5.0]], rx, rx_radius=1.0, n_rays=4000,
                     max_reflections=2)


@pytest.mark.parametrize("cells", [(1, 1, 1), (3, 1, 2), (8, 1, 1), (8, 1, 3), (17, 2, 3)])
@pytest.mark.parametrize("backward", [False, True])
def test_tessellated_faces(O, cells, backward):
    from paper_2112_07115_amd import dcem
    ctx = dcem.Context(0)
    s = _street(cells)
    st, out, ofr = run_pair(ctx, O, s, n_rays=400 if backward else None, visited=True, backward=backward)
    assert_comparable(st)
    assert ctx.paths()["valid"].sum() > 20
    ctx.close()
