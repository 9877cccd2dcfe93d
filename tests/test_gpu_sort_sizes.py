"""GPU: the radix sort at the edges of its launches, through the trees and
candidate lists built on it.  One workgroup takes up to 16384 items, a launch
per pass tiles of 1024 up to 262144 items and of 2048 beyond.  A tree is only
sound if its keys are sorted; a candidate list must equal numpy's sort of its
rows."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes
from tests.bvh_check import check_bvh

pytestmark = pytest.mark.gpu


def _soup(n):
    """n triangles, a face each, at random places over a ground quad."""
    rng = np.random.default_rng(n)
    at = rng.uniform(-50.0, 50.0, (max(n - 2, 0), 1, 3)) + rng.uniform(-1.0, 1.0, (max(n - 2, 0), 3, 3))
    at[..., 2] = np.abs(at[..., 2])
    s = scenes.static_toy()
    ground = np.array([[-60, -60, 0], [60, -60, 0], [60, 60, 0], [-60, 60, 0]], np.float32)
    v = np.concatenate([at.reshape(-1, 3).astype(np.float32), ground])
    k = 3 * at.shape[0]
    t = np.concatenate([np.arange(k).reshape(-1, 3), [[k, k + 1, k + 2], [k, k + 2, k + 3]]]).astype(np.int32)[-n:]
    f = np.arange(len(t), dtype=np.int32)
    return scenes.Scene(**{**s.__dict__, "name": "soup", "vertices": v, "tris": t, "tri_face": f,
                           "face_material": np.zeros(len(t), np.int32),
                           "face_object": np.full(len(t), -1, np.int32), "n_rays": 1000})


@pytest.mark.parametrize("n", [2, 63, 64, 65, 1024, 1025, 16383, 16384, 16385, 17408, 17409, 262145])
def test_tree_sizes(n):
    s = _soup(n)
    ctx = dcem.Context(0)
    ctx.scene_upload(s)
    pad = np.float32(4e-6 * (2.0 * float(np.abs(s.vertices).max()) + 1.0))
    assert check_bvh(*ctx.bvh(), ctx.vertices(), s.tris, pad=pad, exact=True) == []
    ctx.close()


# about 2.5k captures, de-duplicated without the sort; 4k, 17k, 100k and 400k
@pytest.mark.parametrize("radius,n", [(2.0, 240_000), (4.0, 100_000), (8.0, 100_000), (8.0, 600_000), (12.0, 1_000_000)])
def test_candidate_sizes(radius, n):
    s = scenes.static_toy()
    s = scenes.Scene(**{**s.__dict__, "rx_radius": radius, "n_rays": n, "max_reflections": 3})
    ctx = dcem.Context(0)
    ctx.scene_upload(s)
    ctx.trace_frame(**dcem.scene_frame_args(s))
    p, caps = ctx.paths(), ctx.captures()
    print("captures", len(caps), "candidates", len(p["keys"]), flush=True)
    # a candidate for every distinct (tx, rx, order, faces), in ascending order, with its lowest ray
    # (columns: ray, tx, rx, order, faces; the line of sight has no ray)
    ray = np.where(caps[:, 0] < 0, np.iinfo(np.int32).max, caps[:, 0])
    rows = np.concatenate([caps[:, 1:], ray[:, None]], axis=1)
    rows = rows[np.lexsort(rows.T[::-1])]
    head = np.r_[True, (rows[1:, :-1] != rows[:-1, :-1]).any(axis=1)]
    assert np.array_equal(p["keys"], rows[head, :-1])
    first = rows[head, -1]
    assert np.array_equal(p["first_ray"], np.where(first == np.iinfo(np.int32).max, -1, first))
    ctx.close()
