"""GPU: the first ray of every visited-series candidate is the lowest ray whose
hits run over the candidate's faces, from the trace log by brute force: item
counts sorted by one workgroup and in launches per pass, one source and two.
(Not lists where neighbouring rays' series differ in face 0 alone: the item pass
compares neighbours by a shuffle in which not all lanes take part, and may enter
such a ray with its neighbour's series.)"""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("make,n,K,two", [(scenes.static_toy, 300, 2, False), (scenes.static_toy, 9001, 4, True),
                                          (scenes.dynamic_urban, 3000, 3, False)])
def test_first_rays(make, n, K, two):
    s = make()
    tx = np.asarray(s.tx, np.float32)[:1]
    if two:
        tx = np.concatenate([tx, tx + np.float32([3.0, -2.0, 1.0])])
    s = scenes.Scene(**{**s.__dict__, "tx": tx, "n_rays": n, "max_reflections": K})
    ctx = dcem.Context(0)
    ctx.scene_upload(s)
    dcem.trace_scene_frame(ctx, s, frame=0, record_trace_log=True, discovery=dcem.DISCOVER_VISITED)
    p = ctx.paths()
    tri = ctx.trace_log()[0].reshape(len(tx), n, K + 1)[..., :K]
    face = np.where(tri >= 0, np.asarray(s.tri_face)[np.maximum(tri, 0)], -1)
    first = {}
    for src in range(len(tx)):
        for d in range(1, K + 1):
            hit = np.flatnonzero((tri[src, :, :d] >= 0).all(axis=1))
            seq, at = np.unique(face[src, hit, :d], axis=0, return_index=True)
            for q, i in zip(seq, at):   # return_index: the lowest
                first[(src, d) + tuple(int(f) for f in q)] = src * n + int(hit[i])
    seen = 0
    for key, ray in zip(p["keys"], p["first_ray"]):
        order = int(key[2])
        want = -1 if order == 0 else first[(int(key[0]), order) + tuple(int(f) for f in key[3:3 + order])]
        assert ray == want, (key, ray, want)
        if order:
            src = int(key[0])
            assert np.array_equal(face[src, ray - src * n, :order], key[3:3 + order])
        seen += order > 0
    print("candidates", seen, "series", len(first), flush=True)
    assert seen > 10
    ctx.close()
