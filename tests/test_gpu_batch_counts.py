"""GPU: the item counts of a frame are its own: a context whose trace launch left
counts per block, then a frame of a batch without rays or with few, and back."""
import pytest

from paper_2112_07115_amd import dcem, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ctx", [1, 3])
@pytest.mark.parametrize("n", [0, 100])
def test_counts_of_this_frame(n_ctx, n):
    s = scenes.static_toy()
    ctxs = [dcem.Context(0) for _ in range(n_ctx)]
    for c in ctxs:
        c.scene_upload(s)
        c.trace_frame(**dcem.scene_frame_args(s))   # its own launch
        assert c.stats()["segments"] > s.n_rays
    batch = dcem.Batch(ctxs)
    few = dcem.scene_frame_args(scenes.Scene(**{**s.__dict__, "n_rays": n}))
    for frames in ([few] * n_ctx, [dcem.scene_frame_args(s)] * n_ctx, [few] * n_ctx):
        batch.trace(frames)
        for c, f in zip(ctxs, frames):
            st = c.stats()
            rays, top = f["n_rays"], f["n_rays"] * (s.max_reflections + 1)
            print(n_ctx, rays, {k: st[k] for k in ("segments", "nodes_visited", "tri_tests")}, flush=True)
            assert rays <= st["segments"] <= top
            assert (st["nodes_visited"] > 0) == (st["tri_tests"] > 0) == (rays > 0)
    batch.close()
    for c in ctxs:
        c.trace_frame(**few)   # a launch of its own without rays
        assert c.stats()["segments"] <= n * (s.max_reflections + 1)
        c.close()
