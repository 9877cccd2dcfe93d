"""GPU: a packet's rays need more stack entries together than each by itself, and the
capture spheres' tree more than the scene's: with the stacks limited to what single
rays of the scene need at most (found by lowering the limit on a traversal of one ray
per lane), the frame is the unlimited one's; with one entry it is refused."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes

pytestmark = pytest.mark.gpu


def ground(x):
    g = np.stack(np.meshgrid(np.arange(64), np.arange(64)), -1).reshape(-1, 2) * 2.0 - 64
    return scenes.ground_only([[x, 0.2, 2.2]], np.c_[g, np.full(4096, 2.0)].astype(np.float32), rx_radius=1.2,
                              n_rays=1 << 14)


CASES = {"office": (lambda: scenes.indoor_office(n_rays=1 << 14), 8),
         "city": (lambda: scenes.ragged_city(3, 60_000, n_rays=1 << 16), 11),
         "spheres": (lambda: ground(0.3), 11), "far_spheres": (lambda: ground(-300.3), 7)}


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("how", ["frame", "batch"])
def test_what_one_ray_needs(case, how):
    make, limit = CASES[case]
    s = make()
    ctxs = [dcem.Context(0) for _ in range(2)]
    for c in ctxs:
        c.scene_upload(s)
    batch = dcem.Batch(ctxs) if how == "batch" else None

    def frame():
        if batch:
            batch.trace([dcem.scene_frame_args(s)] * 2)
        else:
            ctxs[0].trace_frame(**dcem.scene_frame_args(s))
        return ctxs[0].received_power() + tuple(v for _, v in sorted(ctxs[0].paths().items()))

    want = frame()
    for n in (limit, limit + 1, 40):
        print(case, how, "limit", n, flush=True)
        for c in ctxs:
            c.set_stack_limit(n)
        for a, b in zip(frame(), want):
            assert np.array_equal(a, b)
    if case in ("office", "city"):
        for c in ctxs:
            c.set_stack_limit(1)
        with pytest.raises(dcem.DcemError) as e:
            frame()
        assert e.value.status == dcem.E_CAPACITY
    if batch:
        batch.close()
    for c in ctxs:
        c.close()
