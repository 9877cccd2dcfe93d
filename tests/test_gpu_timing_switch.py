"""GPU: stage timings switched on or off at any point between two calls: the calls go on
and give the same powers (a stage that was not timed reads 0)."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("at", range(6))
@pytest.mark.parametrize("rebuild", [False, True])
def test_switch(at, rebuild):
    s = scenes.box_field(30, 3, half=60.0, n_rays=2000)
    ctx, ref = dcem.Context(0), dcem.Context(0)
    for c in (ctx, ref):
        c.scene_upload(s)
    on = False
    for frame in range(4):
        for c in (ctx, ref):
            mode = dcem.MODE_COHERENT
            steps = [lambda: c.set_object_transforms(s.transforms(frame)),
                     lambda: c.refit_bvh(force_rebuild=rebuild, threshold=float("inf")),
                     lambda: c.trace_frame(**dcem.scene_frame_args(s, frame=frame, mode=mode)),
                     lambda: c.stats(), lambda: c.received_power(), lambda: c.paths()]
            for i, step in enumerate(steps):
                if c is ctx and i == at:
                    on = not on
                    ctx.set_timing(on)
                step()
        for a, b in zip(ctx.received_power(), ref.received_power()):
            assert np.array_equal(a, b)
        st = ctx.stats()
        print(at, rebuild, frame, on, {k: round(v, 3) for k, v in st.items() if k.startswith("ms_")}, flush=True)
        assert all(v >= 0 for k, v in st.items() if k.startswith("ms_"))
    for c in (ctx, ref):
        c.close()
