"""GPU: the packet trace at the edges of its packets: ray counts around the
packet sizes (packets of 64 rays shrink to 4 while a launch would leave the chip
idle), coherent (Fibonacci) and incoherent (random) rays against the oracle, and
lists of re-traced rays, whose lanes start at different segments, against full
traces bitwise."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes
from tests.gpu_frames import assert_comparable, log, run_pair
from tests.test_gpu_coherence import assert_same, frame_outputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def O():
    from oracle import oracle
    oracle.build()
    return oracle


# one ray; one packet less a ray; just above 4096 packets of 4, 16 and 32 rays;
# more than 4096 packets of 64
@pytest.mark.parametrize("n", [1, 3, 255, 4 * 4096 + 1, 16 * 4096 + 1, 32 * 4096 + 3, 64 * 4096 + 63])
@pytest.mark.parametrize("random", [False, True])
def test_ray_counts(O, n, random):
    ctx = dcem.Context(0)
    s = scenes.static_toy()
    dirs = scenes.random_sphere_dirs(n, seed=n) if random else None
    st, out, ofr = run_pair(ctx, O, s, dirs=dirs, n_rays=None if random else n)
    assert_comparable(st)
    ctx.close()


@pytest.mark.parametrize("n", [(1 << 16) + 1, 1 << 18])
def test_long_lists(n):
    """Every box of a dense field moves; launches sized for lists longer than the group trace takes."""
    s = scenes.box_field(100, 257, half=30.0, n_rays=n)
    full, coh = dcem.Context(0), dcem.Context(0)
    for c in (full, coh):
        c.scene_upload(s)
    for frame in range(3):
        dcem.trace_scene_frame(full, s, frame=frame, rebuild=True, record_trace_log=True)
        dcem.trace_scene_frame(coh, s, frame=frame, mode=dcem.MODE_COHERENT, record_trace_log=True)
        assert_same(frame_outputs(full), frame_outputs(coh))
        st = coh.stats()
        log("frame", frame, "traced", st["rays_traced"], "of", n)
        # the first coherent frame sizes its launch for a list of all rays
        assert frame == 2 or st["trace_kernel"] == 0
    full.close()
    coh.close()
