"""GPU: the refinement's two kernels (a block per candidate; four candidates per
wavefront for lists expected to be longer than 4096) give the same bits.  A first
frame's list is sized by its captures, later ones by the last frame's
candidates, so a frame with more captures than 4096 and fewer candidates takes
both kernels in turn."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes

pytestmark = pytest.mark.gpu

CASES = {"toy": (scenes.static_toy, dict(rx_radius=4.0, n_rays=200_000, max_reflections=4)),
         "urban": (scenes.dynamic_urban, dict(rx_radius=2.0, n_rays=1 << 19, freqs_hz=[28e9, 3.5e9, 60e9])),
         "no_reflection": (scenes.static_toy, dict(rx_radius=8.0, n_rays=400_000, max_reflections=0)),
         "office": (scenes.indoor_office, dict(n_rays=6000))}


@pytest.mark.parametrize("name", list(CASES))
def test_both_kernels(name):
    make, change = CASES[name]
    s = make()
    s = scenes.Scene(**{**s.__dict__, **change})
    ctx = dcem.Context(0)
    ctx.scene_upload(s)
    got = []
    for _ in range(2):
        ctx.trace_frame(**dcem.scene_frame_args(s))
        st = ctx.stats()
        print(name, "captures", st["captures"], "candidates", st["unique_candidates"], flush=True)
        assert st["captures"] > 4096 > st["unique_candidates"]
        got.append(ctx.received_power() + tuple(v for _, v in sorted(ctx.paths().items())))
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    assert got[0][0].any()
    ctx.close()
