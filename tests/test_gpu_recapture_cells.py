"""GPU: the captures of kept segments when receivers move, at the edges of the
receivers' grid: one receiver, all on one line along x or along y, one column of
heights, a wide field with large spheres, ragged ray counts.  Coherent frames
equal full traces bitwise."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes

pytestmark = pytest.mark.gpu

N = 40
T = np.linspace(-60.0, 60.0, N)
LAYOUTS = {"one": [[10.0, -35.0, 1.5]],
           "line_x": np.stack([T, np.full(N, 5.0), np.full(N, 1.5)], 1),
           "line_y": np.stack([np.full(N, -3.0), T, np.full(N, 1.5)], 1),
           "column": np.stack([np.full(N, 30.0), np.full(N, 2.0), np.linspace(1.0, 40.0, N)], 1),
           "field": np.stack([80.0 * np.sin(3.0 * np.arange(300)), 80.0 * np.cos(5.0 * np.arange(300)),
                              1.0 + np.arange(300) % 7], 1)}


@pytest.mark.parametrize("layout", list(LAYOUTS))
@pytest.mark.parametrize("radius,n", [(0.5, 20_001), (6.0, 4_000)])
def test_moved_receivers(layout, radius, n):
    s = scenes.box_field(40, 6, half=80.0, n_rays=n)
    rx0 = np.asarray(LAYOUTS[layout], np.float32)
    coh, full = dcem.Context(0), dcem.Context(0)
    for c in (coh, full):
        c.scene_upload(s)
    captures = 0
    for frame in range(4):
        rx = rx0 + np.float32(0.7 * frame) * np.array([1.0, -0.5, 0.1], np.float32)
        got = []
        for c, mode in ((coh, dcem.MODE_COHERENT), (full, dcem.MODE_FULL)):
            c.set_object_transforms(s.transforms(frame))
            c.refit_bvh()
            c.trace_frame(s.tx, rx, radius, n, max_reflections=3, freqs_hz=s.freqs_hz, mode=mode)
            got.append(c.received_power() + tuple(v for _, v in sorted(c.paths().items())))
            st = c.stats()
        for a, b in zip(*got):
            assert np.array_equal(a, b)
        captures += st["captures"]
        print(layout, radius, "frame", frame, "captures", st["captures"], flush=True)
    # (each frame holds the line of sight of every receiver)
    assert coh.stats()["coherent"] == 1 and captures > 4 * len(rx0)
    for c in (coh, full):
        c.close()
