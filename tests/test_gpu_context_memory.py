"""GPU: what a context holds for its traversal stacks does not pay for what its frames
do not use: a small frame's buffers, and moved receivers of more than the tree walk
keeps in LDS (their spill space is sized by the tree), coherent frames against full."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes

pytestmark = pytest.mark.gpu


def test_small_frame():
    s = scenes.static_toy()
    ctx = dcem.Context(0)
    ctx.set_capture_capacity(1 << 16)
    ctx.scene_upload(s)
    dcem.trace_scene_frame(ctx, s, mode=dcem.MODE_COHERENT)
    held = sum(ctx.allocator.live.values())
    print("held", held, flush=True)
    # 2 MB beside the stacks; 32 entries of 4 B for each of the 262144 threads of four
    # blocks of 256 on each of 256 compute units
    assert held < 2 * 2**20 + 4 * 32 * 262144
    ctx.close()


@pytest.mark.parametrize("n_rx", [1, 4, 5, 4096, 4097, 40_000])
def test_moved_receivers(n_rx):
    s = scenes.box_field(30, 3, half=60.0, n_rays=20_000)
    rng = np.random.default_rng(n_rx)
    rx0 = (rng.uniform(-50, 50, (n_rx, 3)) * [1, 1, 0.1] + [0, 0, 6]).astype(np.float32)
    coh, full = dcem.Context(0), dcem.Context(0)
    for c in (coh, full):
        c.scene_upload(s)
    for frame in range(3):
        rx, got = rx0 + np.float32([0.4, -0.3, 0.1]) * np.float32(frame), []
        for c, mode in ((coh, dcem.MODE_COHERENT), (full, dcem.MODE_FULL)):
            c.set_object_transforms(s.transforms(frame))
            c.refit_bvh()
            c.trace_frame(s.tx, rx, 1.0, 20_000, max_reflections=2, freqs_hz=s.freqs_hz, mode=mode)
            got.append(c.received_power() + tuple(v for _, v in sorted(c.paths().items())))
        for a, b in zip(*got):
            assert np.array_equal(a, b)
        print(n_rx, frame, full.stats()["captures"], flush=True)
    assert coh.stats()["coherent"] == 1
    for c in (coh, full):
        c.close()
