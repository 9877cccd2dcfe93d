"""GPU: sources (and branches) of fewer rays than a wavefront has lanes are traced
together: every ray of a frame of many sources equals the ray of its source traced
alone, bitwise, with the segment cache and coherent frames after it, in a batch, backward,
and with transmission branches."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes

pytestmark = pytest.mark.gpu


def outputs(c):
    return c.received_power() + c.trace_log() + tuple(v for _, v in sorted(c.paths().items()))


def same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y, equal_nan=True)


@pytest.mark.parametrize("n_src,n", [(2, 1), (70, 1), (9, 7), (300, 16), (5, 63), (5, 64)])
@pytest.mark.parametrize("backward", [False, True])
def test_each_source_alone(n_src, n, backward):
    s = scenes.static_toy()
    rng = np.random.default_rng(n_src)
    src = (rng.uniform(-40, 40, (n_src, 3)) * [1, 1, 0.1] + [0, 0, 6]).astype(np.float32)
    dirs = scenes.random_sphere_dirs(n, seed=n)

    def trace(c, at):
        tx, rx = (s.rx[:4], at) if backward else (at, s.rx)
        c.trace_frame(tx, rx, 2.0, n, ray_dirs=dirs, max_reflections=3, record_trace_log=True, trace_from_rx=backward)
        caps = c.captures()
        return c.trace_log(), caps[np.lexsort(caps.T[::-1])]

    ctx = dcem.Context(0)
    ctx.scene_upload(s)
    log, caps = trace(ctx, src)
    total = 0
    for j in range(0, n_src, max(1, n_src // 5)):
        one, oc = trace(ctx, src[j:j + 1])
        same([x[j:j + 1] for x in log], one)
        total += len(oc)
        if not backward:   # this source's records, its rays counted from its first
            mine = caps[(caps[:, 0] >= j * n) & (caps[:, 0] < (j + 1) * n)]
            assert len(mine) == (oc[:, 0] >= 0).sum()
    print(n_src, n, backward, "captures", len(caps), "of sources alone", total, flush=True)
    ctx.close()


@pytest.mark.parametrize("n", [3, 63])
@pytest.mark.parametrize("graph", [False, True])
def test_cache_and_batch(n, graph):
    import torch
    s = scenes.dynamic_urban()
    tx = np.asarray(s.tx, np.float32)[:1] + np.float32([[2 * j, j % 3, 0] for j in range(40)])
    s = scenes.Scene(**{**s.__dict__, "tx": tx, "n_rays": n, "rx_radius": 4.0})
    stream = torch.cuda.Stream()
    coh, full, b0, b1 = ctxs = [dcem.Context(0, stream=stream.cuda_stream) for _ in range(4)]
    for c in ctxs:
        c.scene_upload(s)
    batch = dcem.Batch([b0, b1])
    batch.set_graph(graph)
    for frame in range(4):
        for c in ctxs:
            c.set_object_transforms(s.transforms(frame))
            c.refit_bvh(threshold=float("inf"))
        args = [dcem.scene_frame_args(s, mode=m, record_trace_log=True) for m in (dcem.MODE_COHERENT, dcem.MODE_FULL)]
        coh.trace_frame(**args[0])
        full.trace_frame(**args[1])
        batch.trace(args)
        want = outputs(full)
        for c in (coh, b0, b1):
            same(outputs(c), want)
        for k in ("segments", "captures", "rays_traced"):
            assert b1.stats()[k] == full.stats()[k]
    assert coh.stats()["coherent"] == 1 and coh.stats()["rays_traced"] < 40 * n
    assert batch.info()["graph_frames"] >= (3 if graph else 0)
    batch.close()
    for c in ctxs:
        c.close()


@pytest.mark.parametrize("n", [1, 17, 63])
def test_branches(n):
    s = scenes.indoor_office()
    dirs = scenes.random_sphere_dirs(64, seed=5)
    logs = []
    ctx = dcem.Context(0)
    ctx.scene_upload(s)
    for k in (n, 64):   # mixed, then in packets
        dcem.trace_scene_frame(ctx, s, ray_dirs=dirs[:k], record_trace_log=True)
        logs.append([x.reshape(-1, k, x.shape[-1])[:, :n] for x in ctx.trace_log()])
    assert len(logs[0][0]) > 1
    same(*logs)
    ctx.close()
