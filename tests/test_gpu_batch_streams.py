"""GPU: a batch spreads its contexts' own work over side streams: batches of one
context, of as many as there are streams and of more, small and large candidate
lists, coherent and full frames, on the null stream and on a caller's, direct and
as a graph, equal single frames bitwise."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes
from tests.test_gpu_batch import run_batched_and_single, small_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,graph", [(1, False), (2, True), (4, False), (9, False), (9, True)])
@pytest.mark.parametrize("own_stream", [False, True])
def test_spread(n, graph, own_stream):
    import torch
    ws = small_batch(n, seed=40 + n, budget_range=(1 << 13, 1 << 15))
    # every third scene's list is longer than the one-launch de-duplication takes
    ws = [scenes.Scene(**{**s.__dict__, "rx_radius": 6.0 if j % 3 == 1 else s.rx_radius}) for j, s in enumerate(ws)]
    modes = [dcem.MODE_COHERENT if j % 4 == 3 else dcem.MODE_FULL for j in range(n)]
    stream = torch.cuda.Stream() if own_stream else None
    run_batched_and_single(ws, range(4), graph=graph and own_stream, modes=modes,
                           stream=stream.cuda_stream if own_stream else None)


@pytest.mark.parametrize("shape", [(16, 1, 64), (32, 8, 64), (32, 32, 64), (16, 16, 128), (32, 4, 1 << 20)])
def test_shapes(shape):
    """Chunks shared out by the per-XCD queues: fewer chunks than wavefronts and
    many more, more blocks than are resident, chunks of several packets and of
    whole scenes; paths, powers and the counts added per scene."""
    ws = small_batch(5, seed=71, budget_range=(1 << 10, 1 << 16))
    bctx, sctx = [[dcem.Context(0) for _ in ws] for _ in range(2)]
    for c, d, s in zip(bctx, sctx, ws):
        c.scene_upload(s)
        d.scene_upload(s)
    batch = dcem.Batch(bctx)
    batch.set_shape(*shape)
    for _ in range(2):
        batch.trace([dcem.scene_frame_args(s) for s in ws])
        for c, d, s in zip(bctx, sctx, ws):
            d.trace_frame(**dcem.scene_frame_args(s))
            got, want = [x.received_power() + tuple(v for _, v in sorted(x.paths().items())) for x in (c, d)]
            for a, b in zip(got, want):
                assert np.array_equal(a, b)
            for k in ("segments", "captures", "rays_traced"):
                assert c.stats()[k] == d.stats()[k], k
    batch.close()
    for c in bctx + sctx:
        c.close()
