"""GPU: a frame whose buffers cannot be allocated (an allocator that says so at the k-th
request, for every k) is reported as out of memory and leaves no frame: results are refused
until one is traced, refits and trees go on, and the same call then gives what a fresh
context gives, coherent frames after it too."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes

pytestmark = pytest.mark.gpu


class Failing:
    """torch's allocator, failing every request after `left` more (None: never)."""

    def __init__(self):
        base = dcem.TorchAllocator(0)
        self.left, self.refused = None, 0

        def alloc(n, stream, user):
            if self.left is not None:
                if self.left == 0:
                    self.refused += 1
                    return None
                self.left -= 1
            return base._alloc(n, stream, user)

        self._alloc, self._base = dcem._ALLOC_FN(alloc), base
        self.desc = dcem.AllocatorDesc(self._alloc, base._free, None)


def outputs(c):
    return c.received_power() + tuple(v for _, v in sorted(c.paths().items())) + c.trace_log()


def refused(c):
    for read in (c.received_power, c.paths, c.trace_log, c.stats, c.captures, c.power_gradients):
        with pytest.raises(dcem.DcemError) as e:
            read()
        assert e.value.status == dcem.E_STATE


@pytest.mark.parametrize("how", ["frame", "visited", "batch"])
def test_frame(how):
    s = scenes.box_field(40, 3, half=60.0, n_rays=500)
    rx = np.asarray(s.rx, np.float32)
    small = dict(tx=s.tx, rx=rx[:5], rx_radius=1.0, n_rays=500, max_reflections=1, freqs_hz=[28e9], record_trace_log=True,
                 mode=dcem.MODE_COHERENT)
    big = dict(tx=s.tx, rx=rx, rx_radius=2.0, n_rays=20_000, max_reflections=4, freqs_hz=[28e9, 60e9, 3e9],
               record_trace_log=True, mode=dcem.MODE_COHERENT,
               discovery=dcem.DISCOVER_VISITED if how == "visited" else 0)

    def move(c, frame):
        c.set_object_transforms(s.transforms(frame))
        c.refit_bvh(threshold=float("inf"))

    ref = dcem.Context(0)
    ref.scene_upload(s)
    want = []
    for frame in (1, 2):
        move(ref, frame)
        ref.trace_frame(**big)
        want.append(outputs(ref))
    k, done = 0, False
    while not done:
        al = Failing()
        c, other = dcem.Context(0, allocator=al), dcem.Context(0)
        batch = dcem.Batch([other, c]) if how == "batch" else None
        for x in (c, other):
            x.scene_upload(s)
            move(x, 0)
            x.trace_frame(**small)
            x.received_power()
            move(x, 1)
        al.left = k
        try:
            batch.trace([big, big]) if batch else c.trace_frame(**big)
            done = al.refused == 0
            assert done
        except dcem.DcemError as e:
            assert e.status == dcem.E_OUT_OF_MEMORY
            for x in (c, other) if batch else (c,):
                refused(x)
                move(x, 1)
                x.vertices(), x.bvh()
        al.left = None
        for f, frame in enumerate((1, 2)):
            if f:
                move(c, frame), move(other, frame)
            if f or not done:
                batch.trace([big, big]) if batch else c.trace_frame(**big)
            for x in (c, other) if batch else (c,):
                for a, b in zip(outputs(x), want[f]):
                    assert np.array_equal(a, b, equal_nan=True)
        assert c.stats()["coherent"] == 1
        k += 1
        if batch:
            batch.close()
        c.close(), other.close()
    print(how, "allocations", k - 1, flush=True)
    assert k > 10


def test_upload():
    """No scene is left by an upload that cannot allocate; the next one starts anew."""
    small, big = scenes.box_field(5, 2, n_rays=500), scenes.box_field(300, 20, n_rays=4000)
    args = dcem.scene_frame_args(big, record_trace_log=True)
    ref = dcem.Context(0)
    ref.scene_upload(big)
    ref.trace_frame(**args)
    want = outputs(ref)
    k, done = 0, False
    while not done:
        al = Failing()
        c = dcem.Context(0, allocator=al)
        c.scene_upload(small)
        c.trace_frame(**dcem.scene_frame_args(small, record_trace_log=True))
        c.received_power()
        al.left = k
        try:
            c.scene_upload(big)
            done = al.refused == 0
            assert done
        except dcem.DcemError as e:
            assert e.status == dcem.E_OUT_OF_MEMORY
            refused(c)
            for call in (lambda: c.trace_frame(**args), c.refit_bvh, c.vertices, c.bvh,
                         lambda: c.set_object_transforms(big.transforms(1))):
                with pytest.raises(dcem.DcemError) as e2:
                    call()
                assert e2.value.status == dcem.E_STATE
        al.left = None
        if not done:
            c.scene_upload(big)
        c.trace_frame(**args)
        for a, b in zip(outputs(c), want):
            assert np.array_equal(a, b, equal_nan=True)
        c.close()
        k += 1
    print("upload allocations", k - 1, flush=True)
    assert k > 10


def test_refused_upload_keeps_the_scene():
    """An upload with bad arguments changes nothing, a refit still to run included."""
    s = scenes.box_field(40, 3, half=60.0, n_rays=4000)
    bad = scenes.Scene(**{**s.__dict__, "tris": np.where(s.tris == 5, 10**6, s.tris).astype(np.int32)})
    got = []
    for upload in (False, True):
        c = dcem.Context(0)
        c.scene_upload(s)
        c.trace_frame(**dcem.scene_frame_args(s))
        c.received_power()
        c.set_object_transforms(s.transforms(3))
        c.refit_bvh(threshold=float("inf"))
        if upload:
            with pytest.raises(dcem.DcemError) as e:
                c.scene_upload(bad)
            assert e.value.status == dcem.E_INVALID_ARG
        _, box, _ = c.bvh()
        c.trace_frame(**dcem.scene_frame_args(s, record_trace_log=True))
        got.append((box,) + outputs(c))
        c.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b, equal_nan=True)


def test_refused_frames_keep_the_last():
    """Bad arguments of one context of a batch, or of a frame, change no context."""
    s = scenes.box_field(40, 3, half=60.0, n_rays=2000)
    ctxs = [dcem.Context(0) for _ in range(3)]
    batch = dcem.Batch(ctxs)
    good = dcem.scene_frame_args(s, record_trace_log=True)
    more = {**good, "max_reflections": 3, "n_rays": 9000, "freqs_hz": [28e9, 3e9]}
    for c in ctxs:
        c.scene_upload(s)
    batch.trace([good] * 3)
    want = outputs(ctxs[0])
    far = np.asarray(s.rx, np.float32).copy()
    far[3, 1] = np.inf
    dirs = scenes.random_sphere_dirs(50, seed=1)
    dirs[7, 2] = np.nan
    for bad in ({"rx": far}, {"rx_radius": -1.0}, {"freqs_hz": [0.0]}, {"max_reflections": 11}, {"n_rays": -1},
                {"ray_dirs": dirs, "n_rays": 50}, {"tx": np.float32([[0, 0, np.nan]])}):
        for call in (lambda: batch.trace([more, more, {**good, **bad}]), lambda: ctxs[2].trace_frame(**{**good, **bad})):
            with pytest.raises(dcem.DcemError) as e:
                call()
            assert e.value.status == dcem.E_INVALID_ARG, bad
            for c in ctxs:
                for a, b in zip(outputs(c), want):
                    assert np.array_equal(a, b, equal_nan=True)
    batch.close()
    for c in ctxs:
        c.close()
