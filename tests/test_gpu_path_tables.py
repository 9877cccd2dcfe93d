"""GPU: path tables read whole, cut off, with outputs left out, short ones (packed
by one launch) and long ones (copied array by array, above 1 MB): the same rows."""
import ctypes

import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes

pytestmark = pytest.mark.gpu

NAMES = ["keys", "valid", "length", "tau", "aod", "aoa", "amp", "first_ray"]


def _get(ctx, cap, skip=()):
    K, nf = ctx.K, ctx.n_freqs
    rows = max(cap, 1)
    out = {"keys": np.full((rows, 3 + K), -77, np.int32), "valid": np.full(rows, 77, np.uint8),
           "length": np.full(rows, -7.0), "tau": np.full(rows, -7.0), "aod": np.full((rows, 3), -7.0),
           "aoa": np.full((rows, 3), -7.0), "amp": np.full((rows, nf, 3, 2), -7.0),
           "first_ray": np.full(rows, -77, np.int32)}
    n = ctypes.c_int64(0)
    ctx._check(ctx.lib.dcem_get_paths(ctx.handle, cap, *[None if k in skip else out[k].ctypes.data for k in NAMES],
                                      ctypes.byref(n)))
    return out, int(n.value)


@pytest.mark.parametrize("name", ["toy", "toy_los", "office", "bands"])
def test_tables(name):
    s = {"toy": scenes.static_toy, "toy_los": scenes.static_toy, "office": scenes.indoor_office,
         "bands": scenes.static_toy}[name]()
    change = {"toy": dict(rx_radius=2.0, n_rays=30_001, max_reflections=3), "toy_los": dict(max_reflections=0),
              "office": dict(n_rays=80_000), "bands": dict(freqs_hz=list(np.linspace(1e9, 60e9, 64)))}[name]
    s = scenes.Scene(**{**s.__dict__, **change})
    ctx = dcem.Context(0)
    ctx.scene_upload(s)
    ctx.trace_frame(**dcem.scene_frame_args(s))
    ctx.received_power()
    n = _get(ctx, 0)[1]
    whole, _ = _get(ctx, n + 5)
    size = sum(v[:n].nbytes for v in whole.values())
    print(name, "paths", n, "bytes", size, flush=True)
    assert (size > 1 << 20) == (name == "office")
    for k in NAMES:   # every row written, nothing past them
        assert (whole[k][n:] == (77 if k == "valid" else -77 if whole[k].dtype == np.int32 else -7.0)).all()
        assert k == "amp" or not (whole[k][:n] == (77 if k == "valid" else -77)).any()
    # a few rows (packed on every scene), as many as there are, each output alone
    for cap in (1, 7, n):
        cut, total = _get(ctx, cap)
        assert total == n
        for k in NAMES:
            assert np.array_equal(cut[k][:min(cap, n)], whole[k][:min(cap, n)]), (k, cap)
    for k in NAMES:
        one, _ = _get(ctx, min(n, 50), skip=[x for x in NAMES if x != k])
        assert np.array_equal(one[k][:min(n, 50)], whole[k][:min(n, 50)])
        assert all((one[x] == (77 if x == "valid" else -77 if one[x].dtype == np.int32 else -7.0)).all()
                   for x in NAMES if x != k)
    ctx.close()
