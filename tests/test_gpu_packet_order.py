"""GPU: packets of 64 rays are started in an order of their own: several sources,
ray counts with remainders, and chunk counts that the eight queues do not share
evenly, each source's captures against the oracle."""
import numpy as np
import pytest

from paper_2112_07115_amd import dcem, scenes
from tests.gpu_frames import assert_comparable, log, run_pair

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def O():
    from oracle import oracle
    oracle.build()
    return oracle


# just above 4096 packets in all: an order sorted by one workgroup and by several,
# a last packet of 1 ray, 5 rays and 64, directions along the vertical axis only
@pytest.mark.parametrize("n_src,n", [(3, 64 * 1366 + 1), (41, 64 * 103 + 5), (7, 64 * 600)])
@pytest.mark.parametrize("vertical", [False, True])
def test_sources(O, n_src, n, vertical):
    s = scenes.static_toy()
    s.tx = np.asarray(s.tx)[:1] + np.linspace(0.3, 1.0, n_src)[:, None] * np.array([[3.0, 1.0, 1.0]])
    dirs = None
    if vertical:
        dirs = np.zeros((n, 3), np.float32)
        dirs[:, 2] = np.where(np.arange(n) % 3 == 0, -1.0, 1.0)
    ctx = dcem.Context(0)
    log("sources", n_src, "rays", n, "vertical", vertical)
    st, out, ofr = run_pair(ctx, O, s, dirs=dirs, n_rays=None if vertical else n)
    assert_comparable(st)
    ctx.close()
