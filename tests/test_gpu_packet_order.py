"""GPU: one source's packets of 64 rays start in an order of their own, several
sources' by position: ray counts with remainders and packet counts that the eight
queues do not share evenly, with and without transmission branches, against the
oracle."""
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


# just above 4096 packets in all; a last packet of 1 ray, 5 rays and 64; directions
# along the vertical axis only, whose packets all have one key
@pytest.mark.parametrize("n_src,n", [(1, 64 * 4096), (1, 64 * 4102 + 1), (1, 64 * 8193 + 5), (3, 64 * 1366 + 1), (41, 64 * 103 + 5), (7, 64 * 600)])
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


# 11 branches of one source: the shortest order that is used, a last packet of 7 rays,
# and one that gives the queues a remainder of 3 packets
@pytest.mark.parametrize("n", [64 * 372 + 7, 64 * 384 + 1])
def test_branches(O, n):
    s = scenes.indoor_office(n_rays=n)
    assert s.tx.shape[0] == 1
    ctx = dcem.Context(0)
    log("branches", n)
    st, out, ofr = run_pair(ctx, O, s, n_rays=n)
    assert_comparable(st)
    ctx.close()
