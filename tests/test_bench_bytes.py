"""The byte model of bench.py's roofline: what a packet reads once for all its rays is
not counted for each of them; a group of lanes reads for its own ray."""
import bench


def test_trace_bytes():
    s = dict(trace_kernel=0, nodes_visited=10, tri_tests=640, rays_traced=64, segments=100, captures=3)
    assert bench.trace_bytes(s, False) == 128 * 10 + 13 * 64 + 4 * 100 + 8 * 3
    assert bench.trace_bytes(s, True) == bench.trace_bytes(s, False) + 32 * 100
    # the rays' tests say nothing about how often a packet's triangles were read
    assert bench.trace_bytes({**s, "tri_tests": 0}, False) == bench.trace_bytes(s, False)
    g = {**s, "trace_kernel": 1}
    assert bench.trace_bytes(g, True) == 128 * 10 + 16 * 640 + 42 * 64 + 84 * 100 + 8 * 3
