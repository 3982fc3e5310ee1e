"""GPU tests of the packet walks of the single-tree range queries: leaf runs
and packet sizes at their edges, packets cut into tasks early and late, a
pool of tasks that runs out, queries that contain large nodes beside queries
that do not, and packets that mix ordinary and non-finite queries.  Every
result equals the oracle's, bit for bit."""

import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_query_equal, gpu_build, gpu_query, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ws():
    import paper_2402_00665_amd as lb
    return lb.Workspace()


def _check(tree, ref, q, qkind, ws):
    roff, ridx, _ = oracle.query_traverse(qkind, q, ref)
    off, idx = gpu_query(tree, q, qkind, ws)
    assert_query_equal(off, idx, roff, ridx)
    return int(roff[-1])


def _mixed(n, m, rng, kind):
    """Spheres, boxes and segments over [0,1)^3: points, small ones, ones
    that contain large parts of the scene, and a few without an order."""
    c = rng.random((m, 3)).astype(np.float32)
    size = np.where(rng.random(m) < 0.1, 0.5, 0.03).astype(np.float32) * rng.random(m, dtype=np.float32)
    if kind == 0:
        q = workloads.spheres(c, size)
    elif kind == 1:
        q = np.concatenate([c - size[:, None], c + size[:, None]], 1).astype(np.float32)
    else:
        q = workloads.segments_from(c, 0.4, rng)
        q[::17, 4] = 0.0
    if m > 8:
        q[m // 3, 0] = np.nan
        q[m // 2, 1] = np.inf
        q[-1, 2] = -np.inf
    return q


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 256, 257, 513, 3000])
@pytest.mark.parametrize("pkind", [0, 1])
def test_leaf_runs(n, pkind, ws):
    """Trees around the leaf counts at which a node is tested leaf by leaf,
    from one query to more than a packet's."""
    rng = np.random.default_rng([71, n, pkind])
    p = (rng.random((n, 3), dtype=np.float32) if pkind == 0
         else workloads.clustered_boxes(n, rng, components=3, sigma=0.2))
    ref = oracle.build(pkind, p, 63)
    tree, _ = gpu_build(p, pkind, 63, ws)
    for qkind in (0, 1, 2):
        for m in (1, 65):
            _check(tree, ref, _mixed(n, m, rng, qkind), qkind, ws)


@pytest.mark.parametrize("m", [32767, 32768, 65537])
@pytest.mark.parametrize("split2", [2, 7])
def test_packet_sizes_and_cuts(m, split2, ws):
    """Query counts around the packet sizes; with split2 = 2 packets give up
    their walks after three steps, so most of the work goes through tasks."""
    import paper_2402_00665_amd as lb
    rng = np.random.default_rng([73, m, split2])
    old = {k: lb.lbvh_tune(k) for k in ("query_split1", "query_split2")}
    lb.lbvh_tune("query_split2", split2)
    lb.lbvh_tune("query_split1", 2 if split2 == 2 else 12)
    try:
        p = workloads.clustered_boxes(40000, rng, components=6, sigma=0.02)
        ref = oracle.build(1, p, 30)
        tree, _ = gpu_build(p, 1, 30, ws)
        for qkind in (0, 1, 2):
            q = _mixed(p.shape[0], m, rng, qkind)
            if qkind < 2:
                # the large ones few: the result stays small
                big = rng.choice(m, 40, replace=False)
                small = np.ones(m, bool)
                small[big] = False
                c = rng.random((m, 3)).astype(np.float32)
                if qkind == 0:
                    q[small] = workloads.spheres(c, np.float32(0.01))[small]
                else:
                    q[small] = np.concatenate([c - 0.01, c + 0.01], 1).astype(np.float32)[small]
            hits = _check(tree, ref, q, qkind, ws)
            say(f"  qkind {qkind}: {hits} hits")
    finally:
        for k, v in old.items():
            lb.lbvh_tune(k, v)


def test_containing_and_touching_queries_stop_together(ws):
    """Packets in which some queries contain nodes that others only touch,
    given up at every step (patience 3): a query's rest begins behind what it
    has already reported."""
    import paper_2402_00665_amd as lb
    rng = np.random.default_rng(79)
    p = rng.random((60000, 3), dtype=np.float32)
    ref = oracle.build(0, p, 63)
    tree, _ = gpu_build(p, 0, 63, ws)
    old = {k: lb.lbvh_tune(k) for k in ("query_split2", "query_order")}
    lb.lbvh_tune("query_split2", 2)
    try:
        m = 40000
        # neighbours in the order: a thin box, then a box around it
        c = np.sort(rng.random((m, 1)), axis=0) * np.ones((1, 3))
        s = np.where(np.arange(m)[:, None] % 400 == 0, [[0.3, 0.3, 0.3]], [[0.004, 0.004, 0.004]])
        q = np.concatenate([c - s, c + s], 1).astype(np.float32)
        for order in (0, 1):
            lb.lbvh_tune("query_order", order)
            _check(tree, ref, q, 1, ws)
            _check(tree, ref, q[:3000], 1, ws)
    finally:
        for k, v in old.items():
            lb.lbvh_tune(k, v)


def test_pool_of_tasks_runs_out(ws):
    """Thousands of slabs across the whole scene: more tasks than the pool
    holds, so that packets fall back on their own few places."""
    rng = np.random.default_rng(83)
    n, m = 1 << 18, 2500
    p = rng.random((n, 3), dtype=np.float32)
    ref = oracle.build(0, p, 30)
    tree, _ = gpu_build(p, 0, 30, ws)
    z = rng.random(m)
    q = np.zeros((m, 6), np.float32)
    q[:, :2], q[:, 3:5] = -1.0, 2.0
    q[:, 2], q[:, 5] = z - 0.001, z + 0.001
    hits = _check(tree, ref, q, 1, ws)
    assert hits > 500 * m


@pytest.mark.parametrize("m", [(1 << 18) - 1, 1 << 18, (1 << 18) + 8193])
@pytest.mark.parametrize("n", [(1 << 18) - 1, 1 << 18, (1 << 21) - 1, 1 << 21])
def test_query_sort_tile_and_tree_size_lines(n, m, ws):
    """Both sides of the query count where the order's sort takes larger
    tiles (and the scan several rounds of look-back), and of the tree size
    where packets wait longer before they leave their rest and where tasks are
    narrower."""
    rng = np.random.default_rng([59, n, m])
    p = rng.random((n, 3), dtype=np.float32)
    p[: n // 8] = p[: n // 8] * np.float32(0.01) + np.float32(0.5)     # a dense corner
    q = workloads.spheres(rng.random((m, 3), dtype=np.float32), np.float32(0.004))
    q[::9, :3] = np.float32(0.505)
    q[:: m // 40, 3] = np.float32(0.06)                                # a few far longer walks
    ref = oracle.build(0, p, 30)
    tree, _ = gpu_build(p, 0, 30, ws)
    oracle.threads(16)
    try:
        assert _check(tree, ref, q, 0, ws) > m
    finally:
        oracle.threads(1)


def test_pool_of_tasks_runs_out_unevenly(ws):
    """Queries whose rests make from a few to many hundred tasks, in turn,
    more than the pool holds: some packets are refused while smaller ones
    still fit."""
    rng = np.random.default_rng(89)
    n, m = 1 << 20, 1000
    p = rng.random((n, 3), dtype=np.float32)
    ref = oracle.build(0, p, 30)
    tree, _ = gpu_build(p, 0, 30, ws)
    c = rng.random((m, 3))
    half = np.empty((m, 3))
    half[0::4] = [2.0, 2.0, 0.0005]      # slabs
    half[1::4] = [2.0, 0.004, 0.004]     # columns
    half[2::4] = [0.03, 0.03, 0.03]
    half[3::4] = [2.0, 0.3, 0.0005]      # strips
    half[8::64] = [0.4, 0.4, 0.0005]
    q = np.concatenate([c - half, c + half], 1).astype(np.float32)
    for _ in range(3):
        hits = _check(tree, ref, q, 1, ws)
    assert hits > 200 * m


def test_rest_left_at_a_contained_node(ws):
    """20400 queries, thousands of which leave their rest at a large node they
    contain, some nodes waiting: more tasks than the pool holds, so that
    packets are cut from what their walk left or, into their own few places,
    from the root."""
    import torch
    import paper_2402_00665_amd as lb
    rng = np.random.default_rng(113)
    n, k, times = 1 << 18, 24, 850
    p = rng.random((n, 3), dtype=np.float32)
    ref = oracle.build(0, p, 30)
    tree, _ = gpu_build(p, 0, 30, ws)
    c, half = rng.uniform(0.3, 0.7, (k, 3)), rng.uniform(0.2, 0.26, (k, 3))
    q = np.concatenate([c - half, c + half], 1).astype(np.float32)
    roff, ridx, _ = oracle.query_traverse(1, q, ref)
    dq = torch.from_numpy(np.tile(q, (times, 1))).cuda()
    off, idx = lb.query(tree, dq, 1, workspace=ws)
    lb.check_query(ws, k * times)
    counts = (off[1:] - off[:-1]).cpu().numpy().reshape(times, k)
    assert np.array_equal(counts, np.tile(np.diff(roff), (times, 1)))
    first = torch.from_numpy(ridx).cuda()
    for rows in idx.reshape(times, -1).split(50):
        assert bool((rows == first).all())
