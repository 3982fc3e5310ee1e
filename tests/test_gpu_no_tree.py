"""Queries on nodes that are no tree (every id valid, but children that lead
back to their own node or to an empty range): each walk ends, with the error
word set, and the fill stays inside the counted slots.  On a tree the same
calls then pass again."""

import numpy as np
import pytest

import oracle
from gpu_util import assert_query_equal, gpu_build, say

pytestmark = pytest.mark.gpu


def _loop(tree, split):
    """Every internal node splits behind leaf `split`; unit boxes, leaves elsewhere."""
    n = tree.n
    f = np.zeros((2 * n - 1, 8), np.float32)
    f[: n - 1, 4:7] = 1.0
    f[n - 1:, :3], f[n - 1:, 4:7] = 5.0, 6.0
    nodes = f.view(np.int32)
    nodes[: n - 1, 3] = split
    nodes[n - 1:, 3] = np.arange(n)
    nodes[:, 7] = -1
    return nodes


@pytest.mark.parametrize("split", [0, -3])
@pytest.mark.parametrize("m", [1, 2000, 40000])
def test_walks_end(split, m):
    import torch
    import paper_2402_00665_amd as lb
    rng = np.random.default_rng([97, m])
    n = 1000
    p = rng.random((n, 6), dtype=np.float32) * np.float32(0.01)
    p[:, 3:] += p[:, :3]
    tree, _ = gpu_build(p, 1, 30)
    good = tree.nodes.clone()
    bad = torch.from_numpy(_loop(tree, split % n)).view(good.dtype).cuda().reshape(good.shape)
    ws = lb.Workspace()
    ref = oracle.build(1, p, 30)
    # each passes the unit box's test without containing it
    queries = {0: np.float32([[-0.5, 0.5, 0.5, 0.6]]), 1: np.float32([[-1, -1, -1, 0.5, 0.5, 0.5]]),
               2: np.float32([[-1, 0.25, 0.5, 0, 1, 0.125, 0.0625, 9]])}
    for qkind, q in queries.items():
        q = np.repeat(q, m, axis=0)
        d = torch.from_numpy(q).cuda()
        say(f"  qkind {qkind}, m {m}, split {split}")
        tree.nodes.copy_(bad)
        off = lb.query_count(tree, d, qkind, ws)
        with pytest.raises(lb.LbvhError) as e:
            lb.check_query(ws, m)
        assert e.value.status == lb.LBVH_EDEVICE
        total = int(off[-1].item())
        buf = torch.full((total + 4096,), -7, dtype=torch.int32, device="cuda")
        lb.query_fill(tree, d, qkind, buf, ws)
        torch.cuda.synchronize()
        assert bool((buf[total:] == -7).all())
        if qkind == 2:
            lb.query_first(tree, d, workspace=ws)
            with pytest.raises(lb.LbvhError):
                lb.check_query(ws, m)
        tree.nodes.copy_(good)
        few = q[:2000].copy()
        few[:, :3] += rng.random((few.shape[0], 3), dtype=np.float32) * np.float32(0.02)
        off, idx = lb.query(tree, torch.from_numpy(few).cuda(), qkind, workspace=ws)
        lb.check_query(ws, few.shape[0])
        roff, ridx, _ = oracle.query_traverse(qkind, few, ref)
        assert_query_equal(off.cpu().numpy(), idx.cpu().numpy(), roff, ridx)
