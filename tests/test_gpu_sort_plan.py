"""The sort's shape by size, with every knob at its default: builds on both
sides of each size where the digit width or the tile shape changes, and
batches on both sides of the lines between one block per scene and segmented
passes.  Trees must equal the oracle's bit for bit."""

import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_tree_equal, gpu_build
from test_gpu_batched import batched_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [30, 63])
@pytest.mark.parametrize("n", [1 << 17, (1 << 17) + 1, 1 << 19, (1 << 19) + 1, 1 << 21, (1 << 21) + 1,
                               3 << 20, (3 << 20) + 1, (1 << 22) + 1])
def test_single_build_lines(n, bits):
    rng = np.random.default_rng([n, bits])
    prims = rng.random((n, 3), dtype=np.float32)
    prims[n // 3: n // 2] = prims[0]          # one long run of equal codes
    tree, _ = gpu_build(prims, 0, bits)
    assert_tree_equal(tree, oracle.build(0, prims, bits))


@pytest.mark.parametrize("bits", [30, 63])
@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 1023, 1024, 1025, 4095, 4096, 4097])
def test_one_block_build(n, kind, bits):
    import paper_2402_00665_amd as lb
    rng = np.random.default_rng([n, bits, kind])
    prims = np.round(rng.random((n, 3)) * 64).astype(np.float32)   # many equal codes
    if kind == 1:
        prims = np.concatenate([prims, prims + rng.random((n, 3), dtype=np.float32)], axis=1)
    ws = lb.Workspace()
    for _ in range(2):                        # the second into a used workspace
        tree, _ = gpu_build(prims, kind, bits, ws)
        assert_tree_equal(tree, oracle.build(kind, prims, bits))


@pytest.mark.parametrize("bits", [30, 63])
@pytest.mark.parametrize("sizes", [
    [4096, 4095, 1], [4097, 4096, 0],                    # a scene of one tile, and beyond
    [8192, 8191, 3], [8193, 8192],
    [5000] * 128, [5000] * 127 + [4999],                 # 128 times the largest, and below
    [65536, 70000], [65537] * 128,                       # the larger blocks' side
])
def test_batch_lines(sizes, bits):
    rng = np.random.default_rng([sum(sizes), bits])
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    prims = rng.random((int(off[-1]), 3), dtype=np.float32)
    prims[: off[-1] // 4] = np.round(prims[: off[-1] // 4] * 8) / 8   # many equal codes
    batched_parity(prims, off, bits, 0)
