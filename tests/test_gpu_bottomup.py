"""The bottom-up pass at its block edges: chunks of 1024 leaves and
waves of 32 records, and the scene search of batches at powers of 64 scenes,
many of them empty.  Against the oracle, bit
for bit."""

import numpy as np
import pytest

import oracle
from gpu_util import assert_tree_equal, gpu_build
from test_gpu_batched import batched_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [30, 63])
@pytest.mark.parametrize("n", [31, 32, 33, 1023, 1024, 1025, 1055, 1056, 1057, 2047, 2048, 2049, 262144, 262145])
def test_chunk_edges(n, bits):
    rng = np.random.default_rng([n, bits, 5])
    c = rng.random((n, 3), dtype=np.float32)
    prims = np.concatenate([c, c + rng.random((n, 3), dtype=np.float32) * np.float32(0.01)], axis=1)
    prims[n // 2:, :] = prims[n // 2]          # half the leaves in one run of equal codes
    tree, _ = gpu_build(prims, 1, bits)
    assert_tree_equal(tree, oracle.build(1, prims, bits))


@pytest.mark.parametrize("S", [1, 2, 63, 64, 65, 4095, 4096, 4097])
def test_scene_search(S):
    rng = np.random.default_rng([S, 6])
    sizes = rng.choice([0, 0, 0, 1, 2, 40], size=S)
    sizes[rng.integers(0, S, max(1, S // 50))] = 1025
    sizes[S // 2] = 3000
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    batched_parity(rng.random((int(off[-1]), 3), dtype=np.float32), off, 30, 0,
                   check_every=max(1, S // 200))
