"""Sort knobs asked for at their default values ("sort_by_size" off) run as
they say: the number of launches tells which form ran.  And batches on both
sides of the lines between the blocks' shapes.  Trees equal the oracle's bit
for bit."""

import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_tree_equal, gpu_build, say
from test_gpu_batched import batched_parity

pytestmark = pytest.mark.gpu


@pytest.fixture
def by_size():
    import paper_2402_00665_amd as lb

    def turn(on):
        assert lb.lbvh_tune("sort_by_size", on) in (0, 1)

    yield turn
    lb.lbvh_tune("sort_by_size", 1)


def _launches(f):
    """f()'s result and the launches of the sort in it."""
    import torch
    import paper_2402_00665_amd as lb
    lb.lbvh_profile_reset()
    lb.lbvh_profile_enable(True)
    try:
        r = f()
        torch.cuda.synchronize()
        return r, lb.lbvh_profile_read("sort_pass")[1]
    finally:
        lb.lbvh_profile_enable(False)


@pytest.mark.parametrize("n,bits,by_knob,sized", [(100003, 30, 4, 3), (3000, 30, 4, 1), (300, 63, 7, 1),
                                                  (1 << 18, 30, 4, 3), (3300000, 63, 7, 8)])
def test_single_build_runs_the_default_knobs(n, bits, by_knob, sized, by_size):
    rng = np.random.default_rng([103, n, bits])
    p = rng.random((n, 3), dtype=np.float32)
    p[n // 2:] = np.round(p[n // 2:] * 256) / 256      # many equal codes
    ref = oracle.build(0, p, bits)
    for on, want in ((0, by_knob), (1, sized)):
        by_size(on)
        (tree, _), got = _launches(lambda: gpu_build(p, 0, bits))
        assert got == want
        assert_tree_equal(tree, ref)


@pytest.mark.parametrize("bits,passes", [(30, 4), (63, 7)])
def test_segmented_mode_runs_segmented(bits, passes, by_size):
    rng = np.random.default_rng([107, bits])
    sizes = np.array([4097, 1, 4096, 0, 8192, 6000, 33, 2048], np.int64)
    off = np.concatenate([[0], np.cumsum(sizes)])
    p = rng.random((int(off[-1]), 3), dtype=np.float32)
    for on, want in ((0, passes), (1, 1)):
        by_size(on)
        _, got = _launches(lambda: batched_parity(p, off, bits, 0))
        assert got == want


@pytest.mark.timeout(900)
def test_segmented_full_size(by_size):
    """4096 scenes, 35 M points: look-back across many segments."""
    pts, off, q, qoff = workloads.batched()
    by_size(0)
    oracle.threads(16)
    try:
        say("segmented passes over the full batch")
        _, got = _launches(lambda: batched_parity(pts, off, 63, 0, check_every=4))
        assert got == 7
    finally:
        oracle.threads(1)


@pytest.mark.parametrize("bits", [30, 63])
@pytest.mark.parametrize("sizes", [
    [4097] * 256, [4097] * 257,                          # a block a CU, and more
    [24576] * 2 + [12300] * 254 + [24576], [24577] * 2 + [12300] * 256,
    [24577] + [12300] * 512, [24577] + [12400] * 512,    # 256 times the largest, and above
])
def test_block_shape_lines(sizes, bits):
    rng = np.random.default_rng([109, sum(sizes), bits])
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    p = rng.random((int(off[-1]), 3), dtype=np.float32)
    p[: off[-1] // 4] = np.round(p[: off[-1] // 4] * 8) / 8   # many equal codes
    batched_parity(p, off, bits, 0, check_every=max(1, len(sizes) // 40))
