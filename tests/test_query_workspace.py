"""A query workspace that is large enough for m queries is large enough for
fewer: a program keeps one for the most queries it asks at a time."""

import paper_2402_00665_amd as lb


def test_size_never_falls():
    ends = {e + d for k in range(31) for d in range(-66, 67) for e in (1 << k, 4096 * k, 6144 * 64 * k)}
    sizes = sorted(e for e in ends | set(range(70000)) if 0 <= e < 1 << 31)
    for f in (lb.lbvh_query_workspace_bytes, lb.lbvh_query_batched_workspace_bytes):
        most = 0
        for m in sizes:
            assert f(m) >= most, (f.__name__, m)
            most = f(m)
