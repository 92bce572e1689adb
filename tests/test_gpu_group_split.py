"""Grouped moves: the workgroups of a launch dealt out over jobs of unlike sizes, and the
host's count of pending terms as a hint only.  Per job bit for bit its own calls."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (3, 5, 2), (64, 1, 3), (8, 8, 70), (9, 64, 1), (31, 33, 4), (2, 2, 1)]


def _jobs(dtype, delay, sizes=SIZES):
    from paper_2202_05388_amd.job import Job
    out = []
    for ny, nx, m in sizes:
        j = Job(W.tiny(ny, nx, n_mon=m, dtype=dtype, cand_mask=W.MASK_BOTH), device="cuda:0", delay=delay)
        j.init()
        out.append(j)
    return out


def _same(a, b):
    for x, y in zip(a, b):
        x.flush()
        y.flush()
        for u, v in zip(x.host_state(), y.host_state()):
            assert np.array_equal(u, v)
        assert np.array_equal(x.history(), y.history()) and x.status() == y.status()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("delay,calls", [(16, [1, 5, 1, 9, 1]), (64, [3, 1, 20, 1]), (128, [1, 70, 2])])
def test_group_of_unlike_jobs(dtype, delay, calls):
    from paper_2202_05388_amd.job import JobGroup
    print(f"[case] {dtype} delay {delay} calls {calls}", flush=True)
    a, b = _jobs(dtype, delay), _jobs(dtype, delay)
    g = JobGroup(a)
    g.build()
    for n in calls:
        g.steps(n)
        for j in b:
            j.greedy_steps(n)
    _same(a, b)


@pytest.mark.parametrize("n_jobs", [1, 63, 64])
def test_group_counts(n_jobs):
    from paper_2202_05388_amd.job import JobGroup
    sizes = [(4 + i % 5, 3 + i % 7, 1 + i % 3) for i in range(n_jobs)]
    a, b = _jobs("c64", 16, sizes), _jobs("c64", 16, sizes)
    g = JobGroup(a)
    g.build()
    g.steps(6)
    for j in b:
        j.greedy_steps(6)
    _same(a, b)


def test_more_pending_terms_than_the_host_counts():
    from paper_2202_05388_amd.job import JobGroup
    a, b = _jobs("c64", 64), _jobs("c64", 64)
    g = JobGroup(a)
    g.build()
    g.steps(20)
    for j in a:
        j.state.pending_calls = 2
    g.steps(9)
    for j in a:
        j.state.pending_calls = 29
    for j in b:
        j.greedy_steps(29)
    _same(a, b)
