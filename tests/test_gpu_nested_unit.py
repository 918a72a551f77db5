"""The Nested WAIT kernel for unit thresholds at the sizes where its branches
change: every lane-group width, segments of one processing stage, one segment,
short and long calendars, known and drawn lengths, tight memory (evictions of
every kind), full queues; workspaces that pass between it and the general
kernel; and arrival lists, which launches with unit thresholds replay in the
general kernel.  Every field against the oracle."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_util import check, oracle_results, sim_module
from tests.parity_util import compare

pytestmark = pytest.mark.gpu


def _job(rng, m, ends, replicas, room, load=1.0, cap=1 << 12, known=False):
    top = ends[-1]
    l = [int(x) for x in rng.integers(1, 60, m)]
    C = int((max(l) + top) * room) + 1
    kw = dict(out_len=[int(x) for x in rng.integers(1, top, m - 1)] + [top]) if known else dict(
        out_cap=top, out_cdf=np.stack([W.geometric_cdf_table(float(rng.uniform(1.5, top)), top)
                                       for _ in range(m)]))
    wl = W.Workload(prompt_len=l, lam=[float(load * x / m) for x in rng.uniform(0.05, 0.4, m)],
                    d0=float(rng.uniform(0.5, 5.0)), d1=float(rng.uniform(0.0, 0.01)), C=C,
                    policy="nested", n=[1] * len(ends), seg_end=list(ends),
                    hist_edges=W.default_edges(1.0, int(rng.integers(1, 255))),
                    record_capacity=cap, **kw)
    return W.Job(wl, int(rng.integers(0, 2**63)), W.ids(replicas))


ENDS = {4: [3, 9, 40], 8: [1, 2, 3, 30, 31, 64, 200], 16: list(range(2, 30, 2)) + [90],
        1: [25], 2: [1, 2]}


@pytest.mark.parametrize("m", [1, 4, 5, 8, 13, 20, 40])
def test_group_widths(m):
    B = sim_module()
    rng = np.random.default_rng(40 + m)
    jobs = [_job(rng, m, e, r, room, known=kn) for e in ENDS.values() for room in (1.0, 2.5, 9.0)
            for r, kn in ((3, False), (18, True))]
    g, _ = check(B, jobs, 600, f"unit Nested WAIT, {m} types")
    assert g["fallback_evictions"].sum() > 0 and g["evictions"].sum() > g["fallback_evictions"].sum()


def test_full_queues():
    B = sim_module()
    rng = np.random.default_rng(8)
    jobs = [_job(rng, m, [2, 12, 30], 7, 1.5, 6.0, cap) for m in (1, 6) for cap in (16, 64)]
    g, _ = check(B, jobs, 500, "unit Nested WAIT, full queues")
    assert (g["flags"] & B.WS_FLAG_CAPACITY).sum() > 0


def test_queue_full_at_the_launch():
    """Evictions of the repair before a launch that overflow the queue: the
    batch runs, but takes no arrival any more."""
    B = sim_module()
    rng = np.random.default_rng(17)
    jobs = [_job(rng, m, ENDS[e], 24, room, 4.0, 16) for m in (3, 8) for e in (4, 8, 16)
            for room in (1.0, 1.3)]
    g, _ = check(B, jobs, 200, "unit Nested WAIT, queue full at the launch")
    assert (g["flags"] & B.WS_FLAG_CAPACITY).all()


def test_between_kernels():
    """Parts of a run on the unit kernel and on the general one (a traced
    advance), in both orders, end where one advance ends."""
    B = sim_module()
    rng = np.random.default_rng(99)
    jobs = [_job(rng, 3, [4, 20, 50], 21, room) for room in (1.2, 3.0, 20.0)]
    want = oracle_results(jobs, 900)
    for order in ("utu", "tut"):
        sim = B.Simulation(jobs)
        for i, o in enumerate(order):
            if o == "u":
                sim.advance(300, resume=i > 0)
            else:
                sim.advance_traced(300, 4, resume=i > 0)
        compare(sim.results(), want, order)


def _list_job(rng, m, ends, replicas, known, lam=0.0, arrivals=400):
    """A fixed arrival list (some arrivals at one instant) over m types."""
    top = ends[-1]
    lp = [int(x) for x in rng.integers(1, top, m - 1)] + [top]
    times = np.sort(rng.choice(np.linspace(0.0, 900.0, 251), arrivals))
    types = rng.integers(0, m, arrivals)
    l = [int(x) for x in rng.integers(1, 60, m)]
    wl = W.trace_workload("nested", l, lp if known else None, 1.0, 0.01,
                          int((max(l) + top) * rng.uniform(1.0, 4.0)) + 1, [1] * len(ends),
                          times, types, lengths=None if known else rng.integers(1, top + 1, arrivals),
                          seg_end=list(ends), out_cap=0 if known else top,
                          record_capacity=1 << 10)
    wl.lam = [lam] * m
    return W.Job(wl, int(rng.integers(0, 2**63)), W.ids(replicas))


@pytest.mark.parametrize("m", [1, 3, 7, 20])
def test_arrival_lists(m):
    """Unit thresholds and an arrival list, with known and per-request lengths,
    rates of zero and rates that the list replaces: every arrival of the list
    is taken, alone and beside a job that draws its arrivals, and a traced
    advance gives the same."""
    B = sim_module()
    rng = np.random.default_rng(70 + m)
    lists = [_list_job(rng, m, ENDS[e], r, kn, lam) for e in (1, 4) for r, kn in ((2, True), (5, False))
             for lam in (0.0, 0.3)]
    for jobs, ctx in ((lists, "lists"), (lists[:3] + [_job(rng, m, ENDS[4], 9, 2.0)], "lists and draws")):
        g, _ = check(B, jobs, 2500, f"unit Nested WAIT, {m} types, {ctx}")
        # (tight memory can evict a replica's every prompt before its end)
        assert g["completions"].sum() > 0 and (g["arrivals"] > 0).all()
        sim = B.Simulation(jobs)
        sim.prepare()
        sim.advance_traced(2500, 1)
        traced = sim.results()
        for k in g:
            assert np.array_equal(g[k], traced[k]), k
