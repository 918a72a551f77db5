"""The FCFS kernel's lane groups (one lane per type, groups of 1 to 16 lanes)
at the sizes where its branches change: the queue's front in LDS (short and
long queues, few and many replicas per wavefront, admissions past what LDS
holds), cohorts around the 8 records loaded ahead, chunked prefill, full
queues, arrival lists of lengths around what is read ahead; every field against the oracle."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_util import check, sim_module
from tests.test_gpu_wait_lanes import list_jobs

pytestmark = pytest.mark.gpu


def _job(rng, m, replicas, load, chunk=0, cap=1 << 12, room=6.0, lp_hi=12):
    l = [int(x) for x in rng.integers(1, 40, m)]
    lp = [int(x) for x in rng.integers(1, lp_hi, m)]
    C = int(max(a + b for a, b in zip(l, lp)) * rng.uniform(1.2, room)) + 40
    wl = W.Workload(prompt_len=l, lam=[float(load * x / m) for x in rng.uniform(0.1, 1.0, m)],
                    d0=float(rng.uniform(0.5, 5.0)), d1=float(rng.uniform(0.0, 0.01)), C=C,
                    policy="fcfs", n=[], out_len=lp, reserve=0.02 if rng.integers(2) else 0.0,
                    chunk=chunk, hist_edges=W.default_edges(1.0, 64), record_capacity=cap)
    return W.Job(wl, int(rng.integers(0, 2**63)), W.ids(replicas))


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 8, 9, 16])
def test_group_widths(m):
    B = sim_module()
    rng = np.random.default_rng(300 + m)
    jobs = [_job(rng, m, r, load, chunk) for load in (0.1, 1.0, 6.0) for chunk in (0, 1, 24)
            for r in (1, 5, 64)]
    check(B, jobs, 300, f"FCFS, {m} types")


def test_cohorts():
    """Room for many admissions of one batch: more than LDS holds of the
    queue, more completions than are loaded ahead."""
    B = sim_module()
    rng = np.random.default_rng(77)
    jobs = [_job(rng, m, r, load, 0, 1 << 14, 200.0, 4) for m in (1, 3) for load in (5.0, 30.0, 90.0)
            for r in (2, 40)]
    g, _ = check(B, jobs, 200, "FCFS cohorts")
    assert g["completions"].sum() > 20 * g["batches"].sum()


def test_full_queues():
    B = sim_module()
    rng = np.random.default_rng(5)
    jobs = [_job(rng, m, 7, 8.0, chunk, cap) for m in (1, 3, 6) for cap in (16, 64)
            for chunk in (0, 8)]
    g, _ = check(B, jobs, 400, "FCFS full queues")
    assert (g["flags"] & B.WS_FLAG_CAPACITY).sum() > 0


@pytest.mark.parametrize("m", [1, 2, 3, 5, 9, 16])
def test_arrival_lists(m):
    B = sim_module()
    rng = np.random.default_rng(80 + m)
    jobs = list_jobs(rng, "fcfs", m)
    for j in jobs[::2]:
        j.wl.chunk = 13
    g, _ = check(B, jobs, 900, f"FCFS, lists, {m} types")
    assert (g["flags"] & B.WS_FLAG_CAPACITY).sum() > 0
    # a list continued in its middle; lists beside drawn arrivals and rate profiles
    sim = B.Simulation(jobs)
    for i, h in enumerate((3, 90, 807)):
        sim.advance(h, resume=i > 0)
    two = sim.results()
    for k in g:
        assert np.array_equal(g[k], two[k]), k
    rt, rf = W.diurnal_profile(m, 900.0, points=9)
    tv = _job(rng, m, 6, 1.0)
    jobs = jobs[3:7] + [_job(rng, m, 9, 1.0), W.Job(W.with_profile(tv.wl, rt, rf), 5, W.ids(6))]
    check(B, jobs, 400, f"FCFS, lists beside draws, {m} types")
