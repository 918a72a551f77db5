"""The WAIT kernel's lane groups (one lane per type, groups of 1 to 64 lanes)
at the sizes where its branches change: cohorts around the 16 records loaded
ahead and completions around the 8, one type to more than a 32-lane group,
few and many replicas per wavefront, full queues, simultaneous arrivals, arrival
lists of lengths around what is read ahead; every field against the oracle (fp64 sums within the parity bound: the sums
per type and batch are taken type by type)."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import check, sim_module

pytestmark = pytest.mark.gpu


def _job(rng, m, n_lo, n_hi, policy, replicas, cap=1 << 12, load=1.0):
    l = [int(x) for x in rng.integers(1, 40, m)]
    lp = [int(x) for x in rng.integers(1, 12, m)]
    n = [int(x) for x in rng.integers(n_lo, n_hi + 1, m)]
    # memory for one to four full cohorts: completions and evictions both happen
    C = int(max(k * (a + b + 1) for k, a, b in zip(n, l, lp)) * rng.uniform(1.0, 4.0))
    wl = W.Workload(prompt_len=l, lam=[float(load * k * x) for k, x in zip(n, rng.uniform(0.02, 0.4, m))],
                    d0=float(rng.uniform(0.5, 5.0)), d1=float(rng.uniform(0.0, 0.01)), C=C,
                    policy=policy, n=n, out_len=lp, hist_edges=W.default_edges(1.0, 64),
                    record_capacity=cap)
    return W.Job(wl, int(rng.integers(0, 2**63)), W.ids(replicas))


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 8, 9, 16, 17, 33])
def test_group_widths(m):
    B = sim_module()
    rng = np.random.default_rng(900 + m)
    jobs = [_job(rng, m, 1, 5, p, r) for p in ("wait", "wait-nowait") for r in (1, 3, 17, 64)]
    check(B, jobs, 400, f"{m} types, thresholds 1-5")
    check(B, [_job(rng, m, 1, 1, p, r) for p in ("wait", "wait-nowait") for r in (1, 5, 33)],
          400, f"{m} types, unit thresholds")


@pytest.mark.parametrize("n", [7, 8, 9, 15, 16, 17, 24, 65])
def test_cohort_sizes(n):
    B = sim_module()
    rng = np.random.default_rng(700 + n)
    jobs = [_job(rng, m, max(1, n - 1), n, p, r, 1 << 14) for m in (1, 3)
            for p in ("wait", "wait-nowait") for r in (2, 19)]
    g, _ = check(B, jobs, 300, f"cohorts of {n}")
    assert g["evictions"].sum() > 0 and g["completions"].sum() > 0


def test_full_queues():
    """Queues that overflow, in arrivals and in evictions, with cohorts that
    the queue barely holds."""
    B = sim_module()
    rng = np.random.default_rng(31)
    jobs = [_job(rng, m, 1, 16, p, 7, cap, 4.0) for m in (1, 3, 6) for cap in (16, 32, 64)
            for p in ("wait", "wait-nowait")]
    jobs += [_job(rng, 3, 1, 1, "wait", 7, 16, 4.0) for _ in range(3)]
    g, _ = check(B, jobs, 500, "full queues")
    assert (g["flags"] & B.WS_FLAG_CAPACITY).sum() > 0


def test_gaps_below_the_clock():
    """Rates so high that gaps vanish beside the clock: rings of equal arrival
    times, until the queue overflows."""
    B = sim_module()
    jobs = []
    for m, n in ((1, 1), (3, 1), (3, 2)):
        wl = W.Workload(prompt_len=[4, 9, 2][:m], lam=[1e12, 2e-6, 3e11][:m], d0=1e6, d1=1.0,
                        C=400, policy="wait", n=[n] * m, out_len=[3, 5, 2][:m],
                        hist_edges=W.default_edges(1e6, 32), record_capacity=1 << 12)
        slow = dataclasses.replace(wl, lam=[1e-7, 1e-6, 1e-7][:m])
        jobs += [W.Job(wl, 3, W.ids(5)), W.Job(slow, 4, W.ids(5))]
    g, _ = check(B, jobs, 40, "gaps below the clock")
    assert (g["flags"] & B.WS_FLAG_CAPACITY).sum() > 0


def test_more_replicas_than_a_launch_spreads():
    """32 jobs of 1,200 and of 37 replicas: wavefronts full of groups, and the
    narrow ones of a small launch (against the oracle), give the same replicas
    the same bits."""
    B = sim_module()
    rng = np.random.default_rng(12)
    base = [_job(rng, 3, 1, 4, "wait", 1) for _ in range(32)]
    wide = B.run_batch([dataclasses.replace(j, replica_ids=W.ids(1200)) for j in base], 200)
    thin, _ = check(B, [dataclasses.replace(j, replica_ids=W.ids(37)) for j in base], 200,
                    "32 x 37 replicas, three types")
    idx = np.concatenate([1200 * k + np.arange(37) for k in range(32)])
    for k in wide:
        assert np.array_equal(wide[k][idx], thin[k]), k


def list_jobs(rng, policy, m, cap=1 << 9):
    """Arrival lists over m types, several arrivals to an instant: of no more
    entries than a few, around the 8 per lane that are read ahead, long ones;
    a queue that overflows."""
    jobs = []
    for total in (1, 3, 4, 5, 8 * m - 1, 8 * m, 8 * m + 1, 64 * m + 3, 1500):
        span = total * (0.05 if total == 1500 else 4.0)
        times = np.sort(rng.choice(np.linspace(0.0, span, 2 * total + 1), total))
        l = [int(x) for x in rng.integers(1, 40, m)]
        lp = [int(x) for x in rng.integers(1, 12, m)]
        n = [int(x) for x in rng.integers(1, 7, m)]
        wl = W.trace_workload(policy, l, lp, 1.0, 0.005, int((max(l) + 12) * rng.uniform(1.5, 12.0)),
                              [] if policy == "fcfs" else n, times, rng.integers(0, m, total),
                              record_capacity=16 if total == 1500 else cap)
        jobs.append(W.Job(wl, 0, W.ids(int(rng.integers(1, 70)))))
    return jobs


@pytest.mark.parametrize("m", [1, 2, 3, 5, 9, 17, 33])
def test_arrival_lists(m):
    B = sim_module()
    rng = np.random.default_rng(60 + m)
    jobs = list_jobs(rng, "wait", m) + list_jobs(rng, "wait-nowait", m)
    g, _ = check(B, jobs, 700, f"WAIT, lists, {m} types")
    assert (g["flags"] & B.WS_FLAG_CAPACITY).sum() > 0
    # a list continued in its middle; lists beside drawn arrivals and rate profiles
    sim = B.Simulation(jobs)
    for i, h in enumerate((3, 90, 607)):
        sim.advance(h, resume=i > 0)
    two = sim.results()
    for k in g:
        assert np.array_equal(g[k], two[k]), k
    if m <= 16:
        rt, rf = W.diurnal_profile(m, 900.0, points=9)
        tv = _job(rng, m, 1, 3, "wait", 11)
        jobs = jobs[3:7] + [_job(rng, m, 1, 3, "wait", 9), W.Job(W.with_profile(tv.wl, rt, rf), 5, W.ids(6))]
        check(B, jobs, 400, f"WAIT, lists beside draws, {m} types")
