"""Performance cases of the simulator: what its users run, over the real range.

A study is a list of jobs (a model, a policy and a set of replica streams),
made once, whose workspace stays on the device; a pass advances every replica
from the empty system by `horizon` batches and leaves the per-replica results
(counters, censored areas, latency histograms) in the result buffer.  The
listed cases take the workloads of `workloads/` at horizons that reach their
working regime (the KV budget full, the longest outputs completing); two of
them are whole calls (host tables, upload, launch, results on the host; and a
checkpointed continuation).  Integer results and histograms are exact, the
time sums are binary64.
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

import workloads as W
from paper_2504_11320_amd import binding as B

# Per family: the listed sizes (also the largest that draw() gives) and what a
# replica's batch needs on average, counted from the events the workload has:
# lane operations (draws, clock, batch formation, completions, evictions) and
# bytes of request records (32 per arrival and per completion).
FAMILIES = {
    # a two-type toy in overload (about 15 arrivals a batch): the smallest
    # call a notebook makes, tables, upload, launch and results together
    "call": dict(jobs=1, replicas=64, horizon=100, ops=3500, rec=500),
    # the same system kept on the device: few replicas, latency counts
    "small": dict(jobs=1, replicas=64, horizon=1000, ops=3500, rec=500),
    # rate sweep of the Llama-shaped mix under WAIT with unit thresholds
    "wait": dict(jobs=32, replicas=1024, horizon=5000, ops=241, rec=36.5),
    # threshold grid x rates with FCFS on the same streams: many small jobs
    "sweep": dict(jobs=16, replicas=16, horizon=1000, ops=275, rec=25),
    # rates that turn over a day's cycle (thinned arrivals)
    "cyclic": dict(jobs=32, replicas=1024, horizon=2000, ops=334, rec=37.7),
    # FCFS with chunked prefill, the baseline policy of the rate sweep
    "chunked": dict(jobs=32, replicas=1024, horizon=5000, ops=98, rec=12.9),
    # decode server behind a prefill service: WAIT and FCFS, one type,
    # several arrivals a batch
    "decode": dict(jobs=9, replicas=1024, horizon=1000, ops=1134, rec=268),
    # Nested WAIT, geometric outputs, four segments, rate sweep
    "nested": dict(jobs=32, replicas=1024, horizon=4000, ops=163, rec=19.8),
    # Nested WAIT, ten heavy-tailed types, six segments up to 4096 tokens: the
    # benchmark's configuration
    "heavytail": dict(jobs=1, replicas=8192, horizon=10000, ops=235, rec=20.8),
    # Nested WAIT with per-stage caps (a batch-size cap spread over stages)
    "caps": dict(jobs=3, replicas=1001, horizon=3000, ops=250, rec=30),
    # FCFS whose output lengths are drawn per request, ragged sizes
    "drawn-lengths": dict(jobs=5, replicas=333, horizon=3000, ops=120, rec=15),
    # a rate sweep continued from a checkpoint and checkpointed again
    "resume": dict(jobs=7, replicas=301, horizon=1500, ops=241, rec=36.5),
}


def listed():
    return [dict(name=f, family=f, jobs=p["jobs"], replicas=p["replicas"], horizon=p["horizon"])
            for f, p in FAMILIES.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A family and sizes of its range: jobs, replicas per job and horizon
    spread over their logarithms, none above the family's listed case."""
    f = rng.choice(sorted(FAMILIES))
    p = FAMILIES[f]
    return dict(family=f, jobs=_log_int(rng, 1, p["jobs"]),
                replicas=_log_int(rng, min(8, p["replicas"]), p["replicas"]),
                horizon=_log_int(rng, max(20, p["horizon"] // 16), p["horizon"]))


def _capacity(per_batch, horizon):
    """Queue capacity: every arrival of the run fits."""
    return 1 << max(8, math.ceil(math.log2(2.0 * per_batch * horizon + 64)))


def _spread(jobs, n):
    """n of the jobs, from the first to the last."""
    return [jobs[round(i * (len(jobs) - 1) / max(1, n - 1))] for i in range(n)]


def _jobs(case, seed):
    f, n, R, H = case["family"], case["jobs"], case["replicas"], case["horizon"]
    if f in ("call", "small"):
        jobs = W.config1(R, _capacity(16, H))
    elif f in ("wait", "resume"):
        jobs = W.config2(R, n_rates=max(2, n), rate_index=range(n),
                         record_capacity=_capacity(1, H))
    elif f == "sweep":  # n x n thresholds at n rates, and FCFS at the same rates
        jobs = W.config4(R, grid=n, n_rates=max(2, n), record_capacity=_capacity(1, H))
    elif f == "cyclic":
        jobs = W.config_cyclic(R, n_rates=max(2, n), rate_index=range(n),
                               record_capacity=_capacity(2, H), span=8000.0 * H)
    elif f == "chunked":
        jobs = _spread(W.config_chunked(R, record_capacity=_capacity(1, H)), n)
    elif f == "decode":
        both = W.config_pd(R, _capacity(10, H))
        jobs = _spread(both[:9], n) + _spread(both[9:], n)
    elif f == "nested":
        jobs = W.config3(R, n_rates=max(2, n), rate_index=range(n),
                         record_capacity=_capacity(1, H))
    elif f == "heavytail":
        jobs = W.config5(R, _capacity(1, H))
    elif f == "caps":
        jobs = _spread(W.config_p512_mix(R, record_capacity=_capacity(2, H)), n)
    elif f == "drawn-lengths":
        jobs = [W.Job(dataclasses.replace(j.wl, policy="fcfs", n=[], seg_end=None, reserve=0.01),
                      j.seed, j.replica_ids)
                for j in W.config3(R, n_rates=max(2, n), rate_index=range(n),
                                   record_capacity=_capacity(1, H))]
    else:
        raise ValueError(f)
    return [W.Job(j.wl, seed, j.replica_ids) for j in jobs]


def prepare(case, seed):
    """The study's jobs and, but for the whole call, its workspace on the GPU."""
    jobs = _jobs(case, seed)
    state = dict(case=case, jobs=jobs)
    if case["family"] == "call":
        return state
    sim = state["sim"] = B.Simulation(jobs)
    sim.prepare()
    if case["family"] == "resume":  # a run that was saved after `horizon` batches
        sim.advance(case["horizon"])
        state["saved"] = sim.checkpoint()
        # room for the state that the continuation leaves (queues grow)
        state["next"] = torch.empty(2 * state["saved"].numel(), dtype=torch.uint8,
                                    device=state["saved"].device)
    return state


def _results(sim):
    """The result buffer's fields, where they lie on the device."""
    R, hs = sim.R, sim.hist_stride
    n_i, n_f = len(B.I64_FIELDS), len(B.F64_FIELDS)
    out = {f: sim.res[8 * R * i: 8 * R * (i + 1)].view(torch.int64)
           for i, f in enumerate(B.I64_FIELDS)}
    out.update({f: sim.res[8 * R * i: 8 * R * (i + 1)].view(torch.float64)
                for i, f in enumerate(B.F64_FIELDS, n_i)})
    off = 8 * R * (n_i + n_f)
    out["flags"] = sim.res[off: off + 4 * R].view(torch.int32)
    off = (off + 4 * R + 7) // 8 * 8
    out["hist"] = sim.res[off: off + 4 * R * hs].view(torch.int32).view(R, hs)
    return out


def run(state):
    case = state["case"]
    if case["family"] == "call":
        res = B.run_batch(state["jobs"], case["horizon"])
        return {k: v.astype(np.int32) if v.dtype == np.uint32 else v for k, v in res.items()}
    sim = state["sim"]
    if case["family"] == "resume":
        size = sim.run_ex(case["horizon"], state["saved"], state["next"])
        return dict(_results(sim), checkpoint_bytes=size)
    sim.advance(case["horizon"])
    return _results(sim)


def _replicas(case):
    n = case["jobs"]
    jobs = {"sweep": n * n * max(2, n) + max(2, n), "decode": 2 * n}.get(case["family"], n)
    return jobs * case["replicas"]


def work(case):
    p = FAMILIES[case["family"]]
    steps = _replicas(case) * case["horizon"]
    return {"bytes": p["rec"] * steps + 144 * _replicas(case), "flops": p["ops"] * steps}


def tolerance(case):
    # counts are exact; the time sums (areas, latencies) differ from correctly
    # rounded ones by up to 1.8e-14 after 1000 batches, growing with their
    # square root: 6e-14 after 10000, times four
    return {"rel": 2.5e-13}


# ------------------------------------------------------------- in 64 bits --
# WAIT with known output lengths, one request at a time in plain Python.


def _gaps(seed, rid, j, k0, n, lam):
    """Gaps of arrivals k0 .. k0 + n - 1 of type j (Philox4x32-10)."""
    m32 = np.uint64(0xFFFFFFFF)
    c = [np.arange(k0, k0 + n, dtype=np.uint64), np.full(n, j, np.uint64),
         np.full(n, rid, np.uint64), np.zeros(n, np.uint64)]
    k = [seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF]
    for _ in range(10):
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        s = np.uint64(32)
        c = [(p1 >> s) ^ c[1] ^ np.uint64(k[0]), p1 & m32,
             (p0 >> s) ^ c[3] ^ np.uint64(k[1]), p0 & m32]
        k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
    x = (c[0] << np.uint64(20)) | (c[1] >> np.uint64(12))
    return -np.log((2 * x + np.uint64(1)).astype(np.float64) * 2.0 ** -53) / lam


def _wait_replica(wl, seed, rid, horizon):
    m, times, nxt = wl.m, [], [0] * wl.m
    for j in range(m):
        times.append(np.cumsum(_gaps(seed, rid, j, 0, 512, wl.lam[j])))

    def peek():
        best, bj = math.inf, 0
        for j in range(m):
            while nxt[j] >= len(times[j]):
                g = _gaps(seed, rid, j, len(times[j]), len(times[j]), wl.lam[j])
                g[0] += times[j][-1]
                times[j] = np.concatenate([times[j], np.cumsum(g)])
            if times[j][nxt[j]] < best:
                best, bj = float(times[j][nxt[j]]), j
        return best, bj

    queue = [[] for _ in range(m)]      # [arrival, first token]
    here = [[] for _ in range(m)]       # [arrival, first token, stage, batch]
    heads = [0] * m
    out = dict.fromkeys(B.I64_FIELDS, 0)
    lat, ttft, mem, done, busy = [], [], [], [], []
    hist = [0] * (len(wl.hist_edges) + 1)
    t, N, U = 0.0, 0, 0
    held = lambda: sum(wl.prompt_len[j] + p[2] for j in range(m) for p in here[j])  # noqa: E731
    M = 0
    for b in range(horizon):
        while True:
            sel = [j for j in range(m) if len(queue[j]) - heads[j] >= wl.n[j]]
            if sel:
                break
            ta, _ = peek()
            lat.append(N * (ta - t))
            ttft.append(U * (ta - t))
            mem.append(M * (ta - t))
            t = ta
            while peek()[0] == ta:
                j = peek()[1]
                queue[j].append([ta, False])
                nxt[j] += 1
                out["arrivals"] += 1
                N, U = N + 1, U + 1
            out["idle_waits"] += 1
        tokens = prefill = 0
        for j in sel:
            tokens += sum(wl.prompt_len[j] + p[2] for p in here[j]) + wl.n[j] * wl.prompt_len[j]
            prefill += wl.n[j] * wl.prompt_len[j]
            for a, ft in queue[j][heads[j]: heads[j] + wl.n[j]]:
                here[j].append([a, ft, 0, b])
            heads[j] += wl.n[j]
        out["peak_mem"] = max(out["peak_mem"], M + prefill)
        tau = wl.d0 + wl.d1 * tokens
        end = t + tau
        lat.append(N * tau)
        ttft.append(U * tau)
        mem.append((M + prefill) * tau)
        busy.append(tau)
        while True:
            ta, j = peek()
            if ta > end:
                break
            queue[j].append([ta, False])
            nxt[j] += 1
            out["arrivals"] += 1
            N, U = N + 1, U + 1
            lat.append(end - ta)
            ttft.append(end - ta)
        t = end
        for j in sel:
            keep = []
            for p in here[j]:
                if p[2] == 1 and not p[1]:
                    p[1] = True
                    U -= 1
                if p[2] == wl.out_len[j]:
                    done.append(end - p[0])
                    hist[int(np.searchsorted(wl.hist_edges, end - p[0], side="right"))] += 1
                    out["completions"] += 1
                    out["completed_tokens"] += wl.out_len[j]
                    N -= 1
                else:
                    p[2] += 1
                    keep.append(p)
            here[j] = keep
        M = held()
        out["peak_mem"] = max(out["peak_mem"], M)
        while M > wl.C:
            j = max((x for x in range(m) if here[x]), key=lambda x: (here[x][-1][3], x))
            a, ft, stage, _ = here[j].pop()
            queue[j].append([a, ft])
            M -= wl.prompt_len[j] + stage
            out["evictions"] += 1
            out["evicted_tokens"] += stage - 1
        out["batches"] += 1
        out["batch_tokens_sum"] += tokens
    out["waiting_end"] = sum(len(q) - h for q, h in zip(queue, heads))
    out["resident_end"] = sum(len(h) for h in here)
    out.update(t_end=t, busy_time=math.fsum(busy), lat_area=math.fsum(lat),
               ttft_area=math.fsum(ttft), lat_completed_sum=math.fsum(done),
               mem_area=math.fsum(mem), flags=0, hist=hist)
    return out


def exact(case, seed):
    """The two-type WAIT cases replica by replica; the others are 10^6 and more
    replica-batches, hours of plain Python."""
    if case["family"] not in ("call", "small") or case["replicas"] * case["horizon"] > 70000:
        return None
    rows = []
    for job in _jobs(case, seed):
        rows += [_wait_replica(job.wl, seed, int(r), case["horizon"]) for r in job.replica_ids]
    out = {f: np.array([r[f] for r in rows], np.int64) for f in B.I64_FIELDS}
    out.update({f: np.array([r[f] for r in rows], np.float64) for f in B.F64_FIELDS})
    out["flags"] = np.array([r["flags"] for r in rows], np.int32)
    out["hist"] = np.array([r["hist"] for r in rows], np.int32)
    return out
