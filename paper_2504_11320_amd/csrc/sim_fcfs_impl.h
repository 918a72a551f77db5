// sim_fcfs_impl.h -- simulation kernel for FCFS with known output lengths
// (arXiv 2504.11320: Section 4.1; chunked prefill, the baseline of Section 6;
// time-varying rates of the appendix).
//
// A group of G lanes (G = 1, 2, 4, 8 or 16, a power of two >= the job's types)
// runs one replica; lane g of a group owns request type g: its arrival process,
// its resident deque and its resident memory.  Every resident is batched every
// iteration, so a prompt admitted at batch kb completes at batch kb + l'_j and
// the residents of one type complete in admission order: admissions push at
// the back of the type's deque, completions pop at the front, LIFO evictions
// pop at the back.  The external queue is one FIFO of 16-byte records for all
// types; its ends and the batch's scalars are kept identical in every lane of
// the group.  Loops are wavefront-uniform and conditions are lane masks on the
// scalar unit (a group that is done stays in as inactive).
//
// Admission is a serial scan of the queue's head: it stops at the first prompt
// that does not fit, so each head must be known at the launch.  The front of
// the queue is kept in LDS: pushes go there too while everything queued fits,
// and in a longer queue the next records are loaded at a launch and land at
// the batch's completion step, so the scan seldom waits for memory.
//
// Arithmetic is the model's (the same IEEE operations, no FMA contraction), in
// its order but for one sum: a batch's completions sum their latencies per type
// in admission order, then the types in turn (the model adds them one by one).
//
// What bounds it: a wavefront's latency per batch (a replica is a serial chain
// of events).  32 rates x 1024 replicas of the Llama-shaped mix with 512-token
// chunks: 158 vector, 77 scalar and 35 branch instructions per wavefront and
// batch, 11.4 ms per 5,000 batches (18.1 with one lane per replica and per-type
// register arrays); half of the waves' cycles are waits.  2 x 9,216 replicas of one
// type, 6.5 arrivals a batch, beside the same under WAIT: 13.2 against 29.4 ms
// per 1,000 batches (records were loaded one by one as they were popped).
#pragma once

#include "sim_arrivals.h"

namespace wsim {
namespace {

// A queue record in LDS: its prompt length in place of the output length,
// which its type gives.
struct QLds {
  double a_ft;
  int32_t j, l;
};

// TV: the general instantiation (time-varying rates, per-batch trace); LIST:
// arrival lists too.
template <int G, bool TV, bool LIST>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
sim_fcfs_kernel(KArgs A) {
  constexpr int RING = 512;   // arrival times drawn ahead, of a wavefront
  constexpr int QRING = 256;  // queue records in LDS, of a wavefront
  constexpr int NL = G >= 4 ? 1 : 4 / G;  // queue records a lane loads at a time
  // the last records pushed on each deque, for LIFO evictions (in the general
  // instantiations as many as leave room for two wavefronts per SIMD with up to
  // 8 types)
  constexpr int WB = TV ? 4 : 8;
  constexpr int KC = 8;  // records at the front of the deque loaded at the launch
  __shared__ typename Arrivals<G, TV, RING>::Lds s_arr;
  __shared__ DRec s_win[WB][64];
  __shared__ QLds s_q[QRING];
  __shared__ int32_t s_l[G];
  __shared__ double s_edges[WS_MAX_HIST_EDGES + 1];
  __shared__ uint8_t s_htab[kHistTab];
  __shared__ int s_hsteps;

  const int tx = threadIdx.x;
  const int gl = tx & (G - 1);  // lane in the group: type gl
  // the replica list holds A.lanes replicas per 64 entries; a wavefront takes
  // A.nr consecutive ones of them
  const int split = A.lanes / A.nr;
  const int q = tx / G;
  const int64_t row = (int64_t)(blockIdx.x / split) * 64 + (int64_t)(blockIdx.x % split) * A.nr;
  const int32_t *list = (const int32_t *)(A.ws + A.off_list);
  const int32_t r0 = __builtin_amdgcn_readfirstlane(list[row]);
  if (r0 < 0) return;  // nothing but padding
  const int32_t r32 = q < A.nr ? list[row + q] : -1;
  const bool valid = r32 >= 0;
  const int64_t r = valid ? r32 : r0;
  // every replica of a wavefront belongs to the same job: its constants are
  // wavefront-uniform
  const uint32_t jix =
      __builtin_amdgcn_readfirstlane(((const uint32_t *)(A.ws + A.off_job_of))[r0]);
  const JobDev &J = ((const JobDev *)(A.ws + A.off_jobs))[jix];
  const int m = J.m;
  const int n_hist = J.n_hist;
  const int P = TV ? J.n_rate : 0;
  const bool trace = LIST && J.n_trace > 0;
  const bool is_t = gl < m;
  {
    const double *edges_g = (const double *)(A.ws + J.off_edges);
    for (int b = tx; b <= n_hist; b += 64) s_edges[b] = b < n_hist ? edges_g[b] : INFINITY;
    for (int j = tx; j < G; j += 64) s_l[j] = j < m ? J.l[j] : 0;
    if constexpr (TV) {
      if (P > 0) stage_profile(A, J, s_arr.prof);
    }
    __syncthreads();
  }
  const HistIdx hidx = hist_index_build(s_edges, n_hist, s_htab, &s_hsteps);
  const uint64_t seed = ((const uint64_t *)(A.ws + A.off_seed))[r];
  const uint32_t rid = ((const uint32_t *)(A.ws + A.off_rid))[r];

  const double d0 = J.d0, d1 = J.d1;
  const int32_t C = (int32_t)J.C;  // <= 2^30
  const int32_t cap_adm = (int32_t)(J.C - J.reserve_tok);
  const int32_t chunk = J.chunk;  // prefill tokens per iteration (0: whole prefills)
  const uint32_t qmask = (1u << J.qcap_log2) - 1u;
  const uint32_t rec_cap = (uint32_t)J.rec_cap;
  uint32_t *hist = (uint32_t *)(A.ws + A.off_hist) + r * (int64_t)A.hist_stride;
  // this lane's type (lanes without one: type 0's ring, never written)
  const int jt = is_t ? gl : 0;
  uint8_t *blk = A.ws + J.off_ring + (uint64_t)(r - J.replica_begin) * J.ring_stride;
  QRec *qr = (QRec *)(blk + J.off_q[0]);
  DRec *dr = (DRec *)(blk + J.off_d[jt]);
  const uint32_t dmask = (1u << J.dcap_log2[jt]) - 1u;
  const int32_t l = J.l[jt], lp = J.lp[jt];
  const double lam = J.lambda[jt];

  // replica-wide scalars, identical in every lane of the group
  double t, lat_area, ttft_area, lat_sum, mem_area, busy;
  int64_t batches, btok, idle, tridx;
  int32_t peak;
  // resident memory: at most C after a repair, plus one batch's growth (at
  // most C/2: every resident holds >= 2 tokens); admissions stay within C
  int32_t Mres;
  uint32_t qh, qt;  // ends of the external queue
  // chunked prefill: the partially prefilled prompt (at most one, the last
  // admitted), outside the deques until its last chunk: arrival time with
  // first-token flag, type (-1: none) and prompt tokens cached so far
  double part_a = 0.0;
  int32_t part_j = -1, part_pp = 0;
  // this lane's share of the replica's counters
  int64_t arrivals = 0, comps = 0, evicts = 0, etok = 0;
  uint32_t comp32 = 0, evict32 = 0;  // since the 64-bit counts were brought up to date
  uint32_t flags = 0;
  // this lane's type: ends of its deque, resident memory, residents at stage 1
  // without a first token, admission batch of the deque's first record, and
  // the deque's last record
  uint32_t dh, dt, pend, fkb, bkb, bkc;
  int32_t Mj;
  double ba;
  // Of the arrivals taken (in this call, Arrivals::rp) and the earlier ones
  // without a first token, ub have one by now: rp - ub lack one.
  uint32_t ub = 0;
  double t0 = INFINITY;  // a resumed call's pending arrival and its
  uint32_t k0 = 0;       // candidate counter
  uint32_t arr_rp = 0;   // rp when `arrivals` was last brought up to date

  if (!A.resume) {
    t = lat_area = ttft_area = lat_sum = mem_area = busy = 0.0;
    batches = btok = idle = tridx = 0;
    peak = Mres = Mj = 0;
    qh = qt = dh = dt = pend = 0;
    if (valid)  // whole row, padding included
      for (int b = gl; b < A.hist_stride; b += G) hist[b] = 0;
  } else {
    t = slot_f(A, S_T, r);
    lat_area = slot_f(A, S_LAT, r);
    ttft_area = slot_f(A, S_TTFT, r);
    lat_sum = slot_f(A, S_LATSUM, r);
    mem_area = slot_f(A, S_MEM, r);
    busy = slot_f(A, S_BUSY, r);
    batches = slot_i(A, S_BATCHES, r);
    btok = slot_i(A, S_BTOK, r);
    peak = (int32_t)slot_i(A, S_PEAK, r);
    idle = slot_i(A, S_IDLE, r);
    tridx = slot_i(A, S_TRIDX, r);
    Mres = (int32_t)slot_i(A, S_MRES, r);
    flags = (uint32_t)slot_i(A, S_FLAGS, r);
    part_a = slot_f(A, S_PARTA, r);
    part_j = (int32_t)slot_i(A, S_PARTJ, r);
    part_pp = (int32_t)slot_i(A, S_PARTPP, r);
    if (gl == 0) {
      ub = 0u - (uint32_t)slot_i(A, S_U, r);
      arrivals = slot_i(A, S_ARR, r);
      comps = slot_i(A, S_COMP, r);
      evicts = slot_i(A, S_EVICT, r);
      etok = slot_i(A, S_ETOK, r);
    }
    qh = (uint32_t)slot_i(A, S_QH, r);
    qt = (uint32_t)slot_i(A, S_QT, r);
    dh = is_t ? (uint32_t)slot_i(A, S_DH + jt, r) : 0u;
    dt = is_t ? (uint32_t)slot_i(A, S_DT + jt, r) : 0u;
    Mj = is_t ? (int32_t)slot_i(A, S_MJ + jt, r) : 0;
    pend = is_t ? (uint32_t)slot_i(A, S_LNEXT + jt, r) : 0u;
    if (is_t) {
      t0 = slot_f(A, S_TNEXT + jt, r);
      k0 = (uint32_t)slot_i(A, S_K + jt, r);
    }
  }
  const int64_t comps0 = comps;
  const int64_t ctok0 = A.resume && gl == 0 ? slot_i(A, S_CTOK, r) : 0;
  const int64_t batches0 = batches;  // + the batches of this call
  int64_t stop = -1;                 // those of a replica that ended early
  const Mask type_m = ballot(is_t);
  const Mask valid_m = ballot(valid);
  // groups still running
  Mask live = valid_m & ~group_spread<G>(ballot((flags & (kFlagCap | kFlagStall)) != 0));
  if (!in(live)) stop = 0;
  uint32_t wv = 0;  // deque records dt-wv .. dt-1 are in the window
  {  // ends of the deque (an empty one's are stale and not used)
    const DRec b = dr[(dt - 1u) & dmask];
    fkb = dr[dh & dmask].kb;
    ba = b.a_ft;
    bkb = b.kb;
    bkc = b.kc;
  }

  const bool draws = valid && is_t && !trace;
  Arrivals<G, TV, RING> arr(s_arr, A.nr * G, draws, seed, rid, lam, P, A.resume != 0, t0, k0);
  if (!trace) {
    // (one replica that runs low holds up the others of its wavefront: 20 calls of
    // one batch under a rate profile, 4,096 replicas of one type, 1.30 ms with 16
    // draws at the start and 1.16 with 32; a replica alone, 4 of them, 0.62 and 0.77)
    arr.start(live, A.nr > 1 ? 32u : 16u);
    if (draws && !A.resume && arr.limited()) flags |= kFlagThin;
  }
  ListArrivals<G> lst(s_arr.at, s_arr.ak, (const double *)(A.ws + J.off_tr_time),
                      (const int32_t *)(A.ws + J.off_tr_type), J.n_trace, tridx);
  if (trace) lst.start(live);

  // ---- the queue ----------------------------------------------------------
  // Records qh .. qc-1 are in LDS (a power of two of them at most, shared out
  // over the replicas of the wavefront).
  const uint32_t qdepth = min((uint32_t)QRING / (uint32_t)A.nr, 64u);
  QLds *const sq = s_q + (valid ? (uint32_t)q * qdepth : 0u);
  uint32_t qc = qh;
  // Append a record of lane `me`'s type to the queue of each group in `go`.
  // (A full queue ends the replica at its next decision and is not read
  // again, so the stores are unconditional.)
  auto push_q = [&](Mask go, Mask me, double a_ft) __attribute__((always_inline)) {
    const bool near = qc == qt && qt - qh < qdepth;  // everything queued is in LDS
    if (in(me)) {
      QRec rec;
      rec.a_ft = a_ft;
      rec.j = gl;
      rec.L = lp;
      qr[qt & qmask] = rec;
      if (near) {
        QLds x;
        x.a_ft = a_ft;
        x.j = gl;
        x.l = l;
        sq[qt & (qdepth - 1u)] = x;
      }
    }
    if (in(go)) {
      flags |= qt - qh >= rec_cap ? kFlagCap : 0u;
      qc += near ? 1u : 0u;
      qt++;
    }
  };
  // Load the next records behind the ones in LDS (as many as the group's
  // lanes take and LDS has room for); land() stores them there.
  uint4 ld[NL];
  uint32_t ld_n = 0;
  auto load_q = [&](Mask go) __attribute__((always_inline)) {
    if (in(go)) {
      ld_n = min(min(qt - qc, qdepth - (qc - qh)), (uint32_t)(G * NL));
#pragma unroll
      for (int i = 0; i < NL; ++i)
        if ((uint32_t)(gl + i * G) < ld_n) ld[i] = ((const uint4 *)qr)[(qc + (uint32_t)(gl + i * G)) & qmask];
    }
  };
  auto land_q = [&](Mask go) __attribute__((always_inline)) {
    if (in(go)) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        if ((uint32_t)(gl + i * G) < ld_n) {
          QLds x;
          x.a_ft = __longlong_as_double((long long)(((uint64_t)ld[i].y << 32) | ld[i].x));
          x.j = (int32_t)ld[i].z;
          x.l = s_l[x.j & (G - 1)];
          sq[(qc + (uint32_t)(gl + i * G)) & (qdepth - 1u)] = x;
        }
      }
      qc += ld_n;
      ld_n = 0;
    }
    wave_lds_sync();
  };

  // ---- arrivals -------------------------------------------------------------
  // The group's next arrival and the lanes of its type(s).
  auto peek = [&](Mask &mine) __attribute__((always_inline)) -> double {
    if constexpr (LIST) {
      if (trace) {
        mine = ballot(gl == lst.jn);
        return lst.tn;
      }
    }
    const double ta = group_min<G>(arr.tn);
    mine = ballot(arr.tn == ta);
    return ta;
  };
  // One arrival of each group in `go` joins the queue: the lane in `mine` (of
  // simultaneous ones the lowest) takes it at time ta and moves to its
  // type's next arrival.  A group whose queue was full leaves `more`.
  auto take = [&](Mask go, Mask mine, double ta, Mask &more) __attribute__((always_inline)) {
    Mask me = go & mine;
    if constexpr (G > 1) {
      if (__popcll(me) * G != __popcll(go)) me = group_lowest<G>(me);
    }
    // rare: the ring of arrival times runs low, or the queue is full
    const Mask low = arr.low();
    const Mask full = ballot(qt - qh >= rec_cap);
    more &= ~(go & full);
    if ((me & low) != 0) arr.refill(live, me);
    push_q(go, me, ta);
    if (in(me)) {
      if (trace) {
        arr.rp++;
      } else {
        arr.advance();
        if (arr.limited()) flags |= kFlagThin;
      }
    }
    if (trace) lst.advance(go, live);
  };

  // Push a prompt admitted in this batch, at position p, at the back of this
  // lane's deque.
  uint32_t fresh = 0, pnew = 0;  // of them, and those without a first token
  auto push_d = [&](double a, uint32_t kb, uint32_t p) __attribute__((always_inline)) {
    DRec rec;
    rec.a_ft = a;
    rec.kb = kb;
    rec.kc = p;
    dr[dt & dmask] = rec;
    s_win[dt % WB][tx] = rec;
    fkb = dt == dh ? kb : fkb;
    ba = a;
    bkb = kb;
    bkc = p;
    dt++;
    wv = min(wv + 1u, (uint32_t)WB);
    fresh++;
    pnew += has_ft(a) ? 0u : 1u;
  };

  int64_t it = 0;
  for (; it < A.horizon; ++it) {
    if ((it & 255) == 255) {  // 32-bit counts to 64 bits
      arrivals += arr.rp - arr_rp;
      arr_rp = arr.rp;
      comps += comp32;
      comp32 = 0;
      evicts += evict32;
      evict32 = 0;
    }
    // ---- decision: form a batch or wait for the next arrival -----------------
    int32_t N0, U0;
    for (;;) {
      const Mask cap = ballot((flags & kFlagCap) != 0) & live;
      if (cap != 0) {
        const Mask dead = group_spread<G>(cap);
        if (in(dead)) stop = it;
        live &= ~dead;
      }
      const int32_t resident = group_sum32<G>((int32_t)(dt - dh)) + (part_j >= 0 ? 1 : 0);
      N0 = (int32_t)(qt - qh) + resident;
      U0 = group_sum32<G>((int32_t)(arr.rp - ub));
      Mask wait = ballot(N0 == 0) & live;
      if (wait == 0) break;
      Mask mine;
      const double ta = peek(mine);
      const Mask none = wait & ballot(!(ta < INFINITY));
      if (none != 0) {
        if (in(none)) {
          flags |= kFlagStall;
          stop = it;
        }
        live &= ~none;
        wait &= ~none;
      }
      if (in(wait)) {
        const double dtm = ta - t;
        lat_area += (double)N0 * dtm;
        ttft_area += (double)U0 * dtm;
        mem_area += (double)Mres * dtm;
        t = ta;
        idle++;
      }
      // every arrival at this instant joins before the next decision; a full
      // queue ends the replica, which also bounds this loop
      while (wait != 0) {
        take(wait, mine, ta, wait);
        wait &= ballot(peek(mine) == ta);
      }
    }
    if (live == 0) break;

    // ---- launch: admissions and batch tokens ----------------------------------
    const uint32_t bidx = (uint32_t)(batches0 + it);
    const uint32_t before = dt - dh;
    // the deque's front completes in this batch (prompts admitted now never do)
    const Mask fin = ballot(before > 0u) & ballot(fkb + (uint32_t)lp == bidx) & live & type_m;
    int32_t prefill_l = 0, budget = chunk > 0 ? chunk : INT32_MAX;
    uint32_t p = 0;        // position in the batch
    int32_t bt_pre = 0;    // per-batch trace: prefill processings
    fresh = pnew = 0;
    if (chunk > 0) {  // the partially prefilled prompt first
      const Mask part = ballot(part_j >= 0) & live;
      if (part != 0) {
        const int32_t pl = s_l[part_j >= 0 ? part_j : 0];
        const int32_t cq = min(pl - part_pp, budget);
        const Mask whole = part & ballot(part_pp + cq == pl);
        if (in(whole & ballot(gl == part_j))) push_d(part_a, bidx, p);
        if (in(part)) {
          budget -= cq;
          prefill_l = cq;
          part_pp += cq;
          bt_pre = 1;
        }
        if (in(whole)) {  // its last chunk: a fresh resident of its type
          part_j = -1;
          part_pp = 0;
          p = 1;
        }
      }
    }
    // The resident memory includes a partial prompt's earlier chunks, so the
    // batch's tokens are that and the prefill tokens of this batch.
    wave_lds_sync();
    Mask can = live;
    for (;;) {
      can &= ballot(qt != qh) & ballot(budget > 0);
      if (can == 0) break;
      const Mask out = can & ballot(qh == qc);
      if (out != 0) {  // nothing left in LDS: wait for the next records
        load_q(out);
        land_q(out);
      }
      const QLds head = sq[qh & (qdepth - 1u)];
      can &= ballot((uint32_t)Mres + (uint32_t)(prefill_l + head.l) <= (uint32_t)cap_adm);
      if (can == 0) break;
      const int32_t cq = min(head.l, budget);
      const Mask whole = can & ballot(cq == head.l);
      if (in(whole & ballot(gl == head.j))) push_d(head.a_ft, bidx, p);
      if (in(can)) {
        qh++;
        budget -= cq;
        prefill_l += cq;
        bt_pre++;
      }
      if (in(whole)) {
        p++;
      } else if (in(can)) {  // the budget ends inside this prompt
        part_a = head.a_ft;
        part_j = head.j;
        part_pp = cq;
      }
    }
    const int32_t sel_part = part_j >= 0 ? 1 : 0;
    const int32_t tokens = Mres + prefill_l;
    const int32_t m_launch = tokens;
    const double tau = d0 + d1 * (double)tokens;
    const double t_end = t + tau;
    // The records that the completion step uses are loaded now and land then:
    // the front of the deque, and the queue's next ones.
    DRec c[KC];
    if (in(fin)) {
#pragma unroll
      for (int u = 0; u < KC; ++u) c[u] = dr[(dh + (uint32_t)u) & dmask];
    }
    const Mask ahead = ballot(qc != qt) & ballot(qc - qh <= qdepth / 2u) & live;
    load_q(ahead);

    // ---- arrivals during the batch ----------------------------------------
    Mask inb = live;
    if (trace) {
      for (;;) {
        const Mask go = ballot(lst.tn <= t_end) & inb;
        if (go == 0) break;
        const double w = in(go) ? t_end - lst.tn : 0.0;  // (areas are never -0)
        lat_area += w;
        ttft_area += w;
        const Mask me = go & ballot(gl == lst.jn);
        inb &= ~ballot(qt - qh >= rec_cap);
        push_q(go, me, lst.tn);
        if (in(me)) arr.rp++;
        lst.advance(go, live);
      }
    } else {
      for (;;) {
        Mask mine;
        const double ta = peek(mine);
        const Mask go = ballot(ta <= t_end) & inb;
        if (go == 0) break;
        const double w = in(go) ? t_end - ta : 0.0;
        lat_area += w;
        ttft_area += w;
        take(go, mine, ta, inb);
      }
    }
    if (in(live)) {
      lat_area += (double)N0 * tau;
      ttft_area += (double)U0 * tau;
      mem_area += (double)m_launch * tau;
      busy += tau;
      t = t_end;
      peak = max(peak, m_launch);
      btok += tokens;
    }

    // ---- completion transition ----------------------------------------------
    const uint32_t cp0 = comp32, ev0 = evict32;
    uint32_t done = 0;
    if (in(live)) {
      // the stage-1 cohort produces its first tokens
      ub += pend;
      pend = pnew;
    }
    // the loads of the launch arrive here, before the histogram's updates
    // (memory operations complete in order)
    if (ahead != 0) land_q(ahead);
    if (fin != 0) {
      auto count = [&](int bin) __attribute__((always_inline)) {
        __hip_atomic_fetch_add(&hist[bin], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      double part = 0.0;  // the type's latencies in admission order
      // do lanes complete a second prompt?
      const Mask more = ballot(before > 1u) & ballot(c[1].kb + (uint32_t)lp == bidx) & fin;
      if (more == 0) {
        if (in(fin)) {
          part = t_end - arrival_of(c[0].a_ft);
          count(hist_bin_idx(s_edges, s_htab, hidx, part));
          done = 1;
          fkb = c[1].kb;
        }
      } else {
        if (in(fin)) {  // cohorts, KC records at a time
          for (;;) {
            double lat[KC];
            int bin[KC];
            uint32_t n = 0;  // of these, the ones that complete (they lead)
#pragma unroll
            for (int u = 0; u < KC; ++u) {
              lat[u] = t_end - arrival_of(c[u].a_ft);
              const bool ok = done + (uint32_t)u < before && c[u].kb + (uint32_t)lp == bidx;
              n += n == (uint32_t)u && ok ? 1u : 0u;
              fkb = n == (uint32_t)u ? c[u].kb : fkb;
            }
            hist_bins<KC>(s_edges, s_htab, hidx, lat, bin);
#pragma unroll
            for (int u = 0; u < KC; ++u) {
              if ((uint32_t)u < n) {
                part += lat[u];
                count(bin[u]);
              }
            }
            done += n;
            if (n < (uint32_t)KC) break;
#pragma unroll
            for (int u = 0; u < KC; ++u) c[u] = dr[(dh + done + (uint32_t)u) & dmask];
          }
        }
      }
      comp32 += done;
      dh += done;
      lat_sum = add_in_order<G>(lat_sum, part, fin);
    }

    // ---- repair: evict the most recently admitted residents ------------------
    if (in(live))
      Mj += (int32_t)(before - done) + (int32_t)fresh * (l + 1) - (int32_t)done * (l + lp);
    const int32_t Msum = group_sum32<G>(Mj) + (part_j >= 0 ? part_pp : 0);
    Mres = in(live) ? Msum : Mres;
    peak = max(peak, Mres);  // (a replica that has ended keeps its resident memory)
    Mask over = ballot(Mres > C) & live;
    if (over != 0) {
      // a partially prefilled prompt first; it restarts from scratch
      const Mask part = over & ballot(part_j >= 0);
      if (part != 0) {
        push_q(part, part & ballot(gl == part_j), part_a);
        if (in(part)) {
          Mres -= part_pp;
          if (gl == 0) evict32++;
          part_j = -1;
          part_pp = 0;
        }
        over &= ballot(Mres > C);
      }
    }
    // then the largest (batch, position) among the deques' backs
    if (over != 0) {
      uint32_t lost = 0;  // decode tokens
      do {
        const Mask cand = ballot(dt != dh) & over;
        const uint32_t age = in(cand) ? bidx - bkb : ~0u;
        const uint32_t best = group_reduce32<G>(age, [](uint32_t a, uint32_t b) { return min(a, b); });
        const Mask newest = ballot(age == best) & cand;
        const uint32_t pos = in(newest) ? bkc + 1u : 0u;
        const uint32_t last = group_reduce32<G>(pos, [](uint32_t a, uint32_t b) { return max(a, b); });
        const Mask me = ballot(pos == last) & newest;
        over &= group_spread<G>(cand);  // a group without residents has done all it can
        const int32_t stage = (int32_t)(bidx - bkb) + 1;
        const Mask miss = ballot(wv < 2u) & ballot(dt != dh + 1u) & me;
        if (miss != 0) {  // rare: the new back is not in the window
          if (in(miss)) {
            s_win[(dt - 2u) % WB][tx] = dr[(dt - 2u) & dmask];
            wv = 2u;
          }
        }
        // the back record returns to the tail of the queue with its
        // first-token flag
        const bool ft = has_ft(ba);
        push_q(over, me, ft || stage >= 2 ? with_ft(ba) : ba);
        int32_t ch = 0;
        if (in(me)) {
          dt--;
          const DRec b = s_win[(dt - 1u) % WB][tx];  // (not used if the deque is empty)
          wv = wv > 0u ? wv - 1u : 0u;
          ch = l + stage;
          Mj -= ch;
          evict32++;
          lost += (uint32_t)(stage - 1);
          pend -= (stage == 1 && !ft) ? 1u : 0u;
          ba = b.a_ft;
          bkb = b.kb;
          bkc = b.kc;
        }
        Mres -= group_sum32<G>(ch);
        over &= ballot(Mres > C);
      } while (over != 0);
      etok += lost;
    }
    if constexpr (TV) {
      if (A.btrace != nullptr) {
        const int32_t bt_comps = group_sum32<G>((int32_t)(comp32 - cp0));
        const int32_t bt_ev = group_sum32<G>((int32_t)(evict32 - ev0));
        const int32_t bt_sel = group_sum32<G>((int32_t)(before + fresh)) + sel_part;
        const int32_t res = group_sum32<G>((int32_t)(dt - dh)) + (part_j >= 0 ? 1 : 0);
        if (in(live) && gl == 0 && batches0 + it < A.btrace_cap) {
          BatchRec br;
          br.t_launch = t_end - tau;
          br.tau = tau;
          br.tokens = tokens;
          br.prefills = bt_pre;
          br.selected = bt_sel;
          br.completions = bt_comps;
          br.evict_pre = 0;
          br.evict_post = bt_ev;
          br.mem_after = Mres;
          br.waiting_after = (int64_t)(qt - qh);
          br.resident_after = res;
          br.mplus = 0;
          ((BatchRec *)A.btrace)[r * A.btrace_cap + batches0 + it] = br;
        }
      }
    }
  }

  // ---- save state --------------------------------------------------------
  comps += comp32;
  evicts += evict32;
  batches = batches0 + (stop >= 0 ? stop : it);
  const int64_t ctok = group_sum<G>((comps - comps0) * lp + ctok0);
  arrivals = group_sum<G>(arrivals + (int64_t)(arr.rp - arr_rp));
  comps = group_sum<G>(comps);
  evicts = group_sum<G>(evicts);
  etok = group_sum<G>(etok);
  const int32_t U = group_sum32<G>((int32_t)(arr.rp - ub));
  const int32_t N = group_sum32<G>((int32_t)(dt - dh)) + (int32_t)(qt - qh) + (part_j >= 0 ? 1 : 0);
  flags = group_or<G>(flags);
  if (!valid) return;
  if (gl == 0) {
    put_f(A, S_T, r, t);
    put_f(A, S_LAT, r, lat_area);
    put_f(A, S_TTFT, r, ttft_area);
    put_f(A, S_LATSUM, r, lat_sum);
    put_f(A, S_MEM, r, mem_area);
    put_f(A, S_BUSY, r, busy);
    put_i(A, S_BATCHES, r, batches);
    put_i(A, S_ARR, r, arrivals);
    put_i(A, S_COMP, r, comps);
    put_i(A, S_CTOK, r, ctok);
    put_i(A, S_EVICT, r, evicts);
    put_f(A, S_PARTA, r, part_a);
    put_i(A, S_PARTJ, r, part_j);
    put_i(A, S_PARTPP, r, part_pp);
    put_i(A, S_ETOK, r, etok);
    put_i(A, S_FALLBACK, r, 0);
    put_i(A, S_BTOK, r, btok);
    put_i(A, S_PEAK, r, peak);
    put_i(A, S_IDLE, r, idle);
    put_i(A, S_N, r, N);
    put_i(A, S_U, r, U);
    put_i(A, S_MRES, r, Mres);
    put_i(A, S_TRIDX, r, trace ? lst.index() : tridx);
    put_i(A, S_FLAGS, r, (int64_t)flags);
    put_i(A, S_QH, r, qh);
    put_i(A, S_QT, r, qt);
  }
  if (is_t) {
    put_f(A, S_TNEXT + gl, r, draws ? arr.tn : t0);
    put_i(A, S_K + gl, r, draws ? arr.pending() : k0);
    put_i(A, S_DH + gl, r, dh);
    put_i(A, S_DT + gl, r, dt);
    put_i(A, S_MJ + gl, r, Mj);
    put_i(A, S_LNEXT + gl, r, pend);
  }
}

template <int G, bool TV, bool LIST>
hipError_t launch_fcfs_g(KArgs A, hipStream_t s) {
  // replicas per wavefront: what the group width allows, within the list's
  A.nr = 64 / G < A.lanes ? 64 / G : A.lanes;
  if (A.n_list % 64 != 0 || A.lanes % A.nr != 0) return hipErrorInvalidValue;
  while (A.nr > 1 && (int64_t)(A.n_list / 64) * (A.lanes / A.nr) < A.min_waves) A.nr /= 2;
  return launch_checked(sim_fcfs_kernel<G, TV, LIST>, dim3((A.n_list / 64) * (A.lanes / A.nr)), s, A);
}

template <bool TV, bool LIST>
hipError_t launch_fcfs_k(int max_m, const KArgs &A, hipStream_t s) {
  if (max_m <= 1) return launch_fcfs_g<1, TV, LIST>(A, s);
  if (max_m <= 2) return launch_fcfs_g<2, TV, LIST>(A, s);
  if (max_m <= 4) return launch_fcfs_g<4, TV, LIST>(A, s);
  if (max_m <= 8) return launch_fcfs_g<8, TV, LIST>(A, s);
  if (max_m <= 16) return launch_fcfs_g<16, TV, LIST>(A, s);
  return hipErrorInvalidValue;  // more types run in the kernel for drawn lengths
}

}  // namespace
}  // namespace wsim
