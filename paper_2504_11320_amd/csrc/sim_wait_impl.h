// sim_wait_impl.h -- simulation kernel for WAIT with known output lengths
// (arXiv 2504.11320: Algorithm 1; the threshold-without-waiting form and the
// time-varying rates of the appendix; per-stage caps of Section 6).
//
// A group of G lanes (G = 1, 2, 4, ... 64, a power of two >= the job's types)
// runs one replica; lane g of a group owns request type g: its arrival clock
// and draws, its external queue, its resident deque, its services and its
// resident memory, all plain scalars in registers.  What a batch does type by
// type -- eligibility, admissions, completions, evictions of this batch's
// admissions -- runs on the type lanes at once; what couples the types (batch
// tokens, the earliest arrival, the resident memory, the most recent
// admission) are group reductions by DPP lane permutations.  Replica-wide
// scalars (clock, censored areas, resident memory) are kept identical in
// every lane of the group.  Loops are wavefront-uniform (a group that is done
// stays in as inactive), so a draw pass inside them has all 64 lanes.
//
// Records live in HBM rings of the replica's workspace block: per type an
// external queue (8 bytes: arrival time, first-token flag in the sign bit)
// and a resident deque in admission order (16 bytes: DRec).  Under WAIT a
// served type advances every resident prompt of that type (each stage holds
// at most n_j prompts, so min(n_j, n_js) = n_js, as in the resident-memory
// lemma of the Theorem 1 proof): a prompt's stage is the number of services
// of its type since admission and the residents of one type complete in
// admission order, so admissions push at the back of the deque, completions
// pop at the front, LIFO evictions pop at the back, and a step costs
// O(events), not O(stages).
//
// Arithmetic is the model's (the same IEEE operations, no FMA contraction), in
// its order but for three sums: a batch's arrivals and its completions sum their
// area terms and latencies per type, in time and in admission order, then the
// types in turn (the model adds them one by one).
//
// What bounds it: a replica is a serial chain of events, so a wavefront's
// latency per batch.  Per wavefront and batch of the Llama-shaped unit
// threshold sweep (32,768 replicas, 16 to a wavefront, two wavefronts per
// SIMD) it issues 384 vector, 119 scalar and 49 branch instructions (the SIMDs
// issue 70 % of the time); one lane per replica with per-type register arrays
// (select chains, one body per type) took 24.2 ms per 5,000 batches, this 14.2.
// 56 % of a wavefront's cycles are waits, so every record of a batch is loaded
// at its launch and waited for once, at its completion step, before the
// histogram's updates: a wait after them would wait for them too (17.4 ms).
#pragma once

#include "sim_arrivals.h"

namespace wsim {
namespace {

// TV: the general instantiation (time-varying rates, per-stage caps, per-batch
// trace); LIST: arrival lists too.  ONE: every threshold is 1 (at most one
// admission and one completion per type and batch).
template <int G, bool TV, bool ONE, bool LIST>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
sim_wait_kernel(KArgs A) {
  // Arrival times are drawn ahead of use by the whole wavefront into a ring
  // per lane, as deep as the lanes in use leave room for.
  constexpr int RING = ONE ? 1024 : 512;  // ring entries of a wavefront
  // the last records pushed on each deque, for LIFO evictions
  constexpr int WB = 8;
  // records loaded at the launch for use at the completion: a cohort's queue
  // records (a larger cohort enters the deque at the launch) and the records
  // at the front of the deque (fewer with lists, whose state would push 16 and
  // 8 into scratch memory: 124 bytes a lane)
  constexpr int KQ = ONE ? 1 : LIST ? 4 : 16;
  constexpr int VQ = LIST ? 3 : 5;  // of a cohort's records after the first, at a time
  constexpr int KC = ONE || LIST ? 2 : 8;
  __shared__ typename Arrivals<G, TV, RING>::Lds s_arr;
  __shared__ DRec s_win[WB][64];
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
  const bool nowait = J.nowait != 0;
  const uint32_t qmask = (1u << J.qcap_log2) - 1u;
  const uint32_t rec_cap = (uint32_t)J.rec_cap;
  uint32_t *hist = (uint32_t *)(A.ws + A.off_hist) + r * (int64_t)A.hist_stride;
  // this lane's type (lanes without one: type 0's rings, never written)
  const int jt = is_t ? gl : 0;
  uint8_t *blk = A.ws + J.off_ring + (uint64_t)(r - J.replica_begin) * J.ring_stride;
  double *qr = (double *)(blk + J.off_q[jt]);
  DRec *dr = (DRec *)(blk + J.off_d[jt]);
  const uint32_t dmask = (1u << J.dcap_log2[jt]) - 1u;
  const int32_t l = J.l[jt], lp = J.lp[jt], nth = J.n[jt];
  const double lam = J.lambda[jt];
  const int32_t chf = l + 1;              // charge of a prompt admitted in this batch
  const double inv_chf = 1.0 / (double)chf;
  // WAIT per-stage caps (Section 6; general instantiation only): the type
  // takes the caps of its l'_j + 1 stages in turn, one per service, as its
  // threshold and cohort size
  const bool capped = TV && J.has_caps != 0;
  const int32_t *capt = (const int32_t *)(A.ws + J.off_caps);
  if constexpr (TV) {
    if (capped)
      for (int j = 0; j < jt; ++j) capt += J.lp[j] + 1;
  }

  // replica-wide scalars, identical in every lane of the group
  double t, lat_area, ttft_area, lat_sum, mem_area, busy;
  int64_t batches, btok, idle, tridx;
  int32_t peak;
  // resident memory: at most C after a repair, plus one batch's growth (at
  // most C/2: every resident holds >= 2 tokens) and admissions (sum_j n_j
  // (l_j + 1) < 2^29, checked on the host), so < 2^31
  int32_t Mres;
  // this lane's share of the replica's counters
  int64_t arrivals = 0, comps = 0, evicts = 0, etok = 0;
  uint32_t comp32 = 0, evict32 = 0;  // since the 64-bit counts were brought up to date
  uint32_t flags = 0;
  // this lane's type: ends of its queue and deque, services, resident memory,
  // residents at stage 1 without a first token, admission service of the
  // deque's first record, and the deque's last record
  uint32_t qh, qt, dh, dt, svc, pend, fkc, bkb, bkc;
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
    qh = qt = dh = dt = svc = pend = 0;
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
    if (gl == 0) {
      ub = 0u - (uint32_t)slot_i(A, S_U, r);
      arrivals = slot_i(A, S_ARR, r);
      comps = slot_i(A, S_COMP, r);
      evicts = slot_i(A, S_EVICT, r);
      etok = slot_i(A, S_ETOK, r);
    }
    qh = is_t ? (uint32_t)slot_i(A, S_QH + jt, r) : 0u;
    qt = is_t ? (uint32_t)slot_i(A, S_QT + jt, r) : 0u;
    dh = is_t ? (uint32_t)slot_i(A, S_DH + jt, r) : 0u;
    dt = is_t ? (uint32_t)slot_i(A, S_DT + jt, r) : 0u;
    svc = (uint32_t)slot_i(A, S_SVC + jt, r);
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
  auto cap_of = [&](uint32_t services) __attribute__((always_inline)) -> int32_t {
    return TV && capped && is_t ? capt[services % (uint32_t)(lp + 1)] : nth;
  };
  int32_t ncap = cap_of(svc);
  {  // ends of the deque (an empty one's are stale and not used)
    const DRec b = dr[(dt - 1u) & dmask];
    fkc = dr[dh & dmask].kc;
    ba = b.a_ft;
    bkb = b.kb;
    bkc = b.kc;
  }

  const bool draws = valid && is_t && !trace;
  Arrivals<G, TV, RING> arr(s_arr, A.nr * G, draws, seed, rid, lam, P, A.resume != 0, t0, k0);
  if (!trace) {
    arr.start(live);
    if (draws && !A.resume && arr.limited()) flags |= kFlagThin;
  }
  ListArrivals<G> lst(s_arr.at, s_arr.ak, (const double *)(A.ws + J.off_tr_time),
                      (const int32_t *)(A.ws + J.off_tr_type), J.n_trace, tridx);
  if (trace) lst.start(live);

  // ---- arrivals ---------------------------------------------------------------
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
  // One arrival of each group in `go` joins its queue: the lane in `mine` (of
  // simultaneous ones the lowest) takes it at time ta and moves to its
  // type's next arrival.  A group whose queue was full (it ends at its next
  // decision) leaves `more`.  Returns the lanes that took one.
  auto take = [&](Mask go, Mask mine, double ta, Mask &more) __attribute__((always_inline)) -> Mask {
    Mask me = go & mine;
    if constexpr (G > 1) {
      if (__popcll(me) * G != __popcll(go)) me = group_lowest<G>(me);
    }
    // rare: the ring of arrival times runs low, or the queue is full
    const Mask low = arr.low();
    const Mask full = ballot(qt - qh >= rec_cap);
    if ((me & (low | full)) != 0) {
      if (in(me & full)) flags |= kFlagCap;
      more &= ~group_spread<G>(me & full);
      if ((me & low) != 0) arr.refill(live, me);
    }
    if (in(me)) {
      qr[qt & qmask] = ta;  // a full queue is not read again
      qt++;
      if (trace) {
        arr.rp++;
      } else {
        arr.advance();
        if (arr.limited()) flags |= kFlagThin;
      }
    }
    if (trace) lst.advance(go, live);
    return me;
  };

  // This batch's admissions join the deque: the x-th of them is stored; then
  // the deque's ends follow once for all of them.
  uint32_t pnew = 0;  // those without a first token
  auto put_d = [&](uint32_t x, double a, uint32_t kb, uint32_t kcs) __attribute__((always_inline)) {
    DRec rec;
    rec.a_ft = a;
    rec.kb = kb;
    rec.kc = kcs;
    dr[(dt + x) & dmask] = rec;
    s_win[(dt + x) % WB][tx] = rec;
    ba = a;
    pnew += has_ft(a) ? 0u : 1u;
  };
  auto grow_d = [&](uint32_t n, uint32_t kb, uint32_t kcs) __attribute__((always_inline)) {
    fkc = dt == dh ? kcs : fkc;
    bkb = kb;
    bkc = kcs;
    dt += n;
    wv = min(wv + n, (uint32_t)WB);
  };
  // LIFO eviction of this lane's last k records, all admitted in the current
  // batch: they are at stage 1 with the charge l + 1, lose no decode token
  // and keep their first-token flags.
  auto evict_fresh = [&](uint32_t k) __attribute__((always_inline)) {
    const uint32_t t0 = dt;
    for (uint32_t i = 0; i < k; ++i) {
      const double a = dr[(t0 - 1u - i) & dmask].a_ft;
      pend -= has_ft(a) ? 0u : 1u;
      qr[(qt + i) & qmask] = a;
    }
    qt += k;
    dt = t0 - k;
    wv = wv > k ? wv - k : 0u;
    if (dt != dh) {  // the new back record
      if (wv < 1u) {
        s_win[(dt - 1u) % WB][tx] = dr[(dt - 1u) & dmask];
        wv = 1u;
      }
      const DRec b = s_win[(dt - 1u) % WB][tx];
      ba = b.a_ft;
      bkb = b.kb;
      bkc = b.kc;
    }
    Mj -= (int32_t)k * chf;
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
    // ---- decision: the eligible types, or wait for the next arrival ------
    Mask served;
    for (;;) {
      const Mask cap = ballot((flags & kFlagCap) != 0) & live;
      if (cap != 0) {
        const Mask dead = group_spread<G>(cap);
        if (in(dead)) stop = it;
        live &= ~dead;
      }
      const uint32_t waiting = qt - qh;
      served = nowait ? ballot(waiting != 0u) | ballot(dt != dh) : ballot(waiting >= (uint32_t)ncap);
      served &= live & type_m;
      Mask wait = live & ~group_spread<G>(served);
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
      const int32_t N = group_sum32<G>((int32_t)((qt - qh) + (dt - dh)));
      const int32_t U = group_sum32<G>((int32_t)(arr.rp - ub));
      if (in(wait)) {
        const double dtm = ta - t;
        lat_area += (double)N * dtm;
        ttft_area += (double)U * dtm;
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

    // ---- launch: admissions, completions to come, batch tokens --------------
    const uint32_t bidx = (uint32_t)(batches0 + it);
    const uint32_t now = svc + 1u;
    const int32_t N0 = group_sum32<G>((int32_t)((qt - qh) + (dt - dh)));
    const int32_t U0 = group_sum32<G>((int32_t)(arr.rp - ub));
    uint32_t na = nowait ? min(qt - qh, (uint32_t)nth) : (uint32_t)ncap;
    na = in(served) ? na : 0u;
    // the deque's front completes in this batch (prompts admitted now never do)
    const uint32_t before = dt - dh;
    const Mask fin = ballot(before > 0u) & ballot(fkc + (uint32_t)lp == now) & served;
    // The records that the completion step uses are loaded now and waited for
    // then: the queue's first ones (admitted), and the front of the deque.
    double qa[KQ];
    DRec c[KC];
    pnew = 0;
    uint32_t nd = na;  // admitted prompts that join the deque at the completion
    Mask early = 0;
    if constexpr (!ONE) {
      // a cohort larger than KQ enters the deque now, four at a time
      early = ballot(na > (uint32_t)KQ);
      if (in(early)) {
        for (uint32_t x = 0; x < na; x += 4) {
          double nx[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) nx[u] = qr[(qh + x + (uint32_t)u) & qmask];
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (x + (uint32_t)u < na) put_d(x + (uint32_t)u, nx[u], bidx, now);
        }
        grow_d(na, bidx, now);
        nd = 0;
      }
    }
    const Mask adm = ballot(nd > 0u);
#pragma unroll
    for (int u = 0; u < KQ; ++u) qa[u] = 0.0;
    if (in(adm)) qa[0] = qr[qh & qmask];
    if constexpr (!ONE) {
#pragma unroll
      for (int v = 1; v < KQ; v += VQ) {
        if (ballot(nd > (uint32_t)v) != 0) {
#pragma unroll
          for (int u = v; u < v + VQ; ++u) qa[u] = qr[(qh + (uint32_t)u) & qmask];
        }
      }
    }
    if (in(fin)) {
#pragma unroll
      for (int u = 0; u < KC; ++u) c[u] = dr[(dh + (uint32_t)u) & dmask];
    }
    const int32_t pre = (int32_t)na * l;
    const int32_t prefill_l = group_sum32<G>(pre);
    const int32_t tokens = group_sum32<G>(pre + (in(served) ? Mj : 0));
    const int32_t m_launch = Mres + prefill_l;
    const double tau = d0 + d1 * (double)tokens;
    const double t_end = t + tau;
    qh += na;

    // ---- arrivals during the batch ----------------------------------------
    // Each type takes its own, in time order, and sums their area terms; the
    // sums join the areas in type order.  Types need no order between them
    // but where a queue overflows: that ends the group's arrivals at its
    // instant.
    Mask inb = live;
    double part_a = 0.0;
    auto in_order = [&](Mask who, double tm) __attribute__((always_inline)) {
      for (;;) {
        Mask mine;
        const double ta = peek(mine);
        const Mask go = ballot(ta <= t_end) & ballot(ta < tm) & who & inb;
        if (go == 0) break;
        const Mask me = take(go, mine, ta, inb);
        part_a += in(me) ? t_end - ta : 0.0;
      }
    };
    if (trace) {  // the list's next arrival, whichever its type
      for (;;) {
        const Mask go = ballot(lst.tn <= t_end) & inb;
        if (go == 0) break;
        const Mask me = go & ballot(gl == lst.jn);
        if (in(me)) {
          part_a += t_end - lst.tn;
          qr[qt & qmask] = lst.tn;
          qt++;
          arr.rp++;
        }
        const Mask full = ballot(qt - qh > rec_cap) & me;
        if (full != 0) {
          if (in(full)) flags |= kFlagCap;
          inb &= ~group_spread<G>(full);
        }
        lst.advance(go, live);
      }
    } else {
      for (bool stuck = false;;) {
        // up to what every ring of the group knows
        double tm = group_min<G>(arr.te);
        Mask more = ballot(tm <= t_end) & inb;
        if (more != 0) {
          arr.refill(live, inb & ballot(arr.te <= t_end));
          tm = group_min<G>(arr.te);
          more = ballot(tm <= t_end) & inb;
        }
        const uint32_t qt0 = qt, rp0 = arr.rp, flags0 = flags;
        const double pa0 = part_a;
        Mask run = ballot(arr.tn <= t_end) & ballot(arr.tn < tm) & inb;
        if (run == 0 && more != 0 && stuck) {
          // rings full of one instant (gaps below the clock's resolution)
          in_order(live, INFINITY);
          break;
        }
        stuck = run == 0;
        while (run != 0) {
          if (in(run)) {
            part_a += t_end - arr.tn;
            qr[qt & qmask] = arr.tn;
            qt++;
            arr.advance();
            if (arr.limited()) flags |= kFlagThin;
          }
          run &= ballot(arr.tn <= t_end) & ballot(arr.tn < tm);
        }
        const Mask full = ballot(qt - qh > rec_cap) & inb;
        if (full != 0) {  // rare: again in time order, up to the overflow
          const Mask again = group_spread<G>(full);
          if (in(again)) {
            qt = qt0;
            part_a = pa0;
            flags = flags0;
            if (draws) arr.rewind(rp0);
          }
          in_order(again, tm);
        }
        if (more == 0) break;
      }
    }
    {
      const double sum = add_in_order<G>(0.0, part_a, ballot(part_a != 0.0));
      if (in(live)) {
        lat_area += sum;
        ttft_area += sum;
        lat_area += (double)N0 * tau;
        ttft_area += (double)U0 * tau;
        mem_area += (double)m_launch * tau;
        busy += tau;
        t = t_end;
        peak = max(peak, m_launch);
        btok += tokens;
      }
    }

    // ---- completion transition ----------------------------------------------
    const uint32_t cp0 = comp32, ev0 = evict32;
    uint32_t done = 0;
    if (in(served)) {
      // the stage-1 cohort produces its first tokens
      ub += pend;
      svc = now;
      if constexpr (TV) ncap = cap_of(now);
    }
    // the loads of the launch arrive here, before the histogram's updates
    // (memory operations complete in order)
    if constexpr (ONE) {
      qa[0] = opaque(qa[0]);
    } else {
#pragma unroll
      for (int u = 0; u < KQ; ++u) qa[u] = opaque(qa[u]);
    }
    if (fin != 0) {
      auto count = [&](int bin) __attribute__((always_inline)) {
        __hip_atomic_fetch_add(&hist[bin], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      double part = 0.0;  // the type's latencies in admission order
      // do lanes complete a second prompt?
      Mask more = 0;
      if constexpr (!ONE)
        more = ballot(before > 1u) & ballot(c[1].kc + (uint32_t)lp == now) & fin;
      if (more == 0) {
        if (in(fin)) {
          part = t_end - arrival_of(c[0].a_ft);
          count(hist_bin_idx(s_edges, s_htab, hidx, part));
          done = 1;
          fkc = c[1].kc;
        }
      } else if constexpr (!ONE) {
        if (in(fin)) {  // cohorts, KC records at a time
          for (;;) {
            double lat[KC];
            int bin[KC];
            uint32_t n = 0;  // of these, the ones that complete (they lead)
#pragma unroll
            for (int u = 0; u < KC; ++u) {
              lat[u] = t_end - arrival_of(c[u].a_ft);
              const bool ok = done + (uint32_t)u < before && c[u].kc + (uint32_t)lp == now;
              n += n == (uint32_t)u && ok ? 1u : 0u;
              fkc = n == (uint32_t)u ? c[u].kc : fkc;
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
    // This batch's admissions hold the largest keys (batch, type): they go
    // first, highest type first, as many as the memory in excess needs.  Every
    // type lane finds its share from what the higher types can free; the share
    // goes straight back to its queue, the rest joins the deque.
    const int32_t fm = (int32_t)na * chf;
    const int32_t grown = (int32_t)(before - done) - (int32_t)done * (l + lp);
    Mj += in(served) ? grown : 0;
    Mres = group_sum32<G>(Mj + fm);
    peak = max(peak, Mres);  // (a replica that has ended keeps its resident memory)
    Mask over = ballot(Mres > C) & live;
    uint32_t k = 0;  // prompts of this batch that go back
    if (over != 0) {
      const int32_t ex = Mres - C - sum_above<G>(fm, gl);
      const Mask back = ballot(ex > 0) & ballot(na > 0u) & over;
      if constexpr (ONE) {
        k = in(back) ? 1u : 0u;
      } else if (back != 0) {
        // min(na, ceil(ex / chf)): the quotient from a reciprocal is at most
        // one off, and ex is below 2^31
        uint32_t kq = (uint32_t)((double)(min(ex, fm) + chf - 1) * inv_chf);
        if ((int32_t)kq * chf < min(ex, fm)) kq++;
        if (kq > 0u && ((int32_t)kq - 1) * chf >= min(ex, fm)) kq--;
        k = in(back) ? kq : 0u;
      }
      Mres -= group_sum32<G>((int32_t)k * chf);
      over &= ballot(Mres > C);
      evict32 += k;
      if (in(back) && (qt - qh) + k > rec_cap) flags |= kFlagCap;
    }
    // (those that go back leave back first, as single evictions would)
#pragma unroll
    for (int u = 0; u < KQ; ++u) {
      const Mask some = u == 0 ? adm : ballot(nd > (uint32_t)u);
      if (some == 0) break;
      if (in(some)) {
        if ((uint32_t)u < nd - k)
          put_d((uint32_t)u, qa[u], bidx, now);
        else
          qr[(qt + (nd - 1u - (uint32_t)u)) & qmask] = qa[u];
      }
    }
    if (in(adm)) {
      if (nd > k) grow_d(nd - k, bidx, now);
      Mj += (int32_t)(nd - k) * chf;
      qt += k;
    }
    if (in(served)) pend = pnew;
    if constexpr (!ONE) {
      if (in(early)) {
        Mj += fm;
        evict_fresh(k);
      }
    }
    // then the youngest batch among the backs; with unit thresholds it has at
    // most one prompt per type, which leave together as far as needed
    if (over != 0) {
      uint32_t lost = 0;  // decode tokens
      do {
        const Mask cand = ballot(dt != dh) & over;
        const uint32_t age = in(cand) ? bidx - bkb : ~0u;
        const uint32_t best = group_reduce32<G>(age, [](uint32_t a, uint32_t b) { return min(a, b); });
        Mask me = ballot(age == best) & cand;
        over &= group_spread<G>(cand);  // a group without residents has done all it can
        const int32_t stage = (int32_t)(svc - bkc) + 1;
        if constexpr (ONE) {
          const int32_t above = sum_above<G>(in(me) ? l + stage : 0, gl);
          me &= ballot(Mres - C - above > 0);
        } else {
          me = group_highest<G>(me);
        }
        // the back record returns to the tail of its queue with its
        // first-token flag
        int32_t ch = 0;
        const Mask miss = ballot(wv < 2u) & ballot(dt != dh + 1u) & me;
        if (miss != 0) {  // rare: the new back is not in the window
          if (in(miss)) {
            s_win[(dt - 2u) % WB][tx] = dr[(dt - 2u) & dmask];
            wv = 2u;
          }
        }
        if (in(me)) {
          dt--;
          const DRec b = s_win[(dt - 1u) % WB][tx];  // (not used if the deque is empty)
          wv = wv > 0u ? wv - 1u : 0u;
          ch = l + stage;
          Mj -= ch;
          evict32++;
          lost += (uint32_t)(stage - 1);
          const bool ft = has_ft(ba);
          pend -= (stage == 1 && !ft) ? 1u : 0u;
          flags |= qt - qh >= rec_cap ? kFlagCap : 0u;
          // (a full queue ends the replica and is not read again)
          qr[qt & qmask] = ft || stage >= 2 ? with_ft(ba) : ba;
          qt++;
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
        const int32_t bt_pre = group_sum32<G>((int32_t)na);
        const int32_t bt_sel = group_sum32<G>(in(served) ? (int32_t)(before + na) : 0);
        const int32_t bt_comps = group_sum32<G>((int32_t)(comp32 - cp0));
        const int32_t bt_ev = group_sum32<G>((int32_t)(evict32 - ev0));
        const int32_t w = group_sum32<G>((int32_t)(qt - qh));
        const int32_t res = group_sum32<G>((int32_t)(dt - dh));
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
          br.waiting_after = w;
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
  const int32_t N = group_sum32<G>((int32_t)((qt - qh) + (dt - dh)));
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
    put_f(A, S_PARTA, r, 0.0);
    put_i(A, S_PARTJ, r, -1);
    put_i(A, S_PARTPP, r, 0);
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
  }
  if (is_t) {
    put_f(A, S_TNEXT + gl, r, draws ? arr.tn : t0);
    put_i(A, S_K + gl, r, draws ? arr.pending() : k0);
    put_i(A, S_QH + gl, r, qh);
    put_i(A, S_QT + gl, r, qt);
    put_i(A, S_DH + gl, r, dh);
    put_i(A, S_DT + gl, r, dt);
    put_i(A, S_SVC + gl, r, svc);
    put_i(A, S_MJ + gl, r, Mj);
    put_i(A, S_LNEXT + gl, r, pend);
  }
}

template <int G, bool TV, bool ONE, bool LIST>
hipError_t launch_wait_g(KArgs A, hipStream_t s) {
  // replicas per wavefront: what the group width allows, within the list's
  A.nr = 64 / G < A.lanes ? 64 / G : A.lanes;
  if (A.n_list % 64 != 0 || A.lanes % A.nr != 0) return hipErrorInvalidValue;
  while (A.nr > 1 && (int64_t)(A.n_list / 64) * (A.lanes / A.nr) < A.min_waves) A.nr /= 2;
  return launch_checked(sim_wait_kernel<G, TV, ONE, LIST>, dim3((A.n_list / 64) * (A.lanes / A.nr)), s, A);
}

template <bool TV, bool ONE, bool LIST>
hipError_t launch_wait_k(int max_m, const KArgs &A, hipStream_t s) {
  if (max_m <= 1) return launch_wait_g<1, TV, ONE, LIST>(A, s);
  if (max_m <= 2) return launch_wait_g<2, TV, ONE, LIST>(A, s);
  if (max_m <= 4) return launch_wait_g<4, TV, ONE, LIST>(A, s);
  if (max_m <= 8) return launch_wait_g<8, TV, ONE, LIST>(A, s);
  if (max_m <= 16) return launch_wait_g<16, TV, ONE, LIST>(A, s);
  if (max_m <= 32) return launch_wait_g<32, TV, ONE, LIST>(A, s);
  if (max_m <= 64) return launch_wait_g<64, TV, ONE, LIST>(A, s);
  return hipErrorInvalidValue;  // the host admits at most WS_MAX_TYPES types
}

}  // namespace
}  // namespace wsim
