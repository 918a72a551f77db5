// sim_nested_unit_impl.h -- simulation kernel for Nested WAIT with unit
// thresholds and constant arrival rates (arXiv 2504.11320: Algorithm 2,
// Section 5.1; event-driven form Algorithm 4, Appendix B.1).  Other launches
// (larger thresholds, per-stage caps, rate profiles, arrival lists, traces)
// run sim_nested_kernel, whose workspace layout and state this one shares.
//
// A group of G lanes runs one replica; lane g owns request type g (its
// arrival process) and segment g (its services, interior prompts, calendar
// and boundary queue).  With n_k = 1 every service of a segment admits exactly
// one prompt, so the prompt that entered at service c sits in slot c mod
// delta_k of the segment's record ring, and at most one prompt of the segment
// has entered at any service.  A prompt's exit (completion at its own output
// length, or survival to the next boundary queue at r_k) happens at a known
// service, so each segment keeps a calendar: bucket (service mod delta_k)
// heads a linked list of the slots that exit then, in reverse admission
// order.  Loops are wavefront-uniform, conditions are lane masks on the
// scalar unit.
//
// The most recently admitted eviction candidate needs no key: admission order
// is also position order (segment 1, boundary queue 2, segment 2, ...), so it
// is the back of the lowest non-empty boundary queue or, if those are empty,
// the youngest interior prompt of the lowest segment that holds a candidate.
//
// Memory latency: records are written at a prompt's entry and read at its
// exit, thousands of services later, so every read is a miss, a list's second
// record is known only from its first, and memory operations of a wavefront
// complete in order.  So:
//  - what a launch reads is loaded after the walk before it, the walk's
//    first record at the launch;
//  - once the walk's first record is there, the one after it is loaded, and
//    both land during the arrivals.  (Links to the records after that, kept in
//    each record to load them too, cost a line per entering prompt to copy
//    and did not pay: 50.5 against 48.0 ms on the heavy-tailed mix, 8,192
//    replicas x 10,000 batches.)
//  - a prompt that leaves its segment is not marked in its record: that it
//    has left follows from its entry service and its length, and a mark would
//    write the line back once more.  Evictions are marked (L = 0);
//  - the last records of a boundary queue and the last prompts that entered a
//    segment are also in LDS, for evictions;
//  - latencies are counted in LDS (a byte per bin) and added to the
//    histogram in HBM every hundred completions: an update there would be
//    waited for by every later wait.
#pragma once

#include "sim_arrivals.h"

namespace wsim {
namespace {

// A record's type word carries the prompt length with the type.
__device__ __forceinline__ int32_t unit_type_word(int32_t l, int32_t j) { return (l << 8) | j; }
__device__ __forceinline__ int32_t unit_plen(int32_t jw) { return jw >> 8; }

// What the walk needs of a record.
struct URec {
  double a_ft;
  int32_t j, L;
  uint32_t c, next;
};

template <int G>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
sim_nested_unit_kernel(KArgs A) {
  constexpr int NR = 64 / G;  // replicas per wavefront
  constexpr int RING = 512;   // arrivals drawn ahead, of a wavefront
  constexpr int WV = 2;       // boundary-queue records in LDS, per segment
  constexpr int WY = 4;       // entered prompts in LDS, per segment
  constexpr int HB = (WS_MAX_HIST_EDGES + 1) / 4;
  __shared__ typename Arrivals<G, false, RING, true>::Lds s_arr;
  __shared__ uint16_t s_cdfg[G][kCdfGuide + 1];
  __shared__ QRec s_vw[WV][64];
  __shared__ double s_ya[WY][64];
  __shared__ int2 s_yjl[WY][64];
  __shared__ uint32_t s_yc[WY][64];
  __shared__ uint32_t s_hist[NR][HB];
  __shared__ double s_edges[WS_MAX_HIST_EDGES + 1];
  __shared__ uint8_t s_htab[kHistTab];
  __shared__ int s_hsteps;

  const int tx = threadIdx.x;
  const int gl = tx & (G - 1);  // lane in the group: type gl, segment gl
  const int q = tx / G;
  const int32_t *list = (const int32_t *)(A.ws + A.off_list) + (int64_t)blockIdx.x * 64;
  const int32_t r0 = __builtin_amdgcn_readfirstlane(list[0]);
  if (r0 < 0) return;  // nothing but padding
  const int32_t r32 = q < A.lanes ? list[q] : -1;
  const bool valid = r32 >= 0;
  const int64_t r = valid ? r32 : r0;
  // every replica of a wavefront belongs to the same job
  const uint32_t jix =
      __builtin_amdgcn_readfirstlane(((const uint32_t *)(A.ws + A.off_job_of))[r0]);
  const JobDev &J = ((const JobDev *)(A.ws + A.off_jobs))[jix];
  const int m = J.m, L = J.nseg, n_hist = J.n_hist;
  const bool known = J.known != 0;
  const int32_t cap = J.out_cap;
  const uint32_t *cdf_g = (const uint32_t *)(A.ws + J.off_cdf);
  const bool use_guide = !known && cap > 1 && cap <= 65535;
  {
    const double *edges_g = (const double *)(A.ws + J.off_edges);
    for (int b = tx; b <= n_hist; b += 64) s_edges[b] = b < n_hist ? edges_g[b] : INFINITY;
    if (use_guide) {
      for (int x = tx; x < G * (kCdfGuide + 1); x += 64) {
        const int j = x / (kCdfGuide + 1), b = x % (kCdfGuide + 1);
        s_cdfg[j][b] = j < m ? (uint16_t)cdf_guide_entry(cdf_g + (size_t)j * (size_t)(cap - 1), cap, b)
                             : (uint16_t)0;
      }
    }
    for (int x = tx; x < NR * HB; x += 64) s_hist[x / HB][x % HB] = 0;
    for (int w = 0; w < WY; ++w) s_yc[w][tx] = kNil;
    __syncthreads();
  }
  const HistIdx hidx = hist_index_build(s_edges, n_hist, s_htab, &s_hsteps);
  const uint64_t seed = ((const uint64_t *)(A.ws + A.off_seed))[r];
  const uint32_t rid = ((const uint32_t *)(A.ws + A.off_rid))[r];

  const double d0 = J.d0, d1 = J.d1;
  const int32_t C = (int32_t)J.C;  // <= 2^30
  const uint32_t qmask = (1u << J.qcap_log2) - 1u;
  const uint32_t rec_cap = (uint32_t)J.rec_cap;
  uint32_t *hist = (uint32_t *)(A.ws + A.off_hist) + r * (int64_t)A.hist_stride;
  uint8_t *blk = A.ws + J.off_ring + (uint64_t)(r - J.replica_begin) * J.ring_stride;
  QRec *q10 = (QRec *)(blk + J.off_q[0]);
  // this lane's type and segment (lanes without one: the first's, unused)
  const bool is_t = gl < m, is_s = gl < L;
  const int jt = is_t ? gl : 0, k = is_s ? gl : 0;
  const int32_t tword = unit_type_word(J.l[jt], jt), lpk = J.lp[jt];
  const double lam = J.lambda[jt];
  const int32_t rk = J.seg_end[k], ent = J.seg_entry[k];
  const uint32_t delta = (uint32_t)J.seg_delta[k];
  const int32_t rprev = gl > 0 ? ent - 1 : 0;  // r_{k-1}
  NRec *rc = (NRec *)(blk + J.off_rec[k]);
  uint32_t *bk = (uint32_t *)(blk + J.off_bkt[k]);
  NRec *vr = (NRec *)(blk + J.off_v[k >= 1 ? k : 0]);  // (k >= 1)
  const uint32_t vmask = k >= 1 ? (1u << J.vcap_log2[k]) - 1u : 0u;
  const int kn = k + 1 < L ? k + 1 : k;  // survivors join segment kn's queue
  NRec *vrn = (NRec *)(blk + J.off_v[kn >= 1 ? kn : 0]);
  const uint32_t vmaskn = kn >= 1 ? (1u << J.vcap_log2[kn]) - 1u : 0u;
  const bool last = k == L - 1;

  const Mask seg_m = ballot(is_s);
  const Mask bq_m = seg_m & ~group_leaders<G>();  // segments with a boundary queue
  const Mask next_m = ballot(is_s && !last);           // with a segment after them
  const Mask valid_m = ballot(valid);

  // replica-wide scalars, identical in every lane of the group
  double t, lat_area, ttft_area, lat_sum, mem_area, busy;
  int64_t batches, btok, idle, tridx;
  int32_t peak, Mres;
  uint32_t qh, qt;   // ends of Q_{1,0}
  int32_t pendft;    // stage-1 prompts without a first token
  uint32_t flags = 0;
  // this lane's share of the replica's counters
  int64_t arrivals = 0, comps = 0, ctok = 0, evicts = 0, etok = 0, fallback = 0;
  uint32_t comp32 = 0, evict32 = 0, fall32 = 0;
  uint32_t ub = 0, arr_rp = 0;  // (see the WAIT kernel: rp - ub lack a first token)
  double t0 = INFINITY;
  uint32_t k0 = 0;
  int32_t len0 = 1;
  // this lane's segment: services, slot of the last one, interior prompts
  // and their memory, boundary queue's memory and ends; no live interior
  // prompt entered after service ytop
  uint32_t svc = 0, xs = 0, I = 0, vh = 0, vt = 0, ytop = 0;
  int32_t M = 0, Bk = 0;

  if (!A.resume) {
    t = lat_area = ttft_area = lat_sum = mem_area = busy = 0.0;
    batches = btok = idle = tridx = 0;
    peak = Mres = pendft = 0;
    qh = qt = 0;
    if (valid) {
      // calendar buckets start empty: each segment's by the whole group (its size
      // is read before: after a store it would be loaded again)
      for (int kk = 0; kk < L; ++kk) {
        uint32_t *b = (uint32_t *)(blk + J.off_bkt[kk]);
        const int n = J.seg_delta[kk];
        for (int x = gl; x < n; x += G) b[x] = kNil;
      }
      for (int b = gl; b < A.hist_stride; b += G) hist[b] = 0;  // whole row, padding included
    }
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
    pendft = (int32_t)slot_i(A, S_PENDFT, r);
    flags = (uint32_t)slot_i(A, S_FLAGS, r);
    qh = (uint32_t)slot_i(A, S_QH, r);
    qt = (uint32_t)slot_i(A, S_QT, r);
    if (gl == 0) {
      ub = 0u - (uint32_t)slot_i(A, S_U, r);
      arrivals = slot_i(A, S_ARR, r);
      comps = slot_i(A, S_COMP, r);
      ctok = slot_i(A, S_CTOK, r);
      evicts = slot_i(A, S_EVICT, r);
      etok = slot_i(A, S_ETOK, r);
      fallback = slot_i(A, S_FALLBACK, r);
    }
    if (is_t) {
      t0 = slot_f(A, S_TNEXT + jt, r);
      k0 = (uint32_t)slot_i(A, S_K + jt, r);
      len0 = (int32_t)slot_i(A, S_LNEXT + jt, r);
    }
    if (is_s) {
      svc = ytop = (uint32_t)slot_i(A, S_KSVC + k, r);
      I = (uint32_t)slot_i(A, S_KI + k, r);
      M = (int32_t)slot_i(A, S_KM + k, r);
      Bk = (int32_t)slot_i(A, S_KB + k, r);
      vh = (uint32_t)slot_i(A, S_KVH + k, r);
      vt = (uint32_t)slot_i(A, S_KVT + k, r);
      xs = fastmod(svc, fastmod_magic(delta), delta);
    }
  }
  const int64_t batches0 = batches;
  int64_t stop = -1;  // batches of a replica that ended early
  Mask live = valid_m & ~group_spread<G>(ballot((flags & (kFlagCap | kFlagStall)) != 0));
  if (!in(live)) stop = 0;
  uint32_t wv = 0;    // boundary-queue records vt-wv .. vt-1 are in LDS
  uint32_t hcnt = 0;  // the replica's latencies counted in LDS

  const bool draws = valid && is_t;
  Arrivals<G, false, RING, true> arr(s_arr, 64, draws, seed, rid, lam, 0, A.resume != 0, t0, k0);
  arr.law.cdf = cdf_g;
  arr.law.cap = known ? 0 : cap;
  arr.law.guide = use_guide ? s_cdfg : nullptr;
  if (A.resume && draws) s_arr.len[arr.slot(0u, tx)] = (uint16_t)len0;
  arr.start(live);

  // ---- histogram ------------------------------------------------------------
  auto flush_hist = [&](Mask who) __attribute__((always_inline)) {
    wave_lds_sync();
    if (in(who)) {
      for (int b = gl; b < HB; b += G) {
        const uint32_t w = s_hist[q][b];
        if (w != 0u) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t n = (w >> (8 * i)) & 0xFFu;
            if (n != 0u)
              __hip_atomic_fetch_add(&hist[4 * b + i], n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          s_hist[q][b] = 0;
        }
      }
      hcnt = 0;
    }
    wave_lds_sync();
  };

  // ---- the entry queue --------------------------------------------------------
  // Append a record of lane `me` to Q_{1,0} of each group in `go` (a full
  // queue ends the replica at its next decision and is not read again).
  auto push_q = [&](Mask go, Mask me, double a_ft, int32_t j, int32_t len) __attribute__((always_inline)) {
    if (in(me)) {
      QRec rec;
      rec.a_ft = a_ft;
      rec.j = j;
      rec.L = len;
      q10[qt & qmask] = rec;
    }
    if (in(go)) {
      flags |= qt - qh >= rec_cap ? kFlagCap : 0u;
      qt++;
    }
  };
  // One arrival of each group in `go` (of simultaneous ones the lowest type's)
  // joins Q_{1,0} at time ta.
  auto take = [&](Mask go, double ta, Mask &more) __attribute__((always_inline)) {
    Mask me = go & ballot(arr.tn == ta);
    if (__popcll(me) * G != __popcll(go)) me = group_lowest<G>(me);
    const Mask low = arr.low();
    more &= ~(go & ballot(qt - qh >= rec_cap));
    if ((me & low) != 0) arr.refill(live, me);
    const int32_t len = known ? lpk : (int32_t)s_arr.len[arr.slot(arr.rp, tx)];
    push_q(go, me, ta, tword, len);
    if (in(me)) arr.advance();
  };

  // ---- evictions ---------------------------------------------------------------
  auto slot_of = [&](uint32_t c) __attribute__((always_inline)) -> uint32_t {
    const uint32_t d = svc - c;  // < delta
    return xs >= d ? xs - d : xs + delta - d;
  };
  // The WY prompts that entered the segment up to service c, into LDS.
  auto load_y = [&](uint32_t c) __attribute__((always_inline)) {
    double a[WY];
    uint2 jl[WY];
#pragma unroll
    for (int i = 0; i < WY; ++i) {
      // (services before the first, or a whole ring ago: any record, unused)
      const uint32_t ci = c - (uint32_t)i;
      const NRec *b = rc + (ci >= 1u && ci <= c && svc - ci < delta ? slot_of(ci) : 0u);
      a[i] = b->a_ft;
      jl[i] = *(const uint2 *)((const uint8_t *)b + 16);
    }
#pragma unroll
    for (int i = 0; i < WY; ++i) {
      const uint32_t ci = c - (uint32_t)i;
      if (ci >= 1u && ci <= c && svc - ci < delta) {
        s_ya[ci % WY][tx] = a[i];
        s_yjl[ci % WY][tx] = make_int2((int32_t)jl[i].x, (int32_t)jl[i].y);
        s_yc[ci % WY][tx] = ci;
      }
    }
  };
  uint32_t pf_ti = kNil;             // slot whose record the next launch counts as terminal
  uint2 pf_tr = make_uint2(0u, 0u);  // and its (type word, length)
  // Evict the most recently admitted prompt of every group in `over`: among
  // the boundary queues, else among the interiors of the lanes in `inner`.
  // Returns the memory freed (0 in the groups that had none left, which leave
  // `over`).
  auto evict = [&](Mask &over, Mask inner) __attribute__((always_inline)) -> int32_t {
    const Mask mb = group_lowest<G>(ballot(vt != vh) & bq_m & over);
    const Mask mi =
        group_lowest<G>(ballot(I != 0u) & inner & (over & ~group_spread<G>(mb)));
    const Mask me = mb | mi;
    over &= group_spread<G>(me);
    double a = 0.0;
    int32_t j = 0, len = 0;
    uint32_t c = ytop, ci = 0;
    if (mb != 0) {
      const Mask miss = mb & ballot(wv == 0u);
      if (in(mb & ~miss)) {
        const QRec b = s_vw[(vt - 1u) % WV][tx];
        a = b.a_ft;
        j = b.j;
        len = b.L;
      }
      if (miss != 0) {  // not in LDS
        if (in(miss)) {
          const NRec *b = vr + ((vt - 1u) & vmask);
          a = b->a_ft;
          j = b->j;
          len = b->L;
        }
        a = opaque(a);
      }
    }
    if (mi != 0) {  // the youngest live one, from the last known bound down
      Mask look = mi;
      do {
        const Mask near = ballot(s_yc[c % WY][tx] == c) & look;
        if (in(near)) {
          const int2 x = s_yjl[c % WY][tx];
          a = s_ya[c % WY][tx];
          j = x.x;
          len = x.y;
        }
        const Mask far = look & ~near;
        if (far != 0) {  // not in LDS: it and the ones before it
          if (in(far)) {
            load_y(c);
            len = 0;  // looked up again
            c++;
          }
        }
        // a prompt is live if it was not evicted and its exit is to come
        const bool dead = len == 0 || c + (uint32_t)(min(len, rk) - ent) <= svc;
        look &= ballot(dead);
        // (a segment with I > 0 holds a live record among its last delta
        // services; the bound ends the search all the same)
        look &= (ballot(svc - c + 1u < delta) & ballot(c > 1u)) | far;
        if (in(look)) c--;
      } while (look != 0);
      ci = slot_of(c);
    }
    const int32_t stage = ent + (int32_t)(svc - c) + 1;
    const bool b_ = in(mb);
    const bool ft = b_ || has_ft(a) || stage >= 2;  // boundary prompts have their first token
    const int32_t gen = in(me) ? (b_ ? rprev : stage - 1) : 0;
    const int32_t ch = in(me) ? unit_plen(j) + (b_ ? rprev : stage) : 0;
    if (in(mb)) {
      vt--;
      wv = wv > 0u ? wv - 1u : 0u;
      Bk -= ch;
    }
    if (in(mi)) {
      rc[ci].L = 0;  // leaves a hole; the calendar skips it
      if (s_yc[c % WY][tx] == c) s_yjl[c % WY][tx].y = 0;
      if (ci == pf_ti) pf_tr.y = 0u;
      ytop = c - 1u;
      I -= 1u;
      M -= ch;
      fall32++;
    }
    if (in(me)) {
      evict32++;
      etok += gen;
    }
    push_q(over, me, ft ? with_ft(a) : arrival_of(a), j, len);
    const Mask dp = mi & ballot(!ft);
    pendft -= in(group_spread<G>(dp)) ? 1 : 0;
    const int32_t freed = group_sum32<G>(ch);
    Mres -= freed;
    return freed;
  };

  // ---- what the next launch reads first -----------------------------------------
  uint4 pf_q = make_uint4(0u, 0u, 0u, 0u);  // head of Q_{1,0} (lane 0)
  Mask pf_qok = 0;                          // groups whose queue held it
  uint32_t bh = kNil;                       // head of the bucket served next
  double pf_va = 0.0;                       // front of the boundary queue
  uint2 pf_vjl = make_uint2(0u, 0u);
  auto prefetch = [&]() __attribute__((always_inline)) {
    pf_qok = ballot(qt != qh) & live;
    if (in(pf_qok & group_leaders<G>())) pf_q = ((const uint4 *)q10)[qh & qmask];
    const uint32_t nx = xs + 1u == delta ? 0u : xs + 1u;
    const Mask next = live & (group_leaders<G>() | (bq_m & ballot(vt != vh)));
    pf_ti = kNil;
    if (in(next)) {
      bh = bk[nx];
      if (delta >= 2u && svc + 1u >= delta) {
        pf_ti = nx + 1u == delta ? 0u : nx + 1u;  // the oldest slot
        pf_tr = *(const uint2 *)((const uint8_t *)(rc + pf_ti) + 16);
      }
    }
    if (in(next & bq_m)) {
      const NRec *f = vr + (vh & vmask);
      pf_va = f->a_ft;
      pf_vjl = *(const uint2 *)((const uint8_t *)f + 16);
    }
  };
  prefetch();

  int64_t it = 0;
  for (; it < A.horizon; ++it) {
    if ((it & 255) == 255) {  // 32-bit counts to 64 bits
      arrivals += arr.rp - arr_rp;
      arr_rp = arr.rp;
      comps += comp32;
      comp32 = 0;
      evicts += evict32;
      evict32 = 0;
      fallback += fall32;
      fall32 = 0;
    }
    // ---- decision: largest prefix of segments meeting their thresholds -----
    Mask served;
    int32_t N0, U0;
    for (;;) {
      const Mask capf = ballot((flags & kFlagCap) != 0) & live;
      if (capf != 0) {
        const Mask dead = group_spread<G>(capf);
        if (in(dead)) stop = it;
        live &= ~dead;
      }
      const Mask ok = (ballot(qt != qh) & group_leaders<G>()) | (ballot(vt != vh) & bq_m);
      served = live & ~group_fill_up<G>(~ok);
      N0 = group_sum32<G>((int32_t)(I + (vt - vh))) + (int32_t)(qt - qh);
      U0 = group_sum32<G>((int32_t)(arr.rp - ub));
      Mask wait = live & ~group_spread<G>(served);
      if (wait == 0) break;
      const double ta = group_min<G>(arr.tn);
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
      // every arrival at this instant joins before the next decision
      while (wait != 0) {
        take(wait, ta, wait);
        wait &= ballot(group_min<G>(arr.tn) == ta);
      }
    }
    if (live == 0) break;

    // ---- launch: entering prompts, calendar links, batch tokens -----------
    const uint32_t x = svc + 1u;
    const uint32_t slot = xs + 1u == delta ? 0u : xs + 1u;
    const Mask first = served & group_leaders<G>();
    {
      const Mask late = first & ~pf_qok;  // the head arrived after the prefetch
      if (late != 0) {
        if (in(late)) pf_q = ((const uint4 *)q10)[qh & qmask];
      }
    }
    // the entering prompt
    double ea = pf_va;
    int32_t ej = (int32_t)pf_vjl.x, eL = (int32_t)pf_vjl.y;
    if (in(first)) {
      ea = __longlong_as_double((long long)(((uint64_t)pf_q.y << 32) | pf_q.x));
      ej = (int32_t)pf_q.z;
      eL = (int32_t)pf_q.w;
    }
    const int32_t el = unit_plen(ej);
    const int32_t pexit = min(eL, rk);
    // entry stage <= pexit <= r_k: the exit is 0..delta-1 services ahead
    uint32_t b = slot + (uint32_t)(pexit - ent);
    b = b >= delta ? b - delta : b;
    const Mask now_m = served & ballot(pexit == ent);  // exits at this very service
    const Mask link_m = served & ~now_m;
    uint32_t oldh = kNil;  // head of the bucket the prompt joins
    URec c0;
    const Mask walk0 = served & ballot(bh != kNil);
    if (in(walk0)) {  // the walk's first record
      const NRec *p = rc + bh;
      c0.a_ft = p->a_ft;
      c0.j = p->j;
      c0.L = p->L;
      c0.c = p->c;
      c0.next = p->next;
    }
    if (in(link_m)) {
      oldh = bk[b];
      bk[b] = slot;
    }
    int32_t tok = 0, dplus = 0, eB = 0, eM = 0;
    if (in(served)) {
      // (ring of entered prompts)
      s_ya[x % WY][tx] = ea;
      s_yjl[x % WY][tx] = make_int2(ej, eL);
      s_yc[x % WY][tx] = x;
      tok = M + el + (gl > 0 ? ent : 0);  // processed at stage r_{k-1} + 1
      const bool stays = pexit > ent;
      eM = stays ? el + ent + 1 : 0;
      eB = gl > 0 ? el + rprev : 0;
      // projected change of the segment's memory (no early completion)
      if (delta >= 2u) {
        // the terminal slot is live: its prompt stays to the segment's end
        const bool term = pf_ti != kNil && (int32_t)pf_tr.y >= rk;
        dplus = (int32_t)I - (term ? 1 : 0);
        if (last && term) dplus -= unit_plen((int32_t)pf_tr.x) + rk;
        dplus += gl == 0 ? el + 1 : 2;  // l at stage 1; l + r_{k-1} -> l + r_{k-1} + 2
      } else {
        dplus = last ? -(el + rprev) : 1;  // processed at r_k
      }
      vh += gl > 0 ? 1u : 0u;  // still charged in Bk until the completion
    }
    const int32_t prefill_l = group_sum32<G>(in(first) ? el : 0);
    const int32_t tokens = group_sum32<G>(tok);
    const int32_t pend_new = group_sum32<G>(in(first) && !has_ft(ea) ? 1 : 0);
    int32_t mplus = Mres + group_sum32<G>(dplus);
    qh += in(group_spread<G>(first)) ? 1u : 0u;

    // ---- pre-launch repair on the projected state ----------------------------
    {
      Mask over = ballot(mplus > C) & live;
      if (over != 0) {
        const Mask all = over;
        do {
          mplus -= evict(over, seg_m & ~served);
          over &= ballot(mplus > C);
        } while (over != 0);
        if (in(all) && mplus > C) flags |= kFlagOverflow;
        // a replica whose queue an evicted prompt overflowed takes no arrival any
        // more (it ends at its next decision)
        if ((flags & kFlagCap) != 0) arr.tn = INFINITY;
      }
    }
    // The walk's first record is there: the one after it is loaded now.
    uint32_t n1 = kNil;
    URec c1;
    {
      oldh = opaque(oldh);
      if (in(walk0)) n1 = c0.next;
      if (in(walk0 & ballot(n1 < delta))) {
        const NRec *p = rc + n1;
        c1.a_ft = p->a_ft;
        c1.j = p->j;
        c1.L = p->L;
        c1.c = p->c;
        c1.next = p->next;
      }
    }

    const int32_t m_launch = Mres + prefill_l;
    const double tau = d0 + d1 * (double)tokens;
    const double t_end = t + tau;

    // ---- arrivals during the batch -----------------------------------------
    Mask inb = live;
    for (;;) {
      const double ta = group_min<G>(arr.tn);
      const Mask go = ballot(ta <= t_end) & inb;
      if (go == 0) break;
      const double w = in(go) ? t_end - ta : 0.0;  // (areas are never -0)
      lat_area += w;
      ttft_area += w;
      take(go, ta, inb);
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

    // ---- completion transition, every served segment at once ----------------
    // the stage-1 cohort produces its first tokens
    if (in(live)) {
      ub += gl == 0 ? (uint32_t)pendft : 0u;
      pendft = pend_new;
    }
    int32_t Mk = M, dM = 0;
    uint32_t node = kNil;
    if (in(served)) {
      rc[slot].a_ft = ea;
      *(uint4 *)((uint8_t *)(rc + slot) + 16) = make_uint4((uint32_t)ej, (uint32_t)eL, x, oldh);
      bk[slot] = kNil;
      svc = x;
      xs = slot;
      ytop = x;
      Mk = M + (int32_t)I + eM;  // every interior prompt advances
      I += in(link_m) ? 1u : 0u;
      Bk -= eB;
      dM -= eB;
      node = in(now_m) ? slot : bh;
    }
    wave_lds_sync();
    // Walk the buckets served now.  Survivors join the back of segment k+1's
    // boundary queue (its ends from lane k+1; what was pushed goes there after
    // the walk).
    const uint32_t vtn = seg_next<G>(vt), vhn = seg_next<G>(vh);
    uint32_t npush = 0, ndone = 0;
    int32_t bpush = 0;
    double part = 0.0;  // the segment's latencies in traversal order
    Mask walk = ballot(node != kNil) & served;
    uint32_t trips = 0;
    while (walk != 0) {
      // a byte counts 127 and 16 lanes' completions of 8 trips
      if ((++trips & 7u) == 0) {
        hcnt = 128u;
        flush_hist(live);
      }
      // a bucket lists at most delta records: a longer walk could only follow
      // a corrupted link, so it stops the replica
      const Mask bad = walk & ballot(trips > delta + 1u);
      if (bad != 0) {
        if (in(bad)) flags |= kFlagCap;
        walk &= ~bad;
        if (walk == 0) break;
      }
      // the record: the entering one, one of those at hand, or from memory
      URec rec;
      rec.a_ft = ea;
      rec.j = ej;
      rec.L = eL;
      rec.c = x;
      rec.next = bh;
      Mask far = walk & ~(trips == 1u ? now_m : 0);
      if (far != 0) {
        auto pick = [&](uint32_t idx, const URec &o) __attribute__((always_inline)) {
          const Mask hit = far & ballot(node == idx);
          far &= ~hit;
          if (in(hit)) rec = o;
        };
        pick(bh, c0);
        pick(n1, c1);
        if (far != 0) {
          if (in(far)) {
            const NRec *p = rc + node;
            rec.a_ft = p->a_ft;
            rec.j = p->j;
            rec.L = p->L;
            rec.c = p->c;
            rec.next = p->next;
          }
          rec.next = opaque(rec.next);
        }
      }
      const Mask there = walk & ballot(rec.L != 0);  // holes left by evictions are skipped
      const int32_t le = unit_plen(rec.j);
      const int32_t p = min(rec.L, rk);
      const Mask fin = there & ballot(rec.L == p);
      const Mask surv = there & ~fin;
      if (in(there & ballot(rec.c != x))) {  // an interior prompt: it had advanced to p + 1
        Mk -= le + p + 1;
        I -= 1u;
      }
      if (fin != 0) {
        if (in(fin)) {  // completion at its own output length
          const double lat = t_end - arrival_of(rec.a_ft);
          part += lat;
          const int bin = hist_bin_idx(s_edges, s_htab, hidx, lat);
          __hip_atomic_fetch_add(&s_hist[q][bin >> 2], 1u << (8 * (bin & 3)), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WAVEFRONT);
          ndone++;
          ctok += rec.L;
        }
      }
      if (surv != 0) {
        const uint32_t vp = vtn + npush;
        const Mask room = surv & ballot(vp - vhn <= vmaskn) & next_m;
        if (in(surv & ~room)) flags |= kFlagCap;  // bounded by construction; guards the ring
        if (in(room)) {
          QRec w;
          w.a_ft = with_ft(rec.a_ft);
          w.j = rec.j;
          w.L = rec.L;
          NRec *v = vrn + (vp & vmaskn);
          v->a_ft = w.a_ft;
          *(uint2 *)((uint8_t *)v + 16) = make_uint2((uint32_t)w.j, (uint32_t)w.L);
          s_vw[vp % WV][tx + 1] = w;  // a survivor's segment has a next lane
          npush++;
        }
        if (in(surv)) {
          bpush += le + rk;
          dM += le + rk;
        }
      }
      node = rec.next;
      walk &= ballot(node != kNil);
    }
    wave_lds_sync();  // s_vw: a survivor's record, read by the next segment's lane
    comp32 += ndone;
    lat_sum = add_in_order<G>(lat_sum, part, ballot(ndone != 0u));
    {
      const uint32_t np = seg_prev<G>(npush);
      const int32_t bp = (int32_t)seg_prev<G>((uint32_t)bpush);
      if (in(bq_m & live)) {
        Bk += bp;
        vt += np;
        wv = min(wv + np, (uint32_t)WV);
      }
    }
    hcnt += (uint32_t)group_sum32<G>((int32_t)ndone);
    Mres += group_sum32<G>(Mk - M + dM);
    M = Mk;
    peak = max(peak, Mres);
    {
      const Mask full = ballot(hcnt > 127u) & live;
      if (full != 0) flush_hist(full);
    }
    prefetch();

    // ---- repair: boundary prompts first, then interior prompts -------------
    Mask over = ballot(Mres > C) & live;
    while (over != 0) {
      (void)evict(over, seg_m);
      over &= ballot(Mres > C);
    }
    wave_lds_sync();
  }
  flush_hist(valid_m);

  // ---- save state ------------------------------------------------------------
  batches = batches0 + (stop >= 0 ? stop : it);
  arrivals = group_sum<G>(arrivals + (int64_t)(arr.rp - arr_rp));
  comps = group_sum<G>(comps + comp32);
  ctok = group_sum<G>(ctok);
  evicts = group_sum<G>(evicts + evict32);
  etok = group_sum<G>(etok);
  fallback = group_sum<G>(fallback + fall32);
  const int32_t U = group_sum32<G>((int32_t)(arr.rp - ub));
  const int32_t N = group_sum32<G>((int32_t)(I + (vt - vh))) + (int32_t)(qt - qh);
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
    put_i(A, S_ETOK, r, etok);
    put_i(A, S_FALLBACK, r, fallback);
    put_i(A, S_BTOK, r, btok);
    put_i(A, S_PEAK, r, peak);
    put_i(A, S_IDLE, r, idle);
    put_i(A, S_N, r, N);
    put_i(A, S_U, r, U);
    put_i(A, S_MRES, r, Mres);
    put_i(A, S_TRIDX, r, tridx);
    put_i(A, S_PENDFT, r, pendft);
    put_i(A, S_FLAGS, r, (int64_t)flags);
    put_i(A, S_QH, r, qh);
    put_i(A, S_QT, r, qt);
  }
  put_f(A, S_TNEXT + gl, r, is_t ? arr.tn : INFINITY);
  put_i(A, S_K + gl, r, is_t ? arr.pending() : 0u);
  put_i(A, S_LNEXT + gl, r, !is_t ? 1 : known ? lpk : (int32_t)s_arr.len[arr.slot(arr.rp, tx)]);
  if (gl < kMaxSeg) {  // groups wider than the segment limit: lanes without one
    put_i(A, S_KSVC + gl, r, svc);
    put_i(A, S_KI + gl, r, I);
    put_i(A, S_KM + gl, r, M);
    put_i(A, S_KB + gl, r, is_s ? Bk : 0);
    put_i(A, S_KVH + gl, r, is_s ? vh : 0u);
    put_i(A, S_KVT + gl, r, is_s ? vt : 0u);
  }
}

template <int G>
hipError_t launch_unit_g(const KArgs &A, hipStream_t s) {
  return launch_checked(sim_nested_unit_kernel<G>, dim3(A.n_list / 64), s, A);
}

}  // namespace
}  // namespace wsim
