// sim_arrivals.h -- the arrival processes of a replica on a group of G lanes,
// one request type per lane: Poisson at a constant rate, or thinned with a rate
// profile.  An arrival process does not depend on what the simulation does, so
// the whole wavefront draws arrival times ahead of use into a ring per lane.
#pragma once

#include "sim_lanes.h"

namespace wsim {
namespace {

// Output lengths drawn with the arrivals: CDF rows, their cap, search guide.
struct LenLaw {
  const uint32_t *cdf;
  int32_t cap;  // <= 1: no draw, every length is 1; at most 65535
  const uint16_t (*guide)[kCdfGuide + 1];
};

// TV: rate profiles are supported.  RING: ring entries of a wavefront.  LEN:
// output lengths are drawn too (law; constant rates only).
template <int G, bool TV, int RING, bool LEN = false>
struct Arrivals {
  static_assert(!TV || !LEN, "lengths are drawn at constant rates");
  static constexpr int NP = TV ? kMaxRatePts : 1;
  struct Lds {
    double at[RING];
    uint32_t ak[TV ? RING : 1];  // acceptance words, then candidate indices
    uint16_t len[LEN ? RING : 1];
    RateProfLds<TV ? G : 1, NP> prof;
    uint8_t req[64];
  };
  Lds &S;
  int tx, gl, act_log2, gu_log2, P;
  uint32_t dm, gu;  // ring depth - 1; draws added per request
  uint64_t seed;
  uint32_t rid;
  double lam;
  bool tv;
  Mask draw_m;  // lanes that draw
  // The pending arrival (tn) and the next (tn2, if it is known) lead the ring
  // of entries rp .. re-1, whose last is at te; kc is the next candidate to draw, tl the clock
  // it starts from.
  double tn = INFINITY, tn2 = INFINITY, te = INFINITY, tl = 0.0;
  uint32_t rp = 0, re = 0, kc = 0;
  bool ended = false;     // (TV) no further arrivals
  bool thin_end = false;  // (TV) by the limit on rejections in a row
  int cur = -1;           // profile piece of the type's clock
  uint32_t tries = 0;     // rejections in a row
  LenLaw law = {nullptr, 0, nullptr};

  // act: the lanes in use, which share the ring's entries.  A resumed lane's
  // pending arrival is candidate k0 at time t0.
  __device__ __forceinline__ Arrivals(Lds &lds, int act, bool draws, uint64_t seed_, uint32_t rid_,
                                      double lam_, int P_, bool resume, double t0, uint32_t k0)
      : S(lds), tx(threadIdx.x), gl(threadIdx.x & (G - 1)), act_log2(__builtin_ctz(act)), P(P_),
        seed(seed_), rid(rid_), lam(lam_), tv(TV && P_ > 0), draw_m(ballot(draws)) {
    const uint32_t depth = min((uint32_t)(RING / 64) * (64u / (uint32_t)act), 64u);
    dm = depth - 1u;
    gu = depth / 2u;
    gu_log2 = __builtin_ctz(gu);
    if (resume && draws) {  // the pending arrival leads the ring
      tn = te = tl = t0;
      kc = k0 + 1u;
      ended = !(t0 < INFINITY);
      S.at[slot(0u, tx)] = t0;
      if constexpr (TV) S.ak[slot(0u, tx)] = k0;
      re = 1u;
    }
  }
  __device__ __forceinline__ uint32_t slot(uint32_t pos, int ln) const {
    return ((pos & dm) << act_log2) + (uint32_t)ln;
  }

  // Every lane of `live` with room for gu draws asks for them and the
  // wavefront draws all of them together; then each asking lane turns its
  // gaps into arrival times (with a rate profile, its candidates into the
  // kept ones).  Thinning may keep none of them, up to kThinMax in a row, so
  // only the lanes of `need`, whose arrivals are about to be taken, go on until
  // they hold `least`; the others' later arrivals may never be reached.  Every
  // lane of the wavefront takes part.
  __device__ __forceinline__ void refill(Mask live, Mask need, uint32_t least = 2u) {
    Mask again;
    do {
      Mask room = ballot(re - rp <= dm + 1u - gu) & live & draw_m;
      if constexpr (TV) room &= ~ballot(ended);
      if (in(room))
        S.req[__builtin_amdgcn_mbcnt_hi((uint32_t)(room >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)room, 0u))] = (uint8_t)tx;
      wave_lds_sync();
      const int total = __popcll(room) << gu_log2;
      for (int base = 0; base < total; base += 64) {
        const int w = base + tx;
        const int ln = (int)S.req[(w < total ? w : 0) >> gu_log2];
        const uint32_t u = (uint32_t)w & (gu - 1u);
        // the asking lane's key, rate and counters
        const uint64_t sd = __shfl(seed, ln, 64);
        const uint32_t rd = __shfl(rid, ln, 64);
        const double lm = __shfl(lam, ln, 64);
        const uint32_t kl = __shfl(kc, ln, 64), el = __shfl(re, ln, 64);
        uint32_t w3;
        int32_t len = 1;
        const int j = ln & (G - 1);
        const uint32_t *row = nullptr;
        const uint16_t *guide = nullptr;
        if constexpr (LEN) {
          if (law.cap > 1) row = law.cdf + (size_t)j * (size_t)(law.cap - 1);
          if (law.guide != nullptr) guide = law.guide[j];
        }
        const double g = draw_gap(sd, rd, (uint32_t)j, kl + u, lm, LEN ? row : nullptr,
                                  LEN ? law.cap : 0, LEN ? &len : nullptr, TV ? &w3 : nullptr,
                                  LEN ? guide : nullptr);
        if (w < total) {
          S.at[slot(el + u, ln)] = g;
          if constexpr (LEN) S.len[slot(el + u, ln)] = (uint16_t)len;
          if constexpr (TV) S.ak[slot(el + u, ln)] = w3;
        }
      }
      wave_lds_sync();
      if (in(room)) {
        if (!TV || !tv) {
          for (uint32_t u = 0; u < gu; u += 4) {  // depth >= 8: gu is a multiple of 4
            double g[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) g[x] = S.at[slot(re + u + (uint32_t)x, tx)];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              tl = tl + g[x];
              S.at[slot(re + u + (uint32_t)x, tx)] = tl;
              if constexpr (TV) S.ak[slot(re + u + (uint32_t)x, tx)] = kc + u + (uint32_t)x;
            }
          }
          re += gu;
          te = tl;
        } else if constexpr (TV) {  // thinning; kept ones move up
          uint32_t end = re;
          for (uint32_t u = 0; u < gu && !ended; ++u) {
            const double g = S.at[slot(re + u, tx)];
            const uint32_t w3 = S.ak[slot(re + u, tx)];
            const double fmax = S.prof.fmax[gl];
            int d = 1;  // no intensity at all: no arrival
            if (fmax > 0.0) d = thin_decide(tl + g, w3, fmax, S.prof.t, S.prof.f[gl], P, tl, cur);
            const bool limit = d != 0 && fmax > 0.0 && tries + 1u >= kThinMax;
            ended = d == 1 || limit;
            thin_end = thin_end || limit;
            if (d == 0 || ended) {
              te = ended ? INFINITY : tl;
              S.at[slot(end, tx)] = te;
              S.ak[slot(end, tx)] = kc + u;
              end++;
              tries = 0;
            } else {
              ++tries;
            }
          }
          re = end;
        }
        kc += gu;
        tn2 = S.at[slot(rp + 1u, tx)];
      }
      wave_lds_sync();
      again = 0;
      if constexpr (TV) again = ballot(re - rp < least) & ballot(!ended) & live & draw_m & need;
    } while (again != 0);
  }
  // The pending arrivals of the lanes of `live`, after the first refill.  With a
  // rate profile a lane thins its draws one after another, and a call may end
  // after a few batches, so that refill draws `first` at most (and never more than
  // half of a ring): 20 calls of one batch, WAIT, 4 replicas of one type, took 0.75
  // ms with 32 and take 0.59 with 16 (0.58 with 4); 512 replicas 0.84 and 0.68
  // (0.91 with 4, which the batch uses up).
  __device__ __forceinline__ void start(Mask live, uint32_t first = 16u) {
    wave_lds_sync();
    if constexpr (TV) {
      const uint32_t half = gu;
      if (tv) gu = min(half, first);
      gu_log2 = __builtin_ctz(gu);
      refill(live, live, 1u);
      gu = half;
      gu_log2 = __builtin_ctz(half);
    } else {
      refill(live, live, 1u);
    }
    if (in(live & draw_m)) tn = S.at[slot(rp, tx)];
  }
  // Lanes whose ring ends with the next arrival: to refill before they move
  // on (tn2 is then the pending one; what follows it in the ring, if it is
  // not known yet, is set by the refill before it is used).
  __device__ __forceinline__ Mask low() const {
    Mask m = ballot(rp + 2u >= re) & draw_m;
    if constexpr (TV) m &= ~ballot(ended);
    return m;
  }
  // This lane's pending arrival has been taken.
  __device__ __forceinline__ void advance() {
    rp++;
    tn = tn2;
    // (the move first: the read then lands in tn2 itself and is waited for
    // only when tn2 is used)
    __builtin_amdgcn_sched_barrier(0);
    tn2 = S.at[slot(rp + 1u, tx)];
  }
  // Did the process end by the limit on rejections (the flag goes up when its
  // end is reached)?
  __device__ __forceinline__ bool limited() const { return TV && thin_end && !(tn < INFINITY); }
  // Back to entry rp0 of the ring (still there: no refill since).
  __device__ __forceinline__ void rewind(uint32_t rp0) {
    rp = rp0;
    tn = S.at[slot(rp, tx)];
    tn2 = S.at[slot(rp + 1u, tx)];
  }
  // Candidate counter of the pending arrival.
  __device__ __forceinline__ uint32_t pending() const {
    if constexpr (TV) return S.ak[slot(rp, tx)];
    return kc - (re - rp);
  }
};

// A fixed arrival list, read ahead into LDS by the lanes of each group.  A load
// per arrival would be waited for together with every store before it: WAIT, one
// type, 512 replicas x 400 batches of 2.5 arrivals took 1.48 ms with one and takes
// 1.09; FCFS, three types, 32,768 replicas 2.83 and 1.41 (there also because two
// wavefronts per SIMD then fit).
template <int G>
struct ListArrivals {
  static constexpr uint32_t D = 8 * G;  // entries of a group
  double *at;                           // this group's part of LDS, [D] each
  uint32_t *aj;
  const double *time;
  const int32_t *type;
  int64_t n;
  int64_t end;   // the next entry to load
  uint32_t pos;  // the next arrival (low word of its index): tn, jn (at the
                 // end of the list +inf), the one after it: tn2, jn2
  double tn = INFINITY, tn2 = INFINITY;
  int32_t jn = 0, jn2 = 0;

  // at_, aj_: 512 entries of the wavefront's LDS.
  __device__ __forceinline__ ListArrivals(double *at_, uint32_t *aj_, const double *time_,
                                          const int32_t *type_, int64_t n_, int64_t pos_)
      : at(at_ + (threadIdx.x / G) * D), aj(aj_ + (threadIdx.x / G) * D), time(time_), type(type_),
        n(n_), end(pos_), pos((uint32_t)pos_) {}
  __device__ __forceinline__ uint32_t ahead() const { return (uint32_t)end - pos; }
  __device__ __forceinline__ int64_t index() const { return end - (int64_t)ahead(); }
  __device__ __forceinline__ void next2() {
    tn2 = at[(pos + 1u) & (D - 1u)];
    jn2 = (int32_t)aj[(pos + 1u) & (D - 1u)];
  }
  // Every group of `live` with half of its part free loads the next entries,
  // four per lane (each lane of the wavefront takes part).
  __device__ __forceinline__ void fill(Mask live) {
    wave_lds_sync();
    if (in(ballot(ahead() <= D / 2) & live)) {
      const uint32_t gl = threadIdx.x & (G - 1);
      double t[4];
      int32_t j[4];
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i) {
        const int64_t e = end + (int64_t)(gl + i * G);
        const bool left = e < n;
        t[i] = left ? time[e] : INFINITY;
        j[i] = left ? type[e] : 0;
      }
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i) {
        const uint32_t x = ((uint32_t)end + gl + i * G) & (D - 1u);
        at[x] = t[i];
        aj[x] = (uint32_t)j[i];
      }
      end += 4 * G;
    }
    wave_lds_sync();
  }
  __device__ __forceinline__ void start(Mask live) {
    fill(live);
    if (in(live)) {
      tn = at[pos & (D - 1u)];
      jn = (int32_t)aj[pos & (D - 1u)];
      next2();
    }
  }
  // The next arrival of the groups of `go` has been taken (each lane of the
  // wavefront takes part; `live`: the groups still running).
  __device__ __forceinline__ void advance(Mask go, Mask live) {
    if ((ballot(ahead() < 3u) & go) != 0) fill(live);
    if (in(go)) {
      pos++;
      tn = tn2;
      jn = jn2;
      __builtin_amdgcn_sched_barrier(0);  // (as in Arrivals::advance)
      next2();
    }
  }
};

// Stage the rate profile of job J in LDS (every lane of the wavefront).
template <int G, int NP>
__device__ __forceinline__ void stage_profile(const KArgs &A, const JobDev &J,
                                              RateProfLds<G, NP> &prof) {
  const double *rg = (const double *)(A.ws + J.off_rate);
  const int P = J.n_rate, m = J.m, tx = threadIdx.x;
  for (int i = tx; i < P; i += 64) prof.t[i] = rg[i];
  for (int x = tx; x < G * NP; x += 64) {
    const int j = x / NP, i = x % NP;
    prof.f[j][i] = j < m && i < P ? rg[P + j * P + i] : 0.0;
  }
  for (int j = tx; j < G; j += 64) prof.fmax[j] = j < m ? J.rate_fmax[j] : 0.0;
}

}  // namespace
}  // namespace wsim
