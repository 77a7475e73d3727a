// Event loops of small parts, one wavefront per part.
//
// Same model, arithmetic and incremental re-solve as the event loop of
// kernels.hip (finish times and statistics are the same bit for bit), for
// parts that keep few flows active at a time: chained collectives, pipeline
// sends, a training step's trace, the many tiny parts of a what-if batch.
// What bounds such a part is latency: an event is a chain of dependent steps
// on a handful of flows.  A 512-thread workgroup of the block kernel spends
// 10-12 us on one (global-memory round trips for slots, paths, pending list and
// thresholds, a dozen workgroup barriers, an event's code larger than the
// instruction cache).  Here
//   - one wave runs the part, so nothing waits at a barrier: lanes exchange
//     data through shared memory in program order, and reductions are
//     register moves between lanes;
//   - everything an event reads again lives in shared memory: link state, the
//     active flows with their path, remaining bytes and successor range, and
//     the pending list.  Global memory is read for a flow's own data when it
//     is released (one round trip, together with the countdown of its
//     predecessors) and for a finished flow's successors;
//   - the links an event's re-solve touches are listed, so a freezing round
//     looks at those links only;
//   - a part takes a few kB of shared memory instead of the whole pool, so
//     a compute unit runs up to 12 parts at once (149 registers per lane: three
//     waves a SIMD) instead of one.
// Measured (one pass through the C ABI, before: every part in the block kernel):
// ring all-reduce of 64 GPUs 12.0 -> 4.8 ms (981 events), 3D-parallel step on
// 128 GPUs 4.7 -> 1.6 ms, training-step trace of 128 GPUs 252 -> 89 ms (22,872
// events), 33,029 parts of 64 what-if scenarios 5.4 -> 2.9 ms on the device.
// A part whose active or pending flows outgrow the shared-memory lists is
// handed over to the block kernel at that event (its state written out as
// the event loop's own position, see ScenCtl::mid), which wins once there are
// several hundred flows per sweep.
#include "wave.h"

#pragma clang fp contract(off)

namespace netsim_dev {

namespace {

constexpr double WKEEP = 1.0 - 1e-9;

// D: links of the part's longest path, 2, 4 or 6.
template <int D>
struct Wave : WaveLog {
  ScenCtl* C;
  const int nl, sc, pc;
  const bool hist;  // the rollback history is kept
  // shared memory
  int64_t* R;      // [nl + 1] residual capacity
  int64_t* cap;    // [nl + 1] capacity
  double* sh;      // [nl + 1] share of the round
  int32_t* n;      // [nl + 1] unfrozen flows
  int32_t* nact;   // [nl + 1] active flows
  uint32_t* fl;    // [nl + 1] round that blocked the link
  uint16_t* ll;    // [nl + 1] links of the current re-solve
  uint64_t* theta; // [nc]
  double *tau, *rate, *rem, *tref;  // [sc] slots; a new flow's rate is 0, a free slot's id -1
  uint4* path;     // [sc]
  int32_t *id, *k0, *k1, *comp;     // [sc]
  int2* s2;        // [sc] first two successors
  uint16_t *sel, *freed;            // [sc] re-solve list (before it: new flows), free slots
  double* prel;    // [pc] pending flows: release time
  int32_t* pid;    // [pc]
  // the same in every lane
  int nSlots = 0, nFree = 0, nPend = 0, nArr = 0;
  int nSpill = 0, pSpill = 0;       // new and pending flows beyond the lists
  int ndone = 0;                    // flows that left their links in this event
  int vS = 0, vH = 0;               // slots and holes as the block kernel's layout has them
  int e = 0;
  double t = 0.0;
  uint32_t stamp = 0;
  int64_t rounds = 0, fsw = 0, isw = 0, lsw = 0;

  static __host__ __device__ size_t bytes(int nl, int nc, int sc, int pc) {
    const size_t l = (size_t)((nl + 1 + 7) & ~7), s = (size_t)((sc + 7) & ~7), p = (size_t)((pc + 7) & ~7);
    return l * 38 + (size_t)nc * 8 + s * 76 + p * 12 + WLOG + 32;
  }

  __device__ __forceinline__ Wave(const Params& P_, ScenCtl* C_, unsigned char* pool, int sc_, int pc_)
      : WaveLog(P_, C_->f0), C(C_), nl(C_->l1 - C_->l0), sc(sc_), pc(pc_),
        hist(P_.hist != nullptr && C_->hcap > 0) {
    const int l = (nl + 1 + 7) & ~7, s = (sc + 7) & ~7, p = (pc + 7) & ~7;
    unsigned char* b = pool;
    auto take = [&](size_t z) {
      unsigned char* r = b;
      b += z;
      return r;
    };
    path = reinterpret_cast<uint4*>(take((size_t)s * 16));
    ring = reinterpret_cast<Done*>(take(WQ * sizeof(Done)));
    next = reinterpret_cast<int2*>(take(64 * sizeof(int2)));
    s2 = reinterpret_cast<int2*>(take((size_t)s * 8));
    R = reinterpret_cast<int64_t*>(take((size_t)l * 8));
    cap = reinterpret_cast<int64_t*>(take((size_t)l * 8));
    sh = reinterpret_cast<double*>(take((size_t)l * 8));
    tau = reinterpret_cast<double*>(take((size_t)s * 8));
    rate = reinterpret_cast<double*>(take((size_t)s * 8));
    rem = reinterpret_cast<double*>(take((size_t)s * 8));
    tref = reinterpret_cast<double*>(take((size_t)s * 8));
    prel = reinterpret_cast<double*>(take((size_t)p * 8));
    theta = reinterpret_cast<uint64_t*>(take((size_t)C_->nc * 8));
    n = reinterpret_cast<int32_t*>(take((size_t)l * 4));
    nact = reinterpret_cast<int32_t*>(take((size_t)l * 4));
    fl = reinterpret_cast<uint32_t*>(take((size_t)l * 4));
    id = reinterpret_cast<int32_t*>(take((size_t)s * 4));
    k0 = reinterpret_cast<int32_t*>(take((size_t)s * 4));
    k1 = reinterpret_cast<int32_t*>(take((size_t)s * 4));
    comp = reinterpret_cast<int32_t*>(take((size_t)s * 4));
    pid = reinterpret_cast<int32_t*>(take((size_t)p * 4));
    ll = reinterpret_cast<uint16_t*>(take((size_t)l * 2));
    sel = reinterpret_cast<uint16_t*>(take((size_t)s * 2));
    freed = reinterpret_cast<uint16_t*>(take((size_t)s * 2));
  }

  // Flow f becomes active at time t (all lanes call it).
  __device__ __forceinline__ void activate(bool p, int f, const Own& o) {
    const uint64_t m = __ballot(p);
    if (m == 0) return;
    const int c = (int)__popcll(m), r = rank_in(m);
    if (p) {
      const int s = r < nFree ? (int)freed[nFree - 1 - r] : nSlots + r - nFree;
      if (s < sc) {
        tau[s] = WINF;
        rate[s] = 0.0;
        rem[s] = o.nb;
        tref[s] = t;
        path[s] = o.rec;
        id[s] = f;
        k0[s] = o.k0;
        k1[s] = o.k1;
        s2[s] = o.s;
        comp[s] = o.comp - C->c0;
        sel[nArr + r] = (uint16_t)s;
        int lv[D];
        const int deg = unpack<D>(o.rec, nl, lv);
#pragma unroll
        for (int k = 0; k < D; ++k)
          if (k < deg) ladd(&nact[lv[k]], 1);
      } else {
        P.comp1[f0 + nSpill + (s - sc)] = f;
        P.rem[f] = o.nb;
        P.tref[f] = t;
      }
      if (hist) P.eva[f] = e;
    }
    const int used = min(c, nFree), fresh = c - used, over = max(0, nSlots + fresh - sc);
    nFree -= used;
    nSlots = min(nSlots + fresh, sc);
    nSpill += over;
    nArr += c - over;
    vS += c;
  }

  // Counts one predecessor of flow h down; the last one releases it (all
  // lanes call it).  The flow's own data is fetched along with the count.
  __device__ __forceinline__ void countdown(bool p, int h) {
    bool zero = false, act = false, later = false;
    double rl = 0.0;
    Own o{};
    if (p) {
      const int c = __hip_atomic_fetch_add(&P.cnt[h], -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      o = own_of(P, h);
      const double st = P.start[h];
      if (c == 1) {
        double base = t;
        if (P.lat)
          base = __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<uint64_t*>(&P.base[h]),
                                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        rl = st + base;
        P.base[h] = base;
        P.rel[h] = rl;
        if (hist) P.evr[h] = e;
        later = rl > t;
        zero = !later && o.nb == 0.0;
        act = !later && !zero;
      }
    }
    if (zero) {
      P.finish[h] = rl;
      if (hist) {
        P.eva[h] = e;
        P.evd[h] = e;
      }
    }
    push(zero && o.k1 > o.k0, h, o.k0, o.k1, o.s, rl);
    activate(act, h, o);
    const uint64_t m = __ballot(later);
    if (m) {
      const int c = (int)__popcll(m), i = nPend + rank_in(m);
      if (later) {
        if (i < pc) {
          prel[i] = rl;
          pid[i] = h;
        } else {
          P.comp2[f0 + pSpill + (i - pc)] = h;
        }
      }
      const int over = max(0, nPend + c - pc);
      nPend = min(nPend + c, pc);
      pSpill += over;
    }
  }

  // Max-min rates of the nSel flows in sel, by rounds of local-minimum
  // freezing (see kernels.hip); slots get the rate and predicted completion.
  __device__ __forceinline__ int solve(int nSel) {
    int nt = 0;  // links listed
    // take back: remaining bytes up to t, the flow's rate and one unfrozen
    // flow returned to its links; the first flow of a link lists it
    for (int i0 = 0; i0 < nSel; i0 += 64) {
      const bool in = i0 + lane < nSel;
      int lv[D], deg = 0;
      if (in) {
        const int s = sel[i0 + lane];
        const double r = rate[s];
        deg = unpack<D>(path[s], nl, lv);
        if (r != 0.0) {
          const double moved = r * (t - tref[s]);
          rem[s] = rem[s] - moved;
          tref[s] = t;
          const int64_t q = (int64_t)__builtin_rint(r * P.scale);
#pragma unroll
          for (int k = 0; k < D; ++k)
            if (k < deg) ladd(&R[lv[k]], q);
        }
      }
      int old[D];
#pragma unroll
      for (int k = 0; k < D; ++k) {
        old[k] = 1;
        if (in && k < deg)
          old[k] = __hip_atomic_fetch_add(&n[lv[k]], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
#pragma unroll
      for (int k = 0; k < D; ++k) {
        const bool first = old[k] == 0;
        const uint64_t m = __ballot(first);
        if (first) ll[nt + rank_in(m)] = (uint16_t)lv[k];
        nt += (int)__popcll(m);
      }
    }
    wsync();
    if (stamp > 0x7FFFFFFFu) {  // far from wrapping, stamps start over
      for (int l = lane; l <= nl; l += 64) fl[l] = 0;
      stamp = 0;
      wsync();
    }
    int total = nSel, r = 0;
    for (;;) {
      const uint32_t st = ++stamp;
      // shares of the re-solve's links that still carry unfrozen flows
      for (int i0 = 0; i0 < nt; i0 += 64) {
        bool some = false;
        if (i0 + lane < nt) {
          const int l = ll[i0 + lane];
          const int c = n[l];
          some = c > 0;
          if (some) sh[l] = ((double)R[l] / (double)c) * P.inv_scale;
        }
        lsw += __popcll(__ballot(some));
      }
      wsync();
      // smallest share on each path; links above it are blocked
      bool bad = false;
      double m = 0.0;
      uint32_t cm = 0;
      int lv[D], deg = 0, s = 0;
      bool in = false;
      auto look = [&](int i0) {
        in = i0 + lane < total;
        cm = 0;
        if (!in) return;
        s = sel[i0 + lane];
        deg = unpack<D>(path[s], nl, lv);
        isw += deg;
        double sv[D];
#pragma unroll
        for (int k = 0; k < D; ++k) sv[k] = sh[lv[k]];
        m = sv[0];
#pragma unroll
        for (int k = 1; k < D; ++k) m = sv[k] < m ? sv[k] : m;
        const double thr = m * WTHR;
#pragma unroll
        for (int k = 0; k < D; ++k) {
          if (!(sv[k] > thr)) cm |= 1u << k;
          else if (sv[k] < WINF) fl[lv[k]] = st;
        }
        if (!(m > 0.0) || !(m < WINF)) bad = true;
      };
      // flows at the minimum of an unblocked link freeze there; the others
      // stay listed, in place
      int left = 0;
      auto freeze = [&]() {
        bool frozen = false;
        if (in) {
#pragma unroll
          for (int k = 0; k < D; ++k)
            if ((cm >> k) & 1u) frozen |= fl[lv[k]] != st;
          if (frozen) {
            rate[s] = m;
            tau[s] = t + rem[s] / m;
            const int64_t q = (int64_t)__builtin_rint(m * P.scale);
#pragma unroll
            for (int k = 0; k < D; ++k)
              if (k < deg) {
                ladd(&R[lv[k]], -q);
                ladd(&n[lv[k]], -1);
              }
          }
        }
        const bool keep = in && !frozen;
        const uint64_t km = __ballot(keep);
        if (keep) sel[left + rank_in(km)] = (uint16_t)s;
        left += (int)__popcll(km);
      };
      if (total <= 64) {
        look(0);
        wsync();
        freeze();
      } else {
        // the share at the minimum and the links at it wait in the record's
        // spare word and the slot's rate
        for (int i0 = 0; i0 < total; i0 += 64) {
          look(i0);
          if (in) {
            path[s].w = cm;
            rate[s] = m;
          }
        }
        wsync();
        for (int i0 = 0; i0 < total; i0 += 64) {
          in = i0 + lane < total;
          if (in) {
            s = sel[i0 + lane];
            const uint4 rec = path[s];
            cm = rec.w;
            m = rate[s];
            deg = unpack<D>(rec, nl, lv);
          }
          wsync();
          freeze();
          wsync();
        }
      }
      wsync();
      rounds += 1;
      fsw += total;
      if (__ballot(bad) != 0) return ST_BAD_SHARE;
      if (left == 0) return ST_DONE;
      if (left >= total) return ST_BAD_SHARE;  // a round must freeze something
      if (++r > P.max_rounds) return ST_ROUNDS;
      total = left;
    }
  }

  // Active flows to the front of the slots (every sweep looks at all slots).
  __device__ __forceinline__ void compact() {
    int keep = 0;
    for (int s0 = 0; s0 < nSlots; s0 += 64) {
      const int s = s0 + lane;
      const int f = s < nSlots ? id[s] : -1;
      uint4 p{};
      double a = 0.0, b = 0.0, c = 0.0, d = 0.0;
      int x = 0, y = 0, z = 0;
      int2 v{};
      if (f >= 0) {
        p = path[s];
        a = tau[s];
        b = rate[s];
        c = rem[s];
        d = tref[s];
        x = k0[s];
        y = k1[s];
        z = comp[s];
        v = s2[s];
      }
      wsync();
      const uint64_t m = __ballot(f >= 0);
      if (f >= 0) {
        const int to = keep + rank_in(m);
        path[to] = p;
        tau[to] = a;
        rate[to] = b;
        rem[to] = c;
        tref[to] = d;
        id[to] = f;
        k0[to] = x;
        k1[to] = y;
        comp[to] = z;
        s2[to] = v;
      }
      keep += (int)__popcll(m);
      wsync();
    }
    nSlots = keep;
    nFree = 0;
  }

  // Reads the position a launch left (or the start), if the lists hold it.
  __device__ __forceinline__ bool load(bool resume) {
    if (resume && (C->nslots - C->holes > sc || C->npend > pc)) return false;
    if (!resume && C->n_pend0 > pc) return false;
    for (int l = lane; l < nl; l += 64) {
      const int64_t c = P.R0[C->l0 + l];
      R[l] = c;
      cap[l] = c;
      n[l] = 0;
      nact[l] = 0;
      fl[l] = 0;
    }
    if (lane == 0) {
      R[nl] = 0;
      cap[nl] = 0;
      sh[nl] = WINF;
      n[nl] = 0;
      nact[nl] = 0;
      fl[nl] = 0;
    }
    for (int c = lane; c < C->nc; c += 64) theta[c] = (uint64_t)__double_as_longlong(WINF);
    wsync();
    e = resume ? C->e : 0;
    nPend = resume ? C->npend : C->n_pend0;
    const int32_t* pl = (e & 1) ? P.pend1 + f0 : P.pend0 + f0;
    for (int i = lane; i < nPend; i += 64) {
      const int f = pl[i];
      pid[i] = f;
      prel[i] = P.rel[f];
    }
    if (!resume) return true;
    t = C->t;
    vS = C->nslots;
    vH = C->holes;
    const int32_t* ai = C->ab ? P.act1 + f0 : P.act0 + f0;
    const double* at = C->ab ? P.tau1 + f0 : P.tau0 + f0;
    const double* ar = C->ab ? P.srate1 + f0 : P.srate0 + f0;
    for (int i0 = 0; i0 < vS; i0 += 64) {
      const int f = i0 + lane < vS ? ai[i0 + lane] : -1;
      const uint64_t m = __ballot(f >= 0);
      if (f >= 0) {
        const int s = nSlots + rank_in(m);
        const Own o = own_of(P, f);
        const double r = ar[i0 + lane];
        tau[s] = at[i0 + lane];
        rate[s] = r;
        rem[s] = P.rem[f];
        tref[s] = P.tref[f];
        path[s] = o.rec;
        id[s] = f;
        k0[s] = o.k0;
        k1[s] = o.k1;
        s2[s] = o.s;
        comp[s] = o.comp - C->c0;
        const int64_t q = (int64_t)__builtin_rint(r * P.scale);
        int lv[D];
        const int deg = unpack<D>(o.rec, nl, lv);
#pragma unroll
        for (int k = 0; k < D; ++k)
          if (k < deg) {
            ladd(&nact[lv[k]], 1);
            ladd(&R[lv[k]], -q);
          }
      }
      nSlots += (int)__popcll(m);
    }
    wsync();
    return true;
  }

  // Writes the position out as the block kernel's: slots in buffer 0 (those
  // activated in the current event last, from slots0 on, holes before them),
  // pending flows in list pb.  Returns the number of new flows (listed in
  // P.arr).
  __device__ __forceinline__ int dump(int slots0, int pb) {
    int old = 0, fresh = 0;
    const int nNew = vS - slots0;
    for (int s0 = 0; s0 < nSlots; s0 += 64) {
      const int s = s0 + lane;
      const int f = s < nSlots ? id[s] : -1;
      const bool neu = f >= 0 && nNew > 0 && rate[s] == 0.0;
      const uint64_t mo = __ballot(f >= 0 && !neu), mn = __ballot(neu);
      if (f >= 0) {
        const int i = neu ? slots0 + fresh + rank_in(mn) : old + rank_in(mo);
        P.act0[f0 + i] = f;
        P.tau0[f0 + i] = tau[s];
        P.srate0[f0 + i] = rate[s];
        P.rem[f] = rem[s];
        P.tref[f] = tref[s];
        P.rate[f] = rate[s];
        if (neu) P.arr[f0 + i - slots0] = f;
      }
      old += (int)__popcll(mo);
      fresh += (int)__popcll(mn);
    }
    for (int i = lane; i < nSpill; i += 64) {
      const int f = P.comp1[f0 + i], j = slots0 + fresh + i;
      P.act0[f0 + j] = f;
      P.tau0[f0 + j] = WINF;
      P.srate0[f0 + j] = 0.0;
      P.arr[f0 + j - slots0] = f;
    }
    for (int i = old + lane; i < slots0; i += 64) {
      P.act0[f0 + i] = -1;
      P.tau0[f0 + i] = WINF;
      P.srate0[f0 + i] = 0.0;
    }
    int32_t* pl = pb ? P.pend1 + f0 : P.pend0 + f0;
    for (int i = lane; i < nPend; i += 64) pl[i] = pid[i];
    for (int i = lane; i < pSpill; i += 64) pl[nPend + i] = P.comp2[f0 + i];
    return nNew;
  }
};

template <int D>
__device__ __forceinline__ void wave_loop(const Params& P, int part, int sc, int pc, unsigned char* pool) {
  ScenCtl* C = &P.ctl[part];
  Wave<D> w(P, C, pool, sc, pc);
  const int lane = w.lane;
  const bool resume = P.resume && C->started;
  if (!w.load(resume)) {  // more than the lists hold: the block kernel's from here
    if (lane == 0) {
      C->launch_events = 0;
      for (int k = 0; k < 8; ++k) C->ticks[k] = 0;
      P.hlist[__hip_atomic_fetch_add(P.hcount, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)] = part;
    }
    return;
  }
  int64_t events = resume ? C->events : 0, solves = resume ? C->solves : 0;
  int64_t asw = resume ? C->active_swept : 0, psw = resume ? C->pending_swept : 0;
  int64_t nsel = resume ? C->reselected : 0, hp = resume ? C->hpos : 0;
  w.rounds = resume ? C->rounds : 0;
  w.fsw = resume ? C->flows_swept : 0;
  const int64_t events0 = events;
  const int64_t wide = resume ? C->wide_solves : 0, asst = resume ? C->assisted : 0;
  const bool hist = w.hist;
  const int nc = C->nc;
  const bool clk = (P.debug & 2) != 0;
  uint64_t ticks[8] = {}, last = clk ? wall_clock64() : 0;
  auto lap = [&](int k) {
    if (clk) {
      const uint64_t now = wall_clock64();
      ticks[k] += now - last;
      last = now;
    }
  };
  int status = ST_DONE, mid = 0, slots0 = 0;
  for (;;) {
    // next event: earliest predicted completion or release
    double loc = WINF;
    for (int s = lane; s < w.nSlots; s += 64) {
      const double v = w.tau[s];
      loc = v < loc ? v : loc;
    }
    for (int i = lane; i < w.nPend; i += 64) {
      const double v = w.prel[i];
      loc = v < loc ? v : loc;
    }
    asw += w.vS;
    psw += w.nPend;
    const double tn = wmin(loc);
    lap(0);
    if (!(tn < WINF)) break;
    if ((P.max_events > 0 && events - events0 >= P.max_events) || tn > P.until) {
      status = ST_STOPPED;
      break;
    }
    // every event completes or releases a flow, so a part of F flows has at
    // most 2 F events
    if (events - events0 > 2 * (int64_t)(C->f1 - C->f0)) {
      status = ST_OVERFLOW;
      break;
    }
    events += 1;
    const double thr = tn * WTHR;
    w.t = tn;
    w.qh = w.qt = 0;
    w.nArr = w.ndone = 0;
    slots0 = w.vS;
    // completions
    for (int s0 = 0; s0 < w.nSlots; s0 += 64) {
      const int s = s0 + lane;
      const bool due = s < w.nSlots && w.tau[s] <= thr;
      const uint64_t m = __ballot(due);
      if (m == 0) continue;
      int f = 0, a = 0, b = 0;
      int2 next = {0, 0};
      double fin = tn;
      if (due) {
        f = w.id[s];
        a = w.k0[s];
        b = w.k1[s];
        next = w.s2[s];
        const double r = w.rate[s];
        // the last byte leaves now; it arrives the path latency later
        if (P.lat) fin = tn + P.lat[f];
        P.finish[f] = fin;
        if (hist) {
          P.evd[f] = w.e;
          P.rem[f] = w.rem[s];
          P.tref[f] = w.tref[s];
          P.rate[f] = r;
        }
        __hip_atomic_fetch_min(&w.theta[w.comp[s]], (uint64_t)__double_as_longlong(r), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
        const int64_t q = (int64_t)__builtin_rint(r * P.scale);
        int lv[D];
        const int deg = unpack<D>(w.path[s], w.nl, lv);
#pragma unroll
        for (int k = 0; k < D; ++k)
          if (k < deg) {
            ladd(&w.nact[lv[k]], -1);
            ladd(&w.R[lv[k]], q);  // its share returns to the link
          }
        w.id[s] = -1;
        w.tau[s] = WINF;
        w.freed[w.nFree + rank_in(m)] = (uint16_t)s;
      }
      w.push(due && b > a, f, a, b, next, fin);
      const int c = (int)__popcll(m);
      w.nFree += c;
      w.ndone += c;
    }
    w.vH += w.ndone;
    wsync();
    // releases due now; the pending list is compacted in place
    {
      const int np = w.nPend;
      int keep = 0;
      for (int i0 = 0; i0 < np; i0 += 64) {
        const bool in = i0 + lane < np;
        const int f = in ? w.pid[i0 + lane] : 0;
        const double rl = in ? w.prel[i0 + lane] : WINF;
        const bool due = in && rl <= tn;
        if (__ballot(due) != 0) {
          Own o{};
          if (due) o = own_of(P, f);
          const bool zero = due && o.nb == 0.0;
          if (zero) {
            P.finish[f] = rl;
            if (hist) {
              P.eva[f] = w.e;
              P.evd[f] = w.e;
            }
          }
          w.push(zero && o.k1 > o.k0, f, o.k0, o.k1, o.s, rl);
          w.activate(due && !zero, f, o);
        }
        wsync();
        const uint64_t m = __ballot(in && !due);
        if (in && !due) {
          const int i = keep + rank_in(m);
          w.prel[i] = rl;
          w.pid[i] = f;
        }
        keep += (int)__popcll(m);
        wsync();
      }
      w.nPend = keep;
    }
    // dependants of finished flows, to a fixpoint through zero-byte flows
    while (w.qh < w.qt) {
      wsync();
      const int cnt = min(64, w.qt - w.qh);
      if (P.lat) {
        // a dependant starts after the latest arrival among its
        // predecessors: every finished flow raises its dependants' base
        // before it counts them down
        w.successors(cnt, [&](bool in, int g, double fin) {
          if (in)
            __hip_atomic_fetch_max(reinterpret_cast<uint64_t*>(&P.base[g]),
                                   (uint64_t)__double_as_longlong(fin), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        });
        // the raises are performed before a base is read
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
      }
      // entries the countdown appends may reuse the ring slots of this batch
      // (read before the first countdown), never those of later batches that
      // are still in it
      w.successors(cnt, [&](bool in, int g, double) { w.countdown(in, g); });
      w.qh += cnt;
    }
    wsync();
    lap(1);
    const bool changed = w.ndone > 0 || w.vS > slots0;
    if (w.nSpill > 0 || w.pSpill > 0) {
      mid = 1 | (changed ? 2 : 0);
      break;
    }
    if (changed && w.vS - w.vH > 0) {
      // theta of each component: below it every rate stays as it was (see
      // the event loop of kernels.hip); new flows feed the initial share of
      // their links
      for (int i = lane; i < w.nArr; i += 64) {
        const int s = w.sel[i];
        int lv[D];
        const int deg = unpack<D>(w.path[s], w.nl, lv);
        double lo = WINF;
#pragma unroll
        for (int k = 0; k < D; ++k)
          if (k < deg) {
            const double s0 = ((double)w.cap[lv[k]] / (double)w.nact[lv[k]]) * P.inv_scale;
            lo = s0 < lo ? s0 : lo;
          }
        __hip_atomic_fetch_min(&w.theta[w.comp[s]], (uint64_t)__double_as_longlong(lo), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      wsync();
      int nSel = 0;
      for (int s0 = 0; s0 < w.nSlots; s0 += 64) {
        const int s = s0 + lane;
        const int f = s < w.nSlots ? w.id[s] : -1;
        bool take = false;
        if (f >= 0) {
          const double r = w.rate[s];
          take = r == 0.0 || !(r < __longlong_as_double((long long)w.theta[w.comp[s]]) * WKEEP);
        }
        const uint64_t m = __ballot(take);
        if (take) {
          const int i = nSel + rank_in(m);
          w.sel[i] = (uint16_t)s;
          if (hist) {
            // undo record: the flow's values before this event re-solves it
            HistUndo u;
            u.f = f;
            u.ev = w.e;
            u.rem = w.rem[s];
            u.tref = w.tref[s];
            u.rate = w.rate[s];
            P.hist[C->hbase + (hp + i) % C->hcap] = u;
          }
        }
        nSel += (int)__popcll(m);
      }
      wsync();
      for (int c = lane; c < nc; c += 64) w.theta[c] = (uint64_t)__double_as_longlong(WINF);
      wsync();
      lap(7);
      nsel += nSel;
      hp += nSel;
      int rc = 0;
      if (nSel > 0) rc = w.solve(nSel);
      lap(3);
      solves += 1;
      if (rc != 0) {
        status = rc;
        break;
      }
    }
    // the block kernel's compaction rule (its slot count is a statistic)
    if (8 * w.vH > w.vS) {
      w.vS -= w.vH;
      w.vH = 0;
    }
    if (w.nFree == w.nSlots) w.nFree = w.nSlots = 0;
    else if (w.nFree >= 64) w.compact();
    if (hist && lane == 0) {
      HistEv r;
      r.t = w.t;
      r.hpos = hp;
      r.solves = solves;
      r.rounds = w.rounds;
      r.flows_swept = w.fsw;
      r.active_swept = asw;
      r.pending_swept = psw;
      r.reselected = nsel;
      r.wide_solves = wide;
      r.assisted = asst;
      P.hev[C->ebase + (int64_t)w.e % C->ecap] = r;
    }
    w.e += 1;
  }
  wsync();
  const int narr = mid ? w.dump(slots0, (w.e & 1) ^ 1) : w.dump(w.vS, w.e & 1);
  if (mid)
    for (int c = lane; c < nc; c += 64) P.theta[C->c0 + c] = w.theta[c];
  const int64_t isw = wsum(w.isw);
  if (lane == 0) {
    C->started = 1;
    C->mid = mid;
    C->mid_slots0 = slots0;
    C->mid_narr = narr;
    C->e = w.e;
    C->q = 0;
    C->ab = 0;
    C->nslots = w.vS;
    C->holes = w.vH;
    C->npend = w.nPend + w.pSpill;
    C->t = w.t;
    C->events = events;
    C->solves = solves;
    C->rounds = w.rounds;
    C->flows_swept = w.fsw;
    C->incidences_swept = (resume ? C->incidences_swept : 0) + isw;
    C->active_swept = asw;
    C->pending_swept = psw;
    C->reselected = nsel;
    C->wide_solves = wide;
    C->assisted = asst;
    C->links_swept = (resume ? C->links_swept : 0) + w.lsw;
    C->hpos = hp;
    C->launch_events = events - events0;
    C->status = status;
    for (int k = 0; k < 8; ++k) C->ticks[k] = (int64_t)ticks[k];
    if (mid) P.hlist[__hip_atomic_fetch_add(P.hcount, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)] = part;
  }
}

}  // namespace

__global__ __launch_bounds__(64) void netsim_wave_kernel(Params P, const int32_t* list, int sc, int pc) {
  extern __shared__ __align__(16) unsigned char wpool[];
  // a loop over a path's links is unrolled to the longest path of the part:
  // unpacking and guarding six for paths of one or two was a third of a
  // solve's instructions (trace of 128 GPUs 106 -> 88 ms, 3D-parallel step 1.95
  // -> 1.60 ms; one loop that ends on a scalar saved a quarter of that on paths
  // of two links and cost 15% on longer ones, its reads no longer side by side)
  const int part = list[blockIdx.x];
  const int deg = __builtin_amdgcn_readfirstlane(P.ctl[part].deg);
  if (deg <= 2) wave_loop<2>(P, part, sc, pc, wpool);
  else if (deg <= 4) wave_loop<4>(P, part, sc, pc, wpool);
  else wave_loop<6>(P, part, sc, pc, wpool);
}

size_t wave_bytes(int nl, int nc, int sc, int pc) { return Wave<6>::bytes(nl, nc, sc, pc); }

hipError_t launch_wave(const Params& p, const int32_t* list, int parts, int sc, int pc, size_t lds, hipStream_t s) {
  hipError_t e = hipFuncSetAttribute((const void*)netsim_wave_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(netsim_wave_kernel, dim3(parts), dim3(64), lds, s, p, list, sc, pc);
  return hipGetLastError();
}

}  // namespace netsim_dev
