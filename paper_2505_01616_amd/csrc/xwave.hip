// Exact mode's event loop for small scenarios, one wavefront per scenario:
// the arithmetic of exact.hip (the same bits and counters) in the form of
// wave.hip -- no workgroup barriers, active and pending flows and link state
// in shared memory -- for scenarios that keep few flows active at a time.
//
// A solve goes level by level over the active flows, up to 64 * C of them
// held in registers (path and whether unfrozen): a level is a pass over the
// links in use (a few per lane), a minimum by register moves and six gathers
// per flow.  The 512-thread kernel spends 3 to 4 us on a level of a few dozen
// links and flows, in its two barriers and the lists it keeps in global memory.
// Measured (complete runs): gradient rings of 4 x 32 ranks with 200 background
// transfers on a degraded 1024-GPU fat-tree 286 -> 165 ms (7,974 events, 59,094
// levels), chained ring of 46 ranks 85 -> 35 ms, 3D-parallel step 38 -> 28 ms.
// A scenario whose active or pending flows outgrow the lists is handed over
// to the workgroup kernel at that event, before its solve (ScenCtl::mid).
#include "wave.h"

namespace netsim_dev {

namespace {

struct XWave : WaveLog {
  ScenCtl* C;
  const int nl, sc, pc;
  // shared memory; after the links an entry per lane that stands for the
  // absent links of its flows (share +inf, counts that nothing reads), so that
  // path gathers and counts need no guard and no branch
  double *cap, *R, *s;     // [nl + 64] capacity, residual, share of the level
  int32_t *n, *k;          // [nl + 64] unfrozen flows, flows frozen in the level
  uint16_t* ll;            // [nl + 64] links with unfrozen flows
  double *rate, *rem, *tau;  // [sc] slots; a free slot's id is -1
  uint4* path;             // [sc] absent links as nl; w: the degree
  int32_t *id, *k0, *k1;   // [sc]
  int2* s2;                // [sc] first two successors
  uint16_t* freed;         // [sc] free slots
  double* prel;            // [pc] pending flows: release time
  int32_t* pid;            // [pc]
  // the same in every lane
  int nSlots = 0, nFree = 0, nPend = 0, nSpill = 0, pSpill = 0;
  bool changed = false;
  double t = 0.0;
  int64_t rounds = 0, fsw = 0, isw = 0, lsw = 0;

  static __host__ __device__ size_t bytes(int nl, int sc, int pc) {
    const size_t l = (size_t)((nl + 64 + 7) & ~7), z = (size_t)((sc + 7) & ~7), p = (size_t)((pc + 7) & ~7);
    return l * 34 + z * 62 + p * 12 + WLOG + 32;
  }

  __device__ __forceinline__ XWave(const Params& P_, ScenCtl* C_, unsigned char* pool, int sc_, int pc_)
      : WaveLog(P_, C_->f0), C(C_), nl(C_->l1 - C_->l0), sc(sc_), pc(pc_) {
    const int l = (nl + 64 + 7) & ~7, z = (sc + 7) & ~7, p = (pc + 7) & ~7;
    unsigned char* b = pool;
    auto take = [&](size_t x) {
      unsigned char* r = b;
      b += x;
      return r;
    };
    path = reinterpret_cast<uint4*>(take((size_t)z * 16));
    ring = reinterpret_cast<Done*>(take(WQ * sizeof(Done)));
    next = reinterpret_cast<int2*>(take(64 * sizeof(int2)));
    s2 = reinterpret_cast<int2*>(take((size_t)z * 8));
    cap = reinterpret_cast<double*>(take((size_t)l * 8));
    R = reinterpret_cast<double*>(take((size_t)l * 8));
    s = reinterpret_cast<double*>(take((size_t)l * 8));
    rate = reinterpret_cast<double*>(take((size_t)z * 8));
    rem = reinterpret_cast<double*>(take((size_t)z * 8));
    tau = reinterpret_cast<double*>(take((size_t)z * 8));
    prel = reinterpret_cast<double*>(take((size_t)p * 8));
    n = reinterpret_cast<int32_t*>(take((size_t)l * 4));
    k = reinterpret_cast<int32_t*>(take((size_t)l * 4));
    id = reinterpret_cast<int32_t*>(take((size_t)z * 4));
    k0 = reinterpret_cast<int32_t*>(take((size_t)z * 4));
    k1 = reinterpret_cast<int32_t*>(take((size_t)z * 4));
    pid = reinterpret_cast<int32_t*>(take((size_t)p * 4));
    ll = reinterpret_cast<uint16_t*>(take((size_t)l * 2));
    freed = reinterpret_cast<uint16_t*>(take((size_t)z * 2));
  }

  __device__ __forceinline__ void fill(int at, int f, const Own& o, double left, double r) {
    int lv[6];
    const int deg = unpack(o.rec, nl, lv);
    path[at] = make_uint4((uint32_t)lv[0] | (uint32_t)lv[1] << 16, (uint32_t)lv[2] | (uint32_t)lv[3] << 16,
                          (uint32_t)lv[4] | (uint32_t)lv[5] << 16, (uint32_t)deg);
    rate[at] = r;
    rem[at] = left;
    id[at] = f;
    k0[at] = o.k0;
    k1[at] = o.k1;
    s2[at] = o.s;
  }

  // Flow f becomes active (all lanes call it).
  __device__ __forceinline__ void activate(bool p, int f, const Own& o) {
    const uint64_t m = __ballot(p);
    if (m == 0) return;
    const int c = (int)__popcll(m), r = rank_in(m);
    if (p) {
      const int at = r < nFree ? (int)freed[nFree - 1 - r] : nSlots + r - nFree;
      if (at < sc) {
        fill(at, f, o, o.nb, 0.0);
      } else {
        P.comp1[f0 + nSpill + (at - sc)] = f;
        P.rem[f] = o.nb;
      }
    }
    const int used = min(c, nFree), fresh = c - used, over = max(0, nSlots + fresh - sc);
    nFree -= used;
    nSlots = min(nSlots + fresh, sc);
    nSpill += over;
    changed = true;
  }

  // A flow released at rl: it arrives, or (later than t) waits for its
  // release (all lanes call it; `in`: the lane has one).
  __device__ __forceinline__ void arrive(bool in, int f, double rl, const Own& o) {
    const bool later = in && rl > t, zero = in && !later && o.nb == 0.0;
    if (zero) P.finish[f] = rl;
    push(zero && o.k1 > o.k0, f, o.k0, o.k1, o.s, rl);
    activate(in && !later && !zero, f, o);
    const uint64_t m = __ballot(later);
    if (m) {
      const int c = (int)__popcll(m), i = nPend + rank_in(m);
      if (later) {
        if (i < pc) {
          prel[i] = rl;
          pid[i] = f;
        } else {
          P.comp2[f0 + pSpill + (i - pc)] = f;
        }
      }
      const int over = max(0, nPend + c - pc);
      nPend = min(nPend + c, pc);
      pSpill += over;
    }
  }

  // Rates of the active flows, at most 64 * C of them (slots [0, nSlots)).
  template <int CH>
  __device__ __forceinline__ int solve() {
    uint32_t w0[CH], w1[CH], w2[CH];
    int deg[CH];
    int nt = 0, nu = 0;
    // unfrozen counts; the first flow on a link lists it
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      deg[c] = 0;  // degree of an unfrozen flow, else 0
      w0[c] = w1[c] = w2[c] = 0;
      if (c * 64 >= nSlots) continue;
      const int at = c * 64 + lane;
      const bool in = at < nSlots && id[at] >= 0;
      int lv[6];
      if (in) {
        const uint4 r = path[at];
        w0[c] = r.x;
        w1[c] = r.y;
        w2[c] = r.z;
        deg[c] = (int)r.w;
      }
      links(w0[c], w1[c], w2[c], lv);
#pragma unroll
      for (int j = 0; j < 6; ++j) lv[j] = j < deg[c] ? lv[j] : nl + lane;
      w0[c] = (uint32_t)lv[0] | (uint32_t)lv[1] << 16;
      w1[c] = (uint32_t)lv[2] | (uint32_t)lv[3] << 16;
      w2[c] = (uint32_t)lv[4] | (uint32_t)lv[5] << 16;
      int old[6];
#pragma unroll
      for (int j = 0; j < 6; ++j)
        old[j] = __hip_atomic_fetch_add(&n[lv[j]], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
      for (int j = 0; j < 6; ++j) {
        const bool first = old[j] == 0 && j < deg[c];
        const uint64_t m = __ballot(first);
        if (first) ll[nt + rank_in(m)] = (uint16_t)lv[j];
        nt += (int)__popcll(m);
      }
      nu += (int)__popcll(__ballot(in));
    }
    wsync();
    double sprev = 0.0;
    bool first = true;
    int levels = 0;
    while (nu > 0) {
      if (levels >= P.max_rounds) return ST_ROUNDS;
      ++levels;
      // link pass: apply the last level's freezes, new shares, level minimum
      // (three links of a lane in flight; the list is compacted in place)
      double loc = WINF;
      int keep = 0;
      for (int i0 = 0; i0 < nt; i0 += 192) {
        int l[3], c[3], kk[3];
        double r[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          const int i = i0 + u * 64 + lane;
          l[u] = i < nt ? (int)ll[i] : nl + lane;
        }
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          c[u] = n[l[u]];
          kk[u] = k[l[u]];
          r[u] = first ? cap[l[u]] : R[l[u]];
        }
        wsync();
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          // (a link without freezes keeps its bits: its product is zero)
          const double dec = (double)kk[u] * sprev;
          r[u] = r[u] - dec;
          c[u] -= kk[u];
          n[l[u]] = c[u];
          k[l[u]] = 0;
          R[l[u]] = r[u];
          const bool live = i0 + u * 64 + lane < nt && c[u] > 0;
          const double v = live ? r[u] / (double)c[u] : WINF;
          s[l[u]] = v;
          loc = v < loc ? v : loc;
          const uint64_t m = __ballot(live);
          if (live) ll[keep + rank_in(m)] = (uint16_t)l[u];
          keep += (int)__popcll(m);
        }
        wsync();
      }
      nt = keep;
      lsw += nt;
      const double sstar = wmin(loc);
      if (!(sstar > 0.0) || !(sstar < WINF)) return ST_BAD_SHARE;
      first = false;
      rounds += 1;
      fsw += nu;
      const double thr = sstar * WTHR;
      // flows crossing a bottleneck freeze at s*
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        if (c * 64 >= nSlots || __ballot(deg[c] > 0) == 0) continue;
        isw += deg[c];
        int lv[6];
        links(w0[c], w1[c], w2[c], lv);
        bool fz = false;
#pragma unroll
        for (int j = 0; j < 6; ++j) fz |= s[lv[j]] <= thr;
        fz = fz && deg[c] > 0;
        if (fz) {
          rate[c * 64 + lane] = sstar;
#pragma unroll
          for (int j = 0; j < 6; ++j) ladd(&k[lv[j]], 1);
          deg[c] = 0;
        }
        nu -= (int)__popcll(__ballot(fz));
      }
      wsync();
      sprev = sstar;
    }
    // the last level's links go back to rest
    for (int i = lane; i < nt; i += 64) {
      n[ll[i]] = 0;
      k[ll[i]] = 0;
    }
    wsync();
    return ST_DONE;
  }

  static __device__ __forceinline__ void links(uint32_t a, uint32_t b, uint32_t c, int* lv) {
    lv[0] = (int)(a & 0xFFFFu);
    lv[1] = (int)(a >> 16);
    lv[2] = (int)(b & 0xFFFFu);
    lv[3] = (int)(b >> 16);
    lv[4] = (int)(c & 0xFFFFu);
    lv[5] = (int)(c >> 16);
  }

  // Active flows to the front of the slots (every sweep looks at all slots).
  __device__ __forceinline__ void compact() {
    int keep = 0;
    for (int s0 = 0; s0 < nSlots; s0 += 64) {
      const int at = s0 + lane;
      const int f = at < nSlots ? id[at] : -1;
      uint4 p{};
      double a = 0.0, b = 0.0;
      int x = 0, y = 0;
      int2 v{};
      if (f >= 0) {
        p = path[at];
        a = rate[at];
        b = rem[at];
        x = k0[at];
        y = k1[at];
        v = s2[at];
      }
      wsync();
      const uint64_t m = __ballot(f >= 0);
      if (f >= 0) {
        const int to = keep + rank_in(m);
        path[to] = p;
        rate[to] = a;
        rem[to] = b;
        id[to] = f;
        k0[to] = x;
        k1[to] = y;
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
    const int na = resume ? C->nslots : 0, np = resume ? C->npend : C->n_pend0;
    if (na > sc || np > pc) return false;
    for (int l = lane; l < nl + 64; l += 64) {
      cap[l] = l < nl ? P.capf[C->l0 + l] : 0.0;
      R[l] = 0.0;
      s[l] = WINF;
      n[l] = 0;
      k[l] = 0;
    }
    const int32_t* pl = resume && C->e ? P.pend1 + f0 : P.pend0 + f0;
    for (int i = lane; i < np; i += 64) {
      const int f = pl[i];
      pid[i] = f;
      prel[i] = P.rel[f];
    }
    nPend = np;
    if (resume) {
      t = C->t;
      const int32_t* al = C->ab ? P.act1 + f0 : P.act0 + f0;
      for (int i = lane; i < na; i += 64) {
        const int f = al[i];
        fill(i, f, own_of(P, f), P.rem[f], P.rate[f]);
      }
      nSlots = na;
    }
    wsync();
    return true;
  }

  // Writes the position out as the workgroup kernel's (lists in buffer 0);
  // returns the number of active flows.
  __device__ __forceinline__ int dump() {
    int na = 0;
    for (int s0 = 0; s0 < nSlots; s0 += 64) {
      const int at = s0 + lane;
      const int f = at < nSlots ? id[at] : -1;
      const uint64_t m = __ballot(f >= 0);
      if (f >= 0) {
        P.act0[f0 + na + rank_in(m)] = f;
        P.rem[f] = rem[at];
        P.rate[f] = rate[at];
      }
      na += (int)__popcll(m);
    }
    for (int i = lane; i < nSpill; i += 64) P.act0[f0 + na + i] = P.comp1[f0 + i];
    for (int i = lane; i < nPend; i += 64) P.pend0[f0 + i] = pid[i];
    for (int i = lane; i < pSpill; i += 64) P.pend0[f0 + nPend + i] = P.comp2[f0 + i];
    return na + nSpill;
  }
};

__device__ __forceinline__ void xwave_loop(const Params& P, int part, int sc, int pc, unsigned char* pool) {
  ScenCtl* C = &P.ctl[part];
  XWave w(P, C, pool, sc, pc);
  const int lane = w.lane;
  const bool resume = P.resume && C->started;
  if (!w.load(resume)) {  // more than the lists hold: the workgroup kernel's from here
    if (lane == 0) {
      C->launch_events = 0;
      P.hlist[__hip_atomic_fetch_add(P.hcount, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)] = part;
    }
    return;
  }
  int64_t events = resume ? C->events : 0, solves = resume ? C->solves : 0;
  int64_t asw = resume ? C->active_swept : 0, psw = resume ? C->pending_swept : 0;
  w.rounds = resume ? C->rounds : 0;
  w.fsw = resume ? C->flows_swept : 0;
  w.lsw = resume ? C->links_swept : 0;
  const int64_t events0 = events;
  int status = ST_DONE, mid = 0;
  for (;;) {
    const int na = w.nSlots - w.nFree;
    if (na == 0 && w.nPend == 0) break;
    if (P.max_events > 0 && events - events0 >= P.max_events) {
      status = ST_STOPPED;
      break;
    }
    // next event: earliest predicted completion or release
    double loc = WINF;
    for (int at = lane; at < w.nSlots; at += 64) {
      double v = WINF;
      if (w.id[at] >= 0) v = w.t + w.rem[at] / w.rate[at];
      w.tau[at] = v;
      loc = v < loc ? v : loc;
    }
    for (int i = lane; i < w.nPend; i += 64) {
      const double v = w.prel[i];
      loc = v < loc ? v : loc;
    }
    const double tn = wmin(loc);
    asw += na;
    psw += w.nPend;
    if (tn > P.until) {
      status = ST_STOPPED;
      break;
    }
    // every event completes or releases a flow, so a scenario of F flows has
    // at most 2 F events
    if (events - events0 > 2 * (int64_t)(C->f1 - C->f0)) {
      status = ST_OVERFLOW;
      break;
    }
    events += 1;
    const double thr = tn * WTHR;
    const double step = tn - w.t;
    w.t = tn;
    w.qh = w.qt = 0;
    w.changed = false;
    // completions (finish at tn, plus the path latency) and advance
    for (int s0 = 0; s0 < w.nSlots; s0 += 64) {
      const int at = s0 + lane;
      const int f = at < w.nSlots ? w.id[at] : -1;
      const bool due = f >= 0 && w.tau[at] <= thr;
      int a = 0, b = 0;
      int2 next = {0, 0};
      double fin = tn;
      if (due) {
        a = w.k0[at];
        b = w.k1[at];
        next = w.s2[at];
        if (P.lat) fin = tn + P.lat[f];
        P.finish[f] = fin;
        w.id[at] = -1;
      } else if (f >= 0) {
        const double moved = w.rate[at] * step;
        w.rem[at] = w.rem[at] - moved;
      }
      const uint64_t m = __ballot(due);
      if (m == 0) continue;
      if (due) w.freed[w.nFree + rank_in(m)] = (uint16_t)at;
      w.push(due && b > a, f, a, b, next, fin);
      w.nFree += (int)__popcll(m);
      w.changed = true;
    }
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
        wsync();
        const uint64_t m = __ballot(in && !due);
        if (in && !due) {
          const int i = keep + rank_in(m);
          w.prel[i] = rl;
          w.pid[i] = f;
        }
        keep += (int)__popcll(m);
        if (__ballot(due) != 0) {
          Own o{};
          if (due) o = own_of(P, f);
          w.arrive(due, f, rl, o);  // due: none waits on
        }
        wsync();
      }
      w.nPend = keep;
    }
    // dependants, to a fixpoint through zero-byte flows: every finished flow
    // raises its dependants' release base, then counts them down
    while (w.qh < w.qt) {
      wsync();
      const int cnt = min(64, w.qt - w.qh);
      w.successors(cnt, [&](bool in, int g, double fin) {
        if (in)
          __hip_atomic_fetch_max(reinterpret_cast<uint64_t*>(&P.base[g]),
                                 (uint64_t)__double_as_longlong(fin), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
      });
      // the raises are performed before a base is read
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
      __builtin_amdgcn_s_waitcnt(0);
      w.successors(cnt, [&](bool in, int g, double) {
        bool last = false;
        double rl = 0.0;
        Own o{};
        if (in) {
          const int c = __hip_atomic_fetch_add(&P.cnt[g], -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          o = own_of(P, g);
          const double st = P.start[g];
          const double base = __longlong_as_double((long long)__hip_atomic_load(
              reinterpret_cast<uint64_t*>(&P.base[g]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
          last = c == 1;
          rl = st + base;
          if (last) P.rel[g] = rl;
        }
        w.arrive(last, g, rl, o);
      });
      w.qh += cnt;
    }
    wsync();
    if (w.nSpill > 0 || w.pSpill > 0) {
      mid = w.changed ? 3 : 1;
      break;
    }
    if (w.nFree == w.nSlots) w.nFree = w.nSlots = 0;
    else if (w.nFree >= 64) w.compact();
    if (w.changed && w.nSlots > 0) {
      const int rc = w.nSlots <= 128 ? w.solve<2>() : w.solve<8>();
      solves += 1;
      if (rc != ST_DONE) {
        status = rc;
        break;
      }
    }
  }
  wsync();
  const int na = w.dump();
  const int64_t isw = wsum(w.isw);
  if (lane == 0) {
    C->started = 1;
    C->mid = mid;
    C->t = w.t;
    C->ab = 0;
    C->e = 0;
    C->nslots = na;
    C->npend = w.nPend + w.pSpill;
    C->holes = 0;
    C->events = events;
    C->launch_events = events - events0;
    C->solves = solves;
    C->rounds = w.rounds;
    C->flows_swept = w.fsw;
    C->incidences_swept = (resume ? C->incidences_swept : 0) + isw;
    C->links_swept = w.lsw;
    C->active_swept = asw;
    C->pending_swept = psw;
    C->status = status;
    if (mid) P.hlist[__hip_atomic_fetch_add(P.hcount, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)] = part;
  }
}

}  // namespace

__global__ __launch_bounds__(64) void netsim_xwave_kernel(Params P, const int32_t* list, int sc, int pc) {
  extern __shared__ __align__(16) unsigned char wpool[];
  xwave_loop(P, list[blockIdx.x], sc, pc, wpool);
}

size_t xwave_bytes(int nl, int sc, int pc) { return XWave::bytes(nl, sc, pc); }

hipError_t launch_xwave(const Params& p, const int32_t* list, int parts, int sc, int pc, size_t lds, hipStream_t s) {
  hipError_t e = hipFuncSetAttribute((const void*)netsim_xwave_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(netsim_xwave_kernel, dim3(parts), dim3(64), lds, s, p, list, sc, pc);
  return hipGetLastError();
}

}  // namespace netsim_dev
