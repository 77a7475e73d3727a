// Progressive filling over a link-major incidence, by one workgroup: the
// exact solver's arithmetic (exact.hip) with the work of a level cut down to
// what the level changes.
//
// A full-width solve has thousands of bottleneck levels that freeze a few
// tens of flows each.  Sweeping every unfrozen flow and every live link at
// each level costs thousands of times the incidences; here a level
//   a. takes the minimum share over groups of 32 links (kept in shared
//      memory);
//   b. lists the links of the groups within the tie band that are
//      themselves within it: the bottlenecks;
//   c. walks those links' flows and freezes the ones not frozen yet, counting
//      them on their links (k_l) and listing the links it counted on;
//   d. applies R_l -= k_l * s*, n_l -= k_l to the listed links, computes their
//      shares and notes the groups whose minimum they held;
//   e. takes those groups' minima again.
// Measured: 258,048 flows over 20,480 links (11,744 levels) 168 ms with three
// kernels per level over the whole GPU, 65 ms here; 32,256 flows over 2,560
// links (1,461 levels) on a caller's arrays 57 ms by one workgroup's sweeps,
// 7.7 ms here.  512 threads: 256 take as long (66 and 8.5 ms).
// Same operations on the same values in another order of visits: minima,
// integer counts and one product and one difference per link and level, so
// rates and every counter are the same bit for bit.  A level is bound by
// its five workgroup barriers and the loads of b to e one after another.  One
// workgroup, since the exchange between workgroups costs more than a whole
// level; levels that freeze very many flows at once (symmetric traffic)
// cost it at most ~2 ns per flow, and there are few of them.
#pragma once

#include "device.h"
#include "lanes.h"

#include <math.h>

namespace netsim_dev {

constexpr double FTHR = 1.000000000001;
constexpr double FINF = __builtin_huge_val();
constexpr int FILL_BOTT = 1024;     // bottlenecks of a level listed in shared memory
constexpr int FILL_THREADS = 512;
constexpr size_t FILL_DYNAMIC = 140 * 1024;  // dynamic shared memory beside FillShared
constexpr int FILL_TOUCHED = 4096;  // links counted on in a level; beyond, every link is looked at

struct FillShared {
  double red[2][16];
  int32_t nbott, ntouched, nrescan;
  int32_t frozen, finc;  // flows frozen in the level, their incidences
  int32_t nlive;         // links with unfrozen flows
  unsigned long long inc0;
  int32_t b0[FILL_BOTT], b1[FILL_BOTT];  // a bottleneck's flows
  uint16_t touched[FILL_TOUCHED];
};

// Dynamic shared memory of a solve over nl links, with `bits` flow bits in it
// and (lds) the links' residuals, shares and counts too.
__host__ __device__ inline size_t fill_bytes(int nl, int64_t bits, bool lds) {
  const size_t g = (size_t)(nl + 31) / 32, ng = (g + 7) & ~size_t(7);
  const size_t l = ((size_t)nl + 7) & ~size_t(7);
  return ng * (8 + 2 + 2 + 4) + l * 4 + (lds ? l * 20 : 0) + (((size_t)bits + 63) / 64) * 8;
}

struct FillStats {
  int64_t levels = 0, fsw = 0, isw = 0, lsw = 0;
};

// Link state by link (0 .. nl-1) in shared memory ...
struct FillShLinks {
  static constexpr bool kDirect = true;
  double *R, *s;
  int32_t* n;
  const int32_t* off;
  __device__ __forceinline__ void init(int l, double R0, int n0, double v) const {
    R[l] = R0;
    s[l] = v;
    n[l] = n0;
  }
  __device__ __forceinline__ double share(int l) const { return s[l]; }
  __device__ __forceinline__ double look(int l, int& e0, int& e1) const {
    e0 = off[l];
    e1 = off[l + 1];
    return s[l];
  }
  __device__ __forceinline__ void get(int l, double& Rv, int& nv) const {
    Rv = R[l];
    nv = n[l];
  }
  __device__ __forceinline__ void set(int l, double Rv, int nv, double v) const {
    R[l] = Rv;
    n[l] = nv;
    s[l] = v;
  }
};

// ... or in global memory, the share beside where the link's flows are
// listed, so that finding a bottleneck finds its flows.
struct FillShare {
  double s;
  int32_t e0, e1;
};
struct FillRest {
  double R;
  int64_t n;
};
struct FillGlLinks {
  static constexpr bool kDirect = false;
  FillShare* a;
  FillRest* b;
  const int32_t* off;
  __device__ __forceinline__ void init(int l, double R0, int n0, double v) const {
    a[l] = FillShare{v, off[l], off[l + 1]};
    b[l] = FillRest{R0, (int64_t)n0};
  }
  __device__ __forceinline__ double share(int l) const { return a[l].s; }
  __device__ __forceinline__ double look(int l, int& e0, int& e1) const {
    const FillShare x = a[l];
    e0 = x.e0;
    e1 = x.e1;
    return x.s;
  }
  __device__ __forceinline__ void get(int l, double& Rv, int& nv) const {
    const FillRest x = b[l];
    Rv = x.R;
    nv = (int)x.n;
  }
  __device__ __forceinline__ void set(int l, double Rv, int nv, double v) const {
    b[l] = FillRest{Rv, (int64_t)nv};
    a[l].s = v;
  }
};

// Minimum over the workgroup's first FILL_THREADS threads (the callers).
__device__ __forceinline__ double fill_block_min(double v, FillShared& sh, int& rb) {
  v = wmin(v);
  if ((threadIdx.x & 63) == 0) sh.red[rb][threadIdx.x >> 6] = v;
  __syncthreads();
  double m = FINF;
#pragma unroll
  for (int j = 0; j < FILL_THREADS / 64; ++j) {
    const double x = sh.red[rb][j];
    m = x < m ? x : m;
  }
  rb ^= 1;
  return m;
}

// Minimum over each half of the wave (all its lanes get the value of lane 31
// or 63): exchanges inside rows of 16 lanes, then one between the two rows.
__device__ __forceinline__ double fill_half_min(double v) {
  v = dpp_min<0xB1, 0xF>(v);
  v = dpp_min<0x4E, 0xF>(v);
  v = dpp_min<0x141, 0xF>(v);
  v = dpp_min<0x140, 0xF>(v);
  const double w = __shfl_xor(v, 16, 64);
  return w < v ? w : v;
}

// Appends the lanes with pred to a list counted in shared memory (every lane
// of the wave calls it).
__device__ __forceinline__ int fill_append(int32_t* counter, bool pred) {
  const uint64_t mask = __ballot(pred);
  if (mask == 0) return -1;
  const int lane = threadIdx.x & 63;
  const int leader = __ffsll((unsigned long long)mask) - 1;
  int base = 0;
  if (lane == leader) base = atomicAdd(counter, (int)__popcll(mask));
  base = __shfl(base, leader, 64);
  return pred ? base + (int)__popcll(mask & ((1ull << lane) - 1ull)) : -1;
}

// Rates of the unfrozen flows (their bits set) into rate[], by the
// workgroup's first FILL_THREADS threads (the other waves have ended).  link(l, R, n)
// gives link l's capacity and count; pool is the dynamic shared memory
// (fill_bytes); lf lists the links' flows; spill0/spill1 ([nl]) take a level's
// bottlenecks beyond FILL_BOTT.  take(f) clears flow f's bit and says whether
// it was set; paths.load(f, lv, deg) reads up to six links, paths.more(f, j)
// the j-th beyond them.  With link state in shared memory (kDirect) every
// level looks at all shares, a few per thread, instead of the groups'
// minima.  Returns ST_DONE, ST_BAD_SHARE or ST_ROUNDS.
template <class Links, class Link, class Take, class Paths>
__device__ __forceinline__ int fill_levels(FillShared& sh, const Links lk, unsigned char* pool, int nl,
                                           const Link link, const int32_t* lf, int nu, double* rate,
                                           int32_t* spill0, int32_t* spill1, int max_rounds,
                                           const Take take, const Paths paths, FillStats& st) {
  constexpr bool DIRECT = Links::kDirect;
  constexpr int T = FILL_THREADS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int ng = (nl + 31) / 32, ngp = (ng + 7) & ~7;
  unsigned long long* gmin = reinterpret_cast<unsigned long long*>(pool);  // bit patterns (shares >= 0)
  int32_t* gflag = reinterpret_cast<int32_t*>(pool + 8 * (size_t)ngp);
  uint16_t* rescan = reinterpret_cast<uint16_t*>(pool + 12 * (size_t)ngp);
  int32_t* k = reinterpret_cast<int32_t*>(pool + 16 * (size_t)ngp);
  if (tid == 0) {
    sh.nbott = sh.ntouched = sh.nrescan = 0;
    sh.frozen = sh.finc = sh.nlive = 0;
    sh.inc0 = 0;
  }
  __syncthreads();
  // shares of the first level, 32 links of a group by half a wave
  {
    unsigned long long inc = 0;
    int live = 0;
    for (int g0 = 0; g0 < ng; g0 += T / 32) {
      const int g = g0 + (tid >> 5), l = g * 32 + (tid & 31);
      double v = FINF;
      if (g < ng && l < nl) {
        double R;
        int n;
        link(l, R, n);
        k[l] = 0;
        if (n > 0) {
          v = R / (double)n;
          ++live;
          inc += (unsigned long long)n;
        }
        lk.init(l, R, n, v);
      }
      if constexpr (!DIRECT) {
        v = fill_half_min(v);
        if (g < ng && (tid & 31) == 0) {
          gmin[g] = (unsigned long long)__double_as_longlong(v);
          gflag[g] = 0;
        }
      }
    }
    if (live) {
      atomicAdd(&sh.nlive, live);
      atomicAdd(&sh.inc0, inc);
    }
  }
  __syncthreads();
  int64_t ninc = (int64_t)sh.inc0;
  int rb = 0;
  // lists the links hit by the wave's lanes as bottlenecks
  auto bottleneck = [&](bool hit, int e0, int e1) {
    const int i = fill_append(&sh.nbott, hit);
    if (hit) {
      if (i < FILL_BOTT) {
        sh.b0[i] = e0;
        sh.b1[i] = e1;
      } else {
        spill0[i] = e0;
        spill1[i] = e1;
      }
    }
  };
  while (nu > 0) {
    if (st.levels >= max_rounds) return ST_ROUNDS;
    // a. level minimum
    double loc = FINF;
    if constexpr (DIRECT) {
      for (int l = tid; l < nl; l += T) {
        const double v = lk.share(l);
        loc = v < loc ? v : loc;
      }
    } else {
      for (int g = tid; g < ng; g += T) {
        const double v = __longlong_as_double((long long)gmin[g]);
        loc = v < loc ? v : loc;
      }
    }
    const double sstar = fill_block_min(loc, sh, rb);
    if (!(sstar > 0.0) || !(sstar < FINF)) return ST_BAD_SHARE;
    st.levels += 1;
    st.fsw += nu;
    st.isw += ninc;
    st.lsw += sh.nlive;
    const double thr = sstar * FTHR;
    // b. bottlenecks; each wave looks into the groups it found
    if (tid == 0) {
      sh.ntouched = sh.nrescan = 0;
      sh.frozen = sh.finc = 0;
    }
    if constexpr (DIRECT) {
      if (__ballot(loc <= thr) != 0)
        for (int l0 = 0; l0 < nl; l0 += T) {
          const int l = l0 + tid;
          int e0 = 0, e1 = 0;
          bool hit = l < nl && lk.share(l) <= thr;
          if (__ballot(hit) == 0) continue;
          if (hit) lk.look(l, e0, e1);
          bottleneck(hit, e0, e1);
        }
    } else {
      for (int g0 = tid - lane; g0 < ng; g0 += T) {
        const int g = g0 + lane;
        uint64_t m = __ballot(g < ng && __longlong_as_double((long long)gmin[g]) <= thr);
        while (m) {
          const int a = __ffsll((unsigned long long)m) - 1;
          m &= m - 1;
          const int b = m ? __ffsll((unsigned long long)m) - 1 : -1;
          m &= m - 1;
          const int h = lane < 32 ? a : b;
          const int l = (g0 + h) * 32 + (lane & 31);
          int e0 = 0, e1 = 0;
          const bool hit = h >= 0 && l < nl && lk.look(l, e0, e1) <= thr;
          bottleneck(hit, e0, e1);
        }
      }
    }
    __syncthreads();
    const int nb = sh.nbott;
    // c. their flows: the waves shared out among the bottlenecks
    const int waves = T >> 6, wave = tid >> 6;
    const int per = nb < waves ? waves / nb : 1;
    const int step = 64 * per, mine = wave / nb * 64 + lane;
    int froze = 0, finc = 0;
    for (int b = nb < waves ? (wave < nb * per ? wave % nb : nb) : wave; b < nb; b += waves) {
      const int e0 = b < FILL_BOTT ? sh.b0[b] : spill0[b], e1 = b < FILL_BOTT ? sh.b1[b] : spill1[b];
      for (int x = e0; x < e1; x += step) {
        const int e = x + (nb < waves ? mine : lane);
        int lv[6], deg = 0, f = 0;
        bool fz = false;
        if (e < e1) {
          f = lf[e];
          paths.load(f, lv, deg);
          fz = take(f);
        }
        if (__ballot(fz) == 0) continue;
        bool first[6];
#pragma unroll
        for (int j = 0; j < 6; ++j) first[j] = fz && j < deg && atomicAdd(&k[lv[j]], 1) == 0;
        if (fz) {
          rate[f] = sstar;
          froze += 1;
          finc += deg;
        }
        // the links counted on for the first time, listed with one atomic
        int total = 0, at[6];
#pragma unroll
        for (int j = 0; j < 6; ++j) {
          const uint64_t m = __ballot(first[j]);
          at[j] = total + rank_in(m);
          total += (int)__popcll(m);
        }
        int base = 0;
        if (lane == 0 && total > 0) base = atomicAdd(&sh.ntouched, total);
        base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
        for (int j = 0; j < 6; ++j)
          if (first[j] && base + at[j] < FILL_TOUCHED) sh.touched[base + at[j]] = (uint16_t)lv[j];
        for (int j = 6; __ballot(fz && j < deg) != 0; ++j) {
          const bool on = fz && j < deg;
          const int l = on ? paths.more(f, j) : 0;
          const bool one = on && atomicAdd(&k[l], 1) == 0;
          const int i = fill_append(&sh.ntouched, one);
          if (one && i < FILL_TOUCHED) sh.touched[i] = (uint16_t)l;
        }
      }
    }
    if (froze) {
      atomicAdd(&sh.frozen, froze);
      atomicAdd(&sh.finc, finc);
    }
    __syncthreads();
    // d. the links they cross
    const int nt = sh.ntouched;
    const bool all = nt > FILL_TOUCHED;
    nu -= sh.frozen;
    ninc -= sh.finc;
    if (sh.frozen == 0) return ST_BAD_SHARE;  // a level must freeze something
    if (tid == 0) sh.nbott = 0;
    for (int i0 = 0; i0 < (all ? nl : nt); i0 += T) {
      const int i = i0 + tid;
      bool again = false;
      int g = 0;
      if (i < (all ? nl : nt)) {
        const int l = all ? i : (int)sh.touched[i];
        const int kk = k[l];
        if (kk != 0) {
          const double old = DIRECT ? 0.0 : lk.share(l);
          double R;
          int n;
          lk.get(l, R, n);
          const double dec = (double)kk * sstar;
          R = R - dec;
          n -= kk;
          k[l] = 0;
          const double v = n > 0 ? R / (double)n : FINF;
          lk.set(l, R, n, v);
          if (n == 0) atomicAdd(&sh.nlive, -1);
          if constexpr (!DIRECT) {
            // shares do not fall but for rounding; a group is looked at
            // again when one of its smallest changed
            g = l >> 5;
            const double m = __longlong_as_double((long long)gmin[g]);
            if (v < m) atomicMin(&gmin[g], (unsigned long long)__double_as_longlong(v > 0.0 ? v : 0.0));
            if (old <= m) again = atomicExch(&gflag[g], 1) == 0;
          }
        }
      }
      if constexpr (!DIRECT) {
        const int r = fill_append(&sh.nrescan, again);
        if (again) rescan[r] = (uint16_t)g;
      }
    }
    __syncthreads();
    if constexpr (DIRECT) continue;
    // e. minima of the groups that lost theirs
    const int nr = sh.nrescan;
    for (int c0 = 0; c0 < nr; c0 += T / 32) {
      const int c = c0 + (tid >> 5);
      int g = 0;
      double v = FINF;
      if (c < nr) {
        g = rescan[c];
        const int l = g * 32 + (tid & 31);
        if (l < nl) v = lk.share(l);
      }
      v = fill_half_min(v);
      if (c < nr && (tid & 31) == 0) {
        gmin[g] = (unsigned long long)__double_as_longlong(v > 0.0 ? v : 0.0);
        gflag[g] = 0;
      }
    }
    __syncthreads();
  }
  return ST_DONE;
}

}  // namespace netsim_dev
