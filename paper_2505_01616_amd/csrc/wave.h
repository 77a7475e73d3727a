// What the kernels that run a part in one wavefront share (wave.hip: the
// default solver, xwave.hip: exact mode).
#pragma once

#include "device.h"
#include "lanes.h"

#include <math.h>

#pragma clang fp contract(off)

namespace netsim_dev {

namespace {

constexpr double WTHR = 1.000000000001;
constexpr double WINF = __builtin_huge_val();

// Orders this wave's shared-memory accesses for the compiler; the hardware
// performs a wave's LDS operations in order.
__device__ __forceinline__ void wsync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ int64_t wsum(int64_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

template <class T>
__device__ __forceinline__ void ladd(T* p, T v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Finished flows whose successors are still to be counted down: a log of
// flow ids in global memory (a flow finishes once, so it never overflows) and
// the newest WQ entries with their successor range in shared memory.
constexpr int WQ = 64;
struct Done {
  int32_t k0, k1;
  int2 s;  // the first two of them
  double fin;
};
// Shared memory of the log: the entries and a list of successors.
constexpr int WLOG = WQ * (int)sizeof(Done) + 64 * (int)sizeof(int2);

// A flow's own data, read when it is released (its first two successors with
// it: when it ends, and at once for a zero-byte flow, they are counted down
// without a read of the successor list first).
struct Own {
  double nb;
  uint4 rec;
  int k0, k1, comp;
  int2 s;
};

__device__ __forceinline__ Own own_of(const Params& P, int f) {
  Own o;
  o.nb = P.nbytes[f];
  o.rec = P.path16[f];
  o.k0 = P.soff[f];
  o.k1 = P.soff[f + 1];
  o.comp = P.comp[f];
  o.s = P.succ2[f];
  return o;
}

// Unpacks a path record of at most D links into part-local link ids; an absent
// link becomes the sentinel entry nl (share +inf, never stamped).  Returns the
// degree.
template <int D = 6>
__device__ __forceinline__ int unpack(const uint4 rec, int nl, int* lv) {
  const uint32_t w[3] = {rec.x, rec.y, rec.z};
  int deg = 0;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const int u = (int)((w[k >> 1] >> (16 * (k & 1))) & 0xFFFFu);
    deg += u != 0xFFFF;
    lv[k] = min(u, nl);
  }
  return deg;
}

// The log of one event's finished flows.
struct WaveLog {
  const Params& P;
  const int lane, f0;
  Done* ring;       // [WQ], shared memory
  int2* next;       // [64], shared memory: successors and the lanes they belong to
  int qh = 0, qt = 0;  // entries handled, entries

  __device__ __forceinline__ WaveLog(const Params& P_, int first) : P(P_), lane((int)threadIdx.x), f0(first) {}

  // A finished flow joins the log (all lanes call it).
  __device__ __forceinline__ void push(bool p, int f, int a, int b, int2 s, double fin) {
    const uint64_t m = __ballot(p);
    if (m == 0) return;
    if (p) {
      const int q = qt + rank_in(m);
      ring[q & (WQ - 1)] = Done{a, b, s, fin};
      P.comp0[f0 + q] = f;
    }
    qt += (int)__popcll(m);
  }

  // body(in, g, fin) for every successor g of the logged flows
  // [qh, qh + cnt), 64 at a time: a body is a round trip to global memory
  // (about a microsecond with what follows it), so ranges of up to 8 are laid
  // end to end over the lanes; longer ones take the whole wave one by one.
  // (The n-th successors of all flows at a time, each read from the list
  // first: trace of 128 GPUs 111 ms against 106, with latencies and the
  // rollback history 28 against 24.5.)
  template <class Body>
  __device__ __forceinline__ void successors(int cnt, Body body) {
    int a = 0, b = 0;
    int2 s = {0, 0};
    double fin = 0.0;
    if (lane < cnt) {
      const int q = qh + lane;
      if (qt - q <= WQ) {
        const Done d = ring[q & (WQ - 1)];
        a = d.k0;
        b = d.k1;
        s = d.s;
        fin = d.fin;
      } else {
        const int f = P.comp0[f0 + q];
        a = P.soff[f];
        b = P.soff[f + 1];
        s = P.succ2[f];
        fin = P.finish[f];  // (the flow's event stored it before it logged the flow)
      }
    }
    const uint64_t wide = __ballot(b - a > 8);
    const int c = b - a > 8 ? 0 : b - a;
    if (__ballot(c > 1) == 0) {
      if (__ballot(c == 1) != 0) body(c == 1, s.x, fin);
    } else {
      int off = 0, total = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint64_t m = __ballot((c >> k) & 1);
        off += rank_in(m) << k;
        total += (int)__popcll(m) << k;
      }
      for (int i0 = 0; i0 < total; i0 += 64) {
        wsync();
        for (int j = 0; __ballot(j < c) != 0; ++j) {
          const int i = off + j - i0;
          if (j < c && i >= 0 && i < 64) next[i] = make_int2(j == 0 ? s.x : j == 1 ? s.y : ~(a + j), lane);
        }
        wsync();
        const bool in = i0 + lane < total;
        int2 v = {0, 0};
        if (in) {
          v = next[lane];
          if (v.x < 0) v.x = P.succ[~v.x];
        }
        body(in, v.x, __shfl(fin, v.y, 64));
      }
    }
    for (uint64_t m = wide; m != 0; m &= m - 1) {
      const int j = __ffsll((unsigned long long)m) - 1;
      const int z = __shfl(b, j, 64);
      const double fj = __shfl(fin, j, 64);
      for (int k = __shfl(a, j, 64); k < z; k += 64) body(k + lane < z, k + lane < z ? P.succ[k + lane] : 0, fj);
    }
  }
};

}  // namespace

}  // namespace netsim_dev
