// Before and after a run: the dynamic state set back to t = 0, and the
// results gathered into one block that a single copy brings to the host.
//
// Both are bound by bytes: a run of 715,776 flows in 33,029 parts moved 30 MB
// from pageable host memory (initial state, 14 MB of it control blocks) and
// 20 MB back, and permuted and reduced them on one host thread: about 6 ms
// around 2.8 ms of simulation.  The initial state stays on the device, and
// what the host needs (totals, one value per scenario and part, the finish
// times in id order) is 6.0 MB in one copy to pinned memory.  That run's wall
// time went from 9.1 to 3.5 ms, that of a 3D-parallel step on 128
// GPUs from 2.29 to 2.04 ms, and a single rate solve of 258,048 flows (counts
// and rates no longer made on the host) from 4.1 to 3.2 ms.
#include "device.h"

#include <math.h>

namespace netsim_dev {

namespace {

__device__ __forceinline__ int64_t sum_wave(int64_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ uint64_t max_wave(uint64_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t w = __shfl_xor(v, o, 64);
    v = w > v ? w : v;
  }
  return v;
}

}  // namespace

__global__ __launch_bounds__(256) void reset_state_kernel(Params P, Initial I, int64_t F, int64_t L, int64_t ctl_words,
                                                          bool first) {
  const int64_t n = (int64_t)gridDim.x * blockDim.x, i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const double nan = __longlong_as_double(0x7FF8000000000000ll);
  for (int64_t i = i0; i < F; i += n) {
    P.cnt[i] = I.cnt[i];
    P.rel[i] = I.rel[i];
    P.pend0[i] = I.pend[i];
    P.finish[i] = nan;
    P.base[i] = 0.0;
    P.rate[i] = 0.0;
  }
  if (first)  // a handle's first reset: the first two successors of every flow, at its own index
    for (int64_t i = i0; i < F; i += n) {
      const int a = P.soff[i], b = P.soff[i + 1];
      P.succ2[i] = make_int2(a < b ? P.succ[a] : 0, a + 1 < b ? P.succ[a + 1] : 0);
    }
  if (P.hist)
    for (int64_t i = i0; i < F; i += n) {
      P.evr[i] = EV_NEVER;
      P.eva[i] = EV_NEVER;
      P.evd[i] = EV_NEVER;
    }
  for (int64_t l = i0; l < L; l += n) P.nact[l] = 0;
  const uint64_t* src = reinterpret_cast<const uint64_t*>(I.ctl);
  uint64_t* dst = reinterpret_cast<uint64_t*>(P.ctl);
  static_assert(sizeof(ScenCtl) % 8 == 0, "control blocks are copied by words");
  for (int64_t i = i0; i < ctl_words; i += n) dst[i] = src[i];
}

// Releases of the flows [f0, f1) that no predecessor holds back, from their
// present starts (after a rollback to a checkpoint: a flow still pending there
// may have got another start since; the others get the value they had).
__global__ __launch_bounds__(256) void releases_kernel(Params P, int f0, int f1) {
  const int f = f0 + (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (f < f1 && P.cnt[f] == 0) P.rel[f] = P.start[f] + P.base[f];
}

// Synchronisation words, reduction slots and totals of a launch.
__global__ __launch_bounds__(256) void reset_launch_kernel(Params P, Results R, int num_scen_out) {
  const int n = gridDim.x * blockDim.x, i0 = blockIdx.x * blockDim.x + threadIdx.x;
  for (int i = i0; i < BAR_WORDS; i += n) P.bar[i] = 0u;
  for (int i = i0; i < 8; i += n) P.slots[i] = 0x7FF0000000000000ull;
  uint64_t* t = reinterpret_cast<uint64_t*>(R.totals);
  for (int i = i0; i < (int)(sizeof(RunTotals) / 8); i += n) t[i] = 0;
  for (int i = i0; i < num_scen_out; i += n) R.makespan[i] = 0;
}

// Statistics summed over the parts, one thread per part.
__global__ __launch_bounds__(256) void totals_kernel(Params P, Results R) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  const bool in = p < P.num_scen;
  int64_t v[RunTotals::kCounts] = {};
  uint64_t t = 0;
  bool stopped = false, fault = false;
  if (in) {
    const ScenCtl& c = P.ctl[p];
    v[0] = c.events;
    v[1] = c.solves;
    v[2] = c.rounds;
    v[3] = c.flows_swept;
    v[4] = c.incidences_swept;
    v[5] = c.active_swept;
    v[6] = c.pending_swept;
    v[7] = c.reselected;
    v[8] = c.wide_solves;
    v[9] = c.assisted;
    v[10] = c.links_swept;
    v[11] = c.launch_events;
    if (c.t > 0.0) t = (uint64_t)__double_as_longlong(c.t);  // positive doubles order like their bits
    stopped = c.status != 0;
    fault = c.status < 0;
    R.part_t[p] = c.started ? c.t : -__builtin_huge_val();
  }
  const bool first = (threadIdx.x & 63) == 0;
#pragma unroll
  for (int k = 0; k < RunTotals::kCounts; ++k) {
    const int64_t s = sum_wave(v[k]);
    if (first && s != 0) atomicAdd((unsigned long long*)&R.totals->count[k], (unsigned long long)s);
  }
  t = max_wave(t);
  if (first) atomicMax((unsigned long long*)&R.totals->t, (unsigned long long)t);
  const int ns = (int)__popcll(__ballot(stopped)), nf = (int)__popcll(__ballot(fault));
  if (first && ns) atomicAdd((unsigned long long*)&R.totals->stopped, (unsigned long long)ns);
  if (first && nf) atomicAdd((unsigned long long*)&R.totals->faults, (unsigned long long)nf);
  for (int k = 0; k < 8; ++k) {
    const int64_t s = sum_wave(in ? P.ctl[p].ticks[k] : 0);
    if (first && s != 0) atomicAdd((unsigned long long*)&R.totals->ticks[k], (unsigned long long)s);
  }
}

// Finish times in id order, the largest of each scenario and the number of
// flows that have one; 2048 flows per workgroup, whose largest goes to its
// scenario with one atomic when all of them belong to one.
__global__ __launch_bounds__(256) void finish_kernel(Params P, Results R, const int32_t* dev_of, const int32_t* scen_of,
                                                     int64_t F) {
  __shared__ uint64_t wmax[4];
  __shared__ int32_t wdone[4];
  const int64_t i0 = (int64_t)blockIdx.x * 2048, i1 = min(i0 + 2048, F);
  const int32_t s0 = scen_of ? scen_of[i0] : 0;
  uint64_t m = 0;
  int done = 0;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
    const double v = P.finish[dev_of[i]];
    R.finish[i] = v;
    const int32_t s = scen_of ? scen_of[i] : 0;
    if (v == v) {  // finished
      const uint64_t b = v > 0.0 ? (uint64_t)__double_as_longlong(v) : 0;
      ++done;
      if (s == s0) {
        m = b > m ? b : m;
      } else {
        atomicMax((unsigned long long*)&R.makespan[s], (unsigned long long)b);
      }
    }
  }
  m = max_wave(m);
  done = (int)sum_wave(done);
  if ((threadIdx.x & 63) == 0) {
    wmax[threadIdx.x >> 6] = m;
    wdone[threadIdx.x >> 6] = done;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      m = wmax[w] > m ? wmax[w] : m;
      done += wdone[w];
    }
    if (m) atomicMax((unsigned long long*)&R.makespan[s0], (unsigned long long)m);
    if (done) atomicAdd((unsigned long long*)&R.totals->completed, (unsigned long long)done);
  }
}

// Active flows on each link (the solve without an event loop), over the n
// listed flows; out[i] = rate of flow list[i].
__global__ __launch_bounds__(256) void count_active_kernel(Params P, const int32_t* list, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int f = list[i];
    for (int e = P.poff[f]; e < P.poff[f + 1]; ++e) atomicAdd(&P.nact[P.plink[e]], 1);
  }
}
__global__ __launch_bounds__(256) void gather_rates_kernel(Params P, const int32_t* list, int n, double* out) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) out[i] = P.rate[list[i]];
}

hipError_t launch_reset(const Params& P, const Initial& I, int64_t F, int64_t L, int NP, bool first, hipStream_t s) {
  const int64_t words = (int64_t)NP * (int64_t)(sizeof(ScenCtl) / 8);
  const int64_t most = F > words ? F : words;
  const int blocks = (int)((most + 1023) / 1024 < 1 ? 1 : (most + 1023) / 1024 > 2048 ? 2048 : (most + 1023) / 1024);
  hipLaunchKernelGGL(reset_state_kernel, dim3(blocks), dim3(256), 0, s, P, I, F, L, words, first);
  return hipGetLastError();
}

hipError_t launch_releases(const Params& P, int f0, int f1, hipStream_t s) {
  if (f1 <= f0) return hipSuccess;
  hipLaunchKernelGGL(releases_kernel, dim3((unsigned)((f1 - f0 + 255) / 256)), dim3(256), 0, s, P, f0, f1);
  return hipGetLastError();
}

hipError_t launch_reset_words(const Params& P, const Results& R, int scenarios, hipStream_t s) {
  hipLaunchKernelGGL(reset_launch_kernel, dim3(64), dim3(256), 0, s, P, R, scenarios);
  return hipGetLastError();
}

hipError_t launch_results(const Params& P, const Results& R, const int32_t* dev_of, const int32_t* scen_of, int64_t F,
                          hipStream_t s) {
  hipLaunchKernelGGL(totals_kernel, dim3((P.num_scen + 255) / 256), dim3(256), 0, s, P, R);
  hipLaunchKernelGGL(finish_kernel, dim3((unsigned)((F + 2047) / 2048)), dim3(256), 0, s, P, R, dev_of, scen_of, F);
  return hipGetLastError();
}

hipError_t launch_count_active(const Params& P, const int32_t* list, int n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(count_active_kernel, dim3(n < 1024 * 256 ? (n + 255) / 256 : 1024), dim3(256), 0, s, P, list, n);
  return hipGetLastError();
}

hipError_t launch_gather_rates(const Params& P, const int32_t* list, int n, double* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(gather_rates_kernel, dim3(n < 1024 * 256 ? (n + 255) / 256 : 1024), dim3(256), 0, s, P, list, n,
                     out);
  return hipGetLastError();
}

}  // namespace netsim_dev
