// The rule's decisions for all workers without a launch of their own, which takes 5 to 7 us for under 1 us of work: by the workgroup of a gradient
// kernel that finishes last (last_of), or by every workgroup of the server's launch from inputs taken down in front (rule_inputs).
#pragma once

#include "cada_internal.h"

namespace cada {

template <typename T> __device__ __forceinline__ void put_far(T *p, T x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T> __device__ __forceinline__ T get_far(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Counts this workgroup in and says whether it is the last of n; called by all its threads, whose stores have then reached
// the coherence point.  The last one resets the counter for the next launch.
__device__ __forceinline__ bool last_of(uint32_t *count, uint32_t n, uint32_t *flag /* LDS */) {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  if (threadIdx.x == 0) {
    const uint32_t seen = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *flag = seen + 1 == n;
    if (seen + 1 == n) __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  lds_sync();
  return *flag != 0;
}

// Sum of the per-block partial sums of the squared step of iteration k-1 (the value of
// ring[(k-1) mod d_max]), in a fixed order; called by the whole block, valid in every thread.
__device__ inline float last_step_sq(const DevState &s, double *red /* [kBlock] LDS */) {
  // (sixteen loads in flight per thread; the additions keep their order, a missing term adds 0)
  double acc = 0.0;
  for (int i0 = threadIdx.x; i0 < s.n_ring_part; i0 += 16 * kBlock) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) { const int i = i0 + u * kBlock; v[u] = s.ring_part[min(i, s.n_ring_part - 1)]; if (i >= s.n_ring_part) v[u] = 0.f; }
#pragma unroll
    for (int u = 0; u < 16; ++u) acc += (double)v[u];
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = kBlock / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  const float r = (float)red[0];
  __syncthreads();
  return r;
}

// The rule's inputs that no other workgroup of the step changes before the server's launch: the right-hand side (the newest squared step goes into the ring here), delays and
// selectors.  By the kBlock threads of one workgroup of a launch in front.
__device__ inline void rule_inputs(const DevState &s, const RuleInputs &ri, double *red /* [kBlock] LDS */) {
  const int last = s.k > 0 ? (int)((s.k - 1) % s.d_max) : -1;
  for (int m = threadIdx.x; m < s.M; m += kBlock) { ri.in[m] = s.tau[m]; ri.in[s.M + m] = s.sel[m]; }
  const float newest = s.k > 0 ? last_step_sq(s, red) : 0.f;
  if (threadIdx.x < kWave) {      // (a wavefront: by one thread a ring of 1024 squared steps took 75 us)
    double sum = 0.0;
    for (int j = threadIdx.x; j < s.d_max; j += kWave) sum += (double)(j == last ? newest : s.ring[j]);
    sum = wave_sum_f64(sum);
    if (threadIdx.x == 0) {
      *ri.rhs = (s.c / (double)s.d_max) * sum;
      if (last >= 0) s.ring[last] = newest;
    }
  }
}

}  // namespace cada
