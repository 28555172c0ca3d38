// The rule's decisions for all workers without a launch of their own, which costs about 5 us for under 1 us of work: by the workgroup of a gradient
// kernel that finishes last (rule_all), or by every workgroup of the server's launch from inputs taken down in front (rule_inputs).
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
  if (threadIdx.x == 0) {
    double sum = 0.0;
    for (int j = 0; j < s.d_max; ++j) sum += (double)(j == last ? newest : s.ring[j]);
    *ri.rhs = (s.c / (double)s.d_max) * sum;
    if (last >= 0) s.ring[last] = newest;
  }
}

// S3 of the step, by the NT threads of one workgroup: right-hand side, left-hand sides from their partial sums (written
// before by put_far, or by an earlier launch), decisions, tau, pointer swap, trace.  Sums are in double and in a fixed order: a
// wavefront takes four workers at a time (sixteen loads in flight), then a thread decides for one worker.
// lds: rule_lds(NT) bytes.
constexpr int rule_lds(int nt) { return (nt + nt / kWave + 1) * (int)sizeof(double); }
template <int NT>
__device__ __forceinline__ void rule_all(const DevState &s, const uint8_t *replay, void *lds) {
  constexpr int NW = NT / kWave;
  double *lhs_s = static_cast<double *>(lds), *red = lhs_s + NT;
  uint32_t *cnt = reinterpret_cast<uint32_t *>(red + NW);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t k = s.k;
  const int last = k > 0 ? (int)((k - 1) % s.d_max) : -1;
  // squared step of the iteration before: the sum of its blocks' parts
  double acc = 0.0;
  if (k > 0)
    for (int i0 = tid; i0 < s.n_ring_part; i0 += 16 * NT) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) { const int i = i0 + u * NT; v[u] = s.ring_part[min(i, s.n_ring_part - 1)]; if (i >= s.n_ring_part) v[u] = 0.f; }
#pragma unroll
      for (int u = 0; u < 16; ++u) acc += (double)v[u];
    }
  acc = wave_sum_f64(acc);
  if (lane == 0) red[w] = acc;
  if (tid == 0) *cnt = 0u;
  double rhs = 0.0;
  float newest = 0.f;
  const bool tr = k < s.trace_steps;
  for (int mb = 0; mb < s.M; mb += NT) {
    const int mine = mb + tid, mend = min(mb + NT, s.M);
    int32_t tau = 0, sel = 0;
    bool forced = false, up = false;
    if (mine < s.M) {                                  // (asked for before the left-hand sides' parts)
      tau = s.tau[mine]; sel = s.sel[mine];
      if (replay != nullptr) { const uint8_t r = replay[mine]; forced = r != CADA_REPLAY_FREE; up = r != 0; }
    }
    for (int m0 = mb + 4 * w; m0 < mend; m0 += 4 * NW) {
      double l[4] = {0.0, 0.0, 0.0, 0.0};
      for (int t0 = lane; t0 < s.n_lhs_part; t0 += 4 * kWave) {
        float v[4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int t = t0 + u * kWave;
            v[q][u] = get_far(s.lhs_part + (int64_t)min(m0 + q, s.M - 1) * s.n_lhs_part + min(t, s.n_lhs_part - 1));
            if (t >= s.n_lhs_part) v[q][u] = 0.f;
          }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int u = 0; u < 4; ++u) l[q] += (double)v[q][u];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        l[q] = wave_sum_f64(l[q]);
        if (lane == 0 && m0 + q < mend) lhs_s[m0 + q - mb] = l[q];
      }
    }
    lds_sync();
    if (mb == 0) {
      double sum = 0.0;
#pragma unroll
      for (int i = 0; i < NW; ++i) sum += red[i];
      newest = (float)sum;
      sum = 0.0;
      for (int j = lane; j < s.d_max; j += kWave) sum += (double)(j == last ? newest : s.ring[j]);
      rhs = (s.c / (double)s.d_max) * wave_sum_f64(sum);
    }
    uint32_t ups = 0;
    if (mine < s.M) {
      const double lhs = lhs_s[tid];
      const bool own = (s.rule == CADA_RULE_ALWAYS) || (lhs > rhs) || (tau >= s.D);
      if (!forced) up = own;
      if (tr) {
        const int64_t o = k * s.M + mine;
        s.t_mask[o] = up ? 1 : 0;
        s.t_own[o] = own ? 1 : 0;
        s.t_lhs[o] = (float)lhs;
        s.t_tau[o] = tau;
      }
      s.lhs[mine] = (float)lhs;
      s.mask[mine] = up ? 1 : 0;
      s.tau[mine] = up ? 1 : tau + 1;
      if (up) {
        s.sel[mine] = sel ^ 1;       // the fresh row becomes the stored one
        ups = 1;
      } else if (s.rule == CADA_RULE_CADA2 && tau >= s.D) {
        // (only a replay mask can do this: the reference point theta^{k+1-(tau+1)} leaves the D+1 retained iterates)
        atomicOr(s.err, 8u);
      }
    }
    const unsigned long long votes = __ballot(ups != 0);
    if (lane == 0 && votes) atomicAdd(cnt, (uint32_t)__popcll(votes));
    lds_sync();
  }
  if (tid == 0) {
    const uint32_t n = *cnt;
    atomicAdd(reinterpret_cast<unsigned long long *>(s.uploads), (unsigned long long)n);
    s.n_up[k & 1] = n;
    if (last >= 0) s.ring[last] = newest;
    if (tr) s.t_rhs[k] = (float)rhs;
  }
}

}  // namespace cada
