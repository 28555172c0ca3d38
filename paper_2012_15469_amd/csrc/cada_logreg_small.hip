// Whole iterations of Algorithm 1 in one kernel launch, with the rows in LDS: for minibatches that the registers of cada_logreg_steps.hip do not hold (more than 1024 columns or fewer than 4,
// more than 64 rows, or 32 of more than 512 columns); the host side serves both, and asks for both that the rows would fit LDS.  Logistic workloads so small that a
// step is bound by launch and dependency latency rather than by memory (tens of workers, a few
// hundred coordinates): four dependent launches per step cost 20-40 us, the arithmetic well
// under one.  One workgroup per worker:
//   phase A (workgroup m = worker m): both minibatch gradients in the difference form of
//     cada_logreg.hip, the rule's left-hand side, the right-hand side from the ring, the
//     decision, tau, the stored/fresh pointer swap, the trace           [S1-S4 of the step]
//   -- barrier --
//   phase B (EVERY workgroup, all coordinates): aggregate of the stored gradients, the server
//     update, the squared step                                          [S5-S7]
// Launches of several steps (k_small, launched cooperatively, ONE grid-wide barrier per iteration): every workgroup
// keeps the server's vectors (iterate, moments, snapshot) in its LDS and applies the same update
// to them, in the same order, so all copies stay bit for bit equal and the next phase A needs neither a second
// barrier nor the iterate from memory; workgroup (j / 256) mod M writes coordinate j's results to memory for
// the world outside.  What a fast workgroup writes in phase A of step k + 1 while a slow one is still in phase B of
// step k never is what the slow one reads: the fresh gradient goes to the row that is not the stored one, and
// the decisions of step k are published in slot k mod 2 of an array of their own.
// The barrier is that array.  Workgroup m publishes the word {tag of the step, its worker's buffer selector after the
// decision} in slot (step parity, m); a workgroup has passed the barrier when the first wavefront, one lane per worker,
// has seen this step's tag in every word -- and then it holds every decision, which a counter plus a separate array cost
// a memory round trip more.  (Two slots per worker: a workgroup can be one step ahead of another at most, so the word
// that a slow workgroup still waits for is not overwritten.  A tag is never 0, the value of a fresh workspace.)
// Every wait is bounded: one that exceeds the bound sets bit 1 of the error flags and the workgroup stops waiting.
//
// A launch of one step (k_small_one, cada_step): nothing has to wait for another workgroup.  The one that finishes
// phase A last (a counter in the workspace that also collects the decisions) runs phase B alone, with the same
// operations in the same order, so a step ends bit for bit where it ends inside a longer launch.  Without a
// wait among workgroups the launch needs no cooperative dispatch, whose queue hand-over costs more than the step.
//
// What bounds a step is a chain of dependent trips: rows in LDS -> products -> residuals -> gradient -> its stores
// acknowledged -> word published -> words polled -> M rows of gradients -> update.  The kernel is built to shorten it:
//   - eight wavefronts, so that the products of 32 rows are one pass of four rows each and the gradient's rows are
//     split over the threads that have no column of their own; the sums over the lanes of a wavefront's rows are formed
//     together, halving the number of values at each exchange (row_sums);
//   - what one workgroup writes for the others (gradient rows, words) goes through to the coherence point and is read
//     past the XCD's cache (device-scope accesses) instead of a write-back and an invalidation of the whole
//     cache on each side of the barrier;
//   - the stored innovation (CADA1) or gradient (LAG) of the worker, its reference point and the ring stay in LDS,
//     the right-hand side is formed by a wavefront under the products, the next step's rows are asked for while the
//     others arrive (LDS-direct loads into buffers that are free by then);
//   - four workgroup barriers per step, which wait for LDS only; the wait for the gradient's stores is the one exception.
// Measured: twenty steps per call, M = 8, B = 5, p = 2500 (CADA1): 10.9 us per step.  (Shapes that cada_logreg_steps.hip serves now took here: one step per call, M = 10, B = 10, p = 54: 11.2 us; twenty
// steps per call, M = 20, B = 32, p = 784 (CADA1): 11.4 us per step; ten runs of the first side by side: 7.0.)
#include <cstring>
#include <new>
#include <type_traits>

#include "cada_small.h"

namespace cada {

constexpr int S_NT = 512, S_NW = S_NT / kWave;      // threads and wavefronts of a workgroup

__device__ __forceinline__ float sigmoid_s(float a) { return 1.0f / (1.0f + expf(-a)); }

// One LDS-direct load: lane l's 16 (4) bytes at `src` go to LDS byte `dst` + 16 l (4 l).  Written out so that no wait is
// placed before an unrelated LDS access; whoever uses the data waits for vmcnt(0) and a barrier.
template <int BYTES>
__device__ __forceinline__ void lds_direct(const float *src, const float *dst) {
  const uint32_t off = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) float *)dst);
  if constexpr (BYTES == 16) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(off), "v"(src) : "memory", "m0");
  else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" :: "s"(off), "v"(src) : "memory", "m0");
}
// every memory operation of this wavefront has completed, then the workgroup meets
__device__ __forceinline__ void full_sync() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Dynamic LDS, in floats: x [B][ps]; theta, theta_lo, h, vhat, theta - theta_ref [5][ps]; CADA: reference point [2][ps];
// dts: [2][ps]; parts of the gradient pass [groups - 1][2][ps]; r, dr [2][B rounded up to 4]; next rows [B].
__host__ __device__ inline size_t small_floats(int ps, int B, int rule, int groups, int dts) {
  const bool cada = rule == CADA_RULE_CADA1 || rule == CADA_RULE_CADA2;
  return (size_t)B * ps + (size_t)(5 + (cada ? 2 : 0) + (dts ? 2 : 0) + 2 * (groups - 1)) * ps + 2 * (size_t)((B + 3) & ~3) + B;
}

template <bool ONE>
__device__ __forceinline__ void small_body(const SmallArgs &a, const uint32_t *state /* a.s in memory */, const SmallVar &v, Phase ph, int64_t n_steps) {
  extern __shared__ __align__(16) unsigned char small_smem[];
  const DevState &s = a.s;
  const int p = (int)s.p, ps = a.ps, B = s.B, M = s.M, B4 = (s.B + 3) & ~3, nq = ps >> 2, rule = s.rule;
  const bool cada = rule == CADA_RULE_CADA1 || rule == CADA_RULE_CADA2, lds_stored = a.dts != 0;
  float *x_s = reinterpret_cast<float *>(small_smem);      // [B][ps] the minibatch
  float *th_s = x_s + (size_t)B * ps, *tl_s = th_s + ps, *h_s = tl_s + ps, *vh_s = h_s + ps;   // this workgroup's copies
  float *d_s = vh_s + ps;                                  // theta - theta_ref
  float *rf_s = d_s + ps, *rfl_s = rf_s + ps;              // the reference point (CADA rules)
  float *dt_s = d_s + (cada ? 3 : 1) * ps;                 // [2][ps] indexed like the store in memory
  float *part_s = dt_s + (lds_stored ? 2 : 0) * ps;        // [groups - 1][2][ps]
  float *r_s = part_s + 2 * (a.groups - 1) * ps, *dr_s = r_s + B4;      // [B4] residuals (before: labels) and differences
  int32_t *row_n = reinterpret_cast<int32_t *>(dr_s + B4);              // [B] rows of the minibatch to fetch next
  __shared__ float red_l[S_NW], red_q[S_NW];   // per wavefront: left-hand side, squared step
  __shared__ double rhs_s;
  __shared__ float newest_s;
  __shared__ unsigned long long last_s;
  __shared__ float ring_s[CADA_MAX_DMAX];      // the squared steps, kept up to date by every workgroup for itself
  __shared__ unsigned char dk_s[256];          // the workers' buffer selectors after this step's decisions (M <= CUs <= 256)

  // Where the state lies, for what is touched once per step: read from LDS when it is needed.  Kept in scalar registers,
  // of which there are 100, the pointers pushed each other out all over the kernel.
  __shared__ DevState at;

  const int m = blockIdx.x, nb = gridDim.x;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t mp = (int64_t)M * s.p;
  const float invB = 1.0f / (float)B;
  bool dead = false;
  int32_t tau_m = s.tau[m];
  int cur = s.sel[m];
  const int64_t base = s.row_off[m], n_m = s.row_off[m + 1] - base;
  const int32_t *idx = v.idx + (int64_t)m * B;
  const bool x16 = (p & 3) == 0 && (reinterpret_cast<uintptr_t>(s.X) & 15) == 0;
  auto put_row = [&](int b, int64_t r) __attribute__((always_inline)) {
    if (r < 0 || r >= n_m) { atomicOr(s.err, 1u); r = r < 0 ? 0 : n_m - 1; }
    row_n[b] = (int32_t)r;
  };
  // asks for the rows and labels row_n names; wavefronts w0 .. S_NW - 1 share them
  auto fetch = [&](int w0) __attribute__((always_inline)) {
    const int n = S_NW - w0;
    for (int b = w - w0; b < B; b += n) {
      const float *src = s.X + (base + __builtin_amdgcn_readfirstlane(row_n[b])) * s.p;
      float *dst = x_s + (size_t)b * ps;
      if (x16) {
        for (int j0 = 0; j0 < p; j0 += 4 * kWave)
          if (j0 + lane * 4 < p) lds_direct<16>(src + j0 + lane * 4, dst + j0);
      } else {
        for (int j0 = 0; j0 < p; j0 += kWave)
          if (j0 + lane < p) lds_direct<4>(src + j0 + lane, dst + j0);
      }
    }
    for (int b0 = (w - w0) * kWave; b0 < B; b0 += n * kWave)
      if (b0 + lane < B) lds_direct<4>(static_cast<const float *>(s.y) + base + row_n[b0 + lane], r_s + b0);
  };
  // Everything the start needs is asked for before anything is waited for; only the rows depend on their indices.
  const RefPtr ref = !ONE || rule != CADA_RULE_CADA2 ? theta_ref_in(s, tau_m, ph) : theta_ref_in(s, tau_m, Phase{(int32_t)(v.k % s.R), 0, 0});
  const float *stored = (rule == CADA_RULE_CADA1 ? s.dtl : s.gbuf) + (int64_t)cur * mp + (int64_t)m * s.p;
  const int32_t idx0 = tid < B ? idx[tid] : 0;
  const uint32_t state0 = tid < (int)(sizeof(DevState) / 4) ? state[tid] : 0u;
  // (part0: the squared step of the iteration before this launch, in the parts that a server launch or this kernel left)
  const float ring0 = tid < s.d_max ? s.ring[tid] : 0.f, part0 = v.k > 0 && tid < s.n_ring_part ? s.ring_part[tid] : 0.f;
  auto put_vectors = [&](int j, float th, float tl, float hh, float vh, float rf, float rl, float st) __attribute__((always_inline)) {
    th_s[j] = th; tl_s[j] = tl; h_s[j] = hh; vh_s[j] = vh;
    d_s[j] = cada ? (th - rf) + (tl - rl) : 0.f;
    if (cada) { rf_s[j] = rf; rfl_s[j] = rl; }
    if (lds_stored) { dt_s[cur * ps + j] = st; dt_s[(cur ^ 1) * ps + j] = 0.f; }
  };
  const int j0 = min(tid, p - 1);
  const float th0 = s.theta[j0], tl0 = s.theta_lo[j0], h0 = s.h[j0], vh0 = s.vhat[j0];
  const float rf0 = cada ? ref.hi[j0] : 0.f, rl0 = cada ? ref.lo[j0] : 0.f, st0 = lds_stored ? stored[j0] : 0.f;
  if (tid < B) put_row(tid, idx0);
  for (int b = tid + S_NT; b < B; b += S_NT) put_row(b, idx[b]);
  lds_sync();
  fetch(0);
  // under the rows' latency: the vectors, the ring, zeros in the padding (x, r, dr)
  if (tid < (int)(sizeof(DevState) / 4)) reinterpret_cast<uint32_t *>(&at)[tid] = state0;
  if (tid < s.d_max) ring_s[tid] = ring0;
  for (int j = tid + S_NT; j < s.d_max; j += S_NT) ring_s[j] = s.ring[j];
  if (w == 0) {          // (n_ring_part = ceil(p / 256) <= 32)
    const float before = (float)wave_sum_f64((double)part0);
    if (tid < S_NW) red_q[tid] = tid == 0 ? before : 0.f;
  }
  if (tid < p) put_vectors(tid, th0, tl0, h0, vh0, rf0, rl0, st0);
  for (int j = tid + S_NT; j < p; j += S_NT)
    put_vectors(j, s.theta[j], s.theta_lo[j], s.h[j], s.vhat[j], cada ? ref.hi[j] : 0.f, cada ? ref.lo[j] : 0.f, lds_stored ? stored[j] : 0.f);
  if (tid < ps - p) put_vectors(p + tid, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f);
  for (int i = tid; i < B * (ps - p); i += S_NT) x_s[(i / (ps - p)) * ps + p + i % (ps - p)] = 0.f;
  if (tid < B4 - B) { r_s[B + tid] = 0.f; dr_s[B + tid] = 0.f; }
  uint32_t *dec = a.bar + 64;
  const __amdgpu_buffer_rsrc_t store = far_buffer(s.gbuf, 2 * mp);
  // gradient pass: with several row groups thread tid has column quad tid % nq and the rows of group tid / nq
  const int G = a.groups, Bg = G > 1 ? ((B + G - 1) / G + 3) & ~3 : B4;
  const int gg = G > 1 ? tid / nq : 0, c_first = tid - gg * nq;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  for (int64_t step = 0; step < n_steps; ++step) {
    const int64_t k = v.k + step;
    const Phase ph1 = phase_after(s, ph);      // of k + 1
    const int newest_at = ONE ? k > 0 ? (int)((k - 1) % s.d_max) : 0 : ph.d == 0 ? s.d_max - 1 : ph.d - 1;
    const bool more = !ONE && step + 1 < n_steps;
    lds_sync();            // (the wavefronts waited for the rows before they came here)
    int32_t nidx = 0;
    if (more && tid < B) nidx = idx[(step + 1) * (int64_t)M * B + tid];
    // right-hand side: the squared step of iteration k-1 is this workgroup's own sum of the step before
    if (tid == S_NT - kWave) {
      float newest = red_q[0];
#pragma unroll
      for (int i = 1; i < S_NW; ++i) newest += red_q[i];
      if (k > 0) ring_s[newest_at] = newest;
      double sum = 0.0;
#pragma unroll 4
      for (int j = 0; j < s.d_max; ++j) sum += (double)ring_s[j];
      rhs_s = (s.c / (double)s.d_max) * sum;
      newest_s = newest;
    }
    // ------------------------------------------------------------ phase A
    // rows over the wavefronts, RP at a time: z = x.theta, dz = x.d, then the residual and its difference
    auto products = [&](auto RPc) __attribute__((always_inline)) {
      constexpr int RP = decltype(RPc)::value;
      for (int b0 = w; b0 < B; b0 += RP * S_NW) {
        float zd[2 * RP];
        const float *x[RP];
#pragma unroll
        for (int q = 0; q < RP; ++q) { zd[2 * q] = zd[2 * q + 1] = 0.f; x[q] = x_s + min(b0 + q * S_NW, B - 1) * ps; }   // (a row past the end repeats the last one and is dropped)
#pragma unroll 2
        for (int j = lane * 4; j < ps; j += 4 * kWave) {
          const float4 th = *reinterpret_cast<const float4 *>(th_s + j), dd = *reinterpret_cast<const float4 *>(d_s + j);
#pragma unroll
          for (int q = 0; q < RP; ++q) {
            const float4 xv = *reinterpret_cast<const float4 *>(x[q] + j);
            zd[2 * q] = fmaf(xv.x, th.x, zd[2 * q]); zd[2 * q] = fmaf(xv.y, th.y, zd[2 * q]);
            zd[2 * q] = fmaf(xv.z, th.z, zd[2 * q]); zd[2 * q] = fmaf(xv.w, th.w, zd[2 * q]);
            zd[2 * q + 1] = fmaf(xv.x, dd.x, zd[2 * q + 1]); zd[2 * q + 1] = fmaf(xv.y, dd.y, zd[2 * q + 1]);
            zd[2 * q + 1] = fmaf(xv.z, dd.z, zd[2 * q + 1]); zd[2 * q + 1] = fmaf(xv.w, dd.w, zd[2 * q + 1]);
          }
        }
        // value 2 q of a lane is z of row q, value 2 q + 1 its dz: even lanes hold z, odd lanes dz, of the row below
        const float mine = row_sums<2 * RP>(zd, lane), other = dpp_of<0xB1>(mine);
        const bool odd = lane & 1;
        const int b = b0 + S_NW * (row_sums_index<2 * RP>(lane) >> 1);
        const float z = odd ? other : mine, dz = odd ? mine : other;
        const float y = r_s[min(b, B - 1)];
        const float aa = -y * z, bb = aa + y * dz;
        const float sg = sigmoid_s(odd ? -bb : aa);            // even lanes sigma(aa), odd lanes sigma(-bb)
        const float so = dpp_of<0xB1>(sg), em = expm1f(y * dz);
        if (row_sums_owner<2 * RP>(lane) && !odd && b < B) {
          r_s[b] = -y * sg * invB;
          dr_s[b] = y * sg * so * em * invB;
        }
      }
    };
    if (B > 2 * S_NW) products(std::integral_constant<int, 4>{}); else products(std::integral_constant<int, 2>{});
    lds_sync();
    // columns over the threads, four each: fresh gradient, innovation, the rule's left-hand side
    const uint32_t gf_off = (uint32_t)(((int64_t)(1 - cur) * mp + (int64_t)m * s.p) * 4);
    float sq = 0.f;
    auto accumulate = [&](int j, v4s &g, v4s &iv) __attribute__((always_inline)) {      // this thread's rows of columns j .. j + 3
      const int b1 = min(B, (gg + 1) * Bg);
#pragma unroll 2
      for (int b = gg * Bg; b < b1; b += 4) {
        const float4 r4 = *reinterpret_cast<const float4 *>(r_s + b), d4 = *reinterpret_cast<const float4 *>(dr_s + b);   // (zero past B)
        const float rr[4] = {r4.x, r4.y, r4.z, r4.w}, dd[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const v4s xv = *reinterpret_cast<const v4s *>(x_s + min(b + e, B - 1) * ps + j);
#pragma unroll
          for (int u = 0; u < 4; ++u) { g[u] = fmaf(rr[e], xv[u], g[u]); iv[u] = fmaf(dd[e], xv[u], iv[u]); }
        }
      }
    };
    auto finish = [&](int j, v4s g, v4s iv) __attribute__((always_inline)) {
      const int64_t o = (int64_t)m * s.p + j;
      v4s st = {0.f, 0.f, 0.f, 0.f};
      if (rule != CADA_RULE_CADA2) {
        if (lds_stored) {
          st = *reinterpret_cast<const v4s *>(dt_s + cur * ps + j);
        } else {
          const float *q = (rule == CADA_RULE_CADA1 ? s.dtl : s.gbuf) + (int64_t)cur * mp + o;
#pragma unroll
          for (int e = 0; e < 4; ++e) if (j + e < p) st[e] = q[e];
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        g[e] = fmaf(s.lam, th_s[j + e], g[e]);
        iv[e] = fmaf(s.lam, d_s[j + e], iv[e]);
        float lhs_term = iv[e];
        if (rule == CADA_RULE_CADA1) lhs_term = iv[e] - st[e];
        else if (rule != CADA_RULE_CADA2) lhs_term = g[e] - st[e];          // condition (LAGrule): against the stored gradient
        sq = fmaf(lhs_term, lhs_term, sq);                                   // (the padding past p is zero throughout)
      }
      if (j + 4 <= p) {
        store_far(store, (uint32_t)j * 4u, gf_off, g);
        if (rule == CADA_RULE_CADA1) *reinterpret_cast<v4u *>(s.dtl + (int64_t)(1 - cur) * mp + o) = iv;
      } else {
        for (int e = 0; j + e < p; ++e) {
          __hip_atomic_store(s.gbuf + (int64_t)(1 - cur) * mp + o + e, g[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (rule == CADA_RULE_CADA1) s.dtl[(int64_t)(1 - cur) * mp + o + e] = iv[e];
        }
      }
      if (lds_stored) *reinterpret_cast<v4s *>(dt_s + (cur ^ 1) * ps + j) = rule == CADA_RULE_CADA1 ? iv : g;
    };
    if (G > 1) {             // (nq G <= S_NT: one quad per thread)
      v4s g = {0.f, 0.f, 0.f, 0.f}, iv = {0.f, 0.f, 0.f, 0.f};
      const int j = c_first * 4;
      if (gg < G) accumulate(j, g, iv);
      if (gg > 0 && gg < G) {
        *reinterpret_cast<v4s *>(part_s + (gg - 1) * 2 * ps + j) = g;
        *reinterpret_cast<v4s *>(part_s + (gg - 1) * 2 * ps + ps + j) = iv;
      }
      lds_sync();
      if (gg == 0) {
        for (int q = 0; q < G - 1; ++q) {
          g += *reinterpret_cast<const v4s *>(part_s + q * 2 * ps + j);
          iv += *reinterpret_cast<const v4s *>(part_s + q * 2 * ps + ps + j);
        }
        finish(j, g, iv);
      }
    } else {
      for (int j = tid * 4; j < ps; j += 4 * S_NT) {
        v4s g = {0.f, 0.f, 0.f, 0.f}, iv = {0.f, 0.f, 0.f, 0.f};
        accumulate(j, g, iv);
        finish(j, g, iv);
      }
    }
    sq = wave_sum_dpp(sq);
    if (lane == 0) red_l[w] = sq;
    if (more) {
      if (tid < B) put_row(tid, nidx);
      for (int b = tid + S_NT; b < B; b += S_NT) put_row(b, idx[(step + 1) * (int64_t)M * B + b]);
    }
    full_sync();           // the gradient's stores have reached the coherence point
    if (w == 0) {
      // the decision, by every lane of the first wavefront alike
      float lhs = red_l[0];
#pragma unroll
      for (int i = 1; i < S_NW; ++i) lhs += red_l[i];
      const double rhs = rhs_s;
      const bool own = (rule == CADA_RULE_ALWAYS) || ((double)lhs > rhs) || (tau_m >= s.D);
      bool up = own;
      const uint8_t *replay = v.replay ? v.replay + step * M : nullptr;
      if (replay != nullptr && replay[m] != CADA_REPLAY_FREE) up = replay[m] != 0;
      const int sel = up ? cur ^ 1 : cur;
      if constexpr (ONE) {
        // who is last?  Up to 56 workers the decisions travel with the count.
        unsigned long long *cnt = reinterpret_cast<unsigned long long *>(a.bar);
        if (lane == 0) {
          unsigned long long inc = 1ull << 56;
          if (M <= 56) {
            inc |= (unsigned long long)sel << m;
          } else {
            __hip_atomic_store(at.sel + m, sel, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          }
          // (counts past 255 wrap: M <= 256, and the last of 256 sees 255 before it adds)
          const unsigned long long seen = __hip_atomic_fetch_add(cnt, inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          last_s = (seen >> 56) == (unsigned long long)(M - 1) ? ((seen + inc) & ((1ull << 56) - 1)) | (1ull << 63) : 0ull;
        }
      } else {
        const uint32_t tag = ((v.bar_base + (uint32_t)step) & 0x3fffffffu) + 1u;      // (bar_base advances by n_steps M >= n_steps per launch)
        uint32_t *words = dec + (k & 1) * M;
        if (lane == 0) __hip_atomic_store(words + m, (tag << 1) | (uint32_t)sel, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int m0 = 0; m0 < M; m0 += kWave) {
          const int mm = m0 + lane;
          uint32_t word = 0, spins = 0;
          for (;;) {
            if (mm < M) word = __hip_atomic_load(words + mm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const bool ok = mm >= M || (word >> 1) == tag;
            if (dead || __all(ok)) break;
            if (++spins > a.spin_limit) { dead = true; if (lane == 0) atomicOr(at.err, 2u); break; }    // (the whole wavefront: spins is uniform)
            __builtin_amdgcn_s_sleep(1);
          }
          if (mm < M) dk_s[mm] = mm == m ? (unsigned char)sel : (unsigned char)(word & 1u);
        }
      }
      if (lane == 0) {      // the books (after the publication, which nothing should delay)
        if (k < at.trace_steps) {
          const int64_t o = k * M + m;
          at.t_mask[o] = up ? 1 : 0;
          at.t_own[o] = own ? 1 : 0;
          at.t_lhs[o] = lhs;
          at.t_tau[o] = tau_m;
          if (m == 0) at.t_rhs[k] = (float)rhs;
        }
        at.lhs[m] = lhs;
        at.mask[m] = up ? 1 : 0;
        at.tau[m] = up ? 1 : tau_m + 1;
        if (!ONE || M <= 56) at.sel[m] = sel;
        if (up) atomicAdd(reinterpret_cast<unsigned long long *>(at.uploads), 1ull);
        else if (rule == CADA_RULE_CADA2 && tau_m >= s.D) atomicOr(at.err, 8u);   // (a replay mask outlasting the retained iterates)
      }
    } else if (more) {
      fetch(1);            // (x_s and r_s were last read by the gradient pass)
    }
    lds_sync();
    if constexpr (ONE) {
      const unsigned long long last = last_s;
      if (last == 0ull) return;
      if (tid == 0) __hip_atomic_store(reinterpret_cast<unsigned long long *>(a.bar), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      for (int mm = tid; mm < M; mm += S_NT)
        dk_s[mm] = M <= 56 ? (unsigned char)((last >> mm) & 1) : (unsigned char)__hip_atomic_load(at.sel + mm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      lds_sync();
    }
    const bool up_m = (int)dk_s[m] != cur;
    if (up_m) { tau_m = 1; cur ^= 1; } else tau_m += 1;
    // ------------------------------------------------------------ phase B
    if ((ONE || m == 0) && tid == 0 && k > 0) at.ring[newest_at] = newest_s;   // (for the world outside: every workgroup has its own copy)
    float sqs = 0.f;
    const float alpha = stepsize(s, k);
    const bool snap_now = rule == CADA_RULE_CADA1 && (ONE ? (k + 1) % s.D == 0 : ph1.D == 0);
    // the decisions as bits of scalar registers, 64 workers each (M <= 256)
    unsigned long long sel64[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) sel64[i] = 64 * i < M ? __ballot(dk_s[64 * i + lane] != 0) : 0ull;
    const uint32_t mp4 = (uint32_t)mp * 4u, p4 = (uint32_t)p * 4u;
    for (int j = tid * 4; j < ps; j += 4 * S_NT) {
      // The aggregate: the sum over the workers in their order, NG rows asked for before the first is added.  A quad that
      // reaches past p reads up to three floats of what follows the row and drops them.
      v4s nab = {0.f, 0.f, 0.f, 0.f};
      auto aggregate = [&](auto NGc) __attribute__((always_inline)) {
        constexpr int NG = decltype(NGc)::value;
        for (int m0 = 0; m0 < M; m0 += NG) {
          const unsigned long long s64 = m0 < 64 ? sel64[0] : m0 < 128 ? sel64[1] : m0 < 192 ? sel64[2] : sel64[3];
          uint32_t bits = __builtin_amdgcn_readfirstlane((uint32_t)(s64 >> (m0 & 63)));
          asm volatile("" : "+s"(bits));       // (the rows' offsets are formed here, not kept in registers across the loop)
          v4s g[NG];
#pragma unroll
          for (int q = 0; q < NG; ++q) {
            const int qq = min(q, M - 1 - m0);       // (past the last worker: its row again, dropped)
            g[q] = load_far(store, (uint32_t)j * 4u, ((bits >> qq) & 1u) * mp4 + (uint32_t)(m0 + qq) * p4);
          }
#pragma unroll
          for (int q = 0; q < NG; ++q)
            if (m0 + q < M) nab += g[q];
        }
      };
      if (M <= 8) aggregate(std::integral_constant<int, 8>{});
      else if (M <= 16) aggregate(std::integral_constant<int, 16>{});
      else aggregate(std::integral_constant<int, 32>{});
      *reinterpret_cast<v4s *>(d_s + j) = nab;               // (theta - theta_ref has been used: the sums take its place for a moment)
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // (the next minibatch, asked for before, is in LDS too)
    lds_sync();
    // The update, one coordinate per thread: four per thread, as the aggregate has them, are four square roots and eight divisions one after
    // the other, and four times the code, which the first step of a launch fetches from memory.
    for (int j = tid; j < p; j += S_NT) {
      const float nab = d_s[j] / (float)M;
      float hh = h_s[j], vh = vh_s[j], vv, th = th_s[j], tl = tl_s[j];
      const float t0 = th, l0 = tl, stp = server_coordinate(s, alpha, nab, hh, vh, vv, th, tl);
      sqs = fmaf(stp, stp, sqs);
      h_s[j] = hh; vh_s[j] = vh; th_s[j] = th; tl_s[j] = tl;
      if (cada) {
        float rf = rf_s[j], rl = rfl_s[j];
        if (rule == CADA_RULE_CADA2 ? up_m : snap_now) {     // CADA2: theta^k is the next reference point; CADA1: theta^{k+1} the snapshot
          rf = rule == CADA_RULE_CADA2 ? t0 : th; rl = rule == CADA_RULE_CADA2 ? l0 : tl;
          rf_s[j] = rf; rfl_s[j] = rl;
        }
        d_s[j] = (th - rf) + (tl - rl);
      } else {
        d_s[j] = 0.f;
      }
      if (ONE || (j < 256 * nb ? j / 256 : (j / 256) % nb) == m) {
        at.nabla[j] = nab; at.h[j] = hh; at.v[j] = vv; at.vhat[j] = vh; at.theta[j] = th; at.theta_lo[j] = tl;
        if (rule == CADA_RULE_CADA2) {      // (read by other workgroups of this launch below)
          const int64_t o = (ONE ? (k + 1) % s.R : ph1.R) * s.p + j;
          __hip_atomic_store(at.hist + o, th, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(at.hist_lo + o, tl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else if (snap_now) {
          at.snap[j] = th; at.snap_lo[j] = tl;
        }
      }
    }
    for (int j = p + tid; j < ps; j += S_NT) d_s[j] = 0.f;   // (the padding keeps its zeros)
    sqs = wave_sum_dpp(sqs);
    if (lane == 0) red_q[w] = sqs;
    if (more && rule == CADA_RULE_CADA2 && tau_m > s.D) {
      // only a replay mask does this: the worker's reference point has left the retained iterates and the
      // oldest of them, theta^{k + 1 - D}, stands for it (written D steps ago; with D = 1 by the step before)
      full_sync();
      const RefPtr ref = theta_ref_in(at, tau_m, ph1);
      for (int j = tid; j < p; j += S_NT) {
        const float rf = __hip_atomic_load(ref.hi + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const float rl = __hip_atomic_load(ref.lo + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        rf_s[j] = rf; rfl_s[j] = rl;
        d_s[j] = (th_s[j] - rf) + (tl_s[j] - rl);
      }
    }
    ph = ph1;
  }
  // what a later launch, or reading the state out, adds up
  lds_sync();
  if (tid == 0 && (ONE || m == 0)) {
    float newest = red_q[0];
#pragma unroll
    for (int i = 1; i < S_NW; ++i) newest += red_q[i];
    at.ring_part[0] = newest;
    for (int i = 1; i < at.n_ring_part; ++i) at.ring_part[i] = 0.f;
  }
}

// grid (M, runs)
__global__ __launch_bounds__(S_NT) void k_small(const SmallLaunch launch) {
  // (constant address space: scalar loads, so that the compiler knows the values to be the same in all lanes)
  constexpr int n = sizeof(SmallArgs) / 8;
  const auto *src = (const __attribute__((address_space(4))) uint64_t *)(uintptr_t)launch.rep[blockIdx.y];
  uint64_t words[n];
#pragma unroll
  for (int i = 0; i < n; ++i) words[i] = src[i];
  SmallArgs a;
  __builtin_memcpy(&a, words, sizeof(a));
  small_body<false>(a, reinterpret_cast<const uint32_t *>(&launch.rep[blockIdx.y]->s), launch.var[blockIdx.y], launch.ph[blockIdx.y], launch.n_steps);
}

// grid M
// (ph is not looked at: the single step forms the remainders that its rule needs itself.  With them off the arguments p = 2500, M = 8, B = 5, CADA1: 17.95 -> 18.16 us; p = 700, M = 20, B = 40: 16.69 -> 16.93.)
__global__ __launch_bounds__(S_NT) void k_small_one(const SmallArgs a, const SmallVar v, const Phase ph) { small_body<true>(a, reinterpret_cast<const uint32_t *>(&a.s), v, ph, 1); }

// Whether the multi-step kernel serves this configuration.
bool small_plan(Ctx *c, const cada_config *cfg) {
  c->small = 0;
  const int64_t p = cfg->p;
  const int B = cfg->B, M = cfg->M;
  if (p >= 8192) return false;
  // Measured with the rows in LDS against the rows path (cada_logreg_rows.hip), us per step of a 16-step run here / of a single step here / there: M = 10, B = 10,
  // p = 54: 7 / 11.5 / 13; M = 20, B = 32, p = 784: 12 / 17 / 15; M = 64: 15 / 20 / 17; but M = 128: 21 / 26 / 19, M = 200 tiny workers 19 / 23 / 22 (the
  // server phase and the barrier grow with the workers), B = 100 rows of p = 54: 12 / 17 / 13, B = 300: 24 / 28 / 17 (one CU
  // has all rows of a worker): the path is taken by itself up to 64 workers of up to 64 rows.
  if (cfg->path != CADA_PATH_WHOLE_STEPS && (M > 64 || B > 64)) return false;
  int dev = 0, coop = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop) return false;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) return false;
  if (M > cus) return false;
  const int ps = (int)((p + 3) / 4 * 4);
  // the minibatch of a worker and the server's vectors must fit in LDS ...
  constexpr size_t kRoom = 154 * 1024;
  if (small_floats(ps, B, cfg->rule, 1, 0) * sizeof(float) > kRoom) return false;
  // ... the stored innovation or gradient where it also does, and the parts of as many row groups of the gradient pass as
  // threads are left for (of at least eight rows each)
  c->small_dts = cfg->rule != CADA_RULE_CADA2 && small_floats(ps, B, cfg->rule, 1, 1) * sizeof(float) <= kRoom ? 1 : 0;
  c->small_groups = 8;
  while (c->small_groups > 1 && (ps / 4 * c->small_groups > S_NT || (B + c->small_groups - 1) / c->small_groups < 8 ||
                                 small_floats(ps, B, cfg->rule, c->small_groups, c->small_dts) * sizeof(float) > kRoom)) c->small_groups /= 2;
  c->small_lds = small_floats(ps, B, cfg->rule, c->small_groups, c->small_dts) * sizeof(float);
  const StepsKernels steps = steps_kernels(p, B);
  c->small_one = k_small_one; c->small_several = k_small;
  if (steps.one) { c->small_one = steps.one; c->small_several = steps.several; c->small_lds = steps_lds(p); }
  else c->steps_rows = nullptr;
  for (const void *fn : {reinterpret_cast<const void *>(c->small_several), reinterpret_cast<const void *>(c->small_one)})
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRoom) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
  c->small = 1;
  c->small_plain_launch = cfg->plain_launch != 0 ? 1 : 0;
  return true;
}

constexpr uint32_t kSmallSpinLimit = 4000000u;

static SmallArgs small_args_of(Ctx *c) {
  SmallArgs a;
  a.s = c->s;
  a.bar = c->small_bar;
  a.spin_limit = kSmallSpinLimit;
  a.ps = (int)((c->s.p + 3) / 4 * 4);
  a.groups = c->small_groups;
  a.dts = c->small_dts;
  a.rows = c->steps_rows;
  return a;
}

// Writes the launch-invariant arguments of this context into its workspace (for the launches of several steps).
// The source is host memory that lives as long as the context.
int small_publish_args(Ctx *c) {
  if (!c->small) return CADA_OK;
  if (!c->small_args_host) {
    c->small_args_host = new (std::nothrow) unsigned char[sizeof(SmallArgs)];
    if (!c->small_args_host) { set_error("out of host memory"); return CADA_EINVAL; }
  }
  const SmallArgs a = small_args_of(c);
  memcpy(c->small_args_host, &a, sizeof(a));
  const hipError_t e = hipMemcpyAsync(c->small_args, c->small_args_host, sizeof(SmallArgs), hipMemcpyHostToDevice, c->stream);
  if (e != hipSuccess) { set_error("copy of launch arguments failed: %s", hipGetErrorString(e)); return CADA_EHIP; }
  return CADA_OK;
}

void small_free(Ctx *c) {
  delete[] static_cast<unsigned char *>(c->small_args_host);
  c->small_args_host = nullptr;
}

int small_steps_replicas(Ctx *const *cs, int n, const int32_t *const *idx, const uint8_t *const *replay, int64_t n_steps) {
  Ctx *c0 = cs[0];
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    set_error("cannot query the device");
    return CADA_EHIP;
  }
  if ((int64_t)n * c0->s.M > cus) { set_error("n_replicas x M = %lld workgroups exceed the %d CUs that must hold them at once", (long long)n * c0->s.M, cus); return CADA_EINVAL; }
  SmallLaunch l{};
  l.n_steps = n_steps;
  for (int r = 0; r < n; ++r) {
    l.rep[r] = static_cast<const SmallArgs *>(cs[r]->small_args);
    l.var[r] = SmallVar{idx[r], replay ? replay[r] : nullptr, cs[r]->k, cs[r]->small_seq, cs[r]->steps_turn};
    l.ph[r] = phase_of(cs[r]->s, cs[r]->k);
  }
  void *args[] = {&l};
  prof_mark(c0);
  const hipError_t e = hipLaunchCooperativeKernel(reinterpret_cast<const void *>(c0->small_several), dim3((unsigned)c0->s.M, (unsigned)n), dim3(S_NT), args,
                                                  (unsigned)c0->small_lds, c0->stream);
  prof_mark(c0);
  if (e != hipSuccess) {
    set_error("replica launch failed: %s", hipGetErrorString(e));
    return CADA_EHIP;
  }
  // (the barrier counters advance only with a launch that was accepted)
  for (int r = 0; r < n; ++r) {
    cs[r]->small_seq += (uint32_t)(n_steps * cs[r]->s.M);
    cs[r]->steps_turn = (int32_t)((cs[r]->steps_turn + n_steps) % kStepsTurns);
  }
  return CADA_OK;
}

int small_steps(Ctx *c, const int32_t *idx, const uint8_t *replay, int64_t n_steps) {
  if (n_steps == 1) {
    prof_mark(c);
    hipLaunchKernelGGL(c->small_one, dim3((unsigned)c->s.M), dim3(S_NT), c->small_lds, c->stream, small_args_of(c),
                       SmallVar{idx, replay, c->k, 0u, 0}, phase_of(c->s, c->k));
    prof_mark(c);
    const hipError_t e1 = hipGetLastError();
    if (e1 != hipSuccess) { set_error("single-step logistic launch failed: %s", hipGetErrorString(e1)); return CADA_EHIP; }
    return CADA_OK;
  }
  SmallLaunch l{};
  l.n_steps = n_steps;
  l.rep[0] = static_cast<const SmallArgs *>(c->small_args);
  l.var[0] = SmallVar{idx, replay, c->k, c->small_seq, c->steps_turn};
  l.ph[0] = phase_of(c->s, c->k);
  void *args[] = {&l};
  prof_mark(c);
  hipError_t e;
  if (c->small_plain_launch) {      // (at most as many workgroups as CUs: all resident at once on an idle device)
    hipLaunchKernelGGL(c->small_several, dim3((unsigned)c->s.M), dim3(S_NT), c->small_lds, c->stream, l);
    e = hipGetLastError();
  } else {
    e = hipLaunchCooperativeKernel(reinterpret_cast<const void *>(c->small_several), dim3((unsigned)c->s.M), dim3(S_NT), args,
                                   (unsigned)c->small_lds, c->stream);
  }
  prof_mark(c);
  if (e != hipSuccess) {
    set_error("multi-step logistic launch failed: %s", hipGetErrorString(e));
    return CADA_EHIP;
  }
  c->small_seq += (uint32_t)(n_steps * c->s.M);
  c->steps_turn = (int32_t)((c->steps_turn + n_steps) % kStepsTurns);
  return CADA_OK;
}

}  // namespace cada
