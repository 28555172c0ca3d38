// Whole iterations of Algorithm 1 in one kernel launch, as in cada_logreg_small.hip, for minibatches that a workgroup's registers hold: one workgroup per worker, rows of up to
// 1024 columns.  (small_plan still asks that the rows would fit LDS: 32 rows under the CADA rules have up to 1008 columns here.)  A wavefront holds whole rows, four columns per lane and quad, and asks for its rows of the next step at the head of this one: neither the products nor the
// sums of the gradient pass through LDS, and no fetch stands between a step and the next.
//
// What bounds a step is a chain, which has three workgroup barriers and one exchange among the workgroups (each wavefront's instructions count: a dependent one takes 8 cycles):
//   theta and theta - theta_ref from LDS -> z, dz of the wavefront's rows -> residuals -> its part of gradient and innovation -> LDS | -> sums over the wavefronts, left-hand
//   side | -> decision, stored gradient passed on -> all workers' gradients -> update of the thread's own columns, whose state stays in its registers -> LDS |.
// Launches of several steps exchange nothing but the gradients: a worker passes its STORED gradient on after the decision (fresh with an upload, else the one of before, which its
// workgroup keeps in registers), and a word that is not kNotYet has arrived.  No counter, no word of its own, no wait for stores to be acknowledged: what the others wait for is
// the data itself.  Rows of kStepsTurns steps take turns: a worker's row of step k is made ready for step k + 4 at the head of step k + 2.  By then its workgroup
// has all gradients of step k + 1, so every other one has gone past its reads of step k; and the store has been acknowledged when the same wavefront passes the gradient of step
// k + 3 on (it has waited for all its memory operations at the end of step k + 2), without which nobody reads that row for step k + 4.
// A single step waits for nobody: the workgroup that finishes last, which a counter that also collects the decisions tells, runs the server phase alone.
// Measured, us per step, rows in LDS with a grid barrier of tagged words / this.  Launches of twenty steps: M = 20, B = 32, p = 784: 11.4 / 9.1 (the gradients' arrival 2.0, the products 2.4: 256 FMAs of each of two
// wavefronts per SIMD are 0.85, 100 KB of rows another 0.8 of a CU's 64 bytes per cycle); ten runs of M = 10, B = 10, p = 54 side by side: 7.0 / 5.2 (products 1.0, sums 0.9, passing on 0.5,
// arrival 0.9, update 0.5; a cooperative launch 0.7 of each step); M = 64, B = 20, p = 54: 10.1 / 7.7; M = 40, B = 64, p = 512: 13.3 / 9.8; M = 24, B = 24, p = 1000: 10.6 / 10.1.
// A single step: M = 10, B = 10, p = 54: 11.2 / 8.6; M = 64, B = 20: 14.8 / 13.4; M = 12, B = 60, p = 300: 15.4 / 10.7; M = 20, B = 32, p = 784: 17.1 / 14.9.
// (Also tried: the next step's rows in registers of their own, asked for at the head of a step: 64 more of them spill with four quads of four rows, M = 20, p = 784: 205 us per twenty steps against 182;
// 64 rows of one column asked for at once: M = 64: 161 against 155; kernels with several variants of the last workgroup's aggregate: 1 us of fetching code in a single step.)
#include <algorithm>
#include <type_traits>

#include "cada_small.h"

namespace cada {

constexpr int T_NT = 512, T_NW = T_NT / kWave;      // threads and wavefronts of a workgroup
typedef uint32_t u2s __attribute__((ext_vector_type(2)));
constexpr uint32_t kNotYet = 0xffffffffu;           // (a gradient's NaN of that pattern is passed on as another one)
__device__ __forceinline__ v4s passed_on(const v4s &g) {
  u4s u = __builtin_bit_cast(u4s, g);
#pragma unroll
  for (int e = 0; e < 4; ++e) u[e] = u[e] == kNotYet ? kNotYet - 1 : u[e];
  return __builtin_bit_cast(v4s, u);
}
__device__ __forceinline__ float sigmoid_t(float a) { return 1.0f / (1.0f + expf(-a)); }
// what nobody writes during the launch, at a uniform address
template <typename T> __device__ __forceinline__ T uniform_load(const T *p) { return *(const __attribute__((address_space(4))) T *)(uintptr_t)p; }

// Memory through a pointer that itself comes from memory: said to be global (the compiler would make flat accesses of it, for which a wait for LDS waits too).
template <typename T> __device__ __forceinline__ __attribute__((address_space(1))) T *far_of(T *p) {
  static_assert(std::is_arithmetic<std::remove_const_t<T>>::value, "a template's parameter drops the alignment of v4u: far_quad");
  return (__attribute__((address_space(1))) T *)p;
}
// Four floats at any 4-byte aligned address (rows of 54 or 1021 columns, the last quad of a row).
typedef __attribute__((address_space(1))) v4u far_v4u;
__device__ __forceinline__ const far_v4u &far_quad(const float *p) { return *(const far_v4u *)p; }
__device__ __forceinline__ far_v4u &far_quad(float *p) { return *(far_v4u *)p; }

// What seldom happens is laid out behind what does: a jump to code that no workgroup of the CU has run in this launch waits for memory, code in line is fetched ahead.
__device__ __forceinline__ bool rare(bool x) { return __builtin_expect(x, false); }

// CW: quads of a row per lane (256 columns each); RW: rows of a wavefront that are worked on together, NB: such batches (a single step: 1 or 2); ONE: a single step.
// Dynamic LDS, in floats: theta, theta - theta_ref [2][ps]; the wavefronts' parts of gradient and innovation [T_NW][2][ps].
template <int CW, int RW, int NB, bool ONE>
__device__ __forceinline__ void steps_body(const SmallArgs &a, const uint32_t *state /* a.s in memory */, const SmallVar &v, Phase ph, int64_t n_steps) {
  extern __shared__ __align__(16) float steps_smem[];
  constexpr int W = CW <= 2 ? 1 : 2, NV = 2 * RW;      // columns whose server state a thread keeps; z and dz of a wavefront's rows
  const DevState &s = a.s;
  const int p = (int)s.p, ps = a.ps, B = s.B, M = s.M, nq = ps >> 2, rule = s.rule;
  const bool cada = rule == CADA_RULE_CADA1 || rule == CADA_RULE_CADA2;
  float *th_s = steps_smem, *d_s = th_s + ps, *part_s = d_s + ps;
  __shared__ double red_l[T_NW], red_q[T_NW];  // per wavefront: left-hand side, squared step (the rule compares in double)
  __shared__ double rhs_s;
  __shared__ float newest_s;
  __shared__ unsigned long long last_s;
  __shared__ float ring_s[CADA_MAX_DMAX];      // the squared steps, kept up to date by every workgroup for itself
  __shared__ unsigned char dk_s[256];          // a single step: the workers' buffer selectors after its decisions (M <= CUs <= 256)
  // Where the state lies, for what is touched once per step: read from LDS when it is needed (the pointers would push each other out of the scalar registers).
  __shared__ DevState at;

  const int m = blockIdx.x, nb = gridDim.x;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t mp = (int64_t)M * s.p;
  const float invB = 1.0f / (float)B;
  bool dead = false;
  int32_t tau_m = uniform_load(s.tau + m);
  int cur = uniform_load(s.sel + m);
  const int64_t base = uniform_load(s.row_off + m), n_m = uniform_load(s.row_off + m + 1) - base;
  // This wavefront's rows: b0 .. b0 + per - 1 of the minibatch (past its end: the last one again, with weight zero).
  const int per = (B + T_NW - 1) / T_NW, b0 = w * per, waves = (B + per - 1) / per;      // waves that have rows
  const bool busy = w < waves;
  // Indices and labels are vector loads, whose waits no access to LDS stands behind: a lane has those of the row whose z or dz it will hold (row_sums).
  const int q_of = row_sums_index<NV>(lane) >> 1;
  auto ask_idx = [&](int64_t step, int t) __attribute__((always_inline)) { return far_of(v.idx)[(step * M + m) * B + min(b0 + min(t * RW + q_of, per - 1), B - 1)]; };
  auto jb = [&](int i) __attribute__((always_inline)) { return (uint32_t)min((i * kWave + lane) * 4, p - 4); };
  auto dup = [&](int i) __attribute__((always_inline)) { return (i * kWave + lane) * 4 - (int)jb(i); };
  // Rows to be asked for: one uniform pointer each, this lane's label.
  struct Rows { const float *row[RW]; const float *label; };
  auto rows_of = [&](int32_t idx) __attribute__((always_inline)) {
    if (rare(idx < 0 || idx >= n_m)) { atomicOr(s.err, 1u); idx = idx < 0 ? 0 : (int32_t)n_m - 1; }      // (n_m <= idx < 2^31 there)
    Rows r;
#pragma unroll
    for (int q = 0; q < RW; ++q) r.row[q] = s.X + (base + __builtin_amdgcn_readlane(idx, row_sums_lane<NV>(2 * q))) * s.p;
    r.label = static_cast<const float *>(s.y) + base + idx;
    return r;
  };
  v4u x[NB][RW][CW];
  auto ask_quads = [&](const Rows &r, int t, int i) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < RW; ++q) x[t][q][i] = far_quad(r.row[q] + jb(i));
  };
  int32_t idx[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t) idx[t] = ask_idx(0, t);
  const RefPtr ref = theta_ref_in(s, tau_m, ph);
  const uint32_t state0 = tid < (int)(sizeof(DevState) / 4) ? far_of(state)[tid] : 0u;
  // (part0: the squared step of the iteration before this launch, in the parts that a server launch or this kernel left)
  const float ring0 = tid < s.d_max ? far_of(s.ring)[tid] : 0.f, part0 = v.k > 0 && tid < s.n_ring_part ? far_of(s.ring_part)[tid] : 0.f;
  // the server's state of this thread's columns W tid ..
  float th[W], tl[W], hh[W], vh[W], rf[W], rl[W];
#pragma unroll
  for (int e = 0; e < W; ++e) {
    const int j = min(tid * W + e, p - 1);
    th[e] = far_of(s.theta)[j]; tl[e] = far_of(s.theta_lo)[j]; hh[e] = far_of(s.h)[j]; vh[e] = far_of(s.vhat)[j];
    rf[e] = cada ? far_of(ref.hi)[j] : 0.f; rl[e] = cada ? far_of(ref.lo)[j] : 0.f;
  }
  float y[NB] = {};
  static_assert(ONE || NB == 1, "launches of several steps have one batch");
  if (busy) {
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const Rows r = rows_of(idx[t]);
#pragma unroll
      for (int i = 0; i < CW; ++i) ask_quads(r, t, i);
      y[t] = *far_of(r.label);
    }
    if (!ONE && n_steps > 1) idx[0] = ask_idx(1, 0);
  }
  // Thread c < nq sums quad c of the gradient up, thread nq + c that of the innovation (p <= 1024: all of them are there).  kept: of the stored gradient, or (CADA1) innovation.
  const bool is_g = tid < nq, is_iv = tid >= nq && tid < 2 * nq;
  const int jq = (is_g ? tid : is_iv ? tid - nq : 0) * 4;
  v4s kept = {0.f, 0.f, 0.f, 0.f};
  const __amdgpu_buffer_rsrc_t store = far_buffer(s.gbuf, 2 * mp);
  {
    const int64_t o = (int64_t)cur * mp + (int64_t)m * s.p + jq;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (jq + e < p) {
        if (is_g && (!ONE || !cada)) kept[e] = far_of(s.gbuf)[o + e];
        if (is_iv && rule == CADA_RULE_CADA1) kept[e] = far_of(s.dtl)[o + e];
      }
  }
  // under the rows' latency: vectors, ring, zeros in the padding
  if (tid < (int)(sizeof(DevState) / 4)) reinterpret_cast<uint32_t *>(&at)[tid] = state0;
  if (tid < s.d_max) ring_s[tid] = ring0;
  for (int j = tid + T_NT; j < s.d_max; j += T_NT) ring_s[j] = far_of(s.ring)[j];
  if (w == 0) {          // (n_ring_part = ceil(p / 256) <= 4)
    const double before = wave_sum_f64((double)part0);
    if (tid < T_NW) red_q[tid] = tid == 0 ? before : 0.0;
  }
#pragma unroll
  for (int e = 0; e < W; ++e)
    if (tid * W + e < p) { th_s[tid * W + e] = th[e]; d_s[tid * W + e] = cada ? (th[e] - rf[e]) + (tl[e] - rl[e]) : 0.f; }
  if (tid < ps - p) { th_s[p + tid] = 0.f; d_s[p + tid] = 0.f; }
  if (tid < 2 * T_NW)
    for (int j = p; j < ps; ++j) part_s[tid * ps + j] = 0.f;
  const __amdgpu_buffer_rsrc_t rows = far_buffer(a.rows, (int64_t)kStepsTurns * M * ps);
  const uint32_t row4 = (uint32_t)ps * 4u;     // bytes of a row of `rows`
  int turn = v.turn;
  if constexpr (!ONE) {
    // h and vhat of this thread's columns are here before the workgroup's first gradient can be (behind the barrier below): with it all others may update them and write them
    // back, and a wavefront without rows, under a rule without reference points, waits for nothing else until its own update.
#pragma unroll
    for (int e = 0; e < W; ++e) asm volatile("; server state %0 %1" ::"v"(hh[e]), "v"(vh[e]) : "memory");
  }

  for (int64_t step = 0; step < n_steps; ++step) {
    const int64_t k = v.k + step;
    const Phase ph1 = phase_after(s, ph);      // of k + 1
    const int newest_at = ph.d == 0 ? s.d_max - 1 : ph.d - 1;
    const bool more = !ONE && step + 1 < n_steps;
    const uint8_t forced = v.replay ? uniform_load(v.replay + step * M + m) : (uint8_t)CADA_REPLAY_FREE;
    lds_sync();
    if constexpr (!ONE) {
      if (is_g) {
        const float n = __uint_as_float(kNotYet);
        store_far(rows, (uint32_t)jq * 4u, (uint32_t)(((turn + kStepsTurns - 2) & (kStepsTurns - 1)) * M + m) * row4, v4s{n, n, n, n});
      }
    }
    // ------------------------------------------------------------ phase A
    if (busy) {
      v4s g[CW], iv[CW];
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        float zd[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) zd[q] = 0.f;
#pragma unroll
        for (int i = 0; i < CW; ++i) {                   // (a quad at a time: registers)
          float t4[4], d4[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) { t4[e] = e >= dup(i) ? th_s[jb(i) + e] : 0.f; d4[e] = e >= dup(i) ? d_s[jb(i) + e] : 0.f; }
#pragma unroll
          for (int q = 0; q < RW; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) { zd[2 * q] = fmaf(x[t][q][i][e], t4[e], zd[2 * q]); zd[2 * q + 1] = fmaf(x[t][q][i][e], d4[e], zd[2 * q + 1]); }
        }
        const float mine = row_sums<NV>(zd, lane), other = dpp_of<0xB1>(mine);      // lane holds value row_sums_index(lane): z of row / 2 in even, dz in odd lanes
        const bool odd = lane & 1;
        const float z = odd ? other : mine, dz = odd ? mine : other;
        const float aa = -y[t] * z, bb = aa + y[t] * dz;
        const float sg = sigmoid_t(odd ? -bb : aa);        // even lanes sigma(aa), odd lanes sigma(-bb)
        const float so = dpp_of<0xB1>(sg), em = expm1f(y[t] * dz);
        const float r = t * RW + q_of < per && b0 + t * RW + q_of < B ? (odd ? y[t] * so * sg * em * invB : -y[t] * sg * invB) : 0.f;      // even lanes r, odd lanes dr
        float rr[RW], dr[RW];
#pragma unroll
        for (int q = 0; q < RW; ++q) {
          rr[q] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r), row_sums_lane<NV>(2 * q)));
          dr[q] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r), row_sums_lane<NV>(2 * q + 1)));
        }
        // (the rows of the next step come in place of this one's, quad by quad, each when it has been used for the last time)
        Rows next;
        if (more) {
          next = rows_of(idx[0]);
          y[0] = *far_of(next.label);
        }
        float *pg = part_s + w * 2 * ps, *pi = pg + ps;
#pragma unroll
        for (int i = 0; i < CW; ++i) {
          if (t == 0) g[i] = iv[i] = v4s{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int q = 0; q < RW; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) { g[i][e] = fmaf(rr[q], x[t][q][i][e], g[i][e]); iv[i][e] = fmaf(dr[q], x[t][q][i][e], iv[i][e]); }
          if (more) ask_quads(next, 0, i);
          if (t + 1 < NB) continue;
          if (dup(i) == 0) {
            *reinterpret_cast<v4s *>(pg + jb(i)) = g[i];
            *reinterpret_cast<v4s *>(pi + jb(i)) = iv[i];
          } else {
#pragma unroll
            for (int e = 1; e < 4; ++e)
              if (e >= dup(i)) { pg[jb(i) + e] = g[i][e]; pi[jb(i) + e] = iv[i][e]; }
          }
        }
      }
      if (!ONE && step + 2 < n_steps) idx[0] = ask_idx(step + 2, 0);
    }
    lds_sync();
    // four columns per thread: fresh gradient or innovation, the rule's left-hand side
    float sq = 0.f;
    v4s sum = {0.f, 0.f, 0.f, 0.f};
    if (is_g || is_iv) {
      const float *src = part_s + (is_g ? 0 : ps) + jq;
#pragma unroll
      for (int q = 0; q < T_NW; ++q)
        if (q < waves) sum += *reinterpret_cast<const v4s *>(src + q * 2 * ps);
      const v4s at4 = *reinterpret_cast<const v4s *>((is_g ? th_s : d_s) + jq);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sum[e] = fmaf(s.lam, at4[e], sum[e]);
        // condition (workerrule1): against the stored innovation; (workerrule2): the innovation; (LAGrule): against the stored gradient
        const float term = rule == CADA_RULE_CADA2 ? sum[e] : sum[e] - kept[e];
        if (is_iv == cada) sq = fmaf(term, term, sq);                          // (the padding past p is zero throughout)
      }
    }
    const double part_l = wave_sum_f64((double)sq);      // (four terms at a time in float32)
    if (lane == 0) red_l[w] = part_l;
    if (w == T_NW - 1) {   // right-hand side: the squared step of iteration k-1 is this workgroup's own sum of the step before
      double all = red_q[0];
#pragma unroll
      for (int i = 1; i < T_NW; ++i) all += red_q[i];
      const float newest = (float)all;
      double acc = 0.0;
      for (int j = lane; j < s.d_max; j += kWave) acc += (double)(k > 0 && j == newest_at ? newest : ring_s[j]);
      acc = wave_sum_f64(acc);
      if (lane == 0) {
        if (k > 0) ring_s[newest_at] = newest;
        rhs_s = (s.c / (double)s.d_max) * acc;
        newest_s = newest;
      }
    }
    // the fresh gradient and (CADA1) innovation, for the steps to come
    auto put_fresh = [&]() __attribute__((always_inline)) {
      const int64_t of = (int64_t)(1 - cur) * mp + (int64_t)m * s.p + jq;
      if (is_g) {
        if (jq + 4 <= p) store_far(store, (uint32_t)jq * 4u, (uint32_t)(((int64_t)(1 - cur) * mp + (int64_t)m * s.p) * 4), sum);
        else for (int e = 0; jq + e < p; ++e) __hip_atomic_store(far_of(at.gbuf) + of + e, sum[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else if (is_iv && rule == CADA_RULE_CADA1) {
        if (jq + 4 <= p) far_quad(at.dtl + of) = sum;
        else for (int e = 0; jq + e < p; ++e) far_of(at.dtl)[of + e] = sum[e];
      }
    };
    double lhs, rhs;
    bool own, up;
    auto decide = [&]() __attribute__((always_inline)) {
      lhs = red_l[0];
#pragma unroll
      for (int i = 1; i < T_NW; ++i) lhs += red_l[i];
      rhs = rhs_s;
      own = (rule == CADA_RULE_ALWAYS) || (lhs > rhs) || (tau_m >= s.D);
      up = forced != CADA_REPLAY_FREE ? forced != 0 : own;
    };
    auto book = [&]() __attribute__((always_inline)) {
      if (rare(k < at.trace_steps)) {
        const int64_t o = k * M + m;
        far_of(at.t_mask)[o] = up ? 1 : 0;
        far_of(at.t_own)[o] = own ? 1 : 0;
        far_of(at.t_lhs)[o] = (float)lhs;
        far_of(at.t_tau)[o] = tau_m;
        if (m == 0) far_of(at.t_rhs)[k] = (float)rhs;
      }
      far_of(at.lhs)[m] = (float)lhs;
      far_of(at.mask)[m] = up ? 1 : 0;
      far_of(at.tau)[m] = up ? 1 : tau_m + 1;
      if (!ONE || M <= 56) far_of(at.sel)[m] = up ? cur ^ 1 : cur;
      if (up) atomicAdd(reinterpret_cast<unsigned long long *>(at.uploads), 1ull);
      else if (rare(rule == CADA_RULE_CADA2 && tau_m >= s.D)) atomicOr(at.err, 8u);   // (a replay mask outlasting the retained iterates)
    };
    float nab[W];
#pragma unroll
    for (int e = 0; e < W; ++e) nab[e] = 0.f;
    if constexpr (ONE) {
      put_fresh();
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");      // the gradient's stores have reached the coherence point
      if (w == 0) {
        decide();
        // who is last?  Up to 56 workers the decisions travel with the count.
        unsigned long long *cnt = reinterpret_cast<unsigned long long *>(a.bar);
        if (lane == 0) {
          const int sel = up ? cur ^ 1 : cur;
          unsigned long long inc = 1ull << 56;
          if (!rare(M > 56)) {
            inc |= (unsigned long long)sel << m;
          } else {
            __hip_atomic_store(at.sel + m, sel, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          }
          // (counts past 255 wrap: M <= 256, and the last of 256 sees 255 before it adds)
          const unsigned long long seen = __hip_atomic_fetch_add(cnt, inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          last_s = (seen >> 56) == (unsigned long long)(M - 1) ? ((seen + inc) & ((1ull << 56) - 1)) | (1ull << 63) : 0ull;
          book();          // (after the count, which nothing should delay)
        }
      }
      lds_sync();
      const unsigned long long last = last_s;
      if (last == 0ull) return;
      if (tid == 0) __hip_atomic_store(reinterpret_cast<unsigned long long *>(a.bar), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (rare(M > 56)) {
        for (int mm = tid; mm < M; mm += T_NT) dk_s[mm] = (unsigned char)__hip_atomic_load(at.sel + mm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        lds_sync();
      }
      // (whole wavefronts come here: the ballot below takes all lanes; those past the row's end read its last columns once more, and drop them)
      if (w * kWave * W < p) {
        const uint32_t mp4 = (uint32_t)mp * 4u, p4 = (uint32_t)p * 4u, col4 = (uint32_t)min(tid * W, (p - 1) / W * W) * 4u;
        constexpr int NG = 16;
        for (int m0 = 0; m0 < M; m0 += NG) {           // sixteen rows asked for before the first is added
          uint32_t bits = (uint32_t)(last >> (m0 & 63));
          if (rare(M > 56)) bits = (uint32_t)__ballot(m0 + lane < M && lane < NG && dk_s[min(m0 + lane, M - 1)] != 0);
          bits = __builtin_amdgcn_readfirstlane(bits);
          uint32_t gq[NG][W];
#pragma unroll
          for (int q = 0; q < NG; ++q) {
            const int qq = min(q, M - 1 - m0);         // (past the last worker: its row again, dropped)
            const uint32_t off = ((bits >> qq) & 1u) * mp4 + (uint32_t)(m0 + qq) * p4;
            if constexpr (W == 1) gq[q][0] = __builtin_amdgcn_raw_buffer_load_b32(store, col4, off, kFar);
            else {                                     // (the second may lie past the row: dropped)
              const u2s u = __builtin_bit_cast(u2s, __builtin_amdgcn_raw_buffer_load_b64(store, col4, off, kFar));
              gq[q][0] = u.x; gq[q][W - 1] = u.y;
            }
          }
#pragma unroll
          for (int q = 0; q < NG; ++q)
#pragma unroll
            for (int e = 0; e < W; ++e) nab[e] += m0 + q < M ? __uint_as_float(gq[q][e]) : 0.f;
        }
      }
    } else {
      // (with a replay mask a worker may go back to an iterate that others wrote in the step before: below)
      if (rare(v.replay && rule == CADA_RULE_CADA2)) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      lds_sync();
      decide();
      if (is_g) {
        const v4s out = up ? sum : kept;
        store_far(rows, (uint32_t)jq * 4u, (uint32_t)(turn * M + m) * row4, passed_on(out));
        put_fresh();
        kept = out;
      } else if (is_iv && rule == CADA_RULE_CADA1) {
        put_fresh();
        if (up) kept = sum;
      }
      if (tid == T_NT - 1) book();
      // The aggregate: the sum over the workers in their order, up to 32 rows asked for before the first is added, and again until all of them have come.
      if (tid * W < p) {
        auto aggregate = [&](auto NGc) __attribute__((always_inline)) {
          constexpr int NG = decltype(NGc)::value, SURE = NG < 32 ? NG - 7 : 1;      // rows that are there by the choice below
          for (int m0 = 0; m0 < M; m0 += NG) {
            uint32_t gq[NG][W], spins = 0;
            for (;;) {
              uint32_t most = 0, at_row = (uint32_t)(turn * M + m0) * row4;
#pragma unroll
              for (int q = 0; q < NG; ++q) {
                // (of an absent worker: zeros)
#pragma unroll
                for (int e = 0; e < W; ++e) gq[q][e] = 0u;
                if (q < SURE || m0 + q < M) {      // (uniform)
                  if constexpr (W == 1) gq[q][0] = __builtin_amdgcn_raw_buffer_load_b32(rows, (uint32_t)tid * 4u, at_row, kFar);
                  else {
                    const u2s u = __builtin_bit_cast(u2s, __builtin_amdgcn_raw_buffer_load_b64(rows, (uint32_t)tid * 8u, at_row, kFar));
                    gq[q][0] = u.x; gq[q][W - 1] = u.y;
                  }
                }
                at_row += row4;
              }
#pragma unroll
              for (int q = 0; q < NG; ++q)
#pragma unroll
                for (int e = 0; e < W; ++e) most = max(most, gq[q][e]);
              if (dead || __all(most != kNotYet)) break;
              if (rare(++spins > a.spin_limit)) { dead = true; if (lane == 0) atomicOr(at.err, 2u); break; }      // (the whole wavefront: spins is uniform)
            }
#pragma unroll
            for (int q = 0; q < NG; ++q)
#pragma unroll
              for (int e = 0; e < W; ++e) nab[e] += __uint_as_float(gq[q][e]);
          }
        };
        if (M <= 8) aggregate(std::integral_constant<int, 8>{});
        else if (M <= 16) aggregate(std::integral_constant<int, 16>{});
        else if (M <= 24) aggregate(std::integral_constant<int, 24>{});
        else aggregate(std::integral_constant<int, 32>{});
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // (the gradients were the youngest of this wavefront's loads)
      turn = (turn + 1) & (kStepsTurns - 1);
    }
    const bool up_m = ONE ? false : up;                      // (a single step's reference point is not used again)
    if (up_m) { tau_m = 1; cur ^= 1; } else tau_m += 1;
    // ------------------------------------------------------------ phase B
    if ((ONE || m == 0) && tid == 0 && k > 0) far_of(at.ring)[newest_at] = newest_s;   // (for the world outside: every workgroup has its own copy)
    double sqs = 0.0;
    const float alpha = stepsize(at, k);
    const bool snap_now = rule == CADA_RULE_CADA1 && ph1.D == 0;
#pragma unroll
    for (int e = 0; e < W; ++e) {
      const int j = tid * W + e;
      if (j < p) {
        const float mean = nab[e] / (float)M, t0 = th[e], l0 = tl[e];
        float vv;
        const float stp = server_coordinate(s, alpha, mean, hh[e], vh[e], vv, th[e], tl[e]);
        sqs = fma((double)stp, (double)stp, sqs);
        if (rule == CADA_RULE_CADA2 ? up_m : snap_now) {     // CADA2: theta^k is the next reference point; CADA1: theta^{k+1} the snapshot
          rf[e] = rule == CADA_RULE_CADA2 ? t0 : th[e]; rl[e] = rule == CADA_RULE_CADA2 ? l0 : tl[e];
        }
        if constexpr (!ONE) { th_s[j] = th[e]; d_s[j] = cada ? (th[e] - rf[e]) + (tl[e] - rl[e]) : 0.f; }
        if (ONE || (j < 256 * nb ? j / 256 : (j / 256) % nb) == m) {
          far_of(at.nabla)[j] = mean; far_of(at.h)[j] = hh[e]; far_of(at.v)[j] = vv; far_of(at.vhat)[j] = vh[e]; far_of(at.theta)[j] = th[e]; far_of(at.theta_lo)[j] = tl[e];
          if (rule == CADA_RULE_CADA2) {      // (read by other workgroups of this launch below)
            const int64_t o = (int64_t)ph1.R * s.p + j;
            __hip_atomic_store(far_of(at.hist) + o, th[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(far_of(at.hist_lo) + o, tl[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          } else if (snap_now) {
            far_of(at.snap)[j] = th[e]; far_of(at.snap_lo)[j] = tl[e];
          }
        }
      }
    }
    sqs = wave_sum_f64(sqs);
    if (lane == 0) red_q[w] = sqs;
    if (rare(more && rule == CADA_RULE_CADA2 && tau_m > s.D)) {
      // only a replay mask does this: the worker's reference point has left the retained iterates and the oldest of them, theta^{k + 1 - D}, stands for it (written
      // D steps ago; with D = 1 by the step before, whose stores have arrived before anybody passed a gradient of this step on)
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      const RefPtr oldest = theta_ref_in(at, tau_m, ph1);
#pragma unroll
      for (int e = 0; e < W; ++e) {
        const int j = tid * W + e;
        if (j < p) {
          rf[e] = __hip_atomic_load(far_of(oldest.hi) + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          rl[e] = __hip_atomic_load(far_of(oldest.lo) + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          d_s[j] = (th[e] - rf[e]) + (tl[e] - rl[e]);
        }
      }
    }
    ph = ph1;
  }
  // what a later launch, or reading the state out, adds up
  lds_sync();
  if (tid == 0 && (ONE || m == 0)) {
    double newest = red_q[0];
#pragma unroll
    for (int i = 1; i < T_NW; ++i) newest += red_q[i];
    far_of(at.ring_part)[0] = (float)newest;
    for (int i = 1; i < at.n_ring_part; ++i) far_of(at.ring_part)[i] = 0.f;
  }
}

// grid (M, runs)
template <int CW, int RW>
__global__ __launch_bounds__(T_NT) void k_steps(const SmallLaunch launch) {
  // (constant address space: scalar loads, so that the compiler knows the values to be the same in all lanes)
  constexpr int n = sizeof(SmallArgs) / 8;
  const auto *src = (const __attribute__((address_space(4))) uint64_t *)(uintptr_t)launch.rep[blockIdx.y];
  uint64_t words[n];
#pragma unroll
  for (int i = 0; i < n; ++i) words[i] = src[i];
  SmallArgs a;
  __builtin_memcpy(&a, words, sizeof(a));
  steps_body<CW, RW, 1, false>(a, reinterpret_cast<const uint32_t *>(&launch.rep[blockIdx.y]->s), launch.var[blockIdx.y], launch.ph[blockIdx.y], launch.n_steps);
}
// grid M
template <int CW, int RW, int NB = 1>
__global__ __launch_bounds__(T_NT) void k_steps_one(const SmallArgs a, const SmallVar v, const Phase ph) { steps_body<CW, RW, NB, true>(a, reinterpret_cast<const uint32_t *>(&a.s), v, ph, 1); }

StepsKernels steps_kernels(int64_t p, int B) {
  const int per = (B + T_NW - 1) / T_NW;
  if (p < 4 || p > 1024 || per > 8) return StepsKernels{nullptr, nullptr};
  if (p <= 256) return per <= 2 ? StepsKernels{k_steps_one<1, 2>, k_steps<1, 2>} : per <= 4 ? StepsKernels{k_steps_one<1, 4>, k_steps<1, 4>} : StepsKernels{k_steps_one<1, 8>, k_steps<1, 8>};
  if (p <= 512) return per <= 2 ? StepsKernels{k_steps_one<2, 2>, k_steps<2, 2>} : per <= 4 ? StepsKernels{k_steps_one<2, 4>, k_steps<2, 4>} : StepsKernels{k_steps_one<2, 8>, k_steps<2, 8>};
  return per <= 2 ? StepsKernels{k_steps_one<4, 2>, k_steps<4, 2>} : per <= 4 ? StepsKernels{k_steps_one<4, 4>, k_steps<4, 4>} : StepsKernels{nullptr, nullptr};
}
// A single step of more rows than that as well, in two batches, for the path of cada_logreg_rows.hip, which would take them in turn, split them over two workgroups, or both.  us per
// step there / here: M = 10, p = 22, B = 92, LAG: 13.1 / 10.8; M = 32, p = 200, B = 100: 14.3 / 12.4; p = 256, B = 128: 14.5 / 12.3; M = 10, p = 784, B = 60: 16.2 / 14.5; M = 16, p = 1000: 16.6 / 15.1;
// not from 257 to 512 columns, where 65 to 128 rows are 14 quads of registers per lane: p = 500, M = 24, B = 100: 15.1 / 15.4; M = 32: 15.25 / 15.45; p = 300, B = 128: 15.0 / 15.1.
StepsOne steps_one_kernel(int64_t p, int B) {
  const int per = (B + T_NW - 1) / T_NW;
  if (const StepsOne one = steps_kernels(p, B).one) return one;
  if (p < 4 || p > 1024) return nullptr;
  if (p <= 256) return per <= 16 ? k_steps_one<1, 8, 2> : nullptr;
  return p > 512 && per <= 8 ? k_steps_one<4, 4, 2> : nullptr;
}
size_t steps_lds(int64_t p) { return (size_t)(2 + 2 * T_NW) * (size_t)((p + 3) / 4 * 4) * sizeof(float); }
size_t steps_rows_floats(const cada_config *cfg) {
  return cfg->model == CADA_MODEL_LOGREG && cfg->M <= 256 && steps_kernels(cfg->p, cfg->B).one ? (size_t)kStepsTurns * cfg->M * (size_t)((cfg->p + 3) / 4 * 4) : 0;
}

__global__ void k_steps_clear(float *rows, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) rows[i] = __uint_as_float(kNotYet);
}
// No gradient is on its way.
int steps_clear(Ctx *c) {
  if (!c->small || !c->steps_rows) return CADA_OK;
  const int64_t n = (int64_t)kStepsTurns * c->s.M * ((c->s.p + 3) / 4 * 4);
  hipLaunchKernelGGL(k_steps_clear, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1024)), dim3(256), 0, c->stream, c->steps_rows, n);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("launch failed: %s", hipGetErrorString(e)); return CADA_EHIP; }
  c->steps_turn = 0;
  return CADA_OK;
}

}  // namespace cada
