// The communication rule's decision (Algorithm 1: upload iff the condition of Section 2.2
// is violated or tau_m^k >= D; tau bookkeeping) and the server side: stale-gradient
// aggregate nabla^k = (1/M) sum_m (stored gradient of m) and equations (CADA-1)-(CADA-3)
// of Section 1.2, fused with the squared step |theta^{k+1}-theta^k|^2 that the rules'
// right-hand side needs (identity in the proof of Lemma 4 of the supplement:
// |theta^{k+1}-theta^k|^2 = alpha^2 sum_i h_i^2 / (eps + vhat_i)).
#include "cada_rule.h"

namespace cada {

// Left-hand side of condition (LAGrule), Section 2.1: |fresh gradient - stored gradient|^2 per
// worker (the stored one was taken at another iterate on other samples).  grid (blocks, M);
// block b of worker m leaves its sum in lhs_part[m][2 b] and [2 b + 1], the second what the first is rounded by (one part in all: rounded); the
// remaining parts are cleared.  Squares and sums are in double, as the rule compares in double: in float32 over a block a square of 1 swallows all of 2^-25.
// What bounds it: reading, and one round trip: a block takes kLagSpan coordinates at a time, 16 bytes per access, all of them asked for before the first is used (with 2 or 4 bytes per
// access and a block for every 1024 coordinates, 617-301-150-26 with 24 workers and bf16 gradients: 9.7 us in the kernel and 96.0 per step, now 6.3 and 92.5; float32, 300-200-10 with 30 workers: 50.0 us
// per step, now 46.8; 3072-1024-10, always, 36 workers of 128 rows: 572, now 555).
template <bool BF16>
__device__ __forceinline__ double lag_part(const DevState &s, int m) {
  constexpr int E = BF16 ? 8 : 4, ROUNDS = kLagSpan / (E * kBlock);
  typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(4)));
  const int cur = s.sel[m];
  const char *gs = BF16 ? reinterpret_cast<const char *>(s.gbuf16 + ((int64_t)cur * s.M + m) * s.ps16) : reinterpret_cast<const char *>(s.gbuf + ((int64_t)cur * s.M + m) * s.ps);
  const char *gf = BF16 ? reinterpret_cast<const char *>(s.gbuf16 + ((int64_t)(1 - cur) * s.M + m) * s.ps16) : reinterpret_cast<const char *>(s.gbuf + ((int64_t)(1 - cur) * s.M + m) * s.ps);
  double sq[4] = {0.0, 0.0, 0.0, 0.0};
  auto value = [](const u4 &x, int e) __attribute__((always_inline)) { return __uint_as_float(!BF16 ? x[e] : (e & 1) ? x[e >> 1] & 0xffff0000u : x[e >> 1] << 16); };
  for (int64_t i0 = (int64_t)blockIdx.x * kLagSpan + threadIdx.x * E; i0 < s.p; i0 += (int64_t)gridDim.x * kLagSpan) {
    u4 x[ROUNDS], y[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      // (an access that would reach past the row is moved back to end with it: its values come in again, with weight zero.  bf16 rows are padded to whole accesses.)
      const int64_t i = BF16 ? min(i0 + r * E * kBlock, s.ps16 - E) : max(min(i0 + r * E * kBlock, s.p - E), (int64_t)0);
      x[r] = *reinterpret_cast<const u4 *>(gf + i * (BF16 ? 2 : 4));
      y[r] = *reinterpret_cast<const u4 *>(gs + i * (BF16 ? 2 : 4));
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int64_t want = i0 + r * E * kBlock, i = BF16 ? min(want, s.ps16 - E) : max(min(want, s.p - E), (int64_t)0);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const double d = i + e >= want && i + e < s.p ? value(x[r], e) - value(y[r], e) : 0.f;
        sq[e & 3] = fma(d, d, sq[e & 3]);
      }
    }
  }
  return (sq[0] + sq[1]) + (sq[2] + sq[3]);
}
__global__ __launch_bounds__(kBlock) void k_lag_lhs(const DevState s) {
  __shared__ double red[kBlock / kWave];
  const int m = blockIdx.y;
  const double sq = wave_sum_f64(s.gbuf16 ? lag_part<true>(s, m) : lag_part<false>(s, m));      // (bf16 store, always-upload rule, which only records this value: the rows as they are kept)
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sq;
  lds_sync();
  const bool two = 2 * (int)gridDim.x <= s.n_lhs_part;
  float *lp = s.lhs_part + (int64_t)m * s.n_lhs_part;
  if (threadIdx.x == 0) {
    const double tot = (red[0] + red[1]) + (red[2] + red[3]);
    const float hi = (float)tot;
    if (two) {
      lp[2 * blockIdx.x] = hi;
      lp[2 * blockIdx.x + 1] = isinf(hi) ? 0.f : (float)(tot - (double)hi);
    } else {
      lp[blockIdx.x] = hi;
    }
  }
  if (blockIdx.x == 0)
    for (int t = (two ? 2 : 1) * gridDim.x + threadIdx.x; t < s.n_lhs_part; t += kBlock) lp[t] = 0.f;
}

// S3 of the step: RHS, per-worker decision, tau, pointer swap, trace.  One wavefront per
// worker, four workers per block; every block forms the RHS itself (same operations, same
// value), block 0 records it.
__global__ __launch_bounds__(kBlock) void k_rule(const DevState s, const RuleInputs ri, const uint8_t *replay) {
  __shared__ double red[kBlock];
  __shared__ unsigned int cnt;
  const int64_t k = s.k;
  const int last = k > 0 ? (int)((k - 1) % s.d_max) : -1;
  const bool inputs = ri.rhs != nullptr;          // (taken down by an earlier launch of the step)
  const float newest = k > 0 && !inputs ? last_step_sq(s, red) : 0.f;
  double rhs;
  if (inputs) {
    rhs = *ri.rhs;
  } else {
    double sum = 0.0;
    for (int j = 0; j < s.d_max; ++j) sum += (double)(j == last ? newest : s.ring[j]);
    rhs = (s.c / (double)s.d_max) * sum;
  }
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  const bool tr = k < s.trace_steps;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int m = blockIdx.x * (kBlock / kWave) + wv;
  if (m < s.M) {
    double lhs = 0.0;
    const float *lp = s.lhs_part + (int64_t)m * s.n_lhs_part;
    for (int t0 = lane; t0 < s.n_lhs_part; t0 += 16 * kWave) {       // sixteen loads in flight, additions in order
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) { const int t = t0 + u * kWave; v[u] = lp[min(t, s.n_lhs_part - 1)]; if (t >= s.n_lhs_part) v[u] = 0.f; }
#pragma unroll
      for (int u = 0; u < 16; ++u) lhs += (double)v[u];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) lhs += __shfl_xor(lhs, o, 64);   // fixed tree order
    if (lane == 0) {
      const int32_t tau = s.tau[m];
      const bool own = (s.rule == CADA_RULE_ALWAYS) || (lhs > rhs) || (tau >= s.D);
      bool up = own;
      if (replay != nullptr && replay[m] != CADA_REPLAY_FREE) up = replay[m] != 0;
      if (tr) {
        const int64_t o = k * s.M + m;
        s.t_mask[o] = up ? 1 : 0;
        s.t_own[o] = own ? 1 : 0;
        s.t_lhs[o] = (float)lhs;
        s.t_tau[o] = tau;
      }
      s.lhs[m] = (float)lhs;
      s.mask[m] = up ? 1 : 0;
      if (up) {
        s.tau[m] = 1;
        s.sel[m] ^= 1;       // the fresh row becomes the stored one
        atomicAdd(&cnt, 1u);
      } else {
        s.tau[m] = tau + 1;
        // (only a replay mask can do this: the reference point theta^{k+1-(tau+1)} leaves the D+1 retained iterates)
        if (s.rule == CADA_RULE_CADA2 && tau >= s.D) atomicOr(s.err, 8u);
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (cnt) {
      atomicAdd(reinterpret_cast<unsigned long long *>(s.uploads), (unsigned long long)cnt);
      atomicAdd(s.n_up + (k & 1), cnt);
    }
    if (blockIdx.x == 0) {
      if (last >= 0 && !inputs) s.ring[last] = newest;
      if (tr) s.t_rhs[k] = (float)rhs;
    }
  }
}

// One block; used when the state is read out after the last step.
__global__ __launch_bounds__(kBlock) void k_ring_finalize(const DevState s) {
  __shared__ double red[kBlock];
  if (s.k <= 0) return;
  const float newest = last_step_sq(s, red);
  if (threadIdx.x == 0) s.ring[(s.k - 1) % s.d_max] = newest;
}

// S5-S7.  A block owns 256 coordinates, four per lane: consecutive ones read as one 16-byte
// access when every row start is 16-byte aligned (VEC == 4), else the coordinates lane,
// lane + 64, lane + 128, lane + 192 of the block's range (VEC == 1, coalesced scalar accesses).
// Wavefront w sums the stored gradients of workers w, w+4, w+8, ... for them, the four sums
// are combined through LDS in a fixed order, and each thread applies the update to one coordinate (its square root and two divisions are one chain, not
// four in a wavefront that the others wait for).
// grid = n_ring_part = ceil(p / 256) blocks.
// DECIDE: S3 as well.  Every workgroup runs the rule for itself, from the left-hand sides' partial sums and the inputs that an earlier launch has taken down (rule_inputs: nothing
// of what it reads is written in this launch); the first one keeps the books.  As many workgroups as are resident at once then take the coordinates in turn.
constexpr int kDecideSerial = 24;
template <int VEC, bool DECIDE>
__global__ __launch_bounds__(kBlock, 7) void k_server(const DevState s, const RuleInputs ri, const uint8_t *replay) {
  __shared__ __align__(16) float part[DECIDE ? 2 : 1][4][256];
  __shared__ float sq_s[DECIDE ? 2 : 1][4];
  __shared__ double lhs_s[DECIDE ? kDecideWorkers : 1];
  __shared__ uint8_t dec_s[DECIDE ? kDecideWorkers : 1];       // buffer selector after the decision, 2: uploads
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // What the launch reads of its arguments, in one round trip.  us per step without / with it: 128-64-10, always, 50 workers of 40 rows 41.6 / 41.2; 200-150-5, CADA2, 8 of 200 55.7 / 55.2; 20001 columns, LAG,
  // 37 of 75 60.7 / 60.4; but 784-512-10, 64 of 128 164.2 / 164.7 (always), 155.6 / 156.0 (CADA2, bf16 store); 784-1024-10, LAG, 20 of 200 154.9 / 155.4.  (67 / 69 vector registers with the rule.)
  asm volatile("" ::"s"(s.h), "s"(s.vhat), "s"(s.theta), "s"(s.theta_lo), "s"(s.gbuf), "s"(s.gbuf16), "s"(s.sel), "s"(s.n_up), "s"(s.lhs_part), "s"(s.M), "s"(s.p), "s"(s.ps), "s"(s.k), "s"(s.rule),
               "s"(s.D), "s"(s.n_lhs_part), "s"(s.resum), "s"(ri.in), "s"(ri.rhs), "s"(replay));
  int64_t base = (int64_t)blockIdx.x * 256;
  const int64_t mp = (int64_t)s.M * s.ps;
  // coordinate of this lane's v-th value, and whether it exists
  auto coord = [&](int v) -> int64_t { return VEC == 4 ? base + lane * 4 + v : base + lane + 64 * v; };
  auto get = [&](const float *x, float (&o)[4]) {
    if constexpr (VEC == 4) {
      if (coord(0) < s.p) {
        const float4 t = *reinterpret_cast<const float4 *>(x + coord(0));
        o[0] = t.x; o[1] = t.y; o[2] = t.z; o[3] = t.w;
      }
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (coord(v) < s.p) o[v] = x[coord(v)];
    }
  };
  uint32_t n_up = 0;
  struct Bits { unsigned long long a, b, c, d; } sel64{}, up64{};      // DECIDE: the workers' decisions as bits of scalar registers
  if constexpr (DECIDE) {
    const int tid = threadIdx.x, M = s.M, n = s.n_lhs_part;
    const int mine = min(tid, M - 1);
    const int32_t tau = ri.in[mine], sel = ri.in[M + mine];
    const uint8_t forced = replay != nullptr ? replay[mine] : (uint8_t)CADA_REPLAY_FREE;
    const double rhs = *ri.rhs;
    double lhs = 0.0;
    if (n <= kDecideSerial) {            // few parts: each thread adds its worker's up
      const float *lp = s.lhs_part + (int64_t)mine * n;
      float v[kDecideSerial];
#pragma unroll
      for (int i = 0; i < kDecideSerial; ++i) v[i] = lp[min(i, n - 1)];
#pragma unroll
      for (int i = 0; i < kDecideSerial; ++i) lhs += i < n ? (double)v[i] : 0.0;
    } else {
      // a wavefront takes eight workers at a time, three loads of each in flight; up to sixteen workers, two or four wavefronts share their parts
      const int sh = M <= 8 ? 2 : M <= 16 ? 1 : 0, per = (n + (1 << sh) - 1) >> sh, from = (w & ((1 << sh) - 1)) * per, to = min(n, from + per);
      const int m0 = 8 * (w >> sh);
      if (m0 < M) {                      // (M <= 32: decide_plan)
        double l[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (int t0 = from; t0 < to; t0 += 3 * kWave) {
          float v[8][3];
#pragma unroll
          for (int u = 0; u < 3; ++u) {
            if (t0 + u * kWave >= to) break;           // (uniform)
            const uint32_t at = min(t0 + u * kWave + lane, to - 1);
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q][u] = (s.lhs_part + (int64_t)min(m0 + q, M - 1) * n)[at];
          }
#pragma unroll
          for (int u = 0; u < 3; ++u) {
            if (t0 + u * kWave >= to) break;
#pragma unroll
            for (int q = 0; q < 8; ++q) l[q] += t0 + u * kWave + lane < to ? (double)v[q][u] : 0.0;
          }
        }
        const double sum = eight_sums_f64(l, lane);
        const int m = m0 + (lane & 3) + 4 * (lane >> 5);
        if ((lane & 28) == 0 && m < M) lhs_s[(w & ((1 << sh) - 1)) * 64 + m] = sum;
      }
      lds_sync();
      for (int q = 0; q < 1 << sh; ++q) lhs += lhs_s[64 * q + mine];
    }
    const bool own = (s.rule == CADA_RULE_ALWAYS) || (lhs > rhs) || (tau >= s.D);
    const bool up = forced != CADA_REPLAY_FREE ? forced != 0 : own;
    dec_s[tid] = tid < M ? (uint8_t)((up ? sel ^ 1 : sel) | (up ? 2 : 0)) : (uint8_t)0;
    lds_sync();
    const uint32_t d0 = dec_s[lane], d1 = dec_s[64 + lane], d2 = dec_s[128 + lane], d3 = dec_s[192 + lane];
    sel64 = Bits{__ballot(d0 & 1), __ballot(d1 & 1), __ballot(d2 & 1), __ballot(d3 & 1)};
    up64 = Bits{__ballot(d0 & 2), __ballot(d1 & 2), __ballot(d2 & 2), __ballot(d3 & 2)};
    n_up = (uint32_t)(__popcll(up64.a) + __popcll(up64.b) + __popcll(up64.c) + __popcll(up64.d));
    if (blockIdx.x == 0 && tid < M) {      // the books
      if (s.k < s.trace_steps) {
        const int64_t o = s.k * M + tid;
        s.t_mask[o] = up ? 1 : 0;
        s.t_own[o] = own ? 1 : 0;
        s.t_lhs[o] = (float)lhs;
        s.t_tau[o] = tau;
        if (tid == 0) s.t_rhs[s.k] = (float)rhs;
      }
      s.lhs[tid] = (float)lhs;
      s.mask[tid] = up ? 1 : 0;
      s.tau[tid] = up ? 1 : tau + 1;
      s.sel[tid] = dec_s[tid] & 1;
      // (only a replay mask can do this: the reference point theta^{k+1-(tau+1)} leaves the D+1 retained iterates)
      if (!up && s.rule == CADA_RULE_CADA2 && tau >= s.D) atomicOr(s.err, 8u);
      if (tid == 0) {
        *s.uploads += n_up;
        s.n_up[s.k & 1] = n_up;
      }
    }
  } else {
    n_up = s.n_up[s.k & 1];
  }
  auto bit = [](const Bits &x, int m) __attribute__((always_inline)) -> int {
    const unsigned long long word = m < 64 ? x.a : m < 128 ? x.b : m < 192 ? x.c : x.d;
    return (int)(word >> (m & 63)) & 1;
  };
  auto sel_of = [&](int m) __attribute__((always_inline)) -> int { if constexpr (DECIDE) return bit(sel64, m); else return s.sel[m]; };
  // Aggregate.  Plain form: the sum of all M stored gradients (eq. (CADA-1)).  Incremental form of
  // Section 1.2, nabla^k = nabla^{k-1} + (1/M) sum over the uploading workers of (fresh gradient - the
  // gradient it replaces): taken when it reads fewer rows (2 per upload + 1 against M); the plain
  // sum is formed whenever the host asks for it (every D iterations, and when the stored nabla is not that
  // of the step before), so rounding differences between the two forms cannot pile up.  The choice is
  // the same in every block: it depends on the iteration's upload count alone.
  const bool incremental = !s.resum && 2 * (int64_t)n_up + 1 < (int64_t)s.M;
  if (blockIdx.x == 0 && threadIdx.x == 0) s.n_up[(s.k + 1) & 1] = 0u;      // (nobody reads that slot during this launch)
  int turn = 0;
  do {
    // (what the update of this thread's coordinate reads is asked for here)
    const int64_t j = base + threadIdx.x, jr = min(j, s.p - 1);
    float hh = s.h[jr], vh = s.vhat[jr], th = s.theta[jr], tl = s.theta_lo[jr];
    const float prev = incremental ? s.nabla[jr] : 0.f;
    float nab[4] = {0.f, 0.f, 0.f, 0.f};
    auto row_of = [&](int buf, int m) -> const float * { return s.gbuf + (int64_t)buf * mp + (int64_t)m * s.ps; };
    // bf16 store (rows of ps16 elements, 16-byte aligned; VEC == 4 on that path): four coordinates are 8 bytes
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    auto get16 = [&](int buf, int m, float (&o)[4]) {
      if (coord(0) < s.p) {
        const u32x2 t = __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(s.gbuf16 + ((int64_t)buf * s.M + m) * s.ps16 + coord(0)));
        o[0] = __uint_as_float(t.x << 16); o[1] = __uint_as_float(t.x & 0xffff0000u);
        o[2] = __uint_as_float(t.y << 16); o[3] = __uint_as_float(t.y & 0xffff0000u);
      }
    };
    if (incremental) {
      for (int m = w; m < s.M; m += 4) {
        if (DECIDE ? !bit(up64, m) : !s.mask[m]) continue;      // (uniform in the wavefront)
        const int cur = sel_of(m);                       // after the swap: cur holds the fresh gradient, 1 - cur the replaced one
        float a4[4] = {0.f, 0.f, 0.f, 0.f}, b4[4] = {0.f, 0.f, 0.f, 0.f};
        if (VEC == 4 && s.gbuf16) { get16(cur, m, a4); get16(1 - cur, m, b4); }
        else { get(row_of(cur, m), a4); get(row_of(1 - cur, m), b4); }
#pragma unroll
        for (int v = 0; v < 4; ++v) nab[v] += a4[v] - b4[v];
      }
    } else if (VEC == 4 && s.gbuf16) {
#pragma unroll 4
      for (int m = w; m < s.M; m += 4) {
        float t[4] = {0.f, 0.f, 0.f, 0.f};
        get16(sel_of(m), m, t);
#pragma unroll
        for (int v = 0; v < 4; ++v) nab[v] += t[v];
      }
    } else if constexpr (VEC == 4) {
      if (coord(0) < s.p) {
#pragma unroll 5
        for (int m = w; m < s.M; m += 4) {
          typedef float f32x4 __attribute__((ext_vector_type(4)));
          // (the stored gradients are read once per step: non-temporal loads, which stream from HBM faster)
          const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(s.gbuf + (int64_t)sel_of(m) * mp + (int64_t)m * s.ps + coord(0)));
          nab[0] += t.x; nab[1] += t.y; nab[2] += t.z; nab[3] += t.w;
        }
      }
    } else {
#pragma unroll 4
      for (int m = w; m < s.M; m += 4) {
        float t[4] = {0.f, 0.f, 0.f, 0.f};
        const float *gm = s.gbuf + (int64_t)sel_of(m) * mp + (int64_t)m * s.ps;
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (coord(v) < s.p) t[v] = __builtin_nontemporal_load(gm + coord(v));
#pragma unroll
        for (int v = 0; v < 4; ++v) nab[v] += t[v];
      }
    }
    if constexpr (VEC == 4) {
      *reinterpret_cast<v4s *>(&part[turn][w][4 * lane]) = v4s{nab[0], nab[1], nab[2], nab[3]};
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v) part[turn][w][64 * v + lane] = nab[v];
    }
    lds_sync();
    const int i = threadIdx.x;
    const float mean = prev + ((part[turn][0][i] + part[turn][1][i]) + (part[turn][2][i] + part[turn][3][i])) / (float)s.M;
    float vv;
    const float step = server_coordinate(s, s.alpha, mean, hh, vh, vv, th, tl);
    if (j < s.p) {
      s.nabla[j] = mean; s.h[j] = hh; s.v[j] = vv; s.vhat[j] = vh; s.theta[j] = th; s.theta_lo[j] = tl;
      if (s.rule == CADA_RULE_CADA2) {
        const int64_t o = (int64_t)(s.kR + 1 == s.R ? 0 : s.kR + 1) * s.ps + j;
        s.hist[o] = th;
        s.hist_lo[o] = tl;
      } else if (s.snap_next) {
        s.snap[j] = th;
        s.snap_lo[j] = tl;
      }
    }
    const float sq = wave_sum_dpp(j < s.p ? step * step : 0.f);
    if (lane == 0) sq_s[turn][w] = sq;
    lds_sync();
    if (i == 0) s.ring_part[base >> 8] = (sq_s[turn][0] + sq_s[turn][1]) + (sq_s[turn][2] + sq_s[turn][3]);
    base += (int64_t)gridDim.x * 256;
    turn ^= 1;             // (what a turn leaves in LDS is written again two turns later, a barrier behind its readers)
  } while (DECIDE && base < s.p);
}

// The rule in the server's launch saves one, and every workgroup reads all partial sums of the left-hand sides for it.  Measured, us per step with it / with a launch of
// its own, M workers of n parts.  Few parts (rows that are read 16 bytes at a time): p = 20480, n = 20: M = 64: 33.5 / 34.8; 128: 41.3 / 42.2; 256: 58.9 / 59.2; p = 10000, n = 10: M = 64: 24.7 / 25.9; 128: 33.6 /
// 33.5; 256: 47.6 / 45.9; 4 bytes at a time, p = 10001, n = 10: M = 64: 24.7 / 32.2; 256: 47.4 / 69.9; 512-128-10, n = 23: M = 64: 52.0 / 53.5; 256: 106.1 / 106.7; 384-128-10, n = 19: M = 256: 94.9 / 94.0;
// 100-60-5, n = 11: M = 256: 63.2 / 63.1.  LAG and always: 384-120-10, n = 24: M = 64: 46.1 / 47.5; 128: 58.4 / 58.5; 256: 86.2 / 83.7; 150-100-10, n = 8: M = 64: 41.9 / 43.4; 128: 51.8 / 51.5; 256: 67.8 / 64.5;
// 100-60-5, n = 4: M = 256: 54.4 / 54.3.  More parts: 784-500-10, n = 137: M = 10: 58.5 / 60.1; 21: 73.0 / 74.1; 400-300-10, n = 66: M = 32: 58.4 / 60.9; 700-700-10, LAG, n = 246: M = 3: 46.9 / 45.9;
// but 200-150-10, M = 64, n = 28: 68.4 / 67.6; 1000-800-10, M = 16, n = 267: 144.9 / 142.0;
// 2000-500-10, M = 20, n = 281: 154.9 / 153.0; 784-300-10, M = 100: 130.1 / 127.6; 784-512-10, M = 64, n = 137: 174.2 / 171.3; 3072-1024-1024-10, M = 16: 580.9 / 577.1.
// The launch of its own: 784-512-10, M = 64: 4.8 us, 5.9 where it adds the squared step's parts up itself; 3072-1024-1024-10, M = 16: 6.7, 10.7.
constexpr int64_t kDecideParts = 3000;
constexpr int kDecideBlocks = 7 * 256;           // seven workgroups of up to 73 registers per CU
void decide_plan(Ctx *c, char *room) {
  c->rule_in = RuleInputs{reinterpret_cast<double *>(room), reinterpret_cast<int32_t *>(room + 256)};
  const int64_t M = c->s.M, n = c->s.n_lhs_part;
  const bool one_gradient = c->s.rule == CADA_RULE_ALWAYS || c->s.rule == CADA_RULE_LAG;
  c->decide = M <= (c->model == CADA_MODEL_MLP && one_gradient && n > 4 ? kDecideWorkers / 2 : kDecideWorkers) && (n <= kDecideSerial || (M <= 32 && M * n <= kDecideParts));
}

namespace {
int launch_server(Ctx *c, bool decide, const uint8_t *replay) {
  DevState s = c->s;
  set_iteration(s, c->k);
  s.alpha = stepsize(s, s.k);
  s.resum = (c->force_resum || s.k % s.D == 0) ? 1 : 0;
  const dim3 grid(decide ? min(s.n_ring_part, kDecideBlocks) : s.n_ring_part);
  if (c->vec == 4) {
    if (decide) hipLaunchKernelGGL((k_server<4, true>), grid, dim3(kBlock), 0, c->stream, s, c->rule_in, replay);
    else hipLaunchKernelGGL((k_server<4, false>), grid, dim3(kBlock), 0, c->stream, s, c->rule_in, nullptr);
  } else {
    if (decide) hipLaunchKernelGGL((k_server<1, true>), grid, dim3(kBlock), 0, c->stream, s, c->rule_in, replay);
    else hipLaunchKernelGGL((k_server<1, false>), grid, dim3(kBlock), 0, c->stream, s, c->rule_in, nullptr);
  }
  prof_mark(c);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("server launch failed: %s", hipGetErrorString(e)); return CADA_EHIP; }
  c->force_resum = 0;
  return CADA_OK;
}
}  // namespace

int server_step(Ctx *c) { return launch_server(c, false, nullptr); }

int rule_then_server(Ctx *c, const uint8_t *replay) {
  if (c->decide) return launch_server(c, true, replay);
  DevState s = c->s;
  set_iteration(s, c->k);
  hipLaunchKernelGGL(k_rule, dim3((unsigned)((s.M + 3) / 4)), dim3(kBlock), 0, c->stream, s, c->rule_in, replay);
  prof_mark(c);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error("rule launch failed: %s", hipGetErrorString(e));
    return CADA_EHIP;
  }
  return server_step(c);
}

int rule_and_server(Ctx *c, const uint8_t *replay) {
  DevState s = c->s;
  set_iteration(s, c->k);
  if (s.rule == CADA_RULE_LAG || s.rule == CADA_RULE_ALWAYS) {   // (the always-upload rule only records it)
    const int nb = min(max(s.n_lhs_part / 2, 1), lag_blocks(s.p));      // (two parts each; the logistic model: one, of at most 1024 coordinates, or room for two for every 4096)
    hipLaunchKernelGGL(k_lag_lhs, dim3((unsigned)nb, (unsigned)s.M), dim3(kBlock), 0, c->stream, s);
  }
  return rule_then_server(c, replay);
}

int ring_finalize(Ctx *c) {
  DevState s = c->s;
  set_iteration(s, c->k);
  hipLaunchKernelGGL(k_ring_finalize, dim3(1), dim3(kBlock), 0, c->stream, s);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error("ring finalize launch failed: %s", hipGetErrorString(e));
    return CADA_EHIP;
  }
  return CADA_OK;
}

}  // namespace cada
