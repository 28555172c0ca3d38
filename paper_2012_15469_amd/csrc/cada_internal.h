// Internal declarations shared by the HIP translation units of libcada.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "cada.h"

namespace cada {

constexpr int kBlock = 256;          // threads per workgroup = 4 wavefronts of 64
constexpr int kWave = 64;

// Everything the kernels need to find the state; passed by value.
struct DevState {
  // server vectors [p].  The iterate is kept as an unevaluated sum theta + theta_lo of two
  // floats (|theta_lo| <= ulp(theta)/2): theta - theta_ref, which the rules' left-hand side
  // is a function of, is then accurate to float32 relative precision of the DIFFERENCE even
  // when it is a single small step (rounding theta alone perturbs a one-step difference by
  // 1e-5..1e-4 relative, more than the rule comparison tolerates).
  float *theta, *theta_lo, *h, *v, *vhat, *nabla;
  // stored / fresh stochastic gradients: gbuf[s][m][p], s in {0,1}.  Worker m's stored
  // gradient is gbuf[sel[m]][m]; the fresh one of the current step is written to
  // gbuf[1-sel[m]][m] and an upload is sel[m] ^= 1 (no copy).
  float *gbuf;
  // CADA_STORE_BF16: the same two rows per worker as bf16, gbuf16[s][m][ps16] (gbuf is null).  Written rounded to
  // nearest even by the gradient kernels, summed as they are by the server.
  uint16_t *gbuf16;
  // CADA2: hist[R][p], slot j mod R holds theta^j, R = D+1.  theta^{k-tau_m} is read here.
  float *hist, *hist_lo;
  // CADA1: snapshot theta-tilde [p] and innovations dtl[s][m][p] indexed by sel like gbuf.
  float *snap, *snap_lo, *dtl;
  // MLP with CADA1: the stored innovations are kept as bf16, dtl16[s][m][ps16] (dtl is null).  They
  // enter only the rule's left-hand side |fresh - stored|^2, whose other operand comes from bf16
  // contractions anyway; the stored GRADIENTS, which the server sums, stay float32.
  uint16_t *dtl16;
  int64_t ps;               // floats from one row of gbuf / dtl / hist to the next: p, or p rounded up to a
                            // multiple of 4 (MLP) so that every row starts on a 16-byte boundary
  int64_t ps16;             // elements from one row of dtl16 / gbuf16 to the next (a multiple of 8)
  int32_t *tau, *sel;     // [M]
  float *lhs;             // [M]
  float *lhs_part;        // [M][n_lhs_part] partial sums of the left-hand side
  uint8_t *mask;          // [M]
  float *ring;            // [d_max]
  float *ring_part;       // [n_ring_part] per-block partial sums of the last squared step,
                          // folded into ring[(k-1) mod d_max] by the next rule kernel
  uint64_t *uploads;
  uint32_t *n_up;          // [2]: uploads of iteration k in slot k mod 2 (the server kernel clears the other slot)
  int32_t resum;           // this launch: form the aggregate as the plain sum over all workers (0: the kernel may
                           // take the incremental form of Section 1.2 when few workers uploaded)
  int32_t snap_next;        // theta^{k+1} is CADA1's next snapshot
  uint32_t *err;
  // trace
  uint8_t *t_mask, *t_own;
  float *t_lhs, *t_rhs;
  int32_t *t_tau;
  int64_t trace_steps;
  // problem
  const float *X;
  const void *y;
  const int64_t *row_off;   // device [M+1], prefix sums of N_m
  int32_t M, B, d_max, D, R, rule, server_sgd, n_lhs_part, n_ring_part;
  int32_t kR;               // k mod R (the modulo of a 64-bit k is some 130 instructions at the head of a launch)
  int64_t p;
  int64_t k;                // iteration of the launch this copy is passed to
  float alpha, beta1, beta2, omb1, omb2, eps, lam;   // omb = 1 - beta, rounded once from double
  double c;
  double alpha0;            // stepsize constant; alpha above is the stepsize of iteration k
  int64_t alpha_K0;         // 0: constant; else alpha_k = alpha0 K0 / (k + K0)
};

// Where an earlier launch of the step takes the rule's inputs down (rule_inputs, cada_rule.h; else null), so that the server's workgroups can all run the rule: the right-hand
// side, and the workers' delays and buffer selectors [2][M] as they were.  (Not in DevState: 16 bytes more of it cost the whole-step kernel 2 % of a single step.)
struct RuleInputs {
  double *rhs;
  int32_t *in;
};

// Reference point of worker m at iteration k (Algorithm 1: theta-tilde for CADA1,
// theta^{k - tau_m^k} for CADA2).  The always-upload and the stochastic LAG rules evaluate no
// second gradient: their reference point is the iterate itself, so every difference the
// gradient kernels carry is exactly zero.
struct RefPtr { const float *hi, *lo; };
// (for a caller that already holds the worker's delay tau_m^k)
__device__ __forceinline__ RefPtr theta_ref_at(const DevState &s, int32_t tau_m) {
  if (s.rule == CADA_RULE_CADA1) return RefPtr{s.snap, s.snap_lo};
  if (s.rule != CADA_RULE_CADA2) return RefPtr{s.theta, s.theta_lo};
  int32_t slot = s.kR - min(tau_m, s.D);         // tau <= D unless a replay kept m silent longer
  if (slot < 0) slot += s.R;
  return RefPtr{s.hist + (int64_t)slot * s.ps, s.hist_lo + (int64_t)slot * s.ps};
}
// The same by selects, for a kernel that has all of these arguments in registers (the logistic rows' kernels take 0.3 to 0.9 us longer with it).
__device__ __forceinline__ RefPtr theta_ref_of(const DevState &s, int32_t tau_m) {
  const bool c1 = s.rule == CADA_RULE_CADA1, c2 = s.rule == CADA_RULE_CADA2;
  int32_t slot = s.kR - min(tau_m, s.D);
  slot = slot < 0 ? slot + s.R : slot;
  const int64_t at = c2 ? (int64_t)slot * s.ps : 0;
  return RefPtr{(c2 ? s.hist : c1 ? s.snap : s.theta) + at, (c2 ? s.hist_lo : c1 ? s.snap_lo : s.theta_lo) + at};
}
__device__ __forceinline__ RefPtr theta_ref(const DevState &s, int m) {
  return theta_ref_at(s, s.rule == CADA_RULE_CADA2 ? s.tau[m] : 0);
}

// (the single-pass kernel)
__device__ __forceinline__ RefPtr theta_ref(const DevState &s, int m, int64_t k) {
  if (s.rule != CADA_RULE_CADA2) return theta_ref_at(s, 0);
  int64_t slot = (k - (int64_t)min(s.tau[m], s.D)) % s.R;
  if (slot < 0) slot += s.R;
  return RefPtr{s.hist + slot * s.ps, s.hist_lo + slot * s.ps};
}

// The copy of iteration k.  Every launch of a kernel that looks for a reference point or writes one passes such a copy; not the single-pass kernel, which forms the remainders itself, and the evaluation's
// staging, which has no differences to form.
inline void set_iteration(DevState &s, int64_t k) { s.k = k; s.kR = (int32_t)(k % s.R); s.snap_next = s.rule == CADA_RULE_CADA1 && (k + 1) % s.D == 0; }

// Stepsize of iteration k (constant, or the decaying 2/(mu(k+K0)) of Theorem 2).
__host__ __device__ __forceinline__ float stepsize(const DevState &s, int64_t k) {
  return s.alpha_K0 <= 0 ? (float)s.alpha0 : (float)(s.alpha0 * (double)s.alpha_K0 / (double)(k + s.alpha_K0));
}

// bf16 storage: the hardware conversion (v_cvt_pk_bf16_f32: round to nearest even, NaN stays NaN),
// one value, or two packed into a register (first argument in the low half).
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ uint32_t f2bf_pk(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Sum over the 256 threads of a block in a fixed order; result valid in every thread.
__device__ __forceinline__ float block_sum(float x, float *red /* [4] LDS */) {
  x = wave_sum(x);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = x;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// Sum over the 64 lanes without the LDS permute path: four data-parallel-primitive steps inside each row of 16 lanes
// (quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_ror:4, row_ror:8), then the four rows' sums by lane reads.  Every
// lane gets the result; a __shfl_xor butterfly is six dependent LDS-path permutes.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
  v = dpp_add<0xB1>(v); v = dpp_add<0x4E>(v); v = dpp_add<0x124>(v); v = dpp_add<0x128>(v);
  const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0)), r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
  const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32)), r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
  return (r0 + r1) + (r2 + r3);
}

template <int CTRL>
__device__ __forceinline__ double dpp_add_f64(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, true), hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
  return x + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double lane_f64(double x, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  return __builtin_bit_cast(double, ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane));
}
__device__ __forceinline__ double wave_sum_f64(double v) {
  v = dpp_add_f64<0xB1>(v); v = dpp_add_f64<0x4E>(v); v = dpp_add_f64<0x124>(v); v = dpp_add_f64<0x128>(v);
  return (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
}

// Sums over the 64 lanes of eight values at once (as row_sums below, in double): lane l receives the sum of value (l & 3) + 4 (l >> 5), lanes with
// (l & 28) == 0 hold each value once.
template <int CTRL>
__device__ __forceinline__ double dpp_of_f64(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, true), hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double eight_sums_f64(const double (&v)[8], int lane) {
  const bool o1 = lane & 1, o2 = lane & 2, hf = lane & 32;
  double a[4], b[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = (o1 ? v[2 * i + 1] : v[2 * i]) + dpp_of_f64<0xB1>(o1 ? v[2 * i] : v[2 * i + 1]);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    b[i] = (o2 ? a[2 * i + 1] : a[2 * i]) + dpp_of_f64<0x4E>(o2 ? a[2 * i] : a[2 * i + 1]);
    b[i] = dpp_add_f64<0x124>(b[i]);
    b[i] = dpp_add_f64<0x128>(b[i]);
  }
  const double c = (hf ? b[1] : b[0]) + __shfl_xor(hf ? b[0] : b[1], 32, 64);
  return c + __shfl_xor(c, 16, 64);
}

// (An asm block that sets m0 says so, as the compiler uses that register for LDS operations of its own; it warns that the register is reserved.)
#pragma clang diagnostic ignored "-Winline-asm"

// Workgroup barrier for data that is exchanged through LDS: it waits for this wavefront's LDS operations only, not, as
// __syncthreads() does, for the acknowledgement of every global store issued before it (a microsecond each time).
// Data that a thread loaded from memory and passes on through LDS is waited for where it is written to LDS.
__device__ __forceinline__ void lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// block_sum with that barrier and the wavefront sums of wave_sum_dpp
__device__ __forceinline__ float block_sum_lds(float x, float *red /* [4] LDS */) {
  x = wave_sum_dpp(x);
  lds_sync();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  lds_sync();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

template <int CTRL>
__device__ __forceinline__ float dpp_of(float x) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true)); }

// Sums over the 64 lanes of N = 2, 4, 8 or 16 values at once.  Exchanges across lane ^ 1 and lane ^ 2 (N >= 8: and between the halves of
// the wavefront; N = 16: and between neighbouring rows of 16 lanes) halve the number of values, so that the
// whole takes about 17, 27 or 47 instructions instead of N times twenty.  Lane l receives the sum of value
// row_sums_index(l); row_sums_lane(v) is one lane that holds value v, row_sums_owner() the lanes that hold each value once.
template <int N>
__device__ __forceinline__ float row_sums(const float (&v)[N], int lane) {
  static_assert(N == 2 || N == 4 || N == 8 || N == 16, "");
  const bool o1 = lane & 1, o2 = lane & 2;
  constexpr int NB = N == 2 ? 1 : N / 4;
  float a[N / 2], b[NB];
#pragma unroll
  for (int i = 0; i < N / 2; ++i) a[i] = (o1 ? v[2 * i + 1] : v[2 * i]) + dpp_of<0xB1>(o1 ? v[2 * i] : v[2 * i + 1]);
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if constexpr (N == 2) b[i] = dpp_add<0x4E>(a[i]);
    else b[i] = (o2 ? a[2 * i + 1] : a[2 * i]) + dpp_of<0x4E>(o2 ? a[2 * i] : a[2 * i + 1]);
    b[i] = dpp_add<0x124>(b[i]);
    b[i] = dpp_add<0x128>(b[i]);
  }
  // the swap leaves (x.low, y.low) and (x.high, y.high): their sum is x's in the lower and y's in the upper lanes
  auto halves = [](float x, float y) __attribute__((always_inline)) {
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(h[0]) + __uint_as_float(h[1]);
  };
  auto rows = [](float x, float y) __attribute__((always_inline)) {
    const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
  };
  if constexpr (N <= 4) { const float c = halves(b[0], b[0]); return rows(c, c); }
  else if constexpr (N == 8) { const float c = halves(b[0], b[1]); return rows(c, c); }
  else return rows(halves(b[0], b[1]), halves(b[2], b[3]));
}
template <int N> __host__ __device__ constexpr int row_sums_index(int lane) {
  return (lane & (N == 2 ? 1 : 3)) + (N >= 8 ? 4 * (lane >> 5) : 0) + (N == 16 ? 8 * ((lane >> 4) & 1) : 0);
}
template <int N> __host__ __device__ constexpr int row_sums_lane(int v) { return (v & 3) + ((v & 4) ? 32 : 0) + ((v & 8) ? 16 : 0); }
template <int N> __host__ __device__ constexpr bool row_sums_owner(int lane) { return (lane & ((N < 16 ? 16 : 0) | (N < 8 ? 32 : 0) | 12 | (N < 4 ? 2 : 0))) == 0; }

typedef float v4s __attribute__((ext_vector_type(4)));
typedef float v4u __attribute__((ext_vector_type(4), aligned(4)));     // four floats at any 4-byte aligned address

// Four floats to / from the coherence point of the device, past the XCD's own cache: buffer accesses with the device-scope bit (sc1), since
// device-scope accesses exist in the language for four bytes only.  What lies past the buffer's end reads as zero.
constexpr int kFar = 16;
typedef uint32_t u4s __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t far_buffer(float *p, int64_t floats) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)(floats * 4), 0x00020000);
}
__device__ __forceinline__ void store_far(__amdgpu_buffer_rsrc_t r, uint32_t byte_off, uint32_t row_off, v4s x) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4s, x), r, byte_off, row_off, kFar);
}
__device__ __forceinline__ v4s load_far(__amdgpu_buffer_rsrc_t r, uint32_t byte_off, uint32_t row_off) {
  return __builtin_bit_cast(v4s, __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, row_off, kFar));
}
// One coordinate of the server update, equations (CADA-1)-(CADA-3) or the plain SGD step: new h, vhat, v, theta (two floats);
// returns the step.  beta*x + (1-beta)*y is written x + (1-beta)*(y - x): float32(0.999) is off by 1.3e-8 relative, which compounds
// to 1e-5 over the ~1000-step memory of vhat, whereas float32(1-beta) enters only linearly.
__device__ __forceinline__ float server_coordinate(const DevState &s, float alpha, float nab, float &h, float &vh, float &v, float &th, float &tl) {
  const float vo = vh;
  float step;
  v = vo;
  if (s.server_sgd) {          // theta <- theta - alpha * nabla; h, v, vhat keep their zeros
    step = alpha * nab;
  } else {
    h = fmaf(s.omb1, nab - h, h);
    v = fmaf(s.omb2, nab * nab - vo, vo);
    vh = fmaxf(v, vo);
    step = alpha * h / sqrtf(s.eps + vh);
  }
  // (theta, theta_lo) - step in two-float arithmetic (TwoSum, then renormalise)
  const float a = th, ms = -step;
  const float sum = a + ms;
  const float bb = sum - a;
  const float err = (a - (sum - bb)) + (ms - bb);
  const float lo = tl + err;
  th = sum + lo;
  tl = lo - (th - sum);
  return step;
}

constexpr int kCountWords = 32;      // a counter that workgroups count in has a 128-byte line of its own

struct SmallArgs; struct SmallVar; struct Phase; struct SmallLaunch;      // cada_small.h
// Host context.
struct Ctx {
  DevState s;
  hipStream_t stream;
  int64_t k;                 // steps enqueued
  int32_t model, gemm_dtype, n_layers;
  int32_t dims[CADA_MAX_LAYERS + 1];
  size_t state_bytes;        // the part of the workspace that a checkpoint holds
  void *ws_base;             // the caller's workspace
  // logistic launch geometry
  int vec;                   // 4 if rows can be read as float4, else 1
  int n_col_chunks;          // column chunks of the dot-product kernel
  int64_t chunk_cols;
  float *zpart;              // [M][B][n_col_chunks][2]
  int n_server_blocks;
  RuleInputs rule_in;
  int decide;                // the server's workgroups run the rule (k_server<., true>)
  int ring_cap;               // entries of ring_part in the workspace
  // single-pass (register-resident) logistic path, cada_logreg_fused.hip
  int fused, fused_Q, fused_clusters, fused_rs, fused_plain_launch;
  uint32_t fused_seq, fused_seq_per_step;
  unsigned long long *fused_post;
  int fused_tail_f, fused_tail_rows, fused_tail_rem;   // split of the last round's workers over the clusters (0: none)
  float *fused_tail;         // [clusters][2][p]: the clusters' parts of the split workers' sums
  // whole iterations in one launch for small logistic workloads, cada_logreg_small.hip
  int small;
  size_t small_lds;
  int small_groups, small_dts;   // its row groups and whether the stored innovation / gradient stays in LDS
  int small_plain_launch;    // launch it as an ordinary grid (profilers that cannot trace cooperative dispatches)
  uint32_t *small_bar;       // the whole-step kernel's barrier words in the workspace
  uint32_t small_seq;        // its value after everything enqueued so far
  void (*small_one)(const SmallArgs, const SmallVar, const Phase);      // its kernels: of a single step, of launches of several (cada_logreg_small.hip or cada_logreg_steps.hip)
  void (*small_several)(const SmallLaunch);
  float *steps_rows;         // the gradients that the workgroups of cada_logreg_steps.hip pass on (scratch; null: its kernels do not serve the shape)
  int32_t steps_turn;        // turn of the next step of a launch of several
  void *small_args;          // room in the workspace for this context's launch-invariant arguments (launches of several steps)
  void *small_args_host;     // their host copy (owned by the context)
  // one or two launches per step for rows of up to 8192 columns, cada_logreg_rows.hip
  int rows, rows_shares, rows_per_share, rows_per_worker, rows_tail;      // (rows: 1, or 2 for more than 8192 columns, whose shares are WideSplit's)
  size_t rows_lds;
  void (*rows_one)(const SmallArgs, const SmallVar, const Phase);      // small states: the whole step in the single-step kernel of cada_logreg_steps.hip (null: not this shape)
  float *rows_part;          // sums of the shares of a worker's rows
  uint32_t *rows_count;      // [1 + M] counters, kCountWords apart
  char *rule_room;           // rule_in_bytes
  // full-data evaluation scratch (cada_eval)
  double *eval_part;         // [M][kEvalBlocks][2] per-block sums of (loss, correct)
  double *eval_acc;          // [M][2]
  int logreg_group;          // workers per launch pair of the logistic gradient kernels (0 = all)
  int force_resum;           // the stored aggregate does not belong to the state (first step, after cada_set_state)
  void *mlp;                 // MLP plan (cada_mlp.hip), or nullptr
  void *prof;                // profiling events (cada_api.hip), or nullptr
  int n_phases;              // phases per step = marks per step - 1
  const char *phase_names[16];
};

void set_error(const char *fmt, ...);
// Records the next profiling event on the stream when profiling is active (else no-op).
void prof_mark(Ctx *c);

// S1+S2 for the logistic model: fresh gradients into gbuf[1-sel], left-hand sides into lhs_part.
int logreg_gradients(Ctx *c, const int32_t *idx);
bool fused_plan(Ctx *c, const cada_config *cfg);
int logreg_gradients_fused(Ctx *c, const int32_t *idx);
constexpr int64_t kRowsWidest = 10 * 2048;          // columns of the widest row that a workgroup's registers hold
bool rows_serves(const cada_config *cfg);
size_t rows_part_floats(const cada_config *cfg);
bool rows_better(const Ctx *c, const cada_config *cfg);      // the shape is served, and no other kernel is faster
bool rows_plan(Ctx *c, const cada_config *cfg);
int logreg_step_rows(Ctx *c, const int32_t *idx, const uint8_t *replay);   // gradients, rule and server
int small_steps(Ctx *c, const int32_t *idx, const uint8_t *replay, int64_t n_steps);
int small_steps_replicas(Ctx *const *cs, int n, const int32_t *const *idx, const uint8_t *const *replay, int64_t n_steps);
constexpr size_t kSmallArgsBytes = 1024;    // >= sizeof(SmallArgs), checked where it is defined
bool small_plan(Ctx *c, const cada_config *cfg);
int small_publish_args(Ctx *c);             // after the state pointers are final, and after a checkpoint was loaded
int steps_clear(Ctx *c);                    // at init, and where the state is replaced: whatever ended before that, the steps to come start clean
size_t steps_rows_floats(const cada_config *cfg);
void small_free(Ctx *c);
int logreg_init(Ctx *c);                    // LDS allowance of the two-pass kernels
constexpr int kFusedWaves = 8;                      // streaming wavefronts of a single-pass workgroup: one partial sum of the left-hand side each
constexpr size_t kFusedTailFloatsPerP = 2 * 32;     // room for the parts of 32 clusters (one per cluster, two sums)
constexpr size_t kFusedPostWords = 1024 * 4 * 16;   // upper bound: 1024 workgroups x 4 buffers x 16 values
// S1+S2 for the MLP.
int mlp_gradients(Ctx *c, const int32_t *idx);
// Partial sums of the left-hand side, with one per so many columns of a bias innovation (the rules without a second gradient have none of these: k_lag_lhs leaves theirs).
constexpr int kBiasColsState = 256;
inline int mlp_bias_cols(int rule) { return rule == CADA_RULE_CADA1 || rule == CADA_RULE_CADA2 ? 64 : kBiasColsState; }
int mlp_lhs_slots(const cada_config *cfg, int bias_cols);
int mlp_eval(Ctx *c, double *out);
int logreg_eval(Ctx *c, double *out);
int logreg_eval_noalloc(Ctx *c, double *out);   // the same kernels with their scratch in a file-scope device array
int eval_scratch_init();                        // looks that array's address up on the current device
void eval_finish(Ctx *c, double *out, int with_reg);   // out = mean over the workers of eval_acc (+ regulariser)
constexpr int kEvalBlocks = 512;      // blocks per worker of the logistic evaluation kernel
size_t mlp_workspace_bytes(const cada_config *cfg, const int64_t total_rows);
size_t mlp_scratch_bytes(const cada_config *cfg, const int64_t total_rows);      // behind the state: nothing a checkpoint holds
int mlp_plan(Ctx *c, const cada_config *cfg, char *base, size_t offset, size_t scratch, int64_t total_rows);
int mlp_init_state(Ctx *c, const float *theta0);
void mlp_free(Ctx *c);
constexpr int kLagSpan = 4096;              // coordinates of a worker that a block of k_lag_lhs takes at a time; it leaves two parts
inline int lag_blocks(int64_t p) { return (int)((p + kLagSpan - 1) / kLagSpan); }
// Room for the rule's inputs, and whether the server's workgroups run the rule (cada_server.hip: at most so many workers).
constexpr int kDecideWorkers = 256;
constexpr size_t rule_in_bytes(int M) { return 256 + (size_t)M * 2 * sizeof(int32_t); }
void decide_plan(Ctx *c, char *room);
// S3: rule, mask, tau.  S5-S7: aggregate, AMSGrad, ring push.
int rule_and_server(Ctx *c, const uint8_t *replay);
int rule_then_server(Ctx *c, const uint8_t *replay);      // the same, the left-hand side's partial sums being complete for every rule
int server_step(Ctx *c);                           // S5-S7 alone (the rule has been evaluated)

}  // namespace cada
