// Dual minibatch gradient, rule and (small states) server update of the logistic model for rows that one workgroup can
// hold in its registers (p <= 8192), and the rows cross the memory bus once.  A step is
//   ONE launch where the state is small (kServerColumns, kServerState, kServerWorkers): its last workgroup runs rule and server (minibatches that a workgroup's registers hold
//   take the single-step kernel of cada_logreg_steps.hip for it);
//   two, up to kRuleInServer workers: the server's launch runs the rule (cada_server.hip), from inputs that this one takes down;
//   two, up to kRuleWorkers: the last workgroup runs the rule;
//   three with more workers: the rule has a launch of its own.
//
// Workgroup (g, m) takes a share of worker m's minibatch rows.  The rows of a share are read into registers, many at a
// time; z = x.theta and dz = x.d are summed over the lanes, turned into the residual and its difference (formulas as in
// cada_logreg.hip), and the same registers are accumulated into the gradient and the innovation: no second pass.
//   p <= 1024: a wavefront holds whole rows (WC = 1), the eight wavefronts work on rows of their own and add their sums up
//     through LDS at the end: no workgroup barrier per row;
//   p <= 8192: a row lies across the eight wavefronts (WC = 8), which exchange their parts of z, dz through LDS, one barrier per
//     batch of rows.  The next batch is asked for before a batch's products; in every other one the compiled loop waits for it as well.
// Nothing waits for another workgroup: whoever finishes last continues.  The last workgroup of a worker adds the shares'
// sums up in their order, forms the fresh gradient and the left-hand side; the last of those runs the rule for
// all workers, and the server update, where the list above says so.  The partial sums, gradients and left-hand sides that are passed on
// inside the launch are written and read at device scope (past the XCD's cache).
//
// Wider rows, up to 20480 columns: k_rows_wide and k_rows_sum below, two launches, and the server's with the rule in it (more than 256 workers: a launch of its own).
//
// Why: the path replaces four to five dependent launches (two passes over the rows, [left-hand side of the LAG rule],
// rule, server), each about 5 us of fetching arguments, code and first operands for well under 1 us of work.
// Measured per step, against those launches: M = 10, p = 784, B = 60: 23.8 -> 16.2 us (15.5 in the kernel: operands and indices 3.3,
// rows 2.9, share's sums 2.6, gradient 1.5, count 0.7, rule 1.0, aggregate 2.1, update 1.3; in cada_logreg_steps.hip 14.6); M = 100, B = 256, p = 4000 (410 MB of rows): 147 -> 87 us; p = 8192: 308 -> 164 us (5.1 TB/s).
#include <type_traits>

#include "cada_rows_split.h"
#include "cada_rule.h"
#include "cada_small.h"

namespace cada {

constexpr int R_NT = 512, R_NW = R_NT / kWave;
enum { kTailNone = 0, kTailRule = 1, kTailServer = 2 };      // what the workgroup that finishes last does: nothing, the rule, the server update too
// The server update in the launch's last workgroup saves a launch, and costs a pass over the state by one CU.  Measured, us per step with and
// without it, B = 65: M = 10, p = 22: 12.5, 15.0; M = 32, p = 256: 14.0, 15.5; M = 32, p = 500: 14.5, 15.5; M = 48: 15.6, 16.1; M = 64: 16.8,
// 16.7; M = 16, p = 784: 16.5, 17.1; M = 24: 18.1, 17.2; M = 16, p = 1024: 16.4, 17.0; M = 1, p = 1500: 16.5, 16.3; 3000: 22.0, 18.9; 8000: 40.7, 26.6.
// Minibatches that the single-step kernel of cada_logreg_steps.hip takes, in it / with a launch for rule and server: M = 33, p = 22, B = 92, LAG: 13.0, 13.8; M = 48: 13.4, 13.9; M = 64: 15.5, 14.7; M = 48,
// p = 200, B = 100: 13.8, 14.3; M = 64, p = 256: 16.1, 15.0; M = 21, p = 784, B = 60: 16.2, 14.5; M = 17, p = 1024: 16.4, 14.7: the same line for M p; for few columns M could go to 48.
constexpr int kServerColumns = 2 * R_NT, kServerState = 16384, kServerWorkers = 32;      // p, M p and M up to here
// The rule in the last workgroup saves a launch as well; the workgroups count themselves in one after the other for it.  Measured, us with
// and without it: B = 65, p = 22: M = 100: 17.2, 19.9; 256: 23.3, 24.1; 400: 28.6, 30.0; 512: 32.3, 32.4; 1024: 54.9, 53.8; p = 8191, M = 512: 215, 219;
// 1024: 414, 416.
// In the server's launch (cada_server.hip) it needs neither: up to 256 workers.  us per step there / in the last workgroup: p = 54, M = 200, B = 100: 21.6 / 33.7; p = 300,
// M = 100, B = 80: 20.8 / 24.4; p = 784, M = 256, B = 40: 31.8 / 41.9; M = 64, B = 60: 20.7 / 23.7; p = 1500, M = 10, B = 64: 16.6 / 17.7; p = 8192, LAG, M = 16: 34.6 / 36.4;
// p = 4000, M = 100, B = 256: 93.8 / 96.4.  (The server update in the last workgroup stays where it is: p = 784, M = 16, B = 100: 17.0 for 18.0, p = 100, M = 10: 12.1 for 13.8.)
constexpr int kRuleWorkers = 512, kRuleInServer = kDecideWorkers;

struct RowsArgs {
  DevState s;
  const int32_t *idx;        // [M][B]
  const uint8_t *replay;     // [M] or nullptr
  float *part;               // sums of the shares: k_rows [M][shares][2][p rounded up to 4] (shares > 1), k_rows_wide [wide_slots][2][the same]
  uint32_t *count;           // [1 + M], kCountWords apart: workers done; shares done of each worker (zero between launches)
  int shares;                // k_rows: workgroups per worker
  int rows;                  // rows per share (at most)
  int tail;                  // kTail*
  WideSplit wide;            // k_rows_wide, k_rows_sum
};

struct RowsInArgs : RowsArgs { RuleInputs ri; };

__device__ __forceinline__ float sigmoid_r(float a) { return 1.0f / (1.0f + expf(-a)); }

// CW: 16-byte pieces of a row per lane; WC: wavefronts a row lies across; RB: rows per batch.
// dynamic LDS: row offsets int64 [rows], labels [rows] (rounded up to four rows), sums [R_NW / WC][2][p]
// Args RowsInArgs: the launch ends with the left-hand sides and takes the rule's inputs down for the server's launch (a kernel of its own: the code at the end of the
// other one costs that 1 to 3 % of a step of few workers).
template <int CW, int WC, int RB, class Args>
__global__ __launch_bounds__(R_NT) void k_rows(const Args a) {
  extern __shared__ __align__(16) unsigned char rows_smem[];
  const DevState &s = a.s;
  const int p = (int)s.p, ps = (p + 3) & ~3, M = s.M, m = blockIdx.y, share = blockIdx.x, rule = s.rule;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int64_t *off_s = reinterpret_cast<int64_t *>(rows_smem);
  float *y_s = reinterpret_cast<float *>(off_s + ((a.rows + 3) & ~3));
  float *sum_s = y_s + ((a.rows + 3) & ~3);             // [R_NW / WC][2][p rounded up to 4]
  __shared__ float red_s[2][R_NW][2 * RB];
  __shared__ double red_l[R_NW];
  __shared__ uint32_t flag_s, up_s;
  constexpr int NV = 2 * RB;
  static_assert(NV == 4 || NV == 8 || NV == 16, "row_sums");

  const int r0 = share * a.rows, nr = min(a.rows, s.B - r0);        // this share's rows
  const int64_t base = s.row_off[m], n_m = s.row_off[m + 1] - base;
  const int64_t mp = (int64_t)M * s.p;
  const RefPtr ref = theta_ref(s, m);
  // this lane's columns: CW quads; the quad that would reach past p is moved back to end at p, `dup` of its columns belong
  // to the quad before (weight zero here, not stored from here); a quad beyond p has dup >= 4
  int jb[CW], dup[CW];
  float th[CW][4], dd[CW][4], g[CW][4], iv[CW][4];
#pragma unroll
  for (int i = 0; i < CW; ++i) {
    const int j = (((WC == 1 ? 0 : w) * CW + i) * kWave + lane) * 4;
    jb[i] = min(j, p - 4);
    dup[i] = j - jb[i];
  }
  // theta and theta - theta_ref at j .. j + 3 (up to three floats past p: of what follows in the workspace)
  auto diff_at = [&](int j, v4u &t4, v4s &d4) __attribute__((always_inline)) {
    t4 = *reinterpret_cast<const v4u *>(s.theta + j);
    const v4u l4 = *reinterpret_cast<const v4u *>(s.theta_lo + j), rh = *reinterpret_cast<const v4u *>(ref.hi + j), rl = *reinterpret_cast<const v4u *>(ref.lo + j);
#pragma unroll
    for (int e = 0; e < 4; ++e) d4[e] = (t4[e] - rh[e]) + (l4[e] - rl[e]);
  };
  // What the end of the launch needs and nobody changes before it is asked for here, so that its latency passes under the rows'.
  int32_t tau0 = 0, sel0 = 0, rep0 = CADA_REPLAY_FREE;          // of worker tid
  if (tid < M) {
    tau0 = s.tau[tid]; sel0 = s.sel[tid];
    if (a.replay != nullptr) rep0 = a.replay[tid];
  }
  const float ring0 = lane < s.d_max ? s.ring[lane] : 0.f, part0 = lane < s.n_ring_part ? s.ring_part[lane] : 0.f;   // (n_ring_part <= 32)
  auto row_of = [&](int b, int32_t r0_) __attribute__((always_inline)) {
    int64_t r = r0_;
    if (r < 0 || r >= n_m) { atomicOr(s.err, 1u); r = r < 0 ? 0 : n_m - 1; }
    off_s[b] = (base + r) * s.p;
    return base + r;
  };
  const int32_t *idx = a.idx + (int64_t)m * s.B + r0;
  int64_t row0 = 0;
  const int32_t idx0 = tid < nr ? idx[tid] : 0;
  if constexpr (WC == 1) {
    // (every wavefront needs all of theta and the difference: fetched once for the workgroup, through the room of the sums)
    float *d_s = sum_s + ps;
    if (tid * 4 < ps) {                                // (p <= 1024: one quad per thread)
      v4u t4; v4s d4;
      diff_at(tid * 4, t4, d4);
      *reinterpret_cast<v4s *>(sum_s + tid * 4) = t4;
      *reinterpret_cast<v4s *>(d_s + tid * 4) = d4;
    }
  } else {
#pragma unroll
    for (int i = 0; i < CW; ++i) {
      v4u t4; v4s d4;
      diff_at(jb[i], t4, d4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { th[i][e] = e >= dup[i] ? t4[e] : 0.f; dd[i][e] = e >= dup[i] ? d4[e] : 0.f; }
    }
  }
  if (tid < nr) row0 = row_of(tid, idx0);
  for (int b = tid + R_NT; b < nr; b += R_NT) y_s[b] = static_cast<const float *>(s.y)[row_of(b, idx[b])];
  lds_sync();

  const float invB = 1.0f / (float)s.B;
  constexpr int NG = R_NW / WC;                        // row groups: group q takes rows q, q + NG, ...
  const int grp = WC == 1 ? w : 0;
  v4u x[2][RB][CW];
  auto load = [&](v4u (&xb)[RB][CW], int b0) __attribute__((always_inline)) {      // rows b0, b0 + NG, ... (past the end: the last row, with weight zero)
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      const int64_t o = off_s[min(b0 + q * NG, nr - 1)];
      const float *row = s.X + (((int64_t)__builtin_amdgcn_readfirstlane((uint32_t)(o >> 32)) << 32) | __builtin_amdgcn_readfirstlane((uint32_t)o));
#pragma unroll
      for (int i = 0; i < CW; ++i) xb[q][i] = *reinterpret_cast<const v4u *>(row + jb[i]);
    }
  };
  auto work = [&](v4u (&xb)[RB][CW], int b0, int it) __attribute__((always_inline)) {
    float zd[NV];
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      zd[2 * q] = zd[2 * q + 1] = 0.f;
#pragma unroll
      for (int i = 0; i < CW; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) { zd[2 * q] = fmaf(xb[q][i][e], th[i][e], zd[2 * q]); zd[2 * q + 1] = fmaf(xb[q][i][e], dd[i][e], zd[2 * q + 1]); }
    }
    float mine = row_sums<NV>(zd, lane);               // lane holds value v(lane): z of row v / 2 in even, dz in odd lanes
    const int v = row_sums_index<NV>(lane);
    if constexpr (WC > 1) {
      if (row_sums_owner<NV>(lane)) red_s[it & 1][w][v] = mine;
      lds_sync();
      mine = 0.f;
#pragma unroll
      for (int i = 0; i < R_NW; ++i) mine += red_s[it & 1][i][v];
    }
    const float other = dpp_of<0xB1>(mine);
    const bool odd = lane & 1;
    const int b = b0 + (v >> 1) * NG;
    const float z = odd ? other : mine, dz = odd ? mine : other;
    const float y = y_s[min(b, nr - 1)];
    const float aa = -y * z, bb = aa + y * dz;
    const float sg = sigmoid_r(odd ? -bb : aa);        // even lanes sigma(aa), odd lanes sigma(-bb)
    const float so = dpp_of<0xB1>(sg), em = expm1f(y * dz);
    float r = b < nr ? (odd ? y * so * sg * em * invB : -y * sg * invB) : 0.f;      // even lanes r, odd lanes dr
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      const float rr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r), row_sums_lane<NV>(2 * q)));
      const float dr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r), row_sums_lane<NV>(2 * q + 1)));
#pragma unroll
      for (int i = 0; i < CW; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) { g[i][e] = fmaf(rr, xb[q][i][e], g[i][e]); iv[i][e] = fmaf(dr, xb[q][i][e], iv[i][e]); }
    }
  };
  const int64_t k = s.k;
  const int last = k > 0 ? (int)((k - 1) % s.d_max) : -1;
  double rhs;
  float newest;
  {
    int b = grp, it = 0;
    if (b < nr) load(x[0], b);
    const float label = tid < nr ? static_cast<const float *>(s.y)[row0] : 0.f;
    // right-hand side of the rule, by every wavefront alike while its rows are on their way: the squared step of the iteration before is the sum of its blocks' parts
    newest = k > 0 ? (float)wave_sum_f64((double)part0) : 0.f;
    double ring_sum = lane == last ? (double)newest : (double)ring0;
    for (int j = lane + kWave; j < s.d_max; j += kWave) ring_sum += (double)(j == last ? newest : s.ring[j]);
    ring_sum = wave_sum_f64(ring_sum);
    rhs = (s.c / (double)s.d_max) * ring_sum;
#pragma unroll
    for (int i = 0; i < CW; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (WC == 1) {
          th[i][e] = e >= dup[i] ? sum_s[jb[i] + e] : 0.f;
          dd[i][e] = e >= dup[i] ? sum_s[ps + jb[i] + e] : 0.f;
        }
        g[i][e] = iv[i][e] = 0.f;
      }
    if (tid < nr) y_s[tid] = label;
    lds_sync();
    while (b < nr) {                                   // (WC > 1: the same trip count in every wavefront)
      if (b + RB * NG < nr) load(x[1], b + RB * NG);
      work(x[0], b, it);
      b += RB * NG; ++it;
      if (b >= nr) break;
      if (b + RB * NG < nr) load(x[0], b + RB * NG);
      work(x[1], b, it);
      b += RB * NG; ++it;
    }
  }
  // the sums over the share: through LDS, four columns per thread from here on.  (The last quad may reach past p: it reads
  // up to three floats of what follows an array in the workspace and drops them.)
#pragma unroll
  for (int i = 0; i < CW; ++i)
    if (dup[i] == 0) {
      *reinterpret_cast<v4s *>(sum_s + (grp * 2) * ps + jb[i]) = v4s{g[i][0], g[i][1], g[i][2], g[i][3]};
      *reinterpret_cast<v4s *>(sum_s + (grp * 2 + 1) * ps + jb[i]) = v4s{iv[i][0], iv[i][1], iv[i][2], iv[i][3]};
    } else {
#pragma unroll
      for (int e = 1; e < 4; ++e)
        if (e >= dup[i]) { sum_s[(grp * 2) * ps + jb[i] + e] = g[i][e]; sum_s[(grp * 2 + 1) * ps + jb[i] + e] = iv[i][e]; }
    }
  lds_sync();
  auto share_sums = [&](int j, v4s &gs, v4s &is) __attribute__((always_inline)) {
    gs = is = v4s{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < NG; ++q) { gs += *reinterpret_cast<const v4s *>(sum_s + q * 2 * ps + j); is += *reinterpret_cast<const v4s *>(sum_s + (q * 2 + 1) * ps + j); }
  };
  const __amdgpu_buffer_rsrc_t part = far_buffer(a.part + (int64_t)m * a.shares * 2 * ps, (int64_t)a.shares * 2 * ps);
  if (a.shares > 1) {
    for (int j = tid * 4; j < ps; j += R_NT * 4) {
      v4s gs, is;
      share_sums(j, gs, is);
      store_far(part, (uint32_t)j * 4u, (uint32_t)(share * 2 * ps) * 4u, gs);
      store_far(part, (uint32_t)j * 4u, (uint32_t)((share * 2 + 1) * ps) * 4u, is);
    }
    if (!last_of(a.count + kCountWords * (1 + m), (uint32_t)a.shares, &flag_s)) return;
  }
  const int cur = s.sel[m];
  const __amdgpu_buffer_rsrc_t fresh = far_buffer(s.gbuf + (int64_t)(1 - cur) * mp + (int64_t)m * s.p, s.p);
  double sq = 0.0;                                     // (four terms at a time in float32, their sums in double: the rule compares in double)
  for (int j = tid * 4; j < ps; j += R_NT * 4) {
    const int64_t o = (int64_t)m * s.p + j, of = (int64_t)(1 - cur) * mp + o, oc = (int64_t)cur * mp + o;
    const v4u t4 = *reinterpret_cast<const v4u *>(s.theta + j), l4 = *reinterpret_cast<const v4u *>(s.theta_lo + j);
    const v4u rh = *reinterpret_cast<const v4u *>(ref.hi + j), rl = *reinterpret_cast<const v4u *>(ref.lo + j);
    v4u st = {0.f, 0.f, 0.f, 0.f};                     // CADA1: the stored innovation; LAG, always: the stored gradient
    if (rule == CADA_RULE_CADA1) st = *reinterpret_cast<const v4u *>(s.dtl + oc);
    else if (rule != CADA_RULE_CADA2) st = *reinterpret_cast<const v4u *>(s.gbuf + oc);
    v4s gs, is;
    if (a.shares > 1) {
      gs = is = v4s{0.f, 0.f, 0.f, 0.f};
      for (int q0 = 0; q0 < a.shares; q0 += 4) {
        v4s x[4], y[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {                  // (past the last share: that one again, dropped)
          const int at = min(q0 + q, a.shares - 1) * 2 * ps;
          x[q] = load_far(part, (uint32_t)j * 4u, (uint32_t)at * 4u);
          y[q] = load_far(part, (uint32_t)j * 4u, (uint32_t)(at + ps) * 4u);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (q0 + q < a.shares) { gs += x[q]; is += y[q]; }
      }
    } else {
      share_sums(j, gs, is);
    }
    float sq4 = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      gs[e] = fmaf(s.lam, t4[e], gs[e]);
      is[e] = fmaf(s.lam, (t4[e] - rh[e]) + (l4[e] - rl[e]), is[e]);
      const float term = rule == CADA_RULE_CADA2 ? is[e] : (rule == CADA_RULE_CADA1 ? is[e] : gs[e]) - st[e];
      if (j + e < p) sq4 = fmaf(term, term, sq4);
    }
    sq += (double)sq4;
    if (j + 4 <= p) {
      store_far(fresh, (uint32_t)j * 4u, 0u, gs);
      if (rule == CADA_RULE_CADA1) *reinterpret_cast<v4u *>(s.dtl + of) = is;
    } else {
      for (int e = 0; j + e < p; ++e) {
        put_far(s.gbuf + of + e, gs[e]);
        if (rule == CADA_RULE_CADA1) s.dtl[of + e] = is[e];
      }
    }
  }
  sq = wave_sum_f64(sq);
  if (lane == 0) red_l[w] = sq;
  lds_sync();
  uint64_t *lhs_far = reinterpret_cast<uint64_t *>(s.lhs_part);      // [M] two floats whose sum is the left-hand side (n_lhs_part = 2; room for eight)
  if (tid == 0) {
    double l = red_l[0];
#pragma unroll
    for (int i = 1; i < R_NW; ++i) l += red_l[i];
    const float hi = (float)l, lo = isinf(hi) ? 0.f : (float)(l - (double)hi);
    put_far(lhs_far + m, ((uint64_t)__float_as_uint(lo) << 32) | __float_as_uint(hi));
    up_s = 0u;
  }
  if constexpr (std::is_same_v<Args, RowsInArgs>) {
    const RuleInputs ri = a.ri;
    if (m == 0) {                                      // (one workgroup comes here for each worker; M <= R_NT) the rule's inputs for the server's launch
      if (tid < M) { ri.in[tid] = tau0; ri.in[M + tid] = sel0; }
      if (tid == 0) {
        *ri.rhs = rhs;
        if (last >= 0) s.ring[last] = newest;          // (others read this slot too, and put their own sum in its place)
      }
    }
    return;
  }
  if (a.tail == kTailNone) return;
  if (!last_of(a.count, (uint32_t)M, &flag_s)) return;

  // ---- the rule for all workers (last workgroup of the launch)
  uint32_t ups = 0;
  uint8_t *sel_s = reinterpret_cast<uint8_t *>(rows_smem);       // [M], in place of what came before (every wavefront is past it)
  for (int mm = tid; mm < M; mm += R_NT) {
    const uint64_t l2 = get_far(lhs_far + mm);
    const double lhs = (double)__uint_as_float((uint32_t)l2) + (double)__uint_as_float((uint32_t)(l2 >> 32));
    const int32_t tau = mm == tid ? tau0 : s.tau[mm], was = mm == tid ? sel0 : s.sel[mm];
    const int32_t replay = mm == tid ? rep0 : a.replay != nullptr ? (int32_t)a.replay[mm] : CADA_REPLAY_FREE;
    const bool own = (rule == CADA_RULE_ALWAYS) || (lhs > rhs) || (tau >= s.D);
    bool up = own;
    if (replay != CADA_REPLAY_FREE) up = replay != 0;
    if (k < s.trace_steps) {
      const int64_t o = k * M + mm;
      s.t_mask[o] = up ? 1 : 0;
      s.t_own[o] = own ? 1 : 0;
      s.t_lhs[o] = (float)lhs;
      s.t_tau[o] = tau;
    }
    s.lhs[mm] = (float)lhs;
    s.mask[mm] = up ? 1 : 0;
    s.tau[mm] = up ? 1 : tau + 1;
    const int sel = up ? was ^ 1 : was;    // an upload: the fresh row becomes the stored one
    if (a.tail == kTailServer) sel_s[mm] = (uint8_t)sel;
    if (up) { s.sel[mm] = sel; ++ups; }
    else if (rule == CADA_RULE_CADA2 && tau >= s.D) atomicOr(s.err, 8u);   // (only a replay mask can do this)
  }
  if (ups) atomicAdd(&up_s, ups);
  // the server's operands, asked for before the rows of the aggregate
  float h0[2], vh0[2], th0[2], tl0[2];
  if (a.tail == kTailServer) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int j = min(tid + u * R_NT, p - 1);
      h0[u] = s.h[j]; vh0[u] = s.vhat[j]; th0[u] = s.theta[j]; tl0[u] = s.theta_lo[j];
    }
  }
  lds_sync();
  if (tid == 0) {
    atomicAdd(reinterpret_cast<unsigned long long *>(s.uploads), (unsigned long long)up_s);
    s.n_up[k & 1] = up_s;
    if (last >= 0) s.ring[last] = newest;
    if (k < s.trace_steps) s.t_rhs[k] = (float)rhs;
  }
  if (a.tail != kTailServer) return;

  // ---- the server update: sums of four coordinates per thread, then one coordinate per thread (as in cada_logreg_small.hip)
  float *nab_s = reinterpret_cast<float *>(rows_smem + ((M + 15) & ~15));      // [p rounded up to 4]
  const __amdgpu_buffer_rsrc_t store = far_buffer(s.gbuf, 2 * mp);      // (M p <= kServerState)
  for (int j = tid * 4; j < ps; j += R_NT * 4) {
    v4s nab = {0.f, 0.f, 0.f, 0.f};
    for (int m0 = 0; m0 < M; m0 += 16) {               // sixteen rows asked for before the first is added
      v4s v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int mm = min(m0 + q, M - 1);
        v[q] = load_far(store, (uint32_t)j * 4u, __builtin_amdgcn_readfirstlane((uint32_t)(((int64_t)sel_s[mm] * mp + (int64_t)mm * s.p) * 4)));
      }
#pragma unroll
      for (int q = 0; q < 16; ++q)
        if (m0 + q < M) nab += v[q];
    }
    *reinterpret_cast<v4s *>(nab_s + j) = nab;
  }
  lds_sync();
  double sqs = 0.0;
  for (int j = tid; j < p; j += R_NT) {
    const float nab = nab_s[j] / (float)M;
    const bool first = j < R_NT;                         // (p <= kServerColumns)
    float hh = first ? h0[0] : h0[1], vh = first ? vh0[0] : vh0[1], t = first ? th0[0] : th0[1], tl = first ? tl0[0] : tl0[1], vv;
    const float step = server_coordinate(s, s.alpha, nab, hh, vh, vv, t, tl);
    sqs = fma((double)step, (double)step, sqs);
    s.nabla[j] = nab; s.h[j] = hh; s.v[j] = vv; s.vhat[j] = vh; s.theta[j] = t; s.theta_lo[j] = tl;
    if (rule == CADA_RULE_CADA2) {
      const int64_t o = (int64_t)(s.kR + 1 == s.R ? 0 : s.kR + 1) * s.ps + j;
      s.hist[o] = t;
      s.hist_lo[o] = tl;
    } else if (s.snap_next) {
      s.snap[j] = t;
      s.snap_lo[j] = tl;
    }
  }
  sqs = wave_sum_f64(sqs);
  lds_sync();                                          // (red_l has been read)
  if (lane == 0) red_l[w] = sqs;
  lds_sync();
  if (tid < s.n_ring_part) {
    double l = red_l[0];
#pragma unroll
    for (int i = 1; i < R_NW; ++i) l += red_l[i];
    s.ring_part[tid] = tid == 0 ? (float)l : 0.f;
  }
}

// Rows of more than 8192 columns: a workgroup still takes whole rows (z and dz need no other workgroup, hence no cooperative launch and
// no exchange, which cost the cluster kernel of cada_logreg_fused.hip some 50 us per step whatever the size), CW quads of each per lane.
// What bounds it: HBM, at 5.9 TB/s in long shares, and some 7 us of operands and sums at the two ends (a CU takes 64 bytes per cycle: 320 KB of theta,
// theta_lo and the reference point for 20480 columns are 2.5 us).  Measured per step, two passes or the cluster
// kernel in place of these launches: M = 37, B = 75, p = 20001, CADA1: 117 -> 62 us; M = 8, B = 256, p = 8196: 117 -> 35;
// M = 100, B = 256, p = 20480 (2.1 GB of rows): 391 -> 356.  Rows without the non-temporal hint, the last of these: 433 (387 with it then).
// The operands' latency is paid once: asked for piece by piece as the registers of the piece before fell free (with 28 to 40 bytes of them spilled, whose
// reloads drained the rows in flight), p = 20001: 73.8 us, now 66.3; p = 12001: 57.5, 48.6; p = 20480, M = 100, B = 256: 381, 356.
// All workers' rows, one after the other, are cut into one share per workgroup (wide_split); a share that crosses from one worker to
// the next starts new sums there (wide_slot), and k_rows_sum adds a worker's slots up, one block per 1024 columns.  RB rows are worked on together, and the next RB asked for when
// these have landed.  (Two batches in flight, a batch's registers asked for again right after its products: the rows of all CUs then share the memory and the one that is waited
// for comes later: p = 20001: 69.4 us for 66.3, p = 15000, M = 100, B = 64: 96.4 for 88.1, p = 20480, M = 100, B = 256: 355 for 356.)
// DL: theta - theta_ref lies in LDS (the registers of 512 threads hold four vectors of 20480 columns and the rows in flight, not
// five).  SEG: shares may meet several workers (up to 14336 columns: the loop over them costs wider rows registers, 51 -> 59 us).
// dynamic LDS: row offsets int64 [rows], labels [rows] (rounded up to four rows), with DL theta - theta_ref [CW][512] quads
template <int CW, int RB, bool DL, bool SEG>
__global__ __launch_bounds__(R_NT) void k_rows_wide(const RowsArgs a) {
  extern __shared__ __align__(16) unsigned char rows_smem[];
  const DevState &s = a.s;
  const int p = (int)s.p, ps = (p + 3) & ~3;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int64_t *off_s = reinterpret_cast<int64_t *>(rows_smem);
  float *y_s = reinterpret_cast<float *>(off_s + ((a.rows + 3) & ~3));
  v4s *d_s = reinterpret_cast<v4s *>(y_s + ((a.rows + 3) & ~3));
  constexpr int NV = 2 * RB;
  __shared__ float red_s[2][R_NW][NV];

  const int f0 = wide_first(a.wide, blockIdx.x), nr = wide_first(a.wide, blockIdx.x + 1) - f0;        // this share's rows
  // Everything that depends on nothing is asked for at once: this thread's sampled row and its worker's first row, theta, theta_lo, the reference point.
  struct Sample { int64_t base, n; int32_t r; };
  auto ask_row = [&](int b) __attribute__((always_inline)) {
    const int m = (f0 + b) / s.B;
    return Sample{s.row_off[m], s.row_off[m + 1], a.idx[f0 + b]};
  };
  auto row_of = [&](int b, const Sample &x) __attribute__((always_inline)) {          // global row of the share's b-th
    const int64_t n_m = x.n - x.base;
    int64_t r = x.r;
    if (r < 0 || r >= n_m) { atomicOr(s.err, 1u); r = r < 0 ? 0 : n_m - 1; }
    off_s[b] = (x.base + r) * s.p;
    return x.base + r;
  };
  const Sample first = ask_row(min(tid, nr - 1));
  auto delay_of = [&](int m) __attribute__((always_inline)) { return s.rule == CADA_RULE_CADA2 ? s.tau[m] : 0; };
  const int m_first = __builtin_amdgcn_readfirstlane(f0 / s.B);
  const int32_t tau_first = delay_of(m_first);
  // columns as in k_rows: the quad that would reach past p ends at p, its first `dup` columns belong to the quad before
  // (buffer accesses: a uniform base and a 32-bit byte offset per lane, formed where it is used; as global accesses the compiled kernel kept
  // 64-bit offsets of all pieces and spilled)
  const uint32_t j_most = (uint32_t)(p - 4) * 4u;
  auto here = [&]() __attribute__((always_inline)) { int ln = lane; asm volatile("" : "+v"(ln)); return (uint32_t)(w * CW * kWave + ln) * 16u; };
  const uint32_t jl = here();
  auto piece = [&](uint32_t j, int i) __attribute__((always_inline)) { return min(j + (uint32_t)i * (16u * kWave), j_most); };
  auto vec = [&](const float *x) __attribute__((always_inline)) { return far_buffer(const_cast<float *>(x), p); };
  auto quad = [](__amdgpu_buffer_rsrc_t x, uint32_t off) __attribute__((always_inline)) { return __builtin_bit_cast(v4s, __builtin_amdgcn_raw_buffer_load_b128(x, off, 0, 0)); };
  constexpr int kNt = 2;                               // the non-temporal bit of a buffer access
  float th[CW][4], dd[DL ? 1 : CW][4], g[CW][4], iv[CW][4];
  v4s x0[RB][CW], x1[RB][CW], lo[CW], rh[CW], rl[CW];
  // theta_lo and the reference point of a worker, all asked for before the first is used, and before the rows: behind the first batch their data wait
  // for its latency (p = 18000, M = 16, B = 64: 40.0 us for 39.2, and no better with half of them in front)
  auto ask_operands = [&](int32_t tau) __attribute__((always_inline)) {
    const RefPtr ref = theta_ref_at(s, tau);
    const uint32_t j = here();
#pragma unroll
    for (int i = 0; i < CW; ++i) { lo[i] = quad(vec(s.theta_lo), piece(j, i)); rh[i] = quad(vec(ref.hi), piece(j, i)); rl[i] = quad(vec(ref.lo), piece(j, i)); }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int i = 0; i < CW; ++i) {
    const v4s t4 = quad(vec(s.theta), piece(jl, i));
#pragma unroll
    for (int e = 0; e < 4; ++e) th[i][e] = t4[e];      // (zero in the columns of another quad: see below)
  }
  // (labels are asked for behind the rows' offsets and put into LDS behind the first rows' loads: the products' barriers stand between that and their use)
  ask_operands(__builtin_amdgcn_readfirstlane(tau_first));
  int64_t row0 = first.base;
  if (tid < nr) row0 = row_of(tid, first);
  for (int b = tid + R_NT; b < nr; b += R_NT) y_s[b] = static_cast<const float *>(s.y)[row_of(b, ask_row(b))];
  const float label = static_cast<const float *>(s.y)[row0];
  lds_sync();
  int seg = 0, end;                                    // rows of the worker that is worked on
  auto load = [&](v4s (&xb)[RB][CW], int b0) __attribute__((always_inline)) {      // rows b0 .. b0 + RB - 1 (past the end: zeros, of a buffer without bytes)
    const uint32_t j = here();
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      const int64_t o = off_s[min(b0 + q, end - 1)];
      const float *row = s.X + (((int64_t)__builtin_amdgcn_readfirstlane((uint32_t)(o >> 32)) << 32) | __builtin_amdgcn_readfirstlane((uint32_t)o));
#pragma unroll
      for (int i = 0; i < CW; ++i) xb[q][i] = __builtin_bit_cast(v4s, __builtin_amdgcn_raw_buffer_load_b128(far_buffer(const_cast<float *>(row), b0 + q < end ? p : 0), piece(j, i), 0, kNt));
    }
  };
  const float invB = 1.0f / (float)s.B;
  auto work = [&](v4s (&xb)[RB][CW], int b0, int it) __attribute__((always_inline)) {
    int ln = lane;
    asm volatile("" : "+v"(ln));                       // (what follows from it is formed here each time: registers)
    float zd[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) zd[q] = 0.f;
#pragma unroll
    for (int i = 0; i < CW; ++i) {
      v4s d4;
      if (CW >= 10 && i > 0 && i % 3 == 0) __builtin_amdgcn_sched_barrier(0);      // (three quads of the difference at a time: registers)
      if constexpr (DL) d4 = d_s[i * R_NT + w * kWave + ln];
      else d4 = v4s{dd[i][0], dd[i][1], dd[i][2], dd[i][3]};
#pragma unroll
      for (int q = 0; q < RB; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) { zd[2 * q] = fmaf(xb[q][i][e], th[i][e], zd[2 * q]); zd[2 * q + 1] = fmaf(xb[q][i][e], d4[e], zd[2 * q + 1]); }
    }
    float mine = row_sums<NV>(zd, ln);
    const int v = row_sums_index<NV>(ln);
    if (row_sums_owner<NV>(ln)) red_s[it & 1][w][v] = mine;
    lds_sync();
    mine = 0.f;
#pragma unroll
    for (int i = 0; i < R_NW; ++i) mine += red_s[it & 1][i][v];
    const float other = dpp_of<0xB1>(mine);
    const bool odd = ln & 1;
    const int b = b0 + (v >> 1);
    const float z = odd ? other : mine, dz = odd ? mine : other;
    const float y = y_s[min(b, end - 1)];
    const float aa = -y * z, bb = aa + y * dz;
    const float sg = sigmoid_r(odd ? -bb : aa);        // even lanes sigma(aa), odd lanes sigma(-bb)
    const float so = dpp_of<0xB1>(sg), em = expm1f(y * dz);
    const float r = b < end ? (odd ? y * so * sg * em * invB : -y * sg * invB) : 0.f;      // even lanes r, odd lanes dr
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      const float rr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r), row_sums_lane<NV>(2 * q)));
      const float dr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r), row_sums_lane<NV>(2 * q + 1)));
#pragma unroll
      for (int i = 0; i < CW; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) { g[i][e] = fmaf(rr, xb[q][i][e], g[i][e]); iv[i][e] = fmaf(dr, xb[q][i][e], iv[i][e]); }
    }
  };
  int it = 0;
  do {
    const int m = __builtin_amdgcn_readfirstlane((f0 + seg) / s.B);
    end = min(nr, (m + 1) * s.B - f0);
    int b = seg;
    load(x0, b);
    if (seg == 0 && tid < nr) y_s[tid] = label;
    uint32_t j = here();
#pragma unroll
    for (int i = 0; i < CW; ++i) {
      const int dup = (int)(j + (uint32_t)i * (16u * kWave) - piece(j, i)) >> 2;
      v4s d4;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        d4[e] = e >= dup ? (th[i][e] - rh[i][e]) + (lo[i][e] - rl[i][e]) : 0.f;
        if (e < dup) th[i][e] = 0.f;
        if constexpr (!DL) dd[i][e] = d4[e];
        g[i][e] = iv[i][e] = 0.f;
      }
      if constexpr (DL) d_s[i * R_NT + tid] = d4;              // (read back by this lane only)
    }
    // (no branch around the loads: their registers then stay in place)
    for (;; b += 2 * RB) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      load(x1, b + RB);
      work(x0, b, it++);
      load(x0, b + 2 * RB);
      if (b + RB >= end) break;
      work(x1, b + RB, it++);
      if (b + 2 * RB >= end) break;
    }
    const __amdgpu_buffer_rsrc_t pg = far_buffer(a.part + (int64_t)(SEG ? wide_slot(a.wide, blockIdx.x, m) : (int)blockIdx.x) * 2 * ps, 2 * ps);
    j = here();
#pragma unroll
    for (int i = 0; i < CW; ++i) {
      const uint32_t at = piece(j, i);
      const int dup = (int)(j + (uint32_t)i * (16u * kWave) - at) >> 2;
      if (dup == 0) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4s, v4s{g[i][0], g[i][1], g[i][2], g[i][3]}), pg, at, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4s, v4s{iv[i][0], iv[i][1], iv[i][2], iv[i][3]}), pg, at, ps * 4, 0);
      } else {
#pragma unroll
        for (int e = 1; e < 4; ++e)
          if (e >= dup) {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(g[i][e]), pg, at + 4 * e, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(iv[i][e]), pg, at + 4 * e, ps * 4, 0);
          }
      }
    }
    seg = end;
    // (the next worker's first rows may use the exchange buffer of this one's last ones, which a slower wavefront still reads)
    if (SEG && seg < nr) {
      ask_operands(__builtin_amdgcn_readfirstlane(delay_of(m + 1)));
      lds_sync();
    }
  } while (SEG && seg < nr);
}

// Adds up the shares of every worker in their order, adds the regulariser's terms, stores the fresh gradient (CADA1: and the fresh
// innovation) and the left-hand side's partial sums; one block more takes the rule's inputs down.  grid (ceil(p / 1024), M + 1): four
// columns per thread.  (The rule in the block that finishes last, up to 32 workers, cost two trips to counters, the stores' drain and the rule's own reads; in the server's launch it costs less.
// us per step so / now: p = 8193, M = 16, B = 8: 20.2 / 17.8; p = 20480, M = 4, B = 64: 29.1 / 26.7; p = 20001, M = 32: 54.7 / 50.8; p = 14000, LAG, M = 24: 36.8 / 34.0.)  (The last quad may reach past p: it reads up to three floats of what follows in the workspace and drops them.)
__global__ __launch_bounds__(kBlock) void k_rows_sum(const RowsArgs a, const RuleInputs ri) {
  __shared__ float red[4];
  __shared__ double rule_s[kBlock];
  const DevState &s = a.s;
  const int p = (int)s.p, ps = (p + 3) & ~3, m = blockIdx.y, rule = s.rule;
  if (m == s.M) {                                    // (one more row of blocks)
    if (blockIdx.x == 0) rule_inputs(s, ri, rule_s);
    return;
  }
  const int64_t mp = (int64_t)s.M * s.p;
  const int j = (blockIdx.x * kBlock + threadIdx.x) * 4;
  float sq = 0.f;
  if (j < ps) {
    const RefPtr ref = theta_ref(s, m);
    const int cur = s.sel[m];
    const int64_t o = (int64_t)m * s.p + j, of = (int64_t)(1 - cur) * mp + o, oc = (int64_t)cur * mp + o;
    const v4u t4 = *reinterpret_cast<const v4u *>(s.theta + j), l4 = *reinterpret_cast<const v4u *>(s.theta_lo + j);
    const v4u rh = *reinterpret_cast<const v4u *>(ref.hi + j), rl = *reinterpret_cast<const v4u *>(ref.lo + j);
    v4u st = {0.f, 0.f, 0.f, 0.f};                     // CADA1: the stored innovation; LAG, always: the stored gradient
    if (rule == CADA_RULE_CADA1) st = *reinterpret_cast<const v4u *>(s.dtl + oc);
    else if (rule != CADA_RULE_CADA2) st = *reinterpret_cast<const v4u *>(s.gbuf + oc);
    const int c0 = wide_share(a.wide, m * s.B), shares = wide_share(a.wide, (m + 1) * s.B - 1) - c0 + 1;
    const float *pg = a.part + (int64_t)wide_slot(a.wide, c0, m) * 2 * ps + j;
    v4s gs = {0.f, 0.f, 0.f, 0.f}, is = gs;
    for (int q0 = 0; q0 < shares; q0 += 8) {         // eight shares asked for before the first is added
      v4s x[8], y[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float *f = pg + (int64_t)min(q0 + q, shares - 1) * 2 * ps;
        x[q] = *reinterpret_cast<const v4s *>(f);
        y[q] = *reinterpret_cast<const v4s *>(f + ps);
      }
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (q0 + q < shares) { gs += x[q]; is += y[q]; }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      gs[e] = fmaf(s.lam, t4[e], gs[e]);
      is[e] = fmaf(s.lam, (t4[e] - rh[e]) + (l4[e] - rl[e]), is[e]);
      const float term = rule == CADA_RULE_CADA2 ? is[e] : (rule == CADA_RULE_CADA1 ? is[e] : gs[e]) - st[e];
      if (j + e < p) sq = fmaf(term, term, sq);
    }
    if (j + 4 <= p) {
      *reinterpret_cast<v4u *>(s.gbuf + of) = gs;
      if (rule == CADA_RULE_CADA1) *reinterpret_cast<v4u *>(s.dtl + of) = is;
    } else {
      for (int e = 0; j + e < p; ++e) {
        s.gbuf[of + e] = gs[e];
        if (rule == CADA_RULE_CADA1) s.dtl[of + e] = is[e];
      }
    }
  }
  sq = block_sum_lds(sq, red);
  if (threadIdx.x == 0) s.lhs_part[(int64_t)m * s.n_lhs_part + blockIdx.x] = sq;
}

namespace {
using RowsKernel = void (*)(const RowsArgs);
using RowsInKernel = void (*)(const RowsInArgs);
// the variant for rows of p columns: pieces per lane, wavefronts per row, rows per batch
RowsKernel rows_kernel(int64_t p) {
  if (p <= 256) return k_rows<1, 1, 8, RowsArgs>;
  if (p <= 512) return k_rows<2, 1, 4, RowsArgs>;
  if (p <= 1024) return k_rows<4, 1, 4, RowsArgs>;
  if (p <= 2048) return k_rows<1, 8, 8, RowsArgs>;
  if (p <= 4096) return k_rows<2, 8, 4, RowsArgs>;
  return k_rows<4, 8, 2, RowsArgs>;
}
RowsInKernel rows_in_kernel(int64_t p) {
  if (p <= 256) return k_rows<1, 1, 8, RowsInArgs>;
  if (p <= 512) return k_rows<2, 1, 4, RowsInArgs>;
  if (p <= 1024) return k_rows<4, 1, 4, RowsInArgs>;
  if (p <= 2048) return k_rows<1, 8, 8, RowsInArgs>;
  if (p <= 4096) return k_rows<2, 8, 4, RowsInArgs>;
  return k_rows<4, 8, 2, RowsInArgs>;
}
RowsKernel wide_kernel(int64_t p) {
  if (p <= 5 * 2048) return k_rows_wide<5, 2, false, true>;
  if (p <= 6 * 2048) return k_rows_wide<6, 2, false, true>;
  if (p <= 7 * 2048) return k_rows_wide<7, 1, false, true>;
  if (p <= 8 * 2048) return k_rows_wide<8, 1, true, false>;
  if (p <= 9 * 2048) return k_rows_wide<9, 1, true, false>;
  return k_rows_wide<10, 1, true, false>;
}
}  // namespace

bool rows_serves(const cada_config *cfg) {
  return cfg->model == CADA_MODEL_LOGREG && cfg->path != CADA_PATH_TWO_PASS && cfg->p >= 4 && cfg->p <= kRowsWidest &&
         (cfg->p <= 8192 || (int64_t)cfg->M * cfg->B < (1ll << 31) - 1);
}
size_t rows_part_floats(const cada_config *cfg) {
  if (!rows_serves(cfg)) return 0;
  const size_t ps = (size_t)((cfg->p + 3) / 4 * 4);
  if (cfg->p > 8192) return (size_t)wide_slots(wide_split(cfg->M, cfg->B, cfg->p)) * 2 * ps;
  const int shares = rows_split(cfg->M, cfg->B, cfg->p).shares;
  return shares > 1 ? (size_t)cfg->M * shares * 2 * ps : 0;
}

bool rows_better(const Ctx *c, const cada_config *cfg) { return rows_serves(cfg) && rows_preferred(cfg->M, cfg->B, cfg->p, c->vec); }

bool rows_plan(Ctx *c, const cada_config *cfg) {
  c->rows = 0;
  const bool wide = cfg->p > 8192;
  const size_t ps = (size_t)((cfg->p + 3) / 4 * 4);
  int wc;
  c->rows_tail = !wide && cfg->M <= kRuleWorkers ? kTailRule : kTailNone;
  RowsKernel fn;
  if (wide) {
    const WideSplit w = wide_split(cfg->M, cfg->B, cfg->p);
    c->rows_shares = w.shares; c->rows_per_share = w.rows; c->rows_per_worker = w.per;
    fn = wide_kernel(cfg->p);
    c->rows_lds = (size_t)((c->rows_per_share + 3) & ~3) * 12 + (cfg->p > 7 * 2048 ? (size_t)((cfg->p + 2047) / 2048) * R_NT * sizeof(v4s) : 0);
  } else {
    const RowsSplit r = rows_split(cfg->M, cfg->B, cfg->p);
    c->rows_shares = r.shares; c->rows_per_share = r.rows;
    if (cfg->p <= kServerColumns && cfg->M <= kServerWorkers && (int64_t)cfg->M * cfg->p <= kServerState) c->rows_tail = kTailServer;
    fn = rows_kernel(cfg->p);
    wc = cfg->p <= 1024 ? 1 : 8;
    const size_t server = (size_t)((cfg->M + 15) & ~15) + ps * sizeof(float);
    c->rows_lds = (size_t)((c->rows_per_share + 3) & ~3) * 12 + (size_t)(R_NW / wc) * 2 * ps * sizeof(float);
    if (c->rows_tail == kTailServer && c->rows_lds < server) c->rows_lds = server;
  }
  for (const void *k : {reinterpret_cast<const void *>(fn), reinterpret_cast<const void *>(rows_in_kernel(cfg->p))})
    if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
  c->rows_one = c->rows_tail == kTailServer ? steps_one_kernel(cfg->p, cfg->B) : nullptr;
  if (c->rows_one && hipFuncSetAttribute(reinterpret_cast<const void *>(c->rows_one), hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024) != hipSuccess) {
    (void)hipGetLastError();
    c->rows_one = nullptr;
  }
  c->rows = wide ? 2 : 1;
  c->s.n_lhs_part = wide ? (int)((cfg->p + 1023) / 1024) : 2;
  c->n_phases = 0;
  c->phase_names[c->n_phases++] = "logreg_rows";
  if (wide || (c->rows_tail == kTailRule && cfg->M <= kRuleInServer)) decide_plan(c, c->rule_room);
  if (c->decide) c->rows_tail = kTailNone;
  if (c->rows_tail == kTailNone && !c->decide) c->phase_names[c->n_phases++] = "rule";
  if (c->rows_tail != kTailServer) c->phase_names[c->n_phases++] = c->decide ? "rule_and_server_update" : "server_update";
  return true;
}

int logreg_step_rows(Ctx *c, const int32_t *idx, const uint8_t *replay) {
  RowsArgs a;
  a.s = c->s;
  set_iteration(a.s, c->k);
  a.s.alpha = stepsize(a.s, c->k);
  a.idx = idx;
  a.replay = replay;
  a.part = c->rows_part;
  a.count = c->rows_count;
  a.shares = c->rows_shares;
  a.rows = c->rows_per_share;
  a.wide = WideSplit{c->s.M, c->s.B, c->rows_shares, c->rows_per_share, c->rows_per_worker};
  a.tail = c->rows_tail;
  prof_mark(c);
  if (c->rows_one) {
    hipLaunchKernelGGL(c->rows_one, dim3((unsigned)c->s.M), dim3(R_NT), steps_lds(c->s.p), c->stream, SmallArgs{a.s, c->rows_count, 0u, (int)((c->s.p + 3) / 4 * 4), 0, 0, nullptr},
                       SmallVar{idx, replay, c->k, 0u, 0}, phase_of(c->s, c->k));
    prof_mark(c);
    const hipError_t e1 = hipGetLastError();
    if (e1 != hipSuccess) { set_error("logistic step launch failed: %s", hipGetErrorString(e1)); return CADA_EHIP; }
    c->force_resum = 0;
    return CADA_OK;
  }
  const dim3 grid((unsigned)a.shares, c->rows == 2 ? 1u : (unsigned)c->s.M);
  if (c->rows == 1 && c->decide) hipLaunchKernelGGL(rows_in_kernel(c->s.p), grid, dim3(R_NT), c->rows_lds, c->stream, RowsInArgs{a, c->rule_in});
  else hipLaunchKernelGGL(c->rows == 2 ? wide_kernel(c->s.p) : rows_kernel(c->s.p), grid, dim3(R_NT), c->rows_lds, c->stream, a);
  if (c->rows == 2)
    hipLaunchKernelGGL(k_rows_sum, dim3((unsigned)((c->s.p + 1023) / 1024), (unsigned)c->s.M + (c->rule_in.rhs ? 1u : 0u)), dim3(kBlock), 0, c->stream, a, c->rule_in);
  prof_mark(c);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("logistic step launch failed: %s", hipGetErrorString(e)); return CADA_EHIP; }
  if (a.tail == kTailServer) { c->force_resum = 0; return CADA_OK; }
  return a.tail == kTailRule ? server_step(c) : rule_then_server(c, replay);
}

}  // namespace cada
