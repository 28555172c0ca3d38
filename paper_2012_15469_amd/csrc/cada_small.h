// What the two kernels of whole iterations share: cada_logreg_steps.hip (rows in registers) and cada_logreg_small.hip (rows in LDS: what does not fit there).
#pragma once

#include "cada_internal.h"

namespace cada {

// What does not change from launch to launch; kept in the context's workspace for the launches of several steps.
struct SmallArgs {
  DevState s;
  uint32_t *bar;             // [64]: counter of a single-step launch (first 8 bytes); then [2][M] words {tag, selector} of the last two steps
  uint32_t spin_limit;
  int ps;                    // floats from one row to the next in LDS: p rounded up to a multiple of 4
  int groups;                // row groups of the gradient pass (1, 2, 4, 8), each of all columns
  int dts;                   // the worker's stored innovation (CADA1) or gradient (LAG, always) is kept in LDS
  float *rows;               // cada_logreg_steps.hip: [kStepsTurns][M][ps], the gradients that the workers pass on
};
static_assert(sizeof(SmallArgs) <= kSmallArgsBytes && sizeof(SmallArgs) % 8 == 0, "room kept in the workspace");

// What does: schedules, iteration, tag of the first step.
struct SmallVar {
  const int32_t *idx;        // [n_steps][M][B]
  const uint8_t *replay;     // [n_steps][M] or nullptr
  int64_t k;
  uint32_t bar_base;         // sequence number of this launch's first step (monotone over the life of the context)
  int32_t turn;              // cada_logreg_steps.hip: turn of the first step of a launch of several
};
// An iteration k where a launch needs it modulo something: k mod (D + 1) (slot of the iterate history), k mod D (CADA1's snapshots), k mod d_max (ring of
// squared steps).  The host forms the first step's, the others follow: the modulo of a 64-bit k is some 130 instructions in the chain of every step.  Ten runs of 20 steps,
// M = 10, B = 10, p = 54, side by side: 141.8 -> 139.8 us, 20 steps, M = 20, B = 32, p = 784: 234.6 -> 229.5. 
struct Phase { int32_t R, D, d; };
inline Phase phase_of(const DevState &s, int64_t k) { return Phase{(int32_t)(k % s.R), (int32_t)(k % s.D), (int32_t)(k % s.d_max)}; }
__device__ __forceinline__ Phase phase_after(const DevState &s, Phase ph) {
  return Phase{ph.R + 1 == s.R ? 0 : ph.R + 1, ph.D + 1 == s.D ? 0 : ph.D + 1, ph.d + 1 == s.d_max ? 0 : ph.d + 1};
}
__device__ __forceinline__ RefPtr theta_ref_in(const DevState &s, int32_t tau_m, const Phase &ph) {       // theta_ref_at of an iteration in that phase
  if (s.rule == CADA_RULE_CADA1) return RefPtr{s.snap, s.snap_lo};
  if (s.rule != CADA_RULE_CADA2) return RefPtr{s.theta, s.theta_lo};
  int32_t slot = ph.R - min(tau_m, s.D);
  if (slot < 0) slot += s.R;
  return RefPtr{s.hist + (int64_t)slot * s.ps, s.hist_lo + (int64_t)slot * s.ps};
}
// Several independent runs (blockIdx.y picks the run) or one.
struct SmallLaunch {
  const SmallArgs *rep[CADA_MAX_REPLICAS];
  SmallVar var[CADA_MAX_REPLICAS];
  Phase ph[CADA_MAX_REPLICAS];         // of the first step
  int64_t n_steps;
};
static_assert(sizeof(SmallLaunch) <= 4096, "kernel arguments");

// The kernels of cada_logreg_steps.hip for rows of p columns, B per worker: of one step and of launches of several (null: not served).
using StepsOne = void (*)(const SmallArgs, const SmallVar, const Phase);
struct StepsKernels {
  StepsOne one;
  void (*several)(const SmallLaunch);
};
StepsKernels steps_kernels(int64_t p, int B);
StepsOne steps_one_kernel(int64_t p, int B);
constexpr int kStepsTurns = 4;
size_t steps_lds(int64_t p);

}  // namespace cada
