// Objective and accuracy of the MLP on all the data (not part of an iteration): one launch takes every row of X through
// all layers and leaves each row's loss and hit, a second adds them up per worker.  (Few rows: a launch per hidden layer, see eval_plan.)
//
// The rows of all workers lie one after the other, so the data is one matrix.  A workgroup takes RT = 64 NR of its rows at a
// time through the network: for every tile of UT = 128 NU units it sums W X^T over the inputs (split operands, three bf16 MFMA
// products, float32 accumulators as in cada_mlp.hip), eight wavefronts of 32 NU units x 32 NR rows (4 x 2).  The weights are the
// A operand, so a lane of the result holds ONE row and groups of four consecutive units: after bias and ReLU
// these registers are, as they are, the operand of the last layer's product (whose sum over the units may take them in any order, as
// long as the weights follow it).  With one hidden layer nothing but the row's loss leaves the chip; deeper networks
// pass activations on through rows of scratch that belong to the workgroup (L2-resident, never read by another).
// Operands go straight to LDS, weights one step of 32 inputs ahead of the products and rows, which come from HBM, two (one where the launch has several hidden
// layers, whose inputs are written by the launch itself), over the boundaries of unit and row tiles.
//
// What bounds it: the MFMA issue (three products per weight and row; without any loads the launch below takes 630 us, and at the 1.2 PFLOP/s
// that real operands leave the card 790), and the rows' way from HBM: 16 rows x 64 bytes a load, half a line each, of rows that start on no line.
// Measured: 784-512-10 on 384000 rows 3.48 ms as a loop over chunks of M x B rows, 0.90 with the loads of a step in one burst before its products and rows one step
// ahead, now 0.83 - 0.85 (0.31 TFLOP, executed threefold); small minibatches, whose chunks were small too, 10.8 ms -> 73 us.
// Loads in a burst at the head of a step held the wavefronts up before their first product; rows two steps ahead in such a burst gained nothing (0.88), the same loads
// among the first products 0.84 (one by one between all groups of products 0.86).  3072-1024-1024-10 on 50000 rows 2.27 -> 1.84 ms, with the weights at the head, the rows behind the
// first products and the wavefronts that multiply raised over those that wait (either alone 1.94, 2.12; the other way round 1.96).
#include <cstdlib>

#include "cada_mlp.h"

namespace cada {

struct EvalLayer {
  const bf16_t *Wh, *Wl;     // (out, in) chunks
  int64_t kt;                // chunks per 128-unit tile
  int64_t offb;
  int nk, N;                 // steps of 32 inputs, units
};

struct EvalArgs {
  DevState s;
  const bf16_t *Xh, *Xl;     // [rows][ldx]
  int64_t ldx, rows;
  const bf16_t *zeros;       // 16 bytes of zeros
  EvalLayer layer[CADA_MAX_LAYERS];
  int L, C;
  bf16_t *act[2][2];         // [layer parity][hi, lo]: activations [workgroup][RT][lda] (L >= 3)
  int64_t lda;
  float2 *rowval;            // [rows] (loss, hit)
  float *zpart;              // layer by layer: [unit tile][row_pad][32] the logits' parts from each tile of the last hidden layer's units, or
  int64_t row_pad;           //   null: this layer's activations go to act[0] by rows of X
};

// 16 bytes per lane straight to LDS (consecutive in lane order from byte `lds` on).  The compiler does not count these loads; the
// step's barrier waits for them.
__device__ __forceinline__ void to_lds(const bf16_t *g, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory", "m0");
}
__device__ __forceinline__ void to_lds(const bf16_t *base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory", "m0");
}

// HID: hidden layers (2: two or more), or kByLayer: one hidden layer a launch (layer[0]; layer[1] is the next one), one tile of its units a workgroup, or
// kFewSteps: one hidden layer of few inputs
constexpr int kByLayer = 3, kFewSteps = 4;
// Stages of rows in LDS: several hidden layers in a launch have two, as a layer's input is not there before its last step.
constexpr int eval_row_stages(int hid) { return hid == 2 || hid == kFewSteps ? 2 : 3; }
// Rows x units of 256 x 256 then leave no room for the logits.  Lent out and taken back at the end of every tile of units, the stage of weights costs some
// microseconds a row tile, which the third stage of rows earns back where a tile of units has many steps.  Where it has kFewStepsMost or fewer, k_eval_net<4, 2, kFewSteps>
// has two stages, all loads of a step at its head and the logits in room of their own.  us, two stages / three, 60000 and 250000 rows: 64-1024-32 68.5, 239 / 72, 267;
// 256-512-10 71, 237 / 73.5, 248; 512-1024-32 186, 738 / 192, 767; 640-512-10 117, 479 / 119, 473; 640-1024-32 216, 904 / 223, 912; 784-512-10 140, 603 / 139, 566;
// 1024-1024-32 332, 1430 / 334, 1393.
constexpr int kFewStepsMost = 20;
constexpr bool eval_lends(int NR, int NU, int hid) { return eval_row_stages(hid) == 3 && NR == 4 && NU == 2; }
constexpr int eval_lds(int NR, int NU, int hid) { return 64 * NR * 128 * (eval_row_stages(hid) + (eval_lends(NR, NU, hid) ? 0 : 1)) + 2 * 128 * NU * 128; }
template <int NR, int NU, int HID>
__global__ __launch_bounds__(512) void k_eval_net(const EvalArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int RT = 64 * NR, UT = 128 * NU;
  // LDS: XS stages of rows (hi, lo [RT][32]), two of weights (hi, lo [UT][32]), the logits [RT][32] (class c of row r at c ^ (r % 32)), unless they take the
  // stage of weights that is free between two tiles of units
  constexpr int XS = eval_row_stages(HID), XB = RT * 128, WB = UT * 128;
  constexpr bool LEND = eval_lends(NR, NU, HID);
  const DevState &s = a.s;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wu = w & 3, wr = w >> 2;                        // this wavefront's units and rows
  const int half = lane >> 5, l32 = lane & 31;
  const int ntiles = (int)((a.rows + RT - 1) / RT);
  const int nhid = HID != 2 ? 1 : a.L - 1;                   // products in the steps below (no hidden layer: the logits are their result)
  // A loading instruction fills 16 rows of 32 values of a tile: the lane at position `lane` fetches the piece that lds_piece puts there
  const int piece = lds_piece(lane), prow = piece >> 2, pq = piece & 3;

  // Loading cursor: (row tile, layer, unit tile, step).  Row addresses are a scalar plus this lane's part: rows past the last
  // one are read as well (from what follows X's copies in the workspace: at least 256 rows of gathered ones) and dropped.
  int ltile = blockIdx.x, ll = 0, lct = HID == kByLayer ? (int)blockIdx.y : 0, lk = 0;
  EvalLayer le = a.layer[0];
  const bf16_t *src[2];                                     // hi, lo: first row of the tile
  int64_t sld = 0;
  uint32_t xoff = 0;
  auto set_source = [&]() __attribute__((always_inline)) {
    const bool first = HID != 2 || ll == 0;
    sld = first ? a.ldx : a.lda;
    xoff = (uint32_t)(prow * (int)sld + pq * 8) * 2u;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      src[h] = first ? (h ? a.Xl : a.Xh) + (int64_t)ltile * RT * sld : a.act[(ll - 1) & 1][h] + (int64_t)blockIdx.x * RT * sld;
  };
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem_raw;
  auto load_row = [&](int stage, int i) __attribute__((always_inline)) {      // the i-th of this wavefront's NR loads of the cursor's rows
    const int id = w * NR + i, lo = id >= 4 * NR, blk = id & (4 * NR - 1);
    const bf16_t *row = (lo ? src[1] : src[0]) + (int64_t)(blk * 16) * sld + lk * 32;
    const uint32_t to = lds0 + (uint32_t)(stage * XB + id * 1024);
    if ((int64_t)lk * 32 + 32 > sld) {                      // rows of X end at a multiple of 8 values: zeros from there on
      const bf16_t *g = lk * 32 + pq * 8 < (int)sld ? reinterpret_cast<const bf16_t *>(reinterpret_cast<const char *>(row) + xoff) : a.zeros;
      to_lds(g, to);
    } else {
      to_lds(row, xoff, to);
    }
  };
  auto load_rows = [&](int stage) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NR; ++i) load_row(stage, i);
  };
  auto load_weights = [&](int stage) __attribute__((always_inline)) {
    const int last = (le.N + 127) / 128 - 1;
#pragma unroll
    for (int i = 0; i < 2 * NU; ++i) {
      const int id = w * 2 * NU + i, lo = id >= 8 * NU, blk = id & (8 * NU - 1);
      const int ut = min(lct * NU + (blk >> 3), last);      // (units past the last tile: any finite values)
      to_lds((lo ? le.Wl : le.Wh) + (((int64_t)ut * le.kt + lk) << 12) + ((blk & 7) << 9), (uint32_t)piece * 16u, lds0 + (uint32_t)(XS * XB + stage * WB + id * 1024));
    }
  };
  // next step; returns false where it is the first of a layer whose input is still being formed, or past the end
  auto advance = [&](bool &done) __attribute__((always_inline)) -> bool {
    if (++lk < le.nk) return true;
    lk = 0;
    if constexpr (HID != kByLayer) {
      if (++lct * UT < le.N) return true;
      lct = 0;
    }
    if constexpr (HID == 2) {
      if (++ll < nhid) { le = a.layer[ll]; set_source(); return false; }
      ll = 0;
      le = a.layer[0];
    }
    ltile += gridDim.x;
    if (ltile >= ntiles) { done = true; return false; }
    set_source();
    return true;
  };
  // everything has landed, or (rows of the step after the next are on their way) everything but the newest NR loads
  auto landed = [&](bool rows_behind) __attribute__((always_inline)) {
    if (rows_behind) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NR) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };

  if (ltile >= ntiles) return;
  bool done = false;
  int xs = 0, ws = 0;                                       // stages of the step that is worked on
  set_source();
  load_rows(0);
  load_weights(0);
  bool next = true;                                         // XS == 3: the cursor stands at the next step (whose rows have been asked for)
  if constexpr (XS == 3) {
    next = advance(done);
    if (next) load_rows(1);
    landed(next);
  } else {
    landed(false);
  }
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t r0 = (int64_t)tile * RT;
    float *logit_s = reinterpret_cast<float *>(smem_raw + XS * XB + 2 * WB);
    constexpr int NSUM = LEND ? RT * 32 / 512 : 1;
    float sums[NSUM];                                       // LEND: the logits between tiles of units, 512 threads apart
#pragma unroll
    for (int i = 0; i < NSUM; ++i) sums[i] = 0.f;
    for (int l = 0; l < nhid; ++l) {
      const EvalLayer e = a.layer[l];
      const int u1 = HID == kByLayer ? (int)blockIdx.y * UT : 0, u2 = HID == kByLayer ? u1 + 1 : e.N;
      for (int u0 = u1; u0 < u2; u0 += UT) {
        f32x16 acc[NU][NR];
#pragma unroll
        for (int i = 0; i < NU; ++i)
#pragma unroll
          for (int j = 0; j < NR; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
        bool ready = true;
        for (int k = 0; k < e.nk; ++k) {
          const int xn = xs + XS - 1 >= XS ? xs - 1 : xs + XS - 1;      // the stage of the rows that are asked for in this step
          if constexpr (XS != 3) {
            ready = advance(done);
            if (HID == kFewSteps && ready) load_rows(xn);
            if (ready) load_weights(ws ^ 1);
          }
          const bf16_t *sx = reinterpret_cast<const bf16_t *>(smem_raw + xs * XB) + (wr * 32 * NR) * 32;
          const bf16_t *sw = reinterpret_cast<const bf16_t *>(smem_raw + XS * XB + ws * WB) + (wu * 32 * NU) * 32;
          const int fro = lds_piece(l32 * 4 + half) * 8;
#pragma unroll
          for (int ks = 0; ks < 32; ks += 16) {
            if constexpr (HID == 2) __builtin_amdgcn_s_setprio(1);
            bf16x8 wh[NU], wl[NU], xh[NR], xl[NR];
#pragma unroll
            for (int j = 0; j < NR; ++j) {
              xh[j] = *reinterpret_cast<const bf16x8 *>(sx + j * 1024 + (fro ^ ks));
              xl[j] = *reinterpret_cast<const bf16x8 *>(sx + RT * 32 + j * 1024 + (fro ^ ks));
            }
#pragma unroll
            for (int i = 0; i < NU; ++i) {
              wh[i] = *reinterpret_cast<const bf16x8 *>(sw + i * 1024 + (fro ^ ks));
              wl[i] = *reinterpret_cast<const bf16x8 *>(sw + UT * 32 + i * 1024 + (fro ^ ks));
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) {
              if (ks == 0 && q >= 1) {
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (XS == 3) {
                  if (q == 1 && next) { load_weights(ws ^ 1); next = advance(done); }
                  if (q == 2 && next) load_rows(xn);
                } else if (HID != kFewSteps && ready) {
                  if (q == 1) load_rows(xn);
                }
                __builtin_amdgcn_sched_barrier(0);
              }
#pragma unroll
              for (int i = 0; i < NU; ++i)
#pragma unroll
                for (int j = 0; j < NR; ++j)
                  acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q == 1 ? wl[i] : wh[i], q == 0 ? xl[j] : xh[j], acc[i][j], 0, 0, 0);
            }
          }
          if constexpr (HID == 2) __builtin_amdgcn_s_setprio(0);
          landed(XS == 3 && next);
          xs = xs + 1 == XS ? 0 : xs + 1;
          ws ^= 1;
        }
        // accumulator element r of (i, j): unit ub + 32 i + 8 (r / 4) + r % 4, row 32 NR wr + 32 j + lane % 32
        const int ub = u0 + wu * 32 * NU + 4 * half;
        const int rl = wr * 32 * NR + l32;
        if constexpr (HID == 0) {
          if (wu == 0) {
#pragma unroll
            for (int j = 0; j < NR; ++j)
#pragma unroll
              for (int r = 0; r < 16; ++r) logit_s[(rl + 32 * j) * 32 + ((8 * (r >> 2) + 4 * half + (r & 3)) ^ l32)] = acc[0][j][r];
          }
          lds_sync();
        } else {
          // (one block of 32 units after the other: the registers hold the accumulators and the logits, but no more than
          // one block's biases and weights)
          float bias[16];
          const __amdgpu_buffer_rsrc_t bias_buf = __builtin_amdgcn_make_buffer_rsrc(s.theta + e.offb, 0, e.N * 4, 0x00020000);
          auto load_bias = [&](int i) __attribute__((always_inline)) {
            asm volatile("" ::: "memory");
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              const int u = ub + 32 * i + 8 * g;
              const v4s b4 = __builtin_bit_cast(v4s, __builtin_amdgcn_raw_buffer_load_b128(bias_buf, u * 4, 0, 0));      // (zero past the last unit)
#pragma unroll
              for (int q = 0; q < 4; ++q) bias[4 * g + q] = u + q < e.N ? b4[q] : -INFINITY;                    // (no such unit: its value is zero)
            }
          };
          auto value = [&](int i, int j, int r) __attribute__((always_inline)) {
            return fmaxf(acc[i][j][r] + bias[r], 0.f);
          };
          if ((HID == 2 && l + 1 < nhid) || (HID == kByLayer && a.zpart == nullptr)) {
            const int64_t at = ((HID == kByLayer ? r0 : (int64_t)blockIdx.x * RT) + rl) * a.lda + ub;
            bf16_t *dh = a.act[l & 1][0] + at, *dl = a.act[l & 1][1] + at;
            const int ld = a.layer[l + 1].nk * 32;          // (the next layer's steps read whole groups of 32)
#pragma unroll
            for (int i = 0; i < NU; ++i) {
              load_bias(i);
#pragma unroll
              for (int j = 0; j < NR; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                  float x[4];
#pragma unroll
                  for (int q = 0; q < 4; ++q) x[q] = value(i, j, 4 * g + q);
                  uint2 hi, lo;
                  hi.x = f2bf_pk(x[0], x[1]); hi.y = f2bf_pk(x[2], x[3]);
                  lo.x = f2bf_pk(x[0] - __uint_as_float(hi.x << 16), x[1] - __uint_as_float(hi.x & 0xffff0000u));
                  lo.y = f2bf_pk(x[2] - __uint_as_float(hi.y << 16), x[3] - __uint_as_float(hi.y & 0xffff0000u));
                  if (ub + 32 * i + 8 * g < ld) {
                    *reinterpret_cast<uint2 *>(dh + (int64_t)(32 * j) * a.lda + 32 * i + 8 * g) = hi;
                    *reinterpret_cast<uint2 *>(dl + (int64_t)(32 * j) * a.lda + 32 * i + 8 * g) = lo;
                  }
                }
            }
          } else {
            // the last layer's part from these units, from registers to registers: operand slots 8 half .. 8 half + 7 of a
            // product over 16 units hold units {0-3, 8-11} + 4 half, and the weights are read in that order
            const bf16_t *Vh = a.layer[a.L - 1].Wh, *Vl = a.layer[a.L - 1].Wl;
            const int vkt = (int)a.layer[a.L - 1].kt;
            f32x16 lg[NR];
#pragma unroll
            for (int j = 0; j < NR; ++j)
#pragma unroll
              for (int r = 0; r < 16; ++r) lg[j][r] = 0.f;
#pragma unroll
            for (int i = 0; i < NU; ++i) {
              load_bias(i);
              bf16x8 vh[2], vl[2];
              const int64_t o = ((int64_t)min((ub + 32 * i) >> 5, vkt - 1) << 12) + l32 * 32 + 4 * half;
#pragma unroll
              for (int q = 0; q < 2; ++q) {
                const uint2 h0 = *reinterpret_cast<const uint2 *>(Vh + o + 16 * q), h1 = *reinterpret_cast<const uint2 *>(Vh + o + 16 * q + 8);
                const uint2 l0 = *reinterpret_cast<const uint2 *>(Vl + o + 16 * q), l1 = *reinterpret_cast<const uint2 *>(Vl + o + 16 * q + 8);
                vh[q] = __builtin_bit_cast(bf16x8, u32x4{h0.x, h0.y, h1.x, h1.y});
                vl[q] = __builtin_bit_cast(bf16x8, u32x4{l0.x, l0.y, l1.x, l1.y});
              }
#pragma unroll
              for (int j = 0; j < NR; ++j) {
                __builtin_amdgcn_sched_barrier(0);           // (conversions of one block at a time: registers)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                  uint32_t hi[4], lo[4];
#pragma unroll
                  for (int b = 0; b < 4; ++b) {
                    const float x0 = value(i, j, 8 * q + 2 * b), x1 = value(i, j, 8 * q + 2 * b + 1);
                    hi[b] = f2bf_pk(x0, x1);
                    lo[b] = f2bf_pk(x0 - __uint_as_float(hi[b] << 16), x1 - __uint_as_float(hi[b] & 0xffff0000u));
                  }
                  const bf16x8 ah = __builtin_bit_cast(bf16x8, u32x4{hi[0], hi[1], hi[2], hi[3]}), al = __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], lo[2], lo[3]});
                  lg[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vh[q], al, lg[j], 0, 0, 0);
                  lg[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vl[q], ah, lg[j], 0, 0, 0);
                  lg[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vh[q], ah, lg[j], 0, 0, 0);
                }
              }
            }
            // added up over the four wavefronts of the same rows, one after the other
            if constexpr (LEND) logit_s = reinterpret_cast<float *>(smem_raw + XS * XB + (ws ^ 1) * WB);      // (the weights of the step that has just been worked on)
            if (LEND || u0 == u1) {
              for (int i = t; i < RT * 32; i += 512) logit_s[i] = 0.f;
              lds_sync();
            }
            for (int q = 0; q < 4; ++q) {
              if (wu == q) {
#pragma unroll
                for (int j = 0; j < NR; ++j)
#pragma unroll
                  for (int r = 0; r < 16; ++r) {
                    logit_s[(rl + 32 * j) * 32 + ((8 * (r >> 2) + 4 * half + (r & 3)) ^ l32)] += lg[j][r];
                  }
              }
              lds_sync();
            }
            if constexpr (LEND) {
#pragma unroll
              for (int i = 0; i < NSUM; ++i) sums[i] += logit_s[t + 512 * i];
              if (u0 + UT >= u2) {
#pragma unroll
                for (int i = 0; i < NSUM; ++i) logit_s[t + 512 * i] = sums[i];
              }
              lds_sync();
            }
          }
        }
        if (HID == 2 && !ready && !done) {       // the next layer reads what this one has just written
          landed(false);
          load_rows(xs);
          load_weights(ws);
          landed(false);
        }
      }
    }
    if constexpr (HID == kByLayer) {
      if (a.zpart != nullptr)
        for (int i = t; i < RT * 32; i += 512) a.zpart[((int64_t)blockIdx.y * a.row_pad + r0) * 32 + i] = logit_s[(i & ~31) + ((i ^ (i >> 5)) & 31)];
    } else if (t < RT && r0 + t < a.rows) {
      const int64_t r = r0 + t;
      const int label = static_cast<const int32_t *>(s.y)[r];
      const float *bl = s.theta + a.layer[a.L - 1].offb;
      auto z = [&](int c) __attribute__((always_inline)) { return logit_s[t * 32 + (c ^ (t & 31))] + bl[c]; };
      float zmax = -INFINITY, zl = 0.f;
      int arg = 0;
      for (int c = 0; c < a.C; ++c) {
        const float x = z(c);
        if (x > zmax) { zmax = x; arg = c; }
        if (c == label) zl = x;
      }
      float den = 0.f;
      for (int c = 0; c < a.C; ++c) den += expf(z(c) - zmax);
      a.rowval[r] = make_float2(zmax + logf(den) - zl, arg == label ? 1.f : 0.f);
    }
    if constexpr (LEND) lds_sync();                         // (the next tile's first step loads weights to where they lie)
    // (else the next write of the logits is a barrier away)
  }
}

// A row's loss and hit from the parts of its logits, added up in order: 32 lanes a row, one a class.
__global__ __launch_bounds__(kBlock) void k_eval_rows(const EvalArgs a, int parts) {
  const int c = threadIdx.x & 31, half = threadIdx.x & 32;      // (two rows a wavefront)
  const int64_t r = (int64_t)blockIdx.x * (kBlock / 32) + (threadIdx.x >> 5);
  if (r >= a.rows) return;                                      // (whole rows of lanes)
  const bool live = c < a.C;
  float z = 0.f;
  for (int i = 0; i < parts; ++i) z += a.zpart[((int64_t)i * a.row_pad + r) * 32 + c];
  if (live) z += a.s.theta[a.layer[1].offb + c];
  float zmax = live ? z : -INFINITY;
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, o, 32));
  const uint32_t at = (uint32_t)(__ballot(live && z == zmax) >> half);
  const int arg = at ? __ffs(at) - 1 : 0, label = static_cast<const int32_t *>(a.s.y)[r];
  float den = live ? expf(z - zmax) : 0.f;
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) den += __shfl_xor(den, o, 32);
  const float zl = __shfl(z, label & 31, 32);
  if (c == 0) a.rowval[r] = make_float2(zmax + logf(den) - (label >= 0 && label < a.C ? zl : 0.f), arg == label ? 1.f : 0.f);
}

// acc[m] = (mean loss, mean accuracy) of worker m's rows, added up in a fixed order.  One block per worker.
__global__ __launch_bounds__(1024) void k_eval_sums(const DevState s, const float2 *rowval, double *acc) {
  __shared__ double red[1024][2];
  const int m = blockIdx.x, t = threadIdx.x;
  const int64_t r0 = s.row_off[m], n = s.row_off[m + 1] - r0;
  double loss = 0.0, hits = 0.0;
  for (int64_t r = t; r < n; r += 1024) { const float2 v = rowval[r0 + r]; loss += (double)v.x; hits += (double)v.y; }
  red[t][0] = loss; red[t][1] = hits;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if (t < o) { red[t][0] += red[t + o][0]; red[t][1] += red[t + o][1]; }
    __syncthreads();
  }
  if (t < 2) acc[2 * m + t] = red[0][t] / (double)n;
}

namespace {
using EvalKernel = void (*)(const EvalArgs);
constexpr int kEvalGroups = 256;        // workgroups of a launch (one per CU) at most
template <int NU, int HID> EvalKernel eval_kernel_of(int NR) { return NR == 4 ? k_eval_net<4, NU, HID> : NR == 2 ? k_eval_net<2, NU, HID> : k_eval_net<1, NU, HID>; }
struct EvalPlan {
  int nr, nu;                // rows (64 nr) and units (128 nu) of a tile
  bool by_layer;             // a launch per hidden layer
};
bool eval_few_steps(const EvalPlan &e, const MlpPlan &P) { return P.L == 2 && !e.by_layer && e.nr == 4 && e.nu == 2 && (P.d[0] + 31) / 32 <= kFewStepsMost; }
EvalKernel eval_kernel(const EvalPlan &e, const MlpPlan &P) {
  const int L = P.L;
  if (eval_few_steps(e, P)) return k_eval_net<4, 2, kFewSteps>;
  if (e.by_layer) {
    if (e.nu == 2) return e.nr == 2 ? k_eval_net<2, 2, kByLayer> : k_eval_net<1, 2, kByLayer>;
    return eval_kernel_of<1, kByLayer>(e.nr);
  }
  if (L == 1) return eval_kernel_of<1, 0>(e.nr);             // (at most 32 classes)
  if (L == 2) return e.nu == 2 ? eval_kernel_of<2, 1>(e.nr) : eval_kernel_of<1, 1>(e.nr);
  if (e.nu == 2) return e.nr == 2 ? k_eval_net<2, 2, 2> : k_eval_net<1, 2, 2>;
  return eval_kernel_of<1, 2>(e.nr);
}

int eval_hid(const EvalPlan &e, const MlpPlan &P) { return eval_few_steps(e, P) ? kFewSteps : e.by_layer ? kByLayer : min(P.L - 1, 2); }

int64_t eval_row_tiles(const MlpPlan &P, int nr) { return (P.total_rows + 64 * nr - 1) / (64 * nr); }
int eval_unit_tiles(const MlpPlan &P, int l, int nu) { return (int)((P.d[l] + 128 * nu - 1) / (128 * nu)); }

// In cycles of a step a wavefront pair issues 2 x 3 x 2 x 32 per 32 x 32 block; 256 units
// x 64 rows and 128 units x any rows wait for their operands instead (8 KB per 64 rows and 128 units at some 40 bytes per clock).
int64_t eval_step(int r, int u) { return max(384 * u * r, 8192 * (u + 1 + r) / 40 + 200); }
// One tile of 128 u units of layer l.
int64_t eval_tile(const MlpPlan &P, int l, int r, int u) { return (P.d[l - 1] + 31) / 32 * eval_step(r, u) + 2500; }
// Bytes of layer l's input, read once for every tile of units, over the chip's rate.
int64_t eval_reads(const MlpPlan &P, int l, int u) { return P.total_rows * eval_unit_tiles(P, l, u) * P.d[l - 1] * 4 / 5000; }

// One launch takes a row through all layers; the choice of the tile minimises rounds of tiles over the CUs times the time of a tile.  But few
// rows leave CUs idle and pass every tile of units one after the other: there a launch per layer (some 6000 cycles each) puts the tiles
// of units side by side.  Measured, us in one launch / by layers, each with its best tile: 3072-1024-1024-10: 100 rows: 436 / 106, 5000: 439 / 164, 16000: 603 / 381, 40000:
// 1575 / 948; 784-512-10: 100: 64 / 33, 16000: 66 / 55, 40000: 114 / -; 1024-1024-32: 100: 134 / 40, 16000: 139 / 110; 100-1000-10: 16000: 46 / 44; 64-1024-32: 5000: 40 / 30; a
// network of few units: 57-193-470-12: 100: 40 / 31, 16000: 43 / 49.  The model takes the better one except near the line: 617-301-150-26, 40000 rows: 163 (136 by layers);
// 1500-700-10, 16000: 145 (132); 2000-129-7, 5000: 69 (57); 57-193-470-12, 1500: 40 (31).
EvalPlan eval_plan(const MlpPlan &P) {
  const int hidden = P.L > 1 ? P.L - 1 : 1;
  EvalPlan one{1, 1, false}, layers{1, 1, true};
  int64_t best = INT64_MAX, best_layers = INT64_MAX;
  for (int u = 1; u <= (P.L > 1 ? 2 : 1); ++u)
    for (int r = 1; r <= 4; r *= 2) {
      const int64_t tiles = eval_row_tiles(P, r);
      int64_t per = 2000, cost = 6000 * hidden + P.total_rows * eval_unit_tiles(P, hidden, u) * 256 / 2000;      // (with the end of a tile; with the logits' parts)
      for (int l = 1; l <= hidden; ++l) {
        const int64_t ut = eval_unit_tiles(P, l, u), tile = eval_tile(P, l, r, u);
        per += ut * tile;
        cost += (tiles * ut + kEvalGroups - 1) / kEvalGroups * tile + eval_reads(P, l, u);
      }
      per *= (tiles + kEvalGroups - 1) / kEvalGroups;
      const bool big = u == 2 && r == 4;      // (256 x 256 would spill registers except with one hidden layer)
      if (per < best && !(big && P.L > 2)) { best = per; one = EvalPlan{r, u, false}; }
      if (cost < best_layers && !big && tiles < kEvalGroups) { best_layers = cost; layers = EvalPlan{r, u, true}; }
    }
  return P.L > 1 && best_layers < best + eval_reads(P, 1, one.nu) ? layers : one;
}
int64_t eval_groups(const MlpPlan &P, int nr) { return min(eval_row_tiles(P, nr), (int64_t)kEvalGroups); }
int64_t eval_lda(const MlpPlan &P) {     // values per row of the activations that pass through memory (0: none do)
  int64_t w = 0;
  for (int l = 1; l <= P.L - 2; ++l) w = max(w, (int64_t)(P.d[l] + 31) / 32 * 32);
  return w;
}
int64_t eval_act_rows(const MlpPlan &P, const EvalPlan &e) { return (e.by_layer ? eval_row_tiles(P, e.nr) : eval_groups(P, e.nr)) * 64 * e.nr; }
size_t eval_rowval_bytes(const MlpPlan &P) { return ((size_t)P.total_rows * sizeof(float2) + 255) / 256 * 256; }
size_t eval_act_bytes(const MlpPlan &P, const EvalPlan &e) {
  return (size_t)eval_act_rows(P, e) * eval_lda(P) * sizeof(bf16_t) * 2 * (P.L > 3 ? 2 : 1);      // (rows of 64 and groups of 32 values: a multiple of 256 bytes)
}
}  // namespace

// Scratch of the evaluation, behind everything else in the workspace.
size_t mlp_eval_bytes(const MlpPlan &P) {
  const EvalPlan e = eval_plan(P);
  const size_t parts = e.by_layer ? (size_t)eval_unit_tiles(P, P.L - 1, e.nu) * eval_act_rows(P, e) * 32 * sizeof(float) : 0;
  return eval_rowval_bytes(P) + eval_act_bytes(P, e) + parts;
}

int mlp_eval_init(Ctx *c) {
  const MlpPlan &P = *static_cast<MlpPlan *>(c->mlp);
  const EvalPlan p = eval_plan(P);
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(eval_kernel(p, P)), hipFuncAttributeMaxDynamicSharedMemorySize, eval_lds(p.nr, p.nu, eval_hid(p, P)));
  if (e != hipSuccess) { set_error("hipFuncSetAttribute(LDS size) failed: %s", hipGetErrorString(e)); return CADA_EHIP; }
  return CADA_OK;
}

int mlp_eval(Ctx *c, double *out) {
  const MlpPlan &P = *static_cast<MlpPlan *>(c->mlp);
  const EvalPlan p = eval_plan(P);
  EvalArgs a;
  a.s = c->s;
  set_iteration(a.s, c->k);
  a.Xh = P.Xh; a.Xl = P.Xl; a.ldx = P.ldx; a.rows = P.total_rows;
  a.zeros = P.XGh + tm(0, P.ldx, P.kta[0]);      // (columns from ldx on; not read where a row fills its chunks)
  a.L = P.L; a.C = P.d[P.L];
  for (int l = 0; l < P.L; ++l) {
    a.layer[l].Wh = P.WTh + P.wt_off[l]; a.layer[l].Wl = P.WTl + P.wt_off[l]; a.layer[l].kt = P.kta[l];
    a.layer[l].offb = P.offb[l]; a.layer[l].nk = (P.d[l] + 31) / 32; a.layer[l].N = P.d[l + 1];
  }
  a.rowval = reinterpret_cast<float2 *>(P.eval);
  a.lda = eval_lda(P);
  a.zpart = nullptr;
  a.row_pad = eval_act_rows(P, p);
  const int64_t n = a.row_pad * a.lda;
  bf16_t *act = reinterpret_cast<bf16_t *>(P.eval + eval_rowval_bytes(P));
  for (int i = 0; i < 4; ++i) a.act[i >> 1][i & 1] = act + (P.L > 3 ? i : (i & 1)) * n;
  const EvalKernel kernel = eval_kernel(p, P);
  const size_t lds = eval_lds(p.nr, p.nu, eval_hid(p, P));
  mlp_stage_weights(c);
  if (p.by_layer) {
    EvalArgs b = a;
    b.L = 2;
    for (int l = 1; l < P.L; ++l) {
      const int ut = eval_unit_tiles(P, l, p.nu);
      b.layer[0] = a.layer[l - 1]; b.layer[1] = a.layer[l];
      if (l > 1) { b.Xh = a.act[l & 1][0]; b.Xl = a.act[l & 1][1]; b.ldx = a.lda; }
      b.act[0][0] = a.act[(l - 1) & 1][0]; b.act[0][1] = a.act[(l - 1) & 1][1];
      if (l == P.L - 1) b.zpart = reinterpret_cast<float *>(P.eval + eval_rowval_bytes(P) + eval_act_bytes(P, p));
      const int64_t rows = min(eval_row_tiles(P, p.nr), (int64_t)max(1, kEvalGroups / ut));
      hipLaunchKernelGGL(kernel, dim3((unsigned)rows, (unsigned)ut), dim3(512), lds, c->stream, b);
    }
    hipLaunchKernelGGL(k_eval_rows, dim3((unsigned)((P.total_rows + kBlock / 32 - 1) / (kBlock / 32))), dim3(kBlock), 0, c->stream, b, eval_unit_tiles(P, P.L - 1, p.nu));
  } else {
    hipLaunchKernelGGL(kernel, dim3((unsigned)eval_groups(P, p.nr)), dim3(512), lds, c->stream, a);
  }
  hipLaunchKernelGGL(k_eval_sums, dim3((unsigned)P.M), dim3(1024), 0, c->stream, a.s, a.rowval, c->eval_acc);
  eval_finish(c, out, 0);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("evaluation launch failed: %s", hipGetErrorString(e)); return CADA_EHIP; }
  return CADA_OK;
}

}  // namespace cada
