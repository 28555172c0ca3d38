// What the translation units of the MLP path share: operand layout and the plan of a context (cada_mlp.hip: training step,
// cada_mlp_eval.hip: evaluation).
#pragma once

#include "cada_internal.h"

namespace cada {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef uint16_t bf16_t;   // storage type
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // four floats at any 4-byte aligned address
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // 16 bytes in flight (a native vector: stays in registers)
typedef uint32_t u32x2u __attribute__((ext_vector_type(2), aligned(2)));   // four bf16 values at any address (one access: the target runs in its unaligned mode)

static inline int64_t P8(int64_t x) { return (x + 7) / 8 * 8; }

constexpr int BM = 128, BN = 128, BK = 32;
constexpr int TILE = 128 * BK;                    // bf16 elements of one chunk (8 KB)
constexpr int kMaxSlots = 4;

// Operand layout.  Every bf16 tensor a contraction reads is stored in chunks of 128 rows x 32
// contraction indices, each chunk 8 KB of consecutive memory, the chunks of a 128-row tile one
// after the other: element (r, k) of a tensor with kt chunks per row tile lies at
//     ((r / 128) * kt + k / 32) * 4096 + (r % 128) * 32 + k % 32.
// A tile step of the contraction then reads whole 128-byte lines only.  With rows stored one
// after the other a step reads a 64-byte piece of each of 128 rows, and the vector L1, which
// works line by line, delivers those at half the rate (measured from L2: 27 against 51 B/clk
// per CU), which made the loads, not the MFMAs, the longest phase of a step.  Rows and indices
// beyond a tensor's extent, up to whole chunks, exist in memory and stay zero: nothing is
// clamped or masked on the way in.
__host__ __device__ __forceinline__ int64_t tm(int64_t r, int64_t k, int64_t kt) {
  return (((r >> 7) * kt + (k >> 5)) << 12) + ((r & 127) << 5) + (k & 31);
}
static inline int tiles128(int64_t x) { return (int)((x + 127) / 128); }
// chunks per 128-row tile of a tensor with x contraction indices: whole groups of four, so that a
// 128-unit tile of the weight-gradient contractions (which take units as output rows) finds all its
// four chunks; the padding stays zero
static inline int chunks32(int64_t x) { return 4 * (int)((x + 127) / 128); }

// In LDS a chunk keeps its 8 KB (row r at byte 64 r, no padding); the four 16-byte pieces of a row
// are stored in the order q ^ ((r >> 2) & 3).  A fragment read takes one piece of each of 32
// consecutive rows; rows 4 apart lie 256 bytes = one pass over the 64 banks apart, and with this
// order the same piece of 16 consecutive rows covers every bank once.
__device__ __forceinline__ int lds_piece(int piece) {   // piece = 4 row + q  ->  position (16-byte units)
  return piece ^ ((piece >> 4) & 3);
}

struct MlpPlan {
  int L, M, B, Bp, rule, RT;
  int64_t Rp;                     // M * Bp padded rows per step (Bp a multiple of 128: a worker's rows start a tile)
  int64_t total_rows;             // rows of X
  int d[CADA_MAX_LAYERS + 1];
  int64_t offW[CADA_MAX_LAYERS], offb[CADA_MAX_LAYERS];   // offsets into theta, index l-1
  int64_t kta[CADA_MAX_LAYERS + 1];                       // chunks32(d_l): chunks per tile of (row, d_l) tensors
  int64_t wt_off[CADA_MAX_LAYERS], wt_total;              // W_l^T (d_l, d_{l-1}), index l-1
  int64_t wn_off[CADA_MAX_LAYERS], wn_total;              // W_l   (d_{l-1}, d_l), l >= 2
  int lhs_w_slot[CADA_MAX_LAYERS], lhs_b_slot[CADA_MAX_LAYERS];
  int nW;                                                 // delta-weight copies: 1 (CADA1) or M (CADA2)
  bf16_t *Xh, *Xl; int64_t ldx;                           // all features, rows one after the other [total_rows][ldx]
  bf16_t *XGh, *XGl;                                      // gathered minibatch, (padded row, feature)
  int64_t *grow;
  bf16_t *WTh, *WTl, *dWT, *WNh, *WNl, *dWN;
  bf16_t *Ah[CADA_MAX_LAYERS], *Al[CADA_MAX_LAYERS], *dA[CADA_MAX_LAYERS], *Aref[CADA_MAX_LAYERS];   // hidden l, (row, unit)
  bf16_t *Gh[CADA_MAX_LAYERS + 1], *Gl[CADA_MAX_LAYERS + 1], *dG[CADA_MAX_LAYERS + 1], *Gref[CADA_MAX_LAYERS + 1];       // layer l >= 1, (row, unit)
  uint64_t *maskbits[CADA_MAX_LAYERS];                    // hidden l: ReLU mask bits per tile and lane
  int32_t *rep;                                           // CADA2: first worker with the same reference point [M]
  float *dbpart[2], *ddbpart[2];                          // [M][2 RT][max hidden width]: sums per band of 64 rows; those of hidden layer l in (l - 1) mod 2
  size_t band_floats;                                     // of one of them
  char *eval;                                             // scratch of the evaluation (mlp_eval_bytes)
  float *lastb;                                           // [M][Bp / 32][32][2]: last layer, sums of G and dG per block of 32 rows
};

void mlp_stage_weights(Ctx *c);               // WTh, WTl of all layers at the current iterate
size_t mlp_eval_bytes(const MlpPlan &P);      // scratch of the evaluation
int mlp_eval_init(Ctx *c);                    // LDS allowance of its kernel

}  // namespace cada
