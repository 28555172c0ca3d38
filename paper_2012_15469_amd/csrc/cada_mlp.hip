// Dual minibatch gradient of a ReLU MLP with softmax cross-entropy for all workers, bf16
// MFMA contractions with float32 accumulation, and the left-hand side of the communication
// rule (Section 2.2, conditions (workerrule1)/(workerrule2); Algorithm 1, the two gradient
// evaluations on the same samples).
//
// The second gradient is never formed by itself.  With d = theta - theta_ref every quantity
// of the reference evaluation is carried as a difference to the evaluation at theta, and the
// differences are propagated exactly:
//   forward   dZ_1 = A_0 dW_1 + db_1,           dZ_l = dA_{l-1} W_l + Aref_{l-1} dW_l + db_l
//             A_l = relu(Z_l), Aref_l = relu(Z_l - dZ_l), dA_l = A_l - Aref_l
//   loss      G_L = (softmax(Z_L) - onehot)/B,  dG_L = (softmax(Z_L) - softmax(Z_L - dZ_L))/B
//   backward  grad W_l = A_{l-1}^T G_l,         innov W_l = A_{l-1}^T dG_l + dA_{l-1}^T Gref_l
//             GA_{l-1} = G_l W_l^T,             dGA_{l-1} = dG_l W_l^T + Gref_l dW_l^T
//             G_{l-1} = GA_{l-1} [Z>0],         Gref_{l-1} = (GA - dGA)_{l-1} [Zref>0]
// (Gref = G - dG).  Rounding W and W_ref to bf16 separately would bury their difference (one
// Adam step is about one bf16 ulp of a weight); rounding d itself keeps 8 significant bits
// of the difference.
//
// Precision.  The difference of two ReLU-network gradients at nearby points is dominated by
// the few units whose pre-activation changes sign between the two points, so the rule's
// left-hand side is only as good as the pre-activations Z_l are near zero: they must be
// resolved well below |dZ_l| ~ 1e-3 |Z_l|, which a single bf16 product (2^-9 per operand)
// cannot do.  Every contraction of the evaluation at theta (Z_l, grad W_l, GA_l) therefore
// uses split operands x = hi + lo (two bf16 values, 16 significant bits) and three MFMA
// products hi*hi + hi*lo + lo*hi accumulated in float32.  The backward ones need it because
// the server's update divides by sqrt(vhat): a coordinate whose gradient is smaller than its
// rounding error moves by a full alpha-sized step in a random direction, and with single
// bf16 products (0.2% gradient error) the iterate drifts from the fp64 trajectory by
// percents within tens of steps.  The difference contractions are single bf16 products.
//
// Every activation-side tensor (sampled rows, activations, back-propagated signals) exists in ONE
// orientation, (row, unit).  The weight-gradient contractions, which sum over the rows, read the
// same chunks and transpose on the way from LDS into the registers (ds_read_b64_tr_b16).
//
// k_mm5 serves the forward products and the activation gradients, k_dw the weight gradients (where dw_past_caches says so, k_mm5).  For a 128 x 128
// output tile of worker m they accumulate
//     C1 = Ah Bh^T + Ah Bl^T + Al Bh^T          (evaluation at theta, split operands)
//     C2 = Ad Bx^T + Ar Bd^T                    (difference to the reference evaluation)
// from up to four A-side and four B-side bf16 tensors, all stored in chunks of 128 rows x 32
// contraction indices, moved into LDS chunk by chunk, with v_mfma_f32_32x32x16_bf16 on wavefronts
// of 64 x 64.  The epilogues apply bias/ReLU/masks, split results into hi/lo,
// write the tensors the later contractions need, reduce bias gradients
// and the squared norm of the innovation, so no float32 intermediate except the logits
// round-trips through HBM.  k_skinny computes the same products for outputs of at most 32
// columns (the last layer).
#include <algorithm>
#include <cstdlib>
#include <new>
#include <type_traits>

#include "cada_mlp.h"
#include "cada_rule.h"

namespace cada {

enum { EPI_FWD_HIDDEN = 0, EPI_DW = 2, EPI_DA = 3, EPI_LOSS = 4 };

// k_mm5's LDS: a ring of 8 KB slots (one chunk each); behind it 8 KB per multiplying wavefront for the bf16 tensors on their way out, or (weight gradients)
// 32 rows x 64 floats with a pitch of 72: the two half-wavefronts of an accumulator store (rows 4 apart) come into different halves of the banks.
constexpr int kMm5Slots = 15, kDwPitch = 72;
constexpr size_t mm5_lds_bytes(int epi) { return (size_t)kMm5Slots * TILE * sizeof(bf16_t) + 4 * (epi == EPI_DW ? 32 * kDwPitch * sizeof(float) : 8192); }

// Division of 0 <= x < 2^31 by a divisor that the host knows: a product and a shift (as a division it takes the compiler some forty
// instructions, and a tile's three indices two of them, each time at the head of a launch that may have one tile per workgroup).
// With 2^(l-1) < d <= 2^l, m = floor(2^(31+l) / d) + 1 exceeds 2^(31+l) / d by e <= 1, and x e / 2^(31+l) < 2^-l <= 1 / d: the floor is x / d's.
struct Divisor { uint32_t d, m, shift; };
static Divisor divisor(uint32_t d) {
  uint32_t l = 0;
  while ((1u << l) < d) ++l;
  return Divisor{d, (uint32_t)((1ull << (31 + l)) / d + 1), 31 + l};
}
__device__ __forceinline__ int quotient(int x, const Divisor &v) { return (int)(((uint64_t)(uint32_t)x * v.m) >> v.shift); }

// Up to four tensors that share the row index of one side of the product.
struct Side {
  const bf16_t *ptr[kMaxSlots];
  int64_t kt[kMaxSlots];        // chunks per 128-row tile
  int64_t bstride[kMaxSlots];   // elements added per worker
  int n;
};

struct Mm5Args {
  DevState s;
  Side A, B;
  int a_h, a_l, a_d, a_r;       // role -> slot of A (-1: absent)
  int b_h, b_l, b_x, b_d;       // role -> slot of B
  int M, N, K;                  // extents of the tile index spaces and of the contraction
  int workers;
  Divisor gx, gy, nbx;          // k_mm5, k_dw: tiles per row and per column of tiles, workgroups per XCD
  const int32_t *rep;           // optional: the B side of worker m is read at worker rep[m]'s offset (shared reference points)
  int Bp;                       // padded rows per worker (multiple of 128)
  // EPI_FWD_HIDDEN / EPI_DA: bias offset, outputs
  int64_t offb;
  bf16_t *o_h, *o_l, *o_d, *o_r;        // (padded row, column), kto chunks per tile
  int64_t kto;
  uint64_t *maskbits;                   // ReLU mask bits [workers][row tiles][column tiles][256 lanes][2]: written by EPI_FWD_HIDDEN, read by EPI_DA
  float *dbpart, *ddbpart;              // [workers][nband][units], one partial sum per band of 64 rows: written with the signals of a layer's units (EPI_DA, the last
                                        // layer's EPI_DW), read by that layer's EPI_DW.  The order of a band's sum is the same wherever it is formed: the rows with
                                        // row / 4 even one after the other, the other rows one after the other, the one sum plus the other.
  // EPI_DW
  int64_t offW;
  int lhs_slot0;
  int nband;                            // bands per worker
  int bias_here;                        // k_dw: the tiles of the first 128 units form the layer's bias gradient from the bands' sums
  // EPI_LOSS (last layer's forward product with the loss in its epilogue; outputs o_h/o_l/o_d/o_r, bias at offb) and the
  // last layer's EPI_DW, which finishes that layer's bias gradient from the row blocks' sums
  const int64_t *grow;                  // global row of every padded minibatch row (its label)
  float *lastb;                         // [workers][nrb][32][2]: per block of 32 rows, sums over the rows of G and of dG
  int nrb;                              // blocks of 32 rows per worker
  int step_waves;                       // k_skinny<EPI_DW>: wavefronts that take tile steps
  int lhs_slot_b;                       // slot of the bias innovation's part of the left-hand side
  // the last layer's EPI_DW also forms the activation gradient into the units below (null: a single-layer network): W of that layer, its lo part and its difference
  // to the reference point as (unit, class) tensors of w_kt chunks; outputs o_h/o_l/o_d/o_r, maskbits and dbpart/ddbpart as for EPI_DA
  const bf16_t *w_h, *w_l, *w_d;
  int64_t w_kt, w_dstride;
};

__device__ __forceinline__ float delta_theta(const DevState &s, const RefPtr &ref, int64_t i) {
  return (s.theta[i] - ref.hi[i]) + (s.theta_lo[i] - ref.lo[i]);
}
// A value that earlier launches wrote and nobody changes in this one, at a uniform address.
__device__ __forceinline__ int32_t scalar_load(const int32_t *p) { return *(const __attribute__((address_space(4))) int32_t *)(uintptr_t)p; }

// (the selector by a scalar load: the compiler asks for it early, and no wait for it is one for the operands or stores in flight)
__device__ __forceinline__ float *fresh_grad(const DevState &s, int m) {
  return s.gbuf + ((int64_t)(1 - scalar_load(s.sel + m)) * s.M + m) * s.ps;
}
// (bf16 gradient store: the same row of gbuf16; exactly one of the two stores exists)
__device__ __forceinline__ uint16_t *fresh_grad16(const DevState &s, int m) {
  return s.gbuf16 + ((int64_t)(1 - scalar_load(s.sel + m)) * s.M + m) * s.ps16;
}
// coordinate i of worker m's fresh gradient, into whichever store the context keeps
__device__ __forceinline__ void put_fresh_grad(const DevState &s, int m, int64_t i, float v) {
  if (s.gbuf16) fresh_grad16(s, m)[i] = f2bf(v);
  else fresh_grad(s, m)[i] = v;
}

// CADA1's stored innovations (bf16): the row this step writes and the row of the last upload.
__device__ __forceinline__ bf16_t *fresh_innov(const DevState &s, int m) {
  return s.dtl16 + ((int64_t)(1 - scalar_load(s.sel + m)) * s.M + m) * s.ps16;
}
__device__ __forceinline__ const bf16_t *stored_innov(const DevState &s, int m) {
  return s.dtl16 + ((int64_t)scalar_load(s.sel + m) * s.M + m) * s.ps16;
}

__device__ __forceinline__ u32x4 pack8(const bf16_t (&v)[8]) {
  u32x4 o;
  o.x = (uint32_t)v[0] | ((uint32_t)v[1] << 16); o.y = (uint32_t)v[2] | ((uint32_t)v[3] << 16);
  o.z = (uint32_t)v[4] | ((uint32_t)v[5] << 16); o.w = (uint32_t)v[6] | ((uint32_t)v[7] << 16);
  return o;
}

// NA, NB: tensors on the A and the B side (compile-time, so that the loads of a tile step are a
// fixed number of instructions and the waits can count them).  HAS_D: the product Ad Bx^T is present.
// NB == 2 (PL): the rule evaluates no second gradient (always, LAG), so there is no C2 and no difference is carried: three products
// and four operands instead of five and seven.  (The LAG rule's left-hand side stays a launch of its own, k_lag_lhs: the stored
// gradients read in this epilogue made it 12 us longer for the 10 us of that launch, and the server found nothing in the
// caches, 7 -> 11 us; 617-301-150-26, 24 workers.)
//
// A workgroup has eight wavefronts in two roles and works through several tiles.  Wavefronts 4-7
// move chunks from global memory straight into LDS (16-byte LDS-direct loads: no registers, no
// second pass through the LDS write port); wavefronts 0-3 read fragments, issue MFMAs and run the
// epilogue of each tile.  LDS is a ring of 8 KB slots, one chunk each, filled tensor by tensor in
// the order the tile steps read them, across tile boundaries: while the multipliers write one
// tile out, the first steps of the next are already landing.  One barrier per tile step: it
// tells the multipliers that the step has landed, and the movers that the slots of the step before
// are free (NS more loads may go out).  The epilogues use no workgroup barrier, so both roles
// execute the same number of them.  (With four wavefronts doing load, LDS write and multiply in
// turn, the three phases of a step, each near 1000 cycles, ran one after the other.)
// (All eight wavefronts moving and multiplying, the contraction split in two halves of every step that are added up through LDS at the end, with the
// fragments read a step ahead: 1430 instead of 1900 cycles per step, but at 1.54 GHz, what the products' power leaves, in place of 2: 3072-1024-1024-10 within 1 %,
// 512-1024-1024-10 with 64 workers 2 % faster, 300-700-10 with 100 workers, several tiles per workgroup, 2 % slower.  And sums in another order move single units across zero
// a few steps later.  Not kept.)
typedef short i16x4 __attribute__((ext_vector_type(4)));

// Fragment of a transposed operand: 8 consecutive rows (k) of unit (lane % 32) from a [32 rows][32 units]
// block at `blk` (bf16), rows from `krow` on.  ds_read_b64_tr_b16 works on groups of 16 lanes: source lane s
// of a group passes the address of four consecutive units of row s / 4, and lane l receives, for
// e = 0..3, element l % 4 of source lane 4 e + l / 4: unit l of rows 0..3.  The four groups of a
// wavefront are (units 0-15 | 16-31) x (rows 0-7 | 8-15 of the half step, as the MFMA operand wants).
__device__ __forceinline__ bf16x8 tr_fragment(const bf16_t *blk, int lane_off) {
  const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(blk + lane_off));
  const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(blk + lane_off + 4 * 32));
  typedef short i16x8 __attribute__((ext_vector_type(8)));
  const i16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

__device__ __forceinline__ void mm_load(const bf16_t *base, uint32_t byte_off, uint32_t lds) {      // 1 KB, 16 bytes per lane, to `lds` (uniform)
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(byte_off), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory", "m0");
}
// Bias gradient of a hidden layer's units col .. (one per lane) and its innovation, from the sums that the signals' launch left per band of
// 64 rows, and (not PL) the wavefront's 64 units' partial sum of the left-hand side: in the launch of the layer's weight gradient.
template <bool PL, bool CADA1>
__device__ __forceinline__ void hidden_bias(const Mm5Args &g, int wk, int col, int slot, int lane) {
  const DevState &s = g.s;
  float dsum = 0.f;
  if (col < g.N) {
    const float *db = g.dbpart + (int64_t)wk * g.nband * g.N + col, *dd = g.ddbpart + (int64_t)wk * g.nband * g.N + col;
    float gsum = 0.f;
    for (int i = 0; i < (g.K + 63) / 64; ++i) {
      gsum += db[(int64_t)i * g.N];
      if constexpr (!PL) dsum += dd[(int64_t)i * g.N];
    }
    put_fresh_grad(s, wk, g.offb + col, gsum);
    if (CADA1) {
      fresh_innov(s, wk)[g.offb + col] = f2bf(dsum);
      dsum -= bf2f(stored_innov(s, wk)[g.offb + col]);
    }
  }
  if constexpr (!PL) {
    const float tot = wave_sum(dsum * dsum);
    if (lane == 0) s.lhs_part[(int64_t)wk * s.n_lhs_part + slot] = tot;
  }
}

// EPI_DW (rules without a second gradient, float32 store; dw_past_caches): both operands are (row, unit) tensors whose 128-row tiles hold the rows that the
// product sums over.  A step is 32 rows; the operand of a side is the 32 rows x 128 units block of them, which lies in four chunks as 2 KB of
// consecutive memory each, stored in its ring slot as [unit chunk][row][unit] and read with transposing LDS loads.
template <int EPI, int NA, int NB, bool HAS_D>
__global__ __launch_bounds__(2 * kBlock, 1) void k_mm5(const Mm5Args g) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  bf16_t *lds = reinterpret_cast<bf16_t *>(smem_raw);
  constexpr int NS = NA + NB, NSLOT = kMm5Slots;
  constexpr bool PL = NB == 2, TR = EPI == EPI_DW;
  static_assert((EPI == EPI_FWD_HIDDEN || EPI == EPI_DA || (TR && PL)) && NB <= 3, "");
  static_assert(NSLOT >= 2 * NS, "the ring must hold two tile steps");
  const DevState &s = g.s;
  const bool mover = __builtin_amdgcn_readfirstlane((int)threadIdx.x) >= kBlock;   // uniform per wavefront
  const int t = threadIdx.x & (kBlock - 1), lane = t & 63, w = t >> 6;
  const int wy = w >> 1, wx = w & 1;
  // Tiles of this workgroup.  Workgroups are dealt to the 8 XCDs (each with an L2 of its own) in
  // turn; XCD x takes the x-th eighth of the tiles (columns fastest, then rows, then workers), its
  // workgroups every nbx-th of those: an XCD's L2 then sees whole workers, or a few row tiles of
  // one worker with all their column tiles, instead of every worker's operands.
  const int gx = g.gx.d, gy = g.gy.d;
  const int total = gx * gy * g.workers, per = (total + 7) / 8;
  const int nbx = g.nbx.d;
  const int t_first = (blockIdx.x & 7) * per + (blockIdx.x >> 3), t_end = min(((int)(blockIdx.x & 7) + 1) * per, total);
  if (t_first >= t_end) return;
  const int nt = quotient(t_end - t_first + nbx - 1, g.nbx);
  const int nk = (g.K + BK - 1) / BK;
  const int nsteps = nt * nk;

  if (mover) {
    // Instruction c of wavefront w fills the 64 pieces from position 64 (2 w + c) on of a slot;
    // the lane at position P fetches the piece that the LDS order puts there.
    const int lw = __builtin_amdgcn_readfirstlane(w);
    int goff[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      if constexpr (TR) goff[c] = (lw << 12) + (c << 9) + lane * 8;    // kilobyte 2 w + c of the step's operand: half c of unit chunk w
      else goff[c] = lds_piece((2 * lw + c) * 64 + lane) * 8;          // (the order is its own inverse)
    }
    // issue cursor: tile ordinal, step in the tile, first chunk of the tile's rows in every tensor, ring slot
    int ord = 0, h = 0, slot = 0;
    const bf16_t *pa[NA], *pb[NB];
    auto set_tile = [&](int o) __attribute__((always_inline)) {
      const int tix = t_first + o * nbx;
      const int trow = quotient(tix, g.gx), bx = tix - trow * gx, bz = quotient(trow, g.gy), by = trow - bz * gy;
#pragma unroll
      for (int sl = 0; sl < NA; ++sl) pa[sl] = g.A.ptr[sl] + (int64_t)bz * g.A.bstride[sl] + (((int64_t)by * (TR ? 4 : g.A.kt[sl])) << 12);
      const int bzb = g.rep ? scalar_load(g.rep + bz) : bz;
#pragma unroll
      for (int sl = 0; sl < NB; ++sl) pb[sl] = g.B.ptr[sl] + (int64_t)bzb * g.B.bstride[sl] + (((int64_t)bx * (TR ? 4 : g.B.kt[sl])) << 12);
    };
    // next tile step; past the last one the cursor stays (those loads re-read the last chunk into slots nobody reads)
    auto next_step = [&]() __attribute__((always_inline)) {
      if (h + 1 < nk) ++h;
      else if (ord + 1 < nt) { ++ord; h = 0; set_tile(ord); }
    };
    auto load = [&](int sl) __attribute__((always_inline)) {
      const bf16_t *src = sl < NA ? pa[sl < NA ? sl : 0] : pb[sl < NA ? 0 : sl - NA];
      if constexpr (TR) src += (((int64_t)(h >> 2) * (sl < NA ? g.A.kt[0] : g.B.kt[0])) << 12) + ((h & 3) << 10);     // rows 32 h ...: quarter h % 4 of row tile h / 4
      else src += (int64_t)h << 12;
      bf16_t *dst = lds + ((size_t)slot << 12) + (2 * lw << 9);
#pragma unroll
      for (int c = 0; c < 2; ++c)
        __builtin_amdgcn_global_load_lds(src + goff[c], (__attribute__((address_space(3))) void *)(dst + (c << 9)), 16, 0, 0);
      slot = slot + 1 == NSLOT ? 0 : slot + 1;
    };
    set_tile(0);
#pragma unroll
    for (int q = 0; q < NSLOT; ++q) {          // fill the ring
      if (q % NS == 0 && q > 0) next_step();
      load(q % NS);
    }
    // Barrier m: step m has landed when at most the NSLOT - 2 NS tensors issued after it are
    // outstanding (two instructions each); then the NS slots of step m - 1 are free.
    for (int m = 0; m < nsteps; ++m) {
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(2 * (NSLOT - 2 * NS)) : "memory");
      if (m > 0) {
#pragma unroll
        for (int i = 0; i < NS; ++i) {
          constexpr int r0 = NSLOT % NS;
          if ((r0 + i) % NS == 0) next_step();
          load((r0 + i) % NS);
        }
      }
    }
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");     // nothing may land after the workgroup has gone
    return;
  }

  // fragment of this lane inside a 32-row band: row lane % 32, piece lane / 32 (+ 2 in the second half step)
  const int fro = lds_piece((lane & 31) * 4 + (lane >> 5)) * 8;
  const int fro_tr = (8 * (lane >> 5) + ((lane & 15) >> 2)) * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);      // (TR: see tr_fragment)
  int sb = 0;                                  // ring slot of the current step's first tensor
  for (int ord = 0; ord < nt; ++ord) {
  const int tix = t_first + ord * nbx;
  const int trow = quotient(tix, g.gx), bx = tix - trow * gx, wk = quotient(trow, g.gy), by = trow - wk * gy;     // wk: worker
  const int m0 = by * BM, n0 = bx * BN;
  const int rbase = m0 + wy * 64 + 4 * (lane >> 5);
  const int cbase = n0 + wx * 64 + (lane & 31);
  // What the epilogue starts with is asked for here: both columns' biases at theta and at the reference point, or the ReLU masks.
  uint64_t *mbits = nullptr;
  if constexpr (!TR) mbits = g.maskbits + ((((int64_t)wk * gy + by) * gx + bx) * kBlock + t) * 2;
  float bias[2] = {0.f, 0.f}, bias_lo[2] = {0.f, 0.f}, ref_hi[2] = {0.f, 0.f}, ref_lo[2] = {0.f, 0.f};
  u32x4 masks = {0u, 0u, 0u, 0u};
  if constexpr (EPI == EPI_FWD_HIDDEN) {
    const RefPtr ref = theta_ref_at(s, s.rule == CADA_RULE_CADA2 ? scalar_load(s.tau + wk) : 0);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t i = g.offb + min(cbase + j * 32, g.N - 1);
      bias[j] = s.theta[i];
      if constexpr (!PL) { bias_lo[j] = s.theta_lo[i]; ref_hi[j] = ref.hi[i]; ref_lo[j] = ref.lo[i]; }
    }
  }
  if constexpr (EPI == EPI_DA) masks = *reinterpret_cast<const u32x4 *>(mbits);

  f32x16 acc1[2][2], acc2[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) { acc1[i][j][r] = 0.f; acc2[i][j][r] = 0.f; }

  for (int h = 0; h < nk; ++h) {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    auto slot_of = [&](int idx) __attribute__((always_inline)) { const int p = sb + idx; return lds + ((size_t)(p >= NSLOT ? p - NSLOT : p) << 12); };
    const bf16_t *tah = slot_of(g.a_h), *tal = slot_of(g.a_l), *tad = slot_of(HAS_D ? g.a_d : 0), *tar = slot_of(NA == 4 ? g.a_r : 0);
    const bf16_t *tbh = slot_of(NA + g.b_h), *tbl = slot_of(NA + g.b_l), *tbd = slot_of(PL ? NA : NA + g.b_d);
#pragma unroll
    for (int ks = 0; ks < BK; ks += 16) {
      bf16x8 ah[2], al[2], ad[2], ar[2], bh[2], bl[2], bd[2];
      auto frag = [&](const bf16_t *slot, int half, int blk) __attribute__((always_inline)) -> bf16x8 {
        if constexpr (TR) return tr_fragment(slot + (half * 2 + blk) * 1024 + ks * 32, fro_tr);
        else return *reinterpret_cast<const bf16x8 *>(slot + (half * 64 + blk * 32) * BK + (fro ^ ks));
      };
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        ah[i] = frag(tah, wy, i);
        al[i] = frag(tal, wy, i);
        if constexpr (HAS_D) ad[i] = frag(tad, wy, i);
        // with fewer than four A tensors the reference operand is the hi part itself
        if constexpr (NA == 4) ar[i] = frag(tar, wy, i);
        else ar[i] = ah[i];
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        bh[j] = frag(tbh, wx, j);
        bl[j] = frag(tbl, wx, j);
        if constexpr (!PL) bd[j] = frag(tbd, wx, j);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          acc1[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[i], bh[j], acc1[i][j], 0, 0, 0);
          acc1[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bl[j], acc1[i][j], 0, 0, 0);
          acc1[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bh[j], acc1[i][j], 0, 0, 0);
          if constexpr (HAS_D) acc2[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ad[i], bh[j], acc2[i][j], 0, 0, 0);      // (against the hi part)
          if constexpr (!PL) acc2[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ar[i], bd[j], acc2[i][j], 0, 0, 0);
        }
    }
    sb = sb + NS >= NSLOT ? sb + NS - NSLOT : sb + NS;
  }

  // accumulator element (i, j, r) is output (row, col):
  //   row = m0 + wy*64 + i*32 + 8*(r>>2) + 4*(lane>>5) + (r&3),  col = n0 + wx*64 + j*32 + (lane&31)
  const int64_t rp0 = (int64_t)wk * g.Bp;            // first padded row of this worker
  if constexpr (!TR) {
    // Forward: bias, ReLU of both evaluations.  Activation gradient: ReLU masks of the layer
    // below, bias-gradient partial sums.  Both: the result split into hi/lo, its difference and
    // its reference value, each written as a (row, column) tensor.
    // A lane's accumulators are one column and 16 rows of a 32 x 32 quarter: written from there
    // every store instruction would move 2 bytes per lane (some 300 instructions per wavefront and
    // tile; the CU's address unit then needs longer for them than the whole contraction took for
    // small K).  In the chunked layout a quarter is 2 KB of consecutive memory, so each wavefront puts
    // the quarter's values into an LDS buffer of its own in the layout of the destination and
    // copies it out 16 bytes per lane.  (LDS operations of one wavefront are carried out in
    // order, so the buffer needs no barrier.)
    bf16_t *sg = reinterpret_cast<bf16_t *>(smem_raw + (size_t)NSLOT * TILE * sizeof(bf16_t)) + w * 4096;   // 4 x 2 KB
    const int wr0 = m0 + wy * 64, wc0 = n0 + wx * 64;       // first row and column of this wavefront's 64 x 64 part
    bf16_t *const orow_t[4] = {g.o_h, g.o_l, g.o_d, g.o_r};
    auto copy_out = [&](bf16_t *const (&dst)[4], int64_t goff) __attribute__((always_inline)) {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int b = 0; b < (PL ? 2 : 4); ++b)
        if (dst[b] != nullptr) {
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            const int e8 = (hh * 64 + lane) * 8;
            *reinterpret_cast<u32x4 *>(dst[b] + goff + e8) = *reinterpret_cast<const u32x4 *>(sg + b * 1024 + e8);
          }
        }
      asm volatile("" ::: "memory");
    };

    // ReLU masks: one bit per accumulator element, set where the activation is positive (at theta,
    // at the reference point).  The forward contraction of a layer and the activation-gradient
    // contraction into it have the same tiles and the same element-to-lane map, so the forward
    // epilogue leaves each lane's 2 x 64 bits where the backward one finds them: 16 bytes per lane.
    uint64_t bit_on = 0, bit_ref = 0;
    if constexpr (EPI == EPI_DA) {
      bit_on = (uint64_t)masks.x | ((uint64_t)masks.y << 32);
      bit_ref = (uint64_t)masks.z | ((uint64_t)masks.w << 32);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = cbase + j * 32;
      const bool cok = col < g.N;
      const float b = bias[j], db = (bias[j] - ref_hi[j]) + (bias_lo[j] - ref_lo[j]);       // (as delta_theta)
      float sg_sum = 0.f, sd_sum = 0.f;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        // the quarter's four values per element, packed two rows to a register
        uint32_t ph[8], pl[8], pd[8], pr[8];
#pragma unroll
        for (int rp = 0; rp < 8; ++rp) {
          float x[2], xref[2];                      // value at theta, at the reference point; rows r, r + 1
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int r = 2 * rp + e;
            const int row = rbase + i * 32 + 8 * (r >> 2) + (r & 3);
            x[e] = 0.f; xref[e] = 0.f;
            if (cok && row < g.M) {
              if constexpr (EPI == EPI_FWD_HIDDEN) {
                const float z = acc1[i][j][r] + b;
                x[e] = fmaxf(z, 0.f);
                if constexpr (!PL) xref[e] = fmaxf(z - (acc2[i][j][r] + db), 0.f);
              } else {
                const float ga = acc1[i][j][r];
                x[e] = (bit_on >> ((i * 2 + j) * 16 + r)) & 1 ? ga : 0.f;
                if constexpr (!PL) xref[e] = (bit_ref >> ((i * 2 + j) * 16 + r)) & 1 ? (ga - acc2[i][j][r]) : 0.f;
              }
            }
            sg_sum += x[e]; sd_sum += x[e] - xref[e];
          }
          const uint32_t vh = f2bf_pk(x[0], x[1]), vr = f2bf_pk(xref[0], xref[1]);
          ph[rp] = vh; pr[rp] = vr;
          pl[rp] = f2bf_pk(x[0] - __uint_as_float(vh << 16), x[1] - __uint_as_float(vh & 0xffff0000u));
          pd[rp] = f2bf_pk(x[0] - xref[0], x[1] - xref[1]);
          if constexpr (EPI == EPI_FWD_HIDDEN) {      // (the sign of the stored, rounded value)
            const int sh = (i * 2 + j) * 16 + 2 * rp;
            bit_on |= (uint64_t)((__uint_as_float(vh << 16) > 0.f ? 1u : 0u) | (__uint_as_float(vh & 0xffff0000u) > 0.f ? 2u : 0u)) << sh;
            if constexpr (!PL) bit_ref |= (uint64_t)((__uint_as_float(vr << 16) > 0.f ? 1u : 0u) | (__uint_as_float(vr & 0xffff0000u) > 0.f ? 2u : 0u)) << sh;
          }
        }
        // (row, column) layout: element (rl, cl) of the quarter at 32 rl + cl
        if (g.o_h != nullptr && wc0 + j * 32 < (int)g.kto * 32) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int e = (8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * 32 + (lane & 31), sh = 16 * (r & 1);
            sg[e] = (bf16_t)(ph[r >> 1] >> sh); sg[1024 + e] = (bf16_t)(pl[r >> 1] >> sh);
            if constexpr (!PL) { sg[2048 + e] = (bf16_t)(pd[r >> 1] >> sh); sg[3072 + e] = (bf16_t)(pr[r >> 1] >> sh); }
          }
          copy_out(orow_t, tm(rp0 + wr0 + i * 32, wc0 + j * 32, g.kto));
        }
      }
      if constexpr (EPI == EPI_DA) {
        // the other half-wave holds the rows offset by 4: add it, then one value per column and band of 64 rows
        sg_sum += __shfl_xor(sg_sum, 32, 64);
        sd_sum += __shfl_xor(sd_sum, 32, 64);
        if (lane < 32 && cok) {
          const int64_t o = ((int64_t)wk * g.nband + 2 * by + wy) * g.N + col;
          g.dbpart[o] = sg_sum;
          if constexpr (!PL) g.ddbpart[o] = sd_sum;
        }
      }
    }
    if constexpr (EPI == EPI_FWD_HIDDEN) {
      u32x4 mb;
      mb.x = (uint32_t)bit_on; mb.y = (uint32_t)(bit_on >> 32); mb.z = (uint32_t)bit_ref; mb.w = (uint32_t)(bit_ref >> 32);
      *reinterpret_cast<u32x4 *>(mbits) = mb;
    }
  } else {
    // Each wavefront's 64 x 64 part passes through an LDS buffer of its own, 32 rows at a time, and leaves row by row, 16 bytes per lane, 256 bytes per
    // row, past the caches; the stores drain while the next tile's products run.  A lane whose four columns are cut by the matrix's edge goes element by element.
    float *st = reinterpret_cast<float *>(smem_raw + (size_t)NSLOT * TILE * sizeof(bf16_t)) + w * (32 * kDwPitch);
    float *gf = fresh_grad(s, wk) + g.offW;
    const int c4 = (lane & 15) * 4, rr = lane >> 4, colg = n0 + wx * 64 + c4;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int rowb = m0 + wy * 64 + i * 32 + rr;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) st[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * kDwPitch + j * 32 + (lane & 31)] = acc1[i][j][r];
      asm volatile("" ::: "memory");
      if (colg + 4 <= g.N) {
#pragma unroll
        for (int it = 0; it < 8; ++it) {
          const f32x4u v = *reinterpret_cast<const f32x4u *>(st + (rr + 4 * it) * kDwPitch + c4);
          if (rowb + 4 * it < g.M) __builtin_nontemporal_store(v, reinterpret_cast<f32x4u *>(gf + (int64_t)(rowb + 4 * it) * g.N + colg));
        }
      } else {
#pragma unroll
        for (int it = 0; it < 8; ++it)
#pragma unroll
          for (int e = 0; e < 3; ++e)
            if (rowb + 4 * it < g.M && colg + e < g.N) gf[(int64_t)(rowb + 4 * it) * g.N + colg + e] = st[(rr + 4 * it) * kDwPitch + c4 + e];
      }
      asm volatile("" ::: "memory");
    }
    if (g.bias_here && by == 0 && wy == 0 && n0 + wx * 64 < g.N) hidden_bias<true, false>(g, wk, n0 + wx * 64 + lane, 0, lane);
  }
  }   // tiles
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");     // the movers' last barrier
}

// Weight gradient of a layer and its innovation: C1 = A^T G with split operands, C2 = A^T dG [+ dA^T Gref], summed over a worker's rows.  Both
// operands are (row, unit) tensors; a step is 16 rows, 16 rows x 128 units of each of the NS tensors.
//
// What bounds it: a 128 x 128 tile has few steps (16 for B = 256) and then 64 KB of gradient to write (CADA1: 32 KB of innovation read and
// written, too), so products and the way out have to overlap.  Two workgroups of four wavefronts share a CU, half of the register file and 80 KB of
// LDS each: while one writes a tile out, the other has the matrix cores.  Every wavefront moves its part of the operands (LDS-direct), multiplies
// 64 x 64 of the tile and writes them out; no wavefront is there for the moving alone, whose registers would be the second workgroup's.
// With four moving and four multiplying wavefronts on a CU products and stores took turns: first layer of 3072-1024-1024-10, 16 workers of 256
// rows, CADA1: 190 us, now 168; second layer 79, now 71; 784-512-10, 64 workers of 128 rows, CADA2: 51.5, now 44.5.  What is left: a step takes 880 cycles of
// a CU without the way out (products alone 512 by count and 560 measured, loads alone 594), 1010 with it, at the 1.8 GHz that the products' power leaves.
//
// LDS: a ring of 20 slots of 4 KB, one tensor of a step each ([4 chunks of 32 units][16 rows][32 units]: 1 KB of consecutive memory per chunk, moved by
// the wavefront of that number).  A step's fragments are read during the step before, each right after its register's last use, so a step's
// slots are free at its own barrier, and the loads that refill them go out between its products.  A wavefront's loads land in the order of
// issue: the barrier of a step waits until only what was asked for after the next step's operands is outstanding.  At a tile's end the last step's
// freed slots (four of them) are the buffers of the way out, 4 KB per wavefront, and their refill waits until the next tile starts; everything
// else that is in flight then has to land before the first store, so that the next tile's first steps need not wait for the stores behind.
// Asked for in bursts after the barrier, the loads stalled the wavefronts: 1560 cycles per 1024 of products against 1142.
//
// The unit of A is the MFMA's column index: a lane's accumulators are one row of the matrix and groups of four consecutive
// columns, which go through LDS 16 bytes (bf16: 8) at a time and leave as whole rows of 128 bytes.  (Plain stores: with the non-temporal hint, which
// paid for rows of 256 bytes, 201 and 62 us where plain ones took 180 and 44.)
typedef uint32_t u32h __attribute__((aligned(2)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u32x4h __attribute__((ext_vector_type(4), aligned(2)));   // eight bf16 values at any address
constexpr int kDwRows = 16;                                    // rows per step
constexpr int kDwSlots = 20;
constexpr size_t kDwLds = kDwSlots * 4096;

// at: the workgroup's place among its XCD's.
template <int NA, int NB, bool HAS_D, bool CADA1>
__device__ __forceinline__ void weight_gradient(const Mm5Args &g, int at, unsigned char *smem_raw) {
  constexpr int NS = NA + NB, NSLOT = kDwSlots, AHEAD = NSLOT / NS, R0 = NSLOT % NS;
  constexpr int LANDED = (NSLOT - 4) / NS - 1;      // steps of a tile that need not wait for their loads: those had landed before the last tile's way out
  constexpr bool PL = NB == 2;
  static_assert(NS >= 4 && NSLOT >= 2 * NS + 4, "");
  const DevState &s = g.s;
  // (one stride and one number of chunks for all tensors of a side: tiles_fit)
  const int lane0 = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), wy = w >> 1, wx = w & 1;
  // tiles of this workgroup: as in k_mm5
  const int gx = g.gx.d, gy = g.gy.d;
  const int total = gx * gy * g.workers, per = (total + 7) / 8, nbx = g.nbx.d;
  const int t_first = (blockIdx.x & 7) * per + at, t_end = min(((int)(blockIdx.x & 7) + 1) * per, total);
  if (t_first >= t_end) return;
  const int nt = quotient(t_end - t_first + nbx - 1, g.nbx), nk = (g.K + kDwRows - 1) / kDwRows, nsteps = nt * nk;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem_raw;

  // issue cursor: step, tile, step in the tile, slot; this wavefront's chunk of every operand of the tile, and the step's place in it
  int i_step = 0, i_tix = t_first, i_h = 0, i_slot = 0;
  const bf16_t *src[NS];
  int64_t at_a = 0, at_b = 0;
  auto set_tile = [&]() __attribute__((always_inline)) {
    const int trow = quotient(i_tix, g.gx), bx = i_tix - trow * gx, bz = quotient(trow, g.gy), by = trow - bz * gy;
#pragma unroll
    for (int q = 0; q < NA; ++q) src[q] = g.A.ptr[q] + (int64_t)bz * g.A.bstride[0] + ((int64_t)(4 * by + w) << 12);
#pragma unroll
    for (int q = 0; q < NB; ++q) src[NA + q] = g.B.ptr[q] + (int64_t)bz * g.B.bstride[0] + ((int64_t)(4 * bx + w) << 12);
  };
  auto next_step = [&]() __attribute__((always_inline)) {
    ++i_step;
    if (++i_h == nk) { i_h = 0; i_tix += nbx; if (i_tix < t_end) set_tile(); }
    at_a = (((int64_t)(i_h >> 3) * g.A.kt[0]) << 12) + ((i_h & 7) << 9);       // rows 16 i_h .. of the worker: eighth i_h % 8 of row tile i_h / 8
    at_b = (((int64_t)(i_h >> 3) * g.B.kt[0]) << 12) + ((i_h & 7) << 9);
  };
  auto load = [&](int q) __attribute__((always_inline)) {        // tensor q of the cursor's step into the next slot (nothing past the last step)
    if (i_step < nsteps) {
      mm_load(src[q] + (q < NA ? at_a : at_b), lane0 * 16, lds0 + i_slot * 4096 + w * 1024);
      i_slot = i_slot + 1 == NSLOT ? 0 : i_slot + 1;
    }
  };
  auto more = [&](int i) __attribute__((always_inline)) {        // tensor i of the NS that take the slots of a step whose fragments have been read
    if (i >= NS) return;
    if ((R0 + i) % NS == 0) next_step();
    load((R0 + i) % NS);
  };
  set_tile();
#pragma unroll 1
  for (int p = 0; p < AHEAD; ++p) {
    if (p > 0) next_step();
#pragma unroll
    for (int q = 0; q < NS; ++q) load(q);
  }
  if constexpr (R0 > 0) next_step();
#pragma unroll
  for (int q = 0; q < R0; ++q) load(q);
  // The tiles of the first 128 units also form the layer's bias gradient and its innovation.  (A launch of its own cost 5 us.  One wavefront for 256 columns, with fewer partial sums: 784-500-10, B = 12:
  // 81.1 -> 82.8 us per step, 3072-1024-1024-10: 608 -> 615.)  A workgroup's first tile does it while its operands are on their way, a later one before
  // its way out, when the stores of the tile before have drained.
  auto bias_part = [&](int wk, int bx) __attribute__((always_inline)) {
    const int cw = bx * BN + wx * 64;
    if (cw < g.N) hidden_bias<PL, CADA1>(g, wk, cw + lane0, g.lhs_slot_b + 2 * bx + wx, lane0);
  };
  if (g.bias_here && wy == 0) {
    const int trow = quotient(t_first, g.gx), wk = quotient(trow, g.gy);
    if (trow == wk * gy) bias_part(wk, t_first - trow * gx);
  }
  // (the first step; all of them where there are few)
  if (nsteps >= AHEAD) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((AHEAD - 1) * NS) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  // this lane's source address inside a [16 rows][32 units] block (see tr_fragment)
  const int fro = (8 * (lane0 >> 5) + ((lane0 & 15) >> 2)) * 32 + 16 * ((lane0 >> 4) & 1) + 4 * (lane0 & 3);
  int step = 0, sb = 0, landed = 0;             // sb: slot of the first tensor of the step whose fragments are read next
  for (int tix = t_first; tix < t_end; tix += nbx) {
    const int trow = quotient(tix, g.gx), bx = tix - trow * gx, wk = quotient(trow, g.gy), by = trow - wk * gy;     // wk: worker
    f32x16 acc1[2][2], acc2[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) { acc1[i][j][r] = 0.f; acc2[i][j][r] = 0.f; }

    auto slot_of = [&](int q) __attribute__((always_inline)) { const int p = sb + q; return smem_raw + (p >= NSLOT ? p - NSLOT : p) * 4096; };
    auto frag = [&](int q, int blk) __attribute__((always_inline)) { return tr_fragment(reinterpret_cast<const bf16_t *>(slot_of(q) + blk * 1024), fro); };
    bf16x8 ah[2], al[2], ad[2], bh[2], bl[2], bg[2], bd[2];
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (step > 0) {                              // the loads whose slots the last tile's way out lay over
#pragma unroll
      for (int i = NS - 4; i < NS; ++i) more(i);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      al[i] = frag(1, 2 * wy + i); bh[i] = frag(NA, 2 * wx + i); ah[i] = frag(0, 2 * wy + i); bl[i] = frag(NA + 1, 2 * wx + i);
      if constexpr (HAS_D) { ad[i] = frag(2, 2 * wy + i); bg[i] = frag(NA + 2, 2 * wx + i); }
      if constexpr (!PL) bd[i] = frag(NS - 1, 2 * wx + i);
    }
    const int rw = by * BM + wy * 64, cw = bx * BN + wx * 64;     // first row and column of this wavefront's part
    int out_slot = 0;
    u32x4 old[2][4] = {};
    // Step by step each fragment is read for the next step right after its last use, and a load goes out between products.
    for (int h = 0; h < nk; ++h, ++step) {
      const bool last = h + 1 == nk;
      if (last) {
        out_slot = sb + (NS - 4) + w;
        if constexpr (CADA1) {
          // the stored innovations, 16 bytes of row lane / 8 + 8 it from column 8 (lane % 8) on (clamped into the matrix: no load under a branch)
          int ln = lane0;
          asm volatile("" : "+v"(ln));             // (addresses computed here, not kept in registers through the products)
          const int r0 = min(rw, g.M - 1), c0 = min(cw, g.N - 8);
          const bf16_t *ivs = stored_innov(s, wk) + g.offW + (int64_t)r0 * g.N + c0;
          const uint32_t coff = min(cw + 8 * (ln & 7), g.N - 8) - c0;
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int it = 0; it < 4; ++it)
              old[i][it] = *reinterpret_cast<const u32x4h *>(ivs + (uint32_t)min(32 * i + 8 * it + (ln >> 3), g.M - 1 - r0) * (uint32_t)g.N + coff);
        }
      }
#define MM(a, b, c) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, c, 0, 0, 0)
#define KEEP() __builtin_amdgcn_sched_barrier(0)
      auto ask = [&](int i) __attribute__((always_inline)) { if (i < NS - 4 || !last) more(i); };
      sb = sb + NS >= NSLOT ? sb + NS - NSLOT : sb + NS;
      KEEP();
      MM(al[0], bh[0], acc1[0][0]); MM(al[0], bh[1], acc1[0][1]); MM(al[1], bh[0], acc1[1][0]); MM(al[1], bh[1], acc1[1][1]);
      KEEP();
      // this wavefront's part of the next step has landed, and every wavefront has this step's fragments in registers
      const int later = nsteps - step - 2;
      if (last || landed > 0) { --landed; asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
      else if (later * NS >= NSLOT - 2 * NS) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NSLOT - 2 * NS) : "memory");
      else if (later == 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NS) : "memory");
      else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      __builtin_amdgcn_s_setprio(1);
      al[0] = frag(1, 2 * wy); al[1] = frag(1, 2 * wy + 1); KEEP();
      MM(ah[0], bl[0], acc1[0][0]); MM(ah[1], bl[0], acc1[1][0]); KEEP(); bl[0] = frag(NA + 1, 2 * wx); ask(0); KEEP();
      MM(ah[0], bl[1], acc1[0][1]); MM(ah[1], bl[1], acc1[1][1]); KEEP(); bl[1] = frag(NA + 1, 2 * wx + 1); ask(1); KEEP();
      MM(ah[0], bh[0], acc1[0][0]); MM(ah[1], bh[0], acc1[1][0]); KEEP(); bh[0] = frag(NA, 2 * wx); ask(2); KEEP();
      MM(ah[0], bh[1], acc1[0][1]); MM(ah[1], bh[1], acc1[1][1]); KEEP(); bh[1] = frag(NA, 2 * wx + 1); ask(3); KEEP();
      if constexpr (HAS_D) {
        MM(ad[0], bg[0], acc2[0][0]); MM(ad[0], bg[1], acc2[0][1]); KEEP(); ad[0] = frag(2, 2 * wy); ask(4); KEEP();
        MM(ad[1], bg[0], acc2[1][0]); MM(ad[1], bg[1], acc2[1][1]); KEEP(); ad[1] = frag(2, 2 * wy + 1); bg[0] = frag(NA + 2, 2 * wx); bg[1] = frag(NA + 2, 2 * wx + 1); ask(5); KEEP();
      }
      if constexpr (!PL) {
        MM(ah[0], bd[0], acc2[0][0]); MM(ah[0], bd[1], acc2[0][1]); KEEP(); ah[0] = frag(0, 2 * wy); ask(HAS_D ? 6 : 4); KEEP();
        MM(ah[1], bd[0], acc2[1][0]); MM(ah[1], bd[1], acc2[1][1]); KEEP(); ah[1] = frag(0, 2 * wy + 1); bd[0] = frag(NS - 1, 2 * wx); bd[1] = frag(NS - 1, 2 * wx + 1); KEEP();
      } else {
        ah[0] = frag(0, 2 * wy); ah[1] = frag(0, 2 * wy + 1); KEEP();
      }
      __builtin_amdgcn_s_setprio(0);
#undef MM
#undef KEEP
    }
    unsigned char *st = smem_raw + (out_slot >= NSLOT ? out_slot - NSLOT : out_slot) * 4096;

    int lane = lane0;
    asm volatile("" : "+v"(lane));
    const int r32 = lane & 31, hf = lane >> 5;
    // accumulator element (i, j, r): row rw + 32 i + lane % 32 of the matrix, column cw + 32 j + 8 (r / 4) + 4 (lane / 32) + r % 4
    const bool g16 = s.gbuf16 != nullptr;
    // On the way out a lane has 16 bytes of a row: floats 4 (lane % 8) .. of 32 columns, bf16 values 8 (lane % 8) .. of 64, of row lane / 8 + 8 it.
    const int rl = lane >> 3;
    const bool whole = rw + 64 <= g.M && cw + 64 <= g.N;        // (uniform) this wavefront's part lies in the matrix
    if (g.bias_here && by == 0 && wy == 0 && tix != t_first) bias_part(wk, bx);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    landed = LANDED;

    // LDS positions: 16-byte piece p of row r at 128 r + 16 (p ^ r / 2 % 8) (rows 2 apart are one pass over the banks apart); the 8-byte halves of
    // a bf16 piece change places in rows 16 to 31
    auto pos16 = [&](int row, int piece) __attribute__((always_inline)) { return st + row * 128 + ((piece ^ ((row >> 1) & 7)) << 4); };
    auto pos8 = [&](int j, int q) __attribute__((always_inline)) { return pos16(r32, 4 * j + q) + 8 * (hf ^ (r32 >> 4)); };
    auto row16 = [&](int it, u32x4 v) __attribute__((always_inline)) { return it < 2 ? v : u32x4{v.z, v.w, v.x, v.y}; };
    float sq = 0.f;
    auto write_out = [&](auto whole_part) __attribute__((always_inline)) {
      constexpr bool WHOLE = decltype(whole_part)::value;
      const int rows = WHOLE ? 64 : g.M - rw, cols = WHOLE ? 64 : g.N - cw;       // of this wavefront's part (may be none)
      const int64_t at = g.offW + (int64_t)rw * g.N + cw;
      auto put_rows16 = [&](bf16_t *base, int i) __attribute__((always_inline)) {      // 32 rows of 64 bf16 values from LDS to memory
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const u32x4 v = row16(it, *reinterpret_cast<const u32x4 *>(pos16(8 * it + rl, lane & 7)));
          const int row = 32 * i + 8 * it + rl, col = 8 * (lane & 7);
          if (!WHOLE && row >= rows) continue;
          bf16_t *q = base + (uint32_t)row * (uint32_t)g.N + col;
          if (WHOLE || col + 8 <= cols) *reinterpret_cast<u32x4h *>(q) = v;
          else if (col < cols) {               // the one lane at the matrix's edge: (uniform) cols % 8 values
            uint32_t x = v.x, y = v.y;
            if (cols & 4) { *reinterpret_cast<u32x2u *>(q) = u32x2u{x, y}; q += 4; x = v.z; y = v.w; }
            if (cols & 2) { *reinterpret_cast<u32h *>(q) = x; q += 2; x = y; }
            if (cols & 1) *q = (bf16_t)x;
          }
        }
      };
      if constexpr (!PL) {
        bf16_t *ivf = CADA1 ? fresh_innov(s, wk) + at : nullptr;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          if (CADA1) {
#pragma unroll
            for (int it = 0; it < 4; ++it) {
              u32x4 o = old[i][it];
              if constexpr (!WHOLE) {      // (a lane at the matrix's edge was moved back: its values lie that many places further up)
                const int d = min(max(8 * (lane & 7) + 8 - cols, 0), 7);
                uint64_t lo = (uint64_t)o.x | ((uint64_t)o.y << 32), hi = (uint64_t)o.z | ((uint64_t)o.w << 32);
                if (d >= 4) { lo = hi; hi = 0; }
                const int b = 16 * (d & 3);
                if (b > 0) { lo = (lo >> b) | (hi << (64 - b)); hi >>= b; }
                o = u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
              }
              *reinterpret_cast<u32x4 *>(pos16(8 * it + rl, lane & 7)) = row16(it, o);
            }
            asm volatile("" ::: "memory");
          }
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              uint32_t o[2] = {0u, 0u}, nw[2];
              if (CADA1) { const uint64_t x = *reinterpret_cast<const uint64_t *>(pos8(j, q)); o[0] = (uint32_t)x; o[1] = (uint32_t)(x >> 32); }
#pragma unroll
              for (int e = 0; e < 2; ++e) {
                const float x = acc2[i][j][4 * q + 2 * e], y = acc2[i][j][4 * q + 2 * e + 1];
                nw[e] = f2bf_pk(x, y);
                const int row = 32 * i + r32, col = 32 * j + 8 * q + 4 * hf + 2 * e;
                const float dx = WHOLE || (row < rows && col < cols) ? x - __uint_as_float(o[e] << 16) : 0.f;
                const float dy = WHOLE || (row < rows && col + 1 < cols) ? y - __uint_as_float(o[e] & 0xffff0000u) : 0.f;
                sq = fmaf(dx, dx, sq); sq = fmaf(dy, dy, sq);
              }
              if (CADA1) *reinterpret_cast<uint64_t *>(pos8(j, q)) = (uint64_t)nw[0] | ((uint64_t)nw[1] << 32);
            }
          if (CADA1) {
            asm volatile("" ::: "memory");
            put_rows16(ivf, i);
            asm volatile("" ::: "memory");
          }
        }
      }
      if (g16) {
        bf16_t *gf16 = fresh_grad16(s, wk) + at;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
              *reinterpret_cast<uint64_t *>(pos8(j, q)) = (uint64_t)f2bf_pk(acc1[i][j][4 * q], acc1[i][j][4 * q + 1]) |
                                                          ((uint64_t)f2bf_pk(acc1[i][j][4 * q + 2], acc1[i][j][4 * q + 3]) << 32);
          asm volatile("" ::: "memory");
          put_rows16(gf16, i);
          asm volatile("" ::: "memory");
        }
      } else {
        float *gf = fresh_grad(s, wk) + at;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              *reinterpret_cast<v4s *>(pos16(r32, 2 * q + hf)) = v4s{acc1[i][j][4 * q], acc1[i][j][4 * q + 1], acc1[i][j][4 * q + 2], acc1[i][j][4 * q + 3]};
            asm volatile("" ::: "memory");
#pragma unroll
            for (int it = 0; it < 4; ++it) {
              const v4s v = *reinterpret_cast<const v4s *>(pos16(8 * it + rl, lane & 7));
              const int row = 32 * i + 8 * it + rl, col = 32 * j + 4 * (lane & 7);
              if (!WHOLE && row >= rows) continue;
              float *q = gf + (uint32_t)row * (uint32_t)g.N + col;
              if (WHOLE || col + 4 <= cols) *reinterpret_cast<f32x4u *>(q) = v;
              else if (col < cols) {           // (cols % 4 values)
                float x = v.x;
                if (cols & 2) { *reinterpret_cast<f32x2u *>(q) = f32x2u{v.x, v.y}; q += 2; x = v.z; }
                if (cols & 1) *q = x;
              }
            }
            asm volatile("" ::: "memory");
          }
      }
    };
    if (whole) write_out(std::true_type{});
    else write_out(std::false_type{});
    if constexpr (!PL) {
      const float tot = wave_sum(sq);           // one partial sum of the left-hand side per wavefront and tile
      if (lane == 0) s.lhs_part[(int64_t)wk * s.n_lhs_part + g.lhs_slot0 + (by * gx + bx) * 4 + w] = tot;
    }
  }   // tiles
}

template <int NA, int NB, bool HAS_D, bool CADA1>
__global__ __launch_bounds__(kBlock, 2) void k_dw(const Mm5Args g) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  // The arguments of the head and of the way out in one round trip, as in k_skinny.  (784-512-10, 64 workers of 128 rows, with the last layer's launch and the server's: 159.7 -> 157.0 us per step, 784-500-10, 10 of
  // 12: 52.3 -> 51.1.  In k_dw_two and k_mm5 it costs scalar registers that the loop wants: 3072-1024-1024-10: 592.7 -> 594.5, 784-500-500-10, 10 of 12: 104.3 -> 105.3.)
  asm volatile("" ::"s"(g.A.ptr[0]), "s"(g.A.ptr[1]), "s"(g.A.ptr[NA - 1]), "s"(g.B.ptr[0]), "s"(g.B.ptr[1]), "s"(g.B.ptr[NB - 2]), "s"(g.B.ptr[NB - 1]), "s"(g.A.kt[0]), "s"(g.B.kt[0]),
               "s"(g.A.bstride[0]), "s"(g.B.bstride[0]), "s"(g.gx.d), "s"(g.gx.m), "s"(g.gx.shift), "s"(g.gy.d), "s"(g.gy.m), "s"(g.gy.shift), "s"(g.nbx.d), "s"(g.nbx.m), "s"(g.nbx.shift),
               "s"(g.workers), "s"(g.K), "s"(g.M), "s"(g.N), "s"(g.bias_here), "s"(g.s.gbuf), "s"(g.s.gbuf16), "s"(g.s.sel), "s"(g.s.M));
  weight_gradient<NA, NB, HAS_D, CADA1>(g, blockIdx.x >> 3, smem_raw);
}
// The second layer's and the first layer's in one launch (the same number of workgroups per XCD for both; the first layer's tiles are dealt from the other end, so that where
// the tiles are few the two layers have workgroups of their own).  It saves a launch and the first one's last wave.  us per step, two launches / one: 617-301-150-26, always,
// 24 workers of 100 rows: 87.6 / 84.5; 784-512-512-10, LAG, 10 of 12: 82.6 / 78.9; 300-400-300-10, 64 of 60: 174.9 / 167.6; 3072-1024-1024-10, 16 of 256: 572.4 / 562.0.
template <bool PL, bool CADA1>
__global__ __launch_bounds__(kBlock, 2) void k_dw_two(const Mm5Args g2, const Mm5Args g1) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int at = blockIdx.x >> 3, last = g1.nbx.d - 1;
  if constexpr (PL) weight_gradient<2, 2, false, false>(g2, at, smem_raw);
  else weight_gradient<3, 4, true, CADA1>(g2, at, smem_raw);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // (the ring's slots are written again; every load into them has landed)
  if constexpr (PL) weight_gradient<2, 2, false, false>(g1, last - at, smem_raw);
  else weight_gradient<2, 3, false, CADA1>(g1, last - at, smem_raw);
}

__device__ __forceinline__ float group16_sum(float x) {
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// The same products for an output of at most 32 columns (the last layer: C <= 32 classes).  A
// 128 x 128 tile would leave nine tenths of its MFMAs and of its workgroups idle and the launch
// would run on a few CUs (32 tiles for the logits of 16 workers).  Here a workgroup computes
// 32 rows x 32 columns; its wavefronts (eight; fewer for the few steps of a weight gradient) split the
// tile steps (wavefront w takes steps w, w + nw, ...), each through an LDS area of its own, and add their partial accumulators up
// through LDS in a fixed order, the same for any number of workers.  grid (ceil(M / 32), workers, blocks of 32 columns), 64 threads per
// wavefront (EPI_DW: and wavefronts for the way out alone, launch_skinny_as), 2 KB of dynamic LDS per tensor each (EPI_DW: 15.5 KB, for those that take steps).  EPI_FWD_HIDDEN: a hidden layer's forward product where the 128 x 128 tiles are few or mostly
// padding (skinny_forward), with the outputs of k_mm5's.
// EPI_LOSS: the logits stay in the workgroup, whose epilogue is the loss (the signals
// the backward contractions read, and per-block sums for the bias gradient); EPI_DW: weight gradient, innovation, its
// squared norm (slot lhs_slot0 + row band), and (one more workgroup) the last layer's bias gradient from those sums.
// The weight gradient sums over the worker's rows: its operands are (row, unit) tensors, a step's part of
// one is a [32 rows][32 units] block (2 KB of consecutive memory), which the wavefront copies into an
// LDS area of its own and reads back transposed (tr_fragment).
// TWICE (EPI_FWD_HIDDEN): four wavefronts that do the work of eight, each the steps and the partial accumulators of two of them, so that a result does not depend on their number.
template <int EPI, int NA, int NB, bool HAS_D, bool TWICE = false>
__device__ __forceinline__ void skinny(const Mm5Args &g, unsigned char *smem_raw, int bx /* block of 32 rows of the result */) {
  static_assert(EPI == EPI_FWD_HIDDEN || !TWICE, "");
  float *red = reinterpret_cast<float *>(smem_raw);                  // EPI_DW: [8 wavefronts][2 accumulators][16][64]
  const DevState &s = g.s;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int nw = blockDim.x >> 6;          // wavefronts of this launch (1..8)
  const int nsw = EPI == EPI_DW ? g.step_waves : nw;       // those that take tile steps: fewer for short contractions, so that more workgroups fit a CU
  const int m0 = bx * 32, wk = blockIdx.y;
  const int nk = (g.K + BK - 1) / BK;
  constexpr bool PL = NB == 2;
  // (EPI_FWD_HIDDEN: units 32 blockIdx.z ... of the layer; else the only block of columns)
  const int cb = EPI == EPI_FWD_HIDDEN ? (int)blockIdx.z : 0;
  // EPI_FWD_HIDDEN, EPI_LOSS: a wavefront's area of LDS: a step's 32 x 32 blocks, 2 KB each, later its partial results (4 KB, 8 KB with a difference) and a room behind them
  constexpr int AREA = (NA + NB) * 2048, ROOM = PL ? 4096 : 8192;
  auto part_of = [&](int ww, int q) __attribute__((always_inline)) { return reinterpret_cast<float *>(smem_raw + ww * AREA + q * 4096); };      // [16][64]
  if constexpr (EPI == EPI_DW) {
    // The last layer's launch has one workgroup more than tiles: it forms that layer's bias gradient, its innovation
    // and the innovation's part of the left-hand side from the sums that the forward launch left per block of 32 rows
    // (added up in the order of the rows).
    if (g.lastb != nullptr && bx == (g.M + 31) / 32) {
      if (w != 0) return;
      const bool cada1 = s.rule == CADA_RULE_CADA1;
      float sqb = 0.f;
      if (lane < g.N) {
        float gsum = 0.f, iv = 0.f;
        for (int rb = 0; rb < g.nrb; ++rb) {
          const float *q = g.lastb + ((((int64_t)wk * g.nrb + rb) * 32 + lane) << 1);
          gsum += q[0]; iv += q[1];
        }
        put_fresh_grad(s, wk, g.offb + lane, gsum);
        if (cada1) {
          fresh_innov(s, wk)[g.offb + lane] = f2bf(iv);
          iv -= bf2f(stored_innov(s, wk)[g.offb + lane]);
        }
        sqb = iv * iv;
      }
      const float totb = wave_sum(sqb);
      if (!PL && lane == 0) s.lhs_part[(int64_t)wk * s.n_lhs_part + g.lhs_slot_b] = totb;
      return;
    }
  }
  const bool cada1 = !PL && s.rule == CADA_RULE_CADA1;
  bf16_t old_iv[4] = {0, 0, 0, 0};              // EPI_DW: the stored innovations of four of the elements that this thread writes, from e0 on
  auto ask_old = [&](int e0) __attribute__((always_inline)) {
    const bf16_t *ivs = stored_innov(s, wk) + g.offW;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = min(e0 + i * (int)blockDim.x, 16 * 64 - 1), r = e >> 6, ln = e & 63;
      old_iv[i] = ivs[(int64_t)min(m0 + 8 * (r >> 2) + 4 * (ln >> 5) + (r & 3), g.M - 1) * g.N + min(ln & 31, g.N - 1)];
    }
  };
  if constexpr (EPI != EPI_DW) {
    // The arguments that the head needs, in one round trip (left to itself the compiled kernel asks for each where it is used: seven of 0.2 us in a row before the last operands are on their way).
    asm volatile("" ::"s"(g.A.ptr[0]), "s"(g.A.ptr[1]), "s"(g.A.ptr[NA - 2]), "s"(g.A.ptr[NA - 1]), "s"(g.B.ptr[0]), "s"(g.B.ptr[1]), "s"(g.B.ptr[NB - 1]), "s"(g.A.kt[0]), "s"(g.B.kt[0]),
                 "s"(g.A.bstride[0]), "s"(g.B.bstride[NB - 1]), "s"(g.rep), "s"(s.tau), "s"(s.rule), "s"(g.K), "s"(g.M), "s"(g.N), "s"(g.offb), "s"(s.theta), "s"(s.theta_lo), "s"(s.hist), "s"(s.hist_lo),
                 "s"(s.kR), "s"(s.D), "s"(s.R), "s"(s.ps), "s"(EPI == EPI_LOSS ? g.grow : nullptr), "s"(g.Bp));
  } else if constexpr (NB == 4) {
    // (not under the rules without reference points: without / with it 784-500-10, always, 10 workers of 12 rows: 41.8 / 42.5 us per step,
    // 784-512-10, always, 64 of 128: 164.5 / 164.5; CADA2, 784-500-10, 10 of 12: 50.7 / 50.4, 200-150-5, 8 of 200: 55.1 / 55.2, 300-400-300-10, 30 of 60: 111.2 / 111.2)
    asm volatile("" ::"s"(g.A.ptr[0]), "s"(g.A.ptr[1]), "s"(g.A.ptr[NA - 1]), "s"(g.B.ptr[0]), "s"(g.B.ptr[1]), "s"(g.B.ptr[NB - 2]), "s"(g.B.ptr[NB - 1]), "s"(g.A.kt[0]), "s"(g.B.kt[0]),
                 "s"(g.A.bstride[0]), "s"(g.B.bstride[0]), "s"(g.rep), "s"(s.rule), "s"(g.K), "s"(g.M), "s"(g.N), "s"(g.step_waves), "s"(g.lastb), "s"(g.w_h), "s"(g.w_l), "s"(g.w_d), "s"(g.w_kt),
                 "s"(g.w_dstride), "s"(g.maskbits), "s"(s.sel), "s"(s.M), "s"(s.dtl16), "s"(s.ps16));
  }
  const bf16_t *pa[NA], *pb[NB];
  f32x16 acc1, acc2;
#pragma unroll
  for (int r = 0; r < 16; ++r) { acc1[r] = 0.f; acc2[r] = 0.f; }
  f32x16 later1 = acc1, later2 = acc2;            // TWICE: of the wavefront's second share of the steps
  float bz[2] = {0.f, 0.f}, dbz[2] = {0.f, 0.f};
  int label = 0;
  if constexpr (EPI == EPI_DW) {
    // units m0 .. m0 + 31 of the A tensors are chunk m0 / 32 of every row tile, the (at most 32) output
    // columns chunk 0 of the B tensors; step kc covers the worker's rows 32 kc .. 32 kc + 31
#pragma unroll
    for (int sl = 0; sl < NA; ++sl) pa[sl] = g.A.ptr[sl] + (int64_t)wk * g.A.bstride[0] + ((int64_t)(m0 >> 5) << 12);
#pragma unroll
    for (int sl = 0; sl < NB; ++sl) pb[sl] = g.B.ptr[sl] + (int64_t)wk * g.B.bstride[0];
    bf16_t *area = reinterpret_cast<bf16_t *>(smem_raw) + w * (7 * 1024);       // room for seven blocks per wavefront
    if (cada1) ask_old(t);                      // (used after the products)
    u32x4 wh[2], wl[2], wd[2];                  // (activation gradient: 32 units x 32 classes of W, a unit per lane)
    if constexpr (PL || HAS_D) {
      if (g.w_h != nullptr) {
        const int64_t o = (((int64_t)(m0 >> 7) * g.w_kt) << 12) + (((m0 & 127) + (lane & 31)) << 5) + ((lane >> 5) << 3);
        const int64_t od = (int64_t)(g.rep ? scalar_load(g.rep + wk) : wk) * g.w_dstride + o;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          wh[half] = *reinterpret_cast<const u32x4 *>(g.w_h + o + 16 * half);
          wl[half] = *reinterpret_cast<const u32x4 *>(g.w_l + o + 16 * half);
          if constexpr (!PL) wd[half] = *reinterpret_cast<const u32x4 *>(g.w_d + od + 16 * half);
        }
      }
    }
    const int fro_tr = (8 * (lane >> 5) + ((lane & 15) >> 2)) * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    // A band of 64 rows is two steps, which two wavefronts have (in the same round, or the last one and, a round later, the first): the one hands its sums over
    // the first 32 rows on, and the other goes on from there behind the round's barrier, under its conversions.  (Its values left in LDS until then and added up at the end: 784-512-10, 64 workers of
    // 128 rows: 22.5 us, now 21.6; with sums per 32 rows, another order: 21.1.)  What a round leaves is overwritten three rounds later, two barriers behind its reader.
    float2 *const half_sums = reinterpret_cast<float2 *>(smem_raw + nsw * (7 * 2048));     // [3][nsw][64 lanes]
    const bool signals = (PL || HAS_D) && g.w_h != nullptr;
    auto put_band = [&](int kc, float2 v) __attribute__((always_inline)) {
      v.x += __shfl_xor(v.x, 32, 64);            // (the other half-wave: the rows offset by 4)
      v.y += __shfl_xor(v.y, 32, 64);
      if (lane < 32 && m0 + lane < g.M) {
        const int64_t o = ((int64_t)wk * g.nband + (kc >> 1)) * g.M + m0 + lane;
        g.dbpart[o] = v.x;
        if constexpr (!PL) g.ddbpart[o] = v.y;
      }
    };
    for (int round = 0, kc = w; round * nsw < nk; ++round, kc += nsw) {
      auto meet = [&]() __attribute__((always_inline)) { if (signals && nk > 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
      if (w >= nsw || kc >= nk) {               // (uniform: a wavefront without a step in this round)
        meet();
        continue;
      }
      u32x4 v[NA + NB][2];
#pragma unroll
      for (int sl = 0; sl < NA + NB; ++sl) {
        const bf16_t *src = (sl < NA ? pa[sl < NA ? sl : 0] + (((int64_t)(kc >> 2) * g.A.kt[0]) << 12)
                                     : pb[sl < NA ? 0 : sl - NA] + (((int64_t)(kc >> 2) * g.B.kt[0]) << 12)) + ((kc & 3) << 10);
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) v[sl][hh] = *reinterpret_cast<const u32x4 *>(src + (hh * 64 + lane) * 8);
      }
#pragma unroll
      for (int sl = 0; sl < NA + NB; ++sl)
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) *reinterpret_cast<u32x4 *>(area + sl * 1024 + (hh * 64 + lane) * 8) = v[sl][hh];
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // (one wavefront's LDS operations are carried out in order)
#pragma unroll
      for (int ks = 0; ks < BK; ks += 16) {
        auto fr = [&](int sl) __attribute__((always_inline)) { return tr_fragment(area + sl * 1024 + ks * 32, fro_tr); };
        // (roles as below: hi, lo, [difference] on the A side; hi, lo, [reference,] difference on the B side)
        const bf16x8 ah = fr(0), al = fr(1), bh = fr(NA), bl = fr(NA + 1), bd = fr(NA + NB - 1);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, acc1, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, acc1, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc1, 0, 0, 0);
        if constexpr (HAS_D) {
          const bf16x8 ad = fr(2), bx = NB == 4 ? fr(NA + 2) : bh;
          acc2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ad, bx, acc2, 0, 0, 0);
        }
        if constexpr (!PL) acc2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bd, acc2, 0, 0, 0);
      }
      if constexpr (PL || HAS_D) {
        if (signals) {
          // activation gradient of these 32 rows into the units of this block: the signals' block lies in the area as it is, a row per lane
          f32x16 c1, c2;                        // at theta and its difference
#pragma unroll
          for (int r = 0; r < 16; ++r) { c1[r] = 0.f; c2[r] = 0.f; }
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            auto sig = [&](int sl) __attribute__((always_inline)) { return *reinterpret_cast<const bf16x8 *>(area + (NA + sl) * 1024 + (lane & 31) * 32 + half * 16 + 8 * (lane >> 5)); };
            const bf16x8 gh = sig(0), gl = sig(1);
            c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gl, __builtin_bit_cast(bf16x8, wh[half]), c1, 0, 0, 0);
            c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gh, __builtin_bit_cast(bf16x8, wl[half]), c1, 0, 0, 0);
            c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gh, __builtin_bit_cast(bf16x8, wh[half]), c1, 0, 0, 0);
            if constexpr (!PL) {
              c2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sig(NB - 1), __builtin_bit_cast(bf16x8, wh[half]), c2, 0, 0, 0);
              c2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sig(2), __builtin_bit_cast(bf16x8, wd[half]), c2, 0, 0, 0);
            }
          }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          // masks as k_mm5 and this kernel's forward variant leave them: this block is quarter (i, j) of wavefront (wy, wx) of its 128 x 128 tile
          const uint16_t *mb = reinterpret_cast<const uint16_t *>(g.maskbits + ((((int64_t)wk * ((g.K + BM - 1) / BM) + (kc >> 2)) * ((g.M + BN - 1) / BN) + (m0 >> 7)) * kBlock +
                                                                                (((kc >> 1) & 1) * 2 + ((m0 >> 6) & 1)) * 64 + lane) * 2) + (kc & 1) * 2 + ((m0 >> 5) & 1);
          const uint32_t on = mb[0], on_ref = PL ? 0u : mb[4];
          // the values at theta and at the reference point
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const bool live = m0 + (lane & 31) < g.M && 32 * kc + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3) < g.K;
            const float x = live && ((on >> r) & 1) ? c1[r] : 0.f;
            c2[r] = live && ((on_ref >> r) & 1) ? c1[r] - c2[r] : 0.f;
            c1[r] = x;
          }
          float2 sum = make_float2(0.f, 0.f);
          if (!(kc & 1)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) { sum.x += c1[r]; sum.y += c1[r] - c2[r]; }
            if (kc + 1 < nk) half_sums[((round % 3) * nsw + w) * 64 + lane] = sum;
          }
          meet();
          if (kc & 1) sum = half_sums[(w > 0 ? (round % 3) * nsw + w - 1 : ((round + 2) % 3) * nsw + nsw - 1) * 64 + lane];
          const float2 first = sum;
#pragma unroll
          for (int r = 0; r < 16; r += 2) {
            const float x[2] = {c1[r], c1[r + 1]}, xr[2] = {c2[r], c2[r + 1]};
#pragma unroll
            for (int e = 0; e < 2; ++e) { sum.x += x[e]; sum.y += x[e] - xr[e]; }
            const uint32_t vh = f2bf_pk(x[0], x[1]), vr = f2bf_pk(xr[0], xr[1]), vd = f2bf_pk(x[0] - xr[0], x[1] - xr[1]);
            const uint32_t vl = f2bf_pk(x[0] - __uint_as_float(vh << 16), x[1] - __uint_as_float(vh & 0xffff0000u));
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const int o = (8 * (r >> 2) + 4 * (lane >> 5) + ((r + e) & 3)) * 32 + (lane & 31), sh = 16 * e;
              area[o] = (bf16_t)(vh >> sh); area[1024 + o] = (bf16_t)(vl >> sh);
              if constexpr (!PL) { area[2048 + o] = (bf16_t)(vd >> sh); area[3072 + o] = (bf16_t)(vr >> sh); }
            }
          }
          asm volatile("" ::: "memory");
          const int64_t out = tm((int64_t)wk * g.Bp + 32 * kc, m0, g.kto);
          bf16_t *const dst[4] = {g.o_h, g.o_l, g.o_d, g.o_r};
#pragma unroll
          for (int b = 0; b < (PL ? 2 : 4); ++b)
            if (dst[b] != nullptr) {
#pragma unroll
              for (int hh = 0; hh < 2; ++hh) *reinterpret_cast<u32x4 *>(dst[b] + out + (hh * 64 + lane) * 8) = *reinterpret_cast<const u32x4 *>(area + b * 1024 + (hh * 64 + lane) * 8);
            }
          if (kc & 1) put_band(kc, sum);
          else if (kc + 1 == nk) put_band(kc, first);
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the fragments are in registers before the area is written again
    }
    __syncthreads();                                         // the areas are done with: `red` lies over them
  } else {
  // Step kc's block of a tensor is 2 KB of consecutive memory: moved straight to LDS, 1 KB per instruction, its 16-byte pieces in the order of lds_piece.  (Fragments
  // read from memory are 16 bytes of a row each, 64 bytes apart: a wave-load of them took the CU's address unit some 70 cycles, 16300 for the four steps of a wavefront's
  // 784 inputs.  Launches, us: 784-500-10 with 10 workers of 12 rows: hidden layer 10.9, now 9.1, loss 10.8, now 9.0; 617-301-150-26, always, 24 workers of 100: 11.4, now 9.2;
  // loss of 3072-1024-1024-10 with 16 workers of 256: 19.6, now 16.2.)
  const int64_t offa = (((int64_t)(m0 >> 7) * g.A.kt[0]) << 12) + ((m0 & 127) << 5), offb = (((int64_t)(cb >> 2) * g.B.kt[0]) << 12) + ((cb & 3) << 10);
  // (scalar loads: a wait for a vector load's value would be one for all operands in flight)
  // (and without a branch around them: one round trip for both, where a branch each waited for the arguments that it looks at, then for its value)
  const int32_t rep_there = scalar_load((g.rep ? g.rep : s.tau) + wk), tau_there = scalar_load(s.tau + wk);
  int64_t grow = 0;
  if constexpr (EPI == EPI_LOSS) grow = g.grow[(int64_t)wk * g.Bp + min(m0 + (t >> 4), g.M - 1)];
#pragma unroll
  for (int sl = 0; sl < NA; ++sl) pa[sl] = g.A.ptr[sl] + (int64_t)wk * g.A.bstride[0] + offa;      // (one stride for all of A, none for W: launch_mm5)
  const uint32_t area = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem_raw + w * AREA;
  const uint32_t from[2] = {(uint32_t)lds_piece(lane) * 16u, (uint32_t)lds_piece(64 + lane) * 16u};
  auto move = [&](const bf16_t *p, int kc, int sl) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 2; ++c) mm_load(p + ((int64_t)kc << 12), from[c], area + sl * 2048 + c * 1024);
  };
  if (w < nk) {
#pragma unroll
    for (int sl = 0; sl < NA; ++sl) move(pa[sl], w, sl);
  }
  const int rep_wk = g.rep ? rep_there : wk, tau_wk = s.rule == CADA_RULE_CADA2 ? tau_there : 0;
#pragma unroll
  for (int sl = 0; sl < NB; ++sl) pb[sl] = g.B.ptr[sl] + (!PL && sl == NB - 1 ? (int64_t)rep_wk * g.B.bstride[sl] : 0) + offb;
  if (w < nk) {
#pragma unroll
    for (int sl = 0; sl < NB; ++sl) move(pb[sl], w, NA + sl);
  }
  // Sixteen lanes share a row of the 32 x 32 result, each with two of the (at most 32) classes or units.  The biases and their differences to the reference point are
  // asked for behind the first step's operands, the row's label in its products, so that their latency passes under these.
  const int c0 = 32 * cb + 2 * (t & 15);
  {
    const RefPtr ref = theta_ref_of(s, tau_wk);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int64_t i = g.offb + min(c0 + e, g.N - 1);           // (of an absent class: not used)
      bz[e] = s.theta[i];
      if constexpr (!PL) dbz[e] = delta_theta(s, ref, i);
    }
  }
  auto ask_label = [&]() __attribute__((always_inline)) { if constexpr (EPI == EPI_LOSS) label = static_cast<const int32_t *>(s.y)[grow]; };
  if (w >= nk) ask_label();
  const unsigned char *mine = smem_raw + w * AREA;
  const int fro = lds_piece((lane & 31) * 4 + (lane >> 5)) * 16;           // this lane's fragment of the first half step (the second: 32 bytes further, in lds_piece's order)
  // steps first, first + stride, ...; then the steps from `then` on are next (nk: none)
  const int stride = TWICE ? 2 * nw : nw;
  auto walk = [&](int first, int then, f32x16 &acc1, f32x16 &acc2) __attribute__((always_inline)) {
    for (int kc = first; kc < nk; kc += stride) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      u32x4 fa[2][NA], fb[2][NB];          // (kept as integer vectors: arrays of them stay in registers)
#pragma unroll
      for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int sl = 0; sl < NA; ++sl) fa[half][sl] = *reinterpret_cast<const u32x4 *>(mine + sl * 2048 + (fro ^ (32 * half)));
#pragma unroll
        for (int sl = 0; sl < NB; ++sl) fb[half][sl] = *reinterpret_cast<const u32x4 *>(mine + (NA + sl) * 2048 + (fro ^ (32 * half)));
      }
      if (kc == w) ask_label();
      const int next = kc + stride < nk ? kc + stride : then;
      if (next < nk) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // (the fragments are in registers before the area is written again)
#pragma unroll
        for (int sl = 0; sl < NA; ++sl) move(pa[sl], next, sl);
#pragma unroll
        for (int sl = 0; sl < NB; ++sl) move(pb[sl], next, NA + sl);
      }
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        // (the roles of the tensors follow from their number: hi, lo, [difference, [reference]] on the A
        // side, hi, lo, [reference,] difference on the B side; the host checks it)
        auto fr = [&](const u32x4 &v) __attribute__((always_inline)) { return __builtin_bit_cast(bf16x8, v); };
        const bf16x8 ah = fr(fa[half][0]), al = fr(fa[half][1]), bh = fr(fb[half][0]), bl = fr(fb[half][1]), bd = fr(fb[half][NB - 1]);
        const bf16x8 ar = NA == 4 ? fr(fa[half][NA - 1]) : ah;
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, acc1, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, acc1, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc1, 0, 0, 0);
        if constexpr (HAS_D) {
          const bf16x8 ad = fr(fa[half][2]), bx = NB == 4 ? fr(fb[half][2]) : bh;
          acc2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ad, bx, acc2, 0, 0, 0);
        }
        if constexpr (!PL) acc2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ar, bd, acc2, 0, 0, 0);
      }
    }
  };
  walk(w, TWICE ? w + nw : nk, acc1, acc2);
  if constexpr (TWICE) walk(w + nw, nk, later1, later2);
  }
  auto put_part = [&](const f32x16 &acc1, const f32x16 &acc2) __attribute__((always_inline)) {
    float *r1 = EPI == EPI_DW ? red + w * 2 * 1024 : part_of(w, 0), *r2 = EPI == EPI_DW ? r1 + 1024 : part_of(w, 1);      // (not EPI_DW: over this wavefront's own blocks)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      r1[r * 64 + lane] = acc1[r];
      if constexpr (!PL) r2[r * 64 + lane] = acc2[r];
    }
  };
  if (w < nsw) put_part(acc1, acc2);
  lds_sync();
  if constexpr (EPI == EPI_FWD_HIDDEN) {
    // bias and ReLU of both evaluations; the block is 2 KB of consecutive memory of each output tensor
    uint8_t (*pos[2])[33];                          // [32]: value at theta, at the reference point is positive (in the room behind the partial results)
    pos[0] = reinterpret_cast<uint8_t (*)[33]>(smem_raw + ROOM); pos[1] = reinterpret_cast<uint8_t (*)[33]>(smem_raw + AREA + ROOM);
    constexpr int ROWS = TWICE ? 2 : 1, NW = 8 / ROWS;      // rows of a thread; wavefronts of the launch (launch_skinny_as)
    const int c0 = 2 * (t & 15);
    float zs[ROWS][2], ds[ROWS][2];
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
#pragma unroll
      for (int e = 0; e < 2; ++e) { zs[i][e] = bz[e]; ds[i][e] = dbz[e]; }
    auto add_parts = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        const int rl = (t >> 4) + 16 * i, ra = 4 * (rl >> 3) + (rl & 3), lb = 32 * ((rl >> 2) & 1);      // (accumulator element of a row: as below)
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int ww = 0; ww < NW; ++ww) {
            zs[i][e] += part_of(ww, 0)[ra * 64 + lb + c0 + e];
            if constexpr (!PL) ds[i][e] += part_of(ww, 1)[ra * 64 + lb + c0 + e];
          }
      }
    };
    add_parts();
    if (TWICE && nk > nw) {                          // (else the second shares are empty)
      lds_sync();
      put_part(later1, later2);
      lds_sync();
      add_parts();
    }
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const int rl = (t >> 4) + 16 * i;
      float x[2], xref[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const bool live = m0 + rl < g.M && 32 * cb + c0 + e < g.N;             // (else padding: zero)
        x[e] = live ? fmaxf(zs[i][e], 0.f) : 0.f;
        xref[e] = live && !PL ? fmaxf(zs[i][e] - ds[i][e], 0.f) : 0.f;
      }
      const uint32_t vh = f2bf_pk(x[0], x[1]), vr = f2bf_pk(xref[0], xref[1]);
      // ReLU masks where k_mm5's activation gradient looks for them (sign of the stored, rounded values): this block is quarter
      // (i, j) of wavefront (wy, wx) of its 128 x 128 tile, sixteen bits of each of the wavefront's lanes
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        pos[0][rl][c0 + e] = __uint_as_float(e ? vh & 0xffff0000u : vh << 16) > 0.f;
        pos[1][rl][c0 + e] = __uint_as_float(e ? vr & 0xffff0000u : vr << 16) > 0.f;
      }
      const int64_t o = tm((int64_t)wk * g.Bp + m0 + rl, 32 * cb + c0, g.kto);
      *reinterpret_cast<uint32_t *>(g.o_h + o) = vh;
      *reinterpret_cast<uint32_t *>(g.o_l + o) = f2bf_pk(x[0] - __uint_as_float(vh << 16), x[1] - __uint_as_float(vh & 0xffff0000u));
      if constexpr (!PL) {
        *reinterpret_cast<uint32_t *>(g.o_d + o) = f2bf_pk(x[0] - xref[0], x[1] - xref[1]);
        *reinterpret_cast<uint32_t *>(g.o_r + o) = vr;
      }
    }
    lds_sync();
    if (t < 2 * kWave) {
      const int ref = t >> 6;
      uint32_t bits = 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) bits |= (uint32_t)pos[ref][8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)][lane & 31] << r;
      const int by = m0 >> 7, wy = (m0 >> 6) & 1, i = (m0 >> 5) & 1, wx = (cb >> 1) & 1, j = cb & 1;
      const int gx = (g.N + BN - 1) / BN, gy = (g.M + BM - 1) / BM;
      uint64_t *word = g.maskbits + ((((int64_t)wk * gy + by) * gx + (cb >> 2)) * kBlock + (wy * 2 + wx) * 64 + lane) * 2 + ref;
      reinterpret_cast<uint16_t *>(word)[i * 2 + j] = (uint16_t)bits;
    }
    return;
  }
  if constexpr (EPI == EPI_LOSS) {
    // softmax cross-entropy on the tile's rows: G = (P - onehot)/B, dG = (P - Pref)/B.  With e_i = exp(-dz_i) and
    // T = sum_j P_j e_j the reference probabilities are Pref_i = P_i e_i / T, so
    //     P_i - Pref_i = P_i (S - expm1(-dz_i)) / (1 + S),  S = sum_j P_j expm1(-dz_j) = T - 1,
    // which keeps the digits of a small difference (no subtraction of nearly equal probabilities) and
    // is used while every |dz_j| of the row is below 1/2.  For larger differences (a reference point
    // many iterations old) 1 + S cancels instead (T can be far below float32's resolution of 1), so
    // there P_i - Pref_i is formed directly with Pref = softmax(z - dz), the exponents shifted by their
    // maximum; the difference is then no longer small against its operands.
    // Also the sums over the tile's rows of G and dG: the last layer's bias gradient and its innovation, which the
    // weight-gradient launch of that layer adds up over the row blocks.
    auto part = [&](int ww, int cp_) __attribute__((always_inline)) { return reinterpret_cast<float *>(smem_raw + ww * AREA + ROOM) + cp_ * 4; };      // [16][4] per wavefront
    const int rl = t >> 4, cp = t & 15, c0 = 2 * cp;
    const bool on[2] = {c0 < g.N, c0 + 1 < g.N};
    const int row = m0 + rl;
    const bool live = row < g.M;                    // (rows past the minibatch are padding)
    // accumulator element (r, lane) is (row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32) of the tile
    const int ra = 4 * (rl >> 3) + (rl & 3), lb = 32 * ((rl >> 2) & 1);
    const float invB = 1.0f / (float)s.B;
    float z[2], x[2], ndz[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float zs = 0.f, ds = 0.f;
      for (int ww = 0; ww < nw; ++ww) {
        zs += part_of(ww, 0)[ra * 64 + lb + c0 + e];
        if constexpr (!PL) ds += part_of(ww, 1)[ra * 64 + lb + c0 + e];
      }
      z[e] = on[e] ? zs + bz[e] : -INFINITY;
      ndz[e] = on[e] ? -(ds + dbz[e]) : 0.f;
      x[e] = expm1f(ndz[e]);
    }
    const float zr[2] = {z[0] + ndz[0], z[1] + ndz[1]};       // logits at the reference point (-inf for an absent class)
    float nabs = fmaxf(fabsf(ndz[0]), fabsf(ndz[1]));        // (an absent class contributes 0)
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) nabs = fmaxf(nabs, __shfl_xor(nabs, o, 64));
    const bool far = !(nabs < 0.5f);             // (also taken by a NaN, which then shows in the result)
    float zmax = fmaxf(z[0], z[1]);
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, o, 64));
#pragma unroll
    for (int e = 0; e < 2; ++e) z[e] = on[e] ? expf(z[e] - zmax) : 0.f;
    const float den = group16_sum(z[0] + z[1]);
    z[0] = z[0] / den; z[1] = z[1] / den;
    const float S = group16_sum(fmaf(z[0], x[0], z[1] * x[1]));
    // the direct form: Pref = softmax of the reference logits z - dz, shifted by their maximum
    float rmax = fmaxf(zr[0], zr[1]);
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) rmax = fmaxf(rmax, __shfl_xor(rmax, o, 64));
    const float er[2] = {on[0] ? expf(zr[0] - rmax) : 0.f, on[1] ? expf(zr[1] - rmax) : 0.f};
    const float rden = group16_sum(er[0] + er[1]);
    // (row, class) tensors: a row's classes are consecutive, written two at a time (an absent odd
    // class is a zero in the padding)
    uint32_t ph = 0, pl = 0, pd = 0, pr = 0;
    float sumG[2] = {0.f, 0.f}, sumD[2] = {0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      if (on[e] && live) {
        const int c = c0 + e;
        const float gl = (z[e] - (c == label ? 1.f : 0.f)) * invB;
        const float dg = (far ? z[e] - er[e] / rden : z[e] * (S - x[e]) / (1.0f + S)) * invB;
        const bf16_t hi = f2bf(gl), lo = f2bf(gl - bf2f(hi)), bd = f2bf(dg), br = f2bf(gl - dg);
        ph |= (uint32_t)hi << (16 * e); pl |= (uint32_t)lo << (16 * e); pd |= (uint32_t)bd << (16 * e); pr |= (uint32_t)br << (16 * e);
        sumG[e] = gl;
        sumD[e] = dg;
      }
    }
    if (on[0] && live) {
      const int64_t o = tm((int64_t)wk * g.Bp + row, 0, g.kto) + c0;          // classes 0..31 lie in the row's first chunk
      *reinterpret_cast<uint32_t *>(g.o_h + o) = ph; *reinterpret_cast<uint32_t *>(g.o_l + o) = pl;
      if constexpr (!PL) *reinterpret_cast<uint32_t *>(g.o_d + o) = pd;
      if (!PL && g.o_r) *reinterpret_cast<uint32_t *>(g.o_r + o) = pr;
    }
    // sums over the tile's rows in a fixed order: the wavefront's four rows, then the wavefronts
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      sumG[e] += __shfl_xor(sumG[e], 16, 64); sumG[e] += __shfl_xor(sumG[e], 32, 64);
      sumD[e] += __shfl_xor(sumD[e], 16, 64); sumD[e] += __shfl_xor(sumD[e], 32, 64);
    }
    if (lane < 16) *reinterpret_cast<v4s *>(part(w, cp)) = v4s{sumG[0], sumG[1], sumD[0], sumD[1]};
    lds_sync();
    if (w == 0 && lane < g.N) {
      const int c = lane;
      float gsum = 0.f, iv = 0.f;
      for (int ww = 0; ww < nw; ++ww) { gsum += part(ww, c >> 1)[c & 1]; iv += part(ww, c >> 1)[2 + (c & 1)]; }
      float *q = g.lastb + ((((int64_t)wk * g.nrb + bx) * 32 + c) << 1);
      q[0] = gsum; q[1] = iv;
    }
    return;
  }
  // The 16 x 64 sums over the threads, four at a time, each the sum of the wavefronts' partial results in wavefront order
  float sq = 0.f;
  if constexpr (EPI == EPI_DW) {
    float *gf = s.gbuf16 ? nullptr : fresh_grad(s, wk) + g.offW;
    bf16_t *gf16 = s.gbuf16 ? fresh_grad16(s, wk) + g.offW : nullptr;
    bf16_t *ivf = cada1 ? fresh_innov(s, wk) + g.offW : nullptr;
    for (int e0 = t; e0 < 16 * 64; e0 += 4 * (int)blockDim.x) {
      if (cada1 && e0 != t) ask_old(e0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = e0 + i * (int)blockDim.x;
        if (e >= 16 * 64) break;
        float v = 0.f, iv = 0.f;
        for (int ww = 0; ww < nsw; ++ww) {
          v += red[(ww * 2 + 0) * 1024 + e];
          if constexpr (!PL) iv += red[(ww * 2 + 1) * 1024 + e];
        }
        const int r = e >> 6, ln = e & 63, row = m0 + 8 * (r >> 2) + 4 * (ln >> 5) + (r & 3), col = ln & 31;
        if (row < g.M && col < g.N) {
          const int64_t o = (int64_t)row * g.N + col;
          if (gf16) gf16[o] = f2bf(v); else gf[o] = v;
          if constexpr (!PL) {
            if (cada1) { ivf[o] = f2bf(iv); iv -= bf2f(old_iv[i]); }
            sq = fmaf(iv, iv, sq);
          }
        }
      }
    }
  }
  if constexpr (EPI == EPI_DW && !PL) {
    const float ws = wave_sum(sq);
    __syncthreads();
    if (lane == 0) red[w] = ws;
    __syncthreads();
    if (t == 0) {
      float tot = 0.f;
      for (int ww = 0; ww < nw; ++ww) tot += red[ww];
      s.lhs_part[(int64_t)wk * s.n_lhs_part + g.lhs_slot0 + bx] = tot;
    }
  }
}

template <int EPI, int NA, int NB, bool HAS_D, bool TWICE = false>
__global__ __launch_bounds__(TWICE ? kBlock : 2 * kBlock) void k_skinny(const Mm5Args g) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  skinny<EPI, NA, NB, HAS_D, TWICE>(g, smem_raw, blockIdx.x);
}

// The loss and the last layer's weight gradient in one launch, where a worker's rows are one block and the workgroups are all there at once: each of a worker's workgroups forms the
// worker's signals for itself and takes them up again where it has put them (every one the same values to the same place), which costs what the loss costs alone and saves a launch.
template <bool PL>
__global__ __launch_bounds__(2 * kBlock) void k_loss_dw(const Mm5Args loss, const Mm5Args dw) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  if constexpr (PL) skinny<EPI_LOSS, 2, 2, false>(loss, smem_raw, 0);
  else skinny<EPI_LOSS, 4, 3, true>(loss, smem_raw, 0);
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");      // (signals and sums have arrived; the areas are written again)
  if constexpr (PL) skinny<EPI_DW, 2, 2, false>(dw, smem_raw, blockIdx.x);
  else skinny<EPI_DW, 3, 4, true>(dw, smem_raw, blockIdx.x);
}

// ------------------------------------------------------------------------------------------
// plan
// ------------------------------------------------------------------------------------------
namespace {
constexpr size_t kAlignB = 256;
struct Carve {
  char *base; size_t off;
  template <typename T> T *take(size_t n) {
    T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
    off = (off + n * sizeof(T) + kAlignB - 1) / kAlignB * kAlignB;
    return p;
  }
};

// elements of a chunked tensor of r rows and k contraction indices (whole chunks)
size_t tm_elems(int64_t r, int64_t k) { return (size_t)tiles128(r) * chunks32(k) * TILE; }

void layout(MlpPlan &P, const cada_config *cfg, int64_t total_rows, Carve &w) {
  P.L = cfg->n_layers; P.M = cfg->M; P.B = cfg->B; P.rule = cfg->rule;
  P.RT = tiles128(cfg->B);
  P.Bp = P.RT * 128;
  P.Rp = (int64_t)cfg->M * P.Bp;
  P.total_rows = total_rows;
  for (int l = 0; l <= P.L; ++l) { P.d[l] = cfg->layer_dims[l]; P.kta[l] = chunks32(P.d[l]); }
  int64_t o = 0, wt = 0, wn = 0;
  int slot = 0, maxh = 1;
  for (int l = 1; l <= P.L; ++l) {
    P.offW[l - 1] = o; o += (int64_t)P.d[l - 1] * P.d[l];
    P.offb[l - 1] = o; o += P.d[l];
    P.wt_off[l - 1] = wt; wt += (int64_t)tm_elems(P.d[l], P.d[l - 1]);
    P.wn_off[l - 1] = wn; if (l >= 2) wn += (int64_t)tm_elems(P.d[l - 1], P.d[l]);
    P.lhs_w_slot[l - 1] = slot; slot += 4 * tiles128(P.d[l - 1]) * tiles128(P.d[l]);
    P.lhs_b_slot[l - 1] = slot; slot += (P.d[l] + mlp_bias_cols(P.rule) - 1) / mlp_bias_cols(P.rule);
    if (l < P.L && P.d[l] > maxh) maxh = P.d[l];
  }
  P.wt_total = wt; P.wn_total = wn;
  P.nW = (cfg->rule == CADA_RULE_CADA2) ? cfg->M : 1;
  P.ldx = P8(P.d[0]);
  const size_t Rp = (size_t)P.Rp;
  P.Xh = w.take<bf16_t>((size_t)total_rows * P.ldx);
  P.Xl = w.take<bf16_t>((size_t)total_rows * P.ldx);
  P.XGh = w.take<bf16_t>(tm_elems(Rp, P.d[0]));
  P.XGl = w.take<bf16_t>(tm_elems(Rp, P.d[0]));
  P.grow = w.take<int64_t>(Rp);
  P.rep = w.take<int32_t>((size_t)cfg->M);
  P.WTh = w.take<bf16_t>((size_t)wt); P.WTl = w.take<bf16_t>((size_t)wt); P.dWT = w.take<bf16_t>((size_t)wt * P.nW);
  P.WNh = w.take<bf16_t>((size_t)wn + 8); P.WNl = w.take<bf16_t>((size_t)wn + 8); P.dWN = w.take<bf16_t>((size_t)wn * P.nW + 8);
  for (int l = 1; l < P.L; ++l) {
    const size_t n = tm_elems(Rp, P.d[l]);
    P.Ah[l] = w.take<bf16_t>(n); P.Al[l] = w.take<bf16_t>(n); P.dA[l] = w.take<bf16_t>(n); P.Aref[l] = w.take<bf16_t>(n);
    P.maskbits[l] = w.take<uint64_t>((size_t)cfg->M * P.RT * tiles128(P.d[l]) * kBlock * 2);
  }
  for (int l = 1; l <= P.L; ++l) {
    const size_t n = tm_elems(Rp, P.d[l]);
    P.Gh[l] = w.take<bf16_t>(n); P.Gl[l] = w.take<bf16_t>(n); P.dG[l] = w.take<bf16_t>(n);
    P.Gref[l] = l >= 2 ? w.take<bf16_t>(n) : nullptr;       // (the first layer has no propagated difference to pair it with)
  }
  (void)w.take<float>(Rp * P.d[P.L]);             // (not used any more; the room keeps the layout of saved checkpoint blocks)
  (void)w.take<float>(Rp * P.d[P.L]);
  P.dbpart[0] = w.take<float>((size_t)cfg->M * 2 * P.RT * maxh);
  P.ddbpart[0] = w.take<float>((size_t)cfg->M * 2 * P.RT * maxh);
  P.band_floats = (size_t)cfg->M * 2 * P.RT * maxh;
  P.lastb = w.take<float>((size_t)cfg->M * (P.Bp / 32) * 32 * 2);
}
}  // namespace

// Number of partial sums of the left-hand side per worker (four per weight-gradient tile, one per
// bias_cols biases).
int mlp_lhs_slots(const cada_config *cfg, int bias_cols) {
  int slot = 0;
  for (int l = 1; l <= cfg->n_layers; ++l)
    slot += 4 * tiles128(cfg->layer_dims[l - 1]) * tiles128(cfg->layer_dims[l]) + (cfg->layer_dims[l] + bias_cols - 1) / bias_cols;
  return slot;
}

size_t mlp_workspace_bytes(const cada_config *cfg, const int64_t total_rows) {
  if (cfg->gemm_dtype != CADA_GEMM_BF16) { set_error("the MLP model computes its contractions in bf16 (gemm_dtype must be CADA_GEMM_BF16)"); return 0; }
  if (cfg->layer_dims[cfg->n_layers] > 32) { set_error("at most 32 classes"); return 0; }
  for (int l = 0; l <= cfg->n_layers; ++l)    // the kernels index one worker's activations with 32 bits
    if (((int64_t)cfg->B + 128) * (cfg->layer_dims[l] + 32) >= (1ll << 31)) { set_error("B x layer width must stay below 2^31"); return 0; }
  {   // the staging launch numbers its 64 x 64 tiles of the minibatch and of every weight copy in one grid dimension
    const int64_t nz = (cfg->rule == CADA_RULE_CADA2) ? cfg->M + 1 : 2;
    int64_t nblk = ((int64_t)cfg->layer_dims[0] + 71) / 64 * ((cfg->B + 63) / 64) * cfg->M;
    for (int l = 1; l <= cfg->n_layers; ++l)
      nblk += ((int64_t)cfg->layer_dims[l] + 63) / 64 * ((cfg->layer_dims[l - 1] + 63) / 64) * nz;
    if (nblk >= (1ll << 31) - 1) { set_error("too many operand tiles for one launch (M x layer sizes / 4096 must stay below 2^31)"); return 0; }
  }
  MlpPlan P;
  Carve w{nullptr, 0};
  layout(P, cfg, total_rows, w);
  return w.off + kAlignB;
}

// The partial sums of the left-hand side (the rules without a second gradient: two per block of k_lag_lhs) and the rule's inputs, in front of the evaluation's scratch.
static int lhs_parts(const cada_config *cfg) {
  return cfg->rule == CADA_RULE_LAG || cfg->rule == CADA_RULE_ALWAYS ? 2 * lag_blocks(cfg->p) : mlp_lhs_slots(cfg, mlp_bias_cols(cfg->rule));
}
static size_t rule_room(const cada_config *cfg) { return (rule_in_bytes(cfg->M) + kAlignB - 1) / kAlignB * kAlignB; }
static size_t lhs_bytes(const cada_config *cfg) {
  return ((size_t)cfg->M * lhs_parts(cfg) * sizeof(float) + kAlignB - 1) / kAlignB * kAlignB + rule_room(cfg);
}

// The sums per band of the signals of the second, fourth, ... hidden layer (two arrays), behind them.
static size_t bands_bytes(const MlpPlan &P) { return P.L < 3 ? 0 : 2 * ((P.band_floats * sizeof(float) + kAlignB - 1) / kAlignB * kAlignB); }

size_t mlp_scratch_bytes(const cada_config *cfg, const int64_t total_rows) {
  MlpPlan P;
  Carve w{nullptr, 0};
  layout(P, cfg, total_rows, w);
  return lhs_bytes(cfg) + bands_bytes(P) + mlp_eval_bytes(P) + kAlignB;
}

int mlp_plan(Ctx *c, const cada_config *cfg, char *base, size_t offset, size_t scratch, int64_t total_rows) {
  if (mlp_workspace_bytes(cfg, total_rows) == 0) return CADA_EUNSUPPORTED;
  MlpPlan *P = new (std::nothrow) MlpPlan();
  if (!P) { set_error("out of host memory"); return CADA_EINVAL; }
  Carve w{base, (offset + kAlignB - 1) / kAlignB * kAlignB};
  layout(*P, cfg, total_rows, w);
  scratch = (scratch + kAlignB - 1) / kAlignB * kAlignB;
  c->s.lhs_part = reinterpret_cast<float *>(base + scratch);
  c->s.n_lhs_part = lhs_parts(cfg);
  decide_plan(c, base + scratch + lhs_bytes(cfg) - rule_room(cfg));
  if (P->L >= 3) {
    P->dbpart[1] = reinterpret_cast<float *>(base + scratch + lhs_bytes(cfg));
    P->ddbpart[1] = reinterpret_cast<float *>(base + scratch + lhs_bytes(cfg) + bands_bytes(*P) / 2);
  }
  P->eval = base + scratch + lhs_bytes(cfg) + bands_bytes(*P);
  c->mlp = P;
  c->n_phases = 0;
  c->phase_names[c->n_phases++] = "mlp_gradients";
  if (!c->decide) c->phase_names[c->n_phases++] = "rule";
  c->phase_names[c->n_phases++] = c->decide ? "rule_and_server_update" : "server_update";
  return CADA_OK;
}

void mlp_free(Ctx *c) {
  delete static_cast<MlpPlan *>(c->mlp);
  c->mlp = nullptr;
}

// ------------------------------------------------------------------------------------------
// small kernels
// ------------------------------------------------------------------------------------------
// float32 features -> bf16 hi/lo copies with padded leading dimension (once, at init)
__global__ void k_x_to_bf16(const float *X, bf16_t *Xh, bf16_t *Xl, int64_t rows, int d0, int64_t ldx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * ldx) return;
  const int64_t r = i / ldx; const int c = (int)(i % ldx);
  const float x = c < d0 ? X[r * d0 + c] : 0.f;
  const bf16_t hi = f2bf(x);
  Xh[i] = hi;
  Xl[i] = f2bf(x - bf2f(hi));
}

// Per-step staging of the contractions' operands, one launch: the chunked copy of the gathered
// minibatch, and bf16 copies (in both orientations) of every layer's weights and of their
// differences to the reference points.  The blocks of the launch are numbered through the parts
// (minibatch tiles first, then the layers in order); the parts are independent of each other.
struct PrepLayer {
  bf16_t *WTh, *WTl, *dWT, *WNh, *WNl, *dWN;   // already offset to this layer
  int64_t offW;
  int din, dout;
  int64_t ktt, ktn;      // chunks32(din), chunks32(dout)
  int want_n;            // also write the [in][out] orientation (layers >= 2)
  int gx, gy;            // 64 x 64 tiles over (dout, din)
};

struct StageArgs {
  DevState s;
  // minibatch: XG(m*Bp + b, c) = X[grow[m*Bp + b]][c]
  const bf16_t *Xh, *Xl; int64_t ldx;
  const int32_t *idx;    // [M][B] sampled rows, local to each worker's shard
  int64_t *grow;         // out: grow[m*Bp + b] = global row of worker m's b-th sample (b < B)
  bf16_t *XGh, *XGl;
  int d0, B, Bp; int64_t ktx;
  int gx, gy;            // 64 x 64 tiles over (ldx, B)
  // weights
  PrepLayer layer[CADA_MAX_LAYERS];
  int n_layers, nz;      // nz = 1 + groups of blocks for the differences (one for CADA1, none for the rules without)
  int64_t wt_total, wn_total;
  // CADA2 only, else null: workers whose last upload happened at the same iteration share their
  // reference point theta^{k - tau}, hence the difference theta - theta_ref and its bf16 copies;
  // out: rep[m] = the first worker with worker m's (clamped) tau.  Only that worker's difference is computed.
  int32_t *rep;
  int z_groups;          // groups of blocks that share these workers out: k_stage<true>, every block makes the list of them; else a group for every worker, which finds out for itself whether it is a first one
  uint32_t first[CADA_MAX_LAYERS + 2];   // first block of the minibatch part (0), of each layer, and the total
  int rule_block;        // 1: one more block, in front of them, takes the rule's inputs down
  RuleInputs rule_in;
};

// A 64 x 64 tile of the minibatch, moved 16 bytes (8 values) per lane: the sampled rows of X's bf16
// copies go to XG as they are.
__device__ __forceinline__ void stage_minibatch(const StageArgs &a, int bx, int by, int m) {
  const int c0 = bx * 64, b0 = by * 64;
  const int t = threadIdx.x;
  const int cg = (t & 7) * 8;                   // this thread's 8 columns
  const int64_t row0 = a.s.row_off[m], n_m = a.s.row_off[m + 1] - row0;
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int r = (t >> 3) + 32 * pass, b = b0 + r, c = c0 + cg;
    if (b < a.B && c < a.ldx) {                 // (columns from d0 to ldx hold zeros in X's copies)
      int64_t row = a.idx[(int64_t)m * a.B + b];
      if (row < 0 || row >= n_m) {              // reported once per sample, by the tile that also records the row
        if (bx == 0 && cg == 0) atomicOr(a.s.err, 1u);
        row = row < 0 ? 0 : n_m - 1;
      }
      row += row0;
      if (bx == 0 && cg == 0) a.grow[(int64_t)m * a.Bp + b] = row;
      const int64_t src = row * a.ldx + c;
      const u32x4 vh = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(a.Xh + src));      // (a sampled row is not read again soon)
      const u32x4 vl = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(a.Xl + src));
      const int64_t dst = tm((int64_t)m * a.Bp + b, c, a.ktx);
      *reinterpret_cast<u32x4 *>(a.XGh + dst) = vh;
      *reinterpret_cast<u32x4 *>(a.XGl + dst) = vl;
    }
  }
}

constexpr int kStageDelays = 64 * 65;            // delays that the list's table has room for (it lies where a tile does later)
// A 64 x 64 tile of one layer's weights (z = 0: hi and lo parts of W) or of their differences to the
// reference points of group z (worker z - 1's where there is no list), 8 values per lane: rows of W are read (4-byte aligned
// 16-byte loads) and written as they are, and turned through LDS for the other orientation.
// LIST: the differences go by the list of distinct reference points (CADA2, up to 256 workers and 4159 delays); an instance of its own, whose registers the others need not pay for.
template <bool LIST>
__device__ __forceinline__ void stage_weights(const StageArgs &a, const PrepLayer &p, unsigned char *sm, int bx, int by, int z, bool first_tile) {
  const DevState &s = a.s;
  typedef float tile_t[64][65];
  static_assert(sizeof(tile_t) >= kStageDelays * sizeof(int32_t), "");
  tile_t &tile = *reinterpret_cast<tile_t *>(sm);
  const int o0 = bx * 64, i0 = by * 64;
  const int t = threadIdx.x;
  const int og = (t & 7) * 8;
  auto one = [&](const bool is_w, const int m, const int32_t tau) __attribute__((always_inline)) {
    const RefPtr ref = theta_ref_at(s, tau);
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      const int r = (t >> 3) + 32 * pass, i = i0 + r, o = o0 + og;
      float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (i < p.din && o < p.dout) {
        const int64_t src = p.offW + (int64_t)i * p.dout + o;
        // (whole quads also where the row ends inside them: up to seven floats past it, of the next row, the bias or what follows in the workspace, which are not used; the two quads of a tensor
        // one after the other: they share a line, and with the first quads of all four tensors in front 784-512-10, 64 workers of 128 rows, takes 1 us more per step, 23.4 for 22.2 in this launch)
        auto both = [&](const float *from, f32x4u (&x)[2]) __attribute__((always_inline)) { x[0] = *reinterpret_cast<const f32x4u *>(from + src); x[1] = *reinterpret_cast<const f32x4u *>(from + src + 4); __builtin_amdgcn_sched_barrier(0); };
        f32x4u x[2];
        both(s.theta, x);
        if (!is_w) {
          f32x4u xl[2], rh[2], rl[2];
          both(ref.hi, rh); both(s.theta_lo, xl); both(ref.lo, rl);
#pragma unroll
          for (int q = 0; q < 2; ++q) x[q] = (x[q] - rh[q]) + (xl[q] - rl[q]);      // the same expression as delta_theta
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = x[e >> 2][e & 3];
        if (o + 8 > p.dout) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = o + e < p.dout ? v[e] : 0.f;
        }
        if (p.want_n) {                             // (values past dout are zeros, like the padding they land in)
          const int64_t dn = tm(i, o, p.ktn);
          bf16_t h8[8], l8[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) { h8[e] = f2bf(v[e]); l8[e] = f2bf(v[e] - bf2f(h8[e])); }
          if (is_w) { *reinterpret_cast<u32x4 *>(p.WNh + dn) = pack8(h8); *reinterpret_cast<u32x4 *>(p.WNl + dn) = pack8(l8); }
          else *reinterpret_cast<u32x4 *>(p.dWN + (int64_t)m * a.wn_total + dn) = pack8(h8);
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) tile[r][og + e] = v[e];
    }
    __syncthreads();
    const int oo = t & 63;
    if (o0 + oo < p.dout) {
#pragma unroll
      for (int pass = 0; pass < 2; ++pass) {
        const int ig = ((t >> 6) + 4 * pass) * 8;
        if (i0 + ig < p.din) {                      // (rows past din are zeros in the tile)
          bf16_t h8[8], l8[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) { const float x = tile[ig + e][oo]; h8[e] = f2bf(x); l8[e] = f2bf(x - bf2f(h8[e])); }
          const int64_t dt = tm(o0 + oo, i0 + ig, p.ktt);
          if (is_w) { *reinterpret_cast<u32x4 *>(p.WTh + dt) = pack8(h8); *reinterpret_cast<u32x4 *>(p.WTl + dt) = pack8(l8); }
          else *reinterpret_cast<u32x4 *>(p.dWT + (int64_t)m * a.wt_total + dt) = pack8(h8);
        }
      }
    }
  };
  // The first workers with each delay, from a table of the delays (in the tile's room), are dealt to the groups of blocks in turn.
  if constexpr (LIST) {
    __shared__ int32_t tau_s[kBlock];
    __shared__ unsigned long long mine_s[kBlock / kWave];
    if (z == 0) { one(true, 0, 0); return; }
    if (s.M <= kWave) {
      // up to 64 workers: every wavefront makes the list for itself, a ballot per distinct delay (with the table below, which takes six barriers: 784-500-10, 10 workers of 12
      // rows: 2 us more)
      const int lane = t & 63;
      const int32_t mine_tau = lane < s.M ? min(max(s.tau[lane], 0), s.D) : -1;
      unsigned long long left = s.M == kWave ? ~0ull : (1ull << s.M) - 1, mine = 0;
      int r = lane;
      for (int turn = 0; left; turn = turn + 1 == a.z_groups ? 0 : turn + 1) {
        const int i = __ffsll(left) - 1;
        const unsigned long long same = __ballot(mine_tau == __builtin_amdgcn_readlane(mine_tau, i));
        if ((same >> lane) & 1) r = i;
        if (turn == z - 1) mine |= 1ull << i;
        left &= ~same;
      }
      if (first_tile && z == 1 && t < s.M) a.rep[t] = r;
      for (; mine; mine &= mine - 1) {
        const int m = __ffsll(mine) - 1;
        one(false, m, __builtin_amdgcn_readlane(mine_tau, m));
        lds_sync();                                     // (the tile's room is written again)
      }
      return;
    }
    int32_t *first_of = reinterpret_cast<int32_t *>(sm);
    const int32_t tau = t < s.M ? min(max(s.tau[t], 0), s.D) : 0;
    for (int j = t; j <= s.D; j += kBlock) first_of[j] = kBlock;
    lds_sync();
    // (equal delays take their turns at the table's entry: a wavefront's first worker, often one of many with the same, stands for those of its wavefront)
    const int32_t lead = __builtin_amdgcn_readlane(tau, 0);
    if (t < s.M && ((t & 63) == 0 || tau != lead)) atomicMin(&first_of[tau], t);
    lds_sync();
    const int r = t < s.M ? min(first_of[tau], t) : kBlock;
    if (first_tile && z == 1 && t < s.M) a.rep[t] = r;
    const unsigned long long firsts = __ballot(r == t);
    tau_s[t] = tau;
    if ((t & 63) == 0) mine_s[t >> 6] = firsts;
    lds_sync();
    int turn = __popcll(firsts & ((1ull << (t & 63)) - 1));
    for (int i = 0; i < t >> 6; ++i) turn += __popcll(mine_s[i]);
    const unsigned long long mine = __ballot(r == t && turn % a.z_groups == z - 1);
    lds_sync();
    if ((t & 63) == 0) mine_s[t >> 6] = mine;
    lds_sync();
    for (int i = 0; i < kBlock / kWave; ++i)
      for (unsigned long long left = mine_s[i]; left; left &= left - 1) {
        const int m = __builtin_amdgcn_readfirstlane(i * kWave + __ffsll(left) - 1);
        one(false, m, __builtin_amdgcn_readfirstlane(tau_s[m]));
        lds_sync();                                     // (the tile's room is written again)
      }
  } else {
    int m = 0, tau = 0;
    if (z != 0 && a.rep) {
      m = z - 1;
      tau = min(s.tau[m], s.D);
      int r = m;                                          // (every wavefront finds it for itself)
      for (int j0 = 0; j0 < m && r == m; j0 += kWave) {
        const int j = j0 + (t & 63);
        const unsigned long long same = __ballot(j < m && min(s.tau[j], s.D) == tau);
        if (same) r = j0 + __ffsll(same) - 1;
      }
      if (first_tile && t == 0) a.rep[m] = r;
      if (r != m) return;                                 // another worker with the same reference point stands for this one
    }
    one(z == 0, m, tau);
  }
}

template <bool LIST>
__global__ __launch_bounds__(kBlock, LIST ? 5 : 8) void k_stage(const StageArgs a) {
  __shared__ __align__(16) unsigned char sm[64 * 65 * sizeof(float)];     // a weight tile on its way to the other orientation
  if (a.rule_block && blockIdx.x == 0) {
    rule_inputs(a.s, a.rule_in, reinterpret_cast<double *>(sm));
    return;
  }
  const uint32_t blk = blockIdx.x - a.rule_block;
  if (blk < a.first[1]) {
    const uint32_t per = (uint32_t)a.gx * a.gy;
    const uint32_t m = blk / per, r = blk - m * per;
    stage_minibatch(a, (int)(r % a.gx), (int)(r / a.gx), (int)m);
    return;
  }
  int l = 0;
  while (blk >= a.first[l + 2]) ++l;             // (blk < first[n_layers + 1], the grid's size)
  const PrepLayer &p = a.layer[l];
  const uint32_t rel = blk - a.first[l + 1];
  const uint32_t per = (uint32_t)p.gx * p.gy;
  const uint32_t z = rel / per, r = rel - z * per;
  stage_weights<LIST>(a, p, sm, (int)(r % p.gx), (int)(r / p.gx), (int)z, l == 0 && r == 0);
}

// Hidden-layer bias gradient and its innovation from the sums per band of 64 rows.
// grid (ceil(d / 64), M), one wavefront each
__global__ __launch_bounds__(kWave) void k_bias_finish(const DevState s, const float *dbpart, const float *ddbpart, int nband, int bands, int d,
                                                       int64_t offb, int lhs_slot) {
  const int m = blockIdx.y;
  const int c = blockIdx.x * kWave + threadIdx.x;
  float sq = 0.f;
  if (c < d) {
    float gsum = 0.f, dsum = 0.f;
    for (int rb = 0; rb < bands; ++rb) {
      const int64_t at = ((int64_t)m * nband + rb) * d + c;
      gsum += dbpart[at];
      if (ddbpart) dsum += ddbpart[at];
    }
    put_fresh_grad(s, m, offb + c, gsum);
    if (s.rule == CADA_RULE_CADA1) {
      fresh_innov(s, m)[offb + c] = f2bf(dsum);
      dsum -= bf2f(stored_innov(s, m)[offb + c]);
    }
    sq = dsum * dsum;
  }
  const float tot = wave_sum(sq);
  if (ddbpart && threadIdx.x == 0) s.lhs_part[(int64_t)m * s.n_lhs_part + lhs_slot + blockIdx.x] = tot;
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
namespace {

void side_add(Side &sd, const bf16_t *p, int64_t kt, int64_t bstride) {
  sd.ptr[sd.n] = p; sd.kt[sd.n] = kt; sd.bstride[sd.n] = bstride; sd.n += 1;
}

void set_tiles(Mm5Args &g, int per_xcd) { g.gx = divisor((g.N + BN - 1) / BN); g.gy = divisor((g.M + BM - 1) / BM); g.nbx = divisor(per_xcd); }

// The (tensor count, product set) combinations the layers use.
template <int EPI, int NA, int NB, bool HAS_D> hipError_t mm5_allow_lds() {
  return hipFuncSetAttribute(reinterpret_cast<const void *>(k_mm5<EPI, NA, NB, HAS_D>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)mm5_lds_bytes(EPI));
}
template <int EPI, int NA, int NB, bool HAS_D> int launch_mm5_as(Ctx *c, Mm5Args &g) {
  // one workgroup per CU at most (8 XCDs x 32 CUs), each XCD's tiles dealt over its workgroups
  const int total = ((g.N + BN - 1) / BN) * ((g.M + BM - 1) / BM) * g.workers, per = (total + 7) / 8;
  set_tiles(g, per < 32 ? per : 32);
  const dim3 grid(8 * g.nbx.d);
  hipLaunchKernelGGL((k_mm5<EPI, NA, NB, HAS_D>), grid, dim3(2 * kBlock), mm5_lds_bytes(EPI), c->stream, g);
  return CADA_OK;
}
template <int NA, int NB, bool HAS_D, bool CADA1> int launch_dw_as(Ctx *c, Mm5Args &g) {
  // two workgroups per CU at most
  const int total = ((g.N + BN - 1) / BN) * ((g.M + BM - 1) / BM) * g.workers, per = (total + 7) / 8;
  set_tiles(g, per < 64 ? per : 64);
  hipLaunchKernelGGL((k_dw<NA, NB, HAS_D, CADA1>), dim3(8 * g.nbx.d), dim3(kBlock), kDwLds, c->stream, g);
  return CADA_OK;
}
template <bool PL, bool CADA1> int launch_dw_two(Ctx *c, Mm5Args &g2, Mm5Args &g1) {
  int most = 0;
  for (const Mm5Args *g : {&g2, &g1}) most = std::max(most, (((g->N + BN - 1) / BN) * ((g->M + BM - 1) / BM) * g->workers + 7) / 8);
  set_tiles(g2, std::min(most, 64)); set_tiles(g1, std::min(most, 64));
  hipLaunchKernelGGL((k_dw_two<PL, CADA1>), dim3(8 * g1.nbx.d), dim3(kBlock), kDwLds, c->stream, g2, g1);
  return CADA_OK;
}
template <bool PL, bool CADA1> hipError_t dw_two_allow_lds() {
  return hipFuncSetAttribute(reinterpret_cast<const void *>(k_dw_two<PL, CADA1>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDwLds);
}
template <int NA, int NB, bool HAS_D, bool CADA1> hipError_t dw_allow_lds() {
  return hipFuncSetAttribute(reinterpret_cast<const void *>(k_dw<NA, NB, HAS_D, CADA1>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDwLds);
}
// per wavefront: the blocks of a step, over which its partial results (4 or 8 KB) are laid later, and a room of 2 KB at least behind those; weight gradient: the seven blocks it stages (14 KB), over which the partial results are laid later, and behind
// them (1.5 KB) the sums that wavefronts hand on
constexpr int skinny_lds_bytes(int epi, int tensors, int nw = 8) { return nw * (epi == EPI_DW ? 7 * 1024 * (int)sizeof(bf16_t) + 3 * 64 * (int)sizeof(float2) : tensors * 2048); }
// Wavefronts of a launch: one per two tile steps, eight at most.  A weight gradient sums over a worker's few rows (4-8
// steps); with eight wavefronts half of them would idle while their LDS kept other workgroups off the CU.
// A hidden layer's forward product of more blocks than two workgroups of eight wavefronts per CU: four wavefronts with the shares of two each, so that more workgroups are there at once and one's head and
// way out pass under another's products; an inner dimension of more than 512 leaves nothing of that, since the second shares cross LDS after the first.  us per step of inner dimension-400-10, eight / four, CADA2,
// 30 workers of 60 rows, then 40 of 24, always, 30 of 60: 64: 53.8 / 52.5, 51.9 / 50.6, 47.7 / 45.9; 200: 55.9 / 55.8, 57.6 / 57.5, 50.5 / 49.1; 400: 64.1 / 63.7, 68.8 / 68.4, 58.3 / 57.1; 512: 66.3 / 65.7, 71.2 /
// 71.6, 64.0 / 63.8; 700: 80.9 / 80.8, 77.4 / 78.0, 72.7 / 72.5; 1000: 103.1 / 103.0, 103.1 / 104.1, 86.3 / 86.9; 300-400-300-10, 30 of 60: 111.3 / 110.1; 100-300-300-300-10, CADA1, 40 of 50: 170.2 / 162.9.  784-500-10,
// 10 of 12 (160 blocks): 51.6 / 52.4.  (With four shares in all, whose sums are others, 0.2 to 1.3 less from 200 on.)
constexpr int kSkinnyFewWaves = 512, kSkinnyShort = 512;
static int skinny_waves(int epi, int K) {
  const int nk = (K + BK - 1) / BK;
  if (epi != EPI_DW) return 8;
  return nk >= 16 ? 8 : nk >= 2 ? nk / 2 : 1;
}
template <int EPI, int NA, int NB, bool HAS_D> hipError_t skinny_allow_lds() {
  if constexpr (EPI == EPI_FWD_HIDDEN) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_skinny<EPI, NA, NB, HAS_D, true>), hipFuncAttributeMaxDynamicSharedMemorySize, skinny_lds_bytes(EPI, NA + NB, 4));
    if (e != hipSuccess) return e;
  }
  return hipFuncSetAttribute(reinterpret_cast<const void *>(k_skinny<EPI, NA, NB, HAS_D>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             skinny_lds_bytes(EPI, NA + NB));
}
template <int EPI, int NA, int NB, bool HAS_D> int launch_skinny_as(Ctx *c, Mm5Args &g) {
  if constexpr (EPI == EPI_FWD_HIDDEN) {
    const dim3 grid((unsigned)((g.M + 31) / 32), (unsigned)g.workers, (unsigned)((g.N + 31) / 32));
    if ((int64_t)grid.x * grid.y * grid.z > kSkinnyFewWaves && g.K <= kSkinnyShort)
      hipLaunchKernelGGL((k_skinny<EPI, NA, NB, HAS_D, true>), grid, dim3(kBlock), skinny_lds_bytes(EPI, NA + NB, 4), c->stream, g);
    else hipLaunchKernelGGL((k_skinny<EPI, NA, NB, HAS_D>), grid, dim3(2 * kBlock), skinny_lds_bytes(EPI, NA + NB), c->stream, g);
    return CADA_OK;
  }
  const int nw = skinny_waves(EPI, g.K);
  g.step_waves = nw;
  const unsigned extra = (EPI == EPI_DW && g.lastb != nullptr) ? 1u : 0u;      // (the workgroup that finishes the last layer's bias gradient)
  // A weight gradient's way out is spread over four wavefronts at least where the CUs have room for them (with one, 120-80-60-5, 8 workers of 40
  // rows: 12.7 us, now 10.3); with more than two workgroups per CU, whose registers they take, over those of the products (784-512-10, 64 workers of 128 rows:
  // four wavefronts 1.4 us slower than two).
  const int wide = EPI == EPI_DW && nw < 4 && (int64_t)((g.M + 31) / 32 + extra) * g.workers <= 512 ? 4 : nw;
  hipLaunchKernelGGL((k_skinny<EPI, NA, NB, HAS_D>), dim3((unsigned)((g.M + 31) / 32) + extra, g.workers), dim3(64 * wide), skinny_lds_bytes(EPI, NA + NB, nw), c->stream, g);
  return CADA_OK;
}
template <bool PL> hipError_t loss_dw_allow_lds() {
  return hipFuncSetAttribute(reinterpret_cast<const void *>(k_loss_dw<PL>), hipFuncAttributeMaxDynamicSharedMemorySize, skinny_lds_bytes(EPI_LOSS, PL ? 4 : 7));
}
// (M rows of the result and one more workgroup, for each worker)
static int loss_dw_blocks(int units, int workers) { return ((units + 31) / 32 + 1) * workers; }
template <bool PL> int launch_loss_dw(Ctx *c, Mm5Args &loss, Mm5Args &dw) {
  dw.step_waves = 1;                       // (at most 32 rows: one step)
  hipLaunchKernelGGL(k_loss_dw<PL>, dim3((unsigned)((dw.M + 31) / 32 + 1), (unsigned)dw.workers), dim3(2 * kBlock), skinny_lds_bytes(EPI_LOSS, PL ? 4 : 7), c->stream, loss, dw);
  return CADA_OK;
}
// Hidden layers' forward products go through k_skinny while its 32 x 32 blocks fill the chip (two workgroups per CU) at most twice
// over, or a worker has a single block of rows (a 128 x 128 tile would then be three quarters padding).  Few tiles leave CUs
// idle and run through the whole inner dimension one after the other, where k_skinny splits it over eight wavefronts.
// Some two and a half times over as well, where the rows that an XCD meets stay in its L2 (4 MB) from one block of columns to the next: they are read again for each.  They are the same rows
// each time where the row blocks are a multiple of the eight XCDs; where they are not, the products of a second gradient hide what that costs up to half as many rows.
// Measured, us per step with k_skinny and with k_mm5 (inner dimension x units, row blocks), all workers uploading.  CADA2, rows in L2: 3072 x 1024, 40: 215.4, 237.1; 2000 x 500, 80: 145.9, 163.5; 784 x 512, 72:
// 101.9, 110.5; 784 x 500, 70: 90.9, 95.7; 784 x 260, 144: 104.6, 109.7; 784 x 300, 130: 107.3, 107.5; past that: 2000 x 400, 95: 170.0, 169.9 (all delays different: 225.6, 218.8); 3072 x 130, 259: 241.4, 233.6
// (279, 257); 2000 x 130, 259: 183.6, 181.3; 3072 x 257, 140: 207.8, 206.2; but 2000 x 256, 160: 141.8, 155.2.  Always, LAG: 2000 x 500, 80: 129.9, 141.7; 784 x 512, 72: 87.7, 91.8; 64 x 500, 80: 54.0, 54.0;
// no multiple: 784 x 300, 130: 97.2, 93.1; 2000 x 400, 95: 158.7, 147.4; 784 x 500, 70: 77.9, 79.4; past it: 3072 x 128, 320: 214.1, 199.7; 2000 x 64, 640: 205.9, 200.4.
// More blocks, CADA2: 2000-130-10, M = 40, B = 200 (1400): 235.8, 226.7; 100-300-10, M = 60, B = 96 (1800): 81.0, 78.8; 1000-1000-10, M = 16, B = 128 (2048): 192.5, 188.2.
constexpr int64_t kSkinnyBlocks = 1024, kSkinnyBlocksInL2 = 1300, kL2Bytes = 4 << 20;
static bool skinny_forward(const Mm5Args &g, int workers) {
  const int64_t row_blocks = (int64_t)((g.M + 31) / 32) * workers, blocks = row_blocks * ((g.N + 31) / 32);
  if (g.M <= 32 || blocks <= kSkinnyBlocks) return true;
  const bool plain = g.s.rule == CADA_RULE_ALWAYS || g.s.rule == CADA_RULE_LAG;
  const int64_t row_bytes = row_blocks * 32 * g.K * g.A.n * (int64_t)sizeof(bf16_t), room = row_blocks % 8 == 0 ? 8 * kL2Bytes : plain ? 0 : 4 * kL2Bytes;
  return blocks <= kSkinnyBlocksInL2 && row_bytes <= room;
}
// Weight gradients of the rules that read all of them back in the same step, stored ones beside fresh ones (k_lag_lhs).  When they outgrow the 256 MB of
// memory-side cache it pays to write them past the caches: what k_dw's plain stores leave there is written back under that kernel's reads (3072-1024-10, 36 workers of 128
// rows: 206 us, 175 with the other).  Stores of that kind keep k_dw's wavefronts, which load as well as store, waiting (163 us, 151 past the caches); in k_mm5
// the moving wavefronts wait for nothing but loads (140).  Its way out costs more per tile, which few rows per tile do not make up for, least where
// rows start on no line or no 16 bytes.  Measured, us per step, always-upload, k_dw / k_mm5: 3072-1024-10: 177 MB: 100 rows: 281 / 278; 215 MB: 64: 299 / 305, 100: 318 / 313;
// 265 MB: 40: 342 / 343, 64: 347 / 344, 256: 503 / 474; 316 MB: 24: 392 / 394, 40: 392 / 388, 100: 427 / 397; 455 MB: 24: 517 / 518, 40: 575 / 552, 100: 629 / 565;
// 100-1024-1024-10: 300 MB: 100: 552 / 506; 2000-1000-10: 320 MB: 64: 424 / 426, 100: 455 / 436; 450 MB: 40: 540 / 540, 100: 604 / 560; 1021-1021-1021-7:
// 320 MB: 64: 481 / 489, 100: 507 / 490; 450 MB: 64: 611 / 626, 100: 657 / 619.  bf16 gradients (half the bytes, 8 instead of 16 per lane and row): k_dw.
static bool dw_past_caches(const Mm5Args &g) {
  const int64_t bytes = (int64_t)g.workers * g.s.ps * 4;
  return g.s.gbuf16 == nullptr && bytes > 200000000 && bytes * g.K > (g.N % 32 == 0 ? 12000000000ll : 24000000000ll) && (g.N % 4 == 0 || g.K > 64);
}
template <int EPI> bool tiles_fit(const Mm5Args &g) {
  // every tensor must hold the chunks the tile steps walk through: the contraction indices along a row
  // tile, or (weight gradient: units are output rows, the steps walk down the worker's rows) whole
  // 128-unit tiles and the worker's padded rows
  const int64_t needA = EPI == EPI_DW ? 4 * ((g.M + BM - 1) / BM) : (g.K + BK - 1) / BK;
  const int64_t needB = EPI == EPI_DW ? 4 * ((g.N + BN - 1) / BN) : (g.K + BK - 1) / BK;
  for (int i = 1; i < g.A.n; ++i)
    if (g.A.kt[i] != g.A.kt[0] || g.A.bstride[i] != g.A.bstride[0]) { set_error("internal: A tensors with different chunk counts or strides"); return false; }
  for (int i = 1; i < g.B.n; ++i)
    if (EPI == EPI_DW && (g.B.kt[i] != g.B.kt[0] || g.B.bstride[i] != g.B.bstride[0])) { set_error("internal: B tensors with different chunk counts or strides"); return false; }
  for (int i = 0; i < g.A.n; ++i)
    if (g.A.kt[i] < needA) { set_error("internal: A tensor with fewer chunks than the tiles walk through"); return false; }
  for (int i = 0; i < g.B.n; ++i)
    if (g.B.kt[i] < needB) { set_error("internal: B tensor with fewer chunks than the tiles walk through"); return false; }
  if (EPI == EPI_DW && (int64_t)((g.K + BK - 1) / BK) * BK > g.Bp) { set_error("internal: more rows than a worker's padded tile"); return false; }
  return true;
}
// Returns CADA_OK after enqueueing the launch, CADA_EUNSUPPORTED (and launches nothing) when the
// operands do not fit a compiled variant.
template <int EPI> int launch_mm5(Ctx *c, Mm5Args &g, int workers) {
  g.workers = workers;
  const bool has_d = g.a_d >= 0;
  if constexpr (EPI == EPI_DW || EPI == EPI_LOSS || EPI == EPI_FWD_HIDDEN) {
    if (EPI == EPI_FWD_HIDDEN ? skinny_forward(g, workers) : g.N <= 32) {            // (at most 32 output columns: the last layer)
      for (int i = 1; i < g.A.n; ++i)
        if (g.A.kt[i] != g.A.kt[0] || g.A.bstride[i] != g.A.bstride[0]) { set_error("internal: A tensors with different chunk counts or strides"); return CADA_EUNSUPPORTED; }
      if constexpr (EPI == EPI_DW) {
        for (int i = 1; i < g.B.n; ++i)
          if (g.B.kt[i] != g.B.kt[0] || g.B.bstride[i] != g.B.bstride[0]) { set_error("internal: B tensors with different chunk counts or strides"); return CADA_EUNSUPPORTED; }
      } else
        if (g.B.bstride[0] != 0 || g.B.bstride[1] != 0) { set_error("internal: weights of a worker's own"); return CADA_EUNSUPPORTED; }
      if (g.a_h != 0 || g.a_l != 1 || (has_d && g.a_d != 2) || g.a_r != (g.A.n == 4 ? 3 : 0) || g.b_h != 0 || g.b_l != 1 ||
          (has_d && g.b_x != (g.B.n == 4 ? 2 : 0)) || g.b_d != g.B.n - 1) {
        set_error("internal: unexpected tensor roles");
        return CADA_EUNSUPPORTED;
      }
      if (g.A.n == 2 && g.B.n == 2) return launch_skinny_as<EPI, 2, 2, false>(c, g);
      if constexpr (EPI == EPI_DW) {
        if (!has_d && g.A.n == 2 && g.B.n == 3) return launch_skinny_as<EPI, 2, 3, false>(c, g);
        if (has_d && g.A.n == 3 && g.B.n == 4) return launch_skinny_as<EPI, 3, 4, true>(c, g);
      } else {
        if (!has_d && g.A.n == 2 && g.B.n == 3) return launch_skinny_as<EPI, 2, 3, false>(c, g);
        if (has_d && g.A.n == 4 && g.B.n == 3) return launch_skinny_as<EPI, 4, 3, true>(c, g);
      }
    }
  }
  if constexpr (EPI == EPI_LOSS) {
    set_error("internal: the loss epilogue serves at most 32 classes");
    return CADA_EUNSUPPORTED;
  } else {
  if (!tiles_fit<EPI>(g)) return CADA_EUNSUPPORTED;
  if constexpr (EPI == EPI_DW) {
    const bool cada1 = g.s.rule == CADA_RULE_CADA1;
    if (g.A.n == 2 && g.B.n == 2) return dw_past_caches(g) ? launch_mm5_as<EPI, 2, 2, false>(c, g) : launch_dw_as<2, 2, false, false>(c, g);
    if (!has_d && g.A.n == 2 && g.B.n == 3) return cada1 ? launch_dw_as<2, 3, false, true>(c, g) : launch_dw_as<2, 3, false, false>(c, g);
    if (has_d && g.A.n == 3 && g.B.n == 4) return cada1 ? launch_dw_as<3, 4, true, true>(c, g) : launch_dw_as<3, 4, true, false>(c, g);
  } else {
    if (g.A.n == 2 && g.B.n == 2) return launch_mm5_as<EPI, 2, 2, false>(c, g);
    if constexpr (EPI == EPI_FWD_HIDDEN)
      if (!has_d && g.A.n == 2 && g.B.n == 3) return launch_mm5_as<EPI, 2, 3, false>(c, g);
    if (has_d && g.A.n == 4 && g.B.n == 3) return launch_mm5_as<EPI, 4, 3, true>(c, g);
  }
  set_error("internal: no MFMA kernel variant for %d + %d tensors", g.A.n, g.B.n);
  return CADA_EUNSUPPORTED;
  }
}

// The weight gradients of the second layer (g2) and the first (g1) in one launch.  (As above: both or none.)
int launch_weight_gradients_of_two(Ctx *c, Mm5Args &g2, Mm5Args &g1, int workers) {
  g2.workers = g1.workers = workers;
  if (!tiles_fit<EPI_DW>(g2) || !tiles_fit<EPI_DW>(g1)) return CADA_EUNSUPPORTED;
  const bool cada1 = g1.s.rule == CADA_RULE_CADA1;
  if (g1.A.n == 2 && g1.B.n == 2 && g2.A.n == 2 && g2.B.n == 2) return launch_dw_two<true, false>(c, g2, g1);
  if (g1.a_d < 0 && g1.A.n == 2 && g1.B.n == 3 && g2.a_d >= 0 && g2.A.n == 3 && g2.B.n == 4) return cada1 ? launch_dw_two<false, true>(c, g2, g1) : launch_dw_two<false, false>(c, g2, g1);
  set_error("internal: no kernel variant for the weight gradients of %d + %d and %d + %d tensors", g2.A.n, g2.B.n, g1.A.n, g1.B.n);
  return CADA_EUNSUPPORTED;
}

Mm5Args blank(const DevState &s, const MlpPlan &P) {
  Mm5Args g{};
  g.s = s; g.Bp = P.Bp;
  g.a_h = g.a_l = g.a_d = g.a_r = -1;
  g.b_h = g.b_l = g.b_x = g.b_d = -1;
  return g;
}

}  // namespace

// One-time work at init: the bf16 copies of the features and the kernels' LDS allowance.
int mlp_init_state(Ctx *c, const float *) {
  MlpPlan &P = *static_cast<MlpPlan *>(c->mlp);
  hipError_t e = hipSuccess;
  if (const int rc = mlp_eval_init(c)) return rc;
  e = mm5_allow_lds<EPI_FWD_HIDDEN, 2, 3, false>();
  if (e == hipSuccess) e = mm5_allow_lds<EPI_FWD_HIDDEN, 4, 3, true>();
  if (e == hipSuccess) e = mm5_allow_lds<EPI_FWD_HIDDEN, 2, 2, false>();
  if (e == hipSuccess) e = mm5_allow_lds<EPI_DA, 2, 2, false>();
  if (e == hipSuccess) e = mm5_allow_lds<EPI_DW, 2, 2, false>();
  if (e == hipSuccess) e = dw_allow_lds<2, 2, false, false>();
  if (e == hipSuccess) e = skinny_allow_lds<EPI_FWD_HIDDEN, 2, 2, false>();
  if (e == hipSuccess) e = skinny_allow_lds<EPI_FWD_HIDDEN, 2, 3, false>();
  if (e == hipSuccess) e = skinny_allow_lds<EPI_FWD_HIDDEN, 4, 3, true>();
  if (e == hipSuccess) e = skinny_allow_lds<EPI_LOSS, 2, 2, false>();
  if (e == hipSuccess) e = skinny_allow_lds<EPI_DW, 2, 2, false>();
  if (e == hipSuccess) e = dw_allow_lds<2, 3, false, false>();
  if (e == hipSuccess) e = dw_allow_lds<2, 3, false, true>();
  if (e == hipSuccess) e = dw_allow_lds<3, 4, true, false>();
  if (e == hipSuccess) e = dw_allow_lds<3, 4, true, true>();
  if (e == hipSuccess) e = dw_two_allow_lds<true, false>();
  if (e == hipSuccess) e = dw_two_allow_lds<false, false>();
  if (e == hipSuccess) e = dw_two_allow_lds<false, true>();
  if (e == hipSuccess) e = mm5_allow_lds<EPI_DA, 4, 3, true>();
  if (e == hipSuccess) e = skinny_allow_lds<EPI_LOSS, 2, 3, false>();
  if (e == hipSuccess) e = skinny_allow_lds<EPI_LOSS, 4, 3, true>();
  if (e == hipSuccess) e = skinny_allow_lds<EPI_DW, 2, 3, false>();
  if (e == hipSuccess) e = skinny_allow_lds<EPI_DW, 3, 4, true>();
  if (e == hipSuccess) e = loss_dw_allow_lds<true>();
  if (e == hipSuccess) e = loss_dw_allow_lds<false>();
  if (e != hipSuccess) { set_error("hipFuncSetAttribute(LDS size) failed: %s", hipGetErrorString(e)); return CADA_EHIP; }
  const int64_t n = P.total_rows * P.ldx;
  hipLaunchKernelGGL(k_x_to_bf16, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, c->s.X, P.Xh, P.Xl, P.total_rows, P.d[0], P.ldx);
  e = hipGetLastError();
  if (e != hipSuccess) { set_error("feature conversion launch failed: %s", hipGetErrorString(e)); return CADA_EHIP; }
  return CADA_OK;
}

// The rule evaluates no second gradient.
static bool plain_rule(const MlpPlan &P) { return P.rule == CADA_RULE_ALWAYS || P.rule == CADA_RULE_LAG; }

// The bf16 copies of the weights, and with idx the minibatch's rows and the differences to the reference points.
// The differences of CADA2 are formed by groups of blocks that share the distinct reference points out, so many groups as make the blocks fill the chip (eight per CU), eight at
// least.  Every group's blocks start with the list of those points, and more groups than points leave the others' blocks nothing else to do.  Measured, us per step with a group per worker whose blocks
// look for an equal delay before theirs / these groups / 8: every worker at another delay: 784-300-10, 100 workers of 12 rows: 192.2, 193.6, 270; 784-512-10, 64 of 128: 216.4, 217.6, 255; 100-32-10,
// 256 of 8: 51.0, 50.5, 154 (8: with a list made by a walk over the workers as well); 3072-1024-1024-10, 16 of 256: 728.7, 717.3, 738; all workers at one: 113.0, 109.7, 108.5; 165.1, 162.5, 161.7;
// 60.2, 60.5, 60.2; 559, 555, 554.  784-300-10 with 1024 / 4096 blocks: 212.8 / 188.5 and 108.8 / 113.0.
constexpr int kStageBlocks = 2048, kStageGroups = 8;
static void stage(Ctx *c, const MlpPlan &P, const DevState &s, const int32_t *idx) {
  const int L = P.L, M = P.M, B = P.B;
  StageArgs sa;
  sa.s = s;
  sa.Xh = P.Xh; sa.Xl = P.Xl; sa.ldx = P.ldx; sa.idx = idx; sa.grow = P.grow;
  sa.XGh = P.XGh; sa.XGl = P.XGl;
  sa.d0 = P.d[0]; sa.B = B; sa.Bp = P.Bp; sa.ktx = P.kta[0];
  sa.gx = (int)((P.ldx + 63) / 64); sa.gy = (B + 63) / 64;
  int64_t tiles = 0;
  for (int l = 1; l <= L; ++l) tiles += (int64_t)((P.d[l] + 63) / 64) * ((P.d[l - 1] + 63) / 64);
  const bool z_listed = P.rule == CADA_RULE_CADA2 && M <= kBlock && c->s.D < kStageDelays;
  sa.z_groups = z_listed ? (int)std::min<int64_t>(P.nW, std::max<int64_t>(kStageGroups, (kStageBlocks + tiles - 1) / tiles)) : P.nW;
  sa.n_layers = L; sa.nz = idx && !plain_rule(P) ? sa.z_groups + 1 : 1; sa.wt_total = P.wt_total; sa.wn_total = P.wn_total; sa.rep = P.rule == CADA_RULE_CADA2 ? P.rep : nullptr;
  uint64_t nblk = idx ? (uint64_t)sa.gx * sa.gy * M : 0;
  sa.first[0] = 0;
  for (int l = 1; l <= L; ++l) {
    PrepLayer &pl = sa.layer[l - 1];
    pl.WTh = P.WTh + P.wt_off[l - 1]; pl.WTl = P.WTl + P.wt_off[l - 1]; pl.dWT = P.dWT + P.wt_off[l - 1];
    pl.WNh = P.WNh + P.wn_off[l - 1]; pl.WNl = P.WNl + P.wn_off[l - 1]; pl.dWN = P.dWN + P.wn_off[l - 1];
    pl.offW = P.offW[l - 1];
    pl.din = P.d[l - 1]; pl.dout = P.d[l]; pl.ktt = P.kta[l - 1]; pl.ktn = P.kta[l]; pl.want_n = idx && l >= 2;
    pl.gx = (pl.dout + 63) / 64; pl.gy = (pl.din + 63) / 64;
    sa.first[l] = (uint32_t)nblk;
    nblk += (uint64_t)pl.gx * pl.gy * sa.nz;
  }
  for (int l = L + 1; l < CADA_MAX_LAYERS + 2; ++l) sa.first[l] = (uint32_t)nblk;
  sa.rule_block = idx ? 1 : 0;
  sa.rule_in = c->rule_in;
  const dim3 grid((unsigned)(nblk + sa.rule_block));
  if (z_listed && idx) hipLaunchKernelGGL(k_stage<true>, grid, dim3(kBlock), 0, c->stream, sa);
  else hipLaunchKernelGGL(k_stage<false>, grid, dim3(kBlock), 0, c->stream, sa);
}

void mlp_stage_weights(Ctx *c) { stage(c, *static_cast<MlpPlan *>(c->mlp), c->s, nullptr); }

// Gathers the minibatch rows, prepares the bf16 weights and runs the forward contractions, whose last one evaluates the loss.
// One launch for the loss and the last layer's weight gradient: one block of rows per worker, at most a workgroup per CU (their LDS).  us per step, two launches / one: 784-500-10, 10 workers of 12 rows (170
// workgroups): 51.4 / 49.3; 784-500-500-10: 102.0 / 100.0; 617-301-150-26, always, 24 of 30 (144): 68.7 / 67.5; 784-300-10, 23 of 16 (253): 57.1 / 56.3; but 40 of 16 (440): 73.0 / 81.8.
constexpr int kLossDwBlocks = 256;
static bool loss_with_dw(const MlpPlan &P) { return P.L >= 2 && P.B <= 32 && loss_dw_blocks(P.d[P.L - 1], P.M) <= kLossDwBlocks; }

static int mlp_forward(Ctx *c, MlpPlan &P, const DevState &s, const int32_t *idx, Mm5Args &loss /* out: where it has no launch of its own */) {
  const int L = P.L, M = P.M, B = P.B, Bp = P.Bp;
  const bool per_worker = (P.rule == CADA_RULE_CADA2), plain = plain_rule(P);
  const int64_t dwt_stride = per_worker ? P.wt_total : 0;
  int32_t *rep = per_worker ? P.rep : nullptr;
  stage(c, P, s, idx);

  // ---- forward: worker m owns padded rows [m*Bp, m*Bp + B)
  for (int l = 1; l <= L; ++l) {
    const int din = P.d[l - 1], dout = P.d[l];
    Mm5Args g = blank(s, P);
    g.M = B; g.N = dout; g.K = din;
    if (l == 1) {
      const int64_t bs0 = (int64_t)Bp * P.kta[0] * 32;     // a worker's Bp / 128 row tiles
      side_add(g.A, P.XGh, P.kta[0], bs0); side_add(g.A, P.XGl, P.kta[0], bs0);
      g.a_h = 0; g.a_l = 1; g.a_r = 0;                    // dZ_1 = A_0 dW_1
    } else {
      const int64_t bs = (int64_t)Bp * P.kta[l - 1] * 32;
      side_add(g.A, P.Ah[l - 1], P.kta[l - 1], bs); side_add(g.A, P.Al[l - 1], P.kta[l - 1], bs);
      g.a_h = 0; g.a_l = 1; g.a_r = 0;
      if (!plain) {
        side_add(g.A, P.dA[l - 1], P.kta[l - 1], bs); side_add(g.A, P.Aref[l - 1], P.kta[l - 1], bs);
        g.a_d = 2; g.a_r = 3;                             // dZ_l = dA W + Aref dW
      }
    }
    const int64_t ktt = P.kta[l - 1];
    side_add(g.B, P.WTh + P.wt_off[l - 1], ktt, 0); side_add(g.B, P.WTl + P.wt_off[l - 1], ktt, 0);
    g.b_h = 0; g.b_l = 1; g.b_x = 0; g.b_d = 1;
    if (!plain) { side_add(g.B, P.dWT + P.wt_off[l - 1], ktt, dwt_stride); g.b_d = 2; }
    g.rep = rep;
    if (l < L) {
      g.offb = P.offb[l - 1]; g.kto = P.kta[l];
      g.o_h = P.Ah[l]; g.o_l = P.Al[l]; g.o_d = plain ? nullptr : P.dA[l]; g.o_r = plain ? nullptr : P.Aref[l];
      g.maskbits = P.maskbits[l];
      if (const int rc = launch_mm5<EPI_FWD_HIDDEN>(c, g, M)) return rc;
    } else {
      g.offb = P.offb[L - 1]; g.kto = P.kta[L];
      g.o_h = P.Gh[L]; g.o_l = P.Gl[L]; g.o_d = P.dG[L]; g.o_r = P.Gref[L];     // (Gref: null for a single-layer network)
      g.grow = P.grow; g.lastb = P.lastb; g.nrb = Bp / 32;
      if (loss_with_dw(P)) { g.workers = M; loss = g; }
      else if (const int rc = launch_mm5<EPI_LOSS>(c, g, M)) return rc;
    }
  }
  return CADA_OK;
}

// Whether a layer's weight-gradient launch also forms its bias gradient.  That saves a launch of 5 us.  In k_dw a workgroup's first tile does it under its operands' way,
// a later one in front of its way out, which then starts by the latency of those sums later; with many such tiles, or few workgroups that have
// one, that costs as much as it saves.  us per step inside / outside (122 shapes, 12 to 256 rows, three rules): up to the lines below 0.955 to 1.002; beyond them 0.966 to 1.032:
// 784-512-10: M = 64 (256 such tiles): 0.978 - 0.997, M = 200 (800): 0.986 - 0.999; 200-1000-10, M = 100 (800): 0.982 - 1.019; 1024-1024-32: M = 32 (256, M din = 32768):
// 0.98 - 1.002, 64 (512, 65536): 0.997 - 1.013, 100: 1.005 - 1.032; 2000-64-5: M = 64 (64, 128000): 0.974 - 0.991, 200: 0.983 - 1.016; 300-128-10, M = 250 (250, 75000):
// 0.966 - 0.999.  (Up to 32 units k_skinny forms the weight gradient.)
static bool bias_inside(int M, int din, int dout) {
  return dout > 32 && (int64_t)M * tiles128(dout) <= 512 && (int64_t)M * din < 65536;
}

// Where the signals of hidden layer q go, with their masks and the sums for its bias gradient.
static void signals_below(Mm5Args &g, const MlpPlan &P, int q, bool plain) {
  g.kto = P.kta[q];
  g.o_h = P.Gh[q]; g.o_l = P.Gl[q]; g.o_d = plain ? nullptr : P.dG[q]; g.o_r = plain ? nullptr : P.Gref[q];     // (Gref: null for q = 1)
  g.maskbits = P.maskbits[q];
  g.dbpart = P.dbpart[(q - 1) & 1]; g.ddbpart = P.ddbpart[(q - 1) & 1]; g.nband = 2 * P.RT;
}

int mlp_gradients(Ctx *c, const int32_t *idx) {
  MlpPlan &P = *static_cast<MlpPlan *>(c->mlp);
  DevState s = c->s;
  set_iteration(s, c->k);
  hipStream_t st = c->stream;
  const int L = P.L, M = P.M, B = P.B, Bp = P.Bp;
  const bool per_worker = (P.rule == CADA_RULE_CADA2), plain = plain_rule(P);
  const int64_t dwn_stride = per_worker ? P.wn_total : 0;

  prof_mark(c);
  Mm5Args loss;
  if (const int rc = mlp_forward(c, P, s, idx, loss)) return rc;

  // ---- backward
  Mm5Args second;          // the second layer's weight gradient, where it waits for the first layer's
  bool waits = false;
  for (int l = L; l >= 1; --l) {
    const int din = P.d[l - 1], dout = P.d[l];
    {   // weight gradient and its innovation: contraction over the worker's rows, both operands (row, unit) tensors
      Mm5Args g = blank(s, P);
      g.M = din; g.N = dout; g.K = B;
      const int64_t bsA = (int64_t)Bp * P.kta[l - 1] * 32, bsB = (int64_t)Bp * P.kta[l] * 32;     // a worker's Bp / 128 row tiles
      if (l == 1) {
        side_add(g.A, P.XGh, P.kta[0], bsA); side_add(g.A, P.XGl, P.kta[0], bsA);
        g.a_h = 0; g.a_l = 1; g.a_r = 0;
      } else {
        side_add(g.A, P.Ah[l - 1], P.kta[l - 1], bsA); side_add(g.A, P.Al[l - 1], P.kta[l - 1], bsA);
        g.a_h = 0; g.a_l = 1; g.a_r = 0;                  // innov = A^T dG + dA^T Gref
        if (!plain) { side_add(g.A, P.dA[l - 1], P.kta[l - 1], bsA); g.a_d = 2; }
      }
      side_add(g.B, P.Gh[l], P.kta[l], bsB); side_add(g.B, P.Gl[l], P.kta[l], bsB);
      if (plain) {
        g.b_h = 0; g.b_l = 1; g.b_d = 1;
      } else if (l == 1) {     // no dA^T Gref term in the first layer
        side_add(g.B, P.dG[l], P.kta[l], bsB);
        g.b_h = 0; g.b_l = 1; g.b_d = 2;
      } else {
        side_add(g.B, P.Gref[l], P.kta[l], bsB); side_add(g.B, P.dG[l], P.kta[l], bsB);
        g.b_h = 0; g.b_l = 1; g.b_x = 2; g.b_d = 3;
      }
      g.offW = P.offW[l - 1]; g.lhs_slot0 = P.lhs_w_slot[l - 1];
      if (l == L) {     // the last layer's launch also finishes its bias gradient from the forward launch's row-block sums
        g.lastb = P.lastb; g.nrb = Bp / 32; g.offb = P.offb[L - 1]; g.lhs_slot_b = P.lhs_b_slot[L - 1];
        if (l >= 2) {   // and forms the activation gradient into the layer below
          g.w_h = P.WNh + P.wn_off[l - 1]; g.w_l = P.WNl + P.wn_off[l - 1]; g.w_d = P.dWN + P.wn_off[l - 1];
          g.w_kt = P.kta[l]; g.w_dstride = dwn_stride; g.rep = per_worker ? P.rep : nullptr;
          signals_below(g, P, l - 1, plain);
        }
      } else if (bias_inside(M, din, dout)) {       // and the other layers' from the sums of the launch that formed their signals
        g.dbpart = P.dbpart[(l - 1) & 1]; g.ddbpart = P.ddbpart[(l - 1) & 1]; g.nband = 2 * P.RT; g.bias_here = 1; g.offb = P.offb[l - 1]; g.lhs_slot_b = P.lhs_b_slot[l - 1];
      }
      if (l == 2 && l < L && dout > 32 && din > 32) {
        g.workers = M;
        Mm5Args g1 = g;      // (of the first layer, as far as the choice of its kernel goes)
        g1.M = P.d[0]; g1.N = din;
        waits = !(plain && (dw_past_caches(g) || dw_past_caches(g1)));
      }
      if (l == L && loss_with_dw(P)) {
        g.workers = M;
        if (const int rc = plain ? launch_loss_dw<true>(c, loss, g) : launch_loss_dw<false>(c, loss, g)) return rc;
      } else if (l == 2 && waits) second = g;
      else if (const int rc = l == 1 && waits ? launch_weight_gradients_of_two(c, second, g, M) : launch_mm5<EPI_DW>(c, g, M)) return rc;
    }
    if (l >= 2 && l < L) {   // gradient w.r.t. the activations of layer l-1, masks, bias partials
      Mm5Args g = blank(s, P);
      g.M = B; g.N = din; g.K = dout;
      const int64_t bs = (int64_t)Bp * P.kta[l] * 32;
      side_add(g.A, P.Gh[l], P.kta[l], bs); side_add(g.A, P.Gl[l], P.kta[l], bs);
      g.a_h = 0; g.a_l = 1; g.a_r = 0;
      if (!plain) {
        side_add(g.A, P.dG[l], P.kta[l], bs); side_add(g.A, P.Gref[l], P.kta[l], bs);
        g.a_d = 2; g.a_r = 3;                             // dGA = dG W^T + Gref dW^T
      }
      const int64_t ktn = P.kta[l];
      side_add(g.B, P.WNh + P.wn_off[l - 1], ktn, 0); side_add(g.B, P.WNl + P.wn_off[l - 1], ktn, 0);
      g.b_h = 0; g.b_l = 1; g.b_x = 0; g.b_d = 1;
      if (!plain) { side_add(g.B, P.dWN + P.wn_off[l - 1], ktn, dwn_stride); g.b_d = 2; }
      g.rep = per_worker ? P.rep : nullptr;
      signals_below(g, P, l - 1, plain);
      if (const int rc = launch_mm5<EPI_DA>(c, g, M)) return rc;
    }
    if (l >= 2 && !bias_inside(M, P.d[l - 2], din))
      hipLaunchKernelGGL(k_bias_finish, dim3((din + kWave - 1) / kWave, M), dim3(kWave), 0, st, s, P.dbpart[l & 1], plain ? nullptr : P.ddbpart[l & 1], 2 * P.RT, (B + 63) / 64, din,
                         P.offb[l - 2], P.lhs_b_slot[l - 2]);
  }
  prof_mark(c);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error("MLP gradient launch failed: %s", hipGetErrorString(e));
    return CADA_EHIP;
  }
  return CADA_OK;
}

}  // namespace cada
