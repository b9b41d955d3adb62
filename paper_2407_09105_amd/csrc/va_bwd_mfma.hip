// Backward kernels: dQ (query-major) and dK/dV (key-major), bf16 / fp16, head_dim <= 256.
//
// What they compute (see include/varlen_attn.h), from the saved LSE and D = rowsum(dO * O):
//   P_ij = exp(scale q_i.k_j - LSE_i),  dP_ij = dO_i.v_j,  dS_ij = P_ij (dP_ij - D_i)
//   dQ_i = scale sum_j dS_ij k_j;   dK_j = scale sum_i dS_ij q_i;   dV_j = sum_i P_ij dO_i
// over the pairs a <= j <= i of one example (Table 1's mask; bounds from the position-id scan,
// paper Section 3), dK/dV also summed over the query heads that share the KV head.
//
// Two kernels, no atomics, bitwise reproducible:
//   dq_mfma_kernel   : workgroup = (128-query tile, query head); streams K/V blocks of 64 rows.
//                      Lane owns a query row: S^T = K Q^T, dP^T = V dO^T, dQ^T += K^T dS^T.  It also
//                      forms D for its rows (dO . O, then made exact by the row sums of dS) and stores
//                      it for the other kernel, so it runs first.
//   dkdv_mfma_kernel : workgroup = (128- or 64-key tile, KV head); streams Q/dO blocks of 64 rows of
//                      every query head of the group.  Lane owns a key row: S = Q K^T, dP = dO V^T,
//                      dV^T += dO^T P, dK^T += Q^T dS; the dV and the dK halves run on different waves.
// In both, the streamed index lies on the accumulator's register axis and feeds the last
// contraction as a B operand straight from registers (see va_mfma_common.h).
#include <algorithm>
#include <climits>
#include <type_traits>

#include "va_internal.h"
#include "va_mfma_common.h"

namespace va {
namespace {

constexpr int kBT = 128;             // resident rows per workgroup (queries for dQ, keys for dK/dV)
constexpr int kSub = VA_TILE / kBT;  // workgroup tiles per schedule tile
constexpr int kBS = 64;              // streamed rows per LDS block
constexpr int kBlk = kBS * kD;       // elements of one swizzled [64][128] LDS block (16 KB)
constexpr float kLog2e = 1.4426950408889634f;

// ---- where bf16 operands of the second contraction are carried in two parts ----------------------
// P and dS enter the matrix instructions as 16-bit values.  With bf16 (8 significant bits) the
// rounding of the few large entries - rows with a short context, or a peaked softmax - dominates the
// error of dV, dK and dQ (they are sums over many queries and, with grouped heads, over several
// heads).  A 32x32 sub-block that holds a probability above kSplitP (a score gradient above kSplitS
// in magnitude) therefore adds a second pass with the rounding residuals x - bf16(x); elsewhere the
// residuals are below 2^-9 of those thresholds and are dropped.  fp16 operands (11 bits) need none.
constexpr float kSplitP = 0.125f;
constexpr float kSplitS = 1.0f;
// Waves holding queries with fewer keys than this correct their dQ for the rounding of O in
// D = dO . O (see dq_mfma_kernel).
constexpr int kNearCtx = 64;
// k-steps by which the LDS fragment reads of S and dP run ahead of the matrix instructions that use
// them: in the dQ kernel (two products interleaved) and in the dK/dV kernel (one product per wave).
// Depths 2 to 4 measure the same; the rings occupy registers that the next phase's fragments reuse.
constexpr int kAhead = 2;
constexpr int kAheadKv = 3;

template <class E> struct needs_split { static constexpr bool value = false; };
template <> struct needs_split<Bf16> { static constexpr bool value = true; };

// max |x[v]| over a lane's 16 accumulator values.  x must come from vector arithmetic (not straight from
// a matrix instruction: the compiler does not see a hazard through the asm).  Written as three-operand
// maxima with magnitude modifiers, 8 instructions; from fmaxf(fabsf()) the compiler makes 27.
__device__ __forceinline__ float abs_max16(const f32x16 &x) {
  float m = 0.f;
#pragma unroll
  for (int v = 0; v < 16; v += 2) asm("v_max3_f32 %0, |%1|, |%2|, %3" : "=v"(m) : "v"(x[v]), "v"(x[v + 1]), "v"(m));
  return m;
}
// Rounding residuals x[v0..v0+7] - float(hi[0..7]) as a second operand.
template <class E> __device__ __forceinline__ typename E::x8 pack_residual_x8(const f32x16 &x, int v0, typename E::x8 hi) {
  typename E::x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (typename E::elem)(x[v0 + e] - (float)hi[e]);
  return r;
}


// ---------------------------------------------------------------------------------------------
// Template parameters of both kernels: E element type of the inputs (Bf16 / F16); EOut the
// gradients' type (float, or E); kDh head_dim rounded up to 64, 96, 128 or 256 (the unrolling); the
// argument d is the tensors' head_dim (a multiple of 8, <= kDh).  With kDh = 256 a block is two
// 128-column halves and the dQ kernel runs one workgroup per CU (accumulators in AGPRs).
template <class E, class EOut, int kDh>
__global__ void __launch_bounds__(256, kDh > 128 ? 1 : 2)
dq_mfma_kernel(const uint16_t *__restrict__ dO, const uint16_t *__restrict__ Q,
               const uint16_t *__restrict__ K, const uint16_t *__restrict__ V,
               const uint16_t *__restrict__ O, const float *__restrict__ LSE,
               float *__restrict__ delta, void *__restrict__ dQ,
               const int32_t *__restrict__ seg_start, const int32_t *__restrict__ q_tile_order, int N,
               int T, TileMap map, int hq, int hkv, int d, float scale_log2, float scale) {
  constexpr int kKs = kDh / 16, kCb = kDh / 32;
  constexpr int kHf = kDh > 128 ? 2 : 1;   // 128-column sub-blocks per block (head_dim above 128: two)
  constexpr int kBlkT = kBlk * kHf;        // elements of one tensor's streamed block
  constexpr int kTileSub = kBT * kD;       // elements of one sub-block of the tile's own rows
  typedef typename E::x8 x8;
  // two stages of {K block, V block}, swizzled
  __shared__ __attribute__((aligned(16))) uint16_t lds[4 * kBlkT];
  static_assert(4 * kBlk * 2 >= 4 * kStageFloatsPerWave * 4, "staging must fit");

  const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  // schedule tiles hold kSub workgroup tiles; workgroups of one schedule tile are adjacent
  const int wg = xcd_group_remap(blockIdx.x, map);
  const int at = wg / map.heads;  // workgroup tile, in launch order
  const int entry = uniform(q_tile_order[at / kSub]);
  const int tile = order_tile(entry);
  const int sub = at % kSub;
  const int h = (wg - at * hq + head_rotation(entry) * (int)map.group.d) % map.heads;
  const int g = h / map.group;
  const int r = tile / map.tiles, m = tile - r * (int)map.tiles.d;
  const int row_end = (r + 1) * T;
  const int t0 = r * T + m * VA_TILE + sub * kBT;
  if (t0 >= row_end) return;  // workgroup-uniform: the schedule tile is ragged
  const int t_last = min(t0 + kBT, row_end) - 1;
  // Prologue.  The tile's own Q, dO and O rows come in through LDS as whole-row block copies, into
  // the memory of the K/V stages, which is idle until the loop starts (loading the per-lane
  // fragments straight from HBM -- 32 rows x 32 B per instruction -- took 8 us per workgroup):
  //   batch 1: Q -> first half of the stage memory, dO -> second half; scalars (example bounds, LSE)
  //   batch 2: O -> second half, first K/V block -> first half (= stage 0 of the loop)
  // All loads of a batch are requested before any is consumed.
  const int iw0 = t0 + wave * 32;
  const int iw1 = min(iw0 + 31, t_last);
  const bool wave_ok = iw0 <= t_last;
  const bool wave_full = iw0 + 31 <= t_last;
  const int i_abs = iw0 + l32;
  const bool row_ok = i_abs <= t_last;
  const int i_ld = min(i_abs, t_last);  // clamped: loads stay in bounds, results of dead rows are dropped
  const uint32_t row_lane = swz_row_lane_off(lane);
  uint32_t tr_lane[2];
  swz_tr_lane_off(lane, tr_lane);
  typedef __attribute__((address_space(3))) void *lds_void;
  uint16_t *K0 = lds, *V0 = lds + kBlkT, *K1 = lds + 2 * kBlkT, *V1 = lds + 3 * kBlkT;
  const int dma_row = wave * 4 + (lane >> 4);
  bool dma_ok[kHf];  // the same for every transfer of this lane into a sub-block (rows 16 apart)
#pragma unroll
  for (int hf = 0; hf < kHf; ++hf) dma_ok[hf] = dma_lane_ok(lane, dma_row, d - 128 * hf);

  const size_t q_row_bytes = (size_t)hq * d * 2;
  const size_t q_off = (size_t)t0 * q_row_bytes, q_total = (size_t)N * q_row_bytes;
  const uint32_t tile_off = dma_lane_offset(lane, dma_row, q_row_bytes, h, d);
  // 128 rows of one tensor (head h) -> 32 KB per sub-block at dst: 8 transfers of 4 rows per wave
  auto copy_tile = [&](const uint16_t *X, uint16_t *dst) {
    const buffer_t xb = make_buffer((const char *)X + q_off, q_total - q_off);
#pragma unroll
    for (int hf = 0; hf < kHf; ++hf)
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        const uint32_t o = dma_ok[hf] ? tile_off + p * (uint32_t)(16 * q_row_bytes) + hf * 256 : kPastEnd;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(xb, (lds_void)(dst + hf * kTileSub + (4 * p + wave) * 512), 16, o, 0, 0, kOnce);
      }
  };
  copy_tile(Q, K0);
  copy_tile(dO, K1);
  const int ss_t0_v = seg_start[t0];
  const int ss_min_v = seg_start[min(iw0, t_last)];
  const int ss_max_v = seg_start[iw1 < iw0 ? t_last : iw1];
  const int ss_i_v = seg_start[i_ld];
  const float lse_v = LSE[(size_t)h * N + i_ld];

  // Key blocks are counted from the packed row's first token (block jb = tokens jbase + 64 jb ...):
  // a tile's own rows are then exactly its last two blocks whatever T, which the short-context
  // correction after the loop relies on (with blocks counted from token 0 a tile of a row that does
  // not start on a multiple of 64 straddles three).
  const int jbase = (r * T) % kBS;
  const int jb_lo = (uniform(ss_t0_v) - jbase) / kBS, jb_hi = (t_last - jbase) / kBS;  // jb_hi - 1, jb_hi: the tile's own rows
  const int ss_min = uniform(ss_min_v), ss_max = uniform(ss_max_v);
  const int ss_i = row_ok ? ss_i_v : 0x7fffffff;
  f32x16 acc[kCb];
#pragma unroll
  for (int cb = 0; cb < kCb; ++cb)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[cb][v] = 0.f;

  const size_t row_bytes = (size_t)hkv * d * 2;
  const size_t base_off = ((size_t)jb_lo * kBS + jbase) * row_bytes;
  const size_t total = (size_t)N * row_bytes;
  const buffer_t kbuf = make_buffer((const char *)K + base_off, total - base_off);
  const buffer_t vbuf = make_buffer((const char *)V + base_off, total - base_off);
  // HBM -> LDS copy of a 64-row block by the load unit (see the forward kernel): 4 loads per wave and
  // tensor, each 1 KB = 4 rows at LDS address (4 p + wave) KB; lane L lands at row 16 p + 4 wave + L / 16,
  // chunk position L % 16, and fetches global chunk (L % 16) ^ swz(row).
  const uint32_t dma_off = dma_lane_offset(lane, dma_row, row_bytes, g, d);
  const uint32_t blk_bytes = (uint32_t)(kBS * row_bytes);
  const uint32_t p_bytes = (uint32_t)(16 * row_bytes);
  auto copy_block = [&](uint16_t *Kd, uint16_t *Vd, int jb) {  // rows past the tensor arrive as zeros
    const uint32_t off = dma_off + (uint32_t)(jb - jb_lo) * blk_bytes;
#pragma unroll
    for (int hf = 0; hf < kHf; ++hf)
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const uint32_t o = dma_ok[hf] ? off + p * p_bytes + hf * 256 : kPastEnd;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(kbuf, (lds_void)(Kd + hf * kBlk + (4 * p + wave) * 512), 16, o, 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(vbuf, (lds_void)(Vd + hf * kBlk + (4 * p + wave) * 512), 16, o, 0, 0, 0);
      }
  };

  // The example of the tile's first row began fewer than kNearCtx tokens before the tile (workgroup-
  // uniform): the short-context correction of the first waves then needs the kNearCtx K rows before the
  // tile, the end of block jb_prev = jb_hi - 2, which has left the stages by the end of the loop.  They
  // are copied once more during the last iteration, into the V half of the other stage (dead by then).
  // (A tile of at most 64 rows has jb_prev = jb_hi - 1, still in its stage: nothing to copy.)
  static_assert(kNearCtx == 32 || kNearCtx == 64, "the rows kept for the correction are part of one 64-row block");
  // head_dim <= 32 (the smallest instantiation only): the whole correction -c_i sum_j P_ij k_j is kept, in a
  // second accumulator fed by the K^T fragments the dQ product reads anyway.  The softmax scale 1 / sqrt(d)
  // is large there, the same error in D weighs 2..4 times more in dQ than at head_dim 128, and the
  // instantiation has the registers; larger head dims take the correction on the nearest keys only (below).
  constexpr bool kHasPk = kDh == 64;
  const bool pk_on = kHasPk && d <= 32;  // workgroup-uniform
  f32x16 pk[kHasPk ? kCb : 1];
  if constexpr (kHasPk) {
#pragma unroll
    for (int cb = 0; cb < kCb; ++cb)
#pragma unroll
      for (int v = 0; v < 16; ++v) pk[cb][v] = 0.f;
  }
  const int ss_t0 = uniform(ss_t0_v);
  const int jb_prev = (t0 - jbase) / kBS - 1;
  const bool need_prev = !pk_on && ss_t0 < t0 && t0 - ss_t0 < kNearCtx && jb_prev == jb_hi - 2 && jb_prev >= jb_lo;
  auto copy_prev_rows = [&](uint16_t *dst) {
    const uint32_t off = dma_off + (uint32_t)(jb_prev - jb_lo) * blk_bytes;
#pragma unroll
    for (int hf = 0; hf < kHf; ++hf)
#pragma unroll
      for (int p = (kBS - kNearCtx) / 16; p < 4; ++p) {
        const uint32_t o = dma_ok[hf] ? off + p * p_bytes + hf * 256 : kPastEnd;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(kbuf, (lds_void)(dst + hf * kBlk + (4 * p + wave) * 512), 16, o, 0, 0, 0);
      }
  };

  x8 qf[kKs], gf[kKs];  // Q and dO rows of this lane: B operands
  wait_all_loads();
  __syncthreads();  // batch 1 has landed
#pragma unroll
  for (int ks = 0; ks < kKs; ++ks) {
    qf[ks] = swz_read_row<E>(K0 + (ks >> 3) * kTileSub, row_lane, ks & 7, wave * 32);
    gf[ks] = swz_read_row<E>(K1 + (ks >> 3) * kTileSub, row_lane, ks & 7, wave * 32);
  }
  __syncthreads();  // every wave has its Q and dO fragments: the memory is free again
  copy_tile(O, K1);
  copy_block(K0, V0, jb_lo);
  const float lse2 = lse_v * kLog2e;
  wait_all_loads();
  __syncthreads();  // batch 2 has landed
  // D = dO . O of this lane's query row, computed here (each lane of a pair holds half of the row)
  // and left in `delta` for the dK/dV kernel, which runs after this one
  float dl = 0.f;
#pragma unroll
  for (int ks = 0; ks < kKs; ++ks) {
    const x8 of = swz_read_row<E>(K1 + (ks >> 3) * kTileSub, row_lane, ks & 7, wave * 32);
#pragma unroll
    for (int e = 0; e < 8; ++e) dl = fmaf((float)gf[ks][e], (float)of[e], dl);
  }
  dl = pair_sum(dl);  // D~: exact up to the rounding of the stored O; refined below
  float csum = 0.f;   // this lane's share of sum_j dS~_ij
  __syncthreads();  // O has been read: stage 1 may receive the second K/V block

  // One iteration: start the copy of block jb+1 into the other stage (last read before the previous
  // barrier), consume block jb from (Kb, Vb); the barrier at the end publishes the copied block.
  auto iteration = [&](int jb, const uint16_t *__restrict__ Kb, const uint16_t *__restrict__ Vb,
                       uint16_t *__restrict__ Kn, uint16_t *__restrict__ Vn) {
    if (jb < jb_hi) copy_block(Kn, Vn, jb + 1);  // workgroup-uniform
    else if (need_prev) copy_prev_rows(Vn);
    const int j0 = jbase + jb * kBS;
    if (wave_ok && j0 <= iw1 && j0 + kBS - 1 >= ss_min) {  // wave-uniform
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        const int jl = j0 + sb * 32;
        if (jl > iw1 || jl + 31 < ss_min) continue;  // wave-uniform
        f32x16 s, dp;  // dP accumulates onto -D of this lane's query row
#pragma unroll
        for (int v = 0; v < 16; ++v) { s[v] = 0.f; dp[v] = -dl; }
        // Fragment reads run kAhead k-steps ahead of the matrix instructions that use them, in this order
        // (the scheduling barriers keep it): left alone the compiler requests each pair of fragments right
        // before the pair of matrix instructions that uses it, and the wave waits out the LDS latency 8 times.
        x8 kf[kAhead], vf[kAhead];
#pragma unroll
        for (int ks = 0; ks < kAhead; ++ks) {
          kf[ks] = swz_read_row<E>(Kb + (ks >> 3) * kBlk, row_lane, ks & 7, sb * 32);
          vf[ks] = swz_read_row<E>(Vb + (ks >> 3) * kBlk, row_lane, ks & 7, sb * 32);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < kKs; ++ks) {
          s = mfma32(kf[ks % kAhead], qf[ks], s);     // S^T  = K Q^T
          dp = mfma32(vf[ks % kAhead], gf[ks], dp);   // dP^T - D = V dO^T - D
          if (ks + kAhead < kKs) {
            const int kn = ks + kAhead;
            kf[ks % kAhead] = swz_read_row<E>(Kb + (kn >> 3) * kBlk, row_lane, kn & 7, sb * 32);
            vf[ks % kAhead] = swz_read_row<E>(Vb + (kn >> 3) * kBlk, row_lane, kn & 7, sb * 32);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        // K^T fragments of the sub-block's first 16 keys: requested here, in the registers the row
        // fragments have just left, so that they arrive during the vector work below
        x8 kt0[kCb], kt1[kCb];
#pragma unroll
        for (int cb = 0; cb < kCb; ++cb) kt0[cb] = swz_read_tr<E>(Kb + (cb >> 2) * kBlk, tr_lane, cb & 3, sb * 32);
        __builtin_amdgcn_sched_barrier(0);
        const bool interior = wave_full && jl >= ss_max && jl + 31 <= iw0;
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = __builtin_amdgcn_exp2f(fmaf(s[v], scale_log2, -lse2));  // P^T
        if (!interior) hide(s, visible_rows(ss_i - jl, i_abs - jl + 1, half), 0.f);
        x8 pf0, pf1;  // P^T as an operand, where the whole correction is kept
        if constexpr (kHasPk) {
          if (pk_on) { pf0 = pack_x8<E>(s, 0); pf1 = pack_x8<E>(s, 8); }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          s[v] *= dp[v];  // dS~^T = P (dP - D~)
          csum += s[v];
        }
        // large score gradients are carried in two bf16 parts: a second pass with the residuals
        // (wave-uniform choice; rare on long examples)
        const bool split = needs_split<E>::value && __any(abs_max16(s) > kSplitS);
        const x8 df0 = pack_x8<E>(s, 0), df1 = pack_x8<E>(s, 8);
#pragma unroll
        for (int cb = 0; cb < kCb; ++cb) kt1[cb] = swz_read_tr<E>(Kb + (cb >> 2) * kBlk, tr_lane, cb & 3, sb * 32 + 16);
#pragma unroll
        for (int cb = 0; cb < kCb; ++cb) acc[cb] = mfma32(kt0[cb], df0, acc[cb]);  // dQ^T += K^T dS^T
#pragma unroll
        for (int cb = 0; cb < kCb; ++cb) acc[cb] = mfma32(kt1[cb], df1, acc[cb]);
        if constexpr (kHasPk) {
          if (pk_on) {
#pragma unroll
            for (int cb = 0; cb < kCb; ++cb) pk[cb] = mfma32(kt1[cb], pf1, mfma32(kt0[cb], pf0, pk[cb]));  // sum_j k_j P_ij
          }
        }
        if (split) {  // the K^T fragments are simply read again
          const x8 dr0 = pack_residual_x8<E>(s, 0, df0), dr1 = pack_residual_x8<E>(s, 8, df1);
#pragma unroll
          for (int cb = 0; cb < kCb; ++cb)
            acc[cb] = mfma32(swz_read_tr<E>(Kb + (cb >> 2) * kBlk, tr_lane, cb & 3, sb * 32), dr0, acc[cb]);
#pragma unroll
          for (int cb = 0; cb < kCb; ++cb)
            acc[cb] = mfma32(swz_read_tr<E>(Kb + (cb >> 2) * kBlk, tr_lane, cb & 3, sb * 32 + 16), dr1, acc[cb]);
        }
      }
    }
    if (jb < jb_hi) __syncthreads();  // workgroup-uniform; the last block's barrier follows the correction pass below
  };

  for (int jb = jb_lo; jb <= jb_hi; jb += 2) {  // bounds are workgroup-uniform: barriers stay aligned
    iteration(jb, K0, V0, K1, V1);
    if (jb + 1 <= jb_hi) iteration(jb + 1, K1, V1, K0, V0);
  }

  // Softmax rows sum to one, so sum_j P_ij (dP_ij - D_i) = 0 for the exact D_i = sum_j P_ij dP_ij.  The
  // row sum of dS~ is therefore D_i - D~_i, the error that the rounding of the stored O left in
  // D~ = dO . O: the dK/dV kernel gets D_i itself.
  const float c_row = pair_sum(csum);
  if (row_ok && half == 0) delta[(size_t)h * N + i_abs] = dl + c_row;
  // dQ was accumulated with D~: what is missing is -c_i sum_j P_ij k_j.  It matters where the
  // probabilities are large, i.e. for queries with a short context (it falls off as 1 / context^2).
  // Waves that hold queries with fewer than kNearCtx keys recompute P on the key sub-blocks from
  // kNearCtx before their first row on and add K^T (-c P)^T - on the last two key blocks only, which
  // are still in the stage memory (nothing was copied after them): no copy, no extra barrier - and,
  // where the example of the tile's first row began shortly before the tile, on the kNearCtx keys before
  // the tile (copy_prev_rows above: one copy under the last iteration and one barrier).  With 64 instead of
  // 32 the rows whose softmax peaks a few dozen keys back are covered too (dQ of a batch of 8..128-token
  // examples: 1.1e-2 -> 3.7e-3 max-abs) for 7 % of this kernel's time on such a batch, under 2 % elsewhere.
  if constexpr (kHasPk) {
    if (pk_on) {
#pragma unroll
      for (int cb = 0; cb < kCb; ++cb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[cb][v] = fmaf(-c_row, pk[cb][v], acc[cb][v]);
    }
  }
  if (need_prev) {  // workgroup-uniform: the extra rows were requested an iteration ago
    wait_all_loads();
    __syncthreads();
  }
  if (!pk_on && wave_ok && ss_max > iw0 - kNearCtx) {  // wave-uniform
    const int j_first = max(ss_min, iw0 - kNearCtx);
    auto near_sub = [&](const uint16_t *Kb, int row0, int jl) {  // keys jl .. jl + 31 = rows row0 .. of the block at Kb
      f32x16 sc;
#pragma unroll
      for (int v = 0; v < 16; ++v) sc[v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < kKs; ++ks)
        sc = mfma32(swz_read_row<E>(Kb + (ks >> 3) * kBlk, row_lane, ks & 7, row0), qf[ks], sc);
#pragma unroll
      for (int v = 0; v < 16; ++v) sc[v] = -c_row * __builtin_amdgcn_exp2f(fmaf(sc[v], scale_log2, -lse2));
      hide(sc, visible_rows(ss_i - jl, i_abs - jl + 1, half), 0.f);
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        const x8 cf = pack_x8<E>(sc, 8 * s2);
#pragma unroll
        for (int cb = 0; cb < kCb; ++cb)
          acc[cb] = mfma32(swz_read_tr<E>(Kb + (cb >> 2) * kBlk, tr_lane, cb & 3, row0 + s2 * 16), cf, acc[cb]);
      }
    };
    if (need_prev && iw0 - kNearCtx < t0) {  // wave-uniform: this wave's keys begin before the tile
      const uint16_t *Kp = ((jb_hi - jb_lo) & 1) ? V0 : V1;
#pragma unroll 1
      for (int sb = (kBS - kNearCtx) / 32; sb < 2; ++sb) {
        const int jl = t0 - kBS + sb * 32;
        if (jl + 31 >= j_first) near_sub(Kp, sb * 32, jl);
      }
    }
#pragma unroll 1
    for (int jb = max(jb_lo, jb_hi - 1); jb <= jb_hi; ++jb) {
      const uint16_t *Kb = ((jb - jb_lo) & 1) ? K1 : K0;
#pragma unroll 1
      for (int sb = 0; sb < 2; ++sb) {
        const int jl = jbase + jb * kBS + sb * 32;
        if (jl > iw1 || jl + 31 < j_first) continue;  // wave-uniform
        near_sub(Kb, sb * 32, jl);
      }
    }
  }
  __syncthreads();  // every wave is done with the stages: the result staging below overlays them
  float *stage = (float *)lds + wave * kStageFloatsPerWave;
  store_transposed_tile<EOut, kCb>(acc, scale, stage, dQ, iw0, wave_ok ? iw1 - iw0 + 1 : 0, hq, h, d);
}

// ---------------------------------------------------------------------------------------------
// dK/dV with the two gradients on different waves.  Workgroup = 8 waves = (128-key tile, KV head);
// waves 0..3 ("V side") and 4..7 ("K side") each own 32 keys, wave w and w + 4 the same ones, and
// share a SIMD.  Per 32-query sub-block:
//   V side: S = Q K^T (on -LSE / scale), P = exp2, mask; leaves P (fp16) in LDS for its partner;
//           dV^T += dO^T P.
//   K side: dP = dO V^T (on -D); one sub-block later, with that P: dS = P * dP; dK^T += Q^T dS.
// Each wave holds one accumulator tile and one operand tile (about 200 registers), so two waves fit
// per SIMD and one wave's exp / convert / LDS work overlaps the other's matrix instructions.
// head_dim above 128 (kDh = 256): operand and accumulator tiles are twice as large, so a workgroup is
// 4 waves = (64-key tile, KV head), one wave per SIMD with 512 registers each; blocks are two
// 128-column halves, and the tile's own K and V rows pass through the memory of the second stage.
// Two shapes for head_dim <= 128, chosen on the device from the lengths of the packed batch (both are
// launched; the workgroups of the one that does not apply leave at once):
//   large: 8 waves on a 128-key tile, one workgroup per CU: each streamed Q/dO block serves 128 keys
//          (examples of thousands of tokens: 6 % faster than the small shape);
//   small: 4 waves on a 64-key tile, two workgroups per CU that hide each other's prologue, epilogue
//          and barriers (examples of 8..128 tokens: 14 % faster), at twice the block copies per
//          matrix instruction.
// The large shape runs where the mean example has kDkdvLongMean tokens or more, or where the average
// schedule tile streams kDkdvLongBlocks blocks or more: a few long examples among many short ones do most of
// the work, which the mean does not show.  Time of the large over the small shape, 8 head layouts (1 to 9
// query heads per KV head), 8192 to 32768 tokens, d = 64 to 96: 8 to 9 blocks a tile 0.95...1.09 (mean 1.03), 9.5 to 10.5
// blocks 0.98...1.06 (1.01), 12 blocks and more 0.86...1.03 (0.94).  d = 128: 8 to 10.5 blocks 1.02...1.19 (1.10), 12 to 15.5 blocks
// 0.91...1.12 (1.01; long chains cut 0.91...0.94), 18 to 22 blocks 0.98...1.02, beyond 0.89...1.03 (0.94): even between 12 and
// 22, where a later line would gain on some batches (8192 tokens, 32 heads, -6 %) what it loses on others.  Where
// the small shape's tiles may be cut finely (below) no long chain is left for the large one to shorten, and 18 blocks
// give 0.94...1.09: there the mean alone decides.
constexpr int kDkdvLongMean = 1024;
constexpr int kDkdvLongBlocks = 12;
// What a launch asks of the scan's counts, made on the host: nothing but two compares may stand between a workgroup and
// its first load.
struct DkdvPick {
  int select;    // 0: run; 1: run only where the large shape is the better one, 2: only where the small one is
  int examples;  // the small shape: more examples than this
  int blocks;    // and fewer 64-query blocks over all key tiles than this
};
__device__ __forceinline__ bool dkdv_small(int n_examples, int n_blocks, const DkdvPick &pick) {
  return n_examples > pick.examples && n_blocks < pick.blocks;
}
template <int kDh, bool kSmall> struct DkdvShape {
  static_assert(!(kSmall && kDh > 128), "head_dim above 128 has one shape");
  static constexpr int kKg = (kDh > 128 || kSmall) ? 2 : 4;  // key groups (of 32 keys) per workgroup
  static constexpr int kWgPerCu = kSmall ? 2 : 1;
  static constexpr int kWaves = 2 * kKg;                // V side + K side
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kKeys = 32 * kKg;                // keys per workgroup
  static constexpr int kSubTiles = VA_TILE / kKeys;     // workgroup tiles per schedule tile
};

// ---- cutting a key tile's work over several workgroups --------------------------------------------
// A tile's trips (64-query blocks x query heads of the group) form one serial chain.  With few tiles or
// many query heads per KV head the chip then sits idle while the longest chains run (16 heads on one KV
// head, 6141 tokens: 96 workgroups of up to 208 trips, 315 us).  The chain is cut into chunks of whole
// trips, one workgroup each; the chunks of a cut tile leave their fp32 accumulators in the workspace and
// dkdv_merge_kernel adds them, always in the order of the chunks (no atomics): 315 -> 90 us there, 370 ->
// 303 us for one example of 4096 tokens with 4 query heads per KV head.
//   host  : how many chunks a tile may have follows from the number of tiles and the workspace
//           (plan_split below); with many tiles it is one, and no merge kernel is launched.  In between, where
//           grouped heads make chains longer than a resident workgroup's share of the work, only those are cut: dK/dV of
//           three rows of 3735 tokens, 36/4 heads, 510 -> 347 us; 16384 long-tail tokens 640 -> 425; 4248 tokens, 40/8,
//           one example, 540 -> 480.
//   device: whether the batch is cut at all follows from its longest example and its total (dkdv_plan), how many chunks a
//           tile then gets from its own trips.
struct DkdvSplit {
  float *partial;   // slots of 2 * kKeys * kDh floats
  int max_chunks;   // per (tile, KV head) pair; 1: no tile is cut
  bool fine;        // few tiles: every pair has max_chunks slots; otherwise only chunks of cut tiles have one
  int room;         // the slots there are for one KV head (read where only cut tiles have them)
};
// Most chunks of a tile; the workgroups of chunks that it does not get are launched for nothing.  With many tiles 3
// are too few (three rows of 3735 tokens, 36/4 heads: 383 instead of 347 us), more than 4 no faster in 13 batches.
constexpr int kMaxChunks = 32, kMaxChunksMany = 4;
// Trips of a chunk: at least kMinTrips (writing and adding a chunk's 64 KB costs about 5 trips), and so many
// that the batch makes kChunksPerSlot chunks per resident workgroup, for balance.  Measured on six shapes
// with 1..16 heads per KV head and few tiles: 8 per slot 0...25 % faster than 4, 4 twice as fast as 1; at least 6, 8
// or 12 trips within 5 % of each other where total work is small.  With more tiles only chains longer than a slot's
// share of the work are worth a cut: 2 per slot.
constexpr int kMinTrips = 8;
constexpr int kChunksPerSlot = 8, kChunksPerSlotMany = 2;
// What the batch allows, the same in every workgroup.  A batch whose longest chain is no longer than a slot's share of the
// work is not cut: the chunks' sums are 64 KB each, written and read (8192 tokens in examples of 8 to 128, 36/4
// heads: dK/dV cut 94 us, not cut 78; 2048 tokens, 36/4, the share below the chain: 42, not cut 58).  With many tiles
// and long examples alone the bar is 1.5 shares: the tiles' chains then take all lengths up to the longest, and those just
// too short for two chunks, which stay whole, begin after the chunks of the others.  Cut over uncut, examples that fill
// their rows, by the longest chain in shares: 1.9 0.87, 1.8 0.93, 1.6 0.98, 1.45 0.98 and 1.12 (one row and three),
// 1.35 0.98 and 1.08, 1.15 1.02; examples of about 1500 tokens, 6000 in all, 1.09.
struct DkdvPlan {
  int piece;  // least trips of a chunk
  int most;   // no tile gets more chunks
};
__device__ __forceinline__ DkdvPlan dkdv_plan(const int32_t *__restrict__ meta, int keys, int slots, int N, int T, int tiles_per_row,
                                              int hq, int G, const DkdvSplit &split) {
  // 64-query blocks over all schedule tiles (meta[2]) x workgroup tiles in one x heads, over the workgroups the chip holds
  const float per_block = (float)(VA_TILE / keys * hq) * (1.f / slots), share = (float)meta[2] * per_block;
  const int piece = max(kMinTrips, (int)(share * (split.fine ? 1.f / kChunksPerSlot : 1.f / kChunksPerSlotMany)) + 1);
  // The longest chain that the longest example (meta[1]) allows: a tile's blocks reach from at most keys - 1 tokens before
  // an example to the end of it, and begin up to `off` tokens behind a multiple of the block.
  const int off = N == T ? 0 : kBS - min(kBS, T & -T);
  const int chain = ((meta[1] + keys - 2 + off) / kBS + 1) * G;
  const bool all_long = !split.fine && (long long)N >= (long long)kDkdvLongMean * meta[0];
  // Less what the later workgroup tiles of a schedule tile do not stream (16384 tokens in examples of about 100, 36/4 heads,
  // chains of 126 trips: cut 219 us, not cut 237).  `piece` keeps to the larger number, for which slots suffice.
  const float least = share - (float)(N / T * tiles_per_row) * ((VA_TILE - keys) / (2.f * kBS)) * per_block;
  const float bar = all_long ? 1.5f * least : fmaxf(least, 0.f) + (float)kMinTrips;
  return {piece, (float)chain < bar ? 1 : max(1, min(split.max_chunks, chain / piece))};
}
// Chunks of a tile of n_it trips, and the trips of all but the last.  With many tiles the chunks are of one length, whole
// blocks of G heads: the same chunk of neighbouring tiles of an example then streams the same blocks at about the
// same time, as uncut tiles do.  With few they share a tile's trips evenly (even = 0).
struct DkdvChunks {
  int n, even;
  __device__ __forceinline__ int first(int c, int n_it) const { return even ? c * even : (int)((long long)n_it * c / n); }
  __device__ __forceinline__ int end(int c, int n_it) const { return c + 1 == n ? n_it : first(c + 1, n_it); }
};
__device__ __forceinline__ DkdvChunks dkdv_chunks(int n_it, const DkdvPlan &plan, int G, const DkdvSplit &split) {
  if (plan.most == 1) return {1, 0};
  if (split.fine) return {max(1, min(split.max_chunks, n_it / plan.piece)), 0};
  int trips = max(plan.piece, (n_it + split.max_chunks - 1) / split.max_chunks);
  trips = (trips + G - 1) / G * G;
  return {max(1, n_it / trips), trips};
}

// With many tiles: the first slot of tile `u` (in launch order, workgroup tiles) in every KV head's run of slots, from the
// chunks of the cut tiles before it.  The pieces are at least half of a slot's share of the work, so that all chunks
// of cut tiles are at most kChunksPerSlotMany per resident workgroup: 64 MiB whatever the number of tiles.  All threads of
// the workgroup call it; `lds`: an int per wave.  About 3 us, in workgroups of cut tiles only.
template <int kThreads>
__device__ __forceinline__ int dkdv_first_slot(int u, int keys, const int32_t *__restrict__ seg_end, const int32_t *__restrict__ kv_tile_order,
                                               int T, int tiles_per_row, int G, const DkdvPlan &plan, const DkdvSplit &split, int *lds) {
  const int sub_tiles = VA_TILE / keys;
  int sum = 0;
  for (int x = threadIdx.x; x < u; x += kThreads) {
    const int tile = order_tile(kv_tile_order[x / sub_tiles]), r = tile / tiles_per_row, row_end = (r + 1) * T;
    const int t0 = r * T + tile % tiles_per_row * VA_TILE + x % sub_tiles * keys;
    if (t0 >= row_end) continue;
    const int n = dkdv_chunks(((seg_end[min(t0 + keys, row_end) - 1] - 1) / kBS - t0 / kBS + 1) * G, plan, G, split).n;
    if (n > 1) sum += n;
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) sum += __shfl_xor(sum, o, 64);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = sum;
  __syncthreads();
  sum = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) sum += lds[w];
  __syncthreads();
  return uniform(sum);
}

__device__ __forceinline__ void lds_barrier() {  // LDS traffic of this wave done, then workgroup barrier
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// kCut: tiles may be cut (split.max_chunks > 1).  Without it the chunk arithmetic is not compiled in: it costs
// scalar registers, in the head_dim 256 shape 29 spilled ones and 1.5 % of the time.
template <class E, class EOut, int kDh, bool kSmall, bool kCut>
__global__ void __launch_bounds__((DkdvShape<kDh, kSmall>::kThreads), (DkdvShape<kDh, kSmall>::kWgPerCu))
dkdv_mfma_kernel(const uint16_t *__restrict__ dO, const uint16_t *__restrict__ Q,
                  const uint16_t *__restrict__ K, const uint16_t *__restrict__ V,
                  const float *__restrict__ LSE, const float *__restrict__ delta, void *__restrict__ dK,
                  void *__restrict__ dV, const int32_t *__restrict__ seg_end,
                  const int32_t *__restrict__ kv_tile_order, const int32_t *__restrict__ meta, DkdvPick pick,
                  DkdvSplit split, int N, int T, FastDiv tiles, FastDiv heads, int G, int hq, int hkv, int d, float scale_log2,
                  float scale) {
  constexpr int kKs = kDh / 16, kCb = kDh / 32;
  constexpr int kHf = kDh > 128 ? 2 : 1;  // 128-column sub-blocks per block
  constexpr int kBlkT = kBlk * kHf;       // elements of one tensor's streamed block
  typedef DkdvShape<kDh, kSmall> Shape;
  constexpr int kKg = Shape::kKg, kWaves = Shape::kWaves, kKeys = Shape::kKeys, kSubTiles = Shape::kSubTiles;
  constexpr int kKvSub = kKeys * kD;      // elements of one sub-block of the tile's own K (or V) rows
  constexpr bool kKvInStage = kHf > 1 || kSmall;  // no room for a kv_tile of its own: the rows pass through stage 1
  typedef typename E::x8 x8;
  // two stages of {Q block, dO block (swizzled), -LSE / scale [64], -D [64]}; reused as the staging
  // area of the result stores
  constexpr int kStage = 2 * kBlkT + 4 * kBS;
  constexpr int kStagingElems = kWaves * kStageFloatsPerWave * 2;
  constexpr int kStagesElems = kStagingElems > 2 * kStage ? kStagingElems : 2 * kStage;
  static_assert(!kKvInStage || 2 * kHf * kKvSub <= kStage, "the tile's K and V rows must fit in one stage");
  // One LDS object for everything (with several, the compiler makes every LDS read after a block copy
  // wait until the copy has landed: it can tell copy destinations from read addresses by offset inside
  // one object only):
  //   stages: as above
  //   exch:   P hand-over, [key group][parity 2][part 2][lane 64] x 16 B
  //   kv_own: the tile's own K rows and V rows (swizzled like the streamed blocks), only used in the
  //           prologue: each wave takes its 32-row operand from here.  Going through LDS lets the rows
  //           arrive as whole 1 KB transfers; loading the per-lane fragments straight from HBM (32 rows x
  //           32 B per instruction) took 3 us per workgroup.
  constexpr int kExchElems = kKg * 2 * 2 * 64 * 8;
  constexpr int kKvOwnElems = kKvInStage ? 0 : 2 * kKvSub;
  __shared__ __attribute__((aligned(16))) uint16_t lds_all[kStagesElems + kExchElems + kKvOwnElems];
  uint16_t *const stages = lds_all;
  u32x4 *const exch = (u32x4 *)(lds_all + kStagesElems);
  uint16_t *const kv_own = lds_all + kStagesElems + kExchElems;

  const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
  const int kg = wave % kKg;
  const bool k_side = wave >= kKg;
  const int l32 = lane & 31, half = lane >> 5;
  // workgroup -> (tile, KV head) pair `pair` in launch order, chunk `chunk` of its trips.  max_chunks workgroups are
  // launched to a pair; those beyond what the batch allows are numbered last and leave at once.  Numbered among the
  // others they are expensive: workgroups go to the 8 XCDs and the 4 shader engines of each in turn, so that the working
  // ones can all fall to one engine, and are started in order, so that an idle one waits for a place in front of
  // working ones (dK/dV of 2048 tokens in examples of 8 to 60, 32/8 heads: 52 us; numbered last 27; never cut 25).
  int pair = blockIdx.x, chunk = 0;
  // Requested together with the counts that say whether this shape runs.  With the counts first, and the divisions that
  // made their bounds here, dK/dV of 8192 tokens, 32 heads of 128, took 213 us (now 209.5), of 2 x 16384, 40/8 heads, 3232 (3210).
  int entry = kCut ? 0 : uniform(kv_tile_order[pair / heads / kSubTiles]);
  if (pick.select != 0 && dkdv_small(uniform(meta[0]), uniform(meta[2]), pick) != (pick.select == 2)) return;  // workgroup-uniform
  DkdvPlan plan = {0, 1};
  if constexpr (kCut) {
    plan = dkdv_plan(meta, kKeys, 256 * Shape::kWgPerCu, N, T, tiles.d, hq, G, split);
    const int most = plan.most;
    if (blockIdx.x * split.max_chunks >= gridDim.x * most) return;
    if (most > 1 && split.fine) {
      // The tiles in order of their length, a tile's chunks together (16 heads on one KV head, 6141 tokens: 79 us; the
      // first chunks of all tiles, then the second ones, ...: 107 us).  Where `most` is even, the first chunks, which every
      // tile has, would keep to every other engine or XCD: they move on by the digit sum of the tile's number (4096 tokens
      // in examples of 8 to 128, 40/8 heads: 85 -> 57 us; moved on where it is odd, the 1500 tokens of four examples: 48 -> 58).
      const int q = pair / hkv, u = q / most;
      chunk = q - u * most;
      if (most % 2 == 0) {
        for (int x = u; x > 0; x /= most) chunk += x;
        chunk %= most;
      }
      pair += (u - q) * hkv;
    } else if (most > 1) {
      // Most tiles have one chunk: last chunks first, so that the longest tiles start early (three rows of 3735 tokens,
      // 36/4 heads: 347 us, numbered by tile 440).
      const int n_pairs = gridDim.x / split.max_chunks, level = pair / n_pairs;
      chunk = most - 1 - level;
      pair -= level * n_pairs;
    }
  }
  // (cut tiles: plain divisions, for want of scalar registers)
  const int at = kCut ? pair / hkv : pair / heads;  // workgroup tile, in launch order
  if (kCut) entry = uniform(kv_tile_order[at / kSubTiles]);
  const int tile = order_tile(entry);
  const int sub = at % kSubTiles;
  const int turned = pair - at * hkv + head_rotation(entry), g = kCut ? turned % hkv : turned % heads;
  const int tiles_per_row = tiles.d, r = kCut ? tile / tiles_per_row : tile / tiles, m = tile - r * tiles_per_row;
  const int row_end = (r + 1) * T;
  const int t0 = r * T + m * VA_TILE + sub * kKeys;
  if (t0 >= row_end) return;  // workgroup-uniform: the schedule tile is ragged
  const int t_last = min(t0 + kKeys, row_end) - 1;
  const int ib_lo = t0 / kBS;
  // The tile's chunks; with many tiles also its slots, and one chunk where there are too few left.
  int slot0 = pair * split.max_chunks, slot_step = 1;
  auto chunks_of = [&](int n_trips) {
    DkdvChunks c = dkdv_chunks(n_trips, plan, G, split);
    if (c.n > 1 && c.n > chunk && !split.fine) {
      const int before = dkdv_first_slot<Shape::kThreads>(pair / hkv, kKeys, seg_end, kv_tile_order, T, tiles_per_row, G, plan, split, (int *)exch);
      slot0 = before * hkv + pair % hkv;
      slot_step = hkv;
      if (before + c.n > split.room) c = {1, 0};
    }
    return c;
  };
  DkdvChunks c = {1, 0};
  if (kCut && chunk > 0) {
    c = chunks_of((((uniform(seg_end[t_last]) - 1) / kBS) - ib_lo + 1) * G);
    if (chunk >= c.n) return;  // workgroup-uniform
  }

  const size_t row_bytes = (size_t)hq * d * 2;
  const size_t base_off = (size_t)ib_lo * kBS * row_bytes;
  const size_t total = (size_t)N * row_bytes;
  const buffer_t qbuf = make_buffer((const char *)Q + base_off, total - base_off);
  const buffer_t gbuf = make_buffer((const char *)dO + base_off, total - base_off);
  // HBM -> LDS copy of a 64-row block: 16 transfers of 1 KB (4 rows) per tensor and sub-block, shared
  // out over the waves (transfers of one wave are 4 kWaves rows apart: the same swizzle)
  const int dma_row = wave * 4 + (lane >> 4);
  const uint32_t dma_off = dma_lane_offset(lane, dma_row, row_bytes, 0, d);
  bool dma_ok[kHf];
#pragma unroll
  for (int hf = 0; hf < kHf; ++hf) dma_ok[hf] = dma_lane_ok(lane, dma_row, d - 128 * hf);
  const uint32_t blk_bytes = (uint32_t)(kBS * row_bytes);
  const uint32_t p_bytes = (uint32_t)(4 * kWaves * row_bytes);
  typedef __attribute__((address_space(3))) void *lds_void;
  const int stat_row = threadIdx.x & (kBS - 1);
  const bool stat_is_lse = (threadIdx.x & kBS) == 0;
  const float *stat_src = stat_is_lse ? LSE : delta;
  const float stat_mul = stat_is_lse ? -1.f / scale : -1.f;
  float rstat = 0.f;
  uint16_t *const S0 = stages, *const S1 = stages + kStage;
  auto copy_block = [&](uint16_t *dst, int hh, int ib) {
    {  // every thread loads (a load under a condition would be waited for at the end of the branch)
      const int i = min(ib * kBS + stat_row, N - 1);
      rstat = stat_src[(size_t)(g * G + hh) * N + i];
    }
    const uint32_t off = dma_off + (uint32_t)(ib - ib_lo) * blk_bytes + (uint32_t)((g * G + hh) * d * 2);
#pragma unroll
    for (int hf = 0; hf < kHf; ++hf)
#pragma unroll
      for (int p = 0; p < 16 / kWaves; ++p) {
        const uint32_t o = dma_ok[hf] ? off + p * p_bytes + hf * 256 : kPastEnd;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(qbuf, (lds_void)(dst + hf * kBlk + (kWaves * p + wave) * 512), 16, o, 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(gbuf, (lds_void)(dst + kBlkT + hf * kBlk + (kWaves * p + wave) * 512), 16, o, 0, 0, 0);
      }
  };
  auto put_stats = [&](uint16_t *dst) {
    if (threadIdx.x < 2 * kBS) ((float *)(dst + 2 * kBlkT))[threadIdx.x] = rstat * stat_mul;
  };
  if (!kCut || chunk == 0) copy_block(S0, 0, ib_lo);  // needs nothing but the tile: in flight while the bounds arrive

  // Everything else the prologue needs depends on the tile only: all of it is requested before any
  // of it is looked at (a value made wave-uniform right after its load would hold the next load
  // back by a full memory round trip, four times in a row).
  uint16_t *const kv_tile = kKvInStage ? S1 : kv_own;  // K sub-blocks, then V sub-blocks
  const int jw0 = t0 + kg * 32;
  const int jw1 = min(jw0 + 31, t_last);
  const bool wave_ok = jw0 <= t_last;
  const bool wave_full = jw0 + 31 <= t_last;
  const int j_abs = jw0 + l32;
  const bool row_ok = j_abs <= t_last;
  const int j_ld = min(j_abs, t_last);
  const int se_last_v = seg_end[t_last];
  const int se_min_v = seg_end[min(jw0, t_last)];
  const int se_max_v = seg_end[jw1 < jw0 ? t_last : jw1];
  const int se_j_v = seg_end[j_ld];
  {  // K and V rows t0 .. t0 + kKeys - 1 of head g -> kv_tile: 4 transfers of 4 rows per wave, tensor and sub-block
    const size_t kv_row_bytes = (size_t)hkv * d * 2;
    const size_t kv_off = (size_t)t0 * kv_row_bytes, kv_total = (size_t)N * kv_row_bytes;
    const buffer_t kb = make_buffer((const char *)K + kv_off, kv_total - kv_off);
    const buffer_t vb = make_buffer((const char *)V + kv_off, kv_total - kv_off);
    const uint32_t o0 = dma_lane_offset(lane, dma_row, kv_row_bytes, g, d);
    const uint32_t step = (uint32_t)(4 * kWaves * kv_row_bytes);
#pragma unroll
    for (int hf = 0; hf < kHf; ++hf)
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const uint32_t o = dma_ok[hf] ? o0 + p * step + hf * 256 : kPastEnd;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(kb, (lds_void)(kv_tile + hf * kKvSub + (kWaves * p + wave) * 512), 16, o, 0, 0, kOnce);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(vb, (lds_void)(kv_tile + (kHf + hf) * kKvSub + (kWaves * p + wave) * 512), 16, o, 0, 0, kOnce);
      }
  }

  const int ib_hi = (uniform(se_last_v) - 1) / kBS;  // query blocks end with the example of the tile's last key
  int n_it = (ib_hi - ib_lo + 1) * G;
  int n_chunks = 1, it0 = 0;
  if constexpr (kCut) {
    if (chunk == 0) c = chunks_of(n_it);
    n_chunks = c.n;
    it0 = c.first(chunk, n_it);
    n_it = c.end(chunk, n_it) - it0;
  }
  const int se_min = uniform(se_min_v), se_max = uniform(se_max_v);
  const int se_j = row_ok ? se_j_v : 0;  // queries j_abs <= i < se_j see key j_abs

  f32x16 acc[kCb];
#pragma unroll
  for (int cb = 0; cb < kCb; ++cb)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[cb][v] = 0.f;

  const uint32_t row_lane = swz_row_lane_off(lane);
  uint32_t tr_lane[2];
  swz_tr_lane_off(lane, tr_lane);
  u32x4 *const ex = exch + kg * 256 + lane;  // + parity * 128 + part * 64

  x8 rf[kKs];  // this lane's key row: K (the V side computes S) or V (the K side computes dP); set below
  // Order of the streamed blocks.  One query head per KV head: ib_lo, ib_lo + 1, ... ib_hi; neighbouring
  // key tiles of an example, which run next to each other on one XCD, then follow each other two steps
  // apart and find the blocks in L2.  Grouped heads: block ib_lo (the tile's own first rows; needs no
  // bounds, so its copy is in flight while they arrive) for every head of the group, then blocks ib_hi,
  // ib_hi - 1, ... ib_lo + 1, each for every head: the key tiles of one example share ib_hi, so they
  // stream the same block at about the same time, whereas ascending they would run 2 G steps apart per
  // tile and the blocks would have left the L2 (measured traffic of the kernel with 5 query heads per KV
  // head and examples of thousands of tokens: 3.8 GB ascending, 2.9 GB this way; the same run time).
  int ib_nxt = ib_lo, hh_nxt = 0;
  if (kCut && chunk > 0) {  // the chunk's first trip in that order
    const int b = it0 / G;
    hh_nxt = it0 - b * G;
    ib_nxt = G == 1 ? ib_lo + b : b == 0 ? ib_lo : ib_hi + 1 - b;
    copy_block(S0, hh_nxt, ib_nxt);
  }
  int ib_cur = ib_nxt;
  // The K side runs one sub-block behind the V side: in step k the V side computes S(k), P(k) (left in
  // LDS) and dV(k), the K side computes dP(k) and, with the P(k-1) published by the previous barrier,
  // dS(k-1) and dK(k-1).  No wave waits for another inside a step; one barrier ends each step.  The
  // two sides run separate loops (same barriers, same block copies) so that each keeps only its own
  // values in registers.
  auto read_ty = [&](x8 (&ty)[2][kCb], const uint16_t *__restrict__ Ys, int row0) {
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int cb = 0; cb < kCb; ++cb) ty[s2][cb] = swz_read_tr<E>(Ys + (cb >> 2) * kBlk, tr_lane, cb & 3, row0 + s2 * 16);
  };
  auto first_product = [&](f32x16 &x, const uint16_t *__restrict__ Xs, const float *__restrict__ st, int row0) {
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const f32x4 c = *(const f32x4 *)(st + row0 + q4 * 8 + half * 4);
#pragma unroll
      for (int b = 0; b < 4; ++b) x[q4 * 4 + b] = c[b];
    }
    // fragment reads run kAheadKv k-steps ahead of their matrix instructions (see kAhead)
    x8 ax[kAheadKv];
#pragma unroll
    for (int ks = 0; ks < kAheadKv; ++ks) ax[ks] = swz_read_row<E>(Xs + (ks >> 3) * kBlk, row_lane, ks & 7, row0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < kKs; ++ks) {
      x = mfma32(ax[ks % kAheadKv], rf[ks], x);  // S - LSE / scale, or dP - D
      if (ks + kAheadKv < kKs) {
        const int kn = ks + kAheadKv;
        ax[ks % kAheadKv] = swz_read_row<E>(Xs + (kn >> 3) * kBlk, row_lane, kn & 7, row0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // `split` (wave-uniform): x holds entries large enough for their bf16 rounding to matter; their
  // residuals go through the matrix pipe as a second operand (see kSplitP / kSplitS)
  auto second_product = [&](const f32x16 &x, const x8 (&ty)[2][kCb], bool split) {
    const x8 f0 = pack_x8<E>(x, 0), f1 = pack_x8<E>(x, 8);
#pragma unroll
    for (int cb = 0; cb < kCb; ++cb) acc[cb] = mfma32(ty[0][cb], f0, acc[cb]);  // dV^T += dO^T P, dK^T += Q^T dS
#pragma unroll
    for (int cb = 0; cb < kCb; ++cb) acc[cb] = mfma32(ty[1][cb], f1, acc[cb]);
    if (split) {
      const x8 r0 = pack_residual_x8<E>(x, 0, f0), r1 = pack_residual_x8<E>(x, 8, f1);
#pragma unroll
      for (int cb = 0; cb < kCb; ++cb) acc[cb] = mfma32(ty[0][cb], r0, acc[cb]);
#pragma unroll
      for (int cb = 0; cb < kCb; ++cb) acc[cb] = mfma32(ty[1][cb], r1, acc[cb]);
    }
  };
  auto v_step = [&](const uint16_t *__restrict__ cur, int il, int row0, int pw) {
    f32x16 x;
    x8 ty[2][kCb];
    first_product(x, cur, (const float *)(cur + 2 * kBlkT), row0);
    read_ty(ty, cur + kBlkT, row0);
#pragma unroll
    for (int v = 0; v < 16; ++v) x[v] = __builtin_amdgcn_exp2f(x[v] * scale_log2);  // P
    const bool interior = wave_full && il >= jw1 && il + 31 < se_min;
    if (!interior) hide(x, visible_rows(j_abs - il, se_j - il, half), 0.f);
    // P goes to the K side as fp16 whatever the inputs' type: probabilities lie in [0, 1], where fp16
    // keeps 11 significant bits (bf16: 8) down to 6e-5 and absolute 2^-25 below
    ex[pw * 128] = __builtin_bit_cast(u32x4, pack_x8<F16>(x, 0));
    ex[pw * 128 + 64] = __builtin_bit_cast(u32x4, pack_x8<F16>(x, 8));
    second_product(x, ty, needs_split<E>::value && __any(abs_max16(x) > kSplitP));
  };
  auto k_finish = [&](f32x16 &x, const x8 (&ty)[2][kCb], int pr) {  // dS = P (dP - D); dK
    const f16x8 p0 = as_x8<F16>(ex[pr * 128]), p1 = as_x8<F16>(ex[pr * 128 + 64]);
#pragma unroll
    for (int e = 0; e < 8; ++e) {  // written as fma(p, x, +0): one mixed-precision instruction instead of convert + multiply
      x[e] = __builtin_fmaf((float)p0[e], x[e], 0.f);
      x[8 + e] = __builtin_fmaf((float)p1[e], x[8 + e], 0.f);
    }
    second_product(x, ty, needs_split<E>::value && __any(abs_max16(x) > kSplitS));
  };
  bool more = false;
  auto begin_block = [&](int it, uint16_t *__restrict__ nxt) {  // returns the block's first query
    more = it + 1 < n_it;  // workgroup-uniform
    if (++hh_nxt == G) {  // all heads of the group have had this block
      hh_nxt = 0;
      ib_nxt = G == 1 ? ib_nxt + 1 : ib_nxt == ib_lo ? ib_hi : ib_nxt - 1;
    }
    if (more) copy_block(nxt, hh_nxt, ib_nxt);
    const int i0 = ib_cur * kBS;
    ib_cur = ib_nxt;
    return i0;
  };
  auto end_block = [&](uint16_t *__restrict__ nxt) {
    if (more) put_stats(nxt);
    wait_all_loads();
    lds_barrier();  // P published; next block published; every read of this stage is done
  };
  // wave-uniform and the same on both sides: does sub-block [il, il + 32) hold a pair of this wave?
  auto is_active = [&](int il) { return wave_ok && il + 31 >= jw0 && il < se_max; };
  auto v_iteration = [&](int it, const uint16_t *__restrict__ cur, uint16_t *__restrict__ nxt) {
    const int i0 = begin_block(it, nxt);
    if (is_active(i0)) v_step(cur, i0, 0, 0);
    lds_barrier();
    if (is_active(i0 + 32)) v_step(cur, i0 + 32, 32, 1);
    end_block(nxt);
  };
  f32x16 xa, xb;       // K side: dP - D of the two sub-blocks of a block, each waiting for its P
  x8 tyb[2][kCb];      // K side: Q^T fragments of sub-block b (its stage is overwritten before they are used)
  bool act_b = false;  // K side: sub-block b of the previous block is waiting for its P
  auto k_iteration = [&](int it, const uint16_t *__restrict__ cur, uint16_t *__restrict__ nxt) {
    const int i0 = begin_block(it, nxt);
    const float *st = (const float *)(cur + 2 * kBlkT) + kBS;
    const bool act0 = is_active(i0), act1 = is_active(i0 + 32);
    // step 2 it: dP of sub-block a; dS, dK of the previous block's b (P at parity 1)
    if (act0) first_product(xa, cur + kBlkT, st, 0);
    if (act_b) k_finish(xb, tyb, 1);
    lds_barrier();
    // step 2 it + 1: dP of sub-block b; dS, dK of a (P at parity 0)
    if (act1) {
      first_product(xb, cur + kBlkT, st, 32);
      read_ty(tyb, cur, 32);
    }
    if (act0) {
      x8 tya[2][kCb];
      read_ty(tya, cur, 0);
      k_finish(xa, tya, 0);
    }
    act_b = act1;
    end_block(nxt);
  };
  put_stats(S0);
  wait_all_loads();
  lds_barrier();
#pragma unroll
  for (int ks = 0; ks < kKs; ++ks)
    rf[ks] = swz_read_row<E>(kv_tile + ((k_side ? kHf : 0) + (ks >> 3)) * kKvSub, row_lane, ks & 7, kg * 32);
  if (kKvInStage) lds_barrier();  // every wave has its rows before stage 1 receives its first block
  if (!k_side) {
    for (int it = 0; it < n_it; it += 2) {  // bounds are workgroup-uniform: barriers stay aligned
      v_iteration(it, S0, S1);
      if (it + 1 < n_it) v_iteration(it + 1, S1, S0);
    }
  } else {
    for (int it = 0; it < n_it; it += 2) {
      k_iteration(it, S0, S1);
      if (it + 1 < n_it) k_iteration(it + 1, S1, S0);
    }
    if (act_b) k_finish(xb, tyb, 1);  // the last sub-block's dK
  }
  if (kCut && n_chunks > 1) {  // leave the accumulators to the merge kernel: [wave][4-register group][lane] x 16 B
    float *out = split.partial + (size_t)(slot0 + chunk * slot_step) * (2 * kKeys * kDh) +
                 ((kg * 2 + (k_side ? 1 : 0)) * kCb * 4 * 64 + lane) * 4;
#pragma unroll
    for (int cb = 0; cb < kCb; ++cb)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        f32x4 x;
#pragma unroll
        for (int b = 0; b < 4; ++b) x[b] = acc[cb][4 * q4 + b];
        *(f32x4 *)(out + (cb * 4 + q4) * 256) = x;
      }
    return;
  }
  float *stage = (float *)stages + wave * kStageFloatsPerWave;
  const int nrows = wave_ok ? jw1 - jw0 + 1 : 0;
  if (k_side)
    store_transposed_tile<EOut, kCb>(acc, scale, stage, dK, jw0, nrows, hkv, g, d);
  else
    store_transposed_tile<EOut, kCb>(acc, 1.f, stage, dV, jw0, nrows, hkv, g, d);
}

// dK, dV of the tiles whose trips were cut into chunks: the sum of the chunks' accumulators.  One workgroup
// per (schedule tile, KV head, 32-key group): waves 0, 1 add dV, waves 2, 3 dK, each 64 columns at a time, the
// chunks in ascending order.  key_groups: 32-key groups per workgroup tile of the dK/dV kernel that ran (its
// shape, `small` / `large`, is chosen by the same test as there).  Bound: the partial sums, written once and
// read once, mostly from the last-level cache.
template <class EOut, int kDh>
__global__ void __launch_bounds__(256)
dkdv_merge_kernel(void *__restrict__ dK, void *__restrict__ dV, const int32_t *__restrict__ seg_end,
                  const int32_t *__restrict__ kv_tile_order, const int32_t *__restrict__ meta, DkdvPick pick,
                  DkdvSplit small, DkdvSplit large, int N, int T, int tiles_per_row, int hq, int hkv, int d, float scale) {
  constexpr int kCb = kDh / 32;
  __shared__ __attribute__((aligned(16))) float lds[4 * kStageFloatsPerWave];
  const bool is_small = kDh <= 128 && (pick.select == 2 || (pick.select == 0 && dkdv_small(meta[0], meta[2], pick)));
  const DkdvSplit split = is_small ? small : large;
  const int key_groups = is_small || kDh > 128 ? 2 : 4;
  const int sub_tiles = VA_TILE / 32 / key_groups;
  if (split.max_chunks == 1) return;
  const DkdvPlan plan = dkdv_plan(meta, 32 * key_groups, is_small ? 512 : 256, N, T, tiles_per_row, hq, hq / hkv, split);
  if (plan.most == 1) return;  // before any tile is looked up
  const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
  const int kgi = blockIdx.x % (VA_TILE / 32), head_slot = blockIdx.x / (VA_TILE / 32) % hkv;
  const int rank = blockIdx.x / (VA_TILE / 32 * hkv);
  const int sub = kgi / key_groups, kg = kgi % key_groups;
  const int pair = (rank * sub_tiles + sub) * hkv + head_slot;
  const int entry = uniform(kv_tile_order[rank]);
  const int tile = order_tile(entry), g = (head_slot + head_rotation(entry)) % hkv;
  const int r = tile / tiles_per_row, m = tile % tiles_per_row;
  const int row_end = (r + 1) * T;
  const int keys = 32 * key_groups, t0 = r * T + m * VA_TILE + sub * keys;
  if (t0 + kg * 32 >= row_end) return;
  const int t_last = min(t0 + keys, row_end) - 1;
  const int n_it = ((uniform(seg_end[t_last]) - 1) / kBS - t0 / kBS + 1) * (hq / hkv);
  const int n_chunks = dkdv_chunks(n_it, plan, hq / hkv, split).n;
  if (n_chunks == 1) return;  // stored by its only workgroup
  int slot0 = pair * split.max_chunks, slot_step = 1;
  if (!split.fine) {
    const int before = dkdv_first_slot<256>(pair / hkv, keys, seg_end, kv_tile_order, T, tiles_per_row, hq / hkv, plan, split, (int *)lds);
    if (before + n_chunks > split.room) return;  // likewise
    slot0 = before * hkv + head_slot;
    slot_step = hkv;
  }
  const int side = wave >> 1;
  const int nrows = min(32, row_end - (t0 + kg * 32));
  const size_t slot = (size_t)2 * keys * kDh * slot_step;
  const float *src = split.partial + (size_t)slot0 * (2 * keys * kDh) + ((kg * 2 + side) * kCb * 1024 + lane * 4);
#pragma unroll 1
  for (int p = wave & 1; p < (kCb + 1) / 2; p += 2) {
    f32x16 acc[2];
#pragma unroll
    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[cc][v] = 0.f;
    const int n4 = min(2, kCb - 2 * p) * 4;  // 4-register groups of this half
    // kFly chunks are requested together (8 KB each): one at a time is a chain of memory round trips
    auto add = [&](int c0, auto fly) {
      constexpr int kFly = decltype(fly)::value;
      f32x4 x[kFly][8];
#pragma unroll
      for (int f = 0; f < kFly; ++f)
#pragma unroll
        for (int i = 0; i < 8; ++i) x[f][i] = *(const f32x4 *)(src + (c0 + f) * slot + (p * 8 + min(i, n4 - 1)) * 256);
#pragma unroll
      for (int f = 0; f < kFly; ++f)
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int b = 0; b < 4; ++b) acc[i >> 2][(i & 3) * 4 + b] += x[f][i][b];
    };
    int c = 0;
    for (; c + 4 <= n_chunks; c += 4) add(c, std::integral_constant<int, 4>());
    if (c + 2 <= n_chunks) { add(c, std::integral_constant<int, 2>()); c += 2; }
    if (c < n_chunks) add(c, std::integral_constant<int, 1>());
    store_transposed_half<EOut, kCb>(acc, p, side ? scale : 1.f, lds + wave * kStageFloatsPerWave, side ? dK : dV,
                                     t0 + kg * 32, nrows, hkv, g, d);
  }
}

}  // namespace

// How the (tile, KV head) pairs of one workgroup shape may be cut (see DkdvSplit): finely if kDkdvSplitBytes hold
// at least two chunks of every pair; else, with grouped heads and up to kMorePairs pairs per resident workgroup, only the
// longest chains (that is as far as cuts were measured); and not where no row is long enough (longest_chain: trips of one
// that a single example fills).  Cut over uncut there, one such row: 32 trips, 128, 256 and 512 pairs 0.68, 0.91
// and 1.07 (head_dim 64: 1.25); 24 trips, 384 pairs 0.96; 48, 384 0.81; 64, 512 0.88.
// Where a row could hold a long example, but none is, the idle workgroups and the merge launch cost 1 to 5 us.
// slots: workgroups of the shape that the chip holds.
constexpr int kMorePairs = 3;
static DkdvSplit plan_split(const Partials &partial, size_t slot_bytes, long long n_pairs, int hq, int hkv, long long longest_chain, int slots) {
  const DkdvSplit none = {partial.p, 1, true, 0};
  if (longest_chain < 3 * kMinTrips || longest_chain * slots < 6 * kMinTrips * std::min(n_pairs, (long long)slots)) return none;
  const long long trips = longest_chain / kMinTrips;
  if (n_pairs * 2 <= (long long)(kDkdvSplitBytes / slot_bytes)) {
    const int n = (int)std::min({(long long)(partial.bytes / slot_bytes) / n_pairs, trips, (long long)kMaxChunks});
    return n >= 2 ? DkdvSplit{partial.p, n, true, 0} : none;
  }
  const int room = (int)(partial.bytes / slot_bytes) / hkv;
  if (hq == hkv || n_pairs > kMorePairs * slots || room < 2) return none;
  return {partial.p, (int)std::min({2 * kMorePairs * slots / n_pairs, trips, (long long)kMaxChunksMany}), false, room};
}

// The plans of both shapes for rows of T tokens.
template <int kDh> struct DkdvLaunch {
  typedef DkdvShape<kDh, false> Large;
  typedef DkdvShape<kDh, (kDh <= 128)> Small;  // head_dim above 128 has one shape
  long long n_large, n_small;                  // (workgroup tile, KV head) pairs
  DkdvSplit large, small;
  DkdvLaunch(const Partials &partial, int N, int T, int hq, int hkv) {
    const long long tiles = (T + VA_TILE - 1ll) / VA_TILE * (N / T) * hkv;
    n_large = tiles * Large::kSubTiles;
    n_small = tiles * Small::kSubTiles;
    const int off = N == T || T % kBS == 0 ? 0 : kBS - 1;  // a row may begin that far behind a multiple of the block
    const long long longest_chain = ((T - 1ll + off) / kBS + 1) * (hq / hkv);
    large = plan_split(partial, (size_t)2 * Large::kKeys * kDh * 4, n_large, hq, hkv, longest_chain, 256 * Large::kWgPerCu);
    small = plan_split(partial, (size_t)2 * Small::kKeys * kDh * 4, n_small, hq, hkv, longest_chain, 256 * Small::kWgPerCu);
  }
};

template <class F> static auto by_head_dim(int d, F f) {
  if (d <= 64) return f(std::integral_constant<int, 64>());
  if (d <= 96) return f(std::integral_constant<int, 96>());
  if (d <= 128) return f(std::integral_constant<int, 128>());
  return f(std::integral_constant<int, 256>());
}

size_t mfma_partial_bytes(int N, int hq, int hkv, int d) {
  if (d % 8 != 0 || d > 256 || hq % hkv != 0) return 0;
  return by_head_dim(d, [&](auto dh) {  // in one row tiles are fewest and chains longest
    const DkdvLaunch<decltype(dh)::value> l({nullptr, kDkdvSplitBytes}, N, N, hq, hkv);
    return l.large.max_chunks > 1 || l.small.max_chunks > 1 ? kDkdvSplitBytes : (size_t)0;
  });
}

template <class E, class EOut, int kDh>
static void launch_bwd_t(const uint16_t *g, const uint16_t *q, const uint16_t *k, const uint16_t *v,
                         const uint16_t *o, const float *LSE, float *delta, void *dQ, void *dK, void *dV,
                         const va_segments &seg, int N, int T, int tiles_per_row, int hq, int hkv, int d,
                         float scale, unsigned gq, unsigned gkv, const Partials &partial, hipStream_t stream, unsigned stages) {
  const float scale_log2 = scale * kLog2e;
  if (stages & VA_STAGE_DQ)  // first: it also produces D for the dK/dV kernel
    dq_mfma_kernel<E, EOut, kDh><<<gq, 256, 0, stream>>>(g, q, k, v, o, LSE, delta, dQ, seg.seg_start,
                                                         seg.q_tile_order, N, T, tile_map(hq, hkv, tiles_per_row, gq), hq, hkv, d,
                                                         scale_log2, scale);
  if (stages & VA_STAGE_DKDV) {
    typedef typename DkdvLaunch<kDh>::Large Large;
    typedef typename DkdvLaunch<kDh>::Small Small;
    const DkdvLaunch<kDh> l(partial, N, T, hq, hkv);
    const DkdvSplit &sl = l.large, &ss = l.small;
    // Nothing about the lengths is known on the host: both shapes are launched and the device picks, unless
    // the caller's hint names the shape or no example can be as long as calls for the large one: four tiles of a row of 1023
    // tokens, begun 63 tokens behind a multiple of the block, stream at most 17 + 13 + 9 + 5 blocks, 11 a tile.
    static_assert(kDkdvLongMean == 1024 && kBS == 64 && VA_TILE == 256 && kDkdvLongBlocks > 11, "shorter rows may call for the large shape");
    bool run_large = kDh > 128 || !(stages & VA_HINT_SHORT_EXAMPLES);
    bool run_small = kDh <= 128 && !(stages & VA_HINT_LONG_EXAMPLES);
    if (run_small && T < kDkdvLongMean) run_large = false;
    const int select_large = run_small ? 1 : 0, select_small = run_large ? 2 : 0;
    // where tiles may be cut finely the mean decides alone
    const long long long_blocks = (long long)kDkdvLongBlocks * (N / T) * tiles_per_row;
    const int blocks = ss.max_chunks > 1 && ss.fine ? INT_MAX : (int)std::min<long long>(long_blocks, INT_MAX);
    auto pick = [&](int select) { return DkdvPick{select, N / kDkdvLongMean, blocks}; };
    auto launch = [&](auto *kernel, long long pairs, int threads, int select, const DkdvSplit &split) {
      kernel<<<(unsigned)(pairs * split.max_chunks), threads, 0, stream>>>(g, q, k, v, LSE, delta, dK, dV, seg.seg_end, seg.kv_tile_order, seg.meta,
                                                                           pick(select), split, N, T, fast_div(tiles_per_row), fast_div(hkv), hq / hkv, hq, hkv, d,
                                                                           scale_log2, scale);
    };
    if (run_large)
      launch(sl.max_chunks > 1 ? dkdv_mfma_kernel<E, EOut, kDh, false, true> : dkdv_mfma_kernel<E, EOut, kDh, false, false>, l.n_large,
             Large::kThreads, select_large, sl);
    if constexpr (kDh <= 128) {
      if (run_small)
        launch(ss.max_chunks > 1 ? dkdv_mfma_kernel<E, EOut, kDh, true, true> : dkdv_mfma_kernel<E, EOut, kDh, true, false>, l.n_small,
               Small::kThreads, select_small, ss);
    }
    if ((run_large && sl.max_chunks > 1) || (run_small && ss.max_chunks > 1))
      dkdv_merge_kernel<EOut, kDh><<<(unsigned)(gkv / kSub * (VA_TILE / 32)), 256, 0, stream>>>(
          dK, dV, seg.seg_end, seg.kv_tile_order, seg.meta, pick(run_large && run_small ? 0 : run_small ? 2 : 1), ss, sl, N, T,
          tiles_per_row, hq, hkv, d, scale);
  }
}

template <class E, class EOut, class... A>
static void launch_bwd_d(int d, A... a) {
  if (d <= 64) launch_bwd_t<E, EOut, 64>(a...);
  else if (d <= 96) launch_bwd_t<E, EOut, 96>(a...);
  else if (d <= 128) launch_bwd_t<E, EOut, 128>(a...);
  else launch_bwd_t<E, EOut, 256>(a...);
}

hipError_t launch_mfma_bwd(const void *dO, const void *Q, const void *K, const void *V, const void *O,
                           const float *LSE, float *delta, void *dQ, void *dK, void *dV,
                           va_dtype grad_dt, const va_segments &seg, int rows, int T, int hq,
                           int hkv, int d, va_dtype dt, float scale, const Partials &partial, hipStream_t stream, unsigned stages) {
  const int tiles_per_row = ceil_div(T, VA_TILE);
  const long long ntiles = (long long)rows * tiles_per_row * kSub;
  if (ntiles * hq > 0x7fffffffll) return hipErrorInvalidValue;
  const int N = rows * T;
  const uint16_t *q = (const uint16_t *)Q, *k = (const uint16_t *)K, *v = (const uint16_t *)V,
                 *g = (const uint16_t *)dO, *o = (const uint16_t *)O;
  const unsigned gq = (unsigned)(ntiles * hq), gkv = (unsigned)(ntiles * hkv);
  if (dt == VA_F16) {
    if (grad_dt == VA_F32)
      launch_bwd_d<F16, float>(d, g, q, k, v, o, LSE, delta, dQ, dK, dV, seg, N, T, tiles_per_row, hq, hkv, d, scale,
                               gq, gkv, partial, stream, stages);
    else
      launch_bwd_d<F16, F16>(d, g, q, k, v, o, LSE, delta, dQ, dK, dV, seg, N, T, tiles_per_row, hq, hkv, d, scale,
                             gq, gkv, partial, stream, stages);
  } else {
    if (grad_dt == VA_F32)
      launch_bwd_d<Bf16, float>(d, g, q, k, v, o, LSE, delta, dQ, dK, dV, seg, N, T, tiles_per_row, hq, hkv, d, scale,
                                gq, gkv, partial, stream, stages);
    else
      launch_bwd_d<Bf16, Bf16>(d, g, q, k, v, o, LSE, delta, dQ, dK, dV, seg, N, T, tiles_per_row, hq, hkv, d, scale,
                               gq, gkv, partial, stream, stages);
  }
  return hipGetLastError();
}


}  // namespace va
