// Kernels in fp32 arithmetic: any element type (fp32 / bf16 / fp16), any head_dim <= 256.
//
// They serve the fp32 path (where 16-bit matrix operands cannot give the required accuracy) and the
// 16-bit head dims that are not a multiple of 8.  All products run on the fp32 matrix instruction
// v_mfma_f32_16x16x4_f32, D[16x16] += A[16x4] * B[4x16].  Register layout per 64-lane wave (lane l, l16 = l % 16,
// kq = l / 16):
//   A : row l16, k = kq     B : column l16, k = kq     D : column l16, 4 floats v at row 4 kq + v
// The order of the k index of a product is free, as long as A and B agree, and so is the order of the output
// rows; both are chosen so that every operand is loaded straight from memory in 16-byte pieces, without LDS:
//   - contraction over the head_dim (S, dP): the 4 lanes of a row take 4 consecutive columns each of every 16
//     (load_row), so 4 values per 16-byte load serve 4 matrix instructions;
//   - contraction over the streamed tokens (O, dQ, dK, dV): register v of a first-product result is, as it is,
//     the B operand of the k-step that covers tokens 4 kq + v; the A operand of that step are 4 consecutive
//     columns of those tokens (load_cols), which makes output register e hold the columns 4 row + e: a lane ends
//     up with 16 consecutive columns of its row and stores them in 16-byte pieces.
// Tiles are 16 tokens (of the flat stream) x one head; the four waves of a workgroup share out the streamed blocks
// of 32 tokens and add their results through LDS in a fixed order.  Small tiles and that split make short chains
// and many workgroups: fp32 runs are checks of a few hundred to a few thousand tokens and few heads.  (Eight waves
// per workgroup, one workgroup per CU instead of two: the dQ kernel below took 28 us when with four it took 22.)
// The mask is "seg_start[i] <= j <= i" (forward, dQ) or "j <= i < seg_end[j]" (dK/dV) -- Table 1's correct
// cross-attention for contiguous examples.  Tokens outside it leave no trace, whatever they hold: the matrix products
// run on whole blocks with a masked factor of 0, and a wave that meets another factor in such a block that is not finite
// (0 * Inf = NaN) forms its sums again, token by token (`redo`).
// Measured, 1000 tokens, 8 query / 2 KV heads, d = 64, examples of up to 315 tokens, against one wave per output row
// on the vector units: forward 257 -> 14 us, dQ (with D) 214 -> 19 us, dK/dV 484 -> 32 us.  Bound there by the
// matrix instructions of the CUs that hold the longest examples' tiles; one example of 8000 tokens runs the
// forward at 76 TFLOP/s, half of what a large fp32 library product reaches.
#include <algorithm>

#include "va_internal.h"
#include "va_mfma_common.h"

namespace va {
namespace {

constexpr int kRows = 16;    // tokens per workgroup
constexpr int kStep = 32;    // streamed tokens per block (two 16 x 16 sub-blocks)
constexpr int kWaves = 4;    // waves of a workgroup

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// n consecutive elements from p as floats; kVec: p is aligned for one load.
template <typename T, bool kVec, int n> __device__ __forceinline__ void load_n(const T *p, float (&f)[n]) {
  if constexpr (kVec && n > 1) {
    typedef T vec __attribute__((ext_vector_type(n)));
    const vec x = *(const vec *)p;
#pragma unroll
    for (int e = 0; e < n; ++e) f[e] = (float)x[e];
  } else {
#pragma unroll
    for (int e = 0; e < n; ++e) f[e] = (float)p[e];
  }
}
// Columns c .. c + n - 1 of a head vector of d columns, zeros beyond it.  The address is clamped and the value
// selected, not the load made conditional: conditional loads go out one at a time.
template <typename T, bool kVec, int n>
__device__ __forceinline__ void load_cols_at(const T *row, int c, int d, float (&f)[n]) {
  if constexpr (kVec) {  // d a multiple of 4: the n columns lie wholly inside or wholly outside
    load_n<T, true, n>(row + min(c, d - n), f);
#pragma unroll
    for (int e = 0; e < n; ++e) f[e] = c < d ? f[e] : 0.f;
  } else {
#pragma unroll
    for (int e = 0; e < n; ++e) {
      const float x = (float)row[min(c + e, d - 1)];
      f[e] = c + e < d ? x : 0.f;
    }
  }
}
// This lane's share of a row for the products over the head_dim: f[4 i + e] = column 16 i + 4 kq + e.
template <typename T, bool kVec, int kDh>
__device__ __forceinline__ void load_row(const T *row, int kq, int d, float (&f)[kDh / 4]) {
#pragma unroll
  for (int i = 0; i < kDh / 16; ++i) {
    float x[4];
    load_cols_at<T, kVec, 4>(row, 16 * i + 4 * kq, d, x);
#pragma unroll
    for (int e = 0; e < 4; ++e) f[4 * i + e] = x[e];
  }
}

// The products of 16 streamed rows and the tile's 16 rows, over the head_dim, in eight chains of the matrix instruction
// (head_dim 16: four) that are then added in pairs.  An error of a score is an error of its probability, and a single
// chain has two to three times that of the pairwise sums of a wave per row, against 64 bits, scores of about 100,
// head_dim 64: O 1.9e-6 (pairwise 6.7e-7), LSE 1.1e-5 (4.1e-6); two chains 1.1e-6, 6.3e-6; four 7.9e-7, 4.9e-6; eight
// 6.9e-7, 4.3e-6.
template <int kDh> __device__ __forceinline__ f32x4 row_product(const float (&a)[kDh / 4], const float (&b)[kDh / 4]) {
  constexpr int kChains = kDh < 32 ? 4 : 8;
  f32x4 x[kChains];
#pragma unroll
  for (int c = 0; c < kChains; ++c) x[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < kDh / 4; ++i) x[i % kChains] = mfma16(a[i], b[i], x[i % kChains]);
#pragma unroll
  for (int n = kChains / 2; n > 0; n /= 2)
#pragma unroll
    for (int c = 0; c < n; ++c) x[c] += x[c + n];
  return x[0];
}
// dP likewise; up to head_dim 64 it is dP - D, in one chain from -D: more chains take time (backward of 1000 tokens 43.4 ->
// 45.2 us, in two 45.7) and give nothing (dQ 3.7e-6; in eight chains 3.6e-6).  Beyond, D is left to the caller
// (kLessD): eight chains are the faster ones there (backward of 4000 tokens of 128: 1475 us, one from -D 1525).
template <int kDh> constexpr bool kLessD = kDh <= 64;
template <int kDh> __device__ __forceinline__ f32x4 grad_product(const float (&a)[kDh / 4], const float (&b)[kDh / 4], const f32x4 &delta) {
  if constexpr (!kLessD<kDh>) return row_product<kDh>(a, b);
  f32x4 x = -delta;
#pragma unroll
  for (int i = 0; i < kDh / 4; ++i) x = mfma16(a[i], b[i], x);
  return x;
}
// Probability of a scaled score from the row's LSE: the difference is formed before it is scaled for exp2, so that its
// error is that of the score and the LSE, not theirs times the rounding of scale * log2(e).
__device__ __forceinline__ float prob(float s, float scale, float lse) {
  return __builtin_amdgcn_exp2f(fmaf(s, scale, -lse) * 1.4426950408889634f);
}

// Output columns come in groups of 16 kE; within a group, register block e holds the columns kE * row + e.
template <int kDh> struct Cols {
  static constexpr int kE = kDh >= 64 ? 4 : kDh / 16;
  static constexpr int kGroups = kDh / (16 * kE);
};
// This lane's columns of a token, the A operands of one k-step over the tokens, for every column block.
template <typename T, bool kVec, int kDh>
__device__ __forceinline__ void load_cols(const T *row, int l16, int d, float (&x)[Cols<kDh>::kGroups][Cols<kDh>::kE]) {
  constexpr int kE = Cols<kDh>::kE;
#pragma unroll
  for (int g = 0; g < Cols<kDh>::kGroups; ++g) load_cols_at<T, kVec, kE>(row, g * 16 * kE + l16 * kE, d, x[g]);
}
template <int kDh>
__device__ __forceinline__ void add_outer(f32x4 (&acc)[Cols<kDh>::kGroups][Cols<kDh>::kE],
                                          const float (&x)[Cols<kDh>::kGroups][Cols<kDh>::kE], float b) {
#pragma unroll
  for (int g = 0; g < Cols<kDh>::kGroups; ++g)
#pragma unroll
    for (int e = 0; e < Cols<kDh>::kE; ++e) acc[g][e] = mfma16(x[g][e], b, acc[g][e]);
}
// All loads of a block are requested before the first of its products (left alone the compiler requests two
// at a time and waits: eight memory round trips per block), as far as the registers reach: beyond head_dim 64
// the columns are loaded where they are used.
template <int kDh> struct Ahead { static constexpr bool value = kDh <= 64; };
// Workgroups per CU: two up to head_dim 64.  Without the bound the compiler keeps sums in accumulation registers, which every
// rescaling moves to and fro.  The backward keeps to it by requesting the second sub-block's columns only when the rows have been
// used, in their registers (kLateCols).  Forward, 1000 tokens in five examples 14.7 -> 13.7 us, 8000 in one 905 -> 767; dQ
// 19.4 -> 19.0 and 1293 -> 1213, two rows of 1000 tokens, 8 heads of 32, 28.1 -> 18.2.  Not for element-wise loads: dK/dV spills
// 48 registers and more (900 tokens, 8/4 heads of 30: 70 -> 100 us).  Not in dQ up to head_dim 16, where four fit without it
// and the later columns are a second wait: 1105 tokens, 8 heads of 16, 14.3 -> 16.3, 2273 tokens, 2/1, 23.2 -> 26.0.
template <bool kVec, int kDh> constexpr int kPerCu = kVec && kDh <= 64 ? 2 : 1;
template <bool kVec, int kDh> constexpr bool kLateCols = kVec && kDh > 16 && kDh <= 64;
// dK/dV comes in both forms: without the bound it takes 316 registers at head_dim 64, with it it spills 4.  From 768 workgroups
// on, one and a half times what 256 CUs hold at two each, two per CU are faster whatever the lengths (0.78 of the time up to
// 1536, 0.69 beyond; of 2000 random shapes one took 1.06, the others at most 1.02); with four and more query heads per KV head,
// whose chains are longer, from twice as many on (0.82; between 768 and 1536 0.87, but up to 1.16).  With fewer, all are resident
// at once and long chains that begin on one CU stay together, while one at a time is followed by whichever comes next: 256 to
// 512 workgroups take 0.7...1.4 of the time by the lengths, which the host does not know.  Up to head_dim 32 (three per CU)
// the line is at 2048 (0.85; 512 to 768 1.03, up to 1.23) and doubles with two query heads per KV head (2048 to 4096 0.92, up
// to 1.08); up to 16 there is none (1.00...1.08).
template <bool kVec, int kDh> constexpr int kTwoPerCuFrom = !kVec || kDh <= 16 || kDh > 64 ? 0 : kDh <= 32 ? 2048 : 768;
template <int kDh> __device__ __forceinline__ void loads_first() {
  if constexpr (Ahead<kDh>::value) __builtin_amdgcn_sched_barrier(0);
}
template <int kDh> __device__ __forceinline__ void clear(f32x4 (&acc)[Cols<kDh>::kGroups][Cols<kDh>::kE]) {
#pragma unroll
  for (int g = 0; g < Cols<kDh>::kGroups; ++g)
#pragma unroll
    for (int e = 0; e < Cols<kDh>::kE; ++e) acc[g][e] = f32x4{0.f, 0.f, 0.f, 0.f};
}

__device__ __forceinline__ float quad_sum(float x) {  // over the four lanes of a row (l16 + 16 kq)
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}
__device__ __forceinline__ float quad_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16, 64));
  return fmaxf(x, __shfl_xor(x, 32, 64));
}

__device__ __forceinline__ void put(void *out, va_dtype dt, size_t i, float x) {
  if (dt == VA_F32) ((float *)out)[i] = x;
  else if (dt == VA_BF16) ((__bf16 *)out)[i] = (__bf16)x;  // round to nearest even
  else ((_Float16 *)out)[i] = (_Float16)x;
}

// Adds 0 * x to z: z stays 0 as long as all of x is finite.
template <int kDh> __device__ __forceinline__ void probe_finite(float &z, const float (&x)[Cols<kDh>::kGroups][Cols<kDh>::kE]) {
#pragma unroll
  for (int g = 0; g < Cols<kDh>::kGroups; ++g)
#pragma unroll
    for (int e = 0; e < Cols<kDh>::kE; ++e) z = fmaf(x[g][e], 0.f, z);
}
__device__ __forceinline__ bool met_not_finite(float z) { return __any(!(z == 0.f)); }
// For `redo`: the product of two head vectors, the same in the four lanes of a row, and sums = sums * old + w * row for
// this lane's columns (sums: LDS in merge_store's order).  Loops stay loops: unrolled they cost the main loop registers.
template <typename T> __device__ __forceinline__ float dot_token(const T *a, const T *b, int kq, int d) {
  float x = 0.f;
#pragma unroll 1
  for (int c = kq; c < d; c += 4) x = fmaf((float)a[c], (float)b[c], x);
  return quad_sum(x);
}
template <typename T, int kDh>
__device__ __forceinline__ void add_token(float *sums, const T *row, int kq, int d, float old, float w) {
  constexpr int kE = Cols<kDh>::kE;
#pragma unroll 1
  for (int r = 0; r < kDh / 4; ++r) {
    const int c = r / (4 * kE) * (16 * kE) + kq * 4 * kE + r % (4 * kE);
    if (c < d) sums[r * 64] = fmaf(w, (float)row[c], sums[r * 64] * old);
  }
}
template <int kDh> __device__ __forceinline__ void clear_sums(float *sums) {
#pragma unroll 1
  for (int r = 0; r < kDh / 4; ++r) sums[r * 64] = 0.f;
}

// Adds the waves' accumulators (each times its factor f[w] of this lane's row) in the order of the waves and
// stores row `token` of a [N, H, d] tensor.  red: kWaves * (kDh / 4) * 64 floats of LDS.  redone: this wave's sums
// are not in acc, redo(sums) leaves them in its part of red.
template <bool kVec, int kDh, class Redo>
__device__ __forceinline__ void merge_store(const f32x4 (&acc)[Cols<kDh>::kGroups][Cols<kDh>::kE], const float (&f)[kWaves],
                                            float *red, void *out, va_dtype dt, size_t row_off, bool row_ok, int d,
                                            bool redone, Redo redo) {
  constexpr int kE = Cols<kDh>::kE, kRegs = kDh / 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, kq = lane >> 4;
  __syncthreads();  // the previous use of `red` is over
  float *const sums = red + wave * kRegs * 64 + lane;
  if (redone) {
    redo(sums);
  } else {
#pragma unroll
    for (int g = 0; g < Cols<kDh>::kGroups; ++g)
#pragma unroll
      for (int e = 0; e < kE; ++e)
#pragma unroll
        for (int v = 0; v < 4; ++v) sums[((g * 4 + v) * kE + e) * 64] = acc[g][e][v];
  }
  __syncthreads();
  // register r of a lane is column (r / 4kE) * 16 kE + kq * 4 kE + r % 4kE; wave w takes every kWaves-th run of 4
  for (int r0 = wave * 4; r0 < kRegs; r0 += kWaves * 4) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
#pragma unroll
      for (int b = 0; b < 4; ++b) x[b] += f[w] * red[(w * kRegs + r0 + b) * 64 + lane];
    const int c = r0 / (4 * kE) * (16 * kE) + kq * 4 * kE + r0 % (4 * kE);
    if (!row_ok) continue;
    if (kVec && dt == VA_F32) {
      if (c < d) *(f32x4 *)((float *)out + row_off + c) = x;
    } else {
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (c + b < d) put(out, dt, row_off + c + b, x[b]);
    }
  }
}

template <typename T, bool kVec, int kDh>
__global__ void __launch_bounds__(64 * kWaves, (kPerCu<kVec, kDh>))
f32_fwd_kernel(const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V, void *__restrict__ O,
               float *__restrict__ LSE, const int32_t *__restrict__ seg_start, int N, int hq, int hkv, int d,
               va_dtype dt, float scale_log2, float scale) {
  __shared__ float red[kWaves * (kDh / 4) * 64], s_m[kWaves][kRows], s_l[kWaves][kRows];
  const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6), l16 = lane & 15, kq = lane >> 4;
  const int h = blockIdx.x % hq, g = h / (hq / hkv), t0 = (int)(blockIdx.x / hq) * kRows;
  const int hi = min(t0 + kRows, N) - 1, i_abs = t0 + l16, i_ld = min(i_abs, hi);
  const int lo = uniform(seg_start[t0]), ss_i = seg_start[i_ld];
  const size_t kv_row = (size_t)hkv * d;
  const T *Kh = K + (size_t)g * d, *Vh = V + (size_t)g * d;
  float qf[kDh / 4];
  load_row<T, kVec, kDh>(Q + ((size_t)i_ld * hq + h) * d, kq, d, qf);
  f32x4 acc[Cols<kDh>::kGroups][Cols<kDh>::kE];
  clear<kDh>(acc);
  float m = -INFINITY, l = 0.f, z = 0.f;
  for (int j0 = lo + kStep * wave; j0 <= hi; j0 += kStep * kWaves) {
    const bool mixed = __any(j0 < ss_i || j0 + kStep - 1 > i_abs);  // some row of the tile does not see all of the block
    f32x4 s[2];
    float kf[2][kDh / 4], vc[2][4][Cols<kDh>::kGroups][Cols<kDh>::kE];
    auto value_cols = [&](int b, int v) {
      load_cols<T, kVec, kDh>(Vh + (size_t)min(j0 + 16 * b + 4 * kq + v, hi) * kv_row, l16, d, vc[b][v]);
    };
#pragma unroll
    for (int b = 0; b < 2; ++b) load_row<T, kVec, kDh>(Kh + (size_t)min(j0 + 16 * b + l16, hi) * kv_row, kq, d, kf[b]);
    if constexpr (Ahead<kDh>::value) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) value_cols(b, v);
    }
    loads_first<kDh>();
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      s[b] = row_product<kDh>(kf[b], qf);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int j = j0 + 16 * b + 4 * kq + v;
        if (j < ss_i || j > i_abs) s[b][v] = -INFINITY;
      }
    }
    float mx = m;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) mx = fmaxf(mx, s[b][v]);
    mx = quad_max(mx);
    const float base = mx == -INFINITY ? 0.f : mx;  // nothing unmasked yet: exp2(-inf - 0) = 0
    const float alpha = mx == m ? 1.f : __builtin_amdgcn_exp2f((m - base) * scale_log2);
    m = mx;
    l *= alpha;
#pragma unroll
    for (int gr = 0; gr < Cols<kDh>::kGroups; ++gr)
#pragma unroll
      for (int e = 0; e < Cols<kDh>::kE; ++e) acc[gr][e] *= alpha;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float p = __builtin_amdgcn_exp2f((s[b][v] - base) * scale_log2);
        l += p;
        if constexpr (!Ahead<kDh>::value) value_cols(b, v);
        if (mixed) probe_finite<kDh>(z, vc[b][v]);
        add_outer<kDh>(acc, vc[b][v], p);
      }
  }
  const bool redone = met_not_finite(z);
  if (redone) {
    float *const sums = red + wave * (kDh / 4) * 64 + lane;
    clear_sums<kDh>(sums);
    m = -INFINITY;
    l = 0.f;
    for (int j0 = lo + kStep * wave; j0 <= hi; j0 += kStep * kWaves)
      for (int j = j0; j <= min(j0 + kStep - 1, hi); ++j) {
        const float s = dot_token(Q + ((size_t)i_ld * hq + h) * d, Kh + (size_t)j * kv_row, kq, d);
        if (j < ss_i || j > i_abs) continue;  // the same in the four lanes of a row
        const float mx = fmaxf(m, s), base = mx == -INFINITY ? 0.f : mx;
        const float alpha = mx == m ? 1.f : __builtin_amdgcn_exp2f((m - base) * scale_log2);
        const float p = __builtin_amdgcn_exp2f((s - base) * scale_log2);
        m = mx;
        l = l * alpha + (kq == 0 ? p : 0.f);
        add_token<T, kDh>(sums, Vh + (size_t)j * kv_row, kq, d, alpha, p);
      }
  }
  l = quad_sum(l);
  if (kq == 0) { s_m[wave][l16] = m; s_l[wave][l16] = l; }
  __syncthreads();
  float m_all = -INFINITY, l_all = 0.f, f[kWaves];
#pragma unroll
  for (int w = 0; w < kWaves; ++w) m_all = fmaxf(m_all, s_m[w][l16]);
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    f[w] = __builtin_amdgcn_exp2f((s_m[w][l16] - m_all) * scale_log2);
    l_all += f[w] * s_l[w][l16];
  }
#pragma unroll
  for (int w = 0; w < kWaves; ++w) f[w] /= l_all;
  if (wave == 0 && kq == 0 && i_abs <= hi) LSE[(size_t)h * N + i_abs] = m_all * scale + __logf(l_all);
  merge_store<kVec, kDh>(acc, f, red, O, dt, ((size_t)i_ld * hq + h) * d, i_abs <= hi, d, redone, [](float *) {});
}

// dQ; also forms D = dO . O of its rows and leaves it for the dK/dV kernel.
template <typename T, bool kVec, int kDh>
__global__ void __launch_bounds__(64 * kWaves, (kLateCols<kVec, kDh> ? 2 : 1))
f32_dq_kernel(const T *__restrict__ dO, const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V,
              const T *__restrict__ O, const float *__restrict__ LSE, float *__restrict__ delta, void *__restrict__ dQ,
              const int32_t *__restrict__ seg_start, int N, int hq, int hkv, int d, va_dtype gdt, float scale) {
  __shared__ float red[kWaves * (kDh / 4) * 64];
  const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6), l16 = lane & 15, kq = lane >> 4;
  const int h = blockIdx.x % hq, g = h / (hq / hkv), t0 = (int)(blockIdx.x / hq) * kRows;
  const int hi = min(t0 + kRows, N) - 1, i_abs = t0 + l16, i_ld = min(i_abs, hi);
  const int lo = uniform(seg_start[t0]), ss_i = seg_start[i_ld];
  const float lse = LSE[(size_t)h * N + i_ld];
  const size_t kv_row = (size_t)hkv * d, q_off = ((size_t)i_ld * hq + h) * d;
  const T *Kh = K + (size_t)g * d, *Vh = V + (size_t)g * d;
  float qf[kDh / 4], gf[kDh / 4], dl = 0.f;
  load_row<T, kVec, kDh>(Q + q_off, kq, d, qf);
  load_row<T, kVec, kDh>(dO + q_off, kq, d, gf);
  {
    float of[kDh / 4];
    load_row<T, kVec, kDh>(O + q_off, kq, d, of);
#pragma unroll
    for (int i = 0; i < kDh / 4; ++i) dl = fmaf(gf[i], of[i], dl);
  }
  dl = quad_sum(dl);
  if (wave == 0 && kq == 0 && i_abs <= hi) delta[(size_t)h * N + i_abs] = dl;
  f32x4 acc[Cols<kDh>::kGroups][Cols<kDh>::kE];
  clear<kDh>(acc);
  float z = 0.f;
  for (int j0 = lo + kStep * wave; j0 <= hi; j0 += kStep * kWaves) {
    const bool mixed = __any(j0 < ss_i || j0 + kStep - 1 > i_abs);
    f32x4 s[2];
    float kf[2][kDh / 4], vf[2][kDh / 4], kc[2][4][Cols<kDh>::kGroups][Cols<kDh>::kE];
    auto rows = [&](int b) {
      const size_t off = (size_t)min(j0 + 16 * b + l16, hi) * kv_row;
      load_row<T, kVec, kDh>(Kh + off, kq, d, kf[b]);
      load_row<T, kVec, kDh>(Vh + off, kq, d, vf[b]);
    };
    auto key_cols = [&](int b, int v) {
      load_cols<T, kVec, kDh>(Kh + (size_t)min(j0 + 16 * b + 4 * kq + v, hi) * kv_row, l16, d, kc[b][v]);
    };
    if constexpr (Ahead<kDh>::value) {
#pragma unroll
      for (int b = 0; b < 2; ++b) rows(b);
#pragma unroll
      for (int b = 0; b < (kLateCols<kVec, kDh> ? 1 : 2); ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) key_cols(b, v);
    }
    loads_first<kDh>();
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if constexpr (!Ahead<kDh>::value) rows(b);
      s[b] = row_product<kDh>(kf[b], qf);
      const f32x4 dp = grad_product<kDh>(vf[b], gf, f32x4{dl, dl, dl, dl});
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int j = j0 + 16 * b + 4 * kq + v;
        const float p = prob(s[b][v], scale, lse);
        s[b][v] = (j < ss_i || j > i_abs) ? 0.f : p * (kLessD<kDh> ? dp[v] : dp[v] - dl);
      }
    }
    if constexpr (kLateCols<kVec, kDh>) {
#pragma unroll
      for (int v = 0; v < 4; ++v) key_cols(1, v);
      loads_first<kDh>();
    }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if constexpr (!Ahead<kDh>::value) key_cols(b, v);
        if (mixed) probe_finite<kDh>(z, kc[b][v]);
        add_outer<kDh>(acc, kc[b][v], s[b][v]);
      }
  }
  float f[kWaves];
#pragma unroll
  for (int w = 0; w < kWaves; ++w) f[w] = scale;
  auto redo = [&](float *sums) {
    clear_sums<kDh>(sums);
    for (int j0 = lo + kStep * wave; j0 <= hi; j0 += kStep * kWaves)
      for (int j = j0; j <= min(j0 + kStep - 1, hi); ++j) {
        const T *Kj = Kh + (size_t)j * kv_row;
        const float s = dot_token(Q + q_off, Kj, kq, d), dp = dot_token(dO + q_off, Vh + (size_t)j * kv_row, kq, d) - dl;
        if (j < ss_i || j > i_abs) continue;
        add_token<T, kDh>(sums, Kj, kq, d, 1.f, prob(s, scale, lse) * dp);
      }
  };
  merge_store<kVec, kDh>(acc, f, red, dQ, gdt, q_off, i_abs <= hi, d, met_not_finite(z), redo);
}

// dK, dV of 16 keys: the waves share out the (query head of the group, 32-query block) pairs.  With few tiles
// the pairs are also shared out over `parts` workgroups per tile: each then stores its sums as fp32 to
// partial[part] ([2][N, Hkv, d]), and f32_add_parts_kernel adds them in the order of the parts.
template <typename T, bool kVec, int kDh, bool kTwo>
__global__ void __launch_bounds__(64 * kWaves, kTwo ? 2 : 1)
f32_dkdv_kernel(const T *__restrict__ dO, const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V,
                const float *__restrict__ LSE, const float *__restrict__ delta, void *__restrict__ dK, void *__restrict__ dV,
                const int32_t *__restrict__ seg_end, float *__restrict__ partial, int parts, int N, int hq, int hkv, int d, va_dtype gdt,
                float scale) {
  __shared__ float red[kWaves * (kDh / 4) * 64];
  const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6), l16 = lane & 15, kq = lane >> 4;
  const int part = blockIdx.y;
  const int g = blockIdx.x % hkv, G = hq / hkv, t0 = (int)(blockIdx.x / hkv) * kRows;
  const int t_last = min(t0 + kRows, N) - 1, j_abs = t0 + l16, j_ld = min(j_abs, t_last);
  const int end = uniform(seg_end[t_last]);
  const int se_j = j_abs <= t_last ? seg_end[j_ld] : 0;  // queries j_abs <= i < se_j see key j_abs
  const size_t q_row = (size_t)hq * d, kv_off = ((size_t)j_ld * hkv + g) * d;
  float kf[kDh / 4], vf[kDh / 4];
  load_row<T, kVec, kDh>(K + kv_off, kq, d, kf);
  load_row<T, kVec, kDh>(V + kv_off, kq, d, vf);
  f32x4 acc_k[Cols<kDh>::kGroups][Cols<kDh>::kE], acc_v[Cols<kDh>::kGroups][Cols<kDh>::kE];
  clear<kDh>(acc_k);
  clear<kDh>(acc_v);
  const int nb = (end - t0 + kStep - 1) / kStep;
  float z = 0.f;
  for (int it = part * kWaves + wave; it < nb * G; it += kWaves * parts) {
    const int h = g * G + it / nb, i0 = t0 + it % nb * kStep;
    const T *Qh = Q + (size_t)h * d, *Gh = dO + (size_t)h * d;
    const float *Lh = LSE + (size_t)h * N, *Dh = delta + (size_t)h * N;
    const bool mixed = __any(i0 < j_abs || i0 + kStep > se_j);  // some key of the tile is not seen by all of the block
    f32x4 p[2], ds[2];
    float qf[2][kDh / 4], gf[2][kDh / 4], lse[2][4], dl[2][4];
    float qc[2][4][Cols<kDh>::kGroups][Cols<kDh>::kE], gc[2][4][Cols<kDh>::kGroups][Cols<kDh>::kE];
    auto rows = [&](int b) {
      const size_t off = (size_t)min(i0 + 16 * b + l16, end - 1) * q_row;
      load_row<T, kVec, kDh>(Qh + off, kq, d, qf[b]);
      load_row<T, kVec, kDh>(Gh + off, kq, d, gf[b]);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = min(i0 + 16 * b + 4 * kq + v, end - 1);
        lse[b][v] = Lh[i];
        dl[b][v] = Dh[i];
      }
    };
    auto query_cols = [&](int b, int v) {
      const size_t off = (size_t)min(i0 + 16 * b + 4 * kq + v, end - 1) * q_row;
      load_cols<T, kVec, kDh>(Gh + off, l16, d, gc[b][v]);
      load_cols<T, kVec, kDh>(Qh + off, l16, d, qc[b][v]);
    };
    if constexpr (Ahead<kDh>::value) {
#pragma unroll
      for (int b = 0; b < 2; ++b) rows(b);
#pragma unroll
      for (int b = 0; b < (kTwo ? 1 : 2); ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) query_cols(b, v);
    }
    loads_first<kDh>();
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if constexpr (!Ahead<kDh>::value) rows(b);
      const f32x4 s = row_product<kDh>(qf[b], kf), dp = grad_product<kDh>(gf[b], vf, f32x4{dl[b][0], dl[b][1], dl[b][2], dl[b][3]});
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = i0 + 16 * b + 4 * kq + v;
        const bool masked = i < j_abs || i >= se_j;
        p[b][v] = masked ? 0.f : prob(s[v], scale, lse[b][v]);
        ds[b][v] = masked ? 0.f : p[b][v] * (kLessD<kDh> ? dp[v] : dp[v] - dl[b][v]);
      }
    }
    if constexpr (kTwo) {
#pragma unroll
      for (int v = 0; v < 4; ++v) query_cols(1, v);
      loads_first<kDh>();
    }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if constexpr (!Ahead<kDh>::value) query_cols(b, v);
        if (mixed) {
          probe_finite<kDh>(z, gc[b][v]);
          probe_finite<kDh>(z, qc[b][v]);
        }
        add_outer<kDh>(acc_v, gc[b][v], p[b][v]);
        add_outer<kDh>(acc_k, qc[b][v], ds[b][v]);
      }
  }
  if (parts > 1) {
    const size_t n = (size_t)N * hkv * d;
    dV = partial + (size_t)part * 2 * n;
    dK = partial + (size_t)part * 2 * n + n;
    gdt = VA_F32;
  }
  float f[kWaves];
#pragma unroll
  for (int w = 0; w < kWaves; ++w) f[w] = 1.f;
  const bool redone = met_not_finite(z);
  auto redo = [&](float *sums, bool keys) {
    clear_sums<kDh>(sums);
    for (int it = part * kWaves + wave; it < nb * G; it += kWaves * parts) {
      const int h = g * G + it / nb, i0 = t0 + it % nb * kStep;
      for (int i = i0; i < min(i0 + kStep, end); ++i) {
        const T *Qi = Q + (size_t)i * q_row + (size_t)h * d, *Gi = dO + (size_t)i * q_row + (size_t)h * d;
        const float s = dot_token(K + kv_off, Qi, kq, d);
        const float dp = dot_token(V + kv_off, Gi, kq, d) - delta[(size_t)h * N + i];
        if (i < j_abs || i >= se_j) continue;
        const float p = prob(s, scale, LSE[(size_t)h * N + i]);
        add_token<T, kDh>(sums, keys ? Qi : Gi, kq, d, 1.f, keys ? p * dp : p);
      }
    }
  };
  merge_store<kVec, kDh>(acc_v, f, red, dV, gdt, kv_off, j_abs <= t_last, d, redone, [&](float *sums) { redo(sums, false); });
#pragma unroll
  for (int w = 0; w < kWaves; ++w) f[w] = scale;
  merge_store<kVec, kDh>(acc_k, f, red, dK, gdt, kv_off, j_abs <= t_last, d, redone, [&](float *sums) { redo(sums, true); });
}

__global__ void __launch_bounds__(256)
f32_add_parts_kernel(const float *__restrict__ partial, int parts, size_t n, void *__restrict__ dK, void *__restrict__ dV, va_dtype gdt) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= 2 * n) return;
  float x = 0.f;
  for (int p = 0; p < parts; ++p) x += partial[(size_t)p * 2 * n + i];
  if (i < n) put(dV, gdt, i, x);
  else put(dK, gdt, i - n, x);
}

// ---- D on its own --------------------------------------------------------------------------------

// delta[h, i] = sum_c dO[i,h,c] * O[i,h,c]; one wave per (i, h)
template <typename T>
__global__ void __launch_bounds__(256)
delta_kernel(const T *__restrict__ dO, const T *__restrict__ O, float *__restrict__ delta, int N,
             int hq, int d) {
  const int lane = threadIdx.x & 63;
  const long long unit = (long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (unit >= (long long)N * hq) return;
  const int i = (int)(unit / hq), h = (int)(unit % hq);
  float part = 0.f;
  for (int c = lane; c < d; c += 64) {
    const size_t x = ((size_t)i * hq + h) * d + c;
    part += (float)dO[x] * (float)O[x];
  }
  for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
  if (lane == 0) delta[(size_t)h * N + i] = part;
}

// D for the 16-bit types with head_dim a multiple of 8 up to 128: 16 lanes per (token, head) row,
// 16 B of dO and of O per lane; a block handles 64 consecutive tokens of one head, so the [Hq, N]
// result is written 64 B at a time.
template <class E>
__global__ void __launch_bounds__(256)
delta_16bit_kernel(const uint16_t *__restrict__ dO, const uint16_t *__restrict__ O,
                   float *__restrict__ delta, int N, int hq, int d) {
  const int h = blockIdx.y, c = threadIdx.x & 15, ti = threadIdx.x >> 4;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int i = blockIdx.x * 64 + it * 16 + ti;
    float part = 0.f;
    if (i < N && c * 8 < d) {
      const size_t x = ((size_t)i * hq + h) * d + c * 8;
      const typename E::x8 a = as_x8<E>(*(const u32x4 *)(dO + x)), b = as_x8<E>(*(const u32x4 *)(O + x));
#pragma unroll
      for (int e = 0; e < 8; ++e) part += (float)a[e] * (float)b[e];
    }
    for (int o = 8; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
    if (c == 0 && i < N) delta[(size_t)h * N + i] = part;
  }
}

// ---- launches --------------------------------------------------------------------------------------

struct Args {  // one call's tensors and sizes; unused ones stay null
  const void *Q, *K, *V, *O, *dO;
  void *out, *dK, *dV;
  float *LSE, *delta;
  const va_segments *seg;
  int N, T, hq, hkv, d;
  va_dtype out_dt;
  float scale;
  hipStream_t stream;
  unsigned stages;
  Partials partial;
};

template <typename T, bool kVec, int kDh> hipError_t run_fwd(const Args &a) {
  const long long grid = (long long)ceil_div(a.N, kRows) * a.hq;
  if (grid > 0x7fffffffll) return hipErrorInvalidValue;
  f32_fwd_kernel<T, kVec, kDh><<<(unsigned)grid, 64 * kWaves, 0, a.stream>>>(
      (const T *)a.Q, (const T *)a.K, (const T *)a.V, a.out, a.LSE, a.seg->seg_start, a.N, a.hq, a.hkv, a.d, a.out_dt,
      a.scale * 1.4426950408889634f, a.scale);
  return hipGetLastError();
}
// Parts that the work of a dK/dV tile is shared out to: enough workgroups for two per CU, but at least two rounds of the
// waves in the longest chain that a row of T tokens allows.  More parts help long chains (1000 tokens in examples of up to 676,
// 8/2 heads of 64: six instead of four -5 us) and cost short ones, which the host cannot tell apart (1788 tokens in examples of
// up to 28, 4/2 heads: four instead of two +9 us; 2374 of up to 17, 16/4 heads: two instead of one +10).
long long dkdv_parts(int N, int T, int hq, int hkv) {
  const long long units = (N + kRows - 1ll) / kRows * hkv, rounds = (T + kStep - 1ll) / kStep * (hq / hkv) / kWaves;
  return std::max(1ll, std::min(512 / units, rounds / 2));
}
template <typename T, bool kVec, int kDh> hipError_t run_bwd(const Args &a) {
  const long long gq = (long long)ceil_div(a.N, kRows) * a.hq, gkv = (long long)ceil_div(a.N, kRows) * a.hkv;
  if (gq > 0x7fffffffll) return hipErrorInvalidValue;
  if (a.stages & VA_STAGE_DQ)
    f32_dq_kernel<T, kVec, kDh><<<(unsigned)gq, 64 * kWaves, 0, a.stream>>>(
        (const T *)a.dO, (const T *)a.Q, (const T *)a.K, (const T *)a.V, (const T *)a.O, a.LSE, a.delta, a.out,
        a.seg->seg_start, a.N, a.hq, a.hkv, a.d, a.out_dt, a.scale);
  if (a.stages & VA_STAGE_DKDV) {
    const size_t n = (size_t)a.N * a.hkv * a.d;
    const long long parts = std::max(1ll, std::min(dkdv_parts(a.N, a.T, a.hq, a.hkv), (long long)(a.partial.bytes / 8 / n)));
    auto launch = [&](auto *kernel) {
      kernel<<<dim3((unsigned)gkv, (unsigned)parts), 64 * kWaves, 0, a.stream>>>(
          (const T *)a.dO, (const T *)a.Q, (const T *)a.K, (const T *)a.V, a.LSE, a.delta, a.dK, a.dV, a.seg->seg_end,
          a.partial.p, (int)parts, a.N, a.hq, a.hkv, a.d, a.out_dt, a.scale);
    };
    constexpr int kFrom = kTwoPerCuFrom<kVec, kDh>;
    const bool two = kFrom > 0 && gkv >= (a.hq < (kDh <= 32 ? 2 : 4) * a.hkv ? kFrom : 2 * kFrom);
    launch(two ? f32_dkdv_kernel<T, kVec, kDh, (kFrom > 0)> : f32_dkdv_kernel<T, kVec, kDh, false>);
    if (parts > 1)
      f32_add_parts_kernel<<<(unsigned)((2 * n + 255) / 256), 256, 0, a.stream>>>(a.partial.p, (int)parts, n, a.dK, a.dV, a.out_dt);
  }
  return hipGetLastError();
}

// fp32 with d a multiple of 4 and 16-byte aligned tensors loads 16 bytes at a time, unrolled for head dims up to 16, 32,
// 64, 128 and 256; everything else loads element by element and shares the larger three.
template <bool kFwd, typename T, bool kVec> hipError_t by_head_dim(const Args &a) {
  if constexpr (kVec) {
    if (a.d <= 16) { if constexpr (kFwd) return run_fwd<T, kVec, 16>(a); else return run_bwd<T, kVec, 16>(a); }
    if (a.d <= 32) { if constexpr (kFwd) return run_fwd<T, kVec, 32>(a); else return run_bwd<T, kVec, 32>(a); }
  }
  if (a.d <= 64) { if constexpr (kFwd) return run_fwd<T, kVec, 64>(a); else return run_bwd<T, kVec, 64>(a); }
  if (a.d <= 128) { if constexpr (kFwd) return run_fwd<T, kVec, 128>(a); else return run_bwd<T, kVec, 128>(a); }
  if constexpr (kFwd) return run_fwd<T, kVec, 256>(a); else return run_bwd<T, kVec, 256>(a);
}
template <bool kFwd> hipError_t by_type(va_dtype dt, const Args &a) {
  if (dt == VA_BF16) return by_head_dim<kFwd, __bf16, false>(a);
  if (dt == VA_F16) return by_head_dim<kFwd, _Float16, false>(a);
  const uintptr_t bits = (uintptr_t)a.Q | (uintptr_t)a.K | (uintptr_t)a.V | (uintptr_t)a.O | (uintptr_t)a.dO |
                         (uintptr_t)a.out | (uintptr_t)a.dK | (uintptr_t)a.dV;
  return a.d % 4 == 0 && bits % 16 == 0 ? by_head_dim<kFwd, float, true>(a) : by_head_dim<kFwd, float, false>(a);
}

}  // namespace

size_t f32_partial_bytes(int N, int hq, int hkv, int d) {
  const long long parts = dkdv_parts(N, N, hq, hkv);  // one row: the longest chains
  return parts > 1 ? (size_t)parts * 8 * N * hkv * d : 0;
}

hipError_t launch_f32_fwd(const void *Q, const void *K, const void *V, void *O, float *LSE,
                          const va_segments &seg, int N, int hq, int hkv, int d, va_dtype dt,
                          float scale, hipStream_t stream) {
  Args a = {Q, K, V, nullptr, nullptr, O, nullptr, nullptr, LSE, nullptr, &seg, N, 0, hq, hkv, d, dt, scale, stream, 0, {nullptr, 0}};
  return by_type<true>(dt, a);
}

hipError_t launch_f32_bwd(const void *dO, const void *Q, const void *K, const void *V, const void *O,
                          const float *LSE, float *delta, void *dQ, void *dK, void *dV, va_dtype grad_dt,
                          const va_segments &seg, int rows, int T, int hq, int hkv, int d, va_dtype dt, float scale,
                          const Partials &partial, hipStream_t stream, unsigned stages) {
  Args a = {Q, K, V, O, dO, dQ, dK, dV, const_cast<float *>(LSE), delta, &seg, rows * T, T, hq, hkv, d, grad_dt, scale,
            stream, stages, partial};
  return by_type<false>(dt, a);
}

hipError_t launch_delta(const void *dO, const void *O, float *delta, int N, int hq, int d,
                        va_dtype dt, hipStream_t stream) {
  if (dt != VA_F32 && d <= 128 && d % 8 == 0) {
    const dim3 grid((unsigned)((N + 63) / 64), (unsigned)hq);
    if (dt == VA_F16)
      delta_16bit_kernel<F16><<<grid, 256, 0, stream>>>((const uint16_t *)dO, (const uint16_t *)O, delta, N, hq, d);
    else
      delta_16bit_kernel<Bf16><<<grid, 256, 0, stream>>>((const uint16_t *)dO, (const uint16_t *)O, delta, N, hq, d);
    return hipGetLastError();
  }
  const unsigned nb = (unsigned)(((long long)N * hq + 3) / 4);
  if (dt == VA_F16)
    delta_kernel<_Float16><<<nb, 256, 0, stream>>>((const _Float16 *)dO, (const _Float16 *)O, delta, N, hq, d);
  else if (dt == VA_F32)
    delta_kernel<float><<<nb, 256, 0, stream>>>((const float *)dO, (const float *)O, delta, N, hq, d);
  else
    delta_kernel<__bf16><<<nb, 256, 0, stream>>>((const __bf16 *)dO, (const __bf16 *)O, delta, N, hq, d);
  return hipGetLastError();
}

}  // namespace va
