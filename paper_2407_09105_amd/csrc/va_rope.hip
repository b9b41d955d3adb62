// Rotary position embedding driven by the packed stream's position ids (paper, Section 3: a
// model that takes position ids encodes a packed example exactly as if it were alone, because
// the ids restart at 0).  "Rotate-half" pairing: pair c = (x[c], x[c + d/2]) of a head vector
// turns by the angle pos * base^(-2c/d); `inverse` turns by the negative angle (the transpose,
// used for gradients).  HBM-bound: every element is read and written once; the sines and
// cosines of a (token, pair) are computed once and shared by all heads.
#include <algorithm>

#include "va_internal.h"
#include "va_mfma_common.h"

namespace va {
namespace {

// A chunk of kVec consecutive elements of type T (float, __bf16 or _Float16), 16 bytes when wide.
template <typename T, int kVec> struct Chunk {
  typedef T type __attribute__((ext_vector_type(kVec)));
  static __device__ __forceinline__ float get(const type &v, int e) { return (float)v[e]; }
  static __device__ __forceinline__ void set(type &v, int e, float x) { v[e] = (T)x; }  // round to nearest even
};
template <typename T> struct Chunk<T, 1> {
  typedef T type;
  static __device__ __forceinline__ float get(const type &v, int) { return (float)v; }
  static __device__ __forceinline__ void set(type &v, int, float x) { v = (T)x; }
};

// A workgroup takes `tokens` consecutive tokens with all their heads: it forms the cosines and sines of
// its tokens once, in LDS, and then streams their rows - one contiguous piece of memory - in items of one
// chunk of kVec pairs, kItems items of a thread in flight together.
// Bound: HBM, every element read and written once.  Measured (bf16, read + written bytes over time): 69632
// tokens, 32 heads, d = 128: 205 us, 5.6 TB/s; d = 80: 133 us, 5.4 TB/s.  One thread per (token, chunk) that
// walked the heads took 238 and 262 us: its accesses jumped by whole token rows, shared cache lines with
// other workgroups where a head is no multiple of 128 bytes, and every thread formed 8 sines by itself.
// Two or eight items in flight: within 5 %; non-temporal stores: 3 % faster alone, 3...25 % slower together
// with the next reader of y.
constexpr int kThreads = 256;
constexpr int kItems = 4;
constexpr int kMaxPairs = 2048;  // (token, pair) entries of the table: 16 KB
constexpr long long kMinGroups = 512;  // fewer tokens per workgroup rather than fewer than two workgroups per CU,
constexpr int kLeastItems = 64;        // but a wave's worth of items (1000 tokens, one head of 64: 3.1 us, down to one token 4.6)

__device__ __forceinline__ void cos_sin(double pos, int c, double neg2_log2base_over_d, int inverse, float &cs, float &sn) {
  // angle in fp64, reduced to [-pi, pi] before the fp32 sine / cosine: exact to ~1e-7 at any position
  double w = pos * exp2((double)c * neg2_log2base_over_d);
  w -= 6.283185307179586476925 * rint(w * 0.15915494309189533577);
  sincosf((float)w, &sn, &cs);
  if (inverse) sn = -sn;
}

// kDirect: one head, whose table would share nothing; every thread forms the cosines and sines of its only item itself.
template <typename T, int kVec, typename IdT, bool kDirect>
__global__ void __launch_bounds__(kThreads)
rope_kernel(const T *x, T *y, const IdT *__restrict__ pos, long long N, int tokens,  // y may be x (in place)
            int H, int heads, int d, double neg2_log2base_over_d, int inverse) {
  typedef Chunk<T, kVec> C;
  typedef typename C::type chunk_t;
  constexpr int kFly = kDirect ? 1 : kItems, kTable = kDirect ? 1 : kMaxPairs;
  __shared__ __attribute__((aligned(16))) float cs[kTable], sn[kTable];
  const int hd = d / 2, cpt = hd / kVec;
  const long long t0 = (long long)blockIdx.x * tokens;
  const int nt = (int)min((long long)tokens, N - t0);
  const int h0 = blockIdx.y * heads, nh = min(heads, H - h0);
  const size_t token_elems = (size_t)H * d;
  const int n_items = nt * nh * cpt;
  if constexpr (!kDirect) {
    for (int e = threadIdx.x; e < nt * hd; e += kThreads) {
      const int t = e / hd;
      cos_sin((double)pos[t0 + t], e - t * hd, neg2_log2base_over_d, inverse, cs[e], sn[e]);
    }
    __syncthreads();
  }
  const T *const xb = x + (size_t)t0 * token_elems + (size_t)h0 * d;
  T *const yb = y + (size_t)t0 * token_elems + (size_t)h0 * d;
  for (int i0 = threadIdx.x; i0 < n_items; i0 += kFly * kThreads) {
    chunk_t a[kFly], b[kFly];
    size_t off[kFly];
    int e0[kFly];
#pragma unroll
    for (int u = 0; u < kFly; ++u) {  // the last items of a workgroup are loaded more than once, stored once
      const int i = min(i0 + u * kThreads, n_items - 1);
      const int row = i / cpt, c0 = (i - row * cpt) * kVec;
      const int t = kDirect ? row : row / nh;
      off[u] = (size_t)t * token_elems + (size_t)(row - t * nh) * d + c0;
      e0[u] = t * hd + c0;
      a[u] = *(const chunk_t *)(xb + off[u]);
      b[u] = *(const chunk_t *)(xb + off[u] + hd);
    }
#pragma unroll
    for (int u = 0; u < kFly; ++u) {
      if (i0 + u * kThreads >= n_items) break;
      chunk_t ra, rb;
#pragma unroll
      for (int e = 0; e < kVec; ++e) {
        const float x1 = C::get(a[u], e), x2 = C::get(b[u], e);
        float c1, s1;
        if constexpr (kDirect) {
          cos_sin((double)pos[t0 + i0 / cpt], i0 % cpt * kVec + e, neg2_log2base_over_d, inverse, c1, s1);
        } else {
          c1 = cs[e0[u] + e];
          s1 = sn[e0[u] + e];
        }
        C::set(ra, e, x1 * c1 - x2 * s1);
        C::set(rb, e, x2 * c1 + x1 * s1);
      }
      *(chunk_t *)(yb + off[u]) = ra;
      *(chunk_t *)(yb + off[u] + hd) = rb;
    }
  }
}

template <typename T, int kVec, typename IdT>
hipError_t launch(const void *x, void *y, const void *pos, long long N, int H, int d, double base,
                  int inverse, hipStream_t stream) {
  if (N == 0) return hipSuccess;
  const int hd = d / 2, cpt = hd / kVec;
  const long long per_token = (long long)H * cpt;  // items
  // One head and a workgroup of single items per CU: 65536 tokens of 128 12.2 us (with a table 17), 20000 of 64
  // 4.7 (5.7), but 12000 of 64 4.1 (3.9): fewer leave the chip waiting for eight sines in a row.
  const bool direct = H == 1 && N * cpt >= 256 * kThreads;
  long long tokens = direct ? kThreads / cpt : std::max(1ll, std::min(kItems * kThreads / per_token, (long long)kMaxPairs / hd));
  while (!direct && tokens > 1 && N / tokens < kMinGroups && tokens * per_token >= 2 * kLeastItems) tokens /= 2;
  const long long groups = (N + tokens - 1) / tokens;
  if (groups > 0x7fffffffll) return hipErrorInvalidValue;
  // Tokens alone are too few to fill the chip, but have more items than a workgroup keeps in flight: heads are split too
  // (16 tokens, 2048 heads of 256: 47 -> 6.6 us).  A workgroup counts its items in 32 bits.
  const long long parts = std::max({std::min((kMinGroups + groups - 1) / groups, per_token / (kItems * kThreads)), per_token >> 24, 1ll});
  const int heads = (int)((H + parts - 1) / parts);
  auto *kernel = direct ? rope_kernel<T, kVec, IdT, true> : rope_kernel<T, kVec, IdT, false>;
  kernel<<<dim3((unsigned)groups, (unsigned)((H + heads - 1) / heads)), kThreads, 0, stream>>>(
      (const T *)x, (T *)y, (const IdT *)pos, N, (int)tokens, H, heads, d, -2.0 * log2(base) / (double)d, inverse);
  return hipGetLastError();
}

template <typename T, int kWide>
hipError_t pick(const void *x, void *y, const void *pos, va_itype it, long long N, int H, int d,
                double base, int inverse, hipStream_t stream) {
  // 16-byte chunks need both halves of every head vector 16-byte aligned
  const bool wide = (d / 2) % kWide == 0 && (((uintptr_t)x | (uintptr_t)y) & 15) == 0;
  if (it == VA_I64)
    return wide ? launch<T, kWide, int64_t>(x, y, pos, N, H, d, base, inverse, stream)
                : launch<T, 1, int64_t>(x, y, pos, N, H, d, base, inverse, stream);
  return wide ? launch<T, kWide, int32_t>(x, y, pos, N, H, d, base, inverse, stream)
              : launch<T, 1, int32_t>(x, y, pos, N, H, d, base, inverse, stream);
}

}  // namespace

hipError_t launch_rope(const void *x, void *y, va_dtype dt, const void *pos, va_itype it, long long N,
                       int H, int d, double base, int inverse, hipStream_t stream) {
  if (dt == VA_BF16) return pick<__bf16, 8>(x, y, pos, it, N, H, d, base, inverse, stream);
  if (dt == VA_F16) return pick<_Float16, 8>(x, y, pos, it, N, H, d, base, inverse, stream);
  return pick<float, 4>(x, y, pos, it, N, H, d, base, inverse, stream);
}

}  // namespace va
