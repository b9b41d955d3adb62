// Rotary position embedding driven by the packed stream's position ids (paper, Section 3: a
// model that takes position ids encodes a packed example exactly as if it were alone, because
// the ids restart at 0).  "Rotate-half" pairing: pair c = (x[c], x[c + d/2]) of a head vector
// turns by the angle pos * base^(-2c/d); `inverse` turns by the negative angle (the transpose,
// used for gradients).  HBM-bound: every element is read and written once; the sines and
// cosines of a (token, pair) are computed once and shared by all heads.
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
constexpr int kMinGroups = 512;  // fewer tokens per workgroup rather than fewer than two workgroups per CU

template <typename T, int kVec, typename IdT>
__global__ void __launch_bounds__(kThreads)
rope_kernel(const T *x, T *y, const IdT *__restrict__ pos, long long N, int tokens,  // y may be x (in place)
            size_t token_elems, int H, int d, double neg2_log2base_over_d, int inverse) {
  typedef Chunk<T, kVec> C;
  typedef typename C::type chunk_t;
  __shared__ __attribute__((aligned(16))) float cs[kMaxPairs], sn[kMaxPairs];
  const int hd = d / 2, cpt = hd / kVec;
  const long long t0 = (long long)blockIdx.x * tokens;
  const int nt = (int)min((long long)tokens, N - t0);
  const int n_items = nt * H * cpt;
  for (int e = threadIdx.x; e < nt * hd; e += kThreads) {
    const int t = e / hd, c = e - t * hd;
    // angle in fp64, reduced to [-pi, pi] before the fp32 sine / cosine: exact to ~1e-7 at any position
    double w = (double)pos[t0 + t] * exp2((double)c * neg2_log2base_over_d);
    w -= 6.283185307179586476925 * rint(w * 0.15915494309189533577);
    float s1, c1;
    sincosf((float)w, &s1, &c1);
    cs[e] = c1;
    sn[e] = inverse ? -s1 : s1;
  }
  __syncthreads();
  const T *const xb = x + (size_t)t0 * token_elems;
  T *const yb = y + (size_t)t0 * token_elems;
  for (int i0 = threadIdx.x; i0 < n_items; i0 += kItems * kThreads) {
    chunk_t a[kItems], b[kItems];
    size_t off[kItems];
    int e0[kItems];
#pragma unroll
    for (int u = 0; u < kItems; ++u) {  // the last items of a workgroup are loaded more than once, stored once
      const int i = min(i0 + u * kThreads, n_items - 1);
      const int row = i / cpt, c0 = (i - row * cpt) * kVec;
      const int t = row / H;
      off[u] = (size_t)t * token_elems + (size_t)(row - t * H) * d + c0;
      e0[u] = t * hd + c0;
      a[u] = *(const chunk_t *)(xb + off[u]);
      b[u] = *(const chunk_t *)(xb + off[u] + hd);
    }
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
      if (i0 + u * kThreads >= n_items) break;
      chunk_t ra, rb;
#pragma unroll
      for (int e = 0; e < kVec; ++e) {
        const float x1 = C::get(a[u], e), x2 = C::get(b[u], e), c1 = cs[e0[u] + e], s1 = sn[e0[u] + e];
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
  const int h_most = (1 << 24) / cpt;  // heads of one launch: a workgroup counts its items in 32 bits
  for (int h0 = 0; h0 < H; h0 += h_most) {
    const int h = H - h0 < h_most ? H - h0 : h_most;
    long long tokens = kItems * kThreads / ((long long)h * cpt);
    if (tokens > kMaxPairs / hd) tokens = kMaxPairs / hd;
    while (tokens > 1 && N / tokens < kMinGroups) tokens /= 2;
    if (tokens < 1) tokens = 1;
    const long long grid = (N + tokens - 1) / tokens;
    if (grid > 0x7fffffffll) return hipErrorInvalidValue;
    rope_kernel<T, kVec, IdT><<<(unsigned)grid, kThreads, 0, stream>>>(
        (const T *)x + (size_t)h0 * d, (T *)y + (size_t)h0 * d, (const IdT *)pos, N, (int)tokens, (size_t)H * d, h, d,
        -2.0 * log2(base) / (double)d, inverse);
  }
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
