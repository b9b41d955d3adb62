// Device-side padding-free collator (paper, Section 3.4): a minibatch held as a padded
// [n, Lp] batch with per-example lengths becomes one packed row of input_ids, labels (first
// label of every example -> -100) and position_ids (restarting at 0 in every example) --
// the three tensors Section 3.5 prints for its worked example.  Integer work only.
#include "va_internal.h"

namespace va {
namespace {

constexpr int kOffThreads = 1024;

__device__ __forceinline__ int clamp_len(int L, int Lp) { return L < 0 ? 0 : (L > Lp ? Lp : L); }

// offsets[e] = sum of the clamped lengths of examples before e; offsets[n] = total.
// One workgroup walks the lengths in slabs of kOffThreads with a running carry.
__global__ void __launch_bounds__(kOffThreads)
collate_offsets_kernel(const int32_t *__restrict__ lengths, int n, int Lp, int32_t *__restrict__ offsets) {
  __shared__ int32_t wave_sum[kOffThreads / 64];
  __shared__ int32_t carry_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) { carry_s = 0; offsets[0] = 0; }
  __syncthreads();
  for (int base = 0; base < n; base += kOffThreads) {
    const int e = base + tid;
    const int L = e < n ? clamp_len(lengths[e], Lp) : 0;
    int incl = L;  // inclusive scan inside the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int before = carry_s;
    for (int w = 0; w < wave; ++w) before += wave_sum[w];
    if (e < n) offsets[e + 1] = before + incl;
    __syncthreads();
    if (tid == kOffThreads - 1) carry_s = before + incl;
    __syncthreads();
  }
}

// Token t of the output: find its example by bisection over the offsets, then copy.
template <typename IdT>
__device__ __forceinline__ void collate_token(const IdT *__restrict__ ids, const IdT *__restrict__ labels_in,
                                              const int32_t *offsets, int n, int Lp, int t, IdT pad_id,
                                              IdT *__restrict__ input_ids, IdT *__restrict__ labels,
                                              IdT *__restrict__ position_ids) {
  const int total = offsets[n];
  if (t >= total) {  // tail: one pad pseudo-example
    input_ids[t] = pad_id;
    labels[t] = (IdT)-100;
    position_ids[t] = (IdT)(t - total);
    return;
  }
  int lo = 0, hi = n;  // largest e with offsets[e] <= t (empty examples share an offset: take the last)
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (offsets[mid] <= t) lo = mid; else hi = mid;
  }
  const int p = t - offsets[lo];
  const size_t src = (size_t)lo * Lp + p;
  const IdT id = ids[src];
  input_ids[t] = id;
  labels[t] = p == 0 ? (IdT)-100 : (labels_in ? labels_in[src] : id);
  position_ids[t] = (IdT)p;
}

// One thread per output token, the offsets in memory (written by collate_offsets_kernel).
template <typename IdT>
__global__ void __launch_bounds__(256)
collate_tokens_kernel(const IdT *__restrict__ ids, const IdT *__restrict__ labels_in,
                      const int32_t *__restrict__ offsets, int n, int Lp, int n_out, IdT pad_id,
                      IdT *__restrict__ input_ids, IdT *__restrict__ labels, IdT *__restrict__ position_ids) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= n_out) return;
  collate_token(ids, labels_in, offsets, n, Lp, t, pad_id, input_ids, labels, position_ids);
}

// Minibatches of 1 .. kOneMax examples, in one launch: every workgroup sums the lengths into offsets of its own
// in LDS (at most kOneMax ints, read from L2), where the bisection then runs; the first one stores them.
// Bound: launch latency.  1024 examples, 70 thousand tokens: 5.6 us; 4 examples: 4.1 us (offsets and
// tokens in two launches: 10.4 and 5.3 us).  With many examples and many workgroups (of 256 tokens) the sums that
// each repeats cost more than the launch.  One launch / two, us: 2048 examples, 540, 915, 1416, 2120, 8222 workgroups
// 6.3 / 8.6, 7.4 / 8.9, 9.8 / 9.8, 13.5 / 11.5, 37 / 26; 1500, 667, 2079, 4440 5.8 / 8.7, 11.3 / 11.5, 19.2 / 17.3;
// 1024, 3027, 14164 11.9 / 11.9, 37 / 35; 768, 4608 14.7 / 15.6; 512, 14204 28 / 33.
constexpr int kOneMax = 2048, kOneAlways = 512;
constexpr long long kOneWork = 3 << 19;  // examples beyond kOneAlways x workgroups
template <typename IdT>
__global__ void __launch_bounds__(256)
collate_one_kernel(const IdT *__restrict__ ids, const IdT *__restrict__ labels_in, const int32_t *__restrict__ lengths,
                   int n, int Lp, int n_out, IdT pad_id, IdT *__restrict__ input_ids, IdT *__restrict__ labels,
                   IdT *__restrict__ position_ids, int32_t *__restrict__ offsets_out) {
  constexpr int kPer = kOneMax / 256;
  __shared__ int32_t offsets[kOneMax + 1], wave_sum[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int L[kPer], sum = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) L[e] = lengths[min(tid * kPer + e, n - 1)];  // all in flight together
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    L[e] = tid * kPer + e < n ? clamp_len(L[e], Lp) : 0;
    sum += L[e];
  }
  int incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  if (lane == 63) wave_sum[wave] = incl;
  __syncthreads();
  int run = incl - sum;
  for (int w = 0; w < wave; ++w) run += wave_sum[w];
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    offsets[tid * kPer + e] = run;
    run += L[e];
  }
  if (tid == 255) offsets[kOneMax] = run;
  __syncthreads();
  if (blockIdx.x == 0)
    for (int e = tid; e <= n; e += 256) offsets_out[e] = offsets[e];
  const int t = blockIdx.x * 256 + tid;
  if (t < n_out) collate_token(ids, labels_in, offsets, n, Lp, t, pad_id, input_ids, labels, position_ids);
}

}  // namespace

hipError_t launch_collate(const void *ids, const void *labels_in, va_itype it, const int32_t *lengths,
                          int n, int Lp, int n_out, long long pad_id, void *input_ids, void *labels,
                          void *position_ids, int32_t *offsets, hipStream_t stream) {
  const unsigned grid = (unsigned)(n_out > 0 ? ceil_div(n_out, 256) : 1);
  const bool one = n >= 1 && n <= kOneMax && (n - kOneAlways) * (long long)grid <= kOneWork;
  if (!one) {
    collate_offsets_kernel<<<1, kOffThreads, 0, stream>>>(lengths, n, Lp, offsets);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n_out == 0) return e;
  }
  auto tokens = [&](auto pad) {
    typedef decltype(pad) IdT;
    if (one)
      collate_one_kernel<IdT><<<grid, 256, 0, stream>>>((const IdT *)ids, (const IdT *)labels_in, lengths, n, Lp, n_out, pad,
                                                        (IdT *)input_ids, (IdT *)labels, (IdT *)position_ids, offsets);
    else
      collate_tokens_kernel<IdT><<<grid, 256, 0, stream>>>((const IdT *)ids, (const IdT *)labels_in, offsets, n, Lp, n_out,
                                                           pad, (IdT *)input_ids, (IdT *)labels, (IdT *)position_ids);
  };
  if (it == VA_I64) tokens((int64_t)pad_id);
  else tokens((int32_t)pad_id);
  return hipGetLastError();
}

}  // namespace va
