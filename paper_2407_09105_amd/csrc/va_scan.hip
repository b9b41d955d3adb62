// Boundary scan: position_ids -> cu_seqlens, per-token example ids / bounds, tile schedule.
//
// Paper, Section 3: the attention wrapper gets position_ids and derives cu_seq_len from
// them; Section 3.1: ids restart at 0 at each example.  A token starts an example iff it
// is the first of its row or its id is 0.  Integer work only, exact.
//
// Streams of up to 8192 tokens: one launch (pack_single_kernel).  Longer ones: three, over chunks of
// kScanChunk tokens, without any waiting between workgroups:
//   1. per-chunk aggregates: number of starts, last start, first start
//   2. per-chunk final scan, its carries taken from the aggregates -> seg_id, seg_start, seg_end,
//      cu_seqlens, max_seqlen, and a sort key per schedule tile
//   3. the tile order: a rank sort of the keys (heaviest first)
// Bound: launch latency (4 to 6 us each, less when they follow each other closely).  65536 tokens in 256 tiles:
// 15.9 us; 16384 tokens in 64: 12.5 us (with the carries in a launch of their own and each workgroup of the
// ranking making the keys of all tiles: 26.3 and 15.7 us).
#include <type_traits>

#include "va_internal.h"

namespace va {
namespace {

constexpr int kPerThread = kScanChunk / kScanThreads;  // 8 consecutive tokens per thread

// Start flags of the kPerThread consecutive tokens from `base`.  The ids are loaded
// unconditionally (index clamped into the stream) before any of them is looked at: loads under a
// condition would be issued one at a time, each waiting for the one before.
template <typename IdT>
__device__ __forceinline__ void start_flags(const IdT *pos, int base, int N, int T, bool (&flag)[kPerThread]) {
  IdT id[kPerThread];
#pragma unroll
  for (int e = 0; e < kPerThread; ++e) id[e] = pos[min(base + e, N - 1)];
  int r = base % T;  // position inside the packed row, advanced without further divisions
#pragma unroll
  for (int e = 0; e < kPerThread; ++e) {
    flag[e] = base + e < N && (id[e] == 0 || r == 0);
    if (++r == T) r = 0;
  }
}

// ---- block-wide scans over kScanThreads values (LDS, Hillis-Steele per wave + wave carries) ----

__device__ __forceinline__ int wave_incl_add(int x) {
  const int lane = threadIdx.x & 63;
  for (int o = 1; o < 64; o <<= 1) {
    int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}
__device__ __forceinline__ int wave_incl_max(int x) {
  const int lane = threadIdx.x & 63;
  for (int o = 1; o < 64; o <<= 1) {
    int y = __shfl_up(x, o, 64);
    if (lane >= o) x = max(x, y);
  }
  return x;
}
// suffix (right-to-left) inclusive min
__device__ __forceinline__ int wave_suffix_min(int x) {
  const int lane = threadIdx.x & 63;
  for (int o = 1; o < 64; o <<= 1) {
    int y = __shfl_down(x, o, 64);
    if (lane + o < 64) x = min(x, y);
  }
  return x;
}

struct ChunkAgg { int count, last, first; };

// pass 1 (of more than 8192 tokens)
template <typename IdT>
__global__ void __launch_bounds__(kScanThreads)
scan_aggregate_kernel(const IdT *__restrict__ pos, int N, int T, int32_t *__restrict__ agg, int32_t *__restrict__ meta) {
  __shared__ int s_cnt[kScanThreads / 64], s_last[kScanThreads / 64], s_first[kScanThreads / 64];
  const int base = blockIdx.x * kScanChunk + threadIdx.x * kPerThread;
  bool flag[kPerThread];
  start_flags(pos, base, N, T, flag);
  int cnt = 0, last = -1, first = N;
#pragma unroll
  for (int e = 0; e < kPerThread; ++e) {
    const int t = base + e;
    if (flag[e]) {
      ++cnt;
      last = t;
      first = min(first, t);
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    cnt += __shfl_xor(cnt, o, 64);
    last = max(last, __shfl_xor(last, o, 64));
    first = min(first, __shfl_xor(first, o, 64));
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { s_cnt[w] = cnt; s_last[w] = last; s_first[w] = first; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < kScanThreads / 64; ++i) {
      cnt += s_cnt[i]; last = max(last, s_last[i]); first = min(first, s_first[i]);
    }
    agg[3 * blockIdx.x + 0] = cnt;
    agg[3 * blockIdx.x + 1] = last;
    agg[3 * blockIdx.x + 2] = first;
  }
  // meta[1] (max_seqlen) and meta[2] (64-query blocks over all key tiles) are accumulated by the last pass
  if (blockIdx.x == 0 && threadIdx.x < 8) meta[threadIdx.x] = 0;
}

// only for streams of more than kFoldedCarryChunks chunks: carries[3*b] = starts before chunk b,
// [3*b+1] = last start before it, [3*b+2] = first start after it (N if none).
__global__ void __launch_bounds__(64)
scan_carry_kernel(const int32_t *__restrict__ agg, int nchunks, int N, int32_t *__restrict__ carry) {
  const int lane = threadIdx.x;
  int run_cnt = 0, run_last = -1;
  for (int b0 = 0; b0 < nchunks; b0 += 64) {
    const int b = b0 + lane;
    int c = 0, l = -1;
    if (b < nchunks) { c = agg[3 * b]; l = agg[3 * b + 1]; }
    const int ic = wave_incl_add(c);
    const int il = wave_incl_max(l);
    int ec = __shfl_up(ic, 1, 64), el = __shfl_up(il, 1, 64);
    if (lane == 0) { ec = 0; el = -1; }
    if (b < nchunks) {
      carry[3 * b] = run_cnt + ec;
      carry[3 * b + 1] = max(run_last, el);
    }
    run_cnt += __shfl(ic, 63, 64);
    run_last = max(run_last, __shfl(il, 63, 64));
  }
  int run_first = N;
  for (int b0 = ((nchunks - 1) / 64) * 64; b0 >= 0; b0 -= 64) {
    const int b = b0 + lane;
    int f = N;
    if (b < nchunks) f = agg[3 * b + 2];
    const int sf = wave_suffix_min(f);
    int ef = __shfl_down(sf, 1, 64);
    if (lane == 63) ef = N;
    if (b < nchunks) carry[3 * b + 2] = min(run_first, ef);
    run_first = min(run_first, __shfl(sf, 0, 64));
  }
}

// ---- tile schedule -------------------------------------------------------------------------
// Query tile m of row r covers tokens [r*T + m*kTile, min(r*T + (m+1)*kTile, (r+1)*T)).
// Its keys run from seg_start[first token] to its last token: cost = number of 64-key blocks.
// Key tile (same token range): its queries run from its first token to seg_end[last token]:
// cost = number of 64-query blocks.  Every tile has cost >= 1 (the diagonal is never masked).
//
// Order: tiles are sorted by a key (longest governing example first, then that example's start,
// then cost, heaviest first; ties by tile index).  The governing example is the one that fixes the
// streamed range: the example of the first token for a query tile, of the last token for a key
// tile.  Tiles of one long example thus run next to each other -- they stream the same K/V (or
// Q/dO) blocks at about the same time and share them in L2 -- and long work still starts first.
// Examples of at most one schedule tile all rank alike, so their tiles keep the order of the stream:
// a tile whose first example began in the previous tile reads that tile's last K/V rows again (a key
// tile the next tile's first Q/dO rows), and finds them in L2 only if the neighbour ran just before
// it on the same XCD.  With examples of 8..128 tokens that saves 9 % of the step.
constexpr int kShortExample = VA_TILE;
__device__ __forceinline__ unsigned long long tile_key(int len, int start, int cost) {
  return ((unsigned long long)(len <= kShortExample ? 0 : min(len, (1 << 20) - 1)) << 43) |
         ((unsigned long long)(0x7fffffff - start) << 12) | (unsigned long long)min(cost, 4095);
}
// An order entry carries, above the tile index (bits 0..23), the head rotation of its tile (bits
// 24..30; see head_rotation in va_mfma_common.h).  Tiles of an example longer than a schedule tile
// all get one rotation, derived from the example's first token: workgroup w runs on XCD w % 8 and the
// rotation decides which head lands on which XCD, so the tiles of one example - which stream the same
// K/V (or Q/dO) rows - keep each head on one XCD and fetch its rows into one L2 only, while different
// examples start from different rotations.  Tiles of short examples take their rank / 8: over a
// launch every XCD then meets every head (with a fixed assignment every XCD would always read the
// same 256-byte columns of the token rows, i.e. a fixed subset of the memory channels; measured on
// examples of 8..128 tokens, where the kernels are bound by HBM: two XCDs ran 20 % slower than the
// rest), while neighbours in launch order still mostly share an XCD.
__device__ __forceinline__ int32_t order_entry(int tile, unsigned long long key, int rank) {
  const unsigned len_class = (unsigned)(key >> 43);
  const unsigned start = 0x7fffffffu - (unsigned)((key >> 12) & 0x7fffffffu);
  const unsigned rot = len_class ? (start / kTile) * 5u + (start >> 13) : (unsigned)rank >> 3;
  return (int32_t)((unsigned)tile | ((rot & 127u) << 24));
}

// pass 2.  kFoldCarry: the workgroup derives its carries from all chunks' aggregates by itself (a launch less);
// otherwise `agg` holds the carries made by scan_carry_kernel.  The sort keys of the schedule tiles are
// written here too: the key of a query tile needs its first token's example, that of a key tile its last's.
constexpr int kFoldedCarryChunks = 4096;  // 8 M tokens: beyond that re-reading the aggregates costs more than a launch
template <typename IdT, bool kFoldCarry>
__global__ void __launch_bounds__(kScanThreads)
scan_finalize_kernel(const IdT *__restrict__ pos, int N, int T, const int32_t *__restrict__ agg, int nchunks,
                     int tiles_per_row, bool wide, int32_t *__restrict__ cu, int32_t *__restrict__ seg_id,
                     int32_t *__restrict__ seg_start, int32_t *__restrict__ seg_end, int32_t *__restrict__ meta,
                     unsigned long long *__restrict__ key_q, unsigned long long *__restrict__ key_kv) {
  constexpr int kWaves = kScanThreads / 64;
  __shared__ int s_cnt[kWaves], s_last[kWaves], s_first[kWaves];
  __shared__ int c_cnt[kWaves], c_last[kWaves], c_first[kWaves];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int base = blockIdx.x * kScanChunk + threadIdx.x * kPerThread;
  bool flag[kPerThread];
  start_flags(pos, base, N, T, flag);
  if (kFoldCarry) {
    int bc = 0, bl = -1, bf = N;
    for (int b = threadIdx.x; b < nchunks; b += kScanThreads) {
      const int ac = agg[3 * b], al = agg[3 * b + 1], af = agg[3 * b + 2];
      if (b < (int)blockIdx.x) { bc += ac; bl = max(bl, al); }
      if (b > (int)blockIdx.x) bf = min(bf, af);
    }
    for (int o = 32; o > 0; o >>= 1) {
      bc += __shfl_xor(bc, o, 64);
      bl = max(bl, __shfl_xor(bl, o, 64));
      bf = min(bf, __shfl_xor(bf, o, 64));
    }
    if (lane == 0) { c_cnt[w] = bc; c_last[w] = bl; c_first[w] = bf; }
  } else if (lane == 0) {  // one wave brings the carries, the others what leaves them as they are
    c_cnt[w] = w == 0 ? agg[3 * blockIdx.x] : 0;
    c_last[w] = w == 0 ? agg[3 * blockIdx.x + 1] : -1;
    c_first[w] = w == 0 ? agg[3 * blockIdx.x + 2] : N;
  }
  int cnt = 0, last = -1, first = N;
#pragma unroll
  for (int e = 0; e < kPerThread; ++e) {
    const int t = base + e;
    if (flag[e]) { ++cnt; last = t; first = min(first, t); }
  }
  const int icnt = wave_incl_add(cnt), ilast = wave_incl_max(last), sfirst = wave_suffix_min(first);
  if (lane == 63) { s_cnt[w] = icnt; s_last[w] = ilast; }
  if (lane == 0) s_first[w] = sfirst;
  __syncthreads();
  // exclusive values for this thread: wave-exclusive + earlier waves + chunk carry
  int ecnt = __shfl_up(icnt, 1, 64), elast = __shfl_up(ilast, 1, 64), efirst = __shfl_down(sfirst, 1, 64);
  if (lane == 0) { ecnt = 0; elast = -1; }
  if (lane == 63) efirst = N;
  for (int i = 0; i < w; ++i) { ecnt += s_cnt[i]; elast = max(elast, s_last[i]); }
  for (int i = w + 1; i < kWaves; ++i) efirst = min(efirst, s_first[i]);
  for (int i = 0; i < kWaves; ++i) {
    ecnt += c_cnt[i];
    elast = max(elast, c_last[i]);
    efirst = min(efirst, c_first[i]);
  }
  // next start strictly after each of this thread's tokens (right to left)
  int nxt[kPerThread];
  int run = efirst;
#pragma unroll
  for (int e = kPerThread - 1; e >= 0; --e) {
    nxt[e] = run;
    if (flag[e]) run = base + e;
  }
  int c = ecnt, l = elast, longest = 0, blocks = 0;
  int row = base / T, x = base - row * T;  // packed row and position in it, advanced without further divisions
  int id8[kPerThread], ss8[kPerThread];
#pragma unroll
  for (int e = 0; e < kPerThread; ++e) {
    const int t = base + e;
    if (t < N) {
      if (flag[e]) {
        cu[c] = t;
        ++c;
        l = t;
        longest = max(longest, nxt[e] - t);
      }
      const int row_last = t - x + T - 1, m = x / kTile;
      if (x % kTile == 0)  // first token of a schedule tile
        key_q[row * tiles_per_row + m] = tile_key(nxt[e] - l, l, ((t + min(kTile - 1, row_last - t)) >> 6) - (l >> 6) + 1);
      if (x % kTile == kTile - 1 || t == row_last) {  // last token of one
        const int n_blocks = ((nxt[e] - 1) >> 6) - ((t - x % kTile) >> 6) + 1;
        key_kv[row * tiles_per_row + m] = tile_key(nxt[e] - l, l, n_blocks);
        blocks += n_blocks;
      }
      if (t == N - 1) { meta[0] = c; cu[c] = N; }
    }
    id8[e] = c - 1;
    ss8[e] = l;
    if (++x == T) { x = 0; ++row; }
  }
  if (wide && base <= N - kPerThread) {  // wide: the arrays are 16-byte aligned; `base` is a multiple of 8
#pragma unroll
    for (int e = 0; e < kPerThread; e += 4) {
      *(int4 *)(seg_id + base + e) = make_int4(id8[e], id8[e + 1], id8[e + 2], id8[e + 3]);
      *(int4 *)(seg_start + base + e) = make_int4(ss8[e], ss8[e + 1], ss8[e + 2], ss8[e + 3]);
      *(int4 *)(seg_end + base + e) = make_int4(nxt[e], nxt[e + 1], nxt[e + 2], nxt[e + 3]);
    }
  } else {
#pragma unroll
    for (int e = 0; e < kPerThread; ++e)
      if (base + e < N) { seg_id[base + e] = id8[e]; seg_start[base + e] = ss8[e]; seg_end[base + e] = nxt[e]; }
  }
  for (int o = 32; o > 0; o >>= 1) {
    longest = max(longest, __shfl_xor(longest, o, 64));
    blocks += __shfl_xor(blocks, o, 64);
  }
  if (lane == 0 && longest > 0) atomicMax(&meta[1], longest);
  if (lane == 0 && blocks > 0) atomicAdd(&meta[2], blocks);
}

// order[rank] = tile, rank = number of tiles with a larger key (ties: lower index first).  32 tiles per
// workgroup, 8 threads to a tile, each of which compares it with every eighth key of a slab in LDS: one
// thread per tile took 17 us for 272 tiles (a chain of 272 reads and compares, after making all keys), this takes 5.4.
constexpr int kRankTiles = 32;
constexpr int kRankSlab = 512;
__global__ void __launch_bounds__(256)
tile_rank_kernel(const unsigned long long *__restrict__ key_q, const unsigned long long *__restrict__ key_kv,
                 int ntiles, int32_t *__restrict__ order_q, int32_t *__restrict__ order_kv) {
  __shared__ unsigned long long s_q[kRankSlab], s_kv[kRankSlab];
  const int part = threadIdx.x & 7, tile = blockIdx.x * kRankTiles + ((int)threadIdx.x >> 3);
  const unsigned long long cq = key_q[min(tile, ntiles - 1)], ckv = key_kv[min(tile, ntiles - 1)];
  int rq = 0, rkv = 0;
  for (int b0 = 0; b0 < ntiles; b0 += kRankSlab) {
    const int lim = min(kRankSlab, ntiles - b0);
    for (int i = threadIdx.x; i < lim; i += 256) { s_q[i] = key_q[b0 + i]; s_kv[i] = key_kv[b0 + i]; }
    __syncthreads();
    for (int i = part; i < lim; i += 8) {
      const int other = b0 + i;
      rq += (s_q[i] > cq) || (s_q[i] == cq && other < tile);
      rkv += (s_kv[i] > ckv) || (s_kv[i] == ckv && other < tile);
    }
    __syncthreads();
  }
  for (int o = 1; o < 8; o <<= 1) {
    rq += __shfl_xor(rq, o, 64);
    rkv += __shfl_xor(rkv, o, 64);
  }
  if (part == 0 && tile < ntiles) { order_q[rq] = order_entry(tile, cq, rq); order_kv[rkv] = order_entry(tile, ckv, rkv); }
}

// ---- one launch for streams of up to kSingleMaxTokens tokens -----------------------------------
// One workgroup holds the whole stream: boundary scan without carries (8 consecutive tokens per thread),
// then tile keys and ranks after a barrier.  All global traffic is coalesced (thread i touches tokens i,
// i + kThreads, ...): the ids' start flags go through LDS to the threads that scan them, and seg_id /
// seg_start / seg_end come back through LDS to be written out the same way -- one compute unit cannot afford
// 64 cache lines per load or store instruction.  Used when the stream fits, because at this size every extra
// launch costs as much as the work.  Bound: a chain of four barriers, which costs more with more waves, so a
// shorter stream gets a smaller workgroup; with 1024 threads whatever the size and one thread to a tile's rank:
// 16 tokens 7.0 us (now 6.0), 2048 tokens 7.5 (5.8), 8192 tokens 8.7 (8.3).
constexpr int kSingleMaxTokens = 1024 * kPerThread;  // 8192
constexpr int kSingleMaxTiles = 256;

// The values first .. end - 1 that the waves left in v, combined; `id` is the operation's identity.  All are read together: a
// loop up to the own wave is a chain of LDS round trips.
template <int kWaves, class Op> __device__ __forceinline__ int over_waves(const int *v, int first, int end, int id, Op op) {
  int x = id;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) x = op(x, i >= first && i < end ? v[i] : id);
  return x;
}

template <typename IdT, int kThreads>
__global__ void __launch_bounds__(kThreads)
pack_single_kernel(const IdT *__restrict__ pos, int N, int T, int tiles_per_row, int ntiles,
                   int32_t *__restrict__ cu, int32_t *__restrict__ seg_id, int32_t *__restrict__ seg_start,
                   int32_t *__restrict__ seg_end, int32_t *__restrict__ meta, int32_t *__restrict__ order_q,
                   int32_t *__restrict__ order_kv) {
  constexpr int kWaves = kThreads / 64, kTokens = kThreads * kPerThread;
  __shared__ int s_cnt[kWaves], s_last[kWaves], s_first[kWaves];
  __shared__ __attribute__((aligned(16))) int32_t s_ss[kTokens], s_se[kTokens], s_id[kTokens];
  __shared__ __attribute__((aligned(8))) uint8_t s_flag[kTokens];
  __shared__ unsigned long long s_q[kSingleMaxTiles], s_kv[kSingleMaxTiles];
  __shared__ int s_blocks[kWaves];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  {  // start flags, coalesced; all loads in flight together
    IdT id[kPerThread];
#pragma unroll
    for (int e = 0; e < kPerThread; ++e) id[e] = pos[min(e * kThreads + (int)threadIdx.x, N - 1)];
    int r = threadIdx.x % T;
    const int step = kThreads % T;
#pragma unroll
    for (int e = 0; e < kPerThread; ++e) {
      const int t = e * kThreads + threadIdx.x;
      s_flag[t] = t < N && (id[e] == 0 || r == 0);
      r += step;
      if (r >= T) r -= T;
    }
  }
  __syncthreads();
  const int base = threadIdx.x * kPerThread;
  bool flag[kPerThread];
  {
    const unsigned long long f8 = *(const unsigned long long *)(s_flag + base);
#pragma unroll
    for (int e = 0; e < kPerThread; ++e) flag[e] = (f8 >> (8 * e)) & 1;
  }
  int cnt = 0, last = -1, first = N;
#pragma unroll
  for (int e = 0; e < kPerThread; ++e) {
    const int t = base + e;
    if (flag[e]) { ++cnt; last = t; first = min(first, t); }
  }
  const int icnt = wave_incl_add(cnt), ilast = wave_incl_max(last), sfirst = wave_suffix_min(first);
  if (lane == 63) { s_cnt[w] = icnt; s_last[w] = ilast; }
  if (lane == 0) s_first[w] = sfirst;
  __syncthreads();
  int ecnt = __shfl_up(icnt, 1, 64), elast = __shfl_up(ilast, 1, 64), efirst = __shfl_down(sfirst, 1, 64);
  if (lane == 0) { ecnt = 0; elast = -1; }
  if (lane == 63) efirst = N;
  ecnt = over_waves<kWaves>(s_cnt, 0, w, 0, [](int x, int y) { return x + y; }) + ecnt;
  elast = max(elast, over_waves<kWaves>(s_last, 0, w, -1, [](int x, int y) { return max(x, y); }));
  efirst = min(efirst, over_waves<kWaves>(s_first, w + 1, kWaves, N, [](int x, int y) { return min(x, y); }));
  int nxt[kPerThread];
  int run = efirst;
#pragma unroll
  for (int e = kPerThread - 1; e >= 0; --e) {
    nxt[e] = run;
    if (flag[e]) run = base + e;
  }
  int c = ecnt, l = elast, longest = 0;
  int id8[kPerThread], ss8[kPerThread];
#pragma unroll
  for (int e = 0; e < kPerThread; ++e) {
    const int t = base + e;
    if (flag[e]) { cu[c] = t; ++c; l = t; longest = max(longest, nxt[e] - t); }  // never set at t >= N
    id8[e] = c - 1;
    ss8[e] = l;
  }
  // 16-byte LDS stores (a 4-byte store per token, 32 bytes apart over the lanes, is an 8-way bank conflict:
  // 9.8 -> 8.6 us for 8192 tokens); what lies beyond N is never read
#pragma unroll
  for (int e = 0; e < kPerThread; e += 4) {
    *(int4 *)(s_id + base + e) = make_int4(id8[e], id8[e + 1], id8[e + 2], id8[e + 3]);
    *(int4 *)(s_ss + base + e) = make_int4(ss8[e], ss8[e + 1], ss8[e + 2], ss8[e + 3]);
    *(int4 *)(s_se + base + e) = make_int4(nxt[e], nxt[e + 1], nxt[e + 2], nxt[e + 3]);
  }
  for (int o = 32; o > 0; o >>= 1) longest = max(longest, __shfl_xor(longest, o, 64));
  __syncthreads();  // s_cnt free; s_id / s_ss / s_se complete
  if (lane == 0) s_cnt[w] = longest;
  if ((int)threadIdx.x == (N - 1) / kPerThread) {  // the thread holding the last token knows the number of examples
    meta[0] = c;
    for (int i = 3; i < 8; ++i) meta[i] = 0;
    cu[c] = N;
  }
#pragma unroll
  for (int e = 0; e < kPerThread; ++e) {  // coalesced write-out
    const int t = e * kThreads + threadIdx.x;
    if (t < N) { seg_id[t] = s_id[t]; seg_start[t] = s_ss[t]; seg_end[t] = s_se[t]; }
  }
  // tile keys
  int blocks = 0;
  for (int tile = threadIdx.x; tile < ntiles; tile += kThreads) {
    const int r = tile / tiles_per_row, m = tile % tiles_per_row;
    const int t0 = r * T + m * kTile;
    const int t1 = min(t0 + kTile, (r + 1) * T) - 1;
    const int ss0 = s_ss[t0], se0 = s_se[t0], ss1 = s_ss[t1], se1 = s_se[t1];
    s_q[tile] = tile_key(se0 - ss0, ss0, (t1 >> 6) - (ss0 >> 6) + 1);
    const int n_blocks = ((se1 - 1) >> 6) - (t0 >> 6) + 1;
    s_kv[tile] = tile_key(se1 - ss1, ss1, n_blocks);
    blocks += n_blocks;
  }
  for (int o = 32; o > 0; o >>= 1) blocks += __shfl_xor(blocks, o, 64);
  if (lane == 0) s_blocks[w] = blocks;
  __syncthreads();
  if (threadIdx.x == 0) {
    meta[1] = over_waves<kWaves>(s_cnt, 0, kWaves, 0, [](int x, int y) { return max(x, y); });
    meta[2] = over_waves<kWaves>(s_blocks, 0, kWaves, 0, [](int x, int y) { return x + y; });
  }
  // ranks: `parts` threads to a tile (a power of two, so that they share a wave), each compares every parts-th key
  static_assert(kThreads >= kSingleMaxTiles, "a thread to a tile, at least");
  const int parts = min(64, kThreads >> (32 - __clz(max(ntiles - 1, 1))));
  const int part = threadIdx.x & (parts - 1), tile = threadIdx.x / parts;
  const unsigned long long cq = s_q[min(tile, ntiles - 1)], ckv = s_kv[min(tile, ntiles - 1)];
  int rq = 0, rkv = 0;
  for (int o = part; o < ntiles; o += parts) {
    rq += (s_q[o] > cq) || (s_q[o] == cq && o < tile);
    rkv += (s_kv[o] > ckv) || (s_kv[o] == ckv && o < tile);
  }
  for (int o = 1; o < parts; o <<= 1) {
    rq += __shfl_xor(rq, o, 64);
    rkv += __shfl_xor(rkv, o, 64);
  }
  if (part == 0 && tile < ntiles) {
    order_q[rq] = order_entry(tile, cq, rq);
    order_kv[rkv] = order_entry(tile, ckv, rkv);
  }
}

}  // namespace

hipError_t launch_pack(const void *pos, va_itype it, int rows, int T, const va_segments &seg,
                       hipStream_t stream) {
  const int N = rows * T;
  const int nchunks = ceil_div(N, kScanChunk);
  const int tiles_per_row = ceil_div(T, kTile), ntiles = rows * tiles_per_row;
  if (N <= kSingleMaxTokens && ntiles <= kSingleMaxTiles) {
    auto launch = [&](auto *ids, auto threads) {
      typedef std::remove_cv_t<std::remove_pointer_t<decltype(ids)>> IdT;
      pack_single_kernel<IdT, decltype(threads)::value><<<1, decltype(threads)::value, 0, stream>>>(
          ids, N, T, tiles_per_row, ntiles, seg.cu_seqlens, seg.seg_id, seg.seg_start, seg.seg_end, seg.meta, seg.q_tile_order,
          seg.kv_tile_order);
    };
    auto by_size = [&](auto *ids) {
      if (N <= 256 * kPerThread) launch(ids, std::integral_constant<int, 256>());
      else if (N <= 512 * kPerThread) launch(ids, std::integral_constant<int, 512>());
      else launch(ids, std::integral_constant<int, 1024>());
    };
    if (it == VA_I64) by_size((const int64_t *)pos);
    else by_size((const int32_t *)pos);
    return hipGetLastError();
  }
  const bool fold = nchunks <= kFoldedCarryChunks;
  int32_t *agg = seg.scratch;                  // [3 * nchunks]
  int32_t *carry = seg.scratch + 3 * nchunks;  // [3 * nchunks]
  unsigned long long *key_q = (unsigned long long *)(seg.scratch + 8 * nchunks);  // [ntiles] sort keys
  unsigned long long *key_kv = key_q + ntiles;                                    // [ntiles]
  const bool wide = (((uintptr_t)seg.seg_id | (uintptr_t)seg.seg_start | (uintptr_t)seg.seg_end) & 15) == 0;
  auto scan = [&](auto *ids) {
    typedef std::remove_cv_t<std::remove_pointer_t<decltype(ids)>> IdT;
    scan_aggregate_kernel<IdT><<<nchunks, kScanThreads, 0, stream>>>(ids, N, T, agg, seg.meta);
    if (!fold) scan_carry_kernel<<<1, 64, 0, stream>>>(agg, nchunks, N, carry);
    auto *finalize = fold ? scan_finalize_kernel<IdT, true> : scan_finalize_kernel<IdT, false>;
    finalize<<<nchunks, kScanThreads, 0, stream>>>(ids, N, T, fold ? agg : carry, nchunks, tiles_per_row, wide, seg.cu_seqlens,
                                                   seg.seg_id, seg.seg_start, seg.seg_end, seg.meta, key_q, key_kv);
  };
  if (it == VA_I64) scan((const int64_t *)pos);
  else scan((const int32_t *)pos);
  tile_rank_kernel<<<ceil_div(ntiles, kRankTiles), 256, 0, stream>>>(key_q, key_kv, ntiles, seg.q_tile_order, seg.kv_tile_order);
  return hipGetLastError();
}

}  // namespace va
