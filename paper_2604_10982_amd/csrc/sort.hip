// Stable LSD radix sort of (uint32 key, uint32 value) pairs.
//
// Used twice per frame: the visible surfels by FP32 depth bits (32 bits,
// 4 passes) and then the emitted (tile, surfel) pairs by tile id (ceil(log2
// tiles) bits, 2 passes).  Because the pairs are emitted in depth order and
// every pass is stable, the result is the pair list ordered by
// (tile, depth, surfel id) -- an LSD sort of the composite key in which the
// low 32 bits are sorted once per surfel instead of once per pair.
//
// Each pass is reduce-then-scan (no inter-block waiting):
//   upsweep   -- per-block digit histogram (LDS, one sub-histogram per wave);
//   scan      -- one block per digit scans that digit's row over blocks;
//   downsweep -- per block, stable ranks from wave ballots, the tile sorted
//                by digit in LDS, written out bucket by bucket.
// The element count is read on the device, so the launch shape only depends
// on the capacity and no host synchronisation is needed.
#include "common.h"
#include "internal.h"

namespace psm {

__global__ __launch_bounds__(kSortThreads) void k_rs_upsweep(const uint32_t* __restrict__ keys,
                                                            const uint32_t* __restrict__ n_dev, int shift,
                                                            int bits, uint32_t* __restrict__ hist) {
  const uint32_t n = *n_dev;
  const uint32_t nb = (n + kSortTile - 1) / kSortTile;
  if (blockIdx.x >= nb) return;
  __shared__ uint32_t s_h[4][256];
  const int wave = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < 4 * 256; i += kSortThreads) (&s_h[0][0])[i] = 0;
  __syncthreads();
  const uint32_t mask = (1u << bits) - 1u;
  const uint32_t base = blockIdx.x * kSortTile;
#pragma unroll 4
  for (int j = 0; j < kSortItems; ++j) {
    const uint32_t idx = base + j * kSortThreads + threadIdx.x;
    if (idx < n) atomicAdd(&s_h[wave][(keys[idx] >> shift) & mask], 1u);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < (1 << bits); d += kSortThreads)
    hist[(size_t)d * nb + blockIdx.x] = s_h[0][d] + s_h[1][d] + s_h[2][d] + s_h[3][d];
}

// Block d: exclusive scan of digit d's counts over the blocks; the digit's
// total goes to hist[256 * nb_max + d].
__global__ __launch_bounds__(256) void k_rs_scan(const uint32_t* __restrict__ n_dev, uint32_t* __restrict__ hist,
                                                 int64_t nb_max) {
  const uint32_t n = *n_dev;
  const uint32_t nb = (n + kSortTile - 1) / kSortTile;
  const int d = blockIdx.x;
  const int t = threadIdx.x;
  uint32_t* row = hist + (size_t)d * nb;
  __shared__ uint32_t s[256];
  const uint32_t per = (nb + 255) / 256;
  const uint32_t b0 = t * per, b1 = min(nb, b0 + per);
  uint32_t acc = 0;
  for (uint32_t b = b0; b < b1; ++b) acc += row[b];
  s[t] = acc;
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {
    const uint32_t v = t >= o ? s[t - o] : 0u;
    __syncthreads();
    s[t] += v;
    __syncthreads();
  }
  uint32_t run = s[t] - acc;
  for (uint32_t b = b0; b < b1; ++b) {
    const uint32_t v = row[b];
    row[b] = run;
    run += v;
  }
  if (t == 255) hist[256 * nb_max + d] = s[255];
}

// Block-wide (256 threads) exclusive prefix sum of one value per thread;
// red holds 4 words of scratch.  Ends with a barrier, so red can be reused.
__device__ __forceinline__ uint32_t sort_scan_excl(uint32_t v, uint32_t* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) red[wave] = x;
  __syncthreads();
  uint32_t pre = 0;
#pragma unroll
  for (int w = 0; w < 3; ++w) pre += w < wave ? red[w] : 0u;
  __syncthreads();
  return pre + x - v;
}

// One block per tile of kSortTile elements; wave w owns the elements
// [base + w kSortTile / 4, base + (w + 1) kSortTile / 4), kSortItems
// coalesced rows of 64.  (1) Each wave ranks its elements among equal digits
// in index order: wave ballots give the rank within a row, wave-private
// digit counters in LDS carry the count of the rows before (a wave's LDS
// operations complete in program order, so no barrier is needed).  (2) The
// counts are scanned over the waves and the digits, and every element is
// placed in LDS at its block-local position: the tile sorted stably by
// digit.  (3) The tile is written out in that order: consecutive threads
// write consecutive addresses of a digit's bucket.
__global__ __launch_bounds__(kSortThreads) void k_rs_downsweep(
    const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
    uint32_t* __restrict__ vout, const uint32_t* __restrict__ n_dev, int shift, int bits,
    const uint32_t* __restrict__ hist, int64_t nb_max) {
  static_assert(kSortThreads == 256, "one thread per digit of an 8-bit pass");
  const uint32_t n = *n_dev;
  const uint32_t nb = (n + kSortTile - 1) / kSortTile;
  if (blockIdx.x >= nb) return;
  __shared__ uint32_t s_cnt[4][256];  // per-wave digit counts, then the waves' offsets
  __shared__ uint32_t s_gbase[256];   // first global position of each digit for this block
  __shared__ uint32_t s_lbase[256];   // first block-local position of each digit
  __shared__ uint32_t s_red[4];
  __shared__ uint32_t s_k[kSortTile], s_v[kSortTile];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int ndig = 1 << bits;
  const uint32_t mask = (uint32_t)ndig - 1u;
  const uint64_t lt = (1ull << lane) - 1ull;
  const uint32_t base = blockIdx.x * kSortTile;
  const uint32_t wbase = base + (uint32_t)wave * (64 * kSortItems);

  // global start of each digit for this block: all elements of smaller digits
  // plus this digit's elements in earlier blocks
  const uint32_t tot = t < ndig ? hist[256 * nb_max + t] : 0u;
  const uint32_t ex = sort_scan_excl(tot, s_red);
  s_gbase[t] = ex + (t < ndig ? hist[(size_t)t * nb + blockIdx.x] : 0u);
#pragma unroll
  for (int w = 0; w < 4; ++w) s_cnt[w][t] = 0u;
  __syncthreads();

  uint32_t key[kSortItems], val[kSortItems], rank[kSortItems];
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) {
    const uint32_t idx = wbase + j * 64 + lane;
    key[j] = idx < n ? kin[idx] : 0u;
    val[j] = idx < n ? vin[idx] : 0u;
  }
  uint32_t* cnt = s_cnt[wave];
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) {
    const bool valid = wbase + j * 64 + lane < n;
    const uint32_t d = (key[j] >> shift) & mask;
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const uint32_t r = (uint32_t)__popcll(peers & lt);
    const uint32_t c = valid ? cnt[d] : 0u;
    rank[j] = c + r;
    if (valid && r == 0) cnt[d] = c + (uint32_t)__popcll(peers);
  }
  __syncthreads();
  // digit t: the waves' offsets (exclusive over waves) and the digit's
  // block-local start (exclusive over digits)
  const uint32_t c0 = s_cnt[0][t], c1 = s_cnt[1][t], c2 = s_cnt[2][t], c3 = s_cnt[3][t];
  s_cnt[0][t] = 0u;
  s_cnt[1][t] = c0;
  s_cnt[2][t] = c0 + c1;
  s_cnt[3][t] = c0 + c1 + c2;
  s_lbase[t] = sort_scan_excl(c0 + c1 + c2 + c3, s_red);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) {
    if (wbase + j * 64 + lane < n) {
      const uint32_t d = (key[j] >> shift) & mask;
      const uint32_t lp = s_lbase[d] + cnt[d] + rank[j];
      s_k[lp] = key[j];
      s_v[lp] = val[j];
    }
  }
  __syncthreads();
  const uint32_t m = min((uint32_t)kSortTile, n - base);
  for (uint32_t i = t; i < m; i += kSortThreads) {
    const uint32_t k = s_k[i];
    const uint32_t d = (k >> shift) & mask;
    const uint32_t gp = s_gbase[d] + (i - s_lbase[d]);
    kout[gp] = k;
    vout[gp] = s_v[i];
  }
}

// ---- small inputs: one block ---------------------------------------------
// A small call is its launches: the two sorts, the count scan and the ranges
// took 23 of its 27, 3 to 7 us each (100 of the 190 us of a 2k-surfel frame).  One
// block of 16 waves sorts up to kSingleMax pairs in LDS (128 KB), every pass as in
// k_rs_downsweep with the wave's rows in registers, and goes on to what
// follows the sort.  More pairs (the count is on the device, the launch is
// chosen by the capacity) pass through global memory chunk by chunk.
constexpr int kSingleThreads = 1024;
constexpr int kSingleWaves = kSingleThreads / 64;
constexpr int kSingleItems = 16;
constexpr int kSingleMax = kSingleThreads * kSingleItems;

struct SingleShared {
  uint32_t k[kSingleMax], v[kSingleMax];
  uint32_t cnt[kSingleWaves][256];  // per-wave digit counts, then the waves' offsets
  uint32_t lbase[256];              // first block-local position of each digit
  uint32_t gbase[256];              // first global position of each digit (chunked form)
  uint32_t red[kSingleWaves];
};

// Block-wide exclusive prefix sum of one value per thread.
template <typename T>
__device__ __forceinline__ T single_scan_excl(T v, T* red, T& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  T x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const T y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) red[wave] = x;
  __syncthreads();
  T pre = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kSingleWaves; ++w) {
    const T t = red[w];
    pre += w < wave ? t : (T)0;
    tot += t;
  }
  total = tot;
  __syncthreads();
  return pre + x - v;
}

// One stable pass over the m <= kSingleMax pairs given by load(i): ranks by
// wave ballots, the pairs placed in LDS sorted by digit.  The LDS pairs may be
// load's source (all are read before any is placed).
template <class Load>
__device__ __forceinline__ void single_pass(SingleShared& S, uint32_t m, int shift, int bits, Load&& load) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint32_t mask = (1u << bits) - 1u;
  const int rows = (int)((m + kSingleThreads - 1) / kSingleThreads);
  const uint64_t lt = (1ull << lane) - 1ull;
  const uint32_t wbase = (uint32_t)(wave * rows * 64);
  for (int i = t; i < kSingleWaves * 256; i += kSingleThreads) (&S.cnt[0][0])[i] = 0u;
  uint32_t key[kSingleItems], val[kSingleItems], rank[kSingleItems];
#pragma unroll
  for (int j = 0; j < kSingleItems; ++j) {
    key[j] = val[j] = rank[j] = 0u;
    const uint32_t i = wbase + j * 64 + lane;
    if (j < rows && i < m) load(i, key[j], val[j]);
  }
  __syncthreads();
  uint32_t* cnt = S.cnt[wave];
#pragma unroll
  for (int j = 0; j < kSingleItems; ++j) {
    if (j >= rows) continue;  // block-uniform
    const bool valid = wbase + j * 64 + lane < m;
    const uint32_t d = (key[j] >> shift) & mask;
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t q = __ballot(bit);
      peers &= bit ? q : ~q;
    }
    const uint32_t r = (uint32_t)__popcll(peers & lt);
    const uint32_t c = valid ? cnt[d] : 0u;
    rank[j] = c + r;
    if (valid && r == 0) cnt[d] = c + (uint32_t)__popcll(peers);
  }
  __syncthreads();
  uint32_t tot = 0;
  if (t < 256) {
#pragma unroll
    for (int w = 0; w < kSingleWaves; ++w) {
      const uint32_t c = S.cnt[w][t];
      S.cnt[w][t] = tot;
      tot += c;
    }
  }
  uint32_t all;
  const uint32_t ex = single_scan_excl<uint32_t>(tot, S.red, all);
  if (t < 256) S.lbase[t] = ex;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSingleItems; ++j) {
    if (j < rows && wbase + j * 64 + lane < m) {
      const uint32_t d = (key[j] >> shift) & mask;
      const uint32_t lp = S.lbase[d] + cnt[d] + rank[j];
      S.k[lp] = key[j];
      S.v[lp] = val[j];
    }
  }
  __syncthreads();
}

// Stable sort of n pairs (k0, v0) on key bits [0, bits).  Up to kSingleMax: the
// result is left in S.k, S.v and written to (k0, v0).  More: an even number of
// passes between (k0, v0) and (k1, v1).
__device__ __forceinline__ void single_sort(SingleShared& S, uint32_t n, int bits, uint32_t* k0, uint32_t* v0,
                                            uint32_t* k1, uint32_t* v1) {
  const int t = threadIdx.x;
  if (n <= (uint32_t)kSingleMax) {
    const int passes = bits > 8 ? (bits + 7) / 8 : 1;
    int shift = 0;
    for (int p = 0; p < passes; ++p) {
      const int left = passes - p, b = (bits - shift + left - 1) / left;
      if (p == 0)
        single_pass(S, n, shift, b, [&](uint32_t i, uint32_t& k, uint32_t& v) { k = k0[i]; v = v0[i]; });
      else
        single_pass(S, n, shift, b, [&](uint32_t i, uint32_t& k, uint32_t& v) { k = S.k[i]; v = S.v[i]; });
      shift += b;
    }
    for (uint32_t i = t; i < n; i += kSingleThreads) {
      k0[i] = S.k[i];
      v0[i] = S.v[i];
    }
    return;
  }
  int passes = bits > 8 ? (bits + 7) / 8 : 2;
  passes += passes & 1;
  uint32_t *ki = k0, *vi = v0, *ko = k1, *vo = v1;
  int shift = 0;
  for (int p = 0; p < passes; ++p) {
    const int left = passes - p, b = (bits - shift + left - 1) / left;
    const uint32_t mask = (1u << b) - 1u;
    // all digits' counts, then their first positions
    for (int i = t; i < kSingleWaves * 256; i += kSingleThreads) (&S.cnt[0][0])[i] = 0u;
    __syncthreads();
    for (uint32_t i = t; i < n; i += kSingleThreads) atomicAdd(&S.cnt[t >> 6][(ki[i] >> shift) & mask], 1u);
    __syncthreads();
    uint32_t tot = 0, all;
    if (t < 256)
      for (int w = 0; w < kSingleWaves; ++w) tot += S.cnt[w][t];
    const uint32_t ex = single_scan_excl<uint32_t>(tot, S.red, all);
    if (t < 256) S.gbase[t] = ex;
    __syncthreads();
    for (uint32_t c0 = 0; c0 < n; c0 += kSingleMax) {
      const uint32_t m = min((uint32_t)kSingleMax, n - c0);
      single_pass(S, m, shift, b, [&](uint32_t i, uint32_t& k, uint32_t& v) { k = ki[c0 + i]; v = vi[c0 + i]; });
      for (uint32_t i = t; i < m; i += kSingleThreads) {
        const uint32_t k = S.k[i], d = (k >> shift) & mask;
        const uint32_t gp = S.gbase[d] + (i - S.lbase[d]);
        ko[gp] = k;
        vo[gp] = S.v[i];
      }
      __syncthreads();
      if (t < 256) {  // the digit's elements of this chunk
        const uint32_t next = t < 255 ? S.lbase[t + 1] : m;
        S.gbase[t] += next - S.lbase[t];
      }
      __syncthreads();
    }
    uint32_t* x = ki; ki = ko; ko = x;
    x = vi; vi = vo; vo = x;
    shift += b;
    __syncthreads();
  }
}

// Depth sort, exclusive scan of the pair counts in depth order, status words
// and empty tile ranges (the small form of the launches before the emission).
__global__ __launch_bounds__(kSingleThreads) void k_single_depth(
    uint32_t n, uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1, const uint32_t* __restrict__ count, uint32_t* __restrict__ offs,
    uint32_t* __restrict__ status, uint32_t tiles, uint64_t total_bytes, uint32_t cap, uint2* __restrict__ ranges) {
  __shared__ SingleShared S;
  __shared__ uint64_t s_red64[kSingleWaves];
  const int t = threadIdx.x;
  for (uint32_t i = t; i < tiles; i += kSingleThreads) ranges[i] = make_uint2(0u, 0u);
  single_sort(S, n, 32, k0, v0, k1, v1);
  // thread t: the ranks [t per, (t + 1) per)
  const uint32_t per = (n + kSingleThreads - 1) / kSingleThreads;
  uint32_t c[kSingleItems];
  uint64_t sum = 0;
#pragma unroll
  for (int j = 0; j < kSingleItems; ++j) {
    const uint32_t r = (uint32_t)t * per + j;
    c[j] = (uint32_t)j < per && r < n ? count[S.v[r]] : 0u;
    sum += c[j];
  }
  uint64_t all;
  uint64_t run = single_scan_excl<uint64_t>(sum, s_red64, all);
#pragma unroll
  for (int j = 0; j < kSingleItems; ++j) {
    const uint32_t r = (uint32_t)t * per + j;
    if ((uint32_t)j < per && r < n) offs[r] = (uint32_t)run;
    run += c[j];
  }
  if (t < kStWords) status[t] = init_word(t, n, tiles, total_bytes, cap);
  __syncthreads();
  if (t == 0) write_pair_total(status, all, cap);
}

// Pair sort, virtual surfel ids of the sorted pairs, tile ranges and the walk's
// counter lines (the small form of the launches after the emission).
__global__ __launch_bounds__(kSingleThreads) void k_single_pairs(
    uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1, int bits, const uint32_t* __restrict__ sid_emit, const uint32_t* __restrict__ status, uint32_t* __restrict__ pid,
    uint2* __restrict__ ranges, uint64_t* __restrict__ stat, int slots) {
  __shared__ SingleShared S;
  const int t = threadIdx.x;
  const uint32_t P = status[kStP];
  if (t < slots) {
#pragma unroll
    for (int i = 0; i < 3; ++i) stat[t * kStatLine + i] = 0ull;
  }
  single_sort(S, P, bits, k0, v0, k1, v1);
  __syncthreads();
  const bool lds = P <= (uint32_t)kSingleMax;
  const auto key = [&](uint32_t j) { return lds ? S.k[j] : k0[j]; };
  for (uint32_t j = t; j < P; j += kSingleThreads) {
    pid[j] = sid_emit[lds ? S.v[j] : v0[j]];
    const uint32_t tile = key(j);
    if (j == 0 || key(j - 1) != tile) ranges[tile].x = j;
    if (j == P - 1 || key(j + 1) != tile) ranges[tile].y = j + 1;
  }
}

void launch_single_depth(const Layout& L, char* ws, hipStream_t st) {
  hipLaunchKernelGGL(k_single_depth, dim3(1), dim3(kSingleThreads), 0, st, (uint32_t)L.n, (uint32_t*)(ws + L.key0),
                     (uint32_t*)(ws + L.id0), (uint32_t*)(ws + L.key1), (uint32_t*)(ws + L.id1),
                     (const uint32_t*)(ws + L.count), (uint32_t*)(ws + L.offs), (uint32_t*)(ws + L.status),
                     (uint32_t)L.tiles, (uint64_t)L.total, (uint32_t)L.cap, (uint2*)(ws + L.ranges));
}

void launch_single_pairs(const Layout& L, int bits, char* ws, hipStream_t st) {
  hipLaunchKernelGGL(k_single_pairs, dim3(1), dim3(kSingleThreads), 0, st, (uint32_t*)(ws + L.ptile0),
                     (uint32_t*)(ws + L.eid0), (uint32_t*)(ws + L.ptile1), (uint32_t*)(ws + L.eid1), bits,
                     (const uint32_t*)(ws + L.sid_emit), (const uint32_t*)(ws + L.status), (uint32_t*)(ws + L.pid),
                     (uint2*)(ws + L.ranges), (uint64_t*)(ws + L.hist), stat_slots(L));
}

void radix_sort_pairs(uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1, const uint32_t* n_dev,
                      int64_t cap_n, int bits, uint32_t* hist, int64_t nb_max, hipStream_t st) {
  if (cap_n <= 0) return;
  int passes = std::max(2, (bits + 7) / 8);
  if (passes & 1) ++passes;
  const unsigned grid = (unsigned)cdiv(cap_n, kSortTile);
  uint32_t *ki = k0, *vi = v0, *ko = k1, *vo = v1;
  int shift = 0;
  for (int p = 0; p < passes; ++p) {
    const int left = passes - p;
    const int b = (bits - shift + left - 1) / left;
    hipLaunchKernelGGL(k_rs_upsweep, dim3(grid), dim3(kSortThreads), 0, st, ki, n_dev, shift, b, hist);
    hipLaunchKernelGGL(k_rs_scan, dim3(1u << b), dim3(256), 0, st, n_dev, hist, nb_max);
    hipLaunchKernelGGL(k_rs_downsweep, dim3(grid), dim3(kSortThreads), 0, st, ki, vi, ko, vo, n_dev, shift, b,
                       hist, nb_max);
    std::swap(ki, ko);
    std::swap(vi, vo);
    shift += b;
  }
}

}  // namespace psm
