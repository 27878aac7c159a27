// Radix sort of (int64 key, int64 value) pairs by key, for group-by results
// that are asked for in key order and do not come out in it.
//
// Least significant digit first, with the digits that the keys need: a pass
// over the keys finds their least and greatest value, and key - least is sorted
// by an even number of passes over just its bits (even, so that the ping-pong
// ends in the caller's buffers; 6 passes of 6 bits for 33 significant bits).
// A pass is two kernels over the same ranges of tiles, one range a block: the
// first counts the range's digits, the second adds up the counts that lie before
// it (whole groups of 16 ranges, then ranges), ranks each tile by digit, and
// writes the digits' runs from LDS.  Up to kSmallPairs pairs are sorted by one
// block in LDS instead.  The number of pairs is on the device: kernels that it
// leaves nothing to do return at once.
//
// Bound by the pairs' traffic (40 bytes a pair and pass) for large inputs and
// by launches for small ones.  A pass of one kernel, its tiles finding their
// places by looking back over the 256 counts of every earlier tile, measured
// slower (10M pairs: 151 us a pass with four tiles a step, 171 with 32, against
// 18 + 78): 512 tiles are in flight and each step crosses to another XCD's L2.
// Against eight byte passes of histogram, cleared status words, scan and scatter
// (33 launches), a group-by ordered by key measured: 100k rows into 5000 int64
// groups 228 -> 94 us, 900k rows into 300k 348 -> 221 us, 60M rows into 10M
// 2422 -> 2288 us with a key range pass of 125 us that it did not have.
#include "pyst_internal.h"
#include "ranges.h"
#include "table.h"

namespace pyst {

constexpr int kSortBlock = 1024, kSortItems = 4, kSortTile = kSortBlock * kSortItems;
constexpr int kSortWaves = kSortBlock / kWave;
constexpr int kSmallItems = 8, kSmallPairs = kSortBlock * kSmallItems;

struct SortPlan {
  int64_t base;   // least key
  int32_t npass;  // 0: nothing to do here
  int32_t width;  // bits a pass
};

__device__ __forceinline__ int64_t sort_count(const int64_t *d_count, int64_t cap) {
  const int64_t c = *d_count;
  return c < cap ? c : cap;
}

__device__ __forceinline__ void block_key_range(int64_t &lo, int64_t &hi, int64_t *s_lo, int64_t *s_hi, int nwaves) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    const int64_t l = __shfl_xor(lo, o), h = __shfl_xor(hi, o);
    lo = l < lo ? l : lo;
    hi = h > hi ? h : hi;
  }
  if (lane_id() == 0) {
    s_lo[threadIdx.x / kWave] = lo;
    s_hi[threadIdx.x / kWave] = hi;
  }
  __syncthreads();
  for (int w = 0; w < nwaves; ++w) {
    lo = s_lo[w] < lo ? s_lo[w] : lo;
    hi = s_hi[w] > hi ? s_hi[w] : hi;
  }
}

__device__ __forceinline__ int range_bits(int64_t lo, int64_t hi) {
  const uint64_t span = static_cast<uint64_t>(hi) - static_cast<uint64_t>(lo);
  return span ? 64 - __clzll(static_cast<long long>(span)) : 1;
}

// Per-block key range, and every pass's group counts cleared.
__global__ __launch_bounds__(256) void k_sort_range(const int64_t *keys, const int64_t *d_count, int64_t cap, int64_t *lo_out,
                                                    int64_t *hi_out, RangeCounts counts, int passes) {
  __shared__ int64_t s_lo[4], s_hi[4];
  const int64_t n = sort_count(d_count, cap);
  if (n <= kSmallPairs) return;
  const int64_t gtid = int64_t{blockIdx.x} * 256 + threadIdx.x, step = int64_t{gridDim.x} * 256;
  for (int64_t i = gtid; i < int64_t{passes} * counts.ngroups * kRangeDigits; i += step) counts.group[i] = 0;
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  constexpr int U = 8;
  for (int64_t i0 = gtid; i0 < n; i0 += step * U) {
    int64_t k[U];
#pragma unroll
    for (int u = 0; u < U; ++u) k[u] = keys[i0 + u * step < n ? i0 + u * step : i0];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      lo = k[u] < lo ? k[u] : lo;
      hi = k[u] > hi ? k[u] : hi;
    }
  }
  block_key_range(lo, hi, s_lo, s_hi, 4);
  if (threadIdx.x == 0) {
    lo_out[blockIdx.x] = lo;
    hi_out[blockIdx.x] = hi;
  }
}

__global__ __launch_bounds__(kSortBlock) void k_sort_plan(SortPlan *plan, const int64_t *d_count, int64_t cap,
                                                         const int64_t *lo_in, const int64_t *hi_in, int nblocks) {
  __shared__ int64_t s_lo[kSortWaves], s_hi[kSortWaves];
  const int tid = static_cast<int>(threadIdx.x);
  if (sort_count(d_count, cap) <= kSmallPairs) {
    if (tid == 0) plan->npass = 0;
    return;
  }
  int64_t lo = tid < nblocks ? lo_in[tid] : INT64_MAX, hi = tid < nblocks ? hi_in[tid] : INT64_MIN;
  block_key_range(lo, hi, s_lo, s_hi, kSortWaves);
  if (tid == 0) {
    const int bits = range_bits(lo, hi);
    const int np = (bits + 15) / 16 * 2;  // an even number of passes of at most 8 bits
    plan->base = lo;
    plan->npass = np;
    plan->width = (bits + np - 1) / np;
  }
}

__device__ __forceinline__ uint32_t sort_digit(int64_t key, int64_t base, int shift, uint32_t mask) {
  return static_cast<uint32_t>((static_cast<uint64_t>(key) - static_cast<uint64_t>(base)) >> shift) & mask;
}

__global__ __launch_bounds__(kSortBlock, 8) void k_sort_hist(const SortPlan *plan, int pass, const int64_t *keys,
                                                            const int64_t *d_count, int64_t cap, RangeCounts counts) {
  __shared__ uint32_t s_h[kRangeDigits];
  int64_t part, t0, t1;
  if (pass >= plan->npass) return;
  const int64_t n = sort_count(d_count, cap), base = plan->base;
  if (!range_of_block(n, kSortTile, part, t0, t1)) return;
  const int tid = static_cast<int>(threadIdx.x), width = plan->width, shift = pass * width;
  const uint32_t mask = (1u << width) - 1;
  if (tid < kRangeDigits) s_h[tid] = 0;
  __syncthreads();
  const int64_t hi = t1 * kSortTile < n ? t1 * kSortTile : n;
  constexpr int U = 8;
  for (int64_t i0 = t0 * kSortTile + tid; i0 < hi; i0 += kSortBlock * U) {
    int64_t k[U];
#pragma unroll
    for (int u = 0; u < U; ++u) k[u] = keys[i0 + u * kSortBlock < hi ? i0 + u * kSortBlock : i0];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * kSortBlock < hi) atomicAdd(&s_h[sort_digit(k[u], base, shift, mask)], 1u);
  }
  __syncthreads();
  if (tid < kRangeDigits) {
    counts.of_part(part)[tid] = s_h[tid];
    if (s_h[tid]) atomicAdd(&counts.of_group(pass, part / kRangeGroup)[tid], s_h[tid]);
  }
}

// Ranks a wave's ITEMS rows by digit (stable) into pos[] = rank within (wave,
// digit), counting the wave's rows per digit in cnt[].
// Items at or past `used` (wave-uniform) hold nothing.
template <int ITEMS>
__device__ __forceinline__ void rank_digits(const uint32_t (&dig)[ITEMS], const bool (&ok)[ITEMS], int width, int32_t *cnt,
                                            int32_t (&pos)[ITEMS], int used = ITEMS) {
  const int lane = lane_id();
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    if (j >= used) break;
    const uint64_t vm = __ballot(ok[j]);
    const uint64_t peers = match_peers(dig[j], vm, width);
    const int32_t at = ok[j] ? cnt[dig[j]] : 0;
    pos[j] = at + static_cast<int32_t>(mbcnt(peers));
    if (ok[j] && lane == __ffsll(static_cast<unsigned long long>(peers)) - 1) cnt[dig[j]] = at + __popcll(peers);
  }
}

// One pass over a block's range of tiles.  Two blocks of 16 waves per CU.
__global__ __launch_bounds__(kSortBlock, 8) void k_sort_move(const SortPlan *plan, int pass, const int64_t *skeys,
                                                            const int64_t *svals, int64_t *dkeys, int64_t *dvals,
                                                            const int64_t *d_count, int64_t cap, RangeCounts counts) {
  __shared__ int32_t s_cnt[kSortWaves][kRangeDigits];
  __shared__ int64_t s_next[kRangeDigits];  // where the range's next pair of each digit goes
  __shared__ int32_t s_start[kRangeDigits];
  __shared__ RangeOffsets s_off;
  __shared__ uint8_t s_dig[kSortTile];
  __shared__ int64_t s_stage[kSortTile];
  int64_t part, t0, t1;
  if (pass >= plan->npass) return;
  const int64_t n = sort_count(d_count, cap), base = plan->base;
  if (!range_of_block(n, kSortTile, part, t0, t1)) return;
  const int tid = static_cast<int>(threadIdx.x), w = tid / kWave, lane = lane_id();
  range_offsets(counts, pass, static_cast<int>(part), s_off, s_next);
  const int width = plan->width, shift = pass * width;
  const uint32_t mask = (1u << width) - 1;
  for (int64_t t = t0; t < t1; ++t) {  // block-uniform
    for (int i = tid; i < kSortWaves * kRangeDigits; i += kSortBlock) s_cnt[i / kRangeDigits][i % kRangeDigits] = 0;
    int64_t k[kSortItems], v[kSortItems];
    uint32_t dig[kSortItems];
    bool ok[kSortItems];
    int32_t pos[kSortItems];
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
      const int64_t i = t * kSortTile + w * (kWave * kSortItems) + j * kWave + lane;
      ok[j] = i < n;
      k[j] = skeys[ok[j] ? i : n - 1];
      v[j] = svals[ok[j] ? i : n - 1];
    }
    __syncthreads();  // the counters are clear, the previous tile's runs are out
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) dig[j] = sort_digit(k[j], base, shift, mask);
    rank_digits<kSortItems>(dig, ok, width, s_cnt[w], pos);
    __syncthreads();
    int32_t total = 0;
    if (tid < kRangeDigits) {
#pragma unroll
      for (int q = 0; q < kSortWaves; ++q) {
        const int32_t c = s_cnt[q][tid];
        s_cnt[q][tid] = total;
        total += c;
      }
      s_start[tid] = total;
    }
    __syncthreads();
    if (w == 0) {
      int32_t a[4], la = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) la += a[j] = s_start[lane * 4 + j];
      int32_t ra = wave_inclusive_scan(la) - la;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        s_start[lane * 4 + j] = ra;
        s_next[lane * 4 + j] -= ra;  // a pair at LDS position i goes to s_next + i
        ra += a[j];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortItems; ++j)
      if (ok[j]) {
        pos[j] += s_start[dig[j]] + s_cnt[w][dig[j]];
        s_dig[pos[j]] = static_cast<uint8_t>(dig[j]);
        s_stage[pos[j]] = k[j];
      }
    __syncthreads();
    const int rows = static_cast<int>(n - t * kSortTile < kSortTile ? n - t * kSortTile : kSortTile);
    for (int i = tid; i < rows; i += kSortBlock) dkeys[s_next[s_dig[i]] + i] = s_stage[i];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortItems; ++j)
      if (ok[j]) s_stage[pos[j]] = v[j];
    __syncthreads();
    for (int i = tid; i < rows; i += kSortBlock) dvals[s_next[s_dig[i]] + i] = s_stage[i];
    __syncthreads();
    if (tid < kRangeDigits) s_next[tid] += s_start[tid] + total;
  }
}

// Up to kSmallPairs pairs in one block: keys and their 16-bit positions change
// places in LDS, pass by pass; the values are read once at the end, in order.
__global__ __launch_bounds__(kSortBlock) void k_sort_small(int64_t *keys, int64_t *vals, const int64_t *d_count, int64_t cap) {
  __shared__ int32_t s_cnt[kSortWaves][kRangeDigits];
  __shared__ int32_t s_start[kRangeDigits];
  __shared__ int64_t s_key[kSmallPairs];
  __shared__ uint16_t s_idx[kSmallPairs];
  __shared__ int64_t s_lo[kSortWaves], s_hi[kSortWaves];
  const int n = static_cast<int>(sort_count(d_count, cap) <= kSmallPairs ? sort_count(d_count, cap) : 0);
  if (n < 2) return;
  const int tid = static_cast<int>(threadIdx.x), w = tid / kWave, lane = lane_id();
  const int per = (n + kSortBlock - 1) / kSortBlock;  // items in use
  int64_t k[kSmallItems];
  uint16_t x[kSmallItems];
  bool ok[kSmallItems];
  int64_t lo = INT64_MAX, hi = INT64_MIN;
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const int i = w * (kWave * per) + j * kWave + lane;  // a wave's items are consecutive
    ok[j] = j < per && i < n;
    x[j] = static_cast<uint16_t>(ok[j] ? i : n - 1);
    k[j] = keys[x[j]];
    lo = k[j] < lo ? k[j] : lo;
    hi = k[j] > hi ? k[j] : hi;
  }
  block_key_range(lo, hi, s_lo, s_hi, kSortWaves);
  const int bits = range_bits(lo, hi), np = (bits + 7) / 8, width = (bits + np - 1) / np;
  const uint32_t mask = (1u << width) - 1;
  for (int p = 0; p < np; ++p) {
    for (int i = tid; i < kSortWaves * kRangeDigits; i += kSortBlock) s_cnt[i / kRangeDigits][i % kRangeDigits] = 0;
    __syncthreads();  // also: the previous pass's exchange has been read
    uint32_t dig[kSmallItems];
    int32_t pos[kSmallItems];
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) dig[j] = sort_digit(k[j], lo, p * width, mask);
    rank_digits<kSmallItems>(dig, ok, width, s_cnt[w], pos, per);
    __syncthreads();
    if (tid < kRangeDigits) {
      int32_t total = 0;
#pragma unroll
      for (int q = 0; q < kSortWaves; ++q) {
        const int32_t c = s_cnt[q][tid];
        s_cnt[q][tid] = total;
        total += c;
      }
      s_start[tid] = total;
    }
    __syncthreads();
    if (w == 0) {
      int32_t a[4], la = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) la += a[j] = s_start[lane * 4 + j];
      int32_t ra = wave_inclusive_scan(la) - la;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        s_start[lane * 4 + j] = ra;
        ra += a[j];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j)
      if (ok[j]) {
        const int q = pos[j] + s_start[dig[j]] + s_cnt[w][dig[j]];
        s_key[q] = k[j];
        s_idx[q] = x[j];
      }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j)
      if (ok[j]) {
        const int i = w * (kWave * per) + j * kWave + lane;
        k[j] = s_key[i];
        x[j] = s_idx[i];
      }
  }
  int64_t v[kSmallItems];
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) v[j] = vals[x[j]];
  __syncthreads();  // every value is read before any is replaced
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j)
    if (ok[j]) {
      const int i = w * (kWave * per) + j * kWave + lane;
      keys[i] = k[j];
      vals[i] = v[j];
    }
}

// The first min(*d_count, cap) pairs of keys/vals sorted by key, in place.
// key_bits: the keys span at most 2^key_bits values (32 for int32 keys).
pyst_status sort_pairs_by_key(pyst_ctx *ctx, int64_t *keys, int64_t *vals, const int64_t *d_count, int64_t cap,
                              int key_bits, hipStream_t stream) {
  if (cap <= 0) return PYST_OK;
  if (cap > kSmallPairs) {
    const int parts = range_parts(cap, kSortTile);
    const int passes = (key_bits + 15) / 16 * 2;
    Scratch tmp(ctx, 2 * static_cast<size_t>(cap) * sizeof(int64_t), stream);
    Scratch st(ctx, 256 + 2 * parts * sizeof(int64_t) + range_count_words(parts, passes) * sizeof(uint32_t), stream);
    if (!tmp.p || !st.p) return set_error(PYST_ERR_NOMEM, "sort: arena exhausted");
    SortPlan *plan = st.as<SortPlan>();
    int64_t *lo = reinterpret_cast<int64_t *>(static_cast<char *>(st.p) + 256), *hi = lo + parts;
    const RangeCounts counts = range_counts_at(hi + parts, parts);
    k_sort_range<<<parts, 256, 0, stream>>>(keys, d_count, cap, lo, hi, counts, passes);
    PYST_LAUNCH_CHECK("k_sort_range");
    k_sort_plan<<<1, kSortBlock, 0, stream>>>(plan, d_count, cap, lo, hi, parts);
    PYST_LAUNCH_CHECK("k_sort_plan");
    int64_t *bk[2] = {keys, tmp.as<int64_t>()}, *bv[2] = {vals, tmp.as<int64_t>() + cap};
    for (int p = 0; p < passes; ++p) {
      k_sort_hist<<<parts, kSortBlock, 0, stream>>>(plan, p, bk[p & 1], d_count, cap, counts);
      PYST_LAUNCH_CHECK("k_sort_hist");
      k_sort_move<<<parts, kSortBlock, 0, stream>>>(plan, p, bk[p & 1], bv[p & 1], bk[~p & 1], bv[~p & 1], d_count, cap,
                                                   counts);
      PYST_LAUNCH_CHECK("k_sort_move");
    }
  }
  k_sort_small<<<1, kSortBlock, 0, stream>>>(keys, vals, d_count, cap);
  PYST_LAUNCH_CHECK("k_sort_small");
  return PYST_OK;
}

}  // namespace pyst
