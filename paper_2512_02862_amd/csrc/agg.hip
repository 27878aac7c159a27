// Group-by SUM over materialized (key, value) pairs by hash partitioning and
// LDS aggregation.
//
// A hash table in HBM takes two L2 atomics per pair (claim the key, add the
// value), and random atomics on MI355X retire at about 23e9/s chip-wide, so 12M
// pairs cost a millisecond however the table is laid out.  Here the pairs are
// moved twice, 64 ways each time, by 6 bits of a hash of the key: one counting
// pass gives every first-move block's count per final bucket, two exclusive
// scans turn them into both moves' positions, then the first move splits all
// pairs and the second splits each of the 64 parts, so that pairs end in 4096
// contiguous buckets.  One block per bucket then adds its pairs up in
// an LDS hash table (indexed by low bits of the same hash) and writes out the
// groups.  64 ways keep every block's writes to a bucket in a few active lines
// that the L2 combines; one 4096-way move would write 8-byte fragments.
#include "pyst_internal.h"
#include "table.h"

namespace pyst {

constexpr int kAggBlock = 1024;
constexpr int kRadixLg = 6;
constexpr int kRadix = 1 << kRadixLg;
constexpr int kAggBuckets = kRadix * kRadix;   // 4096 buckets after two moves
constexpr int kAggSlotsLg = 13;
constexpr int kAggSlots = 1 << kAggSlotsLg;    // LDS table: 8192 x 16 bytes = 128 KiB per bucket
constexpr int kAggBlocks1 = 512;               // blocks of the first move
constexpr int kAggBlocks2 = 8;                 // blocks per part in the second move
constexpr uint64_t kAggSeed = 0xd6e8feb86659fd93ull;

__device__ __forceinline__ uint64_t agg_hash(int64_t key) { return fmix64(static_cast<uint64_t>(key) ^ kAggSeed); }

// ---------------------------------------------------------------- plan by key range
// A pass over the keys finds their least and greatest value (k_key_range), and
// one block chooses from them how the rows are grouped (k_gb_plan), on the
// device, so nothing is read back:
//   kGbSmall  the keys span at most `small_max` (<= 8192) values: every block
//             adds its rows up in an LDS array indexed by key - kmin and a
//             second kernel adds the blocks' arrays up: the rows are read once
//             more and never moved.  The rule is the LDS: 8192 sums and flags
//             are 72 KiB, two 1024-thread blocks per CU.
//   kGbRange  they span at most 4096 buckets of 8192 values, and a sample finds
//             no crowded bucket or part: the moves split the rows by (key -
//             kmin) >> shift instead of by hash bits, so that a bucket's LDS
//             array is indexed directly (no probing, no compare-and-swap) and
//             the groups come out in key order (no sort).
//   kGbOnce   the same for int32 keys and values that span at most 1024 buckets of
//             16384 values: one move, of 8-byte pairs, does (see k_once_move).
//   kGbFew    the sample finds few different keys, over any range: a table in HBM
//             behind an LDS table per block (gb_insert_rows).  The sample promises
//             nothing: a table that runs full sends the rows on to kGbHash.
//             Every block adds its own table's groups to the one in HBM, so this
//             wants 2048 rows a group (2M rows, int64 keys, against hash buckets:
//             300 groups 144 and 193 us, 900 189 and 200, 1400 224 and 199; 20M
//             into 1400 419 and 770), and room in the blocks' 4096 LDS slots
//             (20M into 2800: 2770 us, 748 hashed).  The same for few rows, which only
//             the device knows of a selection: up to half of the table's slots where
//             nothing else but hash buckets is left (10000 of 20M rows, 64-bit keys
//             over 2^40: 471 -> 64 us, 566 -> 160 ordered), and instead of the moves up
//             to 8192 (whose groups one block sorts; 5000 of 1.1M, 64-bit keys over
//             275000: 94 -> 48, 126 -> 104 ordered) or 1024 of one move (5000 ordered:
//             89 by one move, 98 so).
//   kGbHash   otherwise: hash buckets, each summed in an LDS hash table.
//   kGbTable  the same where hash buckets have no memory or too many groups: the
//             table in HBM (k_gb_insert).
// Measured at 60M rows, start to end, ordered by key: 2407 int32 keys with int64
// values 1953 -> 216 us (kGbSmall: 135 us for the sums, 5.3 TB/s; hash buckets
// left 2407 busy blocks of uneven size), 15M int32 keys with int32 values 2232
// -> 580 us (kGbOnce; 840 with the two moves of kGbRange, whose bucket sums take
// 193 us against 376 with hash tables; nothing is left to sort).  The range costs
// 49 - 66 us there.
constexpr int kDirectSlotsLg = 13;
constexpr int kDirectSlots = 1 << kDirectSlotsLg;  // LDS sums of one direct-addressed table
constexpr int kSamples = 16384;
constexpr int kOnceBuckets = 1024;
constexpr int kOnceShift = 14, kOnceSlots = 1 << kOnceShift;  // LDS sums of one bucket: 128 KiB and 16 KiB of flags
constexpr int kFewKeys = 1500;                    // different keys of the sample, at most
constexpr int64_t kFewRows = 2048;                // rows per different key, at least
constexpr int64_t kFewSlots = int64_t{1} << 16;   // slots of the table in HBM
constexpr int64_t kFewRowsMoves = 8192, kFewRowsOnce = 1024;  // rows that take it instead of two moves, of one

__device__ __forceinline__ bool plan_moves(const GbPlan *p) {
  return !p || plan_mode(p) == kGbHash || plan_mode(p) == kGbRange;
}

// Bucket of a key for both moves: 12 bits, the first move takes the upper 6.
// (Wave-uniform choice; kernels that never see a plan compile it out.)
struct BucketFn {
  int64_t kmin = 0;
  int32_t shift = 0;
  bool ranged = false;
  __device__ __forceinline__ explicit BucketFn(const GbPlan *p) {
    if (p && p->mode == kGbRange) {
      ranged = true;
      kmin = p->kmin;
      shift = p->shift;
    }
  }
  __device__ __forceinline__ uint32_t of_range(int64_t key) const {
    return static_cast<uint32_t>((static_cast<uint64_t>(key) - static_cast<uint64_t>(kmin)) >> shift);
  }
  __device__ __forceinline__ uint32_t wide(int64_t key) const {
    return ranged ? of_range(key) : static_cast<uint32_t>(agg_hash(key) >> (64 - 2 * kRadixLg));
  }
};

// The rows a block of a move reads: with b = xcd_block(blockIdx.x), segment b / bps of the input
// (segment s is [seg_off[s * seg_stride], seg_off[(s + 1) * seg_stride]), or the
// whole input [0, min(*count, cap)) without seg_off), split evenly into bps parts.
struct MoveArgs {
  const int64_t *keys;
  const int64_t *vals;
  const int64_t *count;
  int64_t cap;
  const int32_t *seg_off;
  int seg_stride;
  int bps;
  int sub;  // destination = (bucket >> sub) & (kRadix - 1)
  // With `aligned`, block part of segment seg reads the rows that the first
  // move's blocks [part * G, (part + 1) * G) wrote to it, G = seg_stride / bps
  // (their counts are known from the first pass), instead of an even split.
  int aligned = 0;
  // With kcol set, the pairs are read from the caller's columns instead: pair i
  // is row row_of(sel, i) of (kcol, vcol), int64 or int32 (sign-extended), and
  // an EMPTY key is latched in err (and skipped like any EMPTY key).
  const void *kcol = nullptr;
  const void *vcol = nullptr;
  const int32_t *sel = nullptr;
  int k64 = 0, v64 = 0;
  uint32_t *err = nullptr;
  GbPlan *plan = nullptr;  // null: hash buckets
};

__device__ __forceinline__ int64_t move_key(const MoveArgs &m, int64_t i) {
  return m.kcol ? load_as_i64(m.kcol, m.k64, row_of(m.sel, i)) : m.keys[i];
}

__device__ __forceinline__ int64_t move_val(const MoveArgs &m, int64_t i) {
  return m.kcol ? load_as_i64(m.vcol, m.v64, row_of(m.sel, i)) : m.vals[i];
}

__device__ __forceinline__ void move_range(const MoveArgs &m, int *seg, int *part, int64_t *lo, int64_t *hi) {
  const int blk = static_cast<int>(xcd_block(blockIdx.x, gridDim.x));  // neighbouring ranges on one XCD
  *seg = blk / m.bps;
  *part = blk % m.bps;
  int64_t a, b;
  if (m.seg_off && m.aligned) {
    const int g = m.seg_stride / m.bps;
    *lo = m.seg_off[int64_t{*seg} * m.seg_stride + int64_t{*part} * g];
    *hi = m.seg_off[int64_t{*seg} * m.seg_stride + int64_t{*part + 1} * g];
    return;
  }
  if (m.seg_off) {
    a = m.seg_off[int64_t{*seg} * m.seg_stride];
    b = m.seg_off[int64_t{*seg + 1} * m.seg_stride];
  } else {
    a = 0;
    b = *m.count < m.cap ? *m.count : m.cap;
  }
  const int64_t per = (b - a + m.bps - 1) / m.bps;
  *lo = a + per * *part;
  *hi = *lo + per < b ? *lo + per : b;
  if (*lo > b) *lo = b;
}

// Pairs a thread of the counting pass takes per round, all loads first.
constexpr int kMoveItems = 8;

// Per first-move block: counts of its pairs in each of the 4096 final buckets
// (top 12 bits of the hash: the first move's 6 and the second's 6), from
// which both moves' positions follow (k_narrow_counts), so the second move
// needs no counting pass of its own.
template <bool PLANNED>
__global__ __launch_bounds__(kAggBlock) void k_move_hist_both(MoveArgs m, int32_t *counts) {
  __shared__ int32_t s_c[kAggBuckets];
  if (PLANNED && !plan_moves(m.plan)) return;
  const BucketFn bucket(PLANNED ? m.plan : nullptr);
  for (int i = threadIdx.x; i < kAggBuckets; i += kAggBlock) s_c[i] = 0;
  __syncthreads();
  int seg, part;
  int64_t lo, hi;
  move_range(m, &seg, &part, &lo, &hi);
  for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += int64_t{kAggBlock} * kMoveItems) {
    int64_t k[kMoveItems];
#pragma unroll
    for (int u = 0; u < kMoveItems; ++u) {
      const int64_t i = i0 + int64_t{u} * kAggBlock;
      k[u] = i < hi ? move_key(m, i) : kEmpty64;
      if (m.kcol && i < hi && k[u] == kEmpty64) latch(m.err, kErrKey);
    }
#pragma unroll
    for (int u = 0; u < kMoveItems; ++u)
      if (k[u] != kEmpty64) atomicAdd(&s_c[bucket.wide(k[u])], 1);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kAggBuckets; i += kAggBlock) counts[(int64_t{seg} * m.bps + part) * kAggBuckets + i] = s_c[i];
}

// Writes each block's pairs to its positions (pos: the exclusive scan of the
// per-(segment, bucket, block) counts, in that order).  A tile of kMoveTile pairs is ranked by bucket in LDS
// (per-bucket counts with LDS atomics, one scan over kRadix buckets), laid out
// bucket-major in LDS, and written so that consecutive threads write
// consecutive slots of each bucket's run: every bucket's pairs of a tile leave
// in one contiguous piece (about 512 bytes) instead of as 8-byte fragments.
constexpr int kMoveTileItems = 4;
static_assert(kRadix == kWave, "one wave scans the bucket counts");
constexpr int kMoveTile = kAggBlock * kMoveTileItems;
template <bool PLANNED>
__global__ __launch_bounds__(kAggBlock) void k_move_scatter(MoveArgs m, const int32_t *pos, int64_t *okeys,
                                                           int64_t *ovals) {
  __shared__ int64_t s_k[kMoveTile];
  __shared__ int64_t s_v[kMoveTile];
  __shared__ uint8_t s_b[kMoveTile];
  __shared__ int32_t s_base[kRadix], s_cnt[kRadix], s_off[kRadix + 1];
  if (PLANNED && !plan_moves(m.plan)) return;
  const BucketFn bucket(PLANNED ? m.plan : nullptr);
  int seg, part;
  int64_t lo, hi;
  move_range(m, &seg, &part, &lo, &hi);
  const int tid = static_cast<int>(threadIdx.x);
  if (tid < kRadix) s_base[tid] = pos[(int64_t{seg} * kRadix + tid) * m.bps + part];
  for (int64_t t0 = lo; t0 < hi; t0 += kMoveTile) {  // block-uniform
    if (tid < kRadix) s_cnt[tid] = 0;
    __syncthreads();
    int64_t k[kMoveTileItems], v[kMoveTileItems];
    int bk[kMoveTileItems], rk[kMoveTileItems];
#pragma unroll
    for (int u = 0; u < kMoveTileItems; ++u) {
      const int64_t i = t0 + int64_t{u} * kAggBlock + tid;
      k[u] = i < hi ? move_key(m, i) : kEmpty64;
      v[u] = i < hi ? move_val(m, i) : 0;
    }
#pragma unroll
    for (int u = 0; u < kMoveTileItems; ++u) {
      bk[u] = k[u] != kEmpty64 ? static_cast<int>((bucket.wide(k[u]) >> m.sub) & (kRadix - 1)) : -1;
      rk[u] = bk[u] >= 0 ? atomicAdd(&s_cnt[bk[u]], 1) : 0;
    }
    __syncthreads();
    if (tid < kWave) {  // one wave: exclusive scan of the kRadix (= 64) counts
      const int c = s_cnt[tid];
      const int incl = wave_inclusive_scan(c);
      s_off[tid] = incl - c;
      if (tid == kWave - 1) s_off[kRadix] = incl;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kMoveTileItems; ++u)
      if (bk[u] >= 0) {
        const int p = s_off[bk[u]] + rk[u];
        s_k[p] = k[u];
        s_v[p] = v[u];
        s_b[p] = static_cast<uint8_t>(bk[u]);
      }
    __syncthreads();
    const int n = s_off[kRadix];
    for (int t = tid; t < n; t += kAggBlock) {
      const int b = s_b[t];
      const int64_t o = int64_t{s_base[b]} + (t - s_off[b]);
      okeys[o] = s_k[t];
      ovals[o] = s_v[t];
    }
    __syncthreads();
    if (tid < kRadix) s_base[tid] += s_cnt[tid];
  }
}

// Adds up the pairs of each final bucket in an LDS hash table (indexed by low
// bits of the key hash) and writes out its groups.  One block per CU walks its
// buckets (blockIdx.x, + gridDim.x, ...): the table is cleared as it is written
// out, and the next bucket's first pairs are loaded before the block waits for
// the output position of the current one (one counter atomic per bucket), so a
// bucket costs about one memory round trip.  *d_ngroups must be zero on entry.
__global__ __launch_bounds__(kAggBlock) void k_bucket_groups(const int64_t *keys, const int64_t *vals,
                                                            const int32_t *pos, int bps, int64_t *out_keys,
                                                            int64_t *out_sums, int64_t out_cap, int64_t *d_ngroups,
                                                            uint32_t *err, const GbPlan *plan) {
  if (plan && plan_mode(plan) != kGbHash) return;
  __shared__ uint64_t s_key[kAggSlots];
  __shared__ uint64_t s_sum[kAggSlots];
  __shared__ int32_t s_w[kAggBlock / kWave];
  __shared__ int64_t s_base;
  constexpr int U = 4;  // pairs per thread per round, loaded before any insert
  constexpr int PER = kAggSlots / kAggBlock;  // each thread counts, writes out and clears PER consecutive slots
  const int tid = static_cast<int>(threadIdx.x);
  for (int s = tid; s < kAggSlots; s += kAggBlock) {
    s_key[s] = static_cast<uint64_t>(kEmpty64);
    s_sum[s] = 0;
  }
  bool full = false;
  int64_t kk[U], vv[U];  // the first round of the bucket about to be added up
  auto load_round = [&](int64_t i0, int64_t hi) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + int64_t{u} * kAggBlock;
      kk[u] = i < hi ? keys[i] : kEmpty64;
      vv[u] = i < hi ? vals[i] : 0;
    }
  };
  auto insert_round = [&]() {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (kk[u] == kEmpty64) continue;
      uint32_t s = static_cast<uint32_t>(agg_hash(kk[u])) & (kAggSlots - 1);
      for (int probes = 0;; ++probes) {
        if (probes == kAggSlots) {
          full = true;
          break;
        }
        const uint64_t old = atomicCAS(reinterpret_cast<unsigned long long *>(&s_key[s]),
                                       static_cast<unsigned long long>(kEmpty64), static_cast<unsigned long long>(kk[u]));
        if (old == static_cast<uint64_t>(kEmpty64) || old == static_cast<uint64_t>(kk[u])) {
          atomicAdd(reinterpret_cast<unsigned long long *>(&s_sum[s]), static_cast<unsigned long long>(vv[u]));
          break;
        }
        s = (s + 1) & (kAggSlots - 1);
      }
    }
  };
  int b = static_cast<int>(blockIdx.x);
  if (b < kAggBuckets) load_round(pos[int64_t{b} * bps] + tid, pos[int64_t{b + 1} * bps]);
  __syncthreads();  // the cleared table
  for (; b < kAggBuckets; b += static_cast<int>(gridDim.x)) {  // block-uniform
    const int64_t lo = pos[int64_t{b} * bps], hi = pos[int64_t{b + 1} * bps];
    insert_round();
    for (int64_t i0 = lo + tid + int64_t{kAggBlock} * U; i0 < hi; i0 += int64_t{kAggBlock} * U) {  // large buckets
      load_round(i0, hi);
      insert_round();
    }
    __syncthreads();
    const int s0 = tid * PER;
    int c = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) c += s_key[s0 + j] != static_cast<uint64_t>(kEmpty64);
    const int incl = wave_inclusive_scan(c);
    const int w = tid / kWave;
    if (lane_id() == kWave - 1) s_w[w] = incl;
    __syncthreads();
    // the next bucket's first round goes out before the wait for this one's position
    const int nb = b + static_cast<int>(gridDim.x);
    if (nb < kAggBuckets) load_round(pos[int64_t{nb} * bps] + tid, pos[int64_t{nb + 1} * bps]);
    if (tid == 0) {
      int64_t tot = 0;
      for (int k = 0; k < kAggBlock / kWave; ++k) tot += s_w[k];
      s_base = tot ? static_cast<int64_t>(atomicAdd(reinterpret_cast<unsigned long long *>(d_ngroups),
                                                    static_cast<unsigned long long>(tot)))
                   : 0;
    }
    __syncthreads();
    int64_t p = s_base + incl - c;
    for (int k = 0; k < w; ++k) p += s_w[k];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const uint64_t k = s_key[s0 + j];
      if (k == static_cast<uint64_t>(kEmpty64)) continue;
      if (p < out_cap) {
        out_keys[p] = static_cast<int64_t>(k);
        out_sums[p] = static_cast<int64_t>(s_sum[s0 + j]);
      } else {
        latch(err, kErrCapacity);
      }
      ++p;
      s_key[s0 + j] = static_cast<uint64_t>(kEmpty64);
      s_sum[s0 + j] = 0;
    }
    __syncthreads();  // the table is clear (and s_base read) before the next bucket
  }
  if (full) latch(err, kErrTableFull);
}

// Groups of the pairs [0, min(*count, cap)) of keys/vals (kEmpty64 keys are
// skipped) into out_keys/out_sums, their number into *d_ngroups (which must be
// zero on entry).  keys/vals are overwritten (they hold the second move).
// Fewer than 2^31 pairs; a bucket may hold at most kAggSlots distinct keys
// (about 8192 x 4096 keys in all for keys that hash evenly), else the table-full
// error is latched.
// The moves and the bucket pass; the first move reads `first` (pairs or columns),
// the second writes keys/vals (cap entries each).
// With first.plan, `status` holds kAggBuckets look-back words (cleared by k_gb_plan).
// Without hash_buckets the plan does not choose them.
__global__ void k_narrow_counts(const int32_t *counts, int32_t *c1, int32_t *c2, const GbPlan *plan);
__global__ void k_move_positions(const int32_t *c1, int32_t *p1, const int32_t *c2, int32_t *p2, const GbPlan *plan);
template <bool NARROW>
pyst_status launch_direct_groups(pyst_ctx *ctx, GbPlan *plan, uint64_t *status, const void *pairs, const int64_t *vals,
                                 const int32_t *pos, int bps, int64_t *out_keys, int64_t *out_sums, int64_t out_cap,
                                 int64_t *d_ngroups, hipStream_t stream);

// Scratch of the wide moves: the counts, then the first move's pairs.
static size_t wide_count_bytes() {
  const int64_t n1 = int64_t{kRadix} * kAggBlocks1, n2 = int64_t{kAggBuckets} * kAggBlocks2;
  return ((static_cast<size_t>(kAggBlocks1) * kAggBuckets + static_cast<size_t>(n1 + 1 + n2 + 1) * 2) * sizeof(int32_t) +
          255) / 256 * 256;
}
static size_t wide_groupby_bytes(int64_t cap) { return wide_count_bytes() + static_cast<size_t>(cap) * 16; }

pyst_status pair_groupby_from(pyst_ctx *ctx, MoveArgs first, int64_t *keys, int64_t *vals, const int64_t *count,
                              int64_t cap, int64_t *out_keys, int64_t *out_sums, int64_t out_cap,
                              int64_t *d_ngroups, uint64_t *status, void *ws, bool hash_buckets, hipStream_t stream) {
  if (cap >= (int64_t{1} << 31)) return set_error(PYST_ERR_ARG, "group-by: too many pairs");
  const int64_t n1 = int64_t{kRadix} * kAggBlocks1, n2 = int64_t{kAggBuckets} * kAggBlocks2;
  const size_t counts = wide_count_bytes();
  int32_t *cnt = static_cast<int32_t *>(ws);
  int32_t *h1 = cnt + static_cast<int64_t>(kAggBlocks1) * kAggBuckets, *p1 = h1 + n1 + 1, *h2 = p1 + n1 + 1,
          *p2 = h2 + n2 + 1;
  int64_t *tk = reinterpret_cast<int64_t *>(static_cast<char *>(ws) + counts);
  int64_t *tv = tk + cap;
  // One counting pass over all pairs gives every first-move block's counts
  // per final bucket; the first move's positions are per part (hash bits
  // 58..63), the second's per bucket (bits 52..57) and second-move block.
  MoveArgs m1 = first;
  m1.count = count;
  m1.cap = cap;
  m1.seg_off = nullptr;
  m1.seg_stride = 0;
  m1.bps = kAggBlocks1;
  m1.sub = kRadixLg;
  first.plan ? k_move_hist_both<true><<<kAggBlocks1, kAggBlock, 0, stream>>>(m1, cnt)
             : k_move_hist_both<false><<<kAggBlocks1, kAggBlock, 0, stream>>>(m1, cnt);
  PYST_LAUNCH_CHECK("k_move_hist_both");
  k_narrow_counts<<<static_cast<unsigned>(ceil_div(n1 + n2 + 1, 256)), 256, 0, stream>>>(cnt, h1, h2, first.plan);
  PYST_LAUNCH_CHECK("k_narrow_counts");
  k_move_positions<<<2, kAggBlock, 0, stream>>>(h1, p1, h2, p2, first.plan);
  PYST_LAUNCH_CHECK("k_move_positions");
  first.plan ? k_move_scatter<true><<<kAggBlocks1, kAggBlock, 0, stream>>>(m1, p1, tk, tv)
             : k_move_scatter<false><<<kAggBlocks1, kAggBlock, 0, stream>>>(m1, p1, tk, tv);
  PYST_LAUNCH_CHECK("k_move_scatter");
  // Second move: block j of part p reads what the first move's blocks
  // [64 j, 64 (j + 1)) wrote to part p, and writes it by bucket into keys/vals.
  MoveArgs m2{tk, tv, count, cap, p1, kAggBlocks1, kAggBlocks2, 0};
  m2.aligned = 1;
  m2.plan = first.plan;
  first.plan ? k_move_scatter<true><<<kRadix * kAggBlocks2, kAggBlock, 0, stream>>>(m2, p2, keys, vals)
             : k_move_scatter<false><<<kRadix * kAggBlocks2, kAggBlock, 0, stream>>>(m2, p2, keys, vals);
  PYST_LAUNCH_CHECK("k_move_scatter");
  const int gblocks = static_cast<int>(std::min<int64_t>(kAggBuckets, std::max(1, ctx_num_cus(ctx))));
  if (hash_buckets) {
    k_bucket_groups<<<gblocks, kAggBlock, 0, stream>>>(keys, vals, p2, kAggBlocks2, out_keys, out_sums, out_cap,
                                                       d_ngroups, ctx_err_word(ctx), first.plan);
    PYST_LAUNCH_CHECK("k_bucket_groups");
  }
  if (first.plan) return launch_direct_groups<false>(ctx, first.plan, status, keys, vals, p2, kAggBlocks2, out_keys,
                                                     out_sums, out_cap, d_ngroups, stream);
  return PYST_OK;
}

// ---------------------------------------------------------------- narrow pairs
// Group-by of int32 keys with int32 values: a pair travels as ONE 8-byte word
// (key << 32 | value), half the bytes of the (int64, int64) pairs above, and
// both moves take their counts from one pass over the keys.  The bucket of a
// key is the top 12 bits of a 32-bit hash: bits 26..31 pick its part in the
// first move, bits 20..25 its bucket within the part in the second, bits 0..12
// its LDS slot.  The second move's block j of part p reads exactly the pairs
// that the first move's blocks [j G, (j + 1) G) wrote to part p (G = kNB1 /
// kNB2), so its counts are sums of the first pass's per-block counts and no
// second pass over the pairs is needed to count them.
constexpr int kNB1 = 512;                // blocks of the first move (and of the counting pass)
constexpr int kNB2 = 8;                  // blocks per part in the second move
constexpr int kNG = kNB1 / kNB2;         // first-move blocks behind one second-move block
constexpr int kNItems = 8;               // rows per thread and round of the counting pass
constexpr uint32_t kNarrowSeed = 0x6b43a9b5u;
static_assert(kNB1 % kNB2 == 0, "second-move blocks cover whole groups of first-move blocks");
static_assert(kNB1 == kAggBlocks1 && kNB2 == kAggBlocks2, "the wide pair moves share the count layout");

__device__ __forceinline__ uint32_t narrow_hash(int32_t key) { return fmix32(static_cast<uint32_t>(key) ^ kNarrowSeed); }

struct NarrowArgs {
  const int32_t *kcol;
  const int32_t *vcol;
  const int32_t *sel;    // nullptr: rows 0..count-1
  const int64_t *count;  // rows (or selected rows) to group
  int64_t cap;           // upper bound of *count
  GbPlan *plan;          // null: hash buckets
};

__device__ __forceinline__ uint32_t narrow_bucket(const BucketFn &f, int32_t key) {
  return f.ranged ? f.of_range(key) : narrow_hash(key) >> 20;
}

__device__ __forceinline__ void narrow_range(const NarrowArgs &a, int blk, int nblk, int64_t *lo, int64_t *hi) {
  const int64_t n = *a.count < a.cap ? *a.count : a.cap;
  const int64_t per = (n + nblk - 1) / nblk;
  *lo = per * blk < n ? per * blk : n;
  *hi = *lo + per < n ? *lo + per : n;
}

// Per first-move block: counts of its rows in each of the 4096 buckets.
__global__ __launch_bounds__(kAggBlock) void k_narrow_hist(NarrowArgs a, int32_t *counts) {
  __shared__ int32_t s_c[kAggBuckets];
  if (!plan_moves(a.plan)) return;
  const BucketFn bucket(a.plan);
  for (int i = threadIdx.x; i < kAggBuckets; i += kAggBlock) s_c[i] = 0;
  __syncthreads();
  int64_t lo, hi;
  const int blk = static_cast<int>(xcd_block(blockIdx.x, gridDim.x));  // as k_narrow_move<true>
  narrow_range(a, blk, kNB1, &lo, &hi);
  for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += int64_t{kAggBlock} * kNItems) {
    int32_t k[kNItems];
#pragma unroll
    for (int u = 0; u < kNItems; ++u) {
      const int64_t i = i0 + int64_t{u} * kAggBlock;
      k[u] = i < hi ? a.kcol[row_of(a.sel, i)] : 0;
    }
#pragma unroll
    for (int u = 0; u < kNItems; ++u)
      if (i0 + int64_t{u} * kAggBlock < hi) atomicAdd(&s_c[narrow_bucket(bucket, k[u])], 1);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kAggBuckets; i += kAggBlock) counts[int64_t{blk} * kAggBuckets + i] = s_c[i];
}

// c1[p * kNB1 + b]: rows of first-move block b in part p; c2[(p * 64 + q) * kNB2
// + j]: rows of bucket (p, q) that second-move block j of part p moves.
__global__ void k_narrow_counts(const int32_t *counts, int32_t *c1, int32_t *c2, const GbPlan *plan) {
  if (!plan_moves(plan)) return;
  const int64_t t = blockIdx.x * int64_t{blockDim.x} + threadIdx.x;
  constexpr int64_t n1 = int64_t{kRadix} * kNB1, n2 = int64_t{kAggBuckets} * kNB2;
  if (t < n1) {
    const int p = static_cast<int>(t / kNB1), b = static_cast<int>(t % kNB1);
    int32_t c = 0;
    for (int q = 0; q < kRadix; ++q) c += counts[int64_t{b} * kAggBuckets + p * kRadix + q];
    c1[t] = c;
  } else if (t < n1 + n2) {
    const int64_t u = t - n1;
    const int bucket = static_cast<int>(u / kNB2), j = static_cast<int>(u % kNB2);
    int32_t c = 0;
    for (int b = j * kNG; b < (j + 1) * kNG; ++b) c += counts[int64_t{b} * kAggBuckets + bucket];
    c2[u] = c;
  }
}

// Exclusive scans of both count arrays, one block each; the entry after the
// last is the total.  Every thread holds its 32 counts in registers (eight
// 16-byte loads, tile by tile), so a scan is one memory round trip: 6 us where
// two look-back scans with their cleared status words took 20.
constexpr int kPosLen = kRadix * kNB1;  // entries of c1, and of c2
constexpr int kPosTiles = kPosLen / (4 * kAggBlock);
static_assert(kPosLen == kAggBuckets * kNB2 && kPosLen % (4 * kAggBlock) == 0, "both arrays are whole tiles");
__global__ __launch_bounds__(kAggBlock) void k_move_positions(const int32_t *c1, int32_t *p1, const int32_t *c2,
                                                             int32_t *p2, const GbPlan *plan) {
  constexpr int NW = kAggBlock / kWave;
  __shared__ int32_t s_w[kPosTiles * NW];  // per (tile, wave) sums, then their exclusive prefix
  if (!plan_moves(plan)) return;
  const int32_t *in = blockIdx.x ? c2 : c1;
  int32_t *out = blockIdx.x ? p2 : p1;
  const int tid = static_cast<int>(threadIdx.x), w = tid / kWave, lane = lane_id();
  int32_t v[kPosTiles][4], excl[kPosTiles];
#pragma unroll
  for (int q = 0; q < kPosTiles; ++q)
#pragma unroll
    for (int j = 0; j < 4; ++j) v[q][j] = in[q * 4 * kAggBlock + tid * 4 + j];
#pragma unroll
  for (int q = 0; q < kPosTiles; ++q) {
    const int32_t sum = v[q][0] + v[q][1] + v[q][2] + v[q][3];
    const int32_t incl = wave_inclusive_scan(sum);
    excl[q] = incl - sum;
    if (lane == kWave - 1) s_w[q * NW + w] = incl;
  }
  __syncthreads();
  if (w == 0) {  // kPosTiles * NW = 128 partial sums, two a lane
    static_assert(kPosTiles * NW == 2 * kWave, "two partial sums a lane");
    const int32_t a = s_w[2 * lane], b = s_w[2 * lane + 1];
    const int32_t incl = wave_inclusive_scan(a + b);
    s_w[2 * lane] = incl - a - b;
    s_w[2 * lane + 1] = incl - b;
    if (lane == kWave - 1) out[kPosLen] = incl;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPosTiles; ++q) {
    int32_t run = s_w[q * NW + w] + excl[q];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      out[q * 4 * kAggBlock + tid * 4 + j] = run;
      run += v[q][j];
    }
  }
}

// One move of narrow pairs.  FIRST: block b reads its rows of the columns and
// writes them by part (bits 26..31) at pos1; else block p * kNB2 + j reads the
// pairs of its range of part p and writes them by bucket (bits 20..25) at pos2.
// Each 4096-pair tile is ranked by destination in LDS and every destination's
// pairs of the tile leave as one contiguous run (as k_move_scatter does).
template <bool FIRST>
__global__ __launch_bounds__(kAggBlock) void k_narrow_move(NarrowArgs a, const uint64_t *in, const int32_t *pos1,
                                                          const int32_t *pos2, uint64_t *out) {
  __shared__ uint64_t s_p[kMoveTile];
  __shared__ uint8_t s_b[kMoveTile];
  __shared__ int32_t s_base[kRadix], s_cnt[kRadix], s_off[kRadix + 1];
  if (!plan_moves(a.plan)) return;
  const BucketFn bucket(a.plan);
  const int tid = static_cast<int>(threadIdx.x);
  int64_t lo, hi;
  int part = 0;
  const int blk = static_cast<int>(xcd_block(blockIdx.x, gridDim.x));  // neighbouring ranges on one XCD
  if (FIRST) {
    narrow_range(a, blk, kNB1, &lo, &hi);
    if (tid < kRadix) s_base[tid] = pos1[int64_t{tid} * kNB1 + blk];
  } else {
    part = blk / kNB2;
    const int j = blk % kNB2;
    lo = pos1[int64_t{part} * kNB1 + j * kNG];
    hi = pos1[int64_t{part} * kNB1 + (j + 1) * kNG];
    if (tid < kRadix) s_base[tid] = pos2[(int64_t{part} * kRadix + tid) * kNB2 + j];
  }
  constexpr int sub = FIRST ? kRadixLg : 0;
  for (int64_t t0 = lo; t0 < hi; t0 += kMoveTile) {  // block-uniform
    if (tid < kRadix) s_cnt[tid] = 0;
    __syncthreads();
    uint64_t pr[kMoveTileItems];
    int bk[kMoveTileItems], rk[kMoveTileItems];
#pragma unroll
    for (int u = 0; u < kMoveTileItems; ++u) {
      const int64_t i = t0 + int64_t{u} * kAggBlock + tid;
      if (FIRST) {
        const int64_t r = i < hi ? row_of(a.sel, i) : 0;
        const int32_t k = i < hi ? a.kcol[r] : 0, v = i < hi ? a.vcol[r] : 0;
        pr[u] = (static_cast<uint64_t>(static_cast<uint32_t>(k)) << 32) | static_cast<uint32_t>(v);
      } else {
        pr[u] = i < hi ? in[i] : 0;
      }
    }
#pragma unroll
    for (int u = 0; u < kMoveTileItems; ++u) {
      const int64_t i = t0 + int64_t{u} * kAggBlock + tid;
      bk[u] = i < hi ? static_cast<int>((narrow_bucket(bucket, static_cast<int32_t>(pr[u] >> 32)) >> sub) & (kRadix - 1))
                     : -1;
      rk[u] = bk[u] >= 0 ? atomicAdd(&s_cnt[bk[u]], 1) : 0;
    }
    __syncthreads();
    if (tid < kWave) {
      const int c = s_cnt[tid];
      const int incl = wave_inclusive_scan(c);
      s_off[tid] = incl - c;
      if (tid == kWave - 1) s_off[kRadix] = incl;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kMoveTileItems; ++u)
      if (bk[u] >= 0) {
        const int p = s_off[bk[u]] + rk[u];
        s_p[p] = pr[u];
        s_b[p] = static_cast<uint8_t>(bk[u]);
      }
    __syncthreads();
    const int n = s_off[kRadix];
    for (int t = tid; t < n; t += kAggBlock) {
      const int b = s_b[t];
      out[int64_t{s_base[b]} + (t - s_off[b])] = s_p[t];
    }
    __syncthreads();
    if (tid < kRadix) s_base[tid] += s_cnt[tid];
  }
}

// Inverse of the narrow hash: fmix32 is a bijection (xor-shifts and odd
// multipliers), undone step by step with the multipliers' inverses mod 2^32.
__host__ __device__ constexpr uint32_t inv_odd32(uint32_t c) {
  uint32_t x = c;  // Newton's iteration for the inverse mod 2^32 (c odd): 3, 6, 12, 24, 48 bits
  for (int i = 0; i < 5; ++i) x *= 2u - c * x;
  return x;
}
static_assert(0x85ebca6bu * inv_odd32(0x85ebca6bu) == 1u && 0xc2b2ae35u * inv_odd32(0xc2b2ae35u) == 1u, "inverse");
__device__ __forceinline__ int32_t narrow_unhash(uint32_t h) {
  h ^= h >> 16;
  h *= inv_odd32(0xc2b2ae35u);
  h ^= (h >> 13) ^ (h >> 26);
  h *= inv_odd32(0x85ebca6bu);
  h ^= h >> 16;
  return static_cast<int32_t>(h ^ kNarrowSeed);
}

// Sums every bucket's narrow pairs in an LDS table and writes its groups, one
// block per CU walking the buckets as k_bucket_groups does.  The table holds
// each key's 32-bit hash (slot: its low 13 bits), which identifies the key
// because the hash is a bijection; every hash of bucket b has b as its top 12
// bits, so a hash with other top bits marks an empty slot of that bucket.  A
// slot is read before it is claimed: a key seen before in the bucket costs one
// LDS read and one add instead of a compare-and-swap and an add.  *d_ngroups
// must be zero on entry.
__device__ __forceinline__ uint32_t narrow_empty(int b) { return static_cast<uint32_t>(~b & (kAggBuckets - 1)) << 20; }

__global__ __launch_bounds__(kAggBlock) void k_narrow_groups(const uint64_t *pairs, const int32_t *pos2,
                                                            int64_t *out_keys, int64_t *out_sums, int64_t out_cap,
                                                            int64_t *d_ngroups, uint32_t *err, const GbPlan *plan) {
  if (plan && plan_mode(plan) != kGbHash) return;
  __shared__ uint32_t s_h[kAggSlots];
  __shared__ uint64_t s_sum[kAggSlots];
  __shared__ int32_t s_w[kAggBlock / kWave];
  __shared__ int64_t s_base;
  constexpr int U = 16;  // a whole bucket (14.6k pairs on average at 60M rows) in one round
  constexpr int PER = kAggSlots / kAggBlock;
  const int tid = static_cast<int>(threadIdx.x);
  int b = static_cast<int>(blockIdx.x);
  for (int s = tid; s < kAggSlots; s += kAggBlock) {
    s_h[s] = narrow_empty(b);
    s_sum[s] = 0;
  }
  bool full = false;
  uint64_t pp[U];
  bool have[U];
  auto load_round = [&](int64_t i0, int64_t hi) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + int64_t{u} * kAggBlock;
      have[u] = i < hi;
      pp[u] = have[u] ? pairs[i] : 0;
    }
  };
  // The home slots of all U pairs are read together first; a pair whose key
  // already sits in its home slot (most of them: keys repeat) is added at once,
  // the others walk their runs one by one, claiming an empty slot with a CAS.
  auto insert_round = [&](uint32_t empty) {
    uint32_t h[U], cur[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      h[u] = narrow_hash(static_cast<int32_t>(pp[u] >> 32));
      cur[u] = have[u] ? s_h[h[u] & (kAggSlots - 1)] : 0u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!have[u]) continue;
      const uint64_t val = static_cast<uint64_t>(static_cast<int64_t>(static_cast<int32_t>(pp[u] & 0xffffffffu)));
      uint32_t s = h[u] & (kAggSlots - 1);
      uint32_t c = cur[u];
      for (int probes = 0;; ++probes) {
        if (c == empty) c = atomicCAS(&s_h[s], empty, h[u]);
        if (c == empty || c == h[u]) {
          atomicAdd(reinterpret_cast<unsigned long long *>(&s_sum[s]), static_cast<unsigned long long>(val));
          break;
        }
        if (probes + 1 == kAggSlots) {
          full = true;
          break;
        }
        s = (s + 1) & (kAggSlots - 1);
        c = s_h[s];
      }
    }
  };
  if (b < kAggBuckets) load_round(pos2[int64_t{b} * kNB2] + tid, pos2[int64_t{b + 1} * kNB2]);
  __syncthreads();
  for (; b < kAggBuckets; b += static_cast<int>(gridDim.x)) {  // block-uniform
    const uint32_t empty = narrow_empty(b);
    const int64_t lo = pos2[int64_t{b} * kNB2], hi = pos2[int64_t{b + 1} * kNB2];
    insert_round(empty);
    for (int64_t i0 = lo + tid + int64_t{kAggBlock} * U; i0 < hi; i0 += int64_t{kAggBlock} * U) {
      load_round(i0, hi);
      insert_round(empty);
    }
    __syncthreads();
    // Compact the bucket's groups to the front of the table (each thread holds
    // its PER slots in registers across the barrier), then write them out with
    // consecutive threads on consecutive positions.
    const int s0 = tid * PER;
    uint32_t hh[PER];
    uint64_t ss[PER];
    int c = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      hh[j] = s_h[s0 + j];
      ss[j] = s_sum[s0 + j];
      c += hh[j] != empty;
    }
    const int incl = wave_inclusive_scan(c);
    const int w = tid / kWave;
    if (lane_id() == kWave - 1) s_w[w] = incl;
    __syncthreads();
    const int nb = b + static_cast<int>(gridDim.x);
    if (nb < kAggBuckets) load_round(pos2[int64_t{nb} * kNB2] + tid, pos2[int64_t{nb + 1} * kNB2]);
    int tot = 0, q = incl - c;
    for (int k = 0; k < kAggBlock / kWave; ++k) {
      tot += s_w[k];
      if (k < w) q += s_w[k];
    }
    if (tid == 0)
      s_base = tot ? static_cast<int64_t>(atomicAdd(reinterpret_cast<unsigned long long *>(d_ngroups),
                                                    static_cast<unsigned long long>(tot)))
                   : 0;
#pragma unroll
    for (int j = 0; j < PER; ++j)
      if (hh[j] != empty) {
        s_h[q] = hh[j];
        s_sum[q] = ss[j];
        ++q;
      }
    __syncthreads();
    const int64_t base = s_base;
    for (int i = tid; i < tot; i += kAggBlock) {
      if (base + i < out_cap) {
        out_keys[base + i] = narrow_unhash(s_h[i]);
        out_sums[base + i] = static_cast<int64_t>(s_sum[i]);
      } else {
        latch(err, kErrCapacity);
      }
    }
    __syncthreads();
    const uint32_t next_empty = narrow_empty(nb);
    for (int i = tid; i < kAggSlots; i += kAggBlock) {
      s_h[i] = next_empty;
      s_sum[i] = 0;
    }
    __syncthreads();
  }
  if (full) latch(err, kErrTableFull);
}

// Bytes of scratch narrow_groupby needs for up to `cap` rows.
size_t narrow_groupby_bytes(int64_t cap) {
  const int64_t n1 = int64_t{kRadix} * kNB1, n2 = int64_t{kAggBuckets} * kNB2;
  const size_t counts = static_cast<size_t>(kNB1) * kAggBuckets + 2 * static_cast<size_t>(n1 + 1 + n2 + 1);
  return (counts * sizeof(int32_t) + 255) / 256 * 256 + static_cast<size_t>(cap) * 16 + 256;
}

static pyst_status launch_once(pyst_ctx *ctx, const NarrowArgs &a, void *ws, uint64_t *pairs, uint64_t *status,
                               int64_t *out_keys, int64_t *out_sums, int64_t out_cap, int64_t *d_ngroups, hipStream_t stream);

// GROUP BY key SUM(val) of the rows [0, *count) (of the selection sel) of int32
// columns through narrow pairs, in scratch `ws` of narrow_groupby_bytes(cap).
// *d_ngroups must be zero on entry.  Fewer than 2^31 rows.
pyst_status narrow_groupby(pyst_ctx *ctx, const int32_t *kcol, const int32_t *vcol, const int32_t *sel,
                           const int64_t *count, int64_t cap, void *ws, int64_t *out_keys, int64_t *out_sums,
                           int64_t out_cap, int64_t *d_ngroups, GbPlan *plan, uint64_t *status, bool hash_buckets,
                           hipStream_t stream) {
  if (cap >= (int64_t{1} << 31)) return set_error(PYST_ERR_ARG, "group-by: too many rows");
  const int64_t n1 = int64_t{kRadix} * kNB1, n2 = int64_t{kAggBuckets} * kNB2;
  int32_t *counts = static_cast<int32_t *>(ws);
  int32_t *c1 = counts + static_cast<int64_t>(kNB1) * kAggBuckets, *p1 = c1 + n1 + 1, *c2 = p1 + n1 + 1,
          *p2 = c2 + n2 + 1;
  const size_t cbytes = (static_cast<size_t>(kNB1) * kAggBuckets + 2 * static_cast<size_t>(n1 + 1 + n2 + 1)) *
                        sizeof(int32_t);
  uint64_t *tmp = reinterpret_cast<uint64_t *>(static_cast<char *>(ws) + (cbytes + 255) / 256 * 256);
  uint64_t *pairs = tmp + cap;
  NarrowArgs a{kcol, vcol, sel, count, cap, plan};
  if (plan) {
    const pyst_status st = launch_once(ctx, a, ws, tmp, status, out_keys, out_sums, out_cap, d_ngroups, stream);
    if (st != PYST_OK) return st;
  }
  k_narrow_hist<<<kNB1, kAggBlock, 0, stream>>>(a, counts);
  PYST_LAUNCH_CHECK("k_narrow_hist");
  k_narrow_counts<<<static_cast<unsigned>(ceil_div(n1 + n2 + 1, 256)), 256, 0, stream>>>(counts, c1, c2, plan);
  PYST_LAUNCH_CHECK("k_narrow_counts");
  k_move_positions<<<2, kAggBlock, 0, stream>>>(c1, p1, c2, p2, plan);
  PYST_LAUNCH_CHECK("k_move_positions");
  k_narrow_move<true><<<kNB1, kAggBlock, 0, stream>>>(a, nullptr, p1, p2, tmp);
  PYST_LAUNCH_CHECK("k_narrow_move<1>");
  k_narrow_move<false><<<kRadix * kNB2, kAggBlock, 0, stream>>>(a, tmp, p1, p2, pairs);
  PYST_LAUNCH_CHECK("k_narrow_move<2>");
  const int gblocks = static_cast<int>(std::min<int64_t>(kAggBuckets, std::max(1, ctx_num_cus(ctx))));
  if (hash_buckets) {
    k_narrow_groups<<<gblocks, kAggBlock, 0, stream>>>(pairs, p2, out_keys, out_sums, out_cap, d_ngroups,
                                                       ctx_err_word(ctx), plan);
    PYST_LAUNCH_CHECK("k_narrow_groups");
  }
  if (!plan) return PYST_OK;
  return launch_direct_groups<true>(ctx, plan, status, pairs, nullptr, p2, kNB2, out_keys, out_sums, out_cap, d_ngroups,
                                    stream);
}

pyst_status pair_groupby(pyst_ctx *ctx, int64_t *keys, int64_t *vals, const int64_t *count, int64_t cap,
                         int64_t *out_keys, int64_t *out_sums, int64_t out_cap, int64_t *d_ngroups,
                         hipStream_t stream) {
  MoveArgs first{};
  first.keys = keys;
  first.vals = vals;
  Scratch ws(ctx, wide_groupby_bytes(cap), stream);
  if (!ws.p) return set_error(PYST_ERR_NOMEM, "group-by: arena exhausted");
  return pair_groupby_from(ctx, first, keys, vals, count, cap, out_keys, out_sums, out_cap, d_ngroups, nullptr, ws.p,
                           true, stream);
}

// ---------------------------------------------------------------- planned group-by of columns
// Least and greatest key of the rows (per-block partial results) and a sample
// of the keys at jittered even steps.  One read of the keys bounds it: 16-byte
// loads, four in flight a thread, where there is no selection and the column is
// so aligned (60M int32 keys 49 us, 4.9 TB/s); else 4- or 8-byte loads, eight in
// flight (61 us).  An EMPTY int64 key is latched.  A selection's keys lie in lines
// that other rows share (10M of 20M int64 keys 80 us): where 256 of them already
// span more than any mode takes, their range is left at that (an EMPTY key among
// the others is latched where the rows are read again).
constexpr int kRangeBlocks = 2048, kRangeItems = 8;
constexpr int64_t kPeekRows = int64_t{1} << 19;
__global__ __launch_bounds__(256) void k_key_range(const void *key, int key64, const int32_t *sel, const int64_t *d_nsel,
                                                   int64_t n, int64_t *lo_out, int64_t *hi_out, int64_t *samples,
                                                   GroupDev few, uint64_t *few_status, int64_t few_words, uint32_t *err) {
  __shared__ int64_t s_lo[4], s_hi[4];
  if (few.slots) {  // the table of kGbFew starts empty
    const int64_t g0 = int64_t{blockIdx.x} * 256 + threadIdx.x, step = int64_t{gridDim.x} * 256;
    if (g0 == 0) few.hdr[0] = few.cap_alloc;
    for (int64_t i = g0; i < few.cap_alloc; i += step) {
      few.slots[2 * i] = static_cast<uint64_t>(kEmpty64);
      few.slots[2 * i + 1] = 0;
    }
    for (int64_t i = g0; i < few_words; i += step) few_status[i] = 0;
  }
  int64_t cnt = count_of(d_nsel, n);
  if (cnt > n) cnt = n;
  const int64_t gtid = int64_t{blockIdx.x} * 256 + threadIdx.x;
  if (gtid < kSamples && cnt > 0) {
    const uint64_t jitter = fmix32(static_cast<uint32_t>(gtid) ^ kNarrowSeed) >> 16;
    int64_t i = static_cast<int64_t>(((static_cast<uint64_t>(gtid) << 16) + jitter) * static_cast<uint64_t>(cnt) / (uint64_t{kSamples} << 16));
    samples[gtid] = load_as_i64(key, key64, row_of(sel, i < cnt ? i : cnt - 1));
  }
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  bool bad = false;
  int64_t first = 0;  // rows before it are done
  if (sel && cnt >= kPeekRows) {  // block-uniform, and the same in every block
    const int64_t k = load_as_i64(key, key64, sel[cnt / 256 * static_cast<int>(threadIdx.x)]);
    if (k != kEmpty64) lo = hi = k;
    block_key_range(lo, hi, s_lo, s_hi, 4);
    if (lo <= hi && static_cast<uint64_t>(hi) - static_cast<uint64_t>(lo) >= static_cast<uint64_t>(kAggBuckets) * kDirectSlots) first = cnt;
    __syncthreads();  // s_lo and s_hi are read
  }
  if (!sel && reinterpret_cast<uintptr_t>(key) % 16 == 0) {  // (first is 0)
    // whole 16-byte loads, kRangeItems / 2 in flight a thread
    constexpr int V = kRangeItems / 2;
    const int per = key64 ? 2 : 4;
    const int64_t nv = cnt / per, step = int64_t{gridDim.x} * 256;
    const int4 *kv = static_cast<const int4 *>(key);
    first = nv * per;
    int32_t lo32 = INT32_MAX, hi32 = INT32_MIN;
    for (int64_t v0 = gtid; v0 < nv; v0 += step * V) {
      int4 x[V];
#pragma unroll
      for (int u = 0; u < V; ++u) x[u] = kv[v0 + u * step < nv ? v0 + u * step : v0];
#pragma unroll
      for (int u = 0; u < V; ++u) {
        if (key64) {
          const longlong2 y = __builtin_bit_cast(longlong2, x[u]);
          const int64_t k[2] = {y.x, y.y};
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            if (k[j] == kEmpty64) {
              bad = true;
              continue;
            }
            lo = k[j] < lo ? k[j] : lo;
            hi = k[j] > hi ? k[j] : hi;
          }
        } else {
          lo32 = min(lo32, min(min(x[u].x, x[u].y), min(x[u].z, x[u].w)));
          hi32 = max(hi32, max(max(x[u].x, x[u].y), max(x[u].z, x[u].w)));
        }
      }
    }
    if (!key64 && gtid < nv) {
      lo = lo32;
      hi = hi32;
    }
  }
  for (int64_t i0 = first + gtid; i0 < cnt; i0 += int64_t{gridDim.x} * 256 * kRangeItems) {
    int64_t k[kRangeItems], row[kRangeItems];
#pragma unroll
    for (int u = 0; u < kRangeItems; ++u) {
      const int64_t i = i0 + int64_t{u} * gridDim.x * 256;
      row[u] = i < cnt ? i : i0;
    }
    if (sel) load_items<kRangeItems>(sel, 0, row, cnt, row);
    load_items<kRangeItems>(key, key64, row, n, k);
#pragma unroll
    for (int u = 0; u < kRangeItems; ++u) {
      if (k[u] == kEmpty64) {  // only an int64 column can hold it
        bad = true;
        continue;
      }
      lo = k[u] < lo ? k[u] : lo;
      hi = k[u] > hi ? k[u] : hi;
    }
  }
  if (bad) latch(err, kErrKey);
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
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      lo = s_lo[w] < lo ? s_lo[w] : lo;
      hi = s_hi[w] > hi ? s_hi[w] : hi;
    }
    lo_out[blockIdx.x] = lo;
    hi_out[blockIdx.x] = hi;
  }
}

// One block: reduces the partial ranges, chooses the mode and clears what the
// later kernels start from zero (look-back words, ticket, group count).
// A bucket of the sample with over 1/256 of it, or a part (64 buckets, moved by
// 8 blocks of the second move) with over 1/12, makes the ranged moves and sums
// wait for one block each; such keys take hash buckets.
__global__ __launch_bounds__(kAggBlock) void k_gb_plan(GbPlan *plan, const int64_t *lo_in, const int64_t *hi_in,
                                                      int nblocks, const int64_t *samples, const int64_t *d_nsel,
                                                      int64_t n, int64_t small_max, int allow_range, int allow_once,
                                                      int allow_few, int otherwise, uint64_t *status, int64_t *d_ngroups) {
  __shared__ int32_t s_c[kAggBuckets];
  __shared__ int64_t s_lo[kAggBlock / kWave], s_hi[kAggBlock / kWave];
  __shared__ int32_t s_crowded, s_crowded_once, s_distinct;
  const int tid = static_cast<int>(threadIdx.x);
  for (int i = tid; i < kAggBuckets; i += kAggBlock) {
    s_c[i] = 0;
    status[i] = 0;
  }
  if (tid == 0) s_crowded = s_crowded_once = s_distinct = 0;
  // All that is read, in one round trip (the sample, not held, took ten: 12.6 us in all).
  constexpr int S = kSamples / kAggBlock, B = kRangeBlocks / kAggBlock;
  int64_t sample[S], los[B], his[B];
#pragma unroll
  for (int j = 0; j < B; ++j) {
    const int i = tid + j * kAggBlock;
    los[j] = i < nblocks ? lo_in[i] : INT64_MAX;
    his[j] = i < nblocks ? hi_in[i] : INT64_MIN;
  }
#pragma unroll
  for (int j = 0; j < S; ++j) sample[j] = samples[tid + j * kAggBlock];
  int64_t lo = INT64_MAX, hi = INT64_MIN;
#pragma unroll
  for (int j = 0; j < B; ++j) {
    lo = los[j] < lo ? los[j] : lo;
    hi = his[j] > hi ? his[j] : hi;
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    const int64_t l = __shfl_xor(lo, o), h = __shfl_xor(hi, o);
    lo = l < lo ? l : lo;
    hi = h > hi ? h : hi;
  }
  if (lane_id() == 0) {
    s_lo[tid / kWave] = lo;
    s_hi[tid / kWave] = hi;
  }
  __syncthreads();
  for (int w = 0; w < kAggBlock / kWave; ++w) {
    lo = s_lo[w] < lo ? s_lo[w] : lo;
    hi = s_hi[w] > hi ? s_hi[w] : hi;
  }
  const uint64_t range = lo > hi ? 0 : static_cast<uint64_t>(hi) - static_cast<uint64_t>(lo) + 1;
  const int64_t cnt = std::min(count_of(d_nsel, n), n);
  int32_t mode = otherwise, shift = 0;
  if (range <= static_cast<uint64_t>(small_max)) {
    mode = kGbSmall;
  } else if (allow_few && cnt <= (allow_once ? kFewRowsOnce : kFewRowsMoves)) {  // block-uniform
    mode = kGbFew;
  } else if (allow_range && range <= static_cast<uint64_t>(kAggBuckets) * kDirectSlots) {  // block-uniform
    mode = kGbRange;
    while (((range - 1) >> shift) >= kAggBuckets) ++shift;
#pragma unroll
    for (int j = 0; j < S; ++j) {
      const uint64_t off = static_cast<uint64_t>(sample[j]) - static_cast<uint64_t>(lo);
      if (off < range) atomicAdd(&s_c[off >> shift], 1);
    }
    __syncthreads();
    for (int b = tid; b < kAggBuckets; b += kAggBlock) {
      const int c = s_c[b];
      if (c > kSamples / 256 || wave_sum(c) > kSamples / 12) s_crowded = 1;  // a wave holds one part's 64 buckets
    }
    // kGbOnce: its 1024 buckets are whole groups of these; over 1/128 in one waits for a block
    int once_shift = shift;
    while (((range - 1) >> once_shift) >= kOnceBuckets) ++once_shift;
    if (allow_once && once_shift <= kOnceShift) {  // block-uniform
      const int per = 1 << (once_shift - shift);
      int32_t c = 0;
      for (int j = 0; j < per && tid * per + j < kAggBuckets; ++j) c += s_c[tid * per + j];
      if (c > kSamples / 128) s_crowded_once = 1;
    }
    __syncthreads();
    if (s_crowded) {
      mode = otherwise;
    } else if (allow_once && once_shift <= kOnceShift && !s_crowded_once) {
      mode = kGbOnce;
      shift = once_shift;
    }
  }
  if (mode == otherwise && allow_few && cnt <= kFewSlots / 2) {  // no more groups than rows: the table holds any
    mode = kGbFew;
  } else if (mode == otherwise && allow_few) {  // block-uniform: different keys of the sample, by their hash bits
    constexpr int kBits = kAggBuckets * 32;
    __syncthreads();
    for (int i = tid; i < kAggBuckets; i += kAggBlock) s_c[i] = 0;
    __syncthreads();
    int32_t news = 0;
#pragma unroll
    for (int j = 0; j < S; ++j) {
      const uint32_t h = static_cast<uint32_t>(agg_hash(sample[j])) & (kBits - 1);
      news += !(atomicOr(&s_c[h >> 5], 1 << (h & 31)) >> (h & 31) & 1);
    }
    news = wave_sum(news);
    if (lane_id() == 0) atomicAdd(&s_distinct, news);
    __syncthreads();
    if (s_distinct <= kFewKeys && s_distinct <= cnt / kFewRows) mode = kGbFew;
  }
  if (tid == 0) {
    plan->kmin = lo;
    plan->range = range;
    plan->count = cnt;
    plan->mode = mode;
    plan->shift = shift;
    plan->sort_count = 0;
    plan->few_failed = 0;
    plan->otherwise = otherwise;
    plan->ticket = 0;
    *d_ngroups = 0;
  }
}

// kGbSmall: a block's rows (one contiguous range of them) summed in LDS, then
// written as its partial arrays.  With few keys each lane adds to one of
// `copies` interleaved tables, so that a wave's 64 adds do not all meet in a
// few words.  Bound by the read of the rows (12 bytes each for int32 keys and
// int64 values).
struct SmallLds {
  uint64_t sum[kDirectSlots];
  uint8_t flag[kDirectSlots];
};
__device__ __forceinline__ void small_sums(SmallLds &lds, const void *key, int key64, const void *val, int val64,
                                           const int32_t *sel, int64_t rows, const GbPlan *plan, uint64_t *psum,
                                           uint8_t *pflag) {
  uint64_t *s_sum = lds.sum;
  uint8_t *s_flag = lds.flag;
  if (plan->range == 0) return;
  constexpr int U = 8;
  const int tid = static_cast<int>(threadIdx.x);
  const uint32_t range = static_cast<uint32_t>(plan->range);
  const int64_t kmin = plan->kmin;
  int lgc = 0;  // copies = 1 << lgc
  while (lgc < 4 && (range << (lgc + 1)) <= kDirectSlots) ++lgc;
  for (int i = tid; i < kDirectSlots; i += kAggBlock) {
    s_sum[i] = 0;
    s_flag[i] = 0;
  }
  __syncthreads();
  const int64_t n = plan->count, per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
  const int64_t lo = per * blk < n ? per * blk : n, hi = lo + per < n ? lo + per : n;
  const uint32_t copy = static_cast<uint32_t>(tid) & ((1u << lgc) - 1);
  for (int64_t i0 = lo + tid; i0 < hi; i0 += int64_t{kAggBlock} * U) {
    int64_t k[U], v[U], row[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + int64_t{u} * kAggBlock;
      row[u] = i < hi ? i : i0;
    }
    if (sel) load_items<U>(sel, 0, row, hi, row);
    load_items<U>(key, key64, row, rows, k);
    load_items<U>(val, val64, row, rows, v);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t off = static_cast<uint64_t>(k[u]) - static_cast<uint64_t>(kmin);
      if (i0 + int64_t{u} * kAggBlock >= hi || off >= range) continue;  // past the end, or an EMPTY key
      const uint32_t s = (static_cast<uint32_t>(off) << lgc) | copy;
      atomicAdd(reinterpret_cast<unsigned long long *>(&s_sum[s]), static_cast<unsigned long long>(v[u]));
      s_flag[s] = 1;
    }
  }
  __syncthreads();
  for (uint32_t o = tid; o < range; o += kAggBlock) {
    uint64_t sum = 0;
    uint32_t f = 0;
    for (uint32_t c = 0; c < (1u << lgc); ++c) {
      sum += s_sum[(o << lgc) | c];
      f |= s_flag[(o << lgc) | c];
    }
    psum[blk * range + o] = sum;
    pflag[blk * range + o] = static_cast<uint8_t>(f);
  }
}

// The rows of the modes that read them where they are: kGbSmall, and kGbFew into
// its table.  (One kernel, and one for their groups: each launch that finds
// nothing to do costs the other modes 3 us.)
__global__ __launch_bounds__(kAggBlock, 8) void k_gb_in_place(const void *key, int key64, const void *val, int val64,
                                                             const int32_t *sel, const int64_t *d_nsel, int64_t rows,
                                                             GbPlan *plan, uint64_t *psum, uint8_t *pflag, GroupDev few,
                                                             uint32_t *err) {
  static_assert(kAggBlock == 1024, "blocks of the insertion");
  __shared__ union {
    SmallLds small;
    PreLds pre;
  } lds;
  const int32_t mode = plan->mode;  // (does not change during the launch)
  if (mode == kGbSmall) small_sums(lds.small, key, key64, val, val64, sel, rows, plan, psum, pflag);
  else if (mode == kGbFew) gb_insert_rows(lds.pre, key, key64, val, val64, sel, d_nsel, rows, few, err, 0, plan, true);
}

// Adds up the blocks' partial arrays, 64 keys per block, and writes the groups
// that occur in key order (look-back over the blocks).
__device__ __forceinline__ void small_groups(GbPlan *plan, const uint64_t *psum, const uint8_t *pflag, int nparts,
                                             uint64_t *status, int64_t *out_keys, int64_t *out_sums, int64_t out_cap,
                                             int64_t *d_ngroups, uint32_t *err) {
  constexpr int NW = kAggBlock / kWave, U = 4;
  __shared__ uint64_t s_sum[NW][kWave];
  __shared__ uint32_t s_flag[NW][kWave];
  __shared__ int64_t s_tile;
  const int64_t range = static_cast<int64_t>(plan->range), ntiles = (range + kWave - 1) / kWave;
  if (threadIdx.x == 0) s_tile = static_cast<int64_t>(atomicAdd(&plan->ticket, 1ull));
  __syncthreads();
  const int64_t t = s_tile;
  if (t >= ntiles) return;  // block-uniform
  const int w = static_cast<int>(threadIdx.x) / kWave, lane = lane_id();
  const int64_t o = t * kWave + lane;
  uint64_t sum = 0;
  uint32_t f = 0;
  for (int b0 = w; b0 < nparts; b0 += NW * U) {
    uint64_t x[U];
    uint32_t y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int b = b0 + u * NW;
      const bool ok = b < nparts && o < range;
      x[u] = ok ? psum[int64_t{b} * range + o] : 0;
      y[u] = ok ? pflag[int64_t{b} * range + o] : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      sum += x[u];
      f |= y[u];
    }
  }
  s_sum[w][lane] = sum;
  s_flag[w][lane] = f;
  __syncthreads();
  if (w != 0) return;
  for (int k = 1; k < NW; ++k) {
    sum += s_sum[k][lane];
    f |= s_flag[k][lane];
  }
  const uint64_t m = __ballot(f != 0);
  const int64_t agg = __popcll(m), ex = lookback_exclusive(status, t, agg);
  const int64_t p = ex + mbcnt(m);
  if (f) {
    if (p < out_cap) {
      out_keys[p] = plan->kmin + o;
      out_sums[p] = static_cast<int64_t>(sum);
    } else {
      latch(err, kErrCapacity);
    }
  }
  if (lane == 0 && t == ntiles - 1) *d_ngroups = ex + agg;
}

// The groups of k_gb_in_place.
constexpr int kFewTileItems = 2;
constexpr int64_t kFewTiles = kFewSlots / (kAggBlock * kFewTileItems);
__global__ __launch_bounds__(kAggBlock) void k_gb_in_place_groups(GbPlan *plan, const uint64_t *psum, const uint8_t *pflag,
                                                                 int nparts, uint64_t *status, GroupDev few,
                                                                 uint64_t *few_status, int64_t *out_keys, int64_t *out_sums,
                                                                 int64_t out_cap, int64_t *d_ngroups, uint32_t *err) {
  const int32_t mode = plan_mode(plan);
  if (mode == kGbSmall)
    small_groups(plan, psum, pflag, nparts, status, out_keys, out_sums, out_cap, d_ngroups, err);
  else if (mode == kGbFew)
    gb_compact_tile<kAggBlock, kFewTileItems>(few, out_keys, out_sums, out_cap, d_ngroups, few_status,
                                              reinterpret_cast<unsigned long long *>(few_status + kFewTiles), kFewTiles, err);
}

// kGbRange: the pairs of each bucket summed in an LDS array indexed by the low
// `shift` bits of key - kmin; the groups leave in key order.  Blocks take
// buckets by ticket, in order, and find their output position by look-back, so
// a bucket only waits on buckets that are already running.  Two blocks per CU.
template <bool NARROW>
__global__ __launch_bounds__(kAggBlock, 8) void k_direct_groups(GbPlan *plan, const void *pairs, const int64_t *vals,
                                                               const int32_t *pos, int bps, uint64_t *status,
                                                               int64_t *out_keys, int64_t *out_sums, int64_t out_cap,
                                                               int64_t *d_ngroups, uint32_t *err) {
  constexpr int NW = kAggBlock / kWave, U = NARROW ? 8 : 4, PER = kDirectSlots / kAggBlock;
  __shared__ uint64_t s_sum[kDirectSlots];
  __shared__ uint8_t s_flag[kDirectSlots];
  __shared__ int32_t s_cnt[PER * NW];
  __shared__ int64_t s_base;
  __shared__ int32_t s_b;
  static_assert(PER * NW == 2 * kWave, "one wave scans the counts, two a lane");
  if (plan->mode != kGbRange) return;
  const int tid = static_cast<int>(threadIdx.x), w = tid / kWave, lane = lane_id();
  const int64_t kmin = plan->kmin;
  const int shift = plan->shift;
  const int nbuckets = static_cast<int>((plan->range - 1) >> shift) + 1;
  const uint32_t mask = (1u << shift) - 1;
  const int used = static_cast<int>((mask + kAggBlock) / kAggBlock);  // rounds of 1024 slots in use
  for (int i = tid; i < kDirectSlots; i += kAggBlock) {
    s_sum[i] = 0;
    s_flag[i] = 0;
  }
  while (true) {
    if (tid == 0) s_b = static_cast<int32_t>(atomicAdd(&plan->ticket, 1ull));
    __syncthreads();  // also: the table is clear, s_base and s_cnt are read
    const int b = s_b;
    if (b >= nbuckets) break;  // block-uniform
    const int64_t lo = pos[int64_t{b} * bps], hi = pos[int64_t{b + 1} * bps];
    for (int64_t i0 = lo + tid; i0 < hi; i0 += int64_t{kAggBlock} * U) {
      int64_t k[U], v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t i = i0 + int64_t{u} * kAggBlock < hi ? i0 + int64_t{u} * kAggBlock : i0;
        if (NARROW) {
          const uint64_t pr = static_cast<const uint64_t *>(pairs)[i];
          k[u] = static_cast<int32_t>(pr >> 32);
          v[u] = static_cast<int32_t>(pr & 0xffffffffu);
        } else {
          k[u] = static_cast<const int64_t *>(pairs)[i];
          v[u] = vals[i];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (i0 + int64_t{u} * kAggBlock >= hi) continue;
        const uint32_t s = static_cast<uint32_t>(k[u] - kmin) & mask;
        atomicAdd(reinterpret_cast<unsigned long long *>(&s_sum[s]), static_cast<unsigned long long>(v[u]));
        s_flag[s] = 1;
      }
    }
    __syncthreads();
    uint64_t m[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      m[j] = j < used ? __ballot(s_flag[j * kAggBlock + tid] != 0) : 0;
      if (lane == 0) s_cnt[j * NW + w] = __popcll(m[j]);
    }
    __syncthreads();
    if (w == 0) {
      const int32_t a = s_cnt[2 * lane], c = s_cnt[2 * lane + 1];
      const int32_t incl = wave_inclusive_scan(a + c);
      s_cnt[2 * lane] = incl - a - c;
      s_cnt[2 * lane + 1] = incl - c;
      const int64_t agg = __shfl(incl, kWave - 1);
      const int64_t ex = lookback_exclusive(status, b, agg);
      if (lane == 0) {
        s_base = ex;
        if (b == nbuckets - 1) {
          *d_ngroups = ex + agg;
          if (ex + agg > out_cap) latch(err, kErrCapacity);
        }
      }
    }
    __syncthreads();
    const int64_t base = s_base;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int s = j * kAggBlock + tid;
      if (j < used && ((m[j] >> lane) & 1ull)) {
        const int64_t p = base + s_cnt[j * NW + w] + mbcnt(m[j]);
        if (p < out_cap) {
          out_keys[p] = kmin + ((int64_t{b} << shift) | s);
          out_sums[p] = static_cast<int64_t>(s_sum[s]);
        }
        s_sum[s] = 0;
        s_flag[s] = 0;
      }
    }
  }
}

template <bool NARROW>
pyst_status launch_direct_groups(pyst_ctx *ctx, GbPlan *plan, uint64_t *status, const void *pairs, const int64_t *vals,
                                 const int32_t *pos, int bps, int64_t *out_keys, int64_t *out_sums, int64_t out_cap,
                                 int64_t *d_ngroups, hipStream_t stream) {
  const int blocks = static_cast<int>(std::min<int64_t>(kAggBuckets, 2 * std::max(1, ctx_num_cus(ctx))));
  k_direct_groups<NARROW><<<blocks, kAggBlock, 0, stream>>>(plan, pairs, vals, pos, bps, status, out_keys, out_sums,
                                                           out_cap, d_ngroups, ctx_err_word(ctx));
  PYST_LAUNCH_CHECK("k_direct_groups");
  return PYST_OK;
}

// ---------------------------------------------------------------- one move (kGbOnce)
// int32 keys and values over at most 2^24 values: the pairs are moved once, into
// up to 1024 buckets of the key range, and a bucket's sums fill the LDS of a CU.
// Bound by memory: the rows read and the pairs written (16 bytes a row), the
// pairs read and the groups written.  A move to so many places leaves lines
// half written: 32 blocks of an XCD with 1024 runs each would hold its whole L2
// in such lines, so the blocks of an XCD fill the same places (a cursor per XCD
// and bucket, moved by atomics) and a line is whole before it leaves.  Tiles of
// 16384 pairs (128 KiB of LDS, one block per CU) make runs of 16 pairs.
// 60M pairs over 15M keys: count 34, move 258, sums 172 us, where two moves took
// 40, 235 + 252 and 193; a cursor per block 304 and 198; tiles of 8192 pairs, two
// blocks per CU, 276 and 194.  The call, ordered by key: 840 -> 585 us; 20M over
// 9000 keys 331 -> 211, 1.2M over 300K 123 -> 91, 30M over 16M 490 -> 350.
constexpr int kOnceItems = 16, kOnceTile = kAggBlock * kOnceItems;
constexpr int kOnceParts = 256;  // blocks: contiguous ranges of rows
constexpr int kOnceShare = 32;   // neighbouring ranges (one XCD's) that fill places together

struct OnceWork {
  int32_t *counts;   // [kOnceParts][kOnceBuckets]; then the rows before each range, then cursors
  int32_t *totals;   // [kOnceBuckets]
  uint64_t *pairs;   // (key - kmin) << 32 | value
};

__global__ __launch_bounds__(kAggBlock) void k_once_hist(NarrowArgs a, OnceWork o) {
  __shared__ int32_t s_c[kOnceBuckets];
  if (a.plan->mode != kGbOnce) return;
  const int tid = static_cast<int>(threadIdx.x), shift = a.plan->shift;
  const int32_t kmin = static_cast<int32_t>(a.plan->kmin);
  if (tid < kOnceBuckets) s_c[tid] = 0;
  __syncthreads();
  int64_t lo, hi;
  const int blk = static_cast<int>(xcd_block(blockIdx.x, kOnceParts));
  narrow_range(a, blk, kOnceParts, &lo, &hi);
  constexpr int U = 8;
  for (int64_t i0 = lo + tid; i0 < hi; i0 += int64_t{kAggBlock} * U) {
    int32_t k[U];
#pragma unroll
    for (int u = 0; u < U; ++u) k[u] = a.kcol[row_of(a.sel, i0 + u * kAggBlock < hi ? i0 + u * kAggBlock : i0)];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * kAggBlock < hi) atomicAdd(&s_c[(static_cast<uint32_t>(k[u]) - static_cast<uint32_t>(kmin)) >> shift], 1);
  }
  __syncthreads();
  if (tid < kOnceBuckets) o.counts[blk * kOnceBuckets + tid] = s_c[tid];
}

// Per bucket the exclusive prefix over the ranges, in place, and the total; 64
// buckets a block, 16 ranges a wave.
__global__ __launch_bounds__(kAggBlock) void k_once_counts(const GbPlan *plan, OnceWork o) {
  constexpr int NW = kAggBlock / kWave, PER = kOnceParts / NW;
  __shared__ int32_t s_w[NW][kWave];
  if (plan->mode != kGbOnce) return;
  const int w = threadIdx.x / kWave, lane = lane_id(), b = static_cast<int>(blockIdx.x) * kWave + lane;
  int32_t c[PER], sum = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) c[j] = o.counts[(w * PER + j) * kOnceBuckets + b];
#pragma unroll
  for (int j = 0; j < PER; ++j) sum += c[j];
  s_w[w][lane] = sum;
  __syncthreads();
  int32_t run = 0;
  for (int k = 0; k < w; ++k) run += s_w[k][lane];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    o.counts[(w * PER + j) * kOnceBuckets + b] = run;
    run += c[j];
  }
  if (w == NW - 1) o.totals[b] = run;
}

// s[b]: the exclusive prefix of the bucket totals (all threads; synchronizes).
__device__ __forceinline__ void once_offsets(const int32_t *totals, int32_t *s, int32_t *s_w) {
  static_assert(kOnceBuckets == kAggBlock, "a thread per bucket");
  const int tid = static_cast<int>(threadIdx.x), w = tid / kWave;
  const int32_t c = totals[tid], incl = wave_inclusive_scan(c);
  if (lane_id() == kWave - 1) s_w[w] = incl;
  __syncthreads();
  int32_t before = 0;
  for (int k = 0; k < w; ++k) before += s_w[k];
  s[tid] = before + incl - c;
  __syncthreads();
}

__global__ __launch_bounds__(kAggBlock) void k_once_move(NarrowArgs a, OnceWork o) {
  __shared__ uint64_t s_p[kOnceTile];
  __shared__ int32_t s_cnt[kOnceBuckets], s_off[kOnceBuckets], s_to[kOnceBuckets];
  __shared__ int32_t s_w[kAggBlock / kWave];
  if (a.plan->mode != kGbOnce) return;
  const int tid = static_cast<int>(threadIdx.x), w = tid / kWave, shift = a.plan->shift;
  const uint32_t kmin = static_cast<uint32_t>(static_cast<int32_t>(a.plan->kmin));
  int64_t lo, hi;
  const int blk = static_cast<int>(xcd_block(blockIdx.x, kOnceParts));
  narrow_range(a, blk, kOnceParts, &lo, &hi);
  once_offsets(o.totals, s_to, s_w);
  // thread b: bucket b's start, and the cursor of the places there that these blocks share
  const int32_t start = s_to[tid];
  int32_t *const cursor = o.counts + blk / kOnceShare * kOnceShare * kOnceBuckets + tid;
  uint32_t key[kOnceItems];
  int32_t val[kOnceItems];
  auto load_tile = [&](int64_t t0) {
    const uint32_t n = static_cast<uint32_t>(hi - t0 < kOnceTile ? hi - t0 : kOnceTile);
    if (a.sel) {
      const int32_t *sel = a.sel + t0;
#pragma unroll
      for (int u = 0; u < kOnceItems; ++u) {
        const uint32_t i = static_cast<uint32_t>(u * kAggBlock + tid);
        const int32_t r = sel[i < n ? i : 0];
        key[u] = static_cast<uint32_t>(a.kcol[r]);
        val[u] = a.vcol[r];
      }
    } else {
      const int32_t *kc = a.kcol + t0, *vc = a.vcol + t0;
#pragma unroll
      for (int u = 0; u < kOnceItems; ++u) {
        const uint32_t i = static_cast<uint32_t>(u * kAggBlock + tid);
        if (i < n) key[u] = static_cast<uint32_t>(kc[i]);
        if (i < n) val[u] = vc[i];
      }
    }
  };
  if (lo < hi) load_tile(lo);
  for (int64_t t0 = lo; t0 < hi; t0 += kOnceTile) {  // block-uniform
    s_cnt[tid] = 0;
    uint32_t rk[kOnceItems / 2];  // ranks, two a register
    const int n = static_cast<int>(hi - t0 < kOnceTile ? hi - t0 : kOnceTile);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kOnceItems; ++u) {
      uint32_t r = 0;
      if (u * kAggBlock + tid < n) r = static_cast<uint32_t>(atomicAdd(&s_cnt[(key[u] - kmin) >> shift], 1));
      rk[u / 2] = u % 2 ? rk[u / 2] | r << 16 : r;
    }
    __syncthreads();
    const int32_t c = s_cnt[tid], incl = wave_inclusive_scan(c);
    const int32_t to = c ? atomicAdd(cursor, c) : 0;  // waited for after the pairs are in place
    if (lane_id() == kWave - 1) s_w[w] = incl;
    __syncthreads();
    int32_t at = incl - c;  // bucket b's place in the tile
    for (int k = 0; k < w; ++k) at += s_w[k];
    s_off[tid] = at;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kOnceItems; ++u)
      if (u * kAggBlock + tid < n) {
        const uint32_t off = key[u] - kmin, r = u % 2 ? rk[u / 2] >> 16 : rk[u / 2] & 0xffff;
        s_p[s_off[off >> shift] + r] = static_cast<uint64_t>(off) << 32 | static_cast<uint32_t>(val[u]);
      }
    s_to[tid] = start + to - at;  // the pair at place p goes to s_to + p
    __syncthreads();
    if (t0 + kOnceTile < hi) load_tile(t0 + kOnceTile);  // arrives while this tile leaves
    for (int p = tid; p < n; p += kAggBlock) {
      const uint64_t x = s_p[p];
      o.pairs[s_to[static_cast<uint32_t>(x >> 32) >> shift] + p] = x;
    }
    __syncthreads();
  }
}

// As k_direct_groups, with the whole LDS of a CU for a bucket.
__global__ __launch_bounds__(kAggBlock) void k_once_groups(GbPlan *plan, OnceWork o, uint64_t *status, int64_t *out_keys,
                                                          int64_t *out_sums, int64_t out_cap, int64_t *d_ngroups,
                                                          uint32_t *err) {
  constexpr int NW = kAggBlock / kWave, U = 8, PER = kOnceSlots / kAggBlock;
  __shared__ uint64_t s_sum[kOnceSlots];
  __shared__ uint8_t s_flag[kOnceSlots];
  __shared__ int32_t s_cnt[PER * NW];
  __shared__ int32_t s_w[NW], s_lo[kOnceBuckets];
  __shared__ int64_t s_base;
  __shared__ int32_t s_b;
  static_assert(PER * NW == 4 * kWave, "one wave scans the counts, four a lane");
  if (plan->mode != kGbOnce) return;
  const int tid = static_cast<int>(threadIdx.x), w = tid / kWave, lane = lane_id(), shift = plan->shift;
  const int64_t kmin = plan->kmin;
  const int nbuckets = static_cast<int>((plan->range - 1) >> shift) + 1;
  const uint32_t mask = (1u << shift) - 1;
  const int used = static_cast<int>((mask + kAggBlock) / kAggBlock);
  once_offsets(o.totals, s_lo, s_w);
  for (int i = tid; i < kOnceSlots; i += kAggBlock) {
    s_sum[i] = 0;
    s_flag[i] = 0;
  }
  // A round is 8 pairs a thread; the next round, of this bucket or of the next
  // one, is loaded before this one is added.
  uint64_t x[U];
  int64_t i0 = 0, hi = 0;
  auto load_round = [&]() {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * kAggBlock < hi) x[u] = o.pairs[i0 + u * kAggBlock];
  };
  if (tid == 0) s_b = static_cast<int32_t>(atomicAdd(&plan->ticket, 1ull));
  __syncthreads();
  int b = s_b;
  if (b < nbuckets) {
    i0 = s_lo[b] + tid;
    hi = b + 1 < kOnceBuckets ? s_lo[b + 1] : plan->count;
    load_round();
  }
  while (b < nbuckets) {  // block-uniform
    __syncthreads();      // the table is clear; s_b, s_base and s_cnt are read
    if (tid == 0) s_b = static_cast<int32_t>(atomicAdd(&plan->ticket, 1ull));
    for (; i0 - tid < hi;) {  // block-uniform
      uint64_t y[U];
      const int64_t j0 = i0;
      const int64_t jhi = hi;
#pragma unroll
      for (int u = 0; u < U; ++u) y[u] = x[u];
      i0 += int64_t{kAggBlock} * U;
      load_round();
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (j0 + u * kAggBlock >= jhi) continue;
        const uint32_t s = static_cast<uint32_t>(y[u] >> 32) & mask;
        atomicAdd(reinterpret_cast<unsigned long long *>(&s_sum[s]),
                  static_cast<unsigned long long>(static_cast<int64_t>(static_cast<int32_t>(y[u] & 0xffffffffu))));
        s_flag[s] = 1;
      }
    }
    __syncthreads();
    const int nb = s_b;
    if (nb < nbuckets) {
      i0 = s_lo[nb] + tid;
      hi = nb + 1 < kOnceBuckets ? s_lo[nb + 1] : plan->count;
      load_round();
    }
    uint64_t m[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      m[j] = j < used ? __ballot(s_flag[j * kAggBlock + tid] != 0) : 0;
      if (lane == 0) s_cnt[j * NW + w] = __popcll(m[j]);
    }
    __syncthreads();
    if (w == 0) {
      int32_t c[4], sum = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) sum += c[j] = s_cnt[4 * lane + j];
      const int32_t incl = wave_inclusive_scan(sum);
      int32_t run = incl - sum;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        s_cnt[4 * lane + j] = run;
        run += c[j];
      }
      const int64_t agg = __shfl(incl, kWave - 1);
      const int64_t ex = lookback_exclusive(status, b, agg);
      if (lane == 0) {
        s_base = ex;
        if (b == nbuckets - 1) {
          *d_ngroups = ex + agg;
          if (ex + agg > out_cap) latch(err, kErrCapacity);
        }
      }
    }
    __syncthreads();
    const int64_t base = s_base;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int s = j * kAggBlock + tid;
      if (j < used && ((m[j] >> lane) & 1ull)) {
        const int64_t p = base + s_cnt[j * NW + w] + mbcnt(m[j]);
        if (p < out_cap) {
          out_keys[p] = kmin + ((int64_t{b} << shift) | s);
          out_sums[p] = static_cast<int64_t>(s_sum[s]);
        }
        s_sum[s] = 0;
        s_flag[s] = 0;
      }
    }
    b = nb;
  }
}

// Scratch in the narrow moves' memory: the counts where theirs are, the pairs in
// one of their two buffers.
static pyst_status launch_once(pyst_ctx *ctx, const NarrowArgs &a, void *ws, uint64_t *pairs, uint64_t *status,
                               int64_t *out_keys, int64_t *out_sums, int64_t out_cap, int64_t *d_ngroups, hipStream_t stream) {
  static_assert((kOnceParts + 1) * kOnceBuckets <= kNB1 * kAggBuckets, "the counts of the narrow moves take more");
  OnceWork o;
  o.counts = static_cast<int32_t *>(ws);
  o.totals = o.counts + kOnceParts * kOnceBuckets;
  o.pairs = pairs;
  k_once_hist<<<kOnceParts, kAggBlock, 0, stream>>>(a, o);
  PYST_LAUNCH_CHECK("k_once_hist");
  k_once_counts<<<kOnceBuckets / kWave, kAggBlock, 0, stream>>>(a.plan, o);
  PYST_LAUNCH_CHECK("k_once_counts");
  k_once_move<<<kOnceParts, kAggBlock, 0, stream>>>(a, o);
  PYST_LAUNCH_CHECK("k_once_move");
  k_once_groups<<<std::max(1, ctx_num_cus(ctx)), kAggBlock, 0, stream>>>(a.plan, o, status, out_keys, out_sums, out_cap,
                                                                        d_ngroups, ctx_err_word(ctx));
  PYST_LAUNCH_CHECK("k_once_groups");
  return PYST_OK;
}

// The group count of the hash modes is what remains to be sorted.
__global__ void k_gb_sort_count(GbPlan *plan, const int64_t *d_ngroups) {
  plan->sort_count = plan->mode == kGbSmall || plan->mode == kGbRange || plan->mode == kGbOnce ? 0 : *d_ngroups;
}

// Small scratch of a planned group-by: the plan, the look-back words, the
// blocks' key ranges and the sample.
constexpr size_t kPlanBytes = 256 + sizeof(uint64_t) * kAggBuckets + 2 * sizeof(int64_t) * kRangeBlocks +
                              sizeof(int64_t) * kSamples;

// GROUP BY of key->n >= 2^20 rows (of a selection).  hash_buckets: few enough
// groups (kRadixGroupsMax) for LDS hash tables; else keys without a small range
// take the table in HBM (`bound` groups at most) and the ranged moves are used
// only where the arena also has room for them.
pyst_status planned_groupby(pyst_ctx *ctx, const pyst_col *key, const pyst_col *val, const int32_t *sel,
                            const int64_t *d_nsel, int64_t max_groups, int64_t bound, double max_load,
                            bool hash_buckets, int64_t *out_keys, int64_t *out_sums, int64_t out_cap,
                            int64_t *d_ngroups, int sort_by_key, hipStream_t stream) {
  const int64_t n = key->n;
  const bool narrow = key->dtype == PYST_I32 && val->dtype == PYST_I32;  // 8-byte pairs, else 16-byte ones
  const int k64 = key->dtype == PYST_I64, v64 = val->dtype == PYST_I64;
  uint32_t *err = ctx_err_word(ctx);
  GbPlan *plan = nullptr;
  Scratch ps(ctx, stream);
  {
    const int64_t cap_alloc = hash_buckets ? 0 : table_capacity_host(bound, max_load);
    Scratch table(ctx, stream), words(ctx, stream), ws(ctx, stream), ws2(ctx, stream), few(ctx, stream);
    // what the call cannot do without comes first: what it can must not take its place
    if (!hash_buckets) {
      table.alloc(group_bytes(cap_alloc));
      words.alloc(group_compact_words(cap_alloc) * sizeof(uint64_t));
    }
    const size_t wsb = narrow ? narrow_groupby_bytes(n) : static_cast<size_t>(n) * 16;
    hash_buckets ? ws.alloc(wsb) : ws.try_alloc(wsb);
    if (!narrow && ws.p) hash_buckets ? ws2.alloc(wide_groupby_bytes(n)) : ws2.try_alloc(wide_groupby_bytes(n));
    const bool moves = ws.p && (narrow || ws2.p);
    if (hash_buckets ? !moves : !table.p || !words.p) return set_error(PYST_ERR_NOMEM, "pyst_groupby_sum: arena exhausted");
    ps.try_alloc(kPlanBytes);
    const int64_t *count = d_nsel;
    uint64_t *status = nullptr;
    pyst_status st;
    constexpr int64_t few_words = kFewTiles + 1;
    if (ps.p) few.try_alloc(group_bytes(kFewSlots) + few_words * sizeof(uint64_t));
    if (ps.p) {
      plan = ps.as<GbPlan>();
      count = &plan->count;
      status = reinterpret_cast<uint64_t *>(static_cast<char *>(ps.p) + 256);
      int64_t *lo = reinterpret_cast<int64_t *>(status + kAggBuckets), *hi = lo + kRangeBlocks,
              *samples = hi + kRangeBlocks;
      const GroupDev fg = few.p ? group_view(few.p, kFewSlots) : GroupDev{};
      uint64_t *few_status = few.p ? reinterpret_cast<uint64_t *>(static_cast<char *>(few.p) + group_bytes(kFewSlots)) : nullptr;
      const int rblocks = static_cast<int>(std::min<int64_t>(kRangeBlocks, ceil_div(n, 256 * kRangeItems)));
      // the blocks' partial arrays of kGbSmall take the memory of the moves, or of the table
      const size_t room = moves ? static_cast<size_t>(n) * 16 : group_bytes(cap_alloc);
      const int parts = std::max(1, std::min(512, 2 * ctx_num_cus(ctx)));
      const int64_t small_max = std::min<int64_t>(kDirectSlots, static_cast<int64_t>(room / (parts * 9)));
      k_key_range<<<rblocks, 256, 0, stream>>>(key->data, k64, sel, d_nsel, n, lo, hi, samples, fg, few_status,
                                               few_words, err);
      PYST_LAUNCH_CHECK("k_key_range");
      k_gb_plan<<<1, kAggBlock, 0, stream>>>(plan, lo, hi, rblocks, samples, d_nsel, n, small_max, moves, narrow,
                                             few.p != nullptr, hash_buckets ? kGbHash : kGbTable, status, d_ngroups);
      PYST_LAUNCH_CHECK("k_gb_plan");
      uint64_t *psum = moves ? ws.as<uint64_t>() : table.as<uint64_t>();
      uint8_t *pflag = reinterpret_cast<uint8_t *>(psum + parts * small_max);
      k_gb_in_place<<<parts, kAggBlock, 0, stream>>>(key->data, k64, val->data, v64, sel, d_nsel, n, plan, psum, pflag,
                                                    fg, err);
      PYST_LAUNCH_CHECK("k_gb_in_place");
      const int64_t gblocks = std::max(ceil_div(small_max, kWave), few.p ? kFewTiles : 1);
      k_gb_in_place_groups<<<static_cast<unsigned>(gblocks), kAggBlock, 0, stream>>>(
          plan, psum, pflag, parts, status, fg, few_status, out_keys, out_sums, out_cap, d_ngroups, err);
      PYST_LAUNCH_CHECK("k_gb_in_place_groups");
    } else if (hash_buckets) {  // no room for a plan: hash buckets for any keys
      if ((st = fill_u64(d_ngroups, 1, 0, stream)) != PYST_OK) return st;
      if (!count) {
        if (!ps.alloc(256)) return set_error(PYST_ERR_NOMEM, "pyst_groupby_sum: arena exhausted");
        if ((st = fill_u64(ps.p, 1, static_cast<uint64_t>(n), stream)) != PYST_OK) return st;
        count = ps.as<int64_t>();
      }
    }
    if (hash_buckets || (plan && moves)) {
      if (narrow) {
        st = narrow_groupby(ctx, static_cast<const int32_t *>(key->data), static_cast<const int32_t *>(val->data), sel,
                            count, n, ws.p, out_keys, out_sums, out_cap, d_ngroups, plan, status, hash_buckets, stream);
      } else {
        MoveArgs first{};
        first.kcol = key->data;
        first.vcol = val->data;
        first.sel = sel;
        first.k64 = k64;
        first.v64 = v64;
        first.err = err;
        first.plan = plan;
        int64_t *pk = ws.as<int64_t>();
        st = pair_groupby_from(ctx, first, pk, pk + n, count, n, out_keys, out_sums, out_cap, d_ngroups, status, ws2.p,
                               hash_buckets, stream);
      }
      if (st != PYST_OK) return st;
    }
    if (!hash_buckets) {
      const GroupDev g = group_view(table.p, cap_alloc);
      st = table_groupby(ctx, g, key, val, sel, d_nsel, max_groups, max_load, out_keys, out_sums, out_cap, d_ngroups,
                         plan, kGbTable, words.as<uint64_t>(), stream);
      if (st != PYST_OK) return st;
    }
  }
  if (!sort_by_key) return PYST_OK;
  const int64_t *sort_count = d_ngroups;
  if (plan) {
    k_gb_sort_count<<<1, 1, 0, stream>>>(plan, d_ngroups);
    PYST_LAUNCH_CHECK("k_gb_sort_count");
    sort_count = &plan->sort_count;
  }
  return sort_pairs_by_key(ctx, out_keys, out_sums, sort_count, bound, k64 ? 64 : 32, stream);
}

}  // namespace pyst
