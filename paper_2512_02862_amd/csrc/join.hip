// Equi-join of large sides whose build keys are dense (surrogate keys): the
// build side as an array of row ids indexed by key - least key, built and read
// slice by slice.
//
// A hash join of these sizes is bound by memory lines: every insert and every
// probe of a table far beyond the L2 moves a whole 128-byte line for 4 useful
// bytes (60M inserts 2.9 ms, 160M probes 5.1 ms, at 4 - 5 TB/s of lines).  Here
// both sides are first split by key into slices of 2^18 keys or
// more (1 MiB of the array, which one XCD's L2 holds beside the stream; 2^19
// keys cost the 60M x 160M join 70 us, 2^20 430): a counting and a moving
// kernel over the keys alone.  The stores and loads of the array then hit the
// L2.  Probe rows that no build key can match are dropped by the move.
// The probe rows have to come out in their own order: the move records where
// each row's key went within its tile (2 bytes a row) and which slice each moved
// key of the tile belongs to (1 byte), so that the last kernel reads a tile's
// results back as contiguous runs, puts them in row order through LDS and
// compacts the matches.
//
// Bound by streams: 60M build rows 12 + 20 bytes a row, 160M probe rows about 24
// bytes a row.  60M x 160M with 4 columns a side: build 2911 -> 880 us, probe 5064
// -> 1585 us, the whole join 12.84 -> 7.10 ms (4.6 of them the gathers of the
// columns, at 5.5 TB/s); 5M x 15M 834 -> 406 us.
//
// The choice is made on the device from the build keys' range: direct where the
// keys span no more values than the hash table has slots (and at most 2^32: a key
// travels as its 32-bit offset), else the hash table's
// kernels run and these return at once.  A duplicate key (the caller promised
// none) leaves fewer filled entries than rows, which is reported.
#include "pyst_internal.h"
#include "ranges.h"
#include "table.h"

namespace pyst {

constexpr int kSliceItems = 8, kSliceTile = kRangeThreads * kSliceItems;
constexpr int kSliceLg = 18;
constexpr uint16_t kNoMatchPos = 0xffff;
constexpr int kJoinRangeBlocks = 2048;

// A move of rows to slices and, for probes, the way back.
struct Slices {
  RangeCounts counts;
  int pass;             // row set of the counts
  int64_t *moved;       // rows moved in all
  void *items;          // moved items, then (probes) their results in place
  // probes only:
  uint64_t *status;     // look-back words of the emitting kernel, one per tile
  unsigned long long *ticket;
  int64_t ntiles;       // tiles of all n rows
  uint64_t *found;      // bit per moved item (hash tables; a direct result is -1 for none)
  uint16_t *pos;        // per row: its place among its tile's moved items
  uint8_t *slice;       // per (tile, place): the slice
  uint32_t *goff;       // per (tile, slice): where place 0 of the tile would lie
  int32_t *live;        // per tile: moved items
};

struct DirectJoin {
  JoinPlan *plan;
  int32_t *array;       // row id by key - kmin, -1 for none
  Slices build, probe;
};

template <bool K64>
using ColumnKey = std::conditional_t<K64, int64_t, int32_t>;
template <bool K64>
constexpr ColumnKey<K64> kColumnEmpty = K64 ? static_cast<ColumnKey<K64>>(kEmpty64) : static_cast<ColumnKey<K64>>(kEmpty32);
constexpr uint32_t kDead = 0xffffffffu;  // slice of a row that is not moved

// What moves: the slice of a key and the item that travels for its row.
template <bool K64, bool BUILD>
struct DirectRows {
  static constexpr bool kWide = K64, kProbe = !BUILD;
  using Item = std::conditional_t<BUILD, uint64_t, uint32_t>;
  const JoinPlan *plan;
  int64_t kmin = 0;
  uint64_t range = 0;
  int shift = 0;
  __device__ __forceinline__ bool open() {
    kmin = plan->kmin;
    range = plan->range;
    shift = plan->shift;
    return plan->direct != 0;
  }
  __device__ __forceinline__ uint64_t offset(int64_t k) const { return static_cast<uint64_t>(k) - static_cast<uint64_t>(kmin); }
  __device__ __forceinline__ uint32_t slice(int64_t k) const {
    return offset(k) < range ? static_cast<uint32_t>(offset(k) >> shift) : kDead;
  }
  __device__ __forceinline__ Item item(int64_t k, int32_t row) const {
    if constexpr (BUILD) return static_cast<uint32_t>(offset(k)) | (static_cast<uint64_t>(static_cast<uint32_t>(row)) << 32);
    else return static_cast<uint32_t>(offset(k));
  }
};

// Probe keys of a hash table with 8-byte (int32 keys) or 16-byte slots, by home slot.
template <bool WIDE, bool K64>
struct HashRows {
  static constexpr bool kWide = K64, kProbe = true;
  using Item = std::conditional_t<WIDE, uint64_t, uint32_t>;
  const JoinPlan *plan;  // may be null
  const int64_t *hdr;
  int shift;             // slots a slice
  ProbeRule rule;
  int64_t mask = 0;
  __device__ __forceinline__ bool open() {
    mask = hdr[0] - 1;
    return !(plan && plan->direct) && !rule.not_by_slices();
  }
  __device__ __forceinline__ uint32_t slice(int64_t k) const {
    if constexpr (WIDE) return static_cast<uint32_t>((table_hash64(k) & static_cast<uint64_t>(mask)) >> shift);
    if (K64 && (k <= kEmpty32 || k > INT32_MAX)) return kDead;  // no int32 key of the table
    return static_cast<uint32_t>((table_hash32(static_cast<int32_t>(k)) & static_cast<uint64_t>(mask)) >> shift);
  }
  __device__ __forceinline__ Item item(int64_t k, int32_t) const { return static_cast<Item>(k); }
};

template <bool K64>
__device__ __forceinline__ bool slice_key(const void *key, int64_t row, int64_t &k) {
  if (K64) {
    k = static_cast<const int64_t *>(key)[row];
    return k != kEmpty64;
  }
  k = static_cast<const int32_t *>(key)[row];
  return k != kEmpty32;
}

// Least and greatest build key per block; EMPTY keys are latched and left out.
template <bool K64>
__global__ __launch_bounds__(256) void k_join_range(const void *key, int64_t n, int64_t *lo_out, int64_t *hi_out,
                                                    uint32_t *err) {
  __shared__ int64_t s_lo[4], s_hi[4];
  constexpr int U = 8;
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  bool bad = false;
  const int64_t step = int64_t{gridDim.x} * 256;
  for (int64_t i0 = int64_t{blockIdx.x} * 256 + threadIdx.x; i0 < n; i0 += step * U) {
    int64_t k[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) ok[u] = slice_key<K64>(key, i0 + u * step < n ? i0 + u * step : i0, k[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      bad |= !ok[u];
      lo = ok[u] && k[u] < lo ? k[u] : lo;
      hi = ok[u] && k[u] > hi ? k[u] : hi;
    }
  }
  if (bad) latch(err, kErrKey);
  block_key_range(lo, hi, s_lo, s_hi, 4);
  if (threadIdx.x == 0) {
    lo_out[blockIdx.x] = lo;
    hi_out[blockIdx.x] = hi;
  }
}

__global__ __launch_bounds__(kRangeThreads) void k_join_plan(JoinPlan *plan, const int64_t *lo_in, const int64_t *hi_in,
                                                            int nblocks, uint64_t range_max, RangeCounts counts) {
  __shared__ int64_t s_lo[kRangeThreads / kWave], s_hi[kRangeThreads / kWave];
  const int tid = static_cast<int>(threadIdx.x);
  for (int i = tid; i < 2 * counts.ngroups * kRangeDigits; i += kRangeThreads) counts.group[i] = 0;
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  for (int i = tid; i < nblocks; i += kRangeThreads) {
    lo = lo_in[i] < lo ? lo_in[i] : lo;
    hi = hi_in[i] > hi ? hi_in[i] : hi;
  }
  block_key_range(lo, hi, s_lo, s_hi, kRangeThreads / kWave);
  if (tid == 0) {
    const uint64_t range = lo > hi ? 0 : static_cast<uint64_t>(hi) - static_cast<uint64_t>(lo) + 1;
    int shift = kSliceLg;
    if (range)
      while (((range - 1) >> shift) >= kRangeDigits) ++shift;
    plan->kmin = lo;
    plan->range = range;
    plan->direct = range > 0 && range <= range_max;
    plan->shift = shift;
    plan->moved[0] = plan->moved[1] = 0;
    plan->filled = 0;
    plan->ticket = 0;
  }
}

__global__ __launch_bounds__(256) void k_direct_clear(DirectJoin d) {
  if (!d.plan->direct) return;
  const int64_t i0 = int64_t{blockIdx.x} * 256 + threadIdx.x, step = int64_t{gridDim.x} * 256;
  const int64_t quads = static_cast<int64_t>((d.plan->range + 3) / 4);  // the array has room for whole quads
  const v4i32 none = {-1, -1, -1, -1};
  for (int64_t i = i0; i < quads; i += step) reinterpret_cast<v4i32 *>(d.array)[i] = none;
}

template <typename P>
__global__ __launch_bounds__(kRangeThreads, 8) void k_slice_hist(P p, Slices d, const void *key, const int32_t *sel,
                                                                const int64_t *d_nsel, int64_t n_all) {
  using KeyT = ColumnKey<P::kWide>;
  __shared__ uint32_t s_h[kRangeDigits];
  int64_t part, t0, t1;
  const int64_t n = std::min(count_of(d_nsel, n_all), n_all);
  if (!p.open()) return;
  const int tid = static_cast<int>(threadIdx.x);
  if (P::kProbe)
    for (int64_t i = int64_t{blockIdx.x} * kRangeThreads + tid; i < d.ntiles; i += int64_t{gridDim.x} * kRangeThreads) d.status[i] = 0;
  if (!range_of_block(n, kSliceTile, part, t0, t1)) return;
  if (tid < kRangeDigits) s_h[tid] = 0;
  __syncthreads();
  const int64_t hi = t1 * kSliceTile < n ? t1 * kSliceTile : n;
  for (int64_t i0 = t0 * kSliceTile + tid; i0 < hi; i0 += kSliceTile) {
    int64_t row[kSliceItems];
    KeyT k[kSliceItems];
#pragma unroll
    for (int u = 0; u < kSliceItems; ++u) row[u] = i0 + u * kRangeThreads < hi ? i0 + u * kRangeThreads : i0;
    if (sel) {
#pragma unroll
      for (int u = 0; u < kSliceItems; ++u) row[u] = sel[row[u]];
    }
#pragma unroll
    for (int u = 0; u < kSliceItems; ++u) k[u] = static_cast<const KeyT *>(key)[row[u]];
#pragma unroll
    for (int u = 0; u < kSliceItems; ++u) {
      const uint32_t sl = p.slice(k[u]);
      if (i0 + u * kRangeThreads < hi && k[u] != kColumnEmpty<P::kWide> && sl != kDead) atomicAdd(&s_h[sl], 1u);
    }
  }
  __syncthreads();
  if (tid < kRangeDigits) {
    d.counts.of_part(part)[tid] = s_h[tid];
    if (s_h[tid]) atomicAdd(&d.counts.of_group(d.pass, part / kRangeGroup)[tid], s_h[tid]);
  }
}

// Moves the items of a block's range of tiles to their slices.  A tile is laid
// out by slice in LDS and leaves as one run a slice.  Two blocks of 16 waves per
// CU.
template <typename P>
__global__ __launch_bounds__(kRangeThreads, 8) void k_slice_move(P p, Slices d, const void *key, const int32_t *sel,
                                                                const int64_t *d_nsel, int64_t n_all) {
  using Item = typename P::Item;
  using KeyT = ColumnKey<P::kWide>;
  __shared__ __align__(16) Item s_stage[kSliceTile];
  __shared__ uint8_t s_dig[kSliceTile];
  __shared__ int32_t s_cnt[kRangeDigits], s_start[kRangeDigits];
  __shared__ int64_t s_next[kRangeDigits];
  __shared__ int32_t s_live;
  static_assert(sizeof(RangeOffsets) <= sizeof(s_stage), "the offsets are summed in the staging area");
  static_assert(kSliceTile <= 1 << 16, "a slice and a rank share a word");
  int64_t part, t0, t1;
  const int64_t n = std::min(count_of(d_nsel, n_all), n_all);
  if (!p.open() || !range_of_block(n, kSliceTile, part, t0, t1)) return;
  const int tid = static_cast<int>(threadIdx.x), lane = lane_id();
  const int64_t total = range_offsets(d.counts, d.pass, static_cast<int>(part),
                                      *reinterpret_cast<RangeOffsets *>(s_stage), s_next);
  if (part == 0 && tid == 0) *d.moved = total;
  const int32_t last = static_cast<int32_t>(n) - 1;
  for (int64_t t = t0; t < t1; ++t) {  // block-uniform
    if (tid < kRangeDigits) s_cnt[tid] = 0;
    const int32_t base = static_cast<int32_t>(t) * kSliceTile + tid;
    KeyT k[kSliceItems];
    if (sel) {
#pragma unroll
      for (int u = 0; u < kSliceItems; ++u) k[u] = static_cast<const KeyT *>(key)[sel[std::min(base + u * kRangeThreads, last)]];
    } else {
#pragma unroll
      for (int u = 0; u < kSliceItems; ++u) k[u] = static_cast<const KeyT *>(key)[std::min(base + u * kRangeThreads, last)];
    }
    __syncthreads();  // the counters are clear, the previous tile has left the staging area
    uint32_t at[kSliceItems];  // slice << 16 | rank among the tile's items of the slice; kDead: not moved
#pragma unroll
    for (int u = 0; u < kSliceItems; ++u) {
      const uint32_t sl = p.slice(k[u]);
      at[u] = kDead;
      if (k[u] != kColumnEmpty<P::kWide> && base + u * kRangeThreads <= last && sl != kDead)
        at[u] = sl << 16 | static_cast<uint32_t>(atomicAdd(&s_cnt[sl], 1));
    }
    __syncthreads();
    if (tid < kWave) {
      int32_t a[4], la = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) la += a[j] = s_cnt[lane * 4 + j];
      const int32_t incl = wave_inclusive_scan(la);
      int32_t ra = incl - la;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        s_start[lane * 4 + j] = ra;
        s_next[lane * 4 + j] -= ra;  // the item at place p goes to s_next + p
        ra += a[j];
      }
      if (lane == kWave - 1) s_live = incl;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSliceItems; ++u) {
      const int32_t i = base + u * kRangeThreads;
      int32_t place = kNoMatchPos;
      if (at[u] != kDead) {
        place = s_start[at[u] >> 16] + static_cast<int32_t>(at[u] & 0xffff);
        s_dig[place] = static_cast<uint8_t>(at[u] >> 16);
        s_stage[place] = p.item(k[u], i);
      }
      if (P::kProbe && i <= last) d.pos[i] = static_cast<uint16_t>(place);
    }
    __syncthreads();
    const int live = s_live;
    for (int i = tid; i < live; i += kRangeThreads) {
      const int sl = s_dig[i];
      static_cast<Item *>(d.items)[s_next[sl] + i] = s_stage[i];
      if (P::kProbe) d.slice[t * kSliceTile + i] = static_cast<uint8_t>(sl);
    }
    if (P::kProbe) {
      if (tid < kRangeDigits) d.goff[t * kRangeDigits + tid] = static_cast<uint32_t>(s_next[tid]);
      if (tid == 0) d.live[t] = live;
    }
    __syncthreads();
    if (tid < kRangeDigits) s_next[tid] += s_start[tid] + s_cnt[tid];
  }
}

// Every moved build row into the array.  Blocks take consecutive pieces in
// XCD-major order, so that a slice is written through one L2.  (As many blocks as
// pieces: blocks that walk several drift apart, and with them the slices in use;
// 8 a CU measured 1003 us against 452 for 60M rows, the lookup 649 against 401.)
__global__ __launch_bounds__(256) void k_direct_store(DirectJoin d) {
  if (!d.plan->direct) return;
  constexpr int U = 8;
  const int64_t n = *d.build.moved, blocks = (n + 256 * U - 1) / (256 * U);
  if (blockIdx.x >= blocks) return;
  const int64_t i0 = xcd_block(blockIdx.x, blocks) * (256 * U) + threadIdx.x;
  uint64_t p[U];
#pragma unroll
  for (int u = 0; u < U; ++u) p[u] = i0 + u * 256 < n ? __builtin_nontemporal_load(static_cast<const uint64_t *>(d.build.items) + i0 + u * 256) : 0;
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (i0 + u * 256 < n) d.array[static_cast<uint32_t>(p[u])] = static_cast<int32_t>(p[u] >> 32);
}

__global__ __launch_bounds__(256) void k_direct_filled(DirectJoin d) {
  __shared__ int32_t s_c[4];
  if (!d.plan->direct) return;
  const int64_t range = static_cast<int64_t>(d.plan->range), quads = (range + 3) / 4, step = int64_t{gridDim.x} * 256;
  int32_t c = 0;
  for (int64_t i = int64_t{blockIdx.x} * 256 + threadIdx.x; i < quads; i += step) {
    const v4i32 v = reinterpret_cast<const v4i32 *>(d.array)[i];  // entries past the range are -1
    c += (v.x >= 0) + (v.y >= 0) + (v.z >= 0) + (v.w >= 0);
  }
  c = wave_sum(c);
  if (lane_id() == 0) s_c[threadIdx.x / kWave] = c;
  __syncthreads();
  if (threadIdx.x == 0)
    atomicAdd(&d.plan->filled, static_cast<unsigned long long>(s_c[0] + s_c[1] + s_c[2] + s_c[3]));
}

// The build row of every moved probe key, in place of its offset.
__global__ __launch_bounds__(256) void k_direct_lookup(DirectJoin d) {
  if (!d.plan->direct) return;
  constexpr int U = 8;
  const int64_t n = *d.probe.moved, blocks = (n + 256 * U - 1) / (256 * U);  // the blocks that have rows
  if (blockIdx.x >= blocks) return;
  const int64_t i0 = xcd_block(blockIdx.x, blocks) * (256 * U) + threadIdx.x;
  uint32_t *items = static_cast<uint32_t *>(d.probe.items);
  uint32_t o[U];
  int32_t r[U];
#pragma unroll
  for (int u = 0; u < U; ++u) o[u] = i0 + u * 256 < n ? __builtin_nontemporal_load(&items[i0 + u * 256]) : 0;
#pragma unroll
  for (int u = 0; u < U; ++u) r[u] = d.array[o[u]];
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (i0 + u * 256 < n) __builtin_nontemporal_store(static_cast<uint32_t>(r[u]), &items[i0 + u * 256]);
}

// The payload of every moved probe key of a hash table with unique keys, in
// place of the key, and a bit for those that have one.  A lane's keys walk their
// runs together, in the L2's slice of the table.
template <bool WIDE, bool K64>
__global__ __launch_bounds__(256) void k_hash_lookup(HashRows<WIDE, K64> p, Slices d, const uint64_t *slots) {
  using Item = typename HashRows<WIDE, K64>::Item;
  using Stored = std::conditional_t<WIDE, int64_t, int32_t>;
  constexpr int U = WIDE ? 4 : 8;
  constexpr int64_t GS = WIDE ? 1 : 2;
  if (!p.open()) return;
  const int64_t n = *d.moved, blocks = (n + 256 * U - 1) / (256 * U), mask = p.mask;
  if (blockIdx.x >= blocks) return;
  const int64_t i0 = xcd_block(blockIdx.x, blocks) * (256 * U) + threadIdx.x;
  Item *items = static_cast<Item *>(d.items);
  Stored k[U], pay[U];
  int32_t c[U];
  uint32_t on = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    k[u] = static_cast<Stored>(i0 + u * 256 < n ? __builtin_nontemporal_load(&items[i0 + u * 256]) : 0);
    on |= i0 + u * 256 < n ? 1u << u : 0;
    c[u] = 0;
    pay[u] = 0;
  }
  for (int64_t step = 0; step <= mask && __any(on != 0); step += GS) {
    ulonglong2 g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int64_t s;
      if constexpr (WIDE) s = static_cast<int64_t>((table_hash64(k[u]) & static_cast<uint64_t>(mask)) + step) & mask;
      else s = static_cast<int64_t>((table_hash32(k[u]) & static_cast<uint64_t>(mask) & ~uint64_t{1}) + step) & mask;
      if ((on >> u) & 1) g[u] = *reinterpret_cast<const ulonglong2 *>(&slots[WIDE ? 2 * s : s]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!((on >> u) & 1)) continue;
      bool more;
      if constexpr (WIDE) more = visit_wide(g[u], k[u], 1, c[u], pay[u]);
      else more = visit_pair(g[u], k[u], 1, c[u], pay[u]);
      if (!more) on &= ~(1u << u);
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint64_t m = __ballot(c[u] != 0);
    const int64_t i = i0 + u * 256;
    if (i < n) {
      __builtin_nontemporal_store(static_cast<Item>(pay[u]), &items[i]);
      if (lane_id() == 0) d.found[i / kWave] = m;  // i is a multiple of 64 in lane 0
    }
  }
}

// Matches in ascending probe row: a tile's results back in row order, compacted
// by look-back over the tiles.  HASH: results are payloads with found bits, else
// build rows, -1 for none.
template <typename Item, bool HASH, typename PayT>
__global__ __launch_bounds__(kRangeThreads, 8) void k_slice_emit(const JoinPlan *plan, ProbeRule rule, Slices d, const int32_t *sel,
                                                                const int64_t *d_nsel, int64_t n_all, int32_t *out_row,
                                                                PayT *out_pay, int64_t out_cap, int64_t *d_nout,
                                                                uint32_t *err) {
  constexpr int NW = kRangeThreads / kWave;
  using Res = std::make_signed_t<Item>;
  __shared__ Res s_res[kSliceTile];
  __shared__ uint8_t s_ok[HASH ? kSliceTile : 1];
  __shared__ uint32_t s_goff[kRangeDigits];
  __shared__ int32_t s_w[NW];
  __shared__ int64_t s_tile, s_prefix;
  if (plan && (plan->direct != 0) == HASH) return;
  if (HASH && rule.not_by_slices()) return;
  const int64_t n = std::min(count_of(d_nsel, n_all), n_all), ntiles = (n + kSliceTile - 1) / kSliceTile;
  const int tid = static_cast<int>(threadIdx.x), w = tid / kWave, lane = lane_id();
  if (blockIdx.x >= ntiles) {
    if (ntiles == 0 && blockIdx.x == 0 && tid == 0) *d_nout = 0;
    return;
  }
  if (tid == 0) s_tile = static_cast<int64_t>(atomicAdd(d.ticket, 1ull));
  __syncthreads();
  const int64_t t = s_tile;
  if (!HASH && t == 0 && tid == 0 && plan->filled != static_cast<unsigned long long>(plan->moved[0])) latch(err, kErrDup);
  const int live = d.live[t];
  if (tid < kRangeDigits) s_goff[tid] = d.goff[t * kRangeDigits + tid];
  const int64_t base = t * kSliceTile + w * (kWave * kSliceItems) + lane;
  uint16_t pos[kSliceItems];
  uint8_t sl[kSliceItems];
#pragma unroll
  for (int u = 0; u < kSliceItems; ++u) {
    pos[u] = d.pos[base + u * kWave < n ? base + u * kWave : n - 1];
    sl[u] = d.slice[t * kSliceTile + u * kRangeThreads + tid];  // (undefined past the live ones: not used)
  }
  __syncthreads();
  {
    Res x[kSliceItems];
    uint8_t f[kSliceItems];
#pragma unroll
    for (int u = 0; u < kSliceItems; ++u) {
      const int p = u * kRangeThreads + tid;
      x[u] = -1;
      f[u] = 0;
      if (p < live) {
        const int64_t g = int64_t{s_goff[sl[u]]} + p;
        x[u] = static_cast<Res>(__builtin_nontemporal_load(static_cast<const Item *>(d.items) + g));
        if (HASH) f[u] = reinterpret_cast<const uint8_t *>(d.found)[g >> 3] >> (g & 7) & 1;
      }
    }
#pragma unroll
    for (int u = 0; u < kSliceItems; ++u) {
      s_res[u * kRangeThreads + tid] = x[u];
      if (HASH) s_ok[u * kRangeThreads + tid] = f[u];
    }
  }
  __syncthreads();
  uint64_t m[kSliceItems];
  int cnt = 0;
#pragma unroll
  for (int u = 0; u < kSliceItems; ++u) {
    const bool moved = pos[u] != kNoMatchPos && base + u * kWave < n;
    const bool hit = moved && (HASH ? s_ok[pos[u]] != 0 : s_res[pos[u]] >= 0);
    m[u] = __ballot(hit);
    cnt += __popcll(m[u]);
  }
  if (lane == 0) s_w[w] = cnt;
  __syncthreads();
  if (w == 0) {
    const int64_t c = lane < NW ? s_w[lane] : 0;
    const int64_t agg = wave_sum(c), ex = lookback_exclusive(d.status, t, agg);
    if (lane == 0) {
      s_prefix = ex;
      if (t == ntiles - 1) {
        *d_nout = ex + agg;
        if (ex + agg > out_cap) latch(err, kErrCapacity);
      }
    }
  }
  __syncthreads();
  int64_t at = s_prefix;
  for (int k = 0; k < w; ++k) at += s_w[k];
#pragma unroll
  for (int u = 0; u < kSliceItems; ++u) {
    const int64_t p = at + mbcnt(m[u]);
    if (((m[u] >> lane) & 1ull) && p < out_cap) {
      out_row[p] = static_cast<int32_t>(row_of(sel, base + u * kWave));
      out_pay[p] = static_cast<PayT>(s_res[pos[u]]);
    }
    at += __popcll(m[u]);
  }
}

// Rows below which a side's keys are not split: the hash table of a smaller
// build side lies mostly in the L2s, and fewer probes do not pay for the moves.
constexpr int64_t kDirectBuildMin = int64_t{1} << 21;
constexpr int64_t kDirectProbeMin = int64_t{1} << 21;
constexpr int64_t kDirectRangeMax = int64_t{1} << 32;  // values of an item's offset

bool direct_join_wanted(const pyst_col *build_key, const pyst_col *probe_key, int unique) {
  return unique && build_key->n >= kDirectBuildMin && probe_key->n >= kDirectProbeMin;
}

static size_t align256(size_t b) { return (b + 255) / 256 * 256; }

// A cursor over scratch memory (null: measures).
struct Layout {
  char *mem;
  size_t at = 0;
  template <typename T>
  T *take(size_t bytes) {
    char *p = mem ? mem + at : nullptr;
    at += align256(bytes);
    return reinterpret_cast<T *>(p);
  }
};

// The way back of a probe of np rows whose items take `item` bytes.
static void probe_layout(Layout &l, int64_t np, size_t item, bool found, Slices *s) {
  s->ntiles = ceil_div(np, kSliceTile);
  const size_t tiles = static_cast<size_t>(s->ntiles);
  s->status = l.take<uint64_t>(tiles * 8);
  if (item) s->items = l.take<void>(item * static_cast<size_t>(np));
  s->found = found ? l.take<uint64_t>(static_cast<size_t>(ceil_div(np, kWave)) * 8) : nullptr;
  s->pos = l.take<uint16_t>(2 * static_cast<size_t>(np));
  s->slice = l.take<uint8_t>(tiles * kSliceTile);
  s->goff = l.take<uint32_t>(tiles * kRangeDigits * 4);
  s->live = l.take<int32_t>(tiles * 4);
}

// Scratch of a direct join beside its array, and its layout at `mem`.
static size_t direct_layout(char *mem, int64_t nb, int64_t np, DirectJoin *d, int64_t **lo) {
  const int parts = std::max(range_parts(nb, kSliceTile), range_parts(np, kSliceTile));
  Layout l{mem};
  d->plan = l.take<JoinPlan>(sizeof(JoinPlan));
  *lo = l.take<int64_t>(2 * kJoinRangeBlocks * sizeof(int64_t));
  void *counts = l.take<void>(range_count_words(parts, 2) * sizeof(uint32_t));
  void *items = l.take<void>(std::max<size_t>(8 * static_cast<size_t>(nb), 4 * static_cast<size_t>(np)));
  d->build = d->probe = Slices{};
  probe_layout(l, np, 0, false, &d->probe);
  if (mem) {
    d->build.counts = d->probe.counts = range_counts_at(counts, parts);
    d->build.items = d->probe.items = items;
    d->build.moved = &d->plan->moved[0];
    d->probe.moved = &d->plan->moved[1];
    d->probe.pass = 1;
    d->probe.ticket = &d->plan->ticket;
  }
  return l.at;
}

size_t direct_join_bytes(int64_t nb, int64_t np) {
  DirectJoin d{};
  int64_t *lo;
  return direct_layout(nullptr, nb, np, &d, &lo);
}

template <typename P>
static void launch_slices(const P &p, const Slices &d, const pyst_col *key, const int32_t *sel, const int64_t *d_nsel,
                          hipStream_t stream) {
  const int parts = range_parts(key->n, kSliceTile);
  k_slice_hist<P><<<parts, kRangeThreads, 0, stream>>>(p, d, key->data, sel, d_nsel, key->n);
  k_slice_move<P><<<parts, kRangeThreads, 0, stream>>>(p, d, key->data, sel, d_nsel, key->n);
}

// The build side's plan and, where it is direct, its array in `array` (room for
// range_max entries, a multiple of 4).  *plan: for the hash table's kernels.
pyst_status direct_join_build(pyst_ctx *ctx, const pyst_col *build_key, int64_t np, void *ws, int32_t *array,
                              int64_t range_max, const JoinPlan **plan, hipStream_t stream) {
  DirectJoin d{};
  int64_t *lo = nullptr;
  direct_layout(static_cast<char *>(ws), build_key->n, np, &d, &lo);
  d.array = array;
  *plan = d.plan;
  const int64_t nb = build_key->n;
  const bool k64 = build_key->dtype == PYST_I64;
  const int rblocks = static_cast<int>(std::min<int64_t>(kJoinRangeBlocks, ceil_div(nb, 2048)));
  k64 ? k_join_range<true><<<rblocks, 256, 0, stream>>>(build_key->data, nb, lo, lo + kJoinRangeBlocks, ctx_err_word(ctx))
      : k_join_range<false><<<rblocks, 256, 0, stream>>>(build_key->data, nb, lo, lo + kJoinRangeBlocks, ctx_err_word(ctx));
  PYST_LAUNCH_CHECK("k_join_range");
  k_join_plan<<<1, kRangeThreads, 0, stream>>>(d.plan, lo, lo + kJoinRangeBlocks, rblocks,
                                              static_cast<uint64_t>(std::min(range_max, kDirectRangeMax)), d.build.counts);
  PYST_LAUNCH_CHECK("k_join_plan");
  k_direct_clear<<<grid_for(ctx, range_max / 4, 256, 8), 256, 0, stream>>>(d);
  PYST_LAUNCH_CHECK("k_direct_clear");
  if (k64) launch_slices(DirectRows<true, true>{d.plan}, d.build, build_key, nullptr, nullptr, stream);
  else launch_slices(DirectRows<false, true>{d.plan}, d.build, build_key, nullptr, nullptr, stream);
  PYST_LAUNCH_CHECK("k_slice_move");
  k_direct_store<<<static_cast<unsigned>(ceil_div(nb, 2048)), 256, 0, stream>>>(d);
  PYST_LAUNCH_CHECK("k_direct_store");
  k_direct_filled<<<std::min(512, grid_for(ctx, range_max / 4, 256, 8)), 256, 0, stream>>>(d);
  PYST_LAUNCH_CHECK("k_direct_filled");
  return PYST_OK;
}

pyst_status direct_join_probe(pyst_ctx *ctx, int64_t nb, const pyst_col *probe_key, void *ws, int32_t *array,
                              int32_t *out_row, int32_t *out_build, int64_t out_cap, int64_t *d_nout, hipStream_t stream) {
  DirectJoin d{};
  int64_t *lo = nullptr;
  const int64_t np = probe_key->n;
  direct_layout(static_cast<char *>(ws), nb, np, &d, &lo);
  d.array = array;
  if (probe_key->dtype == PYST_I64) launch_slices(DirectRows<true, false>{d.plan}, d.probe, probe_key, nullptr, nullptr, stream);
  else launch_slices(DirectRows<false, false>{d.plan}, d.probe, probe_key, nullptr, nullptr, stream);
  PYST_LAUNCH_CHECK("k_slice_move");
  k_direct_lookup<<<static_cast<unsigned>(ceil_div(np, 2048)), 256, 0, stream>>>(d);
  PYST_LAUNCH_CHECK("k_direct_lookup");
  k_slice_emit<uint32_t, false, int32_t><<<static_cast<unsigned>(d.probe.ntiles), kRangeThreads, 0, stream>>>(
      d.plan, ProbeRule{}, d.probe, nullptr, nullptr, np, out_row, out_build, out_cap, d_nout, ctx_err_word(ctx));
  PYST_LAUNCH_CHECK("k_slice_emit");
  return PYST_OK;
}

// ---------------------------------------------------------------- hash tables beyond the L2
// Probes of a unique-key hash table far larger than the L2, by slices of 2 MiB of
// its slots (or the table's 256th part), through the same moves and the same way
// back.  From 16 MiB of slots (an XCD's L2 holds 4) and 2^21 probes: below, the
// moves cost what the lines do (600k keys, 2.5M probes 179 -> 164 us; 400k 64-bit
// keys, 8 MiB, stay as they were).  20M probes of a 1M-key table of 16-byte slots
// 680 -> 465 us (counts 43, move 87, lookup 226, way back 109); 50M of 9M int32
// keys with build 1625 -> 1339 us; a 20M x 60M join of sparse 64-bit keys 3993 ->
// 3726 us.  Duplicate keys (any number of matches a row) and arenas without room
// keep k_join_probe; for tables built from a selection the device chooses (ProbeRule).
constexpr int64_t kHashTableMin = int64_t{16} << 20;   // bytes
constexpr int64_t kHashProbeMin = int64_t{1} << 21;    // rows
constexpr int kHashSliceLg = 21;                       // bytes a slice

bool sliced_probe_wanted(const TableDev &t, int unique, const pyst_col *key) {
  return unique && key->n >= kHashProbeMin && t.cap_alloc * t.slot_bytes >= kHashTableMin;
}

struct HashProbe {
  uint32_t *head;  // cleared: ticket, moved rows (nothing writes them where no row is selected), then the group counts
  int64_t head_words;
  Slices s;
};

static size_t hash_probe_layout(char *mem, int64_t np, int slot_bytes, HashProbe *h) {
  const int parts = range_parts(np, kSliceTile);
  Layout l{mem};
  const int64_t groups = ceil_div(parts, kRangeGroup) * kRangeDigits;
  h->head_words = 64 + groups;
  h->head = l.take<uint32_t>(static_cast<size_t>(h->head_words) * 4);
  uint32_t *part = l.take<uint32_t>(static_cast<size_t>(parts) * kRangeDigits * 4);
  h->s = Slices{};
  probe_layout(l, np, slot_bytes == 16 ? 8 : 4, true, &h->s);
  if (mem) {
    h->s.counts.part = part;
    h->s.counts.group = h->head + 64;
    h->s.counts.ngroups = static_cast<int>(ceil_div(parts, kRangeGroup));
    h->s.ticket = reinterpret_cast<unsigned long long *>(h->head);
    h->s.moved = reinterpret_cast<int64_t *>(h->head + 2);
  }
  return l.at;
}

size_t sliced_probe_bytes(const TableDev &t, const pyst_col *key) {
  HashProbe h{};
  return hash_probe_layout(nullptr, key->n, t.slot_bytes, &h);
}

template <bool WIDE, bool K64, typename PayT>
static pyst_status launch_sliced_probe(pyst_ctx *ctx, const TableDev &t, const pyst_col *key, const int32_t *sel,
                                       const int64_t *d_nsel, const HashProbe &h, int32_t *out_row, PayT *out_pay,
                                       int64_t out_cap, int64_t *d_nout, const JoinPlan *plan, const ProbeRule &rule,
                                       hipStream_t stream) {
  using P = HashRows<WIDE, K64>;
  P p{plan, t.hdr, kHashSliceLg - (WIDE ? 4 : 3), rule};
  while (((t.cap_alloc - 1) >> p.shift) >= kRangeDigits) ++p.shift;
  launch_slices(p, h.s, key, sel, d_nsel, stream);
  PYST_LAUNCH_CHECK("k_slice_move");
  k_hash_lookup<WIDE, K64><<<static_cast<unsigned>(ceil_div(key->n, WIDE ? 1024 : 2048)), 256, 0, stream>>>(
      p, h.s, static_cast<const uint64_t *>(t.slots));
  PYST_LAUNCH_CHECK("k_hash_lookup");
  k_slice_emit<typename P::Item, true, PayT><<<static_cast<unsigned>(h.s.ntiles), kRangeThreads, 0, stream>>>(
      plan, rule, h.s, sel, d_nsel, key->n, out_row, out_pay, out_cap, d_nout, ctx_err_word(ctx));
  PYST_LAUNCH_CHECK("k_slice_emit");
  return PYST_OK;
}

ProbeRule sliced_probe_rule(const TableDev &t, const pyst_col *key, const int64_t *d_nsel) {
  ProbeRule r;
  r.hdr = t.hdr;
  r.d_nsel = d_nsel;
  r.n = key->n;
  r.slots_min = kHashTableMin / t.slot_bytes;
  return r;
}

// launch_join_probe's results through slices, in `ws` of `lead` bytes (a multiple
// of 256, cleared with the scratch's head) and sliced_probe_bytes.
template <typename PayT>
pyst_status sliced_probe(pyst_ctx *ctx, const TableDev &t, const pyst_col *key, const int32_t *sel, const int64_t *d_nsel,
                         void *ws, size_t lead, int32_t *out_row, PayT *out_pay, int64_t out_cap, int64_t *d_nout,
                         const JoinPlan *plan, const ProbeRule &rule, hipStream_t stream) {
  HashProbe h{};
  hash_probe_layout(static_cast<char *>(ws) + lead, key->n, t.slot_bytes, &h);
  const pyst_status st = fill_u32(ws, static_cast<int64_t>(lead / 4) + h.head_words, 0, stream);
  if (st != PYST_OK) return st;
  const bool k64 = key->dtype == PYST_I64;
  if (t.slot_bytes == 16)
    return k64 ? launch_sliced_probe<true, true>(ctx, t, key, sel, d_nsel, h, out_row, out_pay, out_cap, d_nout, plan, rule, stream)
               : launch_sliced_probe<true, false>(ctx, t, key, sel, d_nsel, h, out_row, out_pay, out_cap, d_nout, plan, rule, stream);
  return k64 ? launch_sliced_probe<false, true>(ctx, t, key, sel, d_nsel, h, out_row, out_pay, out_cap, d_nout, plan, rule, stream)
             : launch_sliced_probe<false, false>(ctx, t, key, sel, d_nsel, h, out_row, out_pay, out_cap, d_nout, plan, rule, stream);
}
template pyst_status sliced_probe<int32_t>(pyst_ctx *, const TableDev &, const pyst_col *, const int32_t *, const int64_t *,
                                           void *, size_t, int32_t *, int32_t *, int64_t, int64_t *, const JoinPlan *,
                                           const ProbeRule &, hipStream_t);
template pyst_status sliced_probe<int64_t>(pyst_ctx *, const TableDev &, const pyst_col *, const int32_t *, const int64_t *,
                                           void *, size_t, int32_t *, int64_t *, int64_t, int64_t *, const JoinPlan *,
                                           const ProbeRule &, hipStream_t);

}  // namespace pyst
