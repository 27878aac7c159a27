// Equi-join of large sides whose build keys are dense (surrogate keys): the
// build side as an array of row ids indexed by key - least key, built and read
// slice by slice.
//
// A hash join of these sizes is bound by memory lines: every insert and every
// probe of a table far beyond the L2 moves a whole 128-byte line for 4 useful
// bytes (60M inserts 2.9 ms, 160M probes 5.1 ms, at 4 - 5 TB/s of lines).  Here
// both sides are first split by key into slices of 2^19 keys (2 MiB of the
// array, which one XCD's L2 holds beside the stream): a counting and a moving
// kernel over the keys alone.  The stores and loads of the array then hit the
// L2.  Probe rows that no build key can match are dropped by the move.
// The probe rows have to come out in their own order: the move records where
// each row's key went within its tile (2 bytes a row) and which slice each moved
// key of the tile belongs to (1 byte), so that the last kernel reads a tile's
// results back as contiguous runs, puts them in row order through LDS and
// compacts the matches.
//
// Bound by streams: 60M build rows 12 + 20 bytes a row, 160M probe rows about 24
// bytes a row.  Measured: JOIN_FIGURES
//
// The choice is made on the device from the build keys' range: direct where the
// keys span no more values than the hash table has slots, else the hash table's
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

struct DirectJoin {
  JoinPlan *plan;
  int32_t *array;       // row id by key - kmin, -1 for none
  RangeCounts counts;   // pass 0: build, 1: probe
  uint64_t *status;     // look-back words of the emitting kernel, one per probe tile
  int64_t ntiles;       // probe tiles
  uint64_t *pairs;      // moved build rows: offset | row << 32
  uint32_t *moved;      // moved probe offsets, then their build rows (in place)
  uint16_t *pos;        // per probe row: its place in its tile's moved keys
  uint8_t *slice;       // per (tile, place): the slice
  uint32_t *goff;       // per (tile, slice): where place 0 of the tile would lie
  int32_t *live;        // per tile: moved keys
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
  for (int64_t i = i0; i < d.ntiles; i += step) d.status[i] = 0;
}

template <bool K64>
__global__ __launch_bounds__(kRangeThreads, 8) void k_slice_hist(DirectJoin d, int pass, const void *key, int64_t n) {
  __shared__ uint32_t s_h[kRangeDigits];
  int64_t part, t0, t1;
  if (!d.plan->direct || !range_of_block(n, kSliceTile, part, t0, t1)) return;
  const int tid = static_cast<int>(threadIdx.x), shift = d.plan->shift;
  const int64_t kmin = d.plan->kmin;
  const uint64_t range = d.plan->range;
  if (tid < kRangeDigits) s_h[tid] = 0;
  __syncthreads();
  const int64_t hi = t1 * kSliceTile < n ? t1 * kSliceTile : n;
  for (int64_t i0 = t0 * kSliceTile + tid; i0 < hi; i0 += kSliceTile) {
    int64_t k[kSliceItems];
    bool ok[kSliceItems];
#pragma unroll
    for (int u = 0; u < kSliceItems; ++u) {
      const int64_t i = i0 + u * kRangeThreads;
      ok[u] = slice_key<K64>(key, i < hi ? i : i0, k[u]) && i < hi;
    }
#pragma unroll
    for (int u = 0; u < kSliceItems; ++u) {
      const uint64_t off = static_cast<uint64_t>(k[u]) - static_cast<uint64_t>(kmin);
      if (ok[u] && off < range) atomicAdd(&s_h[off >> shift], 1u);
    }
  }
  __syncthreads();
  if (tid < kRangeDigits) {
    d.counts.of_part(part)[tid] = s_h[tid];
    if (s_h[tid]) atomicAdd(&d.counts.of_group(pass, part / kRangeGroup)[tid], s_h[tid]);
  }
}

// Moves the offsets (BUILD: with their rows) of a block's range of tiles to
// their slices.  A tile is laid out by slice in LDS and leaves as one run a
// slice.  Two blocks of 16 waves per CU.
template <bool K64, bool BUILD>
__global__ __launch_bounds__(kRangeThreads, 8) void k_slice_move(DirectJoin d, const void *key, int64_t n) {
  using Item = std::conditional_t<BUILD, uint64_t, uint32_t>;
  using KeyT = std::conditional_t<K64, int64_t, int32_t>;
  constexpr KeyT kColEmpty = K64 ? static_cast<KeyT>(kEmpty64) : static_cast<KeyT>(kEmpty32);
  constexpr uint32_t kDead = 0xffffffffu;
  __shared__ __align__(16) Item s_stage[kSliceTile];
  __shared__ uint8_t s_dig[kSliceTile];
  __shared__ int32_t s_cnt[kRangeDigits], s_start[kRangeDigits];
  __shared__ int64_t s_next[kRangeDigits];
  __shared__ int32_t s_live;
  static_assert(sizeof(RangeOffsets) <= sizeof(s_stage), "the offsets are summed in the staging area");
  int64_t part, t0, t1;
  if (!d.plan->direct || !range_of_block(n, kSliceTile, part, t0, t1)) return;
  const int tid = static_cast<int>(threadIdx.x), lane = lane_id(), shift = d.plan->shift;
  const int64_t kmin = d.plan->kmin;
  const uint64_t range = d.plan->range;
  const int64_t total = range_offsets(d.counts, BUILD ? 0 : 1, static_cast<int>(part),
                                      *reinterpret_cast<RangeOffsets *>(s_stage), s_next);
  if (part == 0 && tid == 0) d.plan->moved[BUILD ? 0 : 1] = total;
  for (int64_t t = t0; t < t1; ++t) {  // block-uniform
    if (tid < kRangeDigits) s_cnt[tid] = 0;
    const int32_t base = static_cast<int32_t>(t) * kSliceTile + tid, last = static_cast<int32_t>(n) - 1;
    KeyT k[kSliceItems];
#pragma unroll
    for (int u = 0; u < kSliceItems; ++u) {
      const int32_t i = base + u * kRangeThreads;
      k[u] = static_cast<const KeyT *>(key)[i < last ? i : last];
    }
    __syncthreads();  // the counters are clear, the previous tile has left the staging area
    uint32_t off[kSliceItems];  // kDead: no row, an EMPTY key, or one outside the build keys' range
    int32_t rank[kSliceItems];
#pragma unroll
    for (int u = 0; u < kSliceItems; ++u) {
      const uint64_t o = static_cast<uint64_t>(static_cast<int64_t>(k[u])) - static_cast<uint64_t>(kmin);
      const bool ok = k[u] != kColEmpty && base + u * kRangeThreads <= last && o < range;
      off[u] = ok ? static_cast<uint32_t>(o) : kDead;
      rank[u] = ok ? atomicAdd(&s_cnt[off[u] >> shift], 1) : 0;
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
        s_next[lane * 4 + j] -= ra;  // the key at place p goes to s_next + p
        ra += a[j];
      }
      if (lane == kWave - 1) s_live = incl;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSliceItems; ++u) {
      const int32_t i = base + u * kRangeThreads;
      int32_t p = kNoMatchPos;
      if (off[u] != kDead) {
        const uint32_t s = off[u] >> shift;
        p = s_start[s] + rank[u];
        s_dig[p] = static_cast<uint8_t>(s);
        if constexpr (BUILD) s_stage[p] = off[u] | (static_cast<uint64_t>(static_cast<uint32_t>(i)) << 32);
        else s_stage[p] = off[u];
      }
      if (!BUILD && i <= last) d.pos[i] = static_cast<uint16_t>(p);
    }
    __syncthreads();
    const int live = s_live;
    for (int p = tid; p < live; p += kRangeThreads) {
      const int s = s_dig[p];
      if constexpr (BUILD) d.pairs[s_next[s] + p] = s_stage[p];
      else {
        d.moved[s_next[s] + p] = s_stage[p];
        d.slice[t * kSliceTile + p] = static_cast<uint8_t>(s);
      }
    }
    if (!BUILD) {
      if (tid < kRangeDigits) d.goff[t * kRangeDigits + tid] = static_cast<uint32_t>(s_next[tid]);
      if (tid == 0) d.live[t] = live;
    }
    __syncthreads();
    if (tid < kRangeDigits) s_next[tid] += s_start[tid] + s_cnt[tid];
  }
}

// Every moved build row into the array.  Blocks take consecutive pieces in
// XCD-major order, so that a slice is written through one L2.
__global__ __launch_bounds__(256) void k_direct_store(DirectJoin d) {
  if (!d.plan->direct) return;
  constexpr int U = 8;
  const int64_t n = d.plan->moved[0], blocks = (n + 256 * U - 1) / (256 * U);
  if (blockIdx.x >= blocks) return;
  const int64_t i0 = xcd_block(blockIdx.x, blocks) * (256 * U) + threadIdx.x;
  uint64_t p[U];
#pragma unroll
  for (int u = 0; u < U; ++u) p[u] = i0 + u * 256 < n ? __builtin_nontemporal_load(&d.pairs[i0 + u * 256]) : 0;
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
  const int64_t n = d.plan->moved[1], blocks = (n + 256 * U - 1) / (256 * U);  // the blocks that have rows
  if (blockIdx.x >= blocks) return;
  const int64_t i0 = xcd_block(blockIdx.x, blocks) * (256 * U) + threadIdx.x;
  uint32_t o[U];
  int32_t r[U];
#pragma unroll
  for (int u = 0; u < U; ++u) o[u] = i0 + u * 256 < n ? __builtin_nontemporal_load(&d.moved[i0 + u * 256]) : 0;
#pragma unroll
  for (int u = 0; u < U; ++u) r[u] = d.array[o[u]];
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (i0 + u * 256 < n) __builtin_nontemporal_store(static_cast<uint32_t>(r[u]), &d.moved[i0 + u * 256]);
}

// Matches in ascending probe row: a tile's results back in row order, compacted
// by look-back over the tiles.
__global__ __launch_bounds__(kRangeThreads, 8) void k_direct_emit(DirectJoin d, int64_t n, int32_t *out_row,
                                                                 int32_t *out_build, int64_t out_cap, int64_t *d_nout,
                                                                 uint32_t *err) {
  constexpr int NW = kRangeThreads / kWave;
  __shared__ int32_t s_res[kSliceTile];
  __shared__ uint32_t s_goff[kRangeDigits];
  __shared__ int32_t s_w[NW];
  __shared__ int64_t s_tile, s_prefix;
  if (!d.plan->direct) return;
  const int tid = static_cast<int>(threadIdx.x), w = tid / kWave, lane = lane_id();
  if (tid == 0) s_tile = static_cast<int64_t>(atomicAdd(&d.plan->ticket, 1ull));
  __syncthreads();
  const int64_t t = s_tile;
  if (t == 0 && tid == 0 && d.plan->filled != static_cast<unsigned long long>(d.plan->moved[0])) latch(err, kErrDup);
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
  int32_t r[kSliceItems];
#pragma unroll
  for (int u = 0; u < kSliceItems; ++u) {
    const int p = u * kRangeThreads + tid;
    r[u] = p < live ? static_cast<int32_t>(__builtin_nontemporal_load(&d.moved[int64_t{s_goff[sl[u]]} + p])) : -1;
  }
#pragma unroll
  for (int u = 0; u < kSliceItems; ++u) s_res[u * kRangeThreads + tid] = r[u];
  __syncthreads();
  uint64_t m[kSliceItems];
  int cnt = 0;
#pragma unroll
  for (int u = 0; u < kSliceItems; ++u) {
    r[u] = pos[u] != kNoMatchPos && base + u * kWave < n ? s_res[pos[u]] : -1;
    m[u] = __ballot(r[u] >= 0);
    cnt += __popcll(m[u]);
  }
  if (lane == 0) s_w[w] = cnt;
  __syncthreads();
  if (w == 0) {
    const int64_t c = lane < NW ? s_w[lane] : 0;
    const int64_t agg = wave_sum(c), ex = lookback_exclusive(d.status, t, agg);
    if (lane == 0) {
      s_prefix = ex;
      if (t == d.ntiles - 1) {
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
    if (r[u] >= 0 && p < out_cap) {
      out_row[p] = static_cast<int32_t>(base + u * kWave);
      out_build[p] = r[u];
    }
    at += __popcll(m[u]);
  }
}

// Rows below which a side's keys are not split: the hash table of a smaller
// build side lies mostly in the L2s, and fewer probes do not pay for the moves.
constexpr int64_t kDirectBuildMin = int64_t{1} << 21;
constexpr int64_t kDirectProbeMin = int64_t{1} << 21;

bool direct_join_wanted(const pyst_col *build_key, const pyst_col *probe_key, int unique) {
  return unique && build_key->n >= kDirectBuildMin && probe_key->n >= kDirectProbeMin;
}

static size_t align256(size_t b) { return (b + 255) / 256 * 256; }

// Scratch beside the array, and its layout at `mem` (null: the size alone).
static size_t direct_layout(char *mem, int64_t nb, int64_t np, DirectJoin *d, int64_t **lo) {
  const int parts = std::max(range_parts(nb, kSliceTile), range_parts(np, kSliceTile));
  const int64_t ntiles = ceil_div(np, kSliceTile);
  size_t at = 0;
  auto take = [&](size_t bytes) {
    char *p = mem ? mem + at : nullptr;
    at += align256(bytes);
    return p;
  };
  char *plan = take(sizeof(JoinPlan)), *part = take(2 * kJoinRangeBlocks * sizeof(int64_t));
  char *counts = take(range_count_words(parts, 2) * sizeof(uint32_t)), *status = take(ntiles * sizeof(uint64_t));
  char *moved = take(std::max<size_t>(8 * static_cast<size_t>(nb), 4 * static_cast<size_t>(np)));
  char *pos = take(2 * static_cast<size_t>(np)), *slice = take(static_cast<size_t>(ntiles) * kSliceTile);
  char *goff = take(static_cast<size_t>(ntiles) * kRangeDigits * 4), *live = take(static_cast<size_t>(ntiles) * 4);
  if (mem) {
    *lo = reinterpret_cast<int64_t *>(part);
    d->plan = reinterpret_cast<JoinPlan *>(plan);
    d->counts = range_counts_at(counts, parts);
    d->status = reinterpret_cast<uint64_t *>(status);
    d->ntiles = ntiles;
    d->pairs = reinterpret_cast<uint64_t *>(moved);
    d->moved = reinterpret_cast<uint32_t *>(moved);
    d->pos = reinterpret_cast<uint16_t *>(pos);
    d->slice = reinterpret_cast<uint8_t *>(slice);
    d->goff = reinterpret_cast<uint32_t *>(goff);
    d->live = reinterpret_cast<int32_t *>(live);
  }
  return at;
}

size_t direct_join_bytes(int64_t nb, int64_t np) { return direct_layout(nullptr, nb, np, nullptr, nullptr); }

template <bool K64>
static void launch_slices(const DirectJoin &d, const pyst_col *key, bool build, hipStream_t stream) {
  const int parts = range_parts(key->n, kSliceTile);
  k_slice_hist<K64><<<parts, kRangeThreads, 0, stream>>>(d, build ? 0 : 1, key->data, key->n);
  if (build) k_slice_move<K64, true><<<parts, kRangeThreads, 0, stream>>>(d, key->data, key->n);
  else k_slice_move<K64, false><<<parts, kRangeThreads, 0, stream>>>(d, key->data, key->n);
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
                                              static_cast<uint64_t>(range_max), d.counts);
  PYST_LAUNCH_CHECK("k_join_plan");
  k_direct_clear<<<grid_for(ctx, range_max / 4, 256, 8), 256, 0, stream>>>(d);
  PYST_LAUNCH_CHECK("k_direct_clear");
  k64 ? launch_slices<true>(d, build_key, true, stream) : launch_slices<false>(d, build_key, true, stream);
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
  probe_key->dtype == PYST_I64 ? launch_slices<true>(d, probe_key, false, stream)
                               : launch_slices<false>(d, probe_key, false, stream);
  PYST_LAUNCH_CHECK("k_slice_move");
  k_direct_lookup<<<static_cast<unsigned>(ceil_div(np, 2048)), 256, 0, stream>>>(d);
  PYST_LAUNCH_CHECK("k_direct_lookup");
  k_direct_emit<<<static_cast<unsigned>(d.ntiles), kRangeThreads, 0, stream>>>(d, np, out_row, out_build, out_cap, d_nout,
                                                                              ctx_err_word(ctx));
  PYST_LAUNCH_CHECK("k_direct_emit");
  return PYST_OK;
}

}  // namespace pyst
