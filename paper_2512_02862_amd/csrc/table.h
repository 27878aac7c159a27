// Hash-table layouts shared by the join, group-by and fused-query kernels.
//
// Join table: power-of-two capacity, linear probing from a 16-byte aligned
// start, so one vector load covers the first 4 (4-byte key slots) or 2
// (8-byte key|payload slots) candidates.  Inserts take the first EMPTY slot of
// the sequence by compare-and-swap, so the occupied slots of any probe
// sequence form a prefix and an EMPTY slot ends a probe.
//
// Group table: 16-byte slots {int64 key, uint64 sum}, key inserted by CAS and
// the sum accumulated with a 64-bit atomic add (wraps modulo 2^64).
//
// Capacity: the smallest power of two >= max(64, cnt / max_load, cnt + 1),
// clamped to the memory reserved for the upper bound.  The device evaluates it
// from the selected-row count it reads from memory, so no host sync is needed.
#pragma once

#include <cmath>

#include "pyst_internal.h"

namespace pyst {

struct TableDev {
  void *slots;     // int32 keys (slot_bytes 4) or uint64 key|payload<<32 (slot_bytes 8)
  int64_t *hdr;    // [0] effective capacity, [1] rows offered for insertion
  uint64_t *sums;  // optional per-slot SUM (group by the join key), else null
  uint8_t *flags;  // optional per-slot "group exists" flags
  uint32_t *bloom; // optional blocked Bloom filter over the inserted keys (fast path)
  int64_t cap_alloc;
  int32_t slot_bytes;
  int32_t selected;  // built from a selection: only the device knows how many slots it uses
};

struct GroupDev {
  uint64_t *slots;  // 2 words per slot
  int64_t *hdr;     // [0] effective capacity
  int64_t cap_alloc;
};

// How the rows of a group-by are grouped: chosen on the device from the keys'
// range (see the planned group-by).  Kernels of the other modes return at once.
enum : int32_t { kGbHash = 0, kGbSmall = 1, kGbRange = 2, kGbTable = 3, kGbFew = 4, kGbOnce = 5 };
struct GbPlan {
  int64_t kmin;
  uint64_t range;      // greatest - least key + 1; 0 without rows
  int64_t count;       // rows to group
  int64_t sort_count;  // groups that still need sorting (0 where they come out in key order)
  int32_t mode;
  int32_t shift;       // kGbRange: bucket = (key - kmin) >> shift
  int32_t few_failed;  // kGbFew: its table had no slot for a group, the mode is `otherwise`
  int32_t otherwise;
  unsigned long long ticket;
};

// How a materializing join of large sides looks its build rows up: chosen on the
// device from the build keys' range (see join.hip).
struct JoinPlan {
  int64_t kmin;
  uint64_t range;             // greatest - least build key + 1
  int32_t direct;             // array indexed by key - kmin, else the hash table
  int32_t shift;              // slice = (key - kmin) >> shift
  int64_t moved[2];           // rows in their slices: build, probe
  unsigned long long filled;  // entries of the array
  unsigned long long ticket;
};
bool direct_join_wanted(const pyst_col *build_key, const pyst_col *probe_key, int unique);
size_t direct_join_bytes(int64_t nb, int64_t np);
pyst_status direct_join_build(pyst_ctx *ctx, const pyst_col *build_key, int64_t np, void *ws, int32_t *array,
                              int64_t range_max, const JoinPlan **plan, hipStream_t stream);
pyst_status direct_join_probe(pyst_ctx *ctx, int64_t nb, const pyst_col *probe_key, void *ws, int32_t *array,
                              int32_t *out_row, int32_t *out_build, int64_t out_cap, int64_t *d_nout, hipStream_t stream);

// How a table that was built from a selection is probed, chosen on the device:
// by slices where it is as large as the host asks of other tables, or half of
// that if the probed column is long (8 MiB of slots, 20M probes 317 us by slices,
// 330 in one pass; 2.5M 73 and 62), or where only a small part of a long column is
// probed (the one-pass probe takes a ticket for every tile of the column, 14 ns
// each: 1000 of 20M rows 140 us, by slices 29); else in one pass (five built rows,
// all of 20M probed: 290 us by slices, 98 in one pass; of 2.5M 72 and 24).  The
// launches that find nothing to do cost 3 to 12 us; a one-pass kernel of few
// blocks that walk its tiles would spare 7 of them, and ran 20 % longer.
struct ProbeRule {
  const int64_t *hdr = nullptr;  // of the table; null: the host has chosen
  const int64_t *d_nsel = nullptr;
  int64_t n = 0, slots_min = 0;
  static constexpr int64_t kLongColumn = int64_t{1} << 22;
  __device__ __forceinline__ bool by_slices() const {
    if (n < kLongColumn) return hdr[0] >= slots_min;
    const int64_t rows = d_nsel ? *d_nsel : n;
    return hdr[0] >= slots_min / 2 || rows < n / 4;
  }
  __device__ __forceinline__ bool not_by_slices() const { return hdr && !by_slices(); }
  __device__ __forceinline__ bool not_in_one_pass() const { return hdr && by_slices(); }
};

__device__ __forceinline__ int32_t plan_mode(const GbPlan *p) {
  return p->mode == kGbFew && p->few_failed ? p->otherwise : p->mode;
}

__host__ __device__ inline int64_t next_pow2(int64_t x) {
  int64_t p = 1;
  while (p < x) p <<= 1;
  return p;
}

__host__ __device__ inline int64_t table_capacity(int64_t cnt, double max_load, int64_t cap_alloc) {
  int64_t need = static_cast<int64_t>(static_cast<double>(cnt) / max_load) + 1;
  if (need < cnt + 1) need = cnt + 1;
  if (need < 64) need = 64;
  int64_t cap = next_pow2(need);
  return cap > cap_alloc ? cap_alloc : cap;
}

inline int64_t table_capacity_host(int64_t n, double max_load) { return table_capacity(n, max_load, INT64_MAX); }

// Header of every table: int64 words (capacity, count, mode, ...) in the
// first 256 bytes; bytes [512, 1024) are one byte per bucket of slot sums.
constexpr size_t kHdrBytes = 1024;

inline size_t table_bytes(int64_t cap, int slot_bytes, bool with_sums) {
  size_t b = kHdrBytes + static_cast<size_t>(cap) * slot_bytes;
  if (with_sums) b += static_cast<size_t>(cap) * (sizeof(uint64_t) + 1);
  return b;
}

inline TableDev table_view(void *mem, int64_t cap, int slot_bytes, bool with_sums) {
  TableDev t{};
  char *p = static_cast<char *>(mem);
  t.hdr = reinterpret_cast<int64_t *>(p);
  t.slots = p + kHdrBytes;
  t.cap_alloc = cap;
  t.slot_bytes = slot_bytes;
  if (with_sums) {
    t.sums = reinterpret_cast<uint64_t *>(p + kHdrBytes + static_cast<size_t>(cap) * slot_bytes);
    t.flags = reinterpret_cast<uint8_t *>(t.sums + cap);
  }
  return t;
}

inline size_t group_bytes(int64_t cap) { return kHdrBytes + static_cast<size_t>(cap) * 16; }

inline GroupDev group_view(void *mem, int64_t cap) {
  GroupDev g{};
  g.hdr = static_cast<int64_t *>(mem);
  g.slots = reinterpret_cast<uint64_t *>(static_cast<char *>(mem) + kHdrBytes);
  g.cap_alloc = cap;
  return g;
}

// Add v to the group of key k (inserting the key if absent).  False: table full,
// or no place within the first `probes` slots.
__device__ __forceinline__ bool group_add(uint64_t *slots, int64_t mask, int64_t k, uint64_t v, int64_t probes) {
  int64_t s = static_cast<int64_t>(table_hash64(k)) & mask;
  for (int64_t step = 0; step < probes; ++step) {
    uint64_t cur = slots[2 * s];
    if (static_cast<int64_t>(cur) == kEmpty64) {
      const uint64_t old = atomicCAS(reinterpret_cast<unsigned long long *>(&slots[2 * s]),
                                     static_cast<unsigned long long>(kEmpty64), static_cast<unsigned long long>(k));
      cur = old == static_cast<uint64_t>(kEmpty64) ? static_cast<uint64_t>(k) : old;
    }
    if (static_cast<int64_t>(cur) == k) {
      atomicAdd(reinterpret_cast<unsigned long long *>(&slots[2 * s + 1]), static_cast<unsigned long long>(v));
      return true;
    }
    s = (s + 1) & mask;
  }
  return false;
}
__device__ __forceinline__ bool group_add(uint64_t *slots, int64_t mask, int64_t k, uint64_t v) {
  return group_add(slots, mask, k, v, mask + 1);
}

// Host helpers implemented in ops.hip / sort.hip.
pyst_status table_init(const TableDev &t, const int64_t *d_nsel, int64_t n, double max_load, hipStream_t stream,
                       const JoinPlan *plan = nullptr);
pyst_status group_init(const GroupDev &g, const int64_t *d_nsel, int64_t n, int64_t max_groups, double max_load,
                       hipStream_t stream);
pyst_status group_insert(pyst_ctx *ctx, const GroupDev &g, const pyst_col *key, const pyst_col *val, const int32_t *sel,
                         const int64_t *d_nsel, int skip_empty, GbPlan *plan, int mode, hipStream_t stream);
pyst_status group_compact(pyst_ctx *ctx, const GroupDev &g, int64_t *out_keys, int64_t *out_sums, int64_t out_cap,
                          int64_t *d_ngroups, hipStream_t stream);
// Group-by of columns through the table `g` in HBM (with a plan: only in `mode`).
// status: group_compact_words of memory (null: taken from the arena).
int64_t group_compact_words(int64_t cap_alloc);
pyst_status table_groupby(pyst_ctx *ctx, const GroupDev &g, const pyst_col *key, const pyst_col *val,
                          const int32_t *sel, const int64_t *d_nsel, int64_t max_groups, double max_load,
                          int64_t *out_keys, int64_t *out_sums, int64_t out_cap, int64_t *d_ngroups, GbPlan *plan,
                          int mode, uint64_t *status, hipStream_t stream);
pyst_status filter_impl(pyst_ctx *ctx, const PredSet &ps, int64_t n, int32_t *sel_out, int64_t *d_nsel,
                        hipStream_t stream);
pyst_status sort_pairs_by_key(pyst_ctx *ctx, int64_t *keys, int64_t *vals, const int64_t *d_count, int64_t cap,
                              int key_bits, hipStream_t stream);
int grid_for(pyst_ctx *ctx, int64_t work, int block, int per_cu);

}  // namespace pyst
