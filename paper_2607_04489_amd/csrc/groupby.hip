// groupby.hip -- group-by with a count and per-column sums, hash-based or
// partition-based, chosen from the HLL distinct-count estimate of the key
// column (Section 3.3: group-by algorithms; Section 4.1: the number of groups,
// estimated with HLL++ before the operator runs, picks the algorithm and sizes
// the hash table; Section 5.3.2: the "Auto" series).
//
//  HASH       one open-addressing table of groups in HBM, sized from the
//             estimate. Every workgroup first aggregates its rows in an LDS
//             table (so a group costs one global update per workgroup, not one
//             per row); rows whose group does not fit in LDS go to the
//             global table; at the end each workgroup merges its LDS groups
//             into the global table, which is then compacted into the output.
//  PARTITION  rows partitioned on the top bits of the key hash (values
//             carried along), then one workgroup per partition aggregates it in
//             LDS and writes its groups straight out (partitions own disjoint
//             keys). A partition with more groups than its LDS table spills
//             into the global table, and its LDS groups are merged there too.
// Group keys live in the tables as sign-extended 64-bit words; a value that is
// not a key (the plan's sentinel) marks empty slots, so a key is claimed with
// one 64-bit CAS.
#include <algorithm>
#include <cmath>
#include <string>
#include <type_traits>

#include "sort.hpp"
#include "variants.hpp"

namespace eiger {

namespace {

constexpr int kGNT = 256;                   // clear and emit workgroups
constexpr int kANT = 512;                   // aggregating workgroup
constexpr uint32_t kGLds = 2048;            // LDS table slots (power of two)
constexpr uint32_t kGLdsOpen = kGLds / 2;   // new groups an LDS table accepts
constexpr int kGMaxVals = 2;
constexpr int kARows = 4;                   // rows a thread loads before aggregating them
constexpr uint32_t kAStep = kANT * kARows;  // rows of a step
constexpr uint32_t kAFold = 31 * kAStep;    // rows between folds: a packed count stays below 2^16
static_assert(kAFold < 65536, "packed counts hold 16 bits");
constexpr int kAOwn = kGLds / kANT;         // slots a thread folds
constexpr uint64_t kGMaxProbe = 4096;       // longest walk in the global table
// rule: HASH while the estimated groups fit one LDS table (beyond it, rows that
// miss the LDS table cost global atomics per row, and PARTITION measured faster
// from 2^14 groups up at 2^28 rows)
constexpr double kGbHashMaxGroups = kGLdsOpen;
constexpr double kGbGroupsPerPartition = 512.0;

struct GbGlobal {
  unsigned long long *key;
  unsigned long long *cnt;
  unsigned long long *sum[kGMaxVals];
  uint64_t mask;
  unsigned long long sentinel;
  uint32_t *overflow;
};

// Value columns: 4-byte values at lo; 8-byte ones at lo, or (after partitioning)
// their low words at lo and high words at hi.
struct GbVals {
  const uint32_t *lo[kGMaxVals];
  const uint32_t *hi[kGMaxVals];
};

// Slot of key k in the global table, claiming an empty one if needed; -1 when
// the whole table was walked (more groups than slots: *overflow is set).
__device__ __forceinline__ int64_t global_slot(const GbGlobal &t, unsigned long long k) {
  uint64_t s = fmix64(k) & t.mask;
  // a table at most half full never needs a walk this long; stopping here keeps
  // an overfull table (a far too low estimate) from costing a whole-table walk
  // per row before the caller plans again with more slots
  const uint64_t limit = t.mask < kGMaxProbe ? t.mask + 1 : kGMaxProbe;
  for (uint64_t step = 0; step < limit; ++step) {
    // a slot changes once, from the sentinel to a key: any other value read is final
    const unsigned long long cur = __atomic_load_n(&t.key[s], __ATOMIC_RELAXED);
    if (cur == k) return static_cast<int64_t>(s);
    if (cur == t.sentinel) {
      const unsigned long long old = atomicCAS(&t.key[s], t.sentinel, k);
      if (old == t.sentinel || old == k) return static_cast<int64_t>(s);
    }
    s = (s + 1) & t.mask;
  }
  atomicOr(t.overflow, 1u);
  return -1;
}

__device__ __forceinline__ void global_add(const GbGlobal &t, unsigned long long k, unsigned long long c,
                                           const unsigned long long *sums, int nv) {
  const int64_t s = global_slot(t, k);
  if (s < 0) return;
  atomicAdd(&t.cnt[s], c);
  for (int v = 0; v < nv; ++v) atomicAdd(&t.sum[v][s], sums[v]);
}

// ---- aggregation in LDS ----------------------------------------------------------
//
// NV value columns, W0 / W1: 8-byte values; kSplit: 8-byte values as two word arrays.
// A workgroup's table: keys in `slots` slots (sign-extended, the plan's sentinel
// marks empty ones), and for each slot `reps` sets of accumulators, a lane using
// the one of its number, so that few groups do not pile a wave's atomics onto few
// LDS words. A 4-byte first column shares its accumulator with the row count:
// count << 48 plus the value made unsigned by adding 2^31, one atomic for both.
// Every kAFold rows the accumulators are folded into registers of the thread that
// owns the slot, so they never run over and reach the global table once per
// workgroup. Four rows a thread and at most 80 registers, so that three workgroups
// of 512 share a CU where their LDS lets them (agg_per_cu): with eight rows and two
// workgroups, 1,000 groups took 1.27 ms instead of 0.91.
template <int NV, bool W0>
constexpr bool kPacked = NV > 0 && !W0;

template <int NV, bool W0>
struct AggLds {
  unsigned long long key[kGLds];
  unsigned long long a[NV > 0 ? kGLds : 1];  // column 0 (with the count when packed)
  unsigned long long b[NV > 1 ? kGLds : 1];  // column 1
  uint32_t c[kPacked<NV, W0> ? 1 : kGLds];   // row counts
  uint32_t used;
  uint32_t spilled;
  unsigned long long scan[kANT / 64];
  unsigned long long at;
};

// Workgroups of a CU: three, or the two whose tables fit its 160 KB of LDS (56 KB each
// where the first of two columns has 8 bytes). The grids are sized by it: with three
// ranges of rows per CU for the two, 2^26 rows of 1,000 groups and two 8-byte sums
// took 517 us, now 424.
template <int NV, bool W0>
constexpr int agg_per_cu = sizeof(AggLds<NV, W0>) * 3 <= 163840 ? 3 : 2;
static_assert(sizeof(AggLds<2, true>) * agg_per_cu<2, true> <= 163840, "the largest table");

// A thread's slots threadIdx.x + j * kANT.
template <int NV>
struct AggOwn {
  uint32_t cnt[kAOwn];  // (a column has fewer than 2^32 rows)
  unsigned long long s[NV > 0 ? NV : 1][kAOwn];
};

struct AggShape {
  uint32_t slots, reps, shift;  // slots * reps = kGLds; shift = 32 - log2(slots)
};

// The whole table, one accumulator a slot.
__host__ __device__ __forceinline__ AggShape agg_whole() { return AggShape{kGLds, 1, 21}; }
static_assert(kGLds == 1u << 11, "agg_whole's shift");

// slots: four per expected group
AggShape agg_shape(double groups) {
  AggShape h{64, 0, 26};
  while (h.slots < kGLds && h.slots < 4 * groups) h.slots <<= 1, --h.shift;
  h.reps = std::min(kGLds / h.slots, 32u);
  return h;
}

__device__ __forceinline__ uint32_t agg_hash(unsigned long long k, uint32_t shift) {
  uint32_t x = static_cast<uint32_t>(k) ^ static_cast<uint32_t>(k >> 32) * 0x85ebca6bu;
  x ^= x >> 16;
  return (x * 0x9e3779b1u) >> shift;
}

template <int NV, bool W0>
__device__ __forceinline__ void agg_clear(AggLds<NV, W0> &L, AggOwn<NV> &own, unsigned long long sentinel) {
  for (uint32_t i = threadIdx.x; i < kGLds; i += kANT) {
    L.key[i] = sentinel;
    if constexpr (NV > 0) L.a[i] = 0;
    if constexpr (NV > 1) L.b[i] = 0;
    if constexpr (!kPacked<NV, W0>) L.c[i] = 0;
  }
#pragma unroll
  for (int j = 0; j < kAOwn; ++j) {
    own.cnt[j] = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) own.s[v][j] = 0;
  }
  if (threadIdx.x == 0) {
    L.used = 0;
    L.spilled = 0;
  }
  __syncthreads();
}

// LDS slot of key k, from slot s on, claiming an empty slot while the table takes
// new groups; kAMiss: not in the table and the table is closed.
constexpr uint32_t kAMiss = 0xFFFFFFFFu, kASkip = 0xFFFFFFFEu;
template <int NV, bool W0>
__device__ __forceinline__ uint32_t agg_slot(AggLds<NV, W0> &L, uint32_t slots, uint32_t s, unsigned long long k,
                                        unsigned long long sentinel) {
  for (uint32_t step = 0; step < slots; ++step) {
    const unsigned long long cur = __atomic_load_n(&L.key[s], __ATOMIC_RELAXED);
    if (cur == k) return s;
    if (cur == sentinel) {
      // closed for new groups once half the slots were claimed; claims racing with the
      // last one can add at most one per thread of the workgroup
      if (__atomic_load_n(&L.used, __ATOMIC_RELAXED) >= slots / 2) return kAMiss;
      const unsigned long long old = atomicCAS(&L.key[s], sentinel, k);
      if (old == sentinel) {
        atomicAdd(&L.used, 1u);
        return s;
      }
      if (old == k) return s;
    }
    s = (s + 1) & (slots - 1);
  }
  return kAMiss;
}

typedef uint32_t V4u __attribute__((ext_vector_type(4)));
typedef V4u V4uWord __attribute__((aligned(4)));  // columns may start at any row

// Four consecutive 4-byte values, or 8-byte ones (one array, or two word arrays).
__device__ __forceinline__ void load4(const uint32_t *p, uint64_t i, uint32_t (&out)[4]) {
  const V4u v = *reinterpret_cast<const V4uWord *>(p + i);
#pragma unroll
  for (int u = 0; u < 4; ++u) out[u] = v[u];
}
template <bool kSplit>
__device__ __forceinline__ void load4(const uint32_t *lo, const uint32_t *hi, uint64_t i, unsigned long long (&out)[4]) {
  const V4u x = *reinterpret_cast<const V4uWord *>(kSplit ? lo + i : lo + 2 * i);
  const V4u y = *reinterpret_cast<const V4uWord *>(kSplit ? hi + i : lo + 2 * i + 4);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if constexpr (kSplit)
      out[u] = (static_cast<unsigned long long>(y[u]) << 32) | x[u];
    else
      out[u] = u < 2 ? (static_cast<unsigned long long>(x[2 * u + 1]) << 32) | x[2 * u]
                     : (static_cast<unsigned long long>(y[2 * u - 3]) << 32) | y[2 * u - 4];
  }
}

// One column of a thread's rows: 4-byte values as words, 8-byte values whole.
template <bool kWide, bool kSplit>
struct AggCol {
  using T = typename std::conditional<kWide, unsigned long long, uint32_t>::type;
  T v[kARows];
  __device__ __forceinline__ void load_full(const uint32_t *lo, const uint32_t *hi, uint64_t base) {
#pragma unroll
    for (int q = 0; q < kARows; q += 4) {
      const uint64_t i = base + (q / 4 * kANT + threadIdx.x) * 4;
      T(&out)[4] = reinterpret_cast<T(&)[4]>(v[q]);
      if constexpr (kWide)
        load4<kSplit>(lo, hi, i, out);
      else
        load4(lo, i, out);
    }
  }
  __device__ __forceinline__ void load_some(const uint32_t *lo, const uint32_t *hi, uint64_t base, uint64_t end) {
#pragma unroll
    for (int q = 0; q < kARows; ++q) {
      const uint64_t i = min(base + (q / 4 * kANT + threadIdx.x) * 4 + q % 4, end - 1);
      if constexpr (!kWide)
        v[q] = lo[i];
      else if constexpr (kSplit)
        v[q] = (static_cast<unsigned long long>(hi[i]) << 32) | lo[i];
      else
        v[q] = (static_cast<unsigned long long>(lo[2 * i + 1]) << 32) | lo[2 * i];
    }
  }
  __device__ __forceinline__ unsigned long long sext64(int q) const {
    if constexpr (kWide)
      return v[q];
    else
      return static_cast<unsigned long long>(static_cast<long long>(static_cast<int32_t>(v[q])));
  }
  // All rows' sum (4-byte values made unsigned first: no high words to hold).
  __device__ __forceinline__ unsigned long long sum() const {
    unsigned long long s = 0;
#pragma unroll
    for (int q = 0; q < kARows; ++q) {
      if constexpr (kWide)
        s += v[q];
      else
        s += v[q] ^ 0x80000000u;
    }
    return kWide ? s : s - (static_cast<unsigned long long>(kARows) << 31);
  }
};

// Sum over the wave, in lane 63, by data-parallel moves: within rows of 16 lanes, then
// from row to row. (Shuffles keep an address a step in registers, here across the
// whole loop.)
template <int kCtrl, int kRowMask>
__device__ __forceinline__ unsigned long long add_moved(unsigned long long v) {
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(v), kCtrl, kRowMask, 0xF, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(v >> 32), kCtrl, kRowMask, 0xF, false);
  return v + ((static_cast<unsigned long long>(hi) << 32) | lo);
}
__device__ __forceinline__ unsigned long long wave_sum_last(unsigned long long v) {
  v = add_moved<0x111, 0xF>(v);  // from 1, 2, 4, 8 lanes below in the row
  v = add_moved<0x112, 0xF>(v);
  v = add_moved<0x114, 0xF>(v);
  v = add_moved<0x118, 0xF>(v);
  v = add_moved<0x142, 0xA>(v);  // a row's last lane to the next row, rows 1 and 3
  return add_moved<0x143, 0xC>(v);  // lane 31 to rows 2 and 3
}

// Adds a step of a wave whose lanes each hold kARows rows of one group in LDS slot s
// (sorted or clustered keys): a lane's rows are summed before they reach the table, and
// the whole wave's if they are of one group, for one atomic instead of 64 * kARows on
// one LDS word (2^26 sorted rows of 1,000 groups: two 4-byte sums 0.24 ms, 0.52 without;
// two 8-byte ones 0.34, 0.74; counts alone 0.12, 0.28).
template <int NV, bool W0, class C0, class C1>
__device__ __forceinline__ void agg_runs(AggLds<NV, W0> &L, const AggShape &h, uint32_t s, const C0 &c0, const C1 &c1) {
  unsigned long long x = 0, y = 0;
  if constexpr (NV > 0) x = c0.sum();
  if constexpr (NV > 1) y = c1.sum();
  uint32_t c = kARows, rep = __lane_id();
  if (__all(s == __builtin_amdgcn_readfirstlane(s))) {
    if constexpr (NV > 0) x = wave_sum_last(x);
    if constexpr (NV > 1) y = wave_sum_last(y);
    if (__lane_id() != 63) return;
    c = 64 * kARows;
    rep = threadIdx.x / 64;
  }
  const uint32_t i = s * h.reps + (rep & (h.reps - 1));
  if constexpr (kPacked<NV, W0>) {  // each value made unsigned by 2^31
    atomicAdd(&L.a[i], (static_cast<unsigned long long>(c) << 48) + x + (static_cast<unsigned long long>(c) << 31));
  } else {
    atomicAdd(&L.c[i], c);
    if constexpr (NV > 0) atomicAdd(&L.a[i], x);
  }
  if constexpr (NV > 1) atomicAdd(&L.b[i], y);
}

// Aggregate this wave's rows of the steps of [lo, hi) (at most kAFold rows) into the
// LDS table; rows that do not fit go global. kGrow: while a larger table can be
// taken, a wave stops instead, before the step in which a row of its does not fit (the
// keys that the step entered stay, with no row yet). kRuns: clustered rows are looked
// for. Returns where the wave stopped.
template <typename K, int NV, bool W0, bool W1, bool kSplit, bool kGrow, bool kRuns>
__device__ __forceinline__ uint64_t agg_rows(AggLds<NV, W0> &L, const AggShape &h, const GbGlobal &g,
                                             const K *__restrict__ keys, const GbVals &vals, uint64_t lo, uint64_t hi) {
  const uint32_t rep = __lane_id() & (h.reps - 1);
  const uint32_t *kw = reinterpret_cast<const uint32_t *>(keys);
  for (uint64_t base = lo; base < hi; base += kAStep) {
    AggCol<sizeof(K) == 8, false> kc;
    AggCol<W0, kSplit> c0;
    AggCol<W1, kSplit> c1;
    const bool full = base + kAStep <= hi;
    if (full) {
      kc.load_full(kw, nullptr, base);
      if constexpr (NV > 0) c0.load_full(vals.lo[0], vals.hi[0], base);
      if constexpr (NV > 1) c1.load_full(vals.lo[1], vals.hi[1], base);
    } else {
      kc.load_some(kw, nullptr, base, hi);
      if constexpr (NV > 0) c0.load_some(vals.lo[0], vals.hi[0], base, hi);
      if constexpr (NV > 1) c1.load_some(vals.lo[1], vals.hi[1], base, hi);
    }
    // all rows' walks take their steps together, so that their LDS reads overlap;
    // a walk ends at its key or an empty slot (or after the whole table)
    unsigned long long k[kARows], at[kARows];
    uint32_t slot[kARows];
#pragma unroll
    for (int q = 0; q < kARows; ++q) {
      k[q] = full || base + (q / 4 * kANT + threadIdx.x) * 4 + q % 4 < hi ? kc.sext64(q) : g.sentinel;
      slot[q] = agg_hash(k[q], h.shift);
      at[q] = __atomic_load_n(&L.key[slot[q]], __ATOMIC_RELAXED);
    }
    for (uint32_t step = 1; step < h.slots; ++step) {
      bool any = false;
#pragma unroll
      for (int q = 0; q < kARows; ++q) {
        const bool on = at[q] != k[q] && at[q] != g.sentinel;
        slot[q] = on ? (slot[q] + 1) & (h.slots - 1) : slot[q];
        any |= on;
      }
      if (!any) break;
      // (unconditional: a read under a condition is waited for on the spot)
#pragma unroll
      for (int q = 0; q < kARows; ++q) at[q] = __atomic_load_n(&L.key[slot[q]], __ATOMIC_RELAXED);
    }
    // rows past the end, and keys new to the workgroup
    bool odd = false;
#pragma unroll
    for (int q = 0; q < kARows; ++q) odd |= at[q] != k[q] || k[q] == g.sentinel;
    if (__any(odd)) {
      bool miss = false;
#pragma unroll
      for (int q = 0; q < kARows; ++q) {
        if (k[q] == g.sentinel)  // (no key equals the sentinel)
          slot[q] = kASkip;
        else if (at[q] != k[q])
          slot[q] = agg_slot<NV, W0>(L, h.slots, slot[q], k[q], g.sentinel);
        miss |= slot[q] == kAMiss;
      }
      if (kGrow && h.slots < kGLds && __any(miss)) return base;
    } else if constexpr (kRuns) {
      bool one = true;
#pragma unroll
      for (int q = 1; q < kARows; ++q) one = one && slot[q] == slot[0];
      if (__all(one)) {
        agg_runs<NV, W0>(L, h, slot[0], c0, c1);
        continue;
      }
    }
#pragma unroll
    for (int q = 0; q < kARows; ++q) {
      if (slot[q] < kGLds) {
        const uint32_t i = slot[q] * h.reps + rep;
        if constexpr (kPacked<NV, W0>)
          atomicAdd(&L.a[i], (1ull << 48) | (static_cast<uint32_t>(c0.v[q]) ^ 0x80000000u));
        else
          atomicAdd(&L.c[i], 1u);
        if constexpr (NV > 0 && W0) atomicAdd(&L.a[i], c0.sext64(q));
        if constexpr (NV > 1) atomicAdd(&L.b[i], c1.sext64(q));
      } else if (slot[q] == kAMiss) {
        L.spilled = 1;
        unsigned long long sv[kGMaxVals] = {0, 0};
        if constexpr (NV > 0) sv[0] = c0.sext64(q);
        if constexpr (NV > 1) sv[1] = c1.sext64(q);
        global_add(g, k[q], 1ull, sv, NV);
      }
    }
  }
  return hi;
}

// Accumulators into the owners' registers, cleared for the rows to come. Barriers.
// Returns whether the table takes no new groups although a larger one would (the same
// for all waves: none takes a row between the barriers).
template <int NV, bool W0>
__device__ __forceinline__ bool agg_fold(AggLds<NV, W0> &L, const AggShape &h, AggOwn<NV> &own) {
  __syncthreads();
  const bool closed = h.slots < kGLds && L.used >= h.slots / 2;
#pragma unroll
  for (int j = 0; j < kAOwn; ++j) {
    const uint32_t s = threadIdx.x + j * kANT;
    if (s >= h.slots) continue;
    for (uint32_t r = 0; r < h.reps; ++r) {
      const uint32_t i = s * h.reps + r;
      if constexpr (kPacked<NV, W0>) {
        const unsigned long long p = L.a[i], c = p >> 48;
        own.cnt[j] += static_cast<uint32_t>(c);
        own.s[0][j] += (p & 0xFFFFFFFFFFFFull) - (c << 31);
        L.a[i] = 0;
      } else {
        own.cnt[j] += L.c[i];
        L.c[i] = 0;
        if constexpr (NV > 0) {
          own.s[0][j] += L.a[i];
          L.a[i] = 0;
        }
      }
      if constexpr (NV > 1) {
        own.s[1][j] += L.b[i];
        L.b[i] = 0;
      }
    }
  }
  __syncthreads();
  return closed;
}

// The folded groups into the global table.
template <int NV, bool W0>
__device__ __forceinline__ void agg_merge(AggLds<NV, W0> &L, const AggShape &h, const AggOwn<NV> &own, const GbGlobal &g) {
#pragma unroll
  for (int j = 0; j < kAOwn; ++j) {
    const uint32_t s = threadIdx.x + j * kANT;
    if (s >= h.slots || L.key[s] == g.sentinel || own.cnt[j] == 0) continue;
    unsigned long long sv[kGMaxVals] = {0, 0};
    for (int v = 0; v < NV; ++v) sv[v] = own.s[v][j];
    global_add(g, L.key[s], own.cnt[j], sv, NV);
  }
}

struct GbOut {
  void *keys;  // key dtype
  unsigned long long *cnt;
  unsigned long long *sum[kGMaxVals];
  uint64_t cap;
  unsigned long long *cursor;
  int kwide;
};

__device__ __forceinline__ void put_group(const GbOut &o, uint64_t pos, unsigned long long k, unsigned long long c,
                                          const unsigned long long *sv, int nv) {
  if (pos >= o.cap || !o.keys) return;
  if (o.kwide)
    static_cast<unsigned long long *>(o.keys)[pos] = k;
  else
    static_cast<uint32_t *>(o.keys)[pos] = static_cast<uint32_t>(k);
  o.cnt[pos] = c;
  for (int v = 0; v < nv; ++v) o.sum[v][pos] = sv[v];
}

// Emit the occupied slots of one table range [lo, hi) of (key, cnt, sums)
// arrays. The whole workgroup walks the range in rounds of kGEmitPer slots per
// thread (each thread a contiguous run), and each round reserves its output
// with ONE atomic: a device-wide counter that every wave hit separately cost
// more than the rest of a group-by with millions of groups. Uniform across
// the workgroup (contains barriers); `scan` holds kGNT / 64 + 1 words of LDS.
constexpr int kGEmitPer = 8;
__device__ __forceinline__ void emit_range(const unsigned long long *key, const unsigned long long *cnt,
                                           const unsigned long long *sum0, const unsigned long long *sum1,
                                           uint64_t lo, uint64_t hi, unsigned long long sentinel, int nv,
                                           const GbOut &o, unsigned long long *scan) {
  constexpr uint64_t round = uint64_t(kGNT) * kGEmitPer;
  for (uint64_t base = lo; base < hi; base += round) {
    const uint64_t mine = base + uint64_t(threadIdx.x) * kGEmitPer;
    uint32_t live = 0;
#pragma unroll
    for (int j = 0; j < kGEmitPer; ++j) {
      const uint64_t i = mine + j;
      if (i < hi && key[i] != sentinel) live |= 1u << j;
    }
    unsigned long long total;
    const unsigned long long off =
        block_exclusive_scan<kGNT, unsigned long long>(static_cast<unsigned long long>(__popc(live)), scan, &total);
    if (total == 0) continue;
    if (threadIdx.x == 0) scan[kGNT / 64] = atomicAdd(o.cursor, total);
    __syncthreads();
    unsigned long long at = scan[kGNT / 64] + off;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kGEmitPer; ++j) {
      if (!((live >> j) & 1u)) continue;
      const uint64_t i = mine + j;
      unsigned long long sv[kGMaxVals] = {0, 0};
      if (nv > 0) sv[0] = sum0[i];
      if (nv > 1) sv[1] = sum1[i];
      put_group(o, at++, key[i], cnt[i], sv, nv);
    }
  }
}

// The global table, the output cursor and the overflow flag.
__global__ void __launch_bounds__(kGNT) k_gb_clear(GbGlobal g, int nv, unsigned long long *cursor) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *cursor = 0;
    *g.overflow = 0;
  }
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i <= g.mask; i += stride) {
    g.key[i] = g.sentinel;
    g.cnt[i] = 0;
    for (int v = 0; v < nv; ++v) g.sum[v][i] = 0;
  }
}

// HASH: a contiguous range of rows per workgroup, LDS aggregation, one merge. `h` is
// the table's shape from the plan's estimate; a workgroup that meets more groups than
// that takes merges what it has and goes on with the whole table, so that a low
// estimate costs one more merge and not a global atomic per row (2^26 rows, two 4-byte
// sums, 1,000 groups planned as one: 0.43 ms, 12.5 while every row that did not fit went
// global; planned as 1,000: 0.39).
// 2^28 rows, two 4-byte sums, 100 groups: 0.57 ms (5.6 TB/s; 1.47 with register
// groups and three 64-bit LDS atomics a row); 1,000 groups: 0.90 ms (2.94), the
// walks in the half-full table.
template <typename K, int NV, bool W0, bool W1, bool kRuns>
__global__ void __launch_bounds__(kANT, (2 * agg_per_cu<NV, W0>)) k_gb_hash(const K *__restrict__ keys, uint64_t n, GbVals vals, AggShape h,
                                                  uint64_t per, GbGlobal g) {
  __shared__ AggLds<NV, W0> L;
  AggOwn<NV> own;
  const uint64_t lo = uint64_t(blockIdx.x) * per, hi = min(n, lo + per);
  agg_clear<NV, W0>(L, own, g.sentinel);
  uint64_t at = lo, end = min(hi, lo + kAFold);  // this wave's next step; the next fold (for all waves)
  for (;;) {
    at = agg_rows<K, NV, W0, W1, false, true, kRuns>(L, h, g, keys, vals, at, end);
    if (agg_fold<NV, W0>(L, h, own)) {
      agg_merge<NV, W0>(L, h, own, g);
      __syncthreads();
      h = agg_whole();
      agg_clear<NV, W0>(L, own, g.sentinel);
      continue;
    }
    if (end >= hi) break;
    at = end;
    end = min(hi, end + kAFold);
  }
  agg_merge<NV, W0>(L, h, own, g);
}

// PARTITION: work item = one of the S equal slices of a partition (S = 1 when
// partitions are small). A whole partition that did not spill writes its groups
// out directly; slices and spilled partitions merge into the global table.
// 2^28 rows, two 4-byte sums, 2^20 groups in 2^11 partitions: 0.72 ms (4.5 TB/s;
// 1.78 with one row's walk at a time).
template <typename K, int NV, bool W0, bool W1>
__global__ void __launch_bounds__(kANT, (2 * agg_per_cu<NV, W0>))
    k_gb_partition(const K *__restrict__ keys, GbVals vals, const uint32_t *__restrict__ off, uint32_t F, uint32_t S,
                   AggShape h, GbGlobal g, GbOut o) {
  __shared__ AggLds<NV, W0> L;
  AggOwn<NV> own;
  const uint64_t items = uint64_t(F) * S;
  for (uint64_t it = blockIdx.x; it < items; it += gridDim.x) {
    const uint32_t p = static_cast<uint32_t>(it / S), sl = static_cast<uint32_t>(it % S);
    const uint64_t plo = off[p], len = off[p + 1] - plo;
    const uint64_t lo = plo + len * sl / S, hi = plo + len * (sl + 1) / S;
    if (lo == hi) continue;
    agg_clear<NV, W0>(L, own, g.sentinel);
    for (uint64_t c = lo; c < hi; c += kAFold) {
      agg_rows<K, NV, W0, W1, true, false, false>(L, h, g, keys, vals, c, min(hi, c + kAFold));
      agg_fold<NV, W0>(L, h, own);
    }
    if (L.spilled || S > 1) {
      agg_merge<NV, W0>(L, h, own, g);
    } else {
      unsigned long long live = 0, total;
#pragma unroll
      for (int j = 0; j < kAOwn; ++j) live += threadIdx.x + j * kANT < h.slots && L.key[threadIdx.x + j * kANT] != g.sentinel;
      unsigned long long at = block_exclusive_scan<kANT, unsigned long long>(live, L.scan, &total);
      if (threadIdx.x == 0) L.at = atomicAdd(o.cursor, total);
      __syncthreads();
      at += L.at;
#pragma unroll
      for (int j = 0; j < kAOwn; ++j) {
        const uint32_t s = threadIdx.x + j * kANT;
        if (s >= h.slots || L.key[s] == g.sentinel) continue;
        unsigned long long sv[kGMaxVals] = {0, 0};
        for (int v = 0; v < NV; ++v) sv[v] = own.s[v][j];
        put_group(o, at++, L.key[s], own.cnt[j], sv, NV);
      }
    }
    __syncthreads();
  }
}

// Compaction of the global table into the output.
__global__ void __launch_bounds__(kGNT) k_gb_emit(GbGlobal g, int nv, GbOut o) {
  const uint64_t slots = g.mask + 1;
  const uint64_t per = (slots + gridDim.x - 1) / gridDim.x;
  const uint64_t lo = uint64_t(blockIdx.x) * per, hi = min(slots, lo + per);
  __shared__ unsigned long long scan[kGNT / 64 + 1];
  emit_range(g.key, g.cnt, g.sum[0], g.sum[1], lo, hi, g.sentinel, nv, o, scan);
}

int gb_sentinel(const eiger_groupby_plan_t &p, unsigned long long *out) {
  *out = static_cast<unsigned long long>(p.sentinel);
  return EIGER_OK;
}

// Slices per partition: few partitions (few groups) are cut into slices so the
// grid still has about four work items per CU of the 256; slices keep at least
// 2^14 rows. With more than one slice every group reaches the global table.
constexpr uint64_t kGTargetItems = 1024;
uint32_t gb_slices(uint64_t n, int bits) {
  const uint64_t F = uint64_t(1) << bits;
  uint32_t S = 1;
  while (uint64_t(S) * F < kGTargetItems && n / (uint64_t(S) * 2 * F) >= (uint64_t(1) << 14)) S <<= 1;
  return S;
}

uint64_t gb_slots(double groups) {
  uint64_t s = 1024;
  while (static_cast<double>(s) < 2.0 * groups + 1.0) s <<= 1;
  return s;
}

struct GbLayout {
  GbGlobal g;
  unsigned long long *cursor;
  uint32_t *overflow;
};

GbLayout gb_layout(Workspace &ws, uint64_t slots, int nv, unsigned long long sentinel) {
  GbLayout L{};
  L.g.key = ws.take<unsigned long long>(slots);
  L.g.cnt = ws.take<unsigned long long>(slots);
  for (int v = 0; v < kGMaxVals; ++v) L.g.sum[v] = v < nv ? ws.take<unsigned long long>(slots) : nullptr;
  L.g.mask = slots - 1;
  L.g.sentinel = sentinel;
  L.cursor = ws.take<unsigned long long>(2);  // the flag in the second word, for one copy to the host
  L.overflow = reinterpret_cast<uint32_t *>(L.cursor + 1);
  L.g.overflow = L.overflow;
  return L;
}

// Launches of the aggregating kernels for the column widths of a call.
struct AggCall {
  GbVals vals;
  AggShape shape;
  GbGlobal g;
  hipStream_t s;
};

template <typename K, int NV, bool W0, bool W1>
int agg_hash_launch(const AggCall &a, const K *keys, uint64_t n) {
  // contiguous ranges of whole steps, all of them in flight together
  const uint64_t steps = (n + kAStep - 1) / kAStep, cap = uint64_t(device_cu_count()) * agg_per_cu<NV, W0>;
  const uint64_t per = (steps + cap - 1) / cap * kAStep;
  const dim3 grid(static_cast<unsigned>((n + per - 1) / per));
  // With four accumulators a slot or more (up to 128 groups) sorted rows cost no more
  // than others (2^26 rows, 100 groups, two 4-byte sums: 210 us, 219 in random order),
  // and the look for clustered ones would cost 3 to 8%.
  if (a.shape.reps <= 2)
    EIGER_LAUNCH("groupby_hash", (k_gb_hash<K, NV, W0, W1, true>), grid, dim3(kANT), 0, a.s, keys, n, a.vals, a.shape, per, a.g);
  else
    EIGER_LAUNCH("groupby_hash", (k_gb_hash<K, NV, W0, W1, false>), grid, dim3(kANT), 0, a.s, keys, n, a.vals, a.shape, per, a.g);
  return EIGER_OK;
}

template <typename K, int NV, bool W0, bool W1>
int agg_partition_launch(const AggCall &a, const K *keys, const uint32_t *off, uint32_t F, uint32_t S, const GbOut &o) {
  const uint64_t cap = uint64_t(device_cu_count()) * agg_per_cu<NV, W0>;
  EIGER_LAUNCH("groupby_partition", (k_gb_partition<K, NV, W0, W1>),
               dim3(static_cast<unsigned>(std::min<uint64_t>(uint64_t(F) * S, cap))), dim3(kANT), 0, a.s, keys, a.vals,
               off, F, S, a.shape, a.g, o);
  return EIGER_OK;
}

#define EIGER_AGG_DISPATCH(FN, ...)                        \
  do {                                                     \
    if (nv == 0) return FN<K, 0, false, false>(__VA_ARGS__); \
    if (nv == 1 && !w0) return FN<K, 1, false, false>(__VA_ARGS__); \
    if (nv == 1) return FN<K, 1, true, false>(__VA_ARGS__);  \
    if (!w0 && !w1) return FN<K, 2, false, false>(__VA_ARGS__); \
    if (!w0) return FN<K, 2, false, true>(__VA_ARGS__);      \
    if (!w1) return FN<K, 2, true, false>(__VA_ARGS__);      \
    return FN<K, 2, true, true>(__VA_ARGS__);                \
  } while (0)

template <typename K>
int run_agg_hash(const AggCall &a, int nv, bool w0, bool w1, const K *keys, uint64_t n) {
  EIGER_AGG_DISPATCH(agg_hash_launch, a, keys, n);
}

template <typename K>
int run_agg_partition(const AggCall &a, int nv, bool w0, bool w1, const K *keys, const uint32_t *off, uint32_t F,
                      uint32_t S, const GbOut &o) {
  EIGER_AGG_DISPATCH(agg_partition_launch, a, keys, off, F, S, o);
}
#undef EIGER_AGG_DISPATCH

// Lays out and (with a workspace base) enqueues the group-by.
template <typename K>
int gb_impl(const eiger_column &keys, const eiger_column *vals, int32_t nv, const eiger_groupby_plan_t &plan,
            const GbOut &out_in, Workspace &ws, GbLayout *lay, hipStream_t s) {
  const uint64_t n = static_cast<uint64_t>(keys.n);
  unsigned long long sentinel;
  gb_sentinel(plan, &sentinel);
  *lay = gb_layout(ws, static_cast<uint64_t>(plan.slots), nv, sentinel);
  PartitionOut part{};
  PartLanes wc{};
  if (plan.variant == EIGER_GB_PARTITION) {
    for (int32_t c = 0; c < nv; ++c) {
      const uint32_t *base = static_cast<const uint32_t *>(vals[c].data);
      if (vals[c].dtype == EIGER_INT64) {
        wc.src[wc.n] = base;
        wc.stride[wc.n++] = 2;
        wc.src[wc.n] = base ? base + 1 : nullptr;
        wc.stride[wc.n++] = 2;
      } else {
        wc.src[wc.n] = base;
        wc.stride[wc.n++] = 1;
      }
    }
    int rc = radix_partition_lanes(static_cast<int>(dtype_size(keys.dtype)), keys.data, n, wc, plan.radix_bits, ws,
                                   &part, n > 0 ? s : nullptr, n > 0);
    if (rc) return rc;
  }
  if (!ws.base) return EIGER_OK;
  const GbGlobal &g = lay->g;
  GbOut o = out_in;
  o.cursor = lay->cursor;
  int rc;
  const unsigned cus = static_cast<unsigned>(device_cu_count());
  EIGER_LAUNCH("groupby_clear", k_gb_clear, dim3(std::min<uint64_t>((plan.slots + kGNT - 1) / kGNT, cus * 8)),
               dim3(kGNT), 0, s, g, nv, lay->cursor);
  if (n == 0) return EIGER_OK;
  const bool w0 = nv > 0 && vals[0].dtype == EIGER_INT64, w1 = nv > 1 && vals[1].dtype == EIGER_INT64;
  AggCall call{};
  call.g = g;
  call.s = s;
  if (plan.variant == EIGER_GB_HASH) {
    for (int32_t c = 0; c < nv; ++c) call.vals.lo[c] = static_cast<const uint32_t *>(vals[c].data);
    call.shape = agg_shape(static_cast<double>(plan.predicted_groups));
    if ((rc = run_agg_hash<K>(call, nv, w0, w1, static_cast<const K *>(keys.data), n))) return rc;
  } else {
    // partitioned values: one word array per lane
    int w = 0;
    for (int32_t c = 0; c < nv; ++c) {
      call.vals.lo[c] = part.words[w++];
      if (vals[c].dtype == EIGER_INT64) call.vals.hi[c] = part.words[w++];
    }
    const uint32_t F = 1u << plan.radix_bits;
    call.shape = agg_whole();  // unevenly filled partitions
    if ((rc = run_agg_partition<K>(call, nv, w0, w1, static_cast<const K *>(part.keys), part.off, F,
                                   gb_slices(n, plan.radix_bits), o)))
      return rc;
  }
  EIGER_LAUNCH("groupby_emit", k_gb_emit, dim3(static_cast<unsigned>(std::min<uint64_t>(
                                              (plan.slots + 4095) / 4096, cus * 4))),
               dim3(kGNT), 0, s, g, nv, o);
  return EIGER_OK;
}

int gb_run(const eiger_column &keys, const eiger_column *vals, int32_t nv, const eiger_groupby_plan_t &plan,
           const GbOut &o, Workspace &ws, GbLayout *lay, hipStream_t s) {
  if (keys.dtype == EIGER_INT64) return gb_impl<int64_t>(keys, vals, nv, plan, o, ws, lay, s);
  return gb_impl<int32_t>(keys, vals, nv, plan, o, ws, lay, s);
}

int gb_check(const eiger_column &keys, const eiger_column *vals, int32_t nv, const eiger_groupby_plan_t *plan) {
  if (!plan) return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: plan is NULL");
  if (keys.dtype != EIGER_INT32 && keys.dtype != EIGER_INT64)
    return fail(EIGER_ERR_DTYPE, "eiger_groupby: key dtype must be EIGER_INT32 or EIGER_INT64");
  if (keys.dtype != plan->key_dtype) return fail(EIGER_ERR_DTYPE, "eiger_groupby: plan.key_dtype differs from the keys");
  if (keys.n < 0) return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: negative row count");
  if (keys.n > EIGER_MAX_ROWS) return fail(EIGER_ERR_TOO_LARGE, "eiger_groupby: more than EIGER_MAX_ROWS rows");
  if (keys.n > 0 && (!keys.data || reinterpret_cast<uintptr_t>(keys.data) % dtype_size(keys.dtype)))
    return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: keys NULL or misaligned");
  if (nv < 0 || nv > kGMaxVals) return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: 0 to 2 value columns");
  if (nv > 0 && !vals) return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: NULL value column array");
  for (int32_t c = 0; c < nv; ++c) {
    if (vals[c].dtype != EIGER_INT32 && vals[c].dtype != EIGER_INT64)
      return fail(EIGER_ERR_DTYPE, "eiger_groupby: value dtype must be EIGER_INT32 or EIGER_INT64");
    if (vals[c].n != keys.n) return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: value column length differs");
    if (keys.n > 0 && (!vals[c].data || reinterpret_cast<uintptr_t>(vals[c].data) % dtype_size(vals[c].dtype)))
      return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: value column NULL or misaligned");
  }
  if (plan->variant != EIGER_GB_HASH && plan->variant != EIGER_GB_PARTITION)
    return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: plan.variant is not an eiger_groupby_variant");
  if (plan->slots < 1024 || (plan->slots & (plan->slots - 1)))
    return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: plan.slots must be a power of two >= 1024");
  if (plan->variant == EIGER_GB_PARTITION && (plan->radix_bits < 1 || plan->radix_bits > 18))
    return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: plan.radix_bits must be in [1, 18]");
  if (plan->flags & EIGER_GB_NO_SENTINEL)
    return fail(EIGER_ERR_UNSUPPORTED, "eiger_groupby: the keys span the whole int64 domain (no free value marks "
                                       "empty slots)");
  return EIGER_OK;
}

}  // namespace
}  // namespace eiger

using namespace eiger;

extern "C" int eiger_groupby_plan(const eiger_stats_t *keys, int32_t selector, const eiger_groupby_plan_t *forced,
                                  eiger_groupby_plan_t *out) {
  if (!keys || !out) return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby_plan: NULL argument");
  if (keys->dtype != EIGER_INT32 && keys->dtype != EIGER_INT64)
    return fail(EIGER_ERR_DTYPE, "eiger_groupby_plan: unsupported key dtype");
  eiger_groupby_plan_t p{};
  p.key_dtype = keys->dtype;
  // a value outside [min, max] marks empty slots; int32 keys never reach INT64_MIN
  if (keys->dtype == EIGER_INT32 || keys->n == 0 || keys->min > INT64_MIN) {
    p.sentinel = INT64_MIN;
  } else if (keys->max < INT64_MAX) {
    p.sentinel = INT64_MAX;
  } else {
    p.flags |= EIGER_GB_NO_SENTINEL;
  }
  const double est = std::max(1.0, std::min(keys->ndv, static_cast<double>(std::max<int64_t>(keys->n, 1))));
  p.predicted_groups = static_cast<int64_t>(std::llround(est));
  if (selector == EIGER_SEL_FORCED) {
    if (!forced) return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby_plan: EIGER_SEL_FORCED needs `forced`");
    p.variant = forced->variant;
    p.radix_bits = forced->radix_bits;
  } else if (selector == EIGER_SEL_RULE || selector == EIGER_SEL_LEARNED) {
    p.variant = est <= kGbHashMaxGroups ? EIGER_GB_HASH : EIGER_GB_PARTITION;
    p.radix_bits = 0;
  } else {
    return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby_plan: selector must be EIGER_SEL_RULE or EIGER_SEL_FORCED");
  }
  if (p.variant == EIGER_GB_PARTITION && (p.radix_bits < 1 || p.radix_bits > 18)) {
    int bits = 1;
    while (bits < 18 && est / std::ldexp(1.0, bits) > kGbGroupsPerPartition) ++bits;
    p.radix_bits = bits;
  }
  // the global table: NDV-sized (twice the estimate) when every group reaches
  // it (HASH, or sliced partitions); unsliced partitions only spill into it
  const bool all_global = p.variant == EIGER_GB_HASH || gb_slices(static_cast<uint64_t>(keys->n), p.radix_bits) > 1;
  p.slots = static_cast<int64_t>(gb_slots(all_global ? est : est / 8.0));
  *out = p;
  return EIGER_OK;
}

extern "C" int eiger_groupby_workspace_size(const eiger_groupby_plan_t *plan, eiger_column keys,
                                            const eiger_column *vals, int32_t n_vals, size_t *bytes) {
  if (!bytes) return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby_workspace_size: bytes is NULL");
  static const int64_t dummy[1] = {0};
  eiger_column k = keys, v[kGMaxVals];
  if (k.n > 0) k.data = dummy;
  if (n_vals < 0 || n_vals > kGMaxVals) return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: 0 to 2 value columns");
  for (int32_t c = 0; c < n_vals; ++c) {
    if (!vals) return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: NULL value column array");
    v[c] = vals[c];
    if (v[c].n > 0) v[c].data = dummy;
  }
  int rc = gb_check(k, v, n_vals, plan);
  if (rc) return rc;
  Workspace ws(nullptr, 0);
  GbLayout lay{};
  if ((rc = gb_run(k, v, n_vals, *plan, GbOut{}, ws, &lay, nullptr))) return rc;
  *bytes = ws.used;
  return EIGER_OK;
}

extern "C" int eiger_groupby(eiger_column keys, const eiger_column *vals, int32_t n_vals,
                             const eiger_groupby_plan_t *plan, void *out_keys, int64_t *out_counts,
                             int64_t *const *out_sums, int64_t out_capacity, int64_t *out_groups, void *ws_ptr,
                             size_t ws_bytes, void *stream) {
  int rc = gb_check(keys, vals, n_vals, plan);
  if (rc) return rc;
  if (!out_groups) return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: out_groups is NULL");
  if (out_capacity < 0) return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: negative out_capacity");
  if (out_capacity > 0 && (!out_keys || !out_counts || (n_vals > 0 && !out_sums)))
    return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: NULL output arrays");
  for (int32_t c = 0; out_capacity > 0 && c < n_vals; ++c)
    if (!out_sums[c]) return fail(EIGER_ERR_INVALID_ARG, "eiger_groupby: NULL sum output");
  {
    Workspace dry(nullptr, 0);
    GbLayout lay{};
    if ((rc = gb_run(keys, vals, n_vals, *plan, GbOut{}, dry, &lay, nullptr))) return rc;
    if (!ws_ptr || dry.used > ws_bytes)
      return fail(EIGER_ERR_WORKSPACE, "eiger_groupby: workspace too small (need " + std::to_string(dry.used) +
                                           " bytes)");
  }
  GbOut o{};
  o.keys = out_capacity > 0 ? out_keys : nullptr;
  o.cnt = reinterpret_cast<unsigned long long *>(out_counts);
  for (int32_t c = 0; c < n_vals; ++c)
    o.sum[c] = out_capacity > 0 ? reinterpret_cast<unsigned long long *>(out_sums[c]) : nullptr;
  o.cap = static_cast<uint64_t>(out_capacity);
  o.kwide = keys.dtype == EIGER_INT64;
  hipStream_t s = static_cast<hipStream_t>(stream);
  Workspace ws(ws_ptr, ws_bytes);
  GbLayout lay{};
  if ((rc = gb_run(keys, vals, n_vals, *plan, o, ws, &lay, s))) return rc;
  struct {
    unsigned long long groups;
    uint32_t overflow;
  } host{};
  static_assert(sizeof(host) == 16, "cursor and flag as they lie in the workspace");
  EIGER_HIP(hipMemcpyAsync(&host, lay.cursor, sizeof(host), hipMemcpyDeviceToHost, s));
  EIGER_HIP(hipStreamSynchronize(s));
  if (host.overflow)
    return fail(EIGER_ERR_TOO_LARGE, "eiger_groupby: more groups than the plan's table slots (the distinct-count "
                                     "estimate was low); raise plan.slots");
  *out_groups = static_cast<int64_t>(host.groups);
  if (host.groups > static_cast<uint64_t>(out_capacity))
    return fail(EIGER_ERR_CAPACITY, "eiger_groupby: " + std::to_string(host.groups) + " groups exceed out_capacity " +
                                        std::to_string(out_capacity));
  return EIGER_OK;
}
