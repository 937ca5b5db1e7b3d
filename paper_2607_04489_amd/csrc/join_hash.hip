// join_hash.hip -- GLOBAL_HASH variant: one open-addressing table in HBM.
//
// This is the non-partitioned hash join of the paper (Section 3.2, Table 1),
// laid out for gfx950: the key, row id and payload of a build row share one
// 16-byte slot (32 bytes when key and payload are both 8 bytes), so a probe
// touches one cache line per slot group instead of gathering keys through
// tuple ids (the cost the paper blames for the hash join's losses, Section
// 5.2.1). Slots are claimed by CAS on the key word with a sentinel key outside
// the build range (duplicates show up during the build), or, when the build
// keys reach both ends of the key domain, by CAS on the row-id word followed
// by a duplicate check. Empty slots have row id 0xFFFFFFFF either way. The
// table is a multiset: duplicate build keys occupy several slots and a probe
// walks (line_walk) until an empty slot.
#include <limits>
#include <type_traits>

#include "join_common.hpp"
#include "variants.hpp"

namespace eiger {

namespace {

// Table sizes at which the probe changes (see hash_impl).
constexpr uint64_t kNearBytes = 8u << 20, kFarBytes = 2ull << 30;

// Probe workgroups of a CU, their threads, and the pairs that a wave stages in the LDS
// that the queues leave: 632 of 4-byte keys and payloads in 16 waves a CU; 652 where one
// has 8 bytes, 492 where both have, in 14 (16 waves with fewer pairs, 2^23 probes of one
// int32 key with int64 payloads: 10% slower). Counting takes 24 or 16.
template <typename K, typename PS, bool kPairs>
constexpr int kPPerCu = !kPairs && sizeof(K) + sizeof(PS) == 8 ? 3 : 2;
template <typename K, typename PS, bool kPairs>
constexpr int kPNT = kPairs && sizeof(K) + sizeof(PS) > 8 ? 448 : 512;
template <typename K, typename PS, bool kPairs>
constexpr uint32_t kPStage = kPairs ? wave_stage<K, PS>(kPNT<K, PS, true> / 64 * kPPerCu<K, PS, true>) : 0;

template <typename K, typename PB>
struct HashTab {
  static constexpr bool kWalk = true;
  using SlotT = Slot<K, PB>;
  using Index = uint64_t;  // a table may hold more than 2^32 slots
  const Slot<K, PB> *__restrict__ slots;
  uint64_t mask;
  const uint32_t *dup;  // device flag: nonzero when some build key occurs twice
  bool unique;          // set in the kernel from *dup

  __device__ __forceinline__ void init() { unique = dup && *dup == 0; }
  __device__ __forceinline__ uint64_t home(K key) const {
    return fmix64(static_cast<uint64_t>(sext(key))) & mask;
  }
  __device__ __forceinline__ uint64_t start(K key, bool &in) const {
    in = true;
    return home(key);
  }
  __device__ __forceinline__ uint64_t walk(uint64_t i, uint32_t steps) const { return line_walk<SlotT>(i, steps, mask); }
  __device__ __forceinline__ SlotT load(uint64_t i) const { return slots[i]; }
};

// The same table of 32-byte slots for a probe that holds each row's walk in its lane:
// the two slots of the first line, the home slot first, then those of the next, each
// one step from the slot before.
template <typename K, typename PB>
struct HashRowTab : HashTab<K, PB> {
  static_assert(sizeof(Slot<K, PB>) == 32, "two slots in 64 bytes");
  static constexpr bool kHashed = true;
  static constexpr bool kRuns = false;
  __device__ __forceinline__ uint64_t next(uint64_t i, uint32_t step) const {
    return step & 1 ? i ^ 1 : ((i ^ 1) + 2) & this->mask;
  }
  template <class F>
  __device__ __forceinline__ void for_each(K key, F f) const {
    uint64_t i = this->home(key);
    for (uint32_t step = 1;; ++step) {
      const Slot<K, PB> s = this->slots[i];
      if (s.rowid == kEmpty) break;
      if (s.key == key) f(s.rowid);
      i = next(i, step);
    }
  }
};

// Sets *dup when some build key occurs more than once: every build row walks its key's
// cluster, 64 bytes a step, until it meets the key again or the flag is found set.
// Afterwards probes of a table with distinct keys stop at their first match. (No key
// lies past an empty slot of its walk, so that all slots of a line can be counted.)
template <typename K, typename PB>
__global__ void k_hash_unique(const K *__restrict__ keys, uint64_t n, HashTab<K, PB> tab,
                              uint32_t *dup) {
  constexpr uint64_t per = 64 / sizeof(Slot<K, PB>);
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t r = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; r < n; r += stride) {
    const K key = keys[r];
    uint64_t at = tab.home(key) & ~(per - 1);
    uint32_t c = 0;
    for (uint32_t line = 0;; ++line) {
      if (line % 16 == 0 && *static_cast<volatile uint32_t *>(dup)) return;
      Slot<K, PB> s[per];
#pragma unroll
      for (uint32_t q = 0; q < per; ++q) s[q] = tab.slots[at + q];
      bool last = false;
#pragma unroll
      for (uint32_t q = 0; q < per; ++q) {
        last |= s[q].rowid == kEmpty;
        c += s[q].rowid != kEmpty && s[q].key == key;
      }
      if (c > 1) atomicOr(dup, 1u);
      if (last || c > 1) break;
      at = (at + per) & tab.mask;
    }
  }
}

template <typename K, typename PB>
__global__ void k_hash_build(const K *__restrict__ keys, const PB *__restrict__ pay, uint64_t n,
                             Slot<K, PB> *__restrict__ slots, uint64_t mask) {
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t r = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; r < n; r += stride) {
    const K key = keys[r];
    const uint64_t home = fmix64(static_cast<uint64_t>(sext(key))) & mask;
    // The table has more slots than rows, so an empty slot is always found.
    for (uint32_t step = 0;; ++step) {
      const uint64_t i = line_walk<Slot<K, PB>>(home, step, mask);
      if (atomicCAS(&slots[i].rowid, kEmpty, static_cast<uint32_t>(r)) == kEmpty) {
        slots[i].key = key;
        slots[i].pay = pay[r];
        break;
      }
    }
  }
}

// Table clear for the key-claiming build: key = sentinel, row id = empty. Slots
// are 16 or 32 bytes (one or two 16-byte words); each workgroup stores one
// contiguous chunk of the table with 16-byte stores, as the library's fills do.
// The first one also zeroes the join's counters and duplicate flag.
template <typename K, typename PB>
__global__ void __launch_bounds__(256) k_hash_clear(Slot<K, PB> *__restrict__ slots, uint64_t n, K sentinel,
                                                    HashCounters *__restrict__ c, uint32_t *__restrict__ dup) {
  static_assert(sizeof(HashCounters) / 8 <= 256, "one word per thread");
  if (blockIdx.x == 0) {
    if (threadIdx.x < sizeof(HashCounters) / 8) reinterpret_cast<uint64_t *>(c)[threadIdx.x] = 0;
    if (threadIdx.x == 0) *dup = 0;
  }
  constexpr int kWords = sizeof(Slot<K, PB>) / 16;
  static_assert(kWords == 1 || kWords == 2, "16- or 32-byte slots");
  Slot<K, PB> e{};
  e.key = sentinel;
  e.rowid = kEmpty;
  uint4 w[kWords];
  __builtin_memcpy(w, &e, sizeof(e));
  uint4 *__restrict__ q = reinterpret_cast<uint4 *>(slots);
  const uint64_t nw = n * kWords;
  const uint64_t per = (nw + gridDim.x - 1) / gridDim.x;
  const uint64_t lo = uint64_t(blockIdx.x) * per, hi = min(nw, lo + per);
  for (uint64_t i = lo + threadIdx.x; i < hi; i += blockDim.x) q[i] = w[i % kWords];
}

// Build that claims a slot by CAS on its key word (empty = a sentinel value no
// build key takes), so a row that meets its own key on the way has found a
// duplicate: the distinctness flag comes out of the build, without a second
// walk per build row. A key equal to the sentinel (the plan's key range was
// wrong) is reported through the counters' flags.
template <typename K, typename PB>
__global__ void k_hash_build_keys(const K *__restrict__ keys, const PB *__restrict__ pay, uint64_t n,
                                  Slot<K, PB> *__restrict__ slots, uint64_t mask, K sentinel, uint32_t *dup,
                                  uint64_t *flags) {
  using W = typename std::conditional<sizeof(K) == 8, unsigned long long, unsigned int>::type;
  const W empty = static_cast<W>(sentinel);
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  bool seen = false;
  for (uint64_t r = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; r < n; r += stride) {
    const K key = keys[r];
    if (key == sentinel) {
      atomicOr(reinterpret_cast<unsigned long long *>(flags), kFlagBuildOutOfRange);
      continue;
    }
    const uint64_t home = fmix64(static_cast<uint64_t>(sext(key))) & mask;
    // The table has more slots than rows, so an empty slot is always found.
    for (uint32_t step = 0;; ++step) {
      const uint64_t i = line_walk<Slot<K, PB>>(home, step, mask);
      const W old = atomicCAS(reinterpret_cast<W *>(&slots[i].key), empty, static_cast<W>(key));
      if (old == empty) {
        slots[i].rowid = static_cast<uint32_t>(r);
        slots[i].pay = pay[r];
        break;
      }
      seen |= old == static_cast<W>(key);
    }
  }
  // One atomic a workgroup, and none once the flag is seen set: they are on one address,
  // 10 ns each (563,000 rows of repeated keys: 79 us, 152 with one a wave).
  if (__syncthreads_or(seen) && threadIdx.x == 0 && __atomic_load_n(dup, __ATOMIC_RELAXED) == 0) atomicOr(dup, 1u);
}

// A key value outside the plan's build range, if the key type has one.
template <typename K>
bool hash_sentinel(const JoinArgs &a, K *out) {
  const int64_t lo = static_cast<int64_t>(std::numeric_limits<K>::min());
  const int64_t hi = static_cast<int64_t>(std::numeric_limits<K>::max());
  if (a.nR == 0 || a.plan.build_min > lo) {
    *out = std::numeric_limits<K>::min();
    return true;
  }
  if (a.plan.build_max < hi) {
    *out = std::numeric_limits<K>::max();
    return true;
  }
  return false;
}

// Each workgroup streams a contiguous range of probe rows (an equal share of
// whole blocks), its waves taking blocks in turn. repeated_only: tables of distinct
// keys are k_probe_rows'.
template <class Tab, typename K, typename PS, int kEager, bool kPairs>
__global__ void __launch_bounds__((kPNT<K, PS, kPairs>)) k_probe(Tab tab, const K *__restrict__ pk,
                                               const PS *__restrict__ pp, uint64_t n, EmitOut o,
                                               bool repeated_only, uint32_t block) {
  constexpr int kNT = kPNT<K, PS, kPairs>;
  constexpr uint32_t kStage = kPStage<K, PS, kPairs>;
  __shared__ WaveLds<K, PS, kStage> L[kNT / 64];
  __shared__ WaveJoint<kNT / 64> J;
  static_assert((sizeof(L) + sizeof(J)) * kPPerCu<K, PS, kPairs> <= 163840, "the workgroups of a CU share its LDS");
  tab.init();
  if (repeated_only && tab.unique) return;
  const uint64_t sub = kNT / 64 * block;
  const uint32_t w = threadIdx.x / 64;
  const uint64_t nsub = (n + sub - 1) / sub;
  const uint64_t per = (nsub + gridDim.x - 1) / gridDim.x;
  const uint64_t lo = blockIdx.x * per * sub;
  const uint64_t hi = lo + per * sub < n ? lo + per * sub : n;
  WaveProbe<Tab, K, PS, kEager, kStage> p(tab, L[w], o);
  p.template run<kNT / 64>(pk, pp, nullptr, lo + w * block, hi, sub, J, block);
}

constexpr int kRowNT = 256;
constexpr int kRowIPT = 5;  // rows per thread
constexpr int kRowSCAP = 4096;

// Each thread holds the walks of its rows to their end, five first slots in flight.
// distinct_only: tables of repeated keys are k_probe's.
template <typename K, typename PB, typename PS>
__global__ void __launch_bounds__(kRowNT) k_probe_rows(HashRowTab<K, PB> tab, const K *__restrict__ pk,
                                                     const PS *__restrict__ pp, uint64_t n, EmitOut o,
                                                     bool distinct_only) {
  __shared__ EmitLds<kRowNT, kRowSCAP> L;
  uint64_t fill = 0, cs = 0;
  tab.init();
  if (distinct_only && !tab.unique) return;
  constexpr uint64_t sub = uint64_t(kRowNT) * kRowIPT;
  const uint64_t nsub = (n + sub - 1) / sub;
  const uint64_t per = (nsub + gridDim.x - 1) / gridDim.x;
  const uint64_t lo = blockIdx.x * per * sub;
  const uint64_t hi = lo + per * sub < n ? lo + per * sub : n;
  probe_range<kRowNT, kRowIPT, kRowSCAP>(tab, pk, pp, static_cast<const uint32_t *>(nullptr), lo, hi, L, fill, o, cs);
  finish(L, o, fill, cs);
}

unsigned grid_for(uint64_t work, uint64_t per_block, int per_cu) {
  uint64_t g = (work + per_block - 1) / per_block;
  const uint64_t cap = uint64_t(device_cu_count()) * per_cu;
  if (g > cap) g = cap;
  return static_cast<unsigned>(g ? g : 1);
}

// Rows that a wave of the probe takes together: 64 * kWaveRows, fewer where the probe side
// leaves waves without any (256 probes of 64 matches each: 49 us of probe, 131 when one
// wave took them all).
template <typename K, typename PS, bool kPairs>
uint32_t probe_block(uint64_t n) {
  const uint64_t waves = uint64_t(device_cu_count()) * kPPerCu<K, PS, kPairs> * (kPNT<K, PS, kPairs> / 64);
  uint32_t block = 64;
  while (block < 64 * kWaveRows && n > waves * block) block *= 2;
  return block;
}

template <typename K, typename PB, typename PS, int kEager, bool kPairs>
int launch_probe(const HashTab<K, PB> &tab, const K *pk, const PS *pp, uint64_t n, const EmitOut &o, bool repeated_only,
                 hipStream_t s) {
  const uint32_t block = probe_block<K, PS, kPairs>(n);
  const dim3 grid(grid_for(n, kPNT<K, PS, kPairs> / 64 * uint64_t(block), kPPerCu<K, PS, kPairs>));
  EIGER_LAUNCH("hash_probe", (k_probe<HashTab<K, PB>, K, PS, kEager, kPairs>), grid, dim3(kPNT<K, PS, kPairs>), 0, s, tab, pk, pp, n, o,
               repeated_only, block);
  return EIGER_OK;
}

template <typename K, typename PB, typename PS>
int hash_impl(const JoinArgs &a, Workspace &ws, JoinCounters **ctr) {
  const uint64_t nslots = hash_slots(a.nR, a.plan.load_factor);
  HashCounters *hc = ws.take<HashCounters>(1);
  uint32_t *dup = ws.take<uint32_t>(1);
  Slot<K, PB> *slots = ws.take<Slot<K, PB>>(nslots);
  if (!ws.base) {  // sizing: there are no counters to point at
    *ctr = nullptr;
    return EIGER_OK;
  }
  JoinCounters *c = &hc->total;
  *ctr = c;
  hipStream_t s = a.s;
  int rc;
  K sentinel;
  const bool by_key = a.nR > 0 && a.nS > 0 && hash_sentinel<K>(a, &sentinel);
  if (!by_key && (rc = fill_u64(reinterpret_cast<uint64_t *>(hc), sizeof(HashCounters) / 8, 0, s))) return rc;
  if (a.nR == 0 || a.nS == 0) return EIGER_OK;
  if (!by_key && (rc = fill_u32(dup, 1, 0, s))) return rc;
  HashTab<K, PB> tab{slots, nslots - 1, dup, false};
  if (by_key) {
    EIGER_LAUNCH("hash_clear", (k_hash_clear<K, PB>),
                 dim3(static_cast<unsigned>(std::min<uint64_t>((nslots + 1023) / 1024, uint64_t(device_cu_count()) * 16))),
                 dim3(256), 0, s, slots, nslots, sentinel, hc, dup);
    EIGER_LAUNCH("hash_build", (k_hash_build_keys<K, PB>), dim3(grid_for(a.nR, 256, 8)), dim3(256), 0, s,
                 static_cast<const K *>(a.bk), static_cast<const PB *>(a.bp), a.nR, slots, nslots - 1, sentinel,
                 dup, &c->flags);
  } else {
    // keys at both ends of the domain: claim by row id, then a duplicate check
    if ((rc = fill_u32(reinterpret_cast<uint32_t *>(slots), nslots * sizeof(Slot<K, PB>) / 4, kEmpty, s)))
      return rc;
    EIGER_LAUNCH("hash_build", (k_hash_build<K, PB>), dim3(grid_for(a.nR, 256, 8)), dim3(256), 0, s,
                 static_cast<const K *>(a.bk), static_cast<const PB *>(a.bp), a.nR, slots, nslots - 1);
    EIGER_LAUNCH("hash_unique", (k_hash_unique<K, PB>), dim3(grid_for(a.nR, 256, 8)), dim3(256), 0, s,
                 static_cast<const K *>(a.bk), a.nR, tab, dup);
  }
  EmitOut o{a.ob, a.op, a.cap, &c->count, &c->checksum, hc->stripe};
  const K *pk = static_cast<const K *>(a.pk);
  const PS *pp = static_cast<const PS *>(a.pp);
  // Which probe (2^27 probes in random order that all match, half-full tables, ms with
  // pairs / count only; one and two: slots a wave loads of every row at first):
  //   32-byte slots   8 MiB: rows 2.65/2.47 one 2.16/1.71 two 2.11/1.71
  //                  16 MiB: rows 2.81/2.61 one 2.67/2.45 two 2.39/2.13
  //                  64 MiB: rows 3.10/2.90 one 3.61/3.41 two 3.01/2.81
  //                   2 GiB: rows 4.08/3.76 one 4.03/3.77 two 3.65/3.19
  //                   4 GiB: rows 4.39/4.10 one 4.70/4.39 two 6.36/6.06
  //   16-byte slots   2 MiB:                one 1.35/1.03 two 1.35/1.00
  //                   8 MiB:                one 1.71/1.43 two 1.70/1.35
  //                  16 MiB:                one 2.34/2.18 two 2.16/1.98
  //                   1 GiB:                one 3.55/3.47 two 3.26/2.97
  //   (8-byte keys)   1 GiB:                one 3.58/3.49 two 3.30/3.00
  //                   4 GiB:                one 3.59/3.46 two 3.55/3.31
  // Small tables are bound by the L1's fills, and a second slot of every row costs more
  // of them than it saves: it loses 2 to 8% of 2^22 probes of 1,000 and 2,000 keys, where
  // the L1 holds some of the table, is even from 2 to 8 MiB (5% behind in a quarter-full
  // table, 9% ahead where no probe matches) and from larger tables comes with the first.
  // Beyond 2 GiB two slots are two address translations in flight instead of one; the
  // line lies where 32-byte slots need it. With 32-byte slots and pairs the rows' probe,
  // whose workgroups write out every 1,280 rows' matches together, is the slower one in
  // random order up to 2 GiB (above), but ahead where most probes stay near, where
  // the waves' falls behind what a thread a row had always taken (sorted probes of
  // 60,000 and 400,000 rows 1.03 to 1.09 times, of one key up to 1.28). Walks among
  // repeated keys are long, and there the waves' probe is the faster (2^22 probes of
  // 4,000 keys of 8 rows: 0.74 ms for 2.00; 2^24 of 250,000 of 4: 2.6 for 5.2). The build
  // tells which it is: both are launched, one returns at once. Small probe sides are left
  // to the waves' alone: with a row a lane the matches of distinct keys fit a wave's stage,
  // and of two kernels the second comes late (90 x 136 rows of repeated keys: 72 us of
  // join, 95 with both).
  const uint64_t bytes = nslots * sizeof(Slot<K, PB>);
  const bool near = bytes <= kNearBytes, far = bytes > kFarBytes;
  bool by_rows = false;
  if constexpr (sizeof(Slot<K, PB>) == 32) {
    by_rows = (a.ob && probe_block<K, PS, true>(a.nS) > 64) || far;
    if (by_rows) {
      HashRowTab<K, PB> rows;
      static_cast<HashTab<K, PB> &>(rows) = tab;
      EIGER_LAUNCH("hash_probe", (k_probe_rows<K, PB, PS>), dim3(grid_for(a.nS, uint64_t(kRowNT) * kRowIPT, 4)),
                   dim3(kRowNT), 0, s, rows, pk, pp, a.nS, o, a.ob != nullptr);
      if (!a.ob) return EIGER_OK;  // (counted pairs of repeated keys: 15.4 ms for 16.3 at 4 GiB)
    }
  }
  if (a.ob)
    return near || far ? launch_probe<K, PB, PS, 1, true>(tab, pk, pp, a.nS, o, by_rows, s)
                       : launch_probe<K, PB, PS, 2, true>(tab, pk, pp, a.nS, o, by_rows, s);
  return near || far ? launch_probe<K, PB, PS, 1, false>(tab, pk, pp, a.nS, o, false, s)
                     : launch_probe<K, PB, PS, 2, false>(tab, pk, pp, a.nS, o, false, s);
}

}  // namespace

uint64_t hash_slots(uint64_t n, float lf) {
  if (!(lf > 0.f) || lf > 0.9f) lf = 0.5f;
  uint64_t want = static_cast<uint64_t>(static_cast<double>(n) / lf) + 1;
  uint64_t s = 64;
  while (s < want) s <<= 1;
  return s;
}

int run_global_hash(const JoinArgs &a, Workspace &ws, JoinCounters **ctr) {
  const bool k64 = a.kdt == EIGER_INT64, b64 = a.bpdt == EIGER_INT64, p64 = a.ppdt == EIGER_INT64;
#define EIGER_DISPATCH(KT, BT, PT) return hash_impl<KT, BT, PT>(a, ws, ctr)
  if (!k64 && !b64 && !p64) EIGER_DISPATCH(int32_t, int32_t, int32_t);
  if (!k64 && !b64 && p64) EIGER_DISPATCH(int32_t, int32_t, int64_t);
  if (!k64 && b64 && !p64) EIGER_DISPATCH(int32_t, int64_t, int32_t);
  if (!k64 && b64 && p64) EIGER_DISPATCH(int32_t, int64_t, int64_t);
  if (k64 && !b64 && !p64) EIGER_DISPATCH(int64_t, int32_t, int32_t);
  if (k64 && !b64 && p64) EIGER_DISPATCH(int64_t, int32_t, int64_t);
  if (k64 && b64 && !p64) EIGER_DISPATCH(int64_t, int64_t, int32_t);
  EIGER_DISPATCH(int64_t, int64_t, int64_t);
#undef EIGER_DISPATCH
}

}  // namespace eiger
