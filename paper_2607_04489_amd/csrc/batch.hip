// batch.hip -- many independent joins in one hipGraph launch.
//
// All joins of a batch go through the same stages, each one persistent kernel
// over a flat list of work items (join, row range) built on the host:
//   reset     per-join state (min/max, counters, flags) and the table arena
//   minmax    min/max of every join's build keys (the statistics the per-join
//             choice needs; Section 4 of the paper: runtime statistics)
//   plan      per join: a table indexed by key - min when the key range fits the
//             join's slot budget (dense keys), else an open-addressing table
//   build     insert build rows; an open-addressing row that meets its own key on
//             the way flags a duplicate
//   unique    the joins whose build could not see duplicates: direct tables (the
//             slot must hold the row itself), and open addressing claimed by row id
//   probe     probe tiles against their join's table, materialize pairs into
//             the join's output range (first-match walks: build keys distinct)
//   radix     joins of size buckets tuned to the partitioned join run the RADIX
//             variant's own kernels (histograms, scans, scatters, LDS-table
//             join) inside the same graph, one join after another, each into
//             its own output range; a collect kernel copies their counters
// Stages never wait on each other inside a kernel, so no workgroup spins.
//
// Each XCD takes one contiguous part of the joins (equal shares of rows), so that a
// join's table is built and probed through one L2: random 16-byte reads run at 255 G/s
// from 4 MB of table and at 59 G/s from 64 MB. (A batch of 256 joins of 2^8..2^18 build
// rows 2.00 ms, 2.28 with items dealt to all XCDs; 64 joins of 2^16..2^18 2.10 and 2.32.)
// Joins whose table exceeds kSharedBytes are dealt: eight tables at a time do not fit
// the 256 MB memory-side cache, one does (eight joins of 2^20 build rows, 64-bit columns,
// 128 MiB tables: 2.75 ms, 2.91 to 3.03 in parts; 32-bit ones, 64 MiB tables: 2.17 either
// way, but with 90% of the probes on one key 1.28 in parts and 1.48 dealt).
#include <algorithm>
#include <type_traits>
#include <vector>

#include "join_common.hpp"
#include "variants.hpp"

namespace eiger {

namespace {

constexpr uint32_t kBuildTile = 2048;
constexpr int kBNT = 256;
// Pairs a probe wave stages. Sixteen waves a CU for every type would leave 312 of 8-byte
// keys and payloads (eight joins of 2^20 rows: 2.2 ms for 2.1; the narrow types gain 1%).
constexpr uint32_t kBStage = 504;
constexpr uint64_t kSharedBytes = 64ull << 20, kFarBytes = 2ull << 30;
constexpr uint32_t kVarDirect = 0, kVarHash = 1, kVarRadix = 2;

struct BatchJoinDev {
  const void *bk, *bp, *pk, *pp;
  uint64_t nR, nS;
  uint64_t out_off;  // first output position of this join
  uint64_t tab_off;  // first slot of this join's table region
  uint64_t slots;    // slots of the region (power of two)
};

struct BatchState {
  int64_t mn, mx;
  uint64_t count, checksum;
  uint32_t variant, flags;
};

struct Item {
  uint32_t join, pad;
  uint64_t lo, hi;
};

// The work items [first[x], first[x + 1]) of XCD x. Workgroup w runs on XCD
// w % kXcds (round-robin dispatch) and takes every (gridDim / kXcds)-th of them; the
// grid is a multiple of kXcds. Only the speed depends on the placement.
constexpr uint32_t kXcds = 8;
struct XcdItems {
  const Item *items;
  uint32_t first[kXcds + 1];
  __device__ __forceinline__ uint32_t begin() const { return first[blockIdx.x % kXcds] + blockIdx.x / kXcds; }
  __device__ __forceinline__ uint32_t end() const { return first[blockIdx.x % kXcds + 1]; }
  __device__ __forceinline__ uint32_t step() const { return gridDim.x / kXcds; }
};

__global__ void k_batch_reset(BatchState *__restrict__ st, int n) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  st[j].mn = INT64_MAX;
  st[j].mx = INT64_MIN;
  st[j].count = 0;
  st[j].checksum = 0;
  st[j].variant = kVarHash;
  st[j].flags = 0;
}

template <typename K>
__global__ void __launch_bounds__(256) k_batch_minmax(XcdItems items,
                                                      const BatchJoinDev *__restrict__ J, BatchState *__restrict__ st) {
  __shared__ int64_t red[2][4];
  for (uint32_t it = items.begin(); it < items.end(); it += items.step()) {
    const Item w = items.items[it];
    const K *keys = static_cast<const K *>(J[w.join].bk);
    int64_t mn = INT64_MAX, mx = INT64_MIN;
    for (uint64_t i = w.lo + threadIdx.x; i < w.hi; i += 256) {
      const int64_t k = sext(keys[i]);
      mn = k < mn ? k : mn;
      mx = k > mx ? k : mx;
    }
    mn = wave_min_i64(mn);
    mx = wave_max_i64(mx);
    if (__lane_id() == 0) {
      red[0][threadIdx.x / 64] = mn;
      red[1][threadIdx.x / 64] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int q = 1; q < 4; ++q) {
        mn = red[0][q] < mn ? red[0][q] : mn;
        mx = red[1][q] > mx ? red[1][q] : mx;
      }
      atomicMin(reinterpret_cast<long long *>(&st[w.join].mn), static_cast<long long>(mn));
      atomicMax(reinterpret_cast<long long *>(&st[w.join].mx), static_cast<long long>(mx));
    }
    __syncthreads();
  }
}

__global__ void k_batch_plan(const BatchJoinDev *__restrict__ J, BatchState *__restrict__ st, int n) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const uint64_t range = static_cast<uint64_t>(st[j].mx) - static_cast<uint64_t>(st[j].mn) + 1;
  st[j].variant = (J[j].nR > 0 && range != 0 && range <= J[j].slots) ? kVarDirect : kVarHash;
}

// Whether a join's open-addressing table is claimed by CAS on the key word: the
// cleared arena's key, -1, has to lie outside the join's key range.
__device__ __forceinline__ bool claims_keys(const BatchState &s) { return s.mn > -1 || s.mx < -1; }

// Inserts build rows, kBuildBatch of a thread loaded ahead. Direct slots are plain
// 16- or 32-byte stores (88-114 G/s against 27 G/s of atomics; k_batch_unique
// finds repeated keys). Open addressing claims the key word, so that a row that
// meets its own key has found a duplicate, or the row-id word where -1 may be a key.
constexpr int kBuildBatch = 4;
template <typename K, typename P>
__global__ void __launch_bounds__(256) k_batch_build(XcdItems items, const BatchJoinDev *__restrict__ J,
                                                     BatchState *__restrict__ st, Slot<K, P> *__restrict__ arena) {
  using W = typename std::conditional<sizeof(K) == 8, unsigned long long, unsigned int>::type;
  for (uint32_t it = items.begin(); it < items.end(); it += items.step()) {
    const Item w = items.items[it];
    const BatchJoinDev d = J[w.join];
    const K *keys = static_cast<const K *>(d.bk);
    const P *pay = static_cast<const P *>(d.bp);
    Slot<K, P> *tab = arena + d.tab_off;
    const BatchState state = st[w.join];
    const bool direct = state.variant == kVarDirect, by_key = claims_keys(state);
    const uint64_t mn = static_cast<uint64_t>(state.mn), mask = d.slots - 1;
    bool seen = false;
    for (uint64_t r0 = w.lo + threadIdx.x; r0 < w.hi; r0 += 256 * kBuildBatch) {
      K key[kBuildBatch];
      P pv[kBuildBatch];
#pragma unroll
      for (int u = 0; u < kBuildBatch; ++u) {
        const uint64_t r = r0 + u * 256;
        if (r < w.hi) {
          key[u] = keys[r];
          pv[u] = pay[r];
        }
      }
#pragma unroll
      for (int u = 0; u < kBuildBatch; ++u) {
        const uint64_t r = r0 + u * 256;
        if (r >= w.hi) continue;
        if (direct) {
          Slot<K, P> v{};
          v.key = key[u];
          v.rowid = static_cast<uint32_t>(r);
          v.pay = pv[u];
          tab[static_cast<uint64_t>(sext(key[u])) - mn] = v;  // < range <= slots
          continue;
        }
        const uint64_t home = fmix64(static_cast<uint64_t>(sext(key[u]))) & mask;
        for (uint32_t step = 0;; ++step) {  // slots >= 2 rows: an empty slot exists
          const uint64_t s = line_walk<Slot<K, P>>(home, step, mask);
          if (by_key) {
            const W old = atomicCAS(reinterpret_cast<W *>(&tab[s].key), ~W(0), static_cast<W>(key[u]));
            if (old == ~W(0)) {
              tab[s].rowid = static_cast<uint32_t>(r);
              tab[s].pay = pv[u];
              break;
            }
            seen |= old == static_cast<W>(key[u]);
          } else if (atomicCAS(&tab[s].rowid, kEmpty, static_cast<uint32_t>(r)) == kEmpty) {
            tab[s].key = key[u];
            tab[s].pay = pv[u];
            break;
          }
        }
      }
    }
    if (seen) atomicOr(&st[w.join].flags, EIGER_BATCH_DUPLICATE_BUILD);
  }
}

// Repeated build keys the build could not see. Direct: of the rows of one key
// the slot holds one, every other finds a row id that is not its own. Open
// addressing claimed by row id: every row counts its key.
template <typename K, typename P>
__global__ void __launch_bounds__(256) k_batch_unique(XcdItems items, const BatchJoinDev *__restrict__ J,
                                                      BatchState *__restrict__ st,
                                                      const Slot<K, P> *__restrict__ arena) {
  for (uint32_t it = items.begin(); it < items.end(); it += items.step()) {
    const Item w = items.items[it];
    const BatchState state = st[w.join];
    const bool direct = state.variant == kVarDirect;
    if (!direct && claims_keys(state)) continue;
    const BatchJoinDev d = J[w.join];
    const K *keys = static_cast<const K *>(d.bk);
    const Slot<K, P> *tab = arena + d.tab_off;
    const uint64_t mn = static_cast<uint64_t>(state.mn), mask = d.slots - 1;
    bool dup = false;
    for (uint64_t r = w.lo + threadIdx.x; r < w.hi; r += 256) {
      const K key = keys[r];
      if (direct) {
        dup |= tab[static_cast<uint64_t>(sext(key)) - mn].rowid != static_cast<uint32_t>(r);
        continue;
      }
      const uint64_t home = fmix64(static_cast<uint64_t>(sext(key))) & mask;
      uint32_t c = 0;
      for (uint32_t step = 0;; ++step) {
        const Slot<K, P> v = tab[line_walk<Slot<K, P>>(home, step, mask)];
        if (v.rowid == kEmpty) break;
        c += v.key == key;
      }
      dup |= c > 1;
    }
    if (dup) atomicOr(&st[w.join].flags, EIGER_BATCH_DUPLICATE_BUILD);
  }
}

template <typename K, typename P>
struct BatchDirectTab {
  static constexpr bool kWalk = false;
  static constexpr bool unique = true;
  using SlotT = Slot<K, P>;
  using Index = uint64_t;
  const Slot<K, P> *slots;
  uint64_t mn, range;
  __device__ __forceinline__ uint64_t start(K key, bool &in) const {
    const uint64_t d = static_cast<uint64_t>(sext(key)) - mn;
    in = d < range;
    return in ? d : 0;
  }
  __device__ __forceinline__ SlotT load(uint64_t i) const { return slots[i]; }
};

template <typename K, typename P>
struct BatchHashTab {
  static constexpr bool kWalk = true;
  static constexpr bool unique = true;
  using SlotT = Slot<K, P>;
  using Index = uint64_t;
  const Slot<K, P> *slots;
  uint64_t mask;
  __device__ __forceinline__ uint64_t start(K key, bool &in) const {
    in = true;
    return fmix64(static_cast<uint64_t>(sext(key))) & mask;
  }
  __device__ __forceinline__ uint64_t walk(uint64_t i, uint32_t steps) const { return line_walk<SlotT>(i, steps, mask); }
  __device__ __forceinline__ SlotT load(uint64_t i) const { return slots[i]; }
};

// An item's rows go to the workgroup's waves in turn; they write their pairs out
// together (256 joins of 2^8..2^18 build rows: 1.11 ms; 1.19 when each wave took its
// own output, for four times the atomics on a join's cursor; 1.81 with a row's walk
// held to its end by its wave). Bound by the random reads of the tables that
// exceed an XCD's L2. Tables beyond kFarBytes: one slot of a row at first (89.9M 64-bit
// build rows, an 8 GiB table, 180M probes: the batch 18.9 ms, 21.4 with two).
template <typename K, typename P>
__global__ void __launch_bounds__(kBNT) k_batch_probe(XcdItems items, const BatchJoinDev *__restrict__ J,
                                                      BatchState *__restrict__ st, const Slot<K, P> *__restrict__ arena,
                                                      uint32_t *ob, uint32_t *op) {
  __shared__ WaveLds<K, P, kBStage> L[kBNT / 64];
  __shared__ WaveJoint<kBNT / 64> joint;
  const uint32_t wave = threadIdx.x / 64;
  constexpr uint64_t block = 64 * kWaveRows, sub = kBNT * kWaveRows;
  for (uint32_t it = items.begin(); it < items.end(); it += items.step()) {
    const Item w = items.items[it];
    const BatchJoinDev d = J[w.join];
    BatchState *s = st + w.join;
    const EmitOut o{ob + d.out_off, op + d.out_off, d.nS, &s->count, &s->checksum};
    const K *pk = static_cast<const K *>(d.pk);
    const P *pp = static_cast<const P *>(d.pp);
    if (s->variant == kVarDirect) {
      const uint64_t mn = static_cast<uint64_t>(s->mn);
      const BatchDirectTab<K, P> tab{arena + d.tab_off, mn, static_cast<uint64_t>(s->mx) - mn + 1};
      WaveProbe<BatchDirectTab<K, P>, K, P, 1, kBStage> p(tab, L[wave], o);
      p.template run<kBNT / 64>(pk, pp, nullptr, w.lo + wave * block, w.hi, sub, joint);
    } else {
      const BatchHashTab<K, P> tab{arena + d.tab_off, d.slots - 1};
      if (d.slots * sizeof(Slot<K, P>) <= kFarBytes) {
        WaveProbe<BatchHashTab<K, P>, K, P, 2, kBStage> p(tab, L[wave], o);
        p.template run<kBNT / 64>(pk, pp, nullptr, w.lo + wave * block, w.hi, sub, joint);
      } else {  // two slots at first would be two address translations in flight for every row
        WaveProbe<BatchHashTab<K, P>, K, P, 1, kBStage> p(tab, L[wave], o);
        p.template run<kBNT / 64>(pk, pp, nullptr, w.lo + wave * block, w.hi, sub, joint);
      }
    }
  }
}

// Counters of a RADIX join run inside the graph -> its batch state.
__global__ void k_batch_collect(const JoinCounters *__restrict__ c, BatchState *__restrict__ st, uint64_t cap) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    st->count = c->count;
    st->checksum = c->checksum;
    st->variant = kVarRadix;
    st->flags = c->count > cap ? EIGER_BATCH_CAPACITY : 0u;
  }
}

int bucket_of_rows(int64_t n) {
  int b = 0;
  while (b < EIGER_BATCH_BUCKETS - 1 && (int64_t(2) << b) <= n) ++b;
  return b;
}

eiger_batch_tune tune_for(const eiger_batch_tune *tune, int64_t n) {
  eiger_batch_tune t{0.5f, 16384, 0};
  if (tune) {
    const eiger_batch_tune &u = tune[bucket_of_rows(n)];
    if (u.load_factor > 0.f && u.load_factor <= 0.9f) t.load_factor = u.load_factor;
    if (u.probe_tile >= 256 && u.probe_tile <= (1 << 20)) t.probe_tile = u.probe_tile;
    if (u.radix_bits >= 1 && u.radix_bits <= 16) t.radix_bits = u.radix_bits;
  }
  return t;
}

// A join of the batch that runs the RADIX variant inside the graph.
struct RadixJob {
  int32_t join;
  JoinArgs args;   // outputs and stream are filled in at capture
  size_t ws_off, ws_bytes;
};

// Work items in the order of the XCDs that take them: XCD x's are [first[x], first[x + 1]).
struct XcdList {
  std::vector<Item> items;
  uint32_t first[kXcds + 1];
};

// Host-side description of a batch (descriptors, work items, sizes).
struct BatchPlan {
  std::vector<BatchJoinDev> joins;
  XcdList build, probe;
  std::vector<RadixJob> radix;
  uint64_t arena_slots = 0, out_total = 0;
  size_t radix_ws = 0;
};

// Puts the items of a batch's joins in the XCDs' order: those of joins with tables up to
// kSharedBytes in one contiguous part per XCD, of equal rows, the others dealt to all.
void order_items(XcdList &l, const std::vector<BatchJoinDev> &joins, size_t slot) {
  std::vector<Item> own, shared;
  uint64_t total = 0, run = 0;
  for (const Item &i : l.items) {
    const bool big = joins[i.join].slots * slot > kSharedBytes;
    (big ? shared : own).push_back(i);
    if (!big) total += i.hi - i.lo;
  }
  l.items.clear();
  size_t at = 0;
  for (uint32_t k = 0; k < kXcds; ++k) {
    l.first[k] = static_cast<uint32_t>(l.items.size());
    const uint64_t upto = total / kXcds * (k + 1) + total % kXcds * (k + 1) / kXcds;
    while (at < own.size() && run < upto) run += own[at].hi - own[at].lo, l.items.push_back(own[at++]);
    for (size_t i = k; i < shared.size(); i += kXcds) l.items.push_back(shared[i]);
  }
  l.first[kXcds] = static_cast<uint32_t>(l.items.size());
}

int plan_batch(const eiger_batch_join *joins, int32_t n, int32_t kdt, int32_t pdt, const eiger_batch_tune *tune,
               BatchPlan *bp) {
  if (!joins || n <= 0) return fail(EIGER_ERR_INVALID_ARG, "batch: no joins");
  if ((kdt != EIGER_INT32 && kdt != EIGER_INT64) || (pdt != EIGER_INT32 && pdt != EIGER_INT64))
    return fail(EIGER_ERR_DTYPE, "batch: dtypes must be EIGER_INT32 or EIGER_INT64");
  bp->joins.resize(n);
  for (int32_t j = 0; j < n; ++j) {
    const eiger_batch_join &q = joins[j];
    if (q.n_build < 0 || q.n_probe < 0) return fail(EIGER_ERR_INVALID_ARG, "batch: negative row count");
    if (q.n_build > EIGER_MAX_ROWS || q.n_probe > EIGER_MAX_ROWS)
      return fail(EIGER_ERR_TOO_LARGE, "batch: a join side has more than EIGER_MAX_ROWS = 2^32 - 2^16 rows");
    if ((q.n_build > 0 && (!q.build_keys || !q.build_payload)) || (q.n_probe > 0 && (!q.probe_keys || !q.probe_payload)))
      return fail(EIGER_ERR_INVALID_ARG, "batch: NULL column of a non-empty side");
    const size_t ks = dtype_size(kdt), ps = dtype_size(pdt);
    if (reinterpret_cast<uintptr_t>(q.build_keys) % ks || reinterpret_cast<uintptr_t>(q.probe_keys) % ks ||
        reinterpret_cast<uintptr_t>(q.build_payload) % ps || reinterpret_cast<uintptr_t>(q.probe_payload) % ps)
      return fail(EIGER_ERR_INVALID_ARG, "batch: column not aligned to its dtype");
    const eiger_batch_tune t = tune_for(tune, q.n_build);
    if (t.radix_bits > 0 && q.n_build > 0 && q.n_probe > 0) {
      BatchJoinDev &d = bp->joins[j];
      d = BatchJoinDev{q.build_keys, q.build_payload, q.probe_keys, q.probe_payload, uint64_t(q.n_build),
                       uint64_t(q.n_probe), bp->out_total, bp->arena_slots, 0};
      RadixJob job{};
      job.join = j;
      JoinArgs &a = job.args;
      a.bk = q.build_keys;
      a.bp = q.build_payload;
      a.pk = q.probe_keys;
      a.pp = q.probe_payload;
      a.nR = uint64_t(q.n_build);
      a.nS = uint64_t(q.n_probe);
      a.kdt = kdt;
      a.bpdt = pdt;
      a.ppdt = pdt;
      a.plan = eiger_plan_t{};
      a.plan.variant = EIGER_RADIX;
      a.plan.key_dtype = kdt;
      a.plan.radix_bits = t.radix_bits;
      a.plan.radix_passes = t.radix_bits > 8 ? 2 : 1;
      a.plan.load_factor = t.load_factor;
      a.cap = uint64_t(q.n_probe);
      Workspace dry(nullptr, 0);
      JoinCounters *unused = nullptr;
      if (int rc = run_join_variant(a, dry, &unused)) return rc;
      // the partitioned joins run one after another on the graph's stream, so
      // they share one workspace region sized for the largest
      job.ws_off = 0;
      job.ws_bytes = dry.used + 256;
      bp->radix_ws = std::max(bp->radix_ws, (job.ws_bytes + 255) & ~size_t(255));
      bp->radix.push_back(job);
      bp->out_total += uint64_t(q.n_probe);
      continue;
    }
    uint64_t slots = 64;
    const double want = static_cast<double>(q.n_build) / t.load_factor + 1.0;
    while (static_cast<double>(slots) < want) slots <<= 1;
    if (slots < 2 * static_cast<uint64_t>(q.n_build)) slots <<= 1;  // >= 2 rows per... keep an empty slot
    BatchJoinDev &d = bp->joins[j];
    d = BatchJoinDev{q.build_keys, q.build_payload, q.probe_keys, q.probe_payload, uint64_t(q.n_build),
                     uint64_t(q.n_probe), bp->out_total, bp->arena_slots, slots};
    bp->out_total += uint64_t(q.n_probe);
    bp->arena_slots += slots;
    for (uint64_t lo = 0; lo < uint64_t(q.n_build); lo += kBuildTile)
      bp->build.items.push_back(Item{uint32_t(j), 0, lo, std::min<uint64_t>(q.n_build, lo + kBuildTile)});
    if (q.n_build > 0)
      for (uint64_t lo = 0; lo < uint64_t(q.n_probe); lo += uint64_t(t.probe_tile))
        bp->probe.items.push_back(Item{uint32_t(j), 0, lo, std::min<uint64_t>(q.n_probe, lo + t.probe_tile)});
  }
  if (bp->build.items.size() >= (1ull << 32) || bp->probe.items.size() >= (1ull << 32))
    return fail(EIGER_ERR_TOO_LARGE, "batch: too many work items");
  order_items(bp->build, bp->joins, slot_bytes(kdt, pdt));
  order_items(bp->probe, bp->joins, slot_bytes(kdt, pdt));
  return EIGER_OK;
}

struct BatchLayout {
  BatchJoinDev *joins;
  BatchState *state;
  Item *build, *probe;
  void *arena;
  char *radix_ws;
};

BatchLayout batch_layout(Workspace &ws, const BatchPlan &bp, size_t slot_bytes_) {
  BatchLayout L;
  L.joins = ws.take<BatchJoinDev>(bp.joins.size());
  L.state = ws.take<BatchState>(bp.joins.size());
  L.build = ws.take<Item>(std::max<size_t>(bp.build.items.size(), 1));
  L.probe = ws.take<Item>(std::max<size_t>(bp.probe.items.size(), 1));
  L.arena = ws.take<char>(bp.arena_slots * slot_bytes_);
  L.radix_ws = ws.take<char>(bp.radix_ws);
  return L;
}

struct BatchHandle {
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  int n = 0;
  BatchState *state = nullptr;
};

XcdItems xcd_items(const XcdList &l, const Item *dev) {
  XcdItems x{};
  x.items = dev;
  std::copy(l.first, l.first + kXcds + 1, x.first);
  return x;
}

// Grid over n work items: per_cu workgroups per CU at most, a multiple of kXcds.
unsigned xcd_grid(unsigned n, unsigned cus, unsigned per_cu) {
  return std::min((n + kXcds - 1) / kXcds * kXcds, std::max(cus / kXcds, 1u) * kXcds * per_cu);
}

template <typename K, typename P>
int enqueue_batch(const BatchPlan &bp, const BatchLayout &L, uint32_t *ob, uint32_t *op, hipStream_t s) {
  const int n = static_cast<int>(bp.joins.size());
  const unsigned nb = static_cast<unsigned>(bp.build.items.size()), np = static_cast<unsigned>(bp.probe.items.size());
  const unsigned cus = static_cast<unsigned>(device_cu_count());
  const XcdItems bi = xcd_items(bp.build, L.build), pi = xcd_items(bp.probe, L.probe);
  int rc;
  EIGER_LAUNCH("batch_reset", k_batch_reset, dim3((n + 255) / 256), dim3(256), 0, s, L.state, n);
  if ((rc = fill_u32(static_cast<uint32_t *>(L.arena), bp.arena_slots * sizeof(Slot<K, P>) / 4, kEmpty, s))) return rc;
  if (nb) {
    EIGER_LAUNCH("batch_minmax", k_batch_minmax<K>, dim3(xcd_grid(nb, cus, 8)), dim3(256), 0, s, bi, L.joins,
                 L.state);
  }
  EIGER_LAUNCH("batch_plan", k_batch_plan, dim3((n + 255) / 256), dim3(256), 0, s, L.joins, L.state, n);
  if (nb) {
    Slot<K, P> *arena = static_cast<Slot<K, P> *>(L.arena);
    EIGER_LAUNCH("batch_build", (k_batch_build<K, P>), dim3(xcd_grid(nb, cus, 8)), dim3(256), 0, s, bi, L.joins,
                 L.state, arena);
    EIGER_LAUNCH("batch_unique", (k_batch_unique<K, P>), dim3(xcd_grid(nb, cus, 8)), dim3(256), 0, s, bi, L.joins,
                 L.state, arena);
  }
  if (np) {
    EIGER_LAUNCH("batch_probe", (k_batch_probe<K, P>), dim3(xcd_grid(np, cus, static_cast<unsigned>(163840 / (sizeof(WaveLds<K, P, kBStage>) * (kBNT / 64))))), dim3(kBNT), 0, s,
                 pi, L.joins, L.state, static_cast<const Slot<K, P> *>(L.arena), ob, op);
  }
  for (const RadixJob &job : bp.radix) {
    JoinArgs a = job.args;
    const uint64_t off = bp.joins[job.join].out_off;
    a.ob = ob + off;
    a.op = op + off;
    a.s = s;
    Workspace w(L.radix_ws + job.ws_off, job.ws_bytes);
    JoinCounters *c = nullptr;
    if ((rc = run_join_variant(a, w, &c))) return rc;
    EIGER_LAUNCH("batch_collect", k_batch_collect, dim3(1), dim3(64), 0, s, c, L.state + job.join, a.cap);
  }
  return EIGER_OK;
}

size_t batch_slot_bytes(int32_t kdt, int32_t pdt) { return slot_bytes(kdt, pdt); }

}  // namespace

}  // namespace eiger

using namespace eiger;

extern "C" int eiger_join_batch_workspace_size(const eiger_batch_join *joins, int32_t n_joins, int32_t key_dtype,
                                               int32_t payload_dtype, const eiger_batch_tune *tune, size_t *bytes) {
  if (!bytes) return fail(EIGER_ERR_INVALID_ARG, "batch: bytes is NULL");
  BatchPlan bp;
  int rc = plan_batch(joins, n_joins, key_dtype, payload_dtype, tune, &bp);
  if (rc) return rc;
  Workspace ws(nullptr, 0);
  batch_layout(ws, bp, batch_slot_bytes(key_dtype, payload_dtype));
  *bytes = ws.used;
  return EIGER_OK;
}

extern "C" int eiger_join_batch_create(const eiger_batch_join *joins, int32_t n_joins, int32_t key_dtype,
                                       int32_t payload_dtype, const eiger_batch_tune *tune, uint32_t *out_build_rowid,
                                       uint32_t *out_probe_rowid, void *ws_ptr, size_t ws_bytes, void *stream,
                                       void **handle) {
  if (!handle) return fail(EIGER_ERR_INVALID_ARG, "batch: handle is NULL");
  *handle = nullptr;
  BatchPlan bp;
  int rc = plan_batch(joins, n_joins, key_dtype, payload_dtype, tune, &bp);
  if (rc) return rc;
  if (bp.out_total > 0 && (!out_build_rowid || !out_probe_rowid))
    return fail(EIGER_ERR_INVALID_ARG, "batch: NULL output arrays");
  Workspace ws(ws_ptr, ws_bytes);
  BatchLayout L = batch_layout(ws, bp, batch_slot_bytes(key_dtype, payload_dtype));
  if (!ws_ptr || ws.used > ws_bytes)
    return fail(EIGER_ERR_WORKSPACE, "batch: workspace too small (need " + std::to_string(ws.used) + " bytes)");
  hipStream_t s = static_cast<hipStream_t>(stream);
  // descriptors and work items, copied once (outside the graph)
  EIGER_HIP(hipMemcpyAsync(L.joins, bp.joins.data(), bp.joins.size() * sizeof(BatchJoinDev), hipMemcpyHostToDevice, s));
  for (const auto &[list, dev] : {std::pair<const XcdList &, Item *>(bp.build, L.build), {bp.probe, L.probe}})
    if (!list.items.empty())
      EIGER_HIP(hipMemcpyAsync(dev, list.items.data(), list.items.size() * sizeof(Item), hipMemcpyHostToDevice, s));
  EIGER_HIP(hipStreamSynchronize(s));
  auto *h = new BatchHandle();
  h->n = n_joins;
  h->state = L.state;
  // The caller's stream may be the legacy default stream, which cannot be
  // captured: record the graph on a private stream (default priority).
  hipStream_t cs = nullptr;
  hipError_t e = hipStreamCreateWithFlags(&cs, hipStreamNonBlocking);
  if (e != hipSuccess) {
    delete h;
    return hip_fail(e, "hipStreamCreateWithFlags");
  }
  e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) {
    (void)hipStreamDestroy(cs);
    delete h;
    return hip_fail(e, "hipStreamBeginCapture");
  }
  const bool k64 = key_dtype == EIGER_INT64, p64 = payload_dtype == EIGER_INT64;
  if (!k64 && !p64) rc = enqueue_batch<int32_t, int32_t>(bp, L, out_build_rowid, out_probe_rowid, cs);
  else if (!k64 && p64) rc = enqueue_batch<int32_t, int64_t>(bp, L, out_build_rowid, out_probe_rowid, cs);
  else if (k64 && !p64) rc = enqueue_batch<int64_t, int32_t>(bp, L, out_build_rowid, out_probe_rowid, cs);
  else rc = enqueue_batch<int64_t, int64_t>(bp, L, out_build_rowid, out_probe_rowid, cs);
  hipGraph_t g = nullptr;
  e = hipStreamEndCapture(cs, &g);
  (void)hipStreamDestroy(cs);
  if (rc || e != hipSuccess) {
    if (g) (void)hipGraphDestroy(g);
    delete h;
    return rc ? rc : hip_fail(e, "hipStreamEndCapture");
  }
  h->graph = g;
  e = hipGraphInstantiate(&h->exec, g, nullptr, nullptr, 0);
  if (e != hipSuccess) {
    (void)hipGraphDestroy(g);
    delete h;
    return hip_fail(e, "hipGraphInstantiate");
  }
  *handle = h;
  return EIGER_OK;
}

extern "C" int eiger_join_batch_launch(void *handle, void *stream) {
  if (!handle) return fail(EIGER_ERR_INVALID_ARG, "batch: handle is NULL");
  auto *h = static_cast<BatchHandle *>(handle);
  EIGER_HIP(hipGraphLaunch(h->exec, static_cast<hipStream_t>(stream)));
  return EIGER_OK;
}

extern "C" int eiger_join_batch_results(void *handle, int64_t *counts, int64_t *checksums, int32_t *variants,
                                        uint32_t *flags, void *stream) {
  if (!handle) return fail(EIGER_ERR_INVALID_ARG, "batch: handle is NULL");
  auto *h = static_cast<BatchHandle *>(handle);
  hipStream_t s = static_cast<hipStream_t>(stream);
  std::vector<BatchState> st(h->n);
  EIGER_HIP(hipMemcpyAsync(st.data(), h->state, sizeof(BatchState) * h->n, hipMemcpyDeviceToHost, s));
  EIGER_HIP(hipStreamSynchronize(s));
  for (int j = 0; j < h->n; ++j) {
    if (counts) counts[j] = static_cast<int64_t>(st[j].count);
    if (checksums) checksums[j] = static_cast<int64_t>(st[j].checksum);
    if (variants)
      variants[j] = st[j].variant == kVarDirect ? EIGER_DIRECT
                    : st[j].variant == kVarRadix ? EIGER_RADIX
                                                 : EIGER_GLOBAL_HASH;
    if (flags) flags[j] = st[j].flags;
  }
  return EIGER_OK;
}

extern "C" int eiger_join_batch_destroy(void *handle) {
  if (!handle) return EIGER_OK;
  auto *h = static_cast<BatchHandle *>(handle);
  if (h->exec) (void)hipGraphExecDestroy(h->exec);
  if (h->graph) (void)hipGraphDestroy(h->graph);
  delete h;
  return EIGER_OK;
}
