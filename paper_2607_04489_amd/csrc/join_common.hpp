// join_common.hpp -- output materialization shared by the join variants.
//
// Every variant probes tiles of NT * IPT probe rows. A probe row may match any
// number of build rows. Matches are compacted per workgroup with a block-wide
// exclusive scan of per-thread match counts and staged in LDS; a full stage is
// flushed with ONE atomic add on the global output cursor and written out with
// consecutive threads on consecutive addresses. The payload aggregate uses
// distributivity mod 2^64: a probe row adds probe_payload * (sum of the payloads
// of its matching build rows).
#pragma once

#include "common.hpp"
#include "variants.hpp"

namespace eiger {

// Slot of a hash table in device memory: key, build row id and build payload
// side by side, 16 bytes (32 when key and payload are both 8 bytes), so one
// probe step is one aligned vector load. rowid == kEmpty marks an empty slot.
template <typename K, typename P>
struct alignas((sizeof(K) + sizeof(P) + 4 <= 16) ? 16 : 32) Slot {
  K key;
  uint32_t rowid;
  P pay;
};

// Probe sequence of the open-addressing tables in device memory (power-of-two
// slots): the slots of the home slot's 64 bytes, wrapping inside them, then the
// next 64 bytes', and so on, so that the second slot costs no second memory access
// (2^28 probes of a 2 GiB table of 32-byte slots, two slots a step: 5.78 ms; in
// 128-byte groups 6.09; first slot and then plain linear probing 6.12).
template <typename SlotT>
__device__ __forceinline__ uint64_t line_walk(uint64_t home, uint32_t steps, uint64_t mask) {
  constexpr uint64_t per = 64 / sizeof(SlotT);
  return (((home | (per - 1)) + 1 - per + (steps & ~uint32_t(per - 1))) & mask) | ((home + steps) & (per - 1));
}

// Where pairs go. ob/op may be null (count-only); positions >= cap are dropped.
struct EmitOut {
  uint32_t *ob;
  uint32_t *op;
  uint64_t cap;
  uint64_t *cursor;    // device u64, zero before the first launch
  uint64_t *checksum;  // device u64, zero before the first launch
  JoinStripe *stripes = nullptr;  // kStripes of them, or null: take cursor and checksum alone
};

template <int NT, int SCAP>
struct EmitLds {
  uint32_t b[SCAP];
  uint32_t p[SCAP];
  uint64_t scan[NT / 64 + 1];
  uint64_t base;
  uint64_t red[NT / 64];
};

__device__ __forceinline__ void put_pair(const EmitOut &o, uint64_t pos, uint32_t b, uint32_t p) {
  if (o.ob && pos < o.cap) {
    o.ob[pos] = b;
    o.op[pos] = p;
  }
}

// Reserve `count` output slots for the whole workgroup; all threads get the base.
template <int NT, int SCAP>
__device__ __forceinline__ uint64_t reserve(EmitLds<NT, SCAP> &L, const EmitOut &o, uint64_t count) {
  if (threadIdx.x == 0) L.base = atomicAdd(reinterpret_cast<unsigned long long *>(o.cursor),
                                           static_cast<unsigned long long>(count));
  __syncthreads();
  const uint64_t base = L.base;
  __syncthreads();
  return base;
}

// Write the staged pairs [0, fill) to the output. Uniform across the workgroup.
template <int NT, int SCAP>
__device__ __forceinline__ void flush(EmitLds<NT, SCAP> &L, const EmitOut &o, uint32_t fill) {
  if (fill == 0) return;
  const uint64_t base = reserve(L, o, fill);
  if (o.ob) {
    for (uint32_t i = threadIdx.x; i < fill; i += NT) put_pair(o, base + i, L.b[i], L.p[i]);
  }
  __syncthreads();
}

// block_exclusive_scan for the emission, whose callers keep whole sub-tiles of rows in
// their registers: the waves' totals are not held in vector registers as well. Four
// waves: in scalar ones (with the totals in vector registers k_probe<DirectTab> took 130
// to 140 of the 128 that its four workgroups a CU leave, and the fourth ran alone: 2^26
// sorted probes of 2^23 dense int32 keys, pairs: 0.87 ms of probe for 0.51). Eight: one
// thread adds them up in LDS, as their scalars spill (k_radix_join, 67M x 268M skewed
// int32 rows: 5.15 ms; 5.26 in scalar registers, 5.20 in vector ones). `scratch` holds
// NT / 64 + 1 words.
template <int NT>
__device__ __forceinline__ uint64_t emit_scan(uint64_t v, uint64_t *scratch, uint64_t *total) {
  constexpr int NW = NT / 64;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / 64);
  const uint64_t inc = wave_inclusive_scan<uint64_t>(v);
  if (__lane_id() == 63) scratch[wave] = inc;
  __syncthreads();
  uint64_t before = 0, all = 0;
  if constexpr (NW <= 4) {
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const uint64_t lds = scratch[w];
      const uint64_t t = (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(static_cast<int>(lds >> 32)))) << 32) |
                         uint32_t(__builtin_amdgcn_readfirstlane(static_cast<int>(lds)));
      before += w < wave ? t : 0;
      all += t;
    }
  } else {
    if (threadIdx.x == 0) {
      for (int w = 0; w < NW; ++w) {
        const uint64_t t = scratch[w];
        scratch[w] = all;
        all += t;
      }
      scratch[NW] = all;
    }
    __syncthreads();
    before = scratch[wave];
    all = scratch[NW];
  }
  *total = all;
  __syncthreads();
  return before + inc - v;
}

// Finish a workgroup's share: flush the stage and add its checksum part. In
// count-only mode `fill` is instead the workgroup's whole pair count (uniform).
template <int NT, int SCAP>
__device__ __forceinline__ void finish(EmitLds<NT, SCAP> &L, const EmitOut &o, uint64_t fill,
                                       uint64_t cs) {
  if (o.ob) {
    flush(L, o, static_cast<uint32_t>(fill));
  } else if (threadIdx.x == 0 && fill) {
    atomicAdd(reinterpret_cast<unsigned long long *>(o.cursor), static_cast<unsigned long long>(fill));
  }
  const uint64_t s = block_sum_u64<NT>(cs, L.red);
  if (threadIdx.x == 0 && s != 0)
    atomicAdd(reinterpret_cast<unsigned long long *>(o.checksum), static_cast<unsigned long long>(s));
}

// ---- wave probes of tables in device memory ----------------------------------
//
// A wave probes on its own. Rows are taken 64 * kWaveRows at a time, their first
// kEager slots loaded at once. Rows whose walk goes on are packed into a queue in
// LDS, and as soon as it holds a full wave of them the next slots of up to
// 64 * kWaveQueued rows are loaded, two at a time. So every round trip carries full
// waves; when a wave walked its rows until the last one ended, it made 8 to 10 for rows
// that need 1.5 on average. A match is staged the moment it is found. Bound by random
// accesses: 255 G/s of them from a table in an XCD's L2, 55-59 G/s from a larger one.
//
// Probes that find their slots in the L1 (sorted ones, one key) are bound by what comes
// between the loads instead: the stage is written out by the whole workgroup, so it
// holds more than one block's matches, and a queue of one wave's rows, not of two,
// leaves the LDS for that and for more waves (2^23 sorted probes of 60,000 int32 keys,
// int64 payloads: 140 us; with stages of 504 pairs, 12 waves a CU and queues of 384
// rows 199; probes in random order 165 and 216).
constexpr int kWaveRows = 4;     // rows a lane takes from the input together
constexpr int kWaveQueued = 2;   // rows a lane takes from the queue together
constexpr uint32_t kWaveFull = 64;  // queued rows that are not left for later
constexpr uint32_t kWaveQueue = 64 * kWaveRows + kWaveFull;
// Pairs that each wave can stage when `waves` of them share a CU's LDS (160 KB, of
// which 1 KB is left for what the workgroups share).
template <typename K, typename PS>
constexpr uint32_t wave_stage(uint32_t waves) {
  return ((163840 - 1024) / waves - kWaveQueue * (sizeof(K) + sizeof(PS) + 8)) / 16 * 2;
}

template <typename K, typename PS, uint32_t kStage>
struct WaveLds {
  static_assert(kStage == 0 || (kStage >= 64 * kWaveRows && kStage >= 64 * 2 * kWaveQueued),
                "a step's matches fit an empty stage");
  K key[kWaveQueue];
  PS pay[kWaveQueue];
  uint32_t row[kWaveQueue], step[kWaveQueue];
  uint32_t ob[kStage ? kStage : 1], op[kStage ? kStage : 1];
};

// What the waves of a workgroup share to write their stages out together; two
// copies, used in turn.
template <int NW>
struct WaveJoint {
  uint64_t base[2];
  uint32_t fill[2][NW];  // bit 31: the wave has more to do
  uint64_t sum[NW], count[NW];
};

// Orders this wave's LDS accesses for the compiler (the hardware keeps a wave's
// LDS operations in order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Tab: SlotT, Index; start(key, in) -> first slot (in: false when the key cannot be
// there), walk(first, steps) -> the slot `steps` further, load(slot); kWalk: keys may
// lie further on; unique: build keys known to be distinct. kStage: pairs staged
// before they are written out (o.ob, o.op given); 0: matches are counted only.
template <class Tab, typename K, typename PS, int kEager, uint32_t kStage>
struct WaveProbe {
  static constexpr bool kPairs = kStage > 0;
  static_assert(kEager == 1 || kEager == 2, "one or two slots at first");
  const Tab &tab;
  WaveLds<K, PS, kStage> &L;
  const EmitOut &o;
  uint64_t fill = 0;    // staged pairs, or all pairs counted (uniform)
  uint32_t queued = 0;  // uniform
  uint64_t cs = 0;      // this lane's share of the checksum

  __device__ __forceinline__ WaveProbe(const Tab &t, WaveLds<K, PS, kStage> &l, const EmitOut &e) : tab(t), L(l), o(e) {}

  // The staged pairs to output positions base, base + 1, ...
  __device__ __forceinline__ void write_out(uint64_t base) {
    wave_lds_fence();
    for (uint32_t i = __lane_id(); i < static_cast<uint32_t>(fill); i += 64) put_pair(o, base + i, L.ob[i], L.op[i]);
    wave_lds_fence();
    fill = 0;
  }

  // Whether the stage takes R more matches a lane.
  __device__ __forceinline__ bool room(int R) const { return !kPairs || fill + 64 * R <= kStage; }

  // Whether the second slot of rows already looked at once can be looked at before the
  // stage is written out: distinct build keys match once in all their slots, so that
  // there is room; others may match in each.
  __device__ __forceinline__ bool second(int R) const { return tab.unique || room(R); }

  // The next slot of R rows a lane: matches are staged; live: the walks that go on.
  template <int R>
  __device__ __forceinline__ void visit(const K (&key)[R], const PS (&pay)[R], const uint32_t (&row)[R], bool (&live)[R],
                                        const typename Tab::SlotT (&sl)[R]) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      live[r] = live[r] && sl[r].rowid != kEmpty;
      const bool hit = live[r] && sl[r].key == key[r];
      if (hit) cs += static_cast<uint64_t>(sext(sl[r].pay)) * static_cast<uint64_t>(sext(pay[r]));
      const uint64_t hits = __ballot(hit);
      if (kPairs && hit) {
        const uint32_t at = static_cast<uint32_t>(fill) + lane_prefix(hits);
        L.ob[at] = sl[r].rowid;
        L.op[at] = row[r];
      }
      fill += __popcll(hits);
      live[r] = live[r] && !(hit && tab.unique);
    }
  }

  // Queues the rows whose walk goes on, `step` slots from their first.
  template <int R>
  __device__ __forceinline__ void enqueue(const K (&key)[R], const PS (&pay)[R], const uint32_t (&row)[R],
                                          const uint32_t (&step)[R], const bool (&live)[R]) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint64_t ons = __ballot(live[r]);
      if (live[r]) {
        const uint32_t at = queued + lane_prefix(ons);
        L.key[at] = key[r];
        L.pay[at] = pay[r];
        L.row[at] = row[r];
        L.step[at] = step[r];
      }
      queued += static_cast<uint32_t>(__popcll(ons));
    }
    wave_lds_fence();
  }

  // The next slots of the last n queued rows (n <= 64 * kWaveQueued, n <= queued): two
  // or, without room for the second's matches, one. Walks among repeated keys are long
  // and stay here while most of them go on.
  __device__ __forceinline__ void advance(uint32_t n) {
    K key[kWaveQueued];
    PS pay[kWaveQueued];
    uint32_t row[kWaveQueued], step[kWaveQueued];
    bool live[kWaveQueued];
    typename Tab::Index home[kWaveQueued];
    typename Tab::SlotT s0[kWaveQueued], s1[kWaveQueued];
    queued -= n;
#pragma unroll
    for (int r = 0; r < kWaveQueued; ++r) {
      const uint32_t i = r * 64 + __lane_id();
      live[r] = i < n;
      const uint32_t e = queued + (live[r] ? i : 0);
      key[r] = L.key[e];
      pay[r] = L.pay[e];
      row[r] = L.row[e];
      step[r] = L.step[e];
      bool in;
      home[r] = tab.start(key[r], in);
    }
    for (;;) {
#pragma unroll
      for (int r = 0; r < kWaveQueued; ++r) {
        s0[r] = tab.load(tab.walk(home[r], step[r]));
        s1[r] = tab.load(tab.walk(home[r], step[r] + 1));
      }
      wave_lds_fence();
      visit<kWaveQueued>(key, pay, row, live, s0);
      const bool both = second(kWaveQueued);
      if (both) visit<kWaveQueued>(key, pay, row, live, s1);
#pragma unroll
      for (int r = 0; r < kWaveQueued; ++r) step[r] += both ? 2 : 1;
      if (tab.unique || !room(kWaveQueued)) break;
      uint32_t on = 0;
#pragma unroll
      for (int r = 0; r < kWaveQueued; ++r) on += static_cast<uint32_t>(__popcll(__ballot(live[r])));
      if (4 * on < 3 * n) break;
    }
    enqueue<kWaveQueued>(key, pay, row, step, live);
  }

  // Probe rows [lo, hi) in blocks of 64 * kWaveRows rows, `stride` rows apart,
  // until every match is written out; a block's columns are loaded while the one
  // before is probed. The waves of the workgroup (all NW call this) write their stages
  // out together whenever one is full, for one atomic: atomics on one cursor run at
  // 10 ns each (2^27 probes, 121M matches: 3.2 ms of them with 380 pairs each).
  template <int NW>
  __device__ __forceinline__ void run(const K *__restrict__ pk, const PS *__restrict__ pp,
                                      const uint32_t *__restrict__ prow, uint64_t lo, uint64_t hi, uint64_t stride,
                                      WaveJoint<NW> &J, uint32_t block = 64 * kWaveRows) {
    K key[kWaveRows], nkey[kWaveRows];
    PS pay[kWaveRows], npay[kWaveRows];
    uint32_t row[kWaveRows], nrow[kWaveRows], step[kWaveRows];
    auto end_of = [&](uint64_t t) { return block < 64 * kWaveRows && t + block < hi ? t + block : hi; };
    auto load = [&](uint64_t t) {
      const uint64_t e = end_of(t);
#pragma unroll
      for (int r = 0; r < kWaveRows; ++r) {
        const uint64_t j = t + r * 64 + __lane_id(), i = j < e ? j : e - 1;
        nkey[r] = pk[i];
        npay[r] = pp[i];
        nrow[r] = prow ? prow[i] : static_cast<uint32_t>(i);
      }
    };
    uint64_t t = lo;
    if (t < hi) load(t);
    for (uint32_t round = 0;; ++round) {
      for (;;) {
        if (Tab::kWalk && (queued >= kWaveFull || (t >= hi && queued))) {
          if (!room(kWaveQueued)) break;
          if constexpr (Tab::kWalk) advance(queued < 64 * kWaveQueued ? queued : 64 * kWaveQueued);
        } else if (t < hi) {
          if (!room(kWaveRows)) break;
          bool live[kWaveRows];
          typename Tab::Index home[kWaveRows];
          typename Tab::SlotT s0[kWaveRows], s1[kWaveRows];
          const uint64_t e = end_of(t);
#pragma unroll
          for (int r = 0; r < kWaveRows; ++r) {
            key[r] = nkey[r];
            pay[r] = npay[r];
            row[r] = nrow[r];
            step[r] = kEager;
            bool in;
            home[r] = tab.start(key[r], in);
            live[r] = in && t + r * 64 + __lane_id() < e;
            s0[r] = tab.load(home[r]);
            if constexpr (Tab::kWalk && kEager > 1) s1[r] = tab.load(tab.walk(home[r], 1));
          }
          t += stride;
          if (t < hi) load(t);
          visit<kWaveRows>(key, pay, row, live, s0);
          if constexpr (Tab::kWalk) {
            if constexpr (kEager > 1) {
              if (second(kWaveRows)) {
                visit<kWaveRows>(key, pay, row, live, s1);
              } else {
#pragma unroll
                for (int r = 0; r < kWaveRows; ++r) step[r] = 1;
              }
            }
            enqueue<kWaveRows>(key, pay, row, step, live);
          } else {
            wave_lds_fence();
          }
        } else {
          break;
        }
      }
      bool done = t >= hi && queued == 0;  // nothing left but the stage
      if constexpr (!kPairs) break;
      const uint32_t w = threadIdx.x / 64, par = round & 1;
      if (__lane_id() == 0) J.fill[par][w] = static_cast<uint32_t>(fill) | (done ? 0u : 1u << 31);
      __syncthreads();
      uint32_t total = 0, before = 0, busy = 0;
#pragma unroll
      for (uint32_t x = 0; x < NW; ++x) {
        const uint32_t f = J.fill[par][x];
        before += x < w ? f & 0x7FFFFFFFu : 0u;
        total += f & 0x7FFFFFFFu;
        busy |= f >> 31;
      }
      if (threadIdx.x == 0 && total)
        J.base[par] = atomicAdd(reinterpret_cast<unsigned long long *>(o.cursor), static_cast<unsigned long long>(total));
      __syncthreads();
      write_out(J.base[par] + before);
      done = !busy;
      if (done) break;
    }
    // totals: the workgroup's in one atomic each
    uint64_t sum = wave_sum_u64(cs), count = kPairs ? 0 : fill;
    if (__lane_id() == 0) {
      J.sum[threadIdx.x / 64] = sum;
      J.count[threadIdx.x / 64] = count;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    sum = count = 0;
    for (int x = 0; x < NW; ++x) {
      sum += J.sum[x];
      count += J.count[x];
    }
    uint64_t *to_sum = o.checksum, *to_count = o.cursor;
    if (o.stripes) {
      to_sum = &o.stripes[blockIdx.x % kStripes].checksum;
      to_count = &o.stripes[blockIdx.x % kStripes].count;
    }
    if (sum) atomicAdd(reinterpret_cast<unsigned long long *>(to_sum), static_cast<unsigned long long>(sum));
    if (count) atomicAdd(reinterpret_cast<unsigned long long *>(to_count), static_cast<unsigned long long>(count));
  }
};

// Registers of one probe sub-tile: up to IPT rows per thread, rows
// lo + k * NT + threadIdx.x. (Holding the next sub-tile in registers as well
// was measured slower on gfx950: the extra registers cost more occupancy than
// the overlap gained.)
template <int IPT, typename K, typename PS>
struct ProbeRegs {
  K key[IPT];
  PS pay[IPT];
  uint32_t rid[IPT];
  uint64_t lo, hi;
};

template <int NT, int IPT, typename K, typename PS>
__device__ __forceinline__ void probe_load(ProbeRegs<IPT, K, PS> &r, const K *__restrict__ pk,
                                           const PS *__restrict__ pp,
                                           const uint32_t *__restrict__ prow, uint64_t lo,
                                           uint64_t hi) {
  r.lo = lo;
  r.hi = hi;
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const uint64_t i = lo + uint64_t(k) * NT + threadIdx.x;
    if (i < hi) {
      r.key[k] = pk[i];
      r.pay[k] = pp[i];
      r.rid[k] = prow ? prow[i] : static_cast<uint32_t>(i);
    }
  }
}

// Count the matches of every loaded row. Tables of two kinds:
//  * hashed tables (Tab::kHashed) expose an index type Index, home(key),
//    next(i, step) (from a walk's slot i to its step-th), load(i) -> slot and a `unique` flag (build keys known to be
//    distinct). The first slot of
//    every row is loaded before any is inspected, so a thread keeps IPT random
//    loads in flight; only rows whose walk is not finished load again, and a
//    unique table stops a walk at its first match.
//  * other tables expose lookup(key, first, payload_sum) -> count, where
//    `first` is the first match's row id, or with Tab::kRuns the start of the
//    key's contiguous run of rows (emit_matches).
template <int NT, int IPT, class Tab, typename K, typename PS>
__device__ __forceinline__ void count_matches(const Tab &tab, const ProbeRegs<IPT, K, PS> &r,
                                              uint32_t (&cnt)[IPT], uint32_t (&first)[IPT],
                                              uint64_t (&psum)[IPT]) {
  bool valid[IPT];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    valid[k] = r.lo + uint64_t(k) * NT + threadIdx.x < r.hi;
    cnt[k] = 0;
    psum[k] = 0;
  }
  if constexpr (Tab::kHashed) {
    typename Tab::Index idx[IPT];
    typename Tab::SlotT sl[IPT];
    bool live[IPT];
#pragma unroll
    for (int k = 0; k < IPT; ++k)
      if (valid[k]) idx[k] = tab.home(r.key[k]);
#pragma unroll
    for (int k = 0; k < IPT; ++k)
      if (valid[k]) sl[k] = tab.load(idx[k]);
    bool any = false;
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      live[k] = valid[k];
      if (!live[k]) continue;
      if (sl[k].rowid == kEmpty) {
        live[k] = false;
      } else {
        if (sl[k].key == r.key[k]) {
          ++cnt[k];
          first[k] = sl[k].rowid;
          psum[k] += static_cast<uint64_t>(sext(sl[k].pay));
          if (tab.unique) live[k] = false;
        }
        if (live[k]) {
          idx[k] = tab.next(idx[k], 1);
          any = true;
        }
      }
    }
    for (uint32_t step = 2; any; ++step) {
      any = false;
#pragma unroll
      for (int k = 0; k < IPT; ++k)
        if (live[k]) sl[k] = tab.load(idx[k]);
#pragma unroll
      for (int k = 0; k < IPT; ++k) {
        if (!live[k]) continue;
        if (sl[k].rowid == kEmpty) {
          live[k] = false;
        } else {
          if (sl[k].key == r.key[k]) {
            ++cnt[k];
            first[k] = sl[k].rowid;
            psum[k] += static_cast<uint64_t>(sext(sl[k].pay));
            if (tab.unique) live[k] = false;
          }
          if (live[k]) {
            idx[k] = tab.next(idx[k], step);
            any = true;
          }
        }
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < IPT; ++k)
      if (valid[k]) cnt[k] = tab.lookup(r.key[k], first[k], psum[k]);
  }
}

// Calls f(build_rowid) for each of the `cnt` matches of a probe row whose
// lookup gave `first`. Tables that keep a key's rows contiguous (Tab::kRuns)
// return the start of the run in `first` and expose row_at(i), so the matches
// are read straight from the run; other tables return the first match's row
// id and walk again (for_each) when there are more.
template <class Tab, typename K, class F>
__device__ __forceinline__ void emit_matches(const Tab &tab, K key, uint32_t cnt, uint32_t first, F f) {
  if constexpr (Tab::kRuns) {
    for (uint32_t j = 0; j < cnt; ++j) f(tab.row_at(first + j));
  } else {
    if (cnt == 1)
      f(first);
    else if (cnt > 1)
      tab.for_each(key, f);
  }
}

// Probe the loaded rows against `tab` and materialize the matches. Tables also
// provide  template <class F> void for_each(K key, F f) const  (f(build_rowid)
// for every match) for rows with more than one match. Match totals are 64-bit:
// a sub-tile of rows that each meet billions of build rows does not wrap.
// Uniform across the workgroup (contains barriers).
template <int NT, int IPT, int SCAP, class Tab, typename K, typename PS>
__device__ __forceinline__ void probe_process(const Tab &tab, const ProbeRegs<IPT, K, PS> &r,
                                              EmitLds<NT, SCAP> &L, uint64_t &fill,
                                              const EmitOut &o, uint64_t &cs) {
  uint32_t cnt[IPT], first[IPT];
  uint64_t psum[IPT];
  count_matches<NT, IPT>(tab, r, cnt, first, psum);
  uint64_t mine = 0;
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    if (cnt[k]) cs += psum[k] * static_cast<uint64_t>(sext(r.pay[k]));
    mine += cnt[k];
  }
  uint64_t total;
  const uint64_t off = emit_scan<NT>(mine, L.scan, &total);
  if (total == 0) return;
  if (!o.ob) {  // count-only: no positions are needed, so nothing is reserved
    fill += total;
    return;
  }
  if (fill + total > SCAP) {
    flush(L, o, static_cast<uint32_t>(fill));
    fill = 0;
  }
  // (probes of 8 rows per thread keep the per-row path below: the row table's
  // registers would cost them occupancy)
  if constexpr (Tab::kRuns && IPT <= 4) {
    static_assert(SCAP >= 2 * NT && NT <= 65536, "the stage holds a round's row table");
    if (total > SCAP) {
      // More matches than the stage holds (duplicated build keys; the stage is
      // empty here). Reserve the sub-tile's output range, then expand one row
      // slot k at a time (NT rows per round): the round's row table goes into
      // the stage arrays, and the pairs are written by consecutive threads at
      // consecutive positions, each reading its build row by index from the
      // key's run.
      const uint64_t base = reserve(L, o, total);
      uint64_t done = 0;  // pairs of this sub-tile placed so far (uniform)
      // row table: rd[i] = run start of row i minus the index of its first
      // pair (mod 2^32), so pair g of row i is build row tab.row_at(rd[i] + g);
      // rq[i] = its probe row id; row_of: the row of each pair of a chunk
      uint32_t *rd = L.b, *rq = L.b + NT;
      uint16_t *row_of = reinterpret_cast<uint16_t *>(L.p);
      constexpr uint32_t CH = 2 * SCAP;
      // every round's offsets from one scan of 16-bit fields when the whole
      // sub-tile has fewer than 2^16 pairs (no field can carry into the next)
      const bool packed = total < (uint64_t(1) << 16);
      uint64_t pk_ok = 0, pk_tot = 0;
      if (packed) {
        uint64_t v = 0;
#pragma unroll
        for (int k = 0; k < IPT; ++k) v |= static_cast<uint64_t>(cnt[k]) << (16 * k);
        pk_ok = emit_scan<NT>(v, L.scan, &pk_tot);
      }
#pragma unroll
      for (int k = 0; k < IPT; ++k) {
        uint64_t tk, ok;
        if (packed) {
          ok = (pk_ok >> (16 * k)) & 0xFFFFu;
          tk = (pk_tot >> (16 * k)) & 0xFFFFu;
        } else {
          ok = emit_scan<NT>(cnt[k], L.scan, &tk);
        }
        if (tk == 0) continue;
        if (tk >= (uint64_t(1) << 32)) {  // offsets do not fit the row table: per row
          uint64_t pos = base + done + ok;
          const uint32_t rr = r.rid[k];
          emit_matches(tab, r.key[k], cnt[k], first[k], [&](uint32_t b) { put_pair(o, pos++, b, rr); });
          done += tk;
          continue;
        }
        rd[threadIdx.x] = first[k] - static_cast<uint32_t>(ok);
        rq[threadIdx.x] = r.rid[k];
        // pairs of the round in chunks of CH: each thread marks its row on its
        // pairs' entries of `row_of`, then consecutive threads take consecutive
        // pairs, so the stores are coalesced
        for (uint64_t c0 = 0; c0 < tk; c0 += CH) {
          const uint64_t c1 = c0 + CH < tk ? c0 + CH : tk;
          const uint64_t a = ok > c0 ? ok : c0;
          const uint64_t e = ok + cnt[k] < c1 ? ok + cnt[k] : c1;
          for (uint64_t g = a; g < e; ++g) row_of[g - c0] = static_cast<uint16_t>(threadIdx.x);
          __syncthreads();
          uint64_t g = c0 + threadIdx.x;
          for (; g + NT < c1; g += 2 * NT) {  // two pairs per step: two lookup chains in flight
            const uint32_t i0 = row_of[g - c0], i1 = row_of[g + NT - c0];
            const uint32_t b0 = tab.row_at(rd[i0] + static_cast<uint32_t>(g));
            const uint32_t b1 = tab.row_at(rd[i1] + static_cast<uint32_t>(g + NT));
            put_pair(o, base + done + g, b0, rq[i0]);
            put_pair(o, base + done + g + NT, b1, rq[i1]);
          }
          if (g < c1) {
            const uint32_t i = row_of[g - c0];
            put_pair(o, base + done + g, tab.row_at(rd[i] + static_cast<uint32_t>(g)), rq[i]);
          }
          __syncthreads();
        }
        done += tk;
      }
      return;
    }
  }
  if (total > SCAP) {
    // More matches than the stage holds (duplicated build keys; the stage is
    // empty here): reserve the sub-tile's whole output range with one atomic,
    // then stage it one row slot k at a time (NT rows per round) and copy each
    // round to its place in the range, so these pairs are also written
    // contiguously; a round that alone overflows the stage writes straight
    // into the range.
    const uint64_t base = reserve(L, o, total);
    uint64_t done = 0;  // pairs of this sub-tile placed so far (uniform)
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      uint64_t tk;
      const uint64_t ok = emit_scan<NT>(cnt[k], L.scan, &tk);
      if (tk == 0) continue;
      if (tk > SCAP) {
        uint64_t pos = base + done + ok;
        const uint32_t rr = r.rid[k];
        emit_matches(tab, r.key[k], cnt[k], first[k], [&](uint32_t b) { put_pair(o, pos++, b, rr); });
        done += tk;
        continue;
      }
      uint32_t pos = static_cast<uint32_t>(ok);
      const uint32_t rr = r.rid[k];
      emit_matches(tab, r.key[k], cnt[k], first[k], [&](uint32_t b) {
        L.b[pos] = b;
        L.p[pos] = rr;
        ++pos;
      });
      __syncthreads();
      for (uint32_t i = threadIdx.x; i < tk; i += NT) put_pair(o, base + done + i, L.b[i], L.p[i]);
      __syncthreads();
      done += tk;
    }
    return;
  }
  uint32_t pos = static_cast<uint32_t>(fill + off);
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const uint32_t rr = r.rid[k];
    emit_matches(tab, r.key[k], cnt[k], first[k], [&](uint32_t b) {
      L.b[pos] = b;
      L.p[pos] = rr;
      ++pos;
    });
  }
  __syncthreads();
  fill += total;
}

// Probe the rows [lo, hi) in sub-tiles of NT * IPT rows. Uniform across the
// workgroup.
template <int NT, int IPT, int SCAP, class Tab, typename K, typename PS>
__device__ __forceinline__ void probe_range(const Tab &tab, const K *__restrict__ pk,
                                            const PS *__restrict__ pp,
                                            const uint32_t *__restrict__ prow, uint64_t lo,
                                            uint64_t hi, EmitLds<NT, SCAP> &L, uint64_t &fill,
                                            const EmitOut &o, uint64_t &cs) {
  constexpr uint64_t sub = uint64_t(NT) * IPT;
  if (lo >= hi) return;
  ProbeRegs<IPT, K, PS> cur;
  for (uint64_t t = lo; t < hi; t += sub) {
    probe_load<NT, IPT>(cur, pk, pp, prow, t, t + sub < hi ? t + sub : hi);
    probe_process<NT, IPT, SCAP>(tab, cur, L, fill, o, cs);
  }
}

}  // namespace eiger
