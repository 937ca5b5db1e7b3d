// sort.hip -- stable LSD radix sort of (key, row id) pairs, keys of 4 or 8 bytes.
//
// Section 3.6 (cases 1 and 2): a single numeric key, or several keys fused into
// one by smart key fusion, are sorted by radix sort. Each pass sorts by one digit
// of at most 8 bits, least significant digit first (a partitioning of many rows: up
// to 10); the number of passes follows
// the key's significant width (the fused key's width), not its type.
//
// One pass = a per-tile digit histogram (k_sort_hist), an exclusive scan over the
// count table, and a scatter (k_sort_scatter). The scatter ranks each tile's items
// stably: every wave walks its own contiguous segment 64 items at a time, finds
// the lanes holding the same digit with one ballot per digit bit, and keeps
// per-wave running digit counts in LDS; keys, then each value lane, are placed
// digit-major into one LDS copy of the tile and leave it in order, so each
// digit's run of the tile goes out as one contiguous block. Few tiles are scanned
// by the scatter's workgroups themselves; an input that fits one workgroup's LDS
// goes through all its passes there (k_sort_block).
#include <type_traits>

#include "common.hpp"
#include "sort.hpp"

namespace eiger {

namespace {

constexpr int kHNT = 256;  // histogram workgroup
constexpr int kSNT = 512;  // scatter workgroup
constexpr int kSWaves = kSNT / 64;
constexpr int kSDigitBits = 8;
constexpr int kSDigits = 1 << kSDigitBits;
static_assert(kSDigits == kHNT && kSDigits <= kSNT, "one thread per digit of 8 bits");

// Tiles. Large inputs: 10,240 items (6,144 of 8-byte keys): longer runs per digit
// against registers (2^28 4-byte pairs, 32 bits, all passes, with histograms
// of 0.30 ms, now 0.25: 12 items per thread 5.14 ms, 16 4.89, 20 4.77, 24 6.27, where
// they spill; 2^27 8-byte pairs: 8 items 4.63 ms, 10 3.77, 12 3.76, 16 4.00). Small
// inputs: 4,096 items, so that there are workgroups for the chip.
constexpr int kItemsSmall = 8;
template <typename K>
constexpr int items_large() {
  return sizeof(K) == 8 ? 12 : 20;
}
// Large tiles from this many of them on (two per CU).
constexpr uint64_t kLargeTiles = 512;
template <typename K>
constexpr uint64_t large_rows() {
  return kLargeTiles * kSNT * items_large<K>();
}
template <typename K>
bool use_large(uint64_t n) {
  return n >= large_rows<K>();
}
// Up to this many tiles the scatter's workgroups sum the count table's columns
// themselves instead of three scan launches.
constexpr uint64_t kSelfScanTiles = 256;
// Workgroups per CU of the histogram's grid; they loop over the remaining tiles.
constexpr uint64_t kHistPerCu = 64;
constexpr uint32_t kXcds = 8;

// Digit of a plain sort: bits [shift, shift + width) of the key.
template <typename K>
struct KeyDigit {
  static constexpr int kBits = kSDigitBits;
  static constexpr bool kStore = false;  // cheap: recomputed from the key
  int shift;
  uint32_t mask;
  __device__ __forceinline__ uint32_t operator()(K k) const { return static_cast<uint32_t>(k >> shift) & mask; }
};

// Digit of a key's partition id, the top `bits` bits of its partition hash
// (hash partitioning).
template <typename K, int B>
struct PartDigit {
  static constexpr int kBits = B;
  // 8-byte keys: a 64-bit hash per item is kept (its digit, in LDS) for the write-out
  static constexpr bool kStore = sizeof(K) == 8;
  int top;  // 64 - partition bits
  int shift;
  uint32_t mask;
  __device__ __forceinline__ uint32_t operator()(K k) const {
    return static_cast<uint32_t>((part_hash(k) >> top) >> shift) & mask;
  }
};

// Workgroups loop over tiles (the grid is sized to the chip): one workgroup
// per tile was limited by how fast workgroups are dispatched, not by memory. Each
// XCD takes a contiguous eighth of the tiles, whose counts share cache lines (2^28
// 4-byte keys 0.25 ms a pass, 4.4 TB/s; dealt round-robin 0.26).
// kVec (16-byte aligned keys): each thread reads 16 bytes of consecutive keys
// per load (counting does not depend on which thread holds which key).
// Counts go out digit-major (cnt[digit * ntiles + tile], for the scan) or, for the
// self-scanning scatter (kTileMajor), as cnt[tile * 256 + digit].
template <typename K, int T, typename D, bool kVec, bool kTileMajor>
__global__ void __launch_bounds__(kHNT) k_sort_hist(const K *__restrict__ keys, uint64_t n, D dig, uint32_t ntiles,
                                                    uint32_t *__restrict__ cnt) {
  constexpr int V = 16 / static_cast<int>(sizeof(K));  // keys per 16-byte load
  constexpr int NV = T / V;                            // 16-byte loads per tile
  static_assert(NV % kHNT == 0, "whole loads");
  constexpr int kDigits = 1 << D::kBits;
  __shared__ uint32_t h[kDigits];
  const uint32_t per_xcd = (ntiles + kXcds - 1) / kXcds;
  for (uint32_t x = blockIdx.x / kXcds; x < per_xcd; x += gridDim.x / kXcds) {
    const uint32_t tile = blockIdx.x % kXcds * per_xcd + x;
    if (tile >= ntiles) break;
#pragma unroll
    for (int d = threadIdx.x; d < kDigits; d += kHNT) h[d] = 0;
    __syncthreads();
    const uint64_t base = static_cast<uint64_t>(tile) * T;
    if constexpr (kVec) {
#pragma unroll
      for (int j = 0; j < NV / kHNT; ++j) {
        const uint64_t i = base + static_cast<uint64_t>(j * kHNT + static_cast<int>(threadIdx.x)) * V;
        if (i + V <= n) {
          K v[V];
          *reinterpret_cast<uint4 *>(v) = *reinterpret_cast<const uint4 *>(keys + i);
#pragma unroll
          for (int u = 0; u < V; ++u) atomicAdd(&h[dig(v[u])], 1u);
        } else {
#pragma unroll
          for (int u = 0; u < V; ++u)
            if (i + u < n) atomicAdd(&h[dig(keys[i + u])], 1u);
        }
      }
    } else {
#pragma unroll 16
      for (int j = 0; j < T / kHNT; ++j) {
        const uint64_t i = base + static_cast<uint64_t>(j) * kHNT + threadIdx.x;
        if (i < n) atomicAdd(&h[dig(keys[i])], 1u);
      }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t d = threadIdx.x; d < kDigits; d += kHNT) {
      if constexpr (kTileMajor)
        cnt[static_cast<uint64_t>(tile) * kDigits + d] = h[d];
      else if (d <= dig.mask)
        cnt[static_cast<uint64_t>(d) * ntiles + tile] = h[d];
    }
    __syncthreads();
  }
}

// 32-bit value lanes moved along with the keys. Lane w of row i is
// src[w][i * stride[w]]; a NULL source lane means the row id i itself.
struct LanesIn {
  const uint32_t *src[kMaxLanes];
  uint32_t stride[kMaxLanes];
  int n;
};
struct LanesOut {
  uint32_t *dst[kMaxLanes];
};

// Stable ranks of a wave's items of one step among the wave's items so far:
// lanes of the same digit are found with one ballot per digit bit, `cnt` (LDS, the
// wave's own) holds the running counts. Returns the item's rank in its digit.
template <int B>
__device__ __forceinline__ uint32_t wave_rank(uint32_t d, bool ok, int bits, uint16_t *cnt) {
  const uint64_t all = __ballot(ok);
  uint32_t plo = static_cast<uint32_t>(all), phi = static_cast<uint32_t>(all >> 32);
#pragma unroll
  for (int b = 0; b < B; ++b) {
    if (b < bits) {
      const uint32_t m = static_cast<uint32_t>(static_cast<int32_t>(d << (31 - b)) >> 31);  // all ones when bit b is set
      const uint64_t bb = __ballot(m != 0);
      plo &= ~(static_cast<uint32_t>(bb) ^ m);
      phi &= ~(static_cast<uint32_t>(bb >> 32) ^ m);
    }
  }
  const uint32_t before = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0u));
  // every lane reads the wave's running count before the group's first lane
  // (the only writer of this digit in this step) stores the new one; LDS
  // operations of one wave complete in order
  const uint32_t pre = ok ? cnt[d] : 0u;
  if (ok && before == 0) cnt[d] = static_cast<uint16_t>(pre + __popc(plo) + __popc(phi));
  return pre + before;
}

// Digits of 2^B a thread of NT sees to in the tile's digit scan: digits
// threadIdx.x * digits_per<NT, B> and on, while there are any.
template <int NT, int B>
constexpr int digits_per = (1 << B) > NT ? (1 << B) / NT : 1;

// Turns the waves' digit counts of a tile into start positions in the tile's
// digit-major order (wave order = item order); ds: the starts of this thread's
// digits. All threads call it (barriers).
template <int NT, int B>
__device__ __forceinline__ void tile_starts(uint16_t (*wcnt)[1 << B], uint32_t *scan_tmp,
                                            uint32_t (&ds)[digits_per<NT, B>]) {
  constexpr int NW = NT / 64, PER = digits_per<NT, B>;
  const int t = threadIdx.x * PER;
  uint32_t c[PER][NW], tot = 0;
  if (t < (1 << B)) {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      ds[e] = tot;
#pragma unroll
      for (int x = 0; x < NW; ++x) {
        c[e][x] = wcnt[x][t + e];
        tot += c[e][x];
      }
    }
  }
  uint32_t all;
  const uint32_t first = block_exclusive_scan<NT, uint32_t>(tot, scan_tmp, &all);
  if (t < (1 << B)) {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      ds[e] += first;
      uint32_t run = ds[e];
#pragma unroll
      for (int x = 0; x < NW; ++x) {
        wcnt[x][t + e] = static_cast<uint16_t>(run);
        run += c[e][x];
      }
    }
  }
}

template <typename K, int kItems, bool kStoreDigit, int B>
struct ScatterLds {
  K sk[kSNT * kItems];  // the tile's keys, then each value lane
  uint8_t sd[kStoreDigit ? kSNT * kItems : 4];
  __align__(4) uint16_t wcnt[kSWaves][1 << B];
  uint32_t adj[1 << B];
  uint32_t scan_tmp[kSWaves];
};

// Keeps the compiler from interleaving more than a few items' address
// arithmetic, which cost registers beyond the 128 that two workgroups per CU allow.
template <int kEvery>
__device__ __forceinline__ void item_fence(int j) {
  if (j % kEvery == kEvery - 1) __builtin_amdgcn_sched_barrier(0);
}

// One tile of a scatter pass. kFull: the tile has all its items. Uniform across
// the workgroup (barriers).
template <typename K, int kItems, typename D, bool kSelfScan, bool kFull>
__device__ __forceinline__ void scatter_tile(ScatterLds<K, kItems, D::kStore, D::kBits> &L, const K *__restrict__ kin,
                                             const LanesIn &vin, uint64_t base, uint32_t in_tile, const D &dig, int bits,
                                             uint32_t tile, uint32_t ntiles, const uint32_t *__restrict__ offs,
                                             K *__restrict__ kout, const LanesOut &vout) {
  uint32_t *sv = reinterpret_cast<uint32_t *>(L.sk);
  const int w = threadIdx.x / 64;
  const uint32_t first = static_cast<uint32_t>(w) * (64 * kItems) + __lane_id();  // this thread's items: first + 64 j
  auto has = [&](uint32_t i) { return kFull || i < in_tile; };
  for (int x = threadIdx.x; x < kSWaves * (1 << D::kBits) / 2; x += kSNT) reinterpret_cast<uint32_t *>(L.wcnt)[x] = 0;
  K key[kItems];
  {
    const K *src = kin + base;
#pragma unroll
    for (int j = 0; j < kItems; ++j) key[j] = has(first + j * 64) ? src[first + j * 64] : K(0);
  }
  __syncthreads();
  uint32_t pos[(kItems + 1) / 2];  // two 16-bit positions each
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t r = wave_rank<D::kBits>(dig(key[j]), has(first + j * 64), bits, L.wcnt[w]);
    pos[j / 2] = j % 2 ? pos[j / 2] | r << 16 : r;
    item_fence<2>(j);
  }
  __syncthreads();
  constexpr int kPer = digits_per<kSNT, D::kBits>;
  uint32_t ds[kPer];
  tile_starts<kSNT, D::kBits>(L.wcnt, L.scan_tmp, ds);
  // global start of this tile's run of digit t, minus its start inside the tile
  const uint32_t t = threadIdx.x;
  if constexpr (kSelfScan) {
    static_assert(D::kBits == kSDigitBits, "one lane per four digits");
    // wave w sums tiles w, w + kSWaves, ...; a lane takes four digits
    uint4 total = make_uint4(0, 0, 0, 0), before = total;
#pragma unroll 8
    for (uint32_t x = w; x < ntiles; x += kSWaves) {
      const uint4 c = reinterpret_cast<const uint4 *>(offs)[x * (kSDigits / 4) + __lane_id()];
      const uint32_t m = x < tile ? ~0u : 0u;
      total.x += c.x; total.y += c.y; total.z += c.z; total.w += c.w;
      before.x += c.x & m; before.y += c.y & m; before.z += c.z & m; before.w += c.w & m;
    }
    static_assert(sizeof(L.sk) >= 2 * kSWaves * kSDigits * 4, "the waves' sums fit the tile's LDS");
    uint4 *part = reinterpret_cast<uint4 *>(L.sk);  // free until the keys are placed
    part[w * (kSDigits / 4) + __lane_id()] = total;
    part[(kSWaves + w) * (kSDigits / 4) + __lane_id()] = before;
    __syncthreads();
    uint32_t tot = 0, bef = 0;
    if (t < kSDigits) {
#pragma unroll
      for (int x = 0; x < kSWaves; ++x) {
        tot += sv[x * kSDigits + t];
        bef += sv[(kSWaves + x) * kSDigits + t];
      }
    }
    uint32_t all;
    const uint32_t start = block_exclusive_scan<kSNT, uint32_t>(tot, L.scan_tmp, &all);
    if (t < kSDigits) L.adj[t] = start + bef - ds[0];
  } else {
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const uint32_t d = t * kPer + e;
      if (d < (1u << D::kBits)) L.adj[d] = d <= dig.mask ? offs[static_cast<uint64_t>(d) * ntiles + tile] - ds[e] : 0u;
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t d = dig(key[j]);
    const uint32_t p = ((pos[j / 2] >> (j % 2 * 16)) & 0xFFFFu) + L.wcnt[w][d];
    pos[j / 2] = j % 2 ? (pos[j / 2] & 0xFFFFu) | p << 16 : (pos[j / 2] & 0xFFFF0000u) | p;
    if (has(first + j * 64)) {
      L.sk[p] = key[j];
      if constexpr (D::kStore) L.sd[p] = static_cast<uint8_t>(d);
    }
    item_fence<8>(j);
  }
  uint32_t val[kItems];
  auto load_lane = [&](int v) {
    if (!vin.src[v]) {  // the row ids
#pragma unroll
      for (int j = 0; j < kItems; ++j) val[j] = static_cast<uint32_t>(base) + first + j * 64;
    } else if (vin.stride[v] == 1) {
      const uint32_t *src = vin.src[v] + base;
#pragma unroll
      for (int j = 0; j < kItems; ++j) val[j] = has(first + j * 64) ? src[first + j * 64] : 0u;
    } else {
      const uint32_t st = vin.stride[v];
      const uint32_t *src = vin.src[v] + base * st;
#pragma unroll
      for (int j = 0; j < kItems; ++j) val[j] = has(first + j * 64) ? src[(first + j * 64) * st] : 0u;
    }
  };
  if (vin.n > 0) load_lane(0);  // in flight while the keys go out
  __syncthreads();
  uint32_t o[kItems];  // where tile position t + j * kSNT goes
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t p = t + j * kSNT;
    o[j] = 0;
    if (has(p)) {
      const K k = L.sk[p];
      uint32_t d;
      if constexpr (D::kStore)
        d = L.sd[p];
      else
        d = dig(k);
      o[j] = L.adj[d] + p;
      kout[o[j]] = k;
    }
    item_fence<8>(j);
  }
  for (int v = 0; v < vin.n; ++v) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      if (has(first + j * 64)) sv[(pos[j / 2] >> (j % 2 * 16)) & 0xFFFFu] = val[j];
      item_fence<8>(j);
    }
    if (v + 1 < vin.n) load_lane(v + 1);
    __syncthreads();
    uint32_t *__restrict__ dst = vout.dst[v];
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      if (has(t + j * kSNT)) dst[o[j]] = sv[t + j * kSNT];
      item_fence<8>(j);
    }
  }
  __syncthreads();
}

// One LSD pass: rank each tile's items stably by digit, place them digit-major
// in LDS, write each digit's run of the tile to its global position. Keys and
// value lanes take turns in one LDS copy of the tile, so the tile's size does not
// depend on the row's width. Bound by memory: 2^28 4-byte pairs move 4.3 GB in
// 0.86 ms a pass (5.0 TB/s; a copy: 4.6 to 4.8); each XCD takes a contiguous
// eighth of the tiles, so that the partial lines at the ends of neighbouring
// tiles' runs meet in one L2 (with tiles dealt round-robin: 1.5 ms).
// One tile per workgroup: a loop over tiles made the compiler keep every item's
// addresses across tiles, and the registers spilled.
// kSelfScan: `offs` holds the raw counts, tile-major, and each workgroup sums
// the columns it needs; else the scanned counts, digit-major.
template <typename K, int kItems, typename D, bool kSelfScan>
__global__ void __launch_bounds__(kSNT, 4) k_sort_scatter(const K *__restrict__ kin, LanesIn vin, uint64_t n, D dig,
                                                          int bits, uint32_t ntiles, const uint32_t *__restrict__ offs,
                                                          K *__restrict__ kout, LanesOut vout) {
  constexpr uint32_t T = kSNT * kItems;
  static_assert(T < 65536, "counts and positions of a tile fit 16 bits");
  __shared__ ScatterLds<K, kItems, D::kStore, D::kBits> L;
  const uint32_t per_xcd = (ntiles + kXcds - 1) / kXcds;
  const uint32_t tile = blockIdx.x % kXcds * per_xcd + blockIdx.x / kXcds;
  if (tile >= ntiles) return;
  const uint64_t base = static_cast<uint64_t>(tile) * T;
  if (n - base >= T)
    scatter_tile<K, kItems, D, kSelfScan, true>(L, kin, vin, base, T, dig, bits, tile, ntiles, offs, kout, vout);
  else
    scatter_tile<K, kItems, D, kSelfScan, false>(L, kin, vin, base, static_cast<uint32_t>(n - base), dig, bits,
                                                     tile, ntiles, offs, kout, vout);
}

// All passes of an input that fits one workgroup's LDS: the pairs stay there
// between passes. (A sort of 1,000 pairs by 32 bits was 20 launches, 210 us.)
constexpr int kBNT = 1024;
template <typename K>
constexpr int block_items_max() {
  return sizeof(K) == 8 ? 8 : 16;
}
template <typename K, int kItems>
__global__ void __launch_bounds__(kBNT) k_sort_block(const K *__restrict__ kin, const uint32_t *__restrict__ vin,
                                                     uint32_t n, int key_bits, K *__restrict__ kout,
                                                     uint32_t *__restrict__ vout) {
  constexpr int T = kBNT * kItems;
  __shared__ K sk[T];
  __shared__ uint32_t sv[T];
  __shared__ __align__(4) uint16_t wcnt[kBNT / 64][kSDigits];
  __shared__ uint32_t scan_tmp[kBNT / 64];
  const int lane = __lane_id();
  const int w = threadIdx.x / 64;
  const uint32_t first = static_cast<uint32_t>(w) * (64 * kItems) + lane;
  K key[kItems];
  uint32_t val[kItems], r[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t i = first + j * 64;
    key[j] = i < n ? kin[i] : K(0);
    val[j] = i < n && vin ? vin[i] : i;
  }
  const int passes = (key_bits + kSDigitBits - 1) / kSDigitBits;
  int shift = 0;
  for (int p = 0; p < passes; ++p) {
    const int bits = (key_bits - shift + (passes - p) - 1) / (passes - p);
    const KeyDigit<K> dig{shift, (1u << bits) - 1u};
    for (int x = threadIdx.x; x < kBNT / 64 * kSDigits / 2; x += kBNT) reinterpret_cast<uint32_t *>(wcnt)[x] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kItems; ++j) r[j] = wave_rank<kSDigitBits>(dig(key[j]), first + j * 64 < n, bits, wcnt[w]);
    __syncthreads();
    uint32_t ds[1];
    tile_starts<kBNT, kSDigitBits>(wcnt, scan_tmp, ds);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      if (first + j * 64 < n) {
        const uint32_t at = wcnt[w][dig(key[j])] + r[j];
        sk[at] = key[j];
        sv[at] = val[j];
      }
    }
    __syncthreads();
    // (the next pass writes sk and sv only after two more barriers)
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const uint32_t i = first + j * 64;
      if (i < n) {
        key[j] = sk[i];
        val[j] = sv[i];
      }
    }
    shift += bits;
  }
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t i = first + j * 64;
    if (i < n) {
      kout[i] = key[j];
      vout[i] = val[j];
    }
  }
}

template <typename K>
__global__ void __launch_bounds__(256) k_sort_copy(const K *__restrict__ kin, const uint32_t *__restrict__ vin,
                                                   uint64_t n, K *__restrict__ kout, uint32_t *__restrict__ vout) {
  const uint64_t stride = static_cast<uint64_t>(gridDim.x) * blockDim.x;
  for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
    kout[i] = kin[i];
    vout[i] = vin ? vin[i] : static_cast<uint32_t>(i);
  }
}

// Count-table and temporaries of `passes` passes over n items in tiles of T.
template <typename K>
struct PassBufs {
  uint64_t ntiles;
  uint32_t *cnt;
  uint64_t *tmp, *total;
  K *k2;
  uint32_t *v2[kMaxLanes];
};

template <typename K>
PassBufs<K> pass_bufs(Workspace &ws, uint64_t n, int T, int lanes, int passes, int digit_bits = kSDigitBits) {
  PassBufs<K> b{};
  b.ntiles = (n + T - 1) / T;
  const uint64_t ncnt = b.ntiles << digit_bits;
  b.cnt = ws.take<uint32_t>(ncnt);
  b.tmp = ws.take<uint64_t>(scan_tmp_elems(ncnt));
  b.total = ws.take<uint64_t>(1);
  if (passes > 1) {
    b.k2 = ws.take<K>(n);
    for (int v = 0; v < lanes; ++v) b.v2[v] = ws.take<uint32_t>(n);
  }
  return b;
}

int pass_count(int bits, int digit_bits = kSDigitBits) { return (bits + digit_bits - 1) / digit_bits; }

// Raises ws, which held `from` bytes before a layout for n rows, to what the most rows
// in small tiles take there: larger tiles need fewer counts and a wider digit fewer
// passes, and a workspace sized for many rows is to take every smaller input.
template <typename K>
void at_least_small(Workspace &ws, size_t from, uint64_t n, int lanes, int passes) {
  if (!use_large<K>(n)) return;
  Workspace small(nullptr, 0);
  small.used = from;
  pass_bufs<K>(small, large_rows<K>() - 1, kSNT * kItemsSmall, lanes, passes);
  ws.used = std::max(ws.used, small.used);
}

// pass_count(total_bits) stable passes of balanced digit widths, least
// significant digit first, alternating between (kout, vout) and the
// temporaries so that the last pass lands in (kout, vout). make(shift, mask)
// gives the pass's digit functor.
template <typename K, int kItems, int B = kSDigitBits, typename MakeDigit>
int lsd_passes(const K *kin, LanesIn vin, uint64_t n, int total_bits, K *kout, LanesOut vout, const PassBufs<K> &b,
               MakeDigit make, hipStream_t s) {
  constexpr int T = kSNT * kItems;
  const int passes = pass_count(total_bits, B);
  const unsigned hist_grid = static_cast<unsigned>(
      std::min<uint64_t>((b.ntiles + kXcds - 1) / kXcds, uint64_t(device_cu_count()) * kHistPerCu / kXcds) * kXcds);
  const unsigned scat_grid = static_cast<unsigned>((b.ntiles + kXcds - 1) / kXcds * kXcds);
  const uint32_t nt = static_cast<uint32_t>(b.ntiles);
  const bool self_scan = kItems == kItemsSmall && b.ntiles <= kSelfScanTiles;
  int shift = 0;
  const K *src_k = kin;
  LanesIn src_v = vin;
  for (int p = 0; p < passes; ++p) {
    const int bits = (total_bits - shift + (passes - p) - 1) / (passes - p);
    const bool to_out = ((passes - 1 - p) % 2) == 0;
    K *dk = to_out ? kout : b.k2;
    LanesOut dv{};
    for (int v = 0; v < vin.n; ++v) dv.dst[v] = to_out ? vout.dst[v] : b.v2[v];
    const auto dig = make(shift, (1u << bits) - 1u);
    using D = std::remove_const_t<decltype(dig)>;
    const bool vec = reinterpret_cast<uintptr_t>(src_k) % 16 == 0;
#define EIGER_HIST(VEC, TM)                                                                                        \
  EIGER_LAUNCH("sort_hist", (k_sort_hist<K, T, D, VEC, TM>), dim3(hist_grid), dim3(kHNT), 0, s, src_k, n, dig, nt, b.cnt)
    if (self_scan) {
      if constexpr (kItems == kItemsSmall) {  // large tiles are never that few
        if (vec) EIGER_HIST(true, true); else EIGER_HIST(false, true);
        EIGER_LAUNCH("sort_scatter", (k_sort_scatter<K, kItems, D, true>), dim3(scat_grid), dim3(kSNT), 0, s, src_k,
                     src_v, n, dig, bits, nt, b.cnt, dk, dv);
      }
    } else {
      if (vec) EIGER_HIST(true, false); else EIGER_HIST(false, false);
      int rc = exclusive_scan_u32(b.cnt, b.cnt, (static_cast<uint64_t>(dig.mask) + 1) * b.ntiles, b.tmp, b.total, s);
      if (rc) return rc;
      EIGER_LAUNCH("sort_scatter", (k_sort_scatter<K, kItems, D, false>), dim3(scat_grid), dim3(kSNT), 0, s, src_k,
                   src_v, n, dig, bits, nt, b.cnt, dk, dv);
    }
#undef EIGER_HIST
    src_k = dk;
    for (int v = 0; v < vin.n; ++v) {
      src_v.src[v] = dv.dst[v];
      src_v.stride[v] = 1;
    }
    shift += bits;
  }
  return EIGER_OK;
}

template <typename K, int kItems>
int sort_block(const K *kin, const uint32_t *vin, uint64_t n, int key_bits, K *kout, uint32_t *vout, hipStream_t s) {
  EIGER_LAUNCH("sort_block", (k_sort_block<K, kItems>), dim3(1), dim3(kBNT), 0, s, kin, vin, static_cast<uint32_t>(n),
               key_bits, kout, vout);
  return EIGER_OK;
}

template <typename K>
int sort_impl(const K *kin, const uint32_t *vin, uint64_t n, int key_bits, K *kout, uint32_t *vout, Workspace &ws,
              hipStream_t s) {
  const bool large = use_large<K>(n);
  const size_t from = ws.used;
  const PassBufs<K> b = pass_bufs<K>(ws, n, kSNT * (large ? items_large<K>() : kItemsSmall), 1, 2);
  at_least_small<K>(ws, from, n, 1, 2);
  if (!ws.base || n == 0) return EIGER_OK;
  if (ws.used > ws.cap) return fail(EIGER_ERR_WORKSPACE, "radix sort: its temporaries exceed the region given");
  if (key_bits == 0 || n == 1) {
    const unsigned grid = static_cast<unsigned>(std::min<uint64_t>((n + 255) / 256, 4096));
    EIGER_LAUNCH("sort_copy", k_sort_copy<K>, dim3(grid), dim3(256), 0, s, kin, vin, n, kout, vout);
    return EIGER_OK;
  }
  if (n <= kBNT) return sort_block<K, 1>(kin, vin, n, key_bits, kout, vout, s);
  if (n <= kBNT * 4) return sort_block<K, 4>(kin, vin, n, key_bits, kout, vout, s);
  if (n <= kBNT * block_items_max<K>()) return sort_block<K, block_items_max<K>()>(kin, vin, n, key_bits, kout, vout, s);
  LanesIn in{};
  in.src[0] = vin;
  in.stride[0] = 1;
  in.n = 1;
  LanesOut out{};
  out.dst[0] = vout;
  const auto make = [](int shift, uint32_t mask) { return KeyDigit<K>{shift, mask}; };
  if (large) return lsd_passes<K, items_large<K>()>(kin, in, n, key_bits, kout, out, b, make, s);
  return lsd_passes<K, kItemsSmall>(kin, in, n, key_bits, kout, out, b, make, s);
}

// Partition bounds: off[p] = first position whose partition id is >= p (the
// rows are sorted by partition id), off[F] = n.
template <typename K>
__global__ void __launch_bounds__(256) k_part_bounds(const K *__restrict__ keys, uint64_t n, int bits, uint32_t F,
                                                     uint32_t *__restrict__ off) {
  const uint32_t stride = gridDim.x * blockDim.x;
  for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p <= F; p += stride) {
    uint64_t a = 0, b = n;
    while (a < b) {
      const uint64_t m = a + (b - a) / 2;
      if ((part_hash(keys[m]) >> (64 - bits)) < p)
        a = m + 1;
      else
        b = m;
    }
    off[p] = static_cast<uint32_t>(a);
  }
}

template <typename K>
void partition_results(uint64_t n, const PartLanes &cols, int bits, Workspace &ws, PartitionOut *out) {
  *out = PartitionOut{};
  out->keys = ws.take<K>(n ? n : 1);
  for (int v = 0; v < cols.n; ++v) out->words[v] = ws.take<uint32_t>(n ? n : 1);
  out->off = ws.take<uint32_t>((uint64_t(1) << bits) + 1);
}

// Digit width of a partitioning. Large inputs of 4-byte keys that need one or two
// bits more than a pass of 8 has take them in one pass of 10: its tile holds 10 items
// per digit instead of 40 and its count table is four times as large, but a whole
// pass over the rows goes (2^28 int32 keys with two int32 lanes, 9 bits: 2.51 +
// 0.42 ms in scatter and histogram as two passes, 1.59 + 0.25 as one; 10 bits 2.55 +
// 0.41 against 1.72 + 0.29; 2^27 rows with two int64 values 2.21 + 0.24 against 1.92
// + 0.13). Digits of 11 bits need smaller tiles and gain nothing (2.58 + 0.42 ms in
// two passes, 2.33 + 0.44 and 0.18 more in the scan in one). Small inputs keep 8
// bits: their tiles of 4,096 items would hold 4 items per digit.
constexpr int kWideBits = 10;
template <typename K>
bool wide_digit(uint64_t n, int bits) {
  return sizeof(K) == 4 && bits > kSDigitBits && bits <= kWideBits && use_large<K>(n);
}

template <typename K>
PassBufs<K> partition_temps(uint64_t n, const PartLanes &cols, int bits, Workspace &ws) {
  const int digit = wide_digit<K>(n, bits) ? kWideBits : kSDigitBits;
  const int items = use_large<K>(n) ? items_large<K>() : kItemsSmall;
  return pass_bufs<K>(ws, n, kSNT * items, cols.n, pass_count(bits, digit), digit);
}

template <typename K>
int partition_run(const K *keys, uint64_t n, const PartLanes &cols, int bits, Workspace &ws, const PartitionOut &out,
                  hipStream_t s) {
  const PassBufs<K> b = partition_temps<K>(n, cols, bits, ws);
  if (ws.used > ws.cap) return fail(EIGER_ERR_WORKSPACE, "radix partition: its temporaries exceed the region given");
  const uint32_t F = 1u << bits;
  K *ok = static_cast<K *>(out.keys);
  if (n > 0) {
    LanesIn in{};
    LanesOut ov{};
    in.n = cols.n;
    for (int v = 0; v < cols.n; ++v) {
      in.src[v] = cols.src[v];
      in.stride[v] = cols.stride[v];
      ov.dst[v] = out.words[v];
    }
    const int top = 64 - bits;
    const auto make = [top](int shift, uint32_t mask) { return PartDigit<K, kSDigitBits>{top, shift, mask}; };
    int rc = EIGER_OK;
    if (wide_digit<K>(n, bits)) {
      if constexpr (sizeof(K) == 4)
        rc = lsd_passes<K, items_large<K>(), kWideBits>(
            keys, in, n, bits, ok, ov, b,
            [top](int shift, uint32_t mask) { return PartDigit<K, kWideBits>{top, shift, mask}; }, s);
    } else if (use_large<K>(n)) {
      rc = lsd_passes<K, items_large<K>()>(keys, in, n, bits, ok, ov, b, make, s);
    } else {
      rc = lsd_passes<K, kItemsSmall>(keys, in, n, bits, ok, ov, b, make, s);
    }
    if (rc) return rc;
  }
  EIGER_LAUNCH("part_bounds", k_part_bounds<K>, dim3(static_cast<unsigned>(std::min<uint64_t>((F + 256) / 256, 1024))),
               dim3(256), 0, s, ok, n, bits, F, out.off);
  return EIGER_OK;
}

}  // namespace

int radix_partition_results(int key_bytes, uint64_t n, const PartLanes &cols, int bits, Workspace &ws,
                            PartitionOut *out) {
  if (bits < 1 || bits > 24 || cols.n < 0 || cols.n > kMaxLanes)
    return fail(EIGER_ERR_INVALID_ARG, "radix partition: bits in [1, 24], at most 9 lanes");
  if (key_bytes == 8)
    partition_results<int64_t>(n, cols, bits, ws, out);
  else
    partition_results<int32_t>(n, cols, bits, ws, out);
  return EIGER_OK;
}

void radix_partition_temps(int key_bytes, uint64_t n, const PartLanes &cols, int bits, Workspace &ws) {
  if (key_bytes == 8)
    partition_temps<int64_t>(n, cols, bits, ws);
  else
    partition_temps<int32_t>(n, cols, bits, ws);
}

int radix_partition_run(int key_bytes, const void *keys, uint64_t n, const PartLanes &cols, int bits, Workspace &ws,
                        const PartitionOut &out, hipStream_t s) {
  if (key_bytes == 8) return partition_run<int64_t>(static_cast<const int64_t *>(keys), n, cols, bits, ws, out, s);
  return partition_run<int32_t>(static_cast<const int32_t *>(keys), n, cols, bits, ws, out, s);
}

int radix_partition_lanes(int key_bytes, const void *keys, uint64_t n, const PartLanes &cols, int bits, Workspace &ws,
                          PartitionOut *out, hipStream_t s, bool run) {
  if (int rc = radix_partition_results(key_bytes, n, cols, bits, ws, out)) return rc;
  const size_t from = ws.used;
  if (ws.base && run) {
    if (int rc = radix_partition_run(key_bytes, keys, n, cols, bits, ws, *out, s)) return rc;
  } else {
    radix_partition_temps(key_bytes, n, cols, bits, ws);
  }
  if (key_bytes == 8)
    at_least_small<int64_t>(ws, from, n, cols.n, pass_count(bits));
  else
    at_least_small<int32_t>(ws, from, n, cols.n, pass_count(bits));
  return EIGER_OK;
}

int radix_sort_pairs(int key_bytes, const void *kin, const uint32_t *vin, uint64_t n, int key_bits, void *kout,
                     uint32_t *vout, Workspace &ws, hipStream_t s) {
  if (key_bytes == 8)
    return sort_impl<uint64_t>(static_cast<const uint64_t *>(kin), vin, n, key_bits, static_cast<uint64_t *>(kout),
                               vout, ws, s);
  return sort_impl<uint32_t>(static_cast<const uint32_t *>(kin), vin, n, key_bits, static_cast<uint32_t *>(kout),
                             vout, ws, s);
}

size_t radix_sort_bytes(int key_bytes, uint64_t n, int tile) {
  Workspace ws(nullptr, 0);
  if (key_bytes == 8)
    pass_bufs<uint64_t>(ws, n, tile, 1, 2);
  else
    pass_bufs<uint32_t>(ws, n, tile, 1, 2);
  return ws.used;
}

}  // namespace eiger

using namespace eiger;

namespace {

int check_sort_args(int32_t key_bytes, int64_t n, int32_t key_bits) {
  if (key_bytes != 4 && key_bytes != 8) return fail(EIGER_ERR_INVALID_ARG, "eiger_sort_pairs: key_bytes must be 4 or 8");
  if (n < 0 || n > EIGER_MAX_ROWS) return fail(EIGER_ERR_TOO_LARGE, "eiger_sort_pairs: n outside [0, EIGER_MAX_ROWS]");
  if (key_bits < 0 || key_bits > 8 * key_bytes)
    return fail(EIGER_ERR_INVALID_ARG, "eiger_sort_pairs: key_bits outside [0, 8 * key_bytes]");
  return EIGER_OK;
}

}  // namespace

extern "C" int eiger_sort_pairs_workspace_size(int32_t key_bytes, int64_t n, int32_t key_bits, size_t *bytes) {
  if (!bytes) return fail(EIGER_ERR_INVALID_ARG, "eiger_sort_pairs_workspace_size: bytes is NULL");
  if (int rc = check_sort_args(key_bytes, n, key_bits)) return rc;
  Workspace ws(nullptr, 0);
  radix_sort_pairs(key_bytes, nullptr, nullptr, static_cast<uint64_t>(n), key_bits, nullptr, nullptr, ws, nullptr);
  *bytes = ws.used + 256;
  return EIGER_OK;
}

extern "C" int eiger_sort_pairs(int32_t key_bytes, const void *keys_in, const uint32_t *vals_in, int64_t n,
                                int32_t key_bits, void *keys_out, uint32_t *vals_out, void *workspace,
                                size_t workspace_bytes, void *stream) {
  if (int rc = check_sort_args(key_bytes, n, key_bits)) return rc;
  if (n > 0 && (!keys_in || !keys_out || !vals_out || !workspace))
    return fail(EIGER_ERR_INVALID_ARG, "eiger_sort_pairs: NULL buffer");
  size_t need = 0;
  eiger_sort_pairs_workspace_size(key_bytes, n, key_bits, &need);
  if (workspace_bytes < need) return fail(EIGER_ERR_WORKSPACE, "eiger_sort_pairs: workspace too small");
  if (n > 0 && (keys_in == keys_out || (vals_in && vals_in == vals_out)))
    return fail(EIGER_ERR_INVALID_ARG, "eiger_sort_pairs: outputs must not alias the inputs");
  Workspace ws(workspace, workspace_bytes);
  return radix_sort_pairs(key_bytes, keys_in, vals_in, static_cast<uint64_t>(n), key_bits, keys_out, vals_out, ws,
                          static_cast<hipStream_t>(stream));
}
