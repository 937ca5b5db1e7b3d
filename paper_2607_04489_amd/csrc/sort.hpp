// sort.hpp -- the radix sort shared by the sort entry points and smart key fusion.
#pragma once

#include "common.hpp"

namespace eiger {

// Stable LSD radix sort of n (key, value) pairs by the low key_bits bits of the
// key (key_bytes 4 or 8). vin == nullptr sorts the row ids 0..n-1 along. Outputs
// must not alias the inputs. With ws.base == nullptr it only sizes the workspace;
// with one, it lays its temporaries out within ws.cap or returns EIGER_ERR_WORKSPACE
// without a launch (so does radix_partition_run).
int radix_sort_pairs(int key_bytes, const void *kin, const uint32_t *vin, uint64_t n, int key_bits, void *kout,
                     uint32_t *vout, Workspace &ws, hipStream_t s);

// Bytes of the temporaries of such a sort in tiles of `tile` pairs (sizing only).
size_t radix_sort_bytes(int key_bytes, uint64_t n, int tile);

// Hash partitioning with value lanes: rows are ordered by partition id, the top
// `bits` bits of the key's partition hash (part_hash), by stable passes of the same
// sort (digits of at most 8 bits, 10 for many rows); up to kMaxLanes 32-bit lanes move along (lane w
// of row i is src[w][i * stride[w]]; a NULL lane is the row id i itself). out receives
// the partitioned keys, the lanes (stride 1) and off[0..2^bits] (partition p is
// [off[p], off[p + 1])). Always lays out the workspace, whose size rises with n;
// enqueues only with a workspace base and `run`.
constexpr int kMaxLanes = 9;  // a row id and eight payload words
struct PartLanes {
  const uint32_t *src[kMaxLanes];
  uint32_t stride[kMaxLanes];
  int n;
};
struct PartitionOut {
  void *keys;
  uint32_t *words[kMaxLanes];
  uint32_t *off;
};
int radix_partition_lanes(int key_bytes, const void *keys, uint64_t n, const PartLanes &cols, int bits, Workspace &ws,
                          PartitionOut *out, hipStream_t s, bool run);
// The same in parts, so that partitionings that run one after another can share
// their temporaries: lay out the results, lay out the temporaries (sizing; no more
// than they take, which may be less for more rows), enqueue (laying out the same
// temporaries in ws).
int radix_partition_results(int key_bytes, uint64_t n, const PartLanes &cols, int bits, Workspace &ws, PartitionOut *out);
void radix_partition_temps(int key_bytes, uint64_t n, const PartLanes &cols, int bits, Workspace &ws);
int radix_partition_run(int key_bytes, const void *keys, uint64_t n, const PartLanes &cols, int bits, Workspace &ws,
                        const PartitionOut &out, hipStream_t s);

}  // namespace eiger
