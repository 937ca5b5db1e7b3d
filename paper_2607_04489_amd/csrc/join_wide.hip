// join_wide.hip -- wide joins: the equi-join with the payload columns of both
// relations materialized for every result pair (the paper's "wide join",
// Section 5.2.1), by either of its two materialization strategies (Section 3.2):
//  GFUR  gather from the untransformed relations: join the keys with any
//        variant into (build row, probe row) pairs, then gather every payload
//        column of both sides from the caller's columns by row id;
//  GFTR  gather from the transformed relations (RADIX only): the payload
//        columns travel with the keys through the partitioning passes, the join
//        emits positions in the partitioned arrays, and each output block
//        gathers its payloads from one partition's contiguous range.
// Both give the same result; which is faster depends on the match ratio and
// the sizes (Section 5.2.3), so EIGER_MAT_AUTO chooses from the plan.
#include <algorithm>
#include <cmath>
#include <string>

#include "variants.hpp"

namespace eiger {

int check_join_inputs_public(const eiger_column &bk, const eiger_column &bp, const eiger_column &pk,
                             const eiger_column &pp, const eiger_plan_t *plan);

namespace {

constexpr int kMaxCols = 4;            // payload columns per side
constexpr float kGftrMinMatch = 0.25f;  // AUTO: GFTR from this estimated match ratio up

// One side's materialization: sources (column c as its low / high 32-bit word
// arrays, hi null for 4-byte columns; GFUR's 8-byte columns are whole at lo), GFTR's
// map from emitted position to row id, and the output columns.
struct GatherSide {
  const uint32_t *rows;
  const uint32_t *lo[kMaxCols];
  const uint32_t *hi[kMaxCols];
  void *dst[kMaxCols];
  int n;
};

constexpr int kGRows = 4;  // result rows of a thread

typedef uint32_t V4u __attribute__((ext_vector_type(4)));
typedef V4u V4uWord __attribute__((aligned(4)));  // outputs may start at any row
typedef uint64_t V2l __attribute__((ext_vector_type(2)));
typedef V2l V2lWord __attribute__((aligned(8)));

// One side's payloads of kGRows consecutive result rows t, t + 1, ... (the first
// `have` of them): all columns' reads are issued before any is stored.
template <bool kMapped>
__device__ __forceinline__ void gather_rows(const GatherSide &g, const uint32_t (&src)[kGRows], uint64_t t, int have) {
  uint64_t val[kMaxCols][kGRows];
#pragma unroll
  for (int c = 0; c < kMaxCols; ++c) {
    if (c >= g.n) break;
    const uint32_t *lo = g.lo[c], *hi = g.hi[c];
    if (hi) {
#pragma unroll
      for (int u = 0; u < kGRows; ++u) {
        if constexpr (kMapped)
          val[c][u] = (uint64_t(hi[src[u]]) << 32) | lo[src[u]];
        else
          val[c][u] = reinterpret_cast<const uint64_t *>(lo)[src[u]];  // an 8-byte column as it is
      }
    } else {
#pragma unroll
      for (int u = 0; u < kGRows; ++u) val[c][u] = lo[src[u]];
    }
  }
#pragma unroll
  for (int c = 0; c < kMaxCols; ++c) {
    if (c >= g.n) break;
    if (g.hi[c]) {
      uint64_t *dst = static_cast<uint64_t *>(g.dst[c]) + t;
      if (have == kGRows) {
        *reinterpret_cast<V2lWord *>(dst) = V2l{val[c][0], val[c][1]};
        *reinterpret_cast<V2lWord *>(dst + 2) = V2l{val[c][2], val[c][3]};
      } else {
#pragma unroll
        for (int u = 0; u < kGRows; ++u)
          if (u < have) dst[u] = val[c][u];
      }
    } else {
      uint32_t *dst = static_cast<uint32_t *>(g.dst[c]) + t;
      if (have == kGRows) {
        *reinterpret_cast<V4uWord *>(dst) = V4u{uint32_t(val[c][0]), uint32_t(val[c][1]), uint32_t(val[c][2]), uint32_t(val[c][3])};
      } else {
#pragma unroll
        for (int u = 0; u < kGRows; ++u)
          if (u < have) dst[u] = static_cast<uint32_t>(val[c][u]);
      }
    }
  }
}

// Row ids of emitted positions (GFTR), in place.
__device__ __forceinline__ void map_rows(uint32_t *__restrict__ ids, const uint32_t *__restrict__ rows,
                                         const uint32_t (&src)[kGRows], uint64_t t, int have) {
  uint32_t r[kGRows];
#pragma unroll
  for (int u = 0; u < kGRows; ++u) r[u] = rows[src[u]];
  if (have == kGRows) {
    *reinterpret_cast<V4uWord *>(ids + t) = V4u{r[0], r[1], r[2], r[3]};
  } else {
#pragma unroll
    for (int u = 0; u < kGRows; ++u)
      if (u < have) ids[t + u] = r[u];
  }
}

// Materialize result rows [0, min(count, cap)): payload words of both sides at
// the emitted (build, probe) indices, then (GFTR) the indices replaced by row ids.
// Four consecutive rows a thread, their reads in flight together. 268M rows of a
// GFTR join, one and two 4-byte columns: 2.01 ms (11 GB, 5.3 TB/s; 3.22 with a row at
// a time). 121M rows of a GFUR join: 1.24 ms, 0.5 of it the random reads of the
// build column (a 128-byte fill each, 255 G/s); 1.41 as one kernel with the other
// strategy, whose branches held the reads back. Rows 64 apart in a thread, so that a
// wave's reads are contiguous: 1.30 there and 2.54 above. Writing the columns from
// the GFTR join itself took 2.95 ms for 1.48 + 2.01: its workgroups' LDS tables leave
// too few waves for the reads.
template <bool kMapped>
__global__ void __launch_bounds__(256)
    k_wide_gather(uint32_t *__restrict__ ob, uint32_t *__restrict__ op, const JoinCounters *__restrict__ ctr,
                  uint64_t cap, GatherSide R, GatherSide S) {
  const uint64_t n = ctr->count < cap ? ctr->count : cap;
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x * kGRows;
  for (uint64_t t = (uint64_t(blockIdx.x) * blockDim.x + threadIdx.x) * kGRows; t < n; t += stride) {
    const int have = static_cast<int>(std::min<uint64_t>(kGRows, n - t));
    uint32_t b[kGRows], p[kGRows];
    if (have == kGRows) {
      const V4u vb = *reinterpret_cast<const V4uWord *>(ob + t), vp = *reinterpret_cast<const V4uWord *>(op + t);
#pragma unroll
      for (int u = 0; u < kGRows; ++u) {
        b[u] = vb[u];
        p[u] = vp[u];
      }
    } else {
#pragma unroll
      for (int u = 0; u < kGRows; ++u) {
        b[u] = ob[u < have ? t + u : t];
        p[u] = op[u < have ? t + u : t];
      }
    }
    gather_rows<kMapped>(R, b, t, have);
    gather_rows<kMapped>(S, p, t, have);
    if constexpr (kMapped) {
      map_rows(ob, R.rows, b, t, have);
      map_rows(op, S.rows, p, t, have);
    }
  }
}

int check_cols(const eiger_column *cols, int32_t n, int64_t rows, const char *what) {
  if (n < 0 || n > kMaxCols)
    return fail(EIGER_ERR_INVALID_ARG, std::string(what) + ": between 0 and 4 payload columns");
  if (n > 0 && !cols) return fail(EIGER_ERR_INVALID_ARG, std::string(what) + ": NULL column array");
  for (int32_t c = 0; c < n; ++c) {
    if (cols[c].dtype != EIGER_INT32 && cols[c].dtype != EIGER_INT64)
      return fail(EIGER_ERR_DTYPE, std::string(what) + ": payload dtype must be EIGER_INT32 or EIGER_INT64");
    if (cols[c].n != rows) return fail(EIGER_ERR_INVALID_ARG, std::string(what) + ": a payload column's row count differs from its keys'");
    if (rows > 0 && !cols[c].data) return fail(EIGER_ERR_INVALID_ARG, std::string(what) + ": NULL payload column");
    if (rows > 0 && reinterpret_cast<uintptr_t>(cols[c].data) % dtype_size(cols[c].dtype))
      return fail(EIGER_ERR_INVALID_ARG, std::string(what) + ": payload column not aligned to its dtype");
  }
  return EIGER_OK;
}

// The columns as word lanes (GFTR carries them through the partitioning).
WordCols word_cols(const eiger_column *cols, int32_t n) {
  WordCols w{};
  for (int32_t c = 0; c < n; ++c) {
    const uint32_t *base = static_cast<const uint32_t *>(cols[c].data);
    if (cols[c].dtype == EIGER_INT64) {
      w.src[w.n] = base;
      w.stride[w.n++] = 2;
      w.src[w.n] = base ? base + 1 : nullptr;
      w.stride[w.n++] = 2;
    } else {
      w.src[w.n] = base;
      w.stride[w.n++] = 1;
    }
  }
  return w;
}

int resolve_mat(const eiger_plan_t *plan, int32_t mat, int32_t nb_cols, int32_t np_cols, int64_t n_probe,
                int32_t *out) {
  if (mat != EIGER_MAT_GFUR && mat != EIGER_MAT_GFTR && mat != EIGER_MAT_AUTO)
    return fail(EIGER_ERR_INVALID_ARG, "eiger_join_wide: materialize must be an eiger_materialize");
  if (mat == EIGER_MAT_GFTR && plan->variant != EIGER_RADIX)
    return fail(EIGER_ERR_UNSUPPORTED, "eiger_join_wide: GFTR needs a RADIX plan (it gathers from the "
                                       "partitioned relations)");
  if (mat == EIGER_MAT_AUTO) {
    const double match = n_probe > 0 ? static_cast<double>(plan->predicted_out) / static_cast<double>(n_probe) : 0.0;
    mat = (plan->variant == EIGER_RADIX && match >= kGftrMinMatch) ? EIGER_MAT_GFTR : EIGER_MAT_GFUR;
  }
  // without payload columns there is nothing to carry: both strategies coincide
  if (nb_cols == 0 && np_cols == 0) mat = EIGER_MAT_GFUR;
  *out = mat;
  return EIGER_OK;
}

JoinArgs key_join_args(const eiger_column &bk, const eiger_column &pk, const eiger_plan_t *plan, uint32_t *ob,
                       uint32_t *op, int64_t cap, void *stream) {
  JoinArgs a{};
  a.bk = bk.data;
  a.bp = bk.data;  // the keys stand in for the narrow join's payloads
  a.pk = pk.data;
  a.pp = pk.data;
  a.nR = static_cast<uint64_t>(bk.n);
  a.nS = static_cast<uint64_t>(pk.n);
  a.kdt = a.bpdt = a.ppdt = bk.dtype;
  a.plan = *plan;
  a.ob = ob;
  a.op = op;
  a.cap = static_cast<uint64_t>(cap);
  a.s = static_cast<hipStream_t>(stream);
  return a;
}

// Lays out (ws.base null: only sizes) and, with a base, runs the key join of
// the chosen strategy. *src* are filled for GFTR.
int run_wide(const JoinArgs &a, int32_t mat, const WordCols &wr, const WordCols &wp, Workspace &ws,
             JoinCounters **ctr, WideSource *srcR, WideSource *srcS) {
  if (mat == EIGER_MAT_GFTR) return run_radix_wide(a, wr, wp, ws, ctr, srcR, srcS);
  return run_join_variant(a, ws, ctr);
}

GatherSide gather_side(const eiger_column *cols, int32_t n, void *const *dst, const WideSource *src) {
  GatherSide g{};
  g.n = n;
  g.rows = src ? src->rows : nullptr;
  int w = 0;
  for (int32_t c = 0; c < n; ++c) {
    const bool wide = cols[c].dtype == EIGER_INT64;
    if (src) {  // transformed: one word array per lane, stride 1
      g.lo[c] = src->words[w];
      g.hi[c] = wide ? src->words[w + 1] : nullptr;
    } else {
      const uint32_t *base = static_cast<const uint32_t *>(cols[c].data);
      g.lo[c] = base;
      g.hi[c] = wide ? base + 1 : nullptr;
    }
    w += wide ? 2 : 1;
    g.dst[c] = dst ? dst[c] : nullptr;
  }
  return g;
}

int check_wide(const eiger_column &bk, const eiger_column *bcols, int32_t nbc, const eiger_column &pk,
               const eiger_column *pcols, int32_t npc, const eiger_plan_t *plan) {
  int rc = check_join_inputs_public(bk, bk, pk, pk, plan);
  if (rc) return rc;
  if ((rc = check_cols(bcols, nbc, bk.n, "build"))) return rc;
  return check_cols(pcols, npc, pk.n, "probe");
}

}  // namespace
}  // namespace eiger

using namespace eiger;

extern "C" int eiger_join_wide_workspace_size(const eiger_plan_t *plan, int32_t materialize, eiger_column build_keys,
                                              const eiger_column *build_cols, int32_t n_build_cols,
                                              eiger_column probe_keys, const eiger_column *probe_cols,
                                              int32_t n_probe_cols, size_t *bytes) {
  if (!bytes) return fail(EIGER_ERR_INVALID_ARG, "eiger_join_wide_workspace_size: bytes is NULL");
  // sizing never reads data: dummy aligned addresses for the checks
  static const int64_t dummy[1] = {0};
  eiger_column bk = build_keys, pk = probe_keys;
  eiger_column bc[kMaxCols], pc[kMaxCols];
  if (bk.n > 0) bk.data = dummy;
  if (pk.n > 0) pk.data = dummy;
  if (n_build_cols < 0 || n_build_cols > kMaxCols || n_probe_cols < 0 || n_probe_cols > kMaxCols)
    return fail(EIGER_ERR_INVALID_ARG, "eiger_join_wide: between 0 and 4 payload columns a side");
  for (int32_t c = 0; c < n_build_cols; ++c) {
    if (!build_cols) return fail(EIGER_ERR_INVALID_ARG, "build: NULL column array");
    bc[c] = build_cols[c];
    if (bc[c].n > 0) bc[c].data = dummy;
  }
  for (int32_t c = 0; c < n_probe_cols; ++c) {
    if (!probe_cols) return fail(EIGER_ERR_INVALID_ARG, "probe: NULL column array");
    pc[c] = probe_cols[c];
    if (pc[c].n > 0) pc[c].data = dummy;
  }
  int rc = check_wide(bk, bc, n_build_cols, pk, pc, n_probe_cols, plan);
  if (rc) return rc;
  int32_t mat;
  if ((rc = resolve_mat(plan, materialize, n_build_cols, n_probe_cols, pk.n, &mat))) return rc;
  JoinArgs a = key_join_args(bk, pk, plan, nullptr, nullptr, 0, nullptr);
  Workspace ws(nullptr, 0);
  JoinCounters *ctr = nullptr;
  WideSource sr{}, sp{};
  if ((rc = run_wide(a, mat, word_cols(bc, n_build_cols), word_cols(pc, n_probe_cols), ws, &ctr, &sr, &sp)))
    return rc;
  *bytes = ws.used;
  return EIGER_OK;
}

extern "C" int eiger_join_wide(eiger_column build_keys, const eiger_column *build_cols, int32_t n_build_cols,
                               eiger_column probe_keys, const eiger_column *probe_cols, int32_t n_probe_cols,
                               const eiger_plan_t *plan, int32_t materialize, uint32_t *out_build_rowid,
                               uint32_t *out_probe_rowid, void *const *out_build_cols, void *const *out_probe_cols,
                               int64_t out_capacity, int64_t *out_count, int32_t *out_materialized, void *ws_ptr,
                               size_t ws_bytes, void *stream) {
  int rc = check_wide(build_keys, build_cols, n_build_cols, probe_keys, probe_cols, n_probe_cols, plan);
  if (rc) return rc;
  if (!out_count) return fail(EIGER_ERR_INVALID_ARG, "eiger_join_wide: out_count is NULL");
  if (out_capacity < 0) return fail(EIGER_ERR_INVALID_ARG, "eiger_join_wide: negative out_capacity");
  if (out_capacity > 0) {
    if (!out_build_rowid || !out_probe_rowid)
      return fail(EIGER_ERR_INVALID_ARG, "eiger_join_wide: out_capacity > 0 needs both row-id output arrays");
    if ((n_build_cols > 0 && !out_build_cols) || (n_probe_cols > 0 && !out_probe_cols))
      return fail(EIGER_ERR_INVALID_ARG, "eiger_join_wide: NULL output column array");
    for (int32_t c = 0; c < n_build_cols; ++c)
      if (!out_build_cols[c]) return fail(EIGER_ERR_INVALID_ARG, "eiger_join_wide: NULL build output column");
    for (int32_t c = 0; c < n_probe_cols; ++c)
      if (!out_probe_cols[c]) return fail(EIGER_ERR_INVALID_ARG, "eiger_join_wide: NULL probe output column");
  } else if (out_build_rowid || out_probe_rowid) {
    return fail(EIGER_ERR_INVALID_ARG, "eiger_join_wide: out_capacity == 0 takes NULL outputs (count only)");
  }
  int32_t mat;
  if ((rc = resolve_mat(plan, materialize, n_build_cols, n_probe_cols, probe_keys.n, &mat))) return rc;
  if (out_materialized) *out_materialized = mat;
  const WordCols wr = word_cols(build_cols, n_build_cols), wp = word_cols(probe_cols, n_probe_cols);
  JoinArgs a = key_join_args(build_keys, probe_keys, plan, out_capacity > 0 ? out_build_rowid : nullptr,
                             out_capacity > 0 ? out_probe_rowid : nullptr, out_capacity, stream);
  {
    Workspace dry(nullptr, 0);
    JoinCounters *unused = nullptr;
    WideSource sr{}, sp{};
    if ((rc = run_wide(a, mat, wr, wp, dry, &unused, &sr, &sp))) return rc;
    if (!ws_ptr || dry.used > ws_bytes)
      return fail(EIGER_ERR_WORKSPACE,
                  "eiger_join_wide: workspace too small (need " + std::to_string(dry.used) + " bytes)");
  }
  Workspace ws(ws_ptr, ws_bytes);
  JoinCounters *ctr = nullptr;
  WideSource sr{}, sp{};
  if ((rc = run_wide(a, mat, wr, wp, ws, &ctr, &sr, &sp))) return rc;
  hipStream_t s = a.s;
  if (out_capacity > 0 && build_keys.n > 0 && probe_keys.n > 0) {
    const bool tr = mat == EIGER_MAT_GFTR;
    const GatherSide gr = gather_side(build_cols, n_build_cols, out_build_cols, tr ? &sr : nullptr);
    const GatherSide gp = gather_side(probe_cols, n_probe_cols, out_probe_cols, tr ? &sp : nullptr);
    const uint64_t want = static_cast<uint64_t>(out_capacity);
    uint64_t g = (want + 256 * kGRows - 1) / (256 * kGRows);
    const uint64_t gmax = uint64_t(device_cu_count()) * 64;
    if (g > gmax) g = gmax;
    const dim3 grid(unsigned(g ? g : 1));
    if (tr)
      EIGER_LAUNCH("wide_gather", k_wide_gather<true>, grid, dim3(256), 0, s, out_build_rowid, out_probe_rowid, ctr, want,
                   gr, gp);
    else
      EIGER_LAUNCH("wide_gather", k_wide_gather<false>, grid, dim3(256), 0, s, out_build_rowid, out_probe_rowid, ctr, want,
                   gr, gp);
  }
  JoinCounters host{};
  if ((rc = read_counters(plan->variant, ctr, &host, s))) return rc;
  if (host.flags & kFlagBuildOutOfRange)
    return fail(EIGER_ERR_INVALID_ARG, "eiger_join_wide: a build key lies outside the plan's [build_min, build_max]");
  *out_count = static_cast<int64_t>(host.count);
  if (out_capacity > 0 && host.count > static_cast<uint64_t>(out_capacity))
    return fail(EIGER_ERR_CAPACITY, "eiger_join_wide: " + std::to_string(host.count) +
                                        " result rows exceed out_capacity " + std::to_string(out_capacity));
  return EIGER_OK;
}
