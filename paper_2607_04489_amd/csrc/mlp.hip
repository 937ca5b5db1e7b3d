// mlp.hip -- forward, loss, backward and Adam kernels of the selector MLP.
//
// Network: x[16] -> relu(x W1 + b1)[64] -> relu(h1 W2 + b2)[64] -> h2 W3 + b3 [16].
// Every sum runs over its index in increasing order with explicit fused
// multiply-adds, and every batch reduction is a fixed loop or a fixed-shape tree,
// so the kernels are deterministic (no float atomics) and the host forward in
// selector.hip reproduces the device forward bit for bit.
#include <algorithm>
#include <cmath>
#include <string>

#include "common.hpp"
#include "mlp.hpp"

namespace eiger {

namespace {

// The training step is four launches: forward by rows, loss, backward by rows,
// weight gradients with the Adam update. None of it is bound by memory or by the
// matrix units: a step at 4,050 rows reads 3 MB and makes 71 MFLOP, and every sum
// has to run in index order, so the step costs its serial chains and its launches.
// At 4,050 rows: 7 us forward, 11 us loss, 9 us backward, 42 us weight gradients.
// (With one thread per output reading global memory at each link of its chain, the
// step took 2.93 ms, 2.86 of it in the weight gradients.)
constexpr int kRowsPer = 4;   // rows a wave takes together
constexpr int kRowWaves = 4;  // waves of a row kernel's workgroup
static_assert(kHid == 64 && kOut * kRowsPer == 64 && kIn <= 64, "one lane per hidden unit, or per (row, output)");

// Forward: h1, h2, y of kRowsPer rows per wave and step. A lane holds its unit's
// weight columns in registers; the rows' four chains run side by side.
__global__ void __launch_bounds__(64 * kRowWaves)
    k_mlp_forward_train(const float *__restrict__ P, const float *__restrict__ x, int batch, float *__restrict__ h1,
                        float *__restrict__ h2, float *__restrict__ y) {
  __shared__ __align__(16) float xs[kRowWaves][kRowsPer][kIn], hs[2][kRowWaves][kRowsPer][kHid];
  const MlpOffsets o;
  const int j = threadIdx.x % 64, w = threadIdx.x / 64, q3 = j / kOut, j3 = j % kOut;
  float w1[kIn], w2[kHid], w3[kHid];
#pragma unroll
  for (int i = 0; i < kIn; ++i) w1[i] = P[o.W1 + i * kHid + j];
#pragma unroll
  for (int i = 0; i < kHid; ++i) w2[i] = P[o.W2 + i * kHid + j];
#pragma unroll
  for (int i = 0; i < kHid; ++i) w3[i] = P[o.W3 + i * kOut + j3];
  const float c1 = P[o.b1 + j], c2 = P[o.b2 + j], c3 = P[o.b3 + j3];
  const int64_t step = int64_t(gridDim.x) * kRowWaves * kRowsPer;
  // every wave of the workgroup runs the same number of steps (barriers below)
  for (int64_t base = int64_t(blockIdx.x) * kRowWaves * kRowsPer; base < batch; base += step) {
    const int64_t r0 = base + int64_t(w) * kRowsPer;
    const int nr = r0 < batch ? static_cast<int>(std::min<int64_t>(kRowsPer, batch - r0)) : 0;
    if (j < kRowsPer * kIn) xs[w][j / kIn][j % kIn] = j / kIn < nr ? x[r0 * kIn + j] : 0.f;
    __syncthreads();
    float acc[kRowsPer] = {};
#pragma unroll
    for (int i = 0; i < kIn; ++i)
#pragma unroll
      for (int q = 0; q < kRowsPer; ++q) acc[q] = fmaf(xs[w][q][i], w1[i], acc[q]);
#pragma unroll
    for (int q = 0; q < kRowsPer; ++q) {
      const float v = acc[q] + c1;
      hs[0][w][q][j] = v < 0.f ? 0.f : v;
      if (q < nr) h1[(r0 + q) * kHid + j] = v < 0.f ? 0.f : v;
      acc[q] = 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kHid; ++i)
#pragma unroll
      for (int q = 0; q < kRowsPer; ++q) acc[q] = fmaf(hs[0][w][q][i], w2[i], acc[q]);
#pragma unroll
    for (int q = 0; q < kRowsPer; ++q) {
      const float v = acc[q] + c2;
      hs[1][w][q][j] = v < 0.f ? 0.f : v;
      if (q < nr) h2[(r0 + q) * kHid + j] = v < 0.f ? 0.f : v;
    }
    __syncthreads();
    float out = 0.f;
#pragma unroll
    for (int i = 0; i < kHid; ++i) out = fmaf(hs[1][w][q3][i], w3[i], out);
    if (q3 < nr) y[(r0 + q3) * kOut + j3] = out + c3;
    __syncthreads();
  }
}

// Masked squared error: one workgroup, fixed-shape reduction. Writes
// out[0] = *loss = sum mask*(y-t)^2 / sum mask (0 when the mask is empty), out[1] =
// sum mask. A thread's kLossBatch terms are loaded before any is added.
constexpr int kLossBatch = 16;
__global__ void __launch_bounds__(1024) k_mlp_loss(const float *__restrict__ y, const float *__restrict__ t,
                                                   const float *__restrict__ m, int64_t n,
                                                   float *__restrict__ out, float *__restrict__ loss) {
  __shared__ float se[1024], sm[1024];
  float a = 0.f, c = 0.f;
  for (int64_t i0 = threadIdx.x; i0 < n; i0 += 1024 * kLossBatch) {
    float vy[kLossBatch], vt[kLossBatch], vm[kLossBatch];
#pragma unroll
    for (int u = 0; u < kLossBatch; ++u) {
      const int64_t i = i0 + int64_t(u) * 1024;
      if (i < n) {
        vy[u] = y[i];
        vt[u] = t[i];
        vm[u] = m[i];
      }
    }
#pragma unroll
    for (int u = 0; u < kLossBatch; ++u) {
      if (i0 + int64_t(u) * 1024 < n) {
        const float d = vy[u] - vt[u];
        a = fmaf(vm[u] * d, d, a);
        c += vm[u];
      }
    }
  }
  se[threadIdx.x] = a;
  sm[threadIdx.x] = c;
  __syncthreads();
  for (int w = 512; w >= 1; w >>= 1) {
    if (threadIdx.x < w) {
      se[threadIdx.x] += se[threadIdx.x + w];
      sm[threadIdx.x] += sm[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = sm[0] > 0.f ? se[0] / sm[0] : 0.f;
    out[1] = sm[0];
    *loss = out[0];
  }
}

// Backward by rows: dY = 2 * mask * (y - t) / sum(mask), then per hidden layer
// da[b][i] = (sum_j dz[b][j] * W[i][j]) * [act[b][i] > 0] (ReLU derivative). A lane
// holds its unit's weight rows in registers.
__global__ void __launch_bounds__(64 * kRowWaves)
    k_mlp_backward_rows(const float *__restrict__ P, const float *__restrict__ y, const float *__restrict__ t,
                        const float *__restrict__ m, const float *__restrict__ lossv, const float *__restrict__ h1,
                        const float *__restrict__ h2, int batch, float *__restrict__ dy, float *__restrict__ dh2,
                        float *__restrict__ dh1) {
  __shared__ __align__(16) float ys[kRowWaves][kRowsPer][kOut], hs[kRowWaves][kRowsPer][kHid];
  const MlpOffsets o;
  const int j = threadIdx.x % 64, w = threadIdx.x / 64, q3 = j / kOut;
  float w3[kOut], w2[kHid];
#pragma unroll
  for (int i = 0; i < kOut; ++i) w3[i] = P[o.W3 + j * kOut + i];
#pragma unroll
  for (int i = 0; i < kHid; ++i) w2[i] = P[o.W2 + j * kHid + i];
  const float msum = lossv[1];
  const int64_t step = int64_t(gridDim.x) * kRowWaves * kRowsPer;
  for (int64_t base = int64_t(blockIdx.x) * kRowWaves * kRowsPer; base < batch; base += step) {
    const int64_t r0 = base + int64_t(w) * kRowsPer;
    const int nr = r0 < batch ? static_cast<int>(std::min<int64_t>(kRowsPer, batch - r0)) : 0;
    float a1[kRowsPer], a2[kRowsPer];
#pragma unroll
    for (int q = 0; q < kRowsPer; ++q) {
      a2[q] = q < nr ? h2[(r0 + q) * kHid + j] : 0.f;
      a1[q] = q < nr ? h1[(r0 + q) * kHid + j] : 0.f;
    }
    float d = 0.f;
    if (q3 < nr) {
      const int64_t i = r0 * kOut + j;
      d = msum > 0.f ? 2.f * m[i] * (y[i] - t[i]) / msum : 0.f;
      dy[i] = d;
    }
    ys[w][q3][j % kOut] = d;
    __syncthreads();
    float acc[kRowsPer] = {};
#pragma unroll
    for (int i = 0; i < kOut; ++i)
#pragma unroll
      for (int q = 0; q < kRowsPer; ++q) acc[q] = fmaf(ys[w][q][i], w3[i], acc[q]);
#pragma unroll
    for (int q = 0; q < kRowsPer; ++q) {
      const float v = a2[q] > 0.f ? acc[q] : 0.f;
      hs[w][q][j] = v;
      if (q < nr) dh2[(r0 + q) * kHid + j] = v;
      acc[q] = 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kHid; ++i)
#pragma unroll
      for (int q = 0; q < kRowsPer; ++q) acc[q] = fmaf(hs[w][q][i], w2[i], acc[q]);
#pragma unroll
    for (int q = 0; q < kRowsPer; ++q)
      if (q < nr) dh1[(r0 + q) * kHid + j] = a1[q] > 0.f ? acc[q] : 0.f;
    __syncthreads();
  }
}

// One layer's weight gradients: dW[i][j] = sum_b a[b][i] * dz[b][j] (at g[i * OUT + j]),
// db[j] = sum_b dz[b][j] (i == IN: the bias block follows the weights).
struct GradLayer {
  const float *a, *dz;
  int64_t at;  // offset of the layer's weights in the parameter arrays
};
struct AdamArgs {
  float *p, *m, *v, *g;
  float lr, c1, c2;
};
typedef float F4 __attribute__((ext_vector_type(4)));
typedef F4 F4Word __attribute__((aligned(4)));  // the workspace may be aligned to 4 bytes only
constexpr int kGradNT = 128;
constexpr int kGradRows = 128;  // rows of an LDS tile: 32 KB of dz and 1 KB of a at OUT = 64
constexpr int kGradLds = kGradRows * 66;
constexpr int kGradStep = 16;   // rows whose LDS reads are in flight together
static_assert(kGradRows % (2 * kGradStep) == 0, "a tile is whole double steps");

// One chain per thread, kGradNT consecutive ones per workgroup. The chain's length
// (batch) is its cost, so its links must not wait for memory: tiles of kGradRows
// rows go through LDS, the next tile's loads in flight in registers while the
// chains walk this one. 25 clocks a link at 4,050 rows; two waves a workgroup, so
// that a compute unit's LDS reads (256 bytes a wave and link) keep up: four waves
// 57 us, two 42. Then Adam with bias correction (Kingma & Ba 2015) on the
// thread's own parameter.
template <int IN, int OUT>
__device__ __forceinline__ void grad_chains(const GradLayer &l, int block, int batch, const AdamArgs &A, float *lds) {
  constexpr int NI = kGradNT / OUT;                // inputs i of a workgroup
  constexpr int VZ = kGradRows * OUT / 4 / kGradNT;  // 16-byte loads of dz per thread and tile
  constexpr int VA = kGradRows * NI / kGradNT;       // words of a per thread and tile
  static_assert(VZ * 4 * kGradNT == kGradRows * OUT && VA * kGradNT == kGradRows * NI, "a tile is whole loads");
  static_assert(kGradRows * (OUT + NI) <= kGradLds, "the tile fits");
  float *zs = lds, *as = lds + kGradRows * OUT;  // as: NI columns of kGradRows rows
  const int i0 = block * NI, il = threadIdx.x / OUT, j = threadIdx.x % OUT;
  F4 z[VZ];
  float v[VA];
  // Every load is unconditional: a load under a condition was waited for on the
  // spot. A partial last tile clamps its places to the last row (what lies past
  // the batch is not used), a whole one keeps 32-bit offsets from one base.
  const uint32_t ic = min(i0 + static_cast<int>(threadIdx.x) % NI, IN - 1);
  auto load = [&](int64_t r0) {
    const float *zsrc = l.dz + r0 * OUT, *asrc = l.a + r0 * IN;
    if (r0 + kGradRows <= batch) {
#pragma unroll
      for (int u = 0; u < VZ; ++u) z[u] = *reinterpret_cast<const F4Word *>(zsrc + (u * kGradNT + threadIdx.x) * 4);
#pragma unroll
      for (int u = 0; u < VA; ++u) v[u] = asrc[((u * kGradNT + threadIdx.x) / NI) * IN + ic];
    } else {
      const uint32_t rows = static_cast<uint32_t>(batch - r0), last = rows * OUT - 4;
#pragma unroll
      for (int u = 0; u < VZ; ++u)
        z[u] = *reinterpret_cast<const F4Word *>(zsrc + min((u * kGradNT + threadIdx.x) * 4, last));
#pragma unroll
      for (int u = 0; u < VA; ++u) v[u] = asrc[min((u * kGradNT + threadIdx.x) / NI, rows - 1) * IN + ic];
    }
  };
  load(0);
  float acc = 0.f;
  for (int64_t r0 = 0; r0 < batch; r0 += kGradRows) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < VZ; ++u) *reinterpret_cast<F4 *>(zs + (u * kGradNT + threadIdx.x) * 4) = z[u];
#pragma unroll
    for (int u = 0; u < VA; ++u) {
      const int e = u * kGradNT + threadIdx.x;
      as[(e % NI) * kGradRows + e / NI] = i0 + e % NI < IN ? v[u] : 1.f;  // the bias sums 1 * dz
    }
    __syncthreads();
    if (r0 + kGradRows < batch) load(r0 + kGradRows);
    const int rows = static_cast<int>(std::min<int64_t>(kGradRows, batch - r0));
    const float *ac = as + il * kGradRows, *zc = zs + j;
    // kGradStep rows' values are read from LDS while the chain walks the
    // kGradStep before them (rows past `rows` are read, inside the tile, and not used)
    float av[2][kGradStep], zv[2][kGradStep];
    auto fetch = [&](int r, int b) {
#pragma unroll
      for (int u = 0; u < kGradStep; u += 4)
        *reinterpret_cast<float4 *>(&av[b][u]) = *reinterpret_cast<const float4 *>(ac + r + u);
#pragma unroll
      for (int u = 0; u < kGradStep; ++u) zv[b][u] = zc[(r + u) * OUT];
    };
    fetch(0, 0);
    int r = 0;
    for (; r + 2 * kGradStep <= rows; r += 2 * kGradStep) {
      fetch(r + kGradStep, 1);
#pragma unroll
      for (int u = 0; u < kGradStep; ++u) acc = fmaf(av[0][u], zv[0][u], acc);
      if (r + 2 * kGradStep < kGradRows) fetch(r + 2 * kGradStep, 0);
#pragma unroll
      for (int u = 0; u < kGradStep; ++u) acc = fmaf(av[1][u], zv[1][u], acc);
    }
    for (; r < rows; ++r) acc = fmaf(ac[r], zc[r * OUT], acc);
  }
  if (i0 + il > IN) return;
  const int64_t i = l.at + (i0 + il) * OUT + j;
  const float beta1 = 0.9f, beta2 = 0.999f, eps = 1e-8f;
  const float gi = acc;
  A.g[i] = gi;
  const float mi = beta1 * A.m[i] + (1.f - beta1) * gi;
  const float vi = beta2 * A.v[i] + (1.f - beta2) * gi * gi;
  A.m[i] = mi;
  A.v[i] = vi;
  const float mh = mi / A.c1, vh = vi / A.c2;
  A.p[i] -= A.lr * mh / (sqrtf(vh) + eps);
}

template <int IN, int OUT>
constexpr int grad_blocks() {
  return (IN + 1 + kGradNT / OUT - 1) / (kGradNT / OUT);
}
constexpr int kGradB2 = grad_blocks<kHid, kHid>(), kGradB3 = grad_blocks<kHid, kOut>(), kGradB1 = grad_blocks<kIn, kHid>();

// All three layers in one launch.
__global__ void __launch_bounds__(kGradNT) k_mlp_grad_adam(GradLayer l1, GradLayer l2, GradLayer l3, int batch, AdamArgs A) {
  __shared__ __align__(16) float lds[kGradLds];
  const int b = blockIdx.x;
  if (b < kGradB2)
    grad_chains<kHid, kHid>(l2, b, batch, A, lds);
  else if (b < kGradB2 + kGradB3)
    grad_chains<kHid, kOut>(l3, b - kGradB2, batch, A, lds);
  else
    grad_chains<kIn, kHid>(l1, b - kGradB2 - kGradB3, batch, A, lds);
}

// Inference without scratch memory: one 64-thread workgroup per row at a time,
// hidden activations in LDS; each output is the same ordered fused sum as in
// k_mlp_forward_train, so the result equals the training forward bit for bit.
__global__ void __launch_bounds__(64) k_mlp_forward_rows(const float *__restrict__ P, const float *__restrict__ x,
                                                         int batch, float *__restrict__ y) {
  __shared__ float xs[kIn], h1[kHid], h2[kHid];
  const MlpOffsets o;
  const int j = threadIdx.x;
  for (int b = blockIdx.x; b < batch; b += gridDim.x) {
    if (j < kIn) xs[j] = x[int64_t(b) * kIn + j];
    __syncthreads();
    float acc = 0.f;
    for (int i = 0; i < kIn; ++i) acc = fmaf(xs[i], P[o.W1 + i * kHid + j], acc);
    acc += P[o.b1 + j];
    h1[j] = acc < 0.f ? 0.f : acc;
    __syncthreads();
    acc = 0.f;
    for (int i = 0; i < kHid; ++i) acc = fmaf(h1[i], P[o.W2 + i * kHid + j], acc);
    acc += P[o.b2 + j];
    h2[j] = acc < 0.f ? 0.f : acc;
    __syncthreads();
    if (j < kOut) {
      acc = 0.f;
      for (int i = 0; i < kHid; ++i) acc = fmaf(h2[i], P[o.W3 + i * kOut + j], acc);
      y[int64_t(b) * kOut + j] = acc + P[o.b3 + j];
    }
    __syncthreads();
  }
}

struct TrainWs {
  float *h1, *h2, *y, *dy, *dh2, *dh1, *lossv;
};

TrainWs train_layout(Workspace &ws, int batch) {
  TrainWs w;
  const size_t B = static_cast<size_t>(batch);
  w.h1 = ws.take<float>(B * kHid);
  w.h2 = ws.take<float>(B * kHid);
  w.y = ws.take<float>(B * kOut);
  w.dy = ws.take<float>(B * kOut);
  w.dh2 = ws.take<float>(B * kHid);
  w.dh1 = ws.take<float>(B * kHid);
  w.lossv = ws.take<float>(2);
  return w;
}

}  // namespace

}  // namespace eiger

using namespace eiger;

extern "C" int64_t eiger_mlp_param_count(void) { return kParams; }

extern "C" size_t eiger_mlp_train_workspace_size(int32_t batch) {
  if (batch <= 0) return 0;
  Workspace ws(nullptr, 0);
  train_layout(ws, batch);
  return ws.used;
}

extern "C" int eiger_mlp_forward(const float *params, const float *x, int32_t batch, float *y, void *stream) {
  if (!params || !y || batch < 0 || (batch > 0 && !x))
    return fail(EIGER_ERR_INVALID_ARG, "eiger_mlp_forward: bad arguments");
  if (batch == 0) return EIGER_OK;
  if (batch > (1 << 24)) return fail(EIGER_ERR_TOO_LARGE, "eiger_mlp_forward: batch above 2^24");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const unsigned grid = static_cast<unsigned>(std::min<int64_t>(batch, int64_t(device_cu_count()) * 16));
  EIGER_LAUNCH("mlp_forward_rows", k_mlp_forward_rows, dim3(grid), dim3(64), 0, s, params, x, batch, y);
  return EIGER_OK;
}

extern "C" int eiger_mlp_train_step(float *params, float *adam_m, float *adam_v, float *grads, const float *x,
                                    const float *target, const float *mask, int32_t batch, float lr,
                                    int32_t step, float *loss, void *ws_ptr, size_t ws_bytes, void *stream) {
  if (!params || !adam_m || !adam_v || !grads || !x || !target || !mask || !loss)
    return fail(EIGER_ERR_INVALID_ARG, "eiger_mlp_train_step: NULL pointer");
  if (batch <= 0 || batch > (1 << 24)) return fail(EIGER_ERR_INVALID_ARG, "eiger_mlp_train_step: batch out of range");
  if (step < 1) return fail(EIGER_ERR_INVALID_ARG, "eiger_mlp_train_step: step must be >= 1");
  if (!(lr > 0.f)) return fail(EIGER_ERR_INVALID_ARG, "eiger_mlp_train_step: lr must be > 0");
  Workspace ws(ws_ptr, ws_bytes);
  TrainWs w = train_layout(ws, batch);
  if (!ws_ptr || ws.used > ws_bytes)
    return fail(EIGER_ERR_WORKSPACE, "eiger_mlp_train_step: workspace too small (need " +
                                         std::to_string(ws.used) + " bytes)");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const MlpOffsets o;
  const unsigned grid = static_cast<unsigned>(std::min<int64_t>(
      (int64_t(batch) + kRowWaves * kRowsPer - 1) / (kRowWaves * kRowsPer), int64_t(device_cu_count()) * 8));
  EIGER_LAUNCH("mlp_forward", k_mlp_forward_train, dim3(grid), dim3(64 * kRowWaves), 0, s, params, x, batch, w.h1,
               w.h2, w.y);
  EIGER_LAUNCH("mlp_loss", k_mlp_loss, dim3(1), dim3(1024), 0, s, w.y, target, mask, int64_t(batch) * kOut, w.lossv,
               loss);
  EIGER_LAUNCH("mlp_backward", k_mlp_backward_rows, dim3(grid), dim3(64 * kRowWaves), 0, s, params, w.y, target, mask,
               w.lossv, w.h1, w.h2, batch, w.dy, w.dh2, w.dh1);
  const float c1 = 1.f - std::pow(0.9f, static_cast<float>(step));
  const float c2 = 1.f - std::pow(0.999f, static_cast<float>(step));
  EIGER_LAUNCH("mlp_grad_adam", k_mlp_grad_adam, dim3(kGradB1 + kGradB2 + kGradB3), dim3(kGradNT), 0, s,
               GradLayer{x, w.dh1, o.W1}, GradLayer{w.h1, w.dh2, o.W2}, GradLayer{w.h2, w.dy, o.W3}, batch,
               AdamArgs{params, adam_m, adam_v, grads, lr, c1, c2});
  return EIGER_OK;
}
