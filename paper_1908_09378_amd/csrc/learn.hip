// Training of the extraction-threshold model (an addition to the paper's
// method: a small MLP that picks how many minima a parDijkstra round pulls).
//
//  k_trace_labels  label of a traced round = log2 of the longest prefix of
//                  B_0 (in key order) whose keys are already final distances
//                  (pulling that many minima wastes no relaxation)
//  k_feat_stats    per-feature mean and standard deviation of the dataset
//  k_mlp_grad      one mini-batch: forward 8 -> 64 -> 64 -> 1 (GELU, weights
//                  rounded to bfloat16, FP32 accumulation), mean squared error,
//                  backward to the FP32 master weights (the rounding is taken
//                  as identity); one share of the sums per workgroup
//  k_mlp_sum       the shares' sum and the Adam step on the master weights
//
// Layout of the parameter blob: see sssp_opts.k_model in include/pbh.h.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>

#include "../../include/pbh.h"
#include "pbh_core.h"

namespace bkt {

constexpr int H = MLP_H;
constexpr int F = NFEAT;
constexpr int OW1 = 0, OB1 = F * H, OW2 = OB1 + H, OB2 = OW2 + H * H, OW3 = OB2 + H, OB3 = OW3 + H;
constexpr int OMU = MLP_PARAMS, OSD = OMU + F, OSC = OSD + F;

__device__ __forceinline__ float gelu_d(float x) {
  // d/dx [x Phi(x)] = Phi(x) + x phi(x)
  const float phi = 0.3989422804014327f * expf(-0.5f * x * x);
  return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * phi;
}

// Every record names a query < nq, and every traced id (padding keys KINF
// aside) is a vertex of that query's graph; *bad != 0 otherwise.
__global__ void k_trace_check(const u64* tk, const u32* tv, const u32* tq, u32 count, const u32* dist_n, u32 nq,
                              u32* bad) {
  for (u32 r = blockIdx.x * blockDim.x + threadIdx.x; r < count; r += gridDim.x * blockDim.x) {
    const u32 q = tq[r];
    bool b = q >= nq;
    if (!b) {
      const u32 n = dist_n[q];
      for (int k = 0; k < TRACE_K; ++k)
        b = b || (tk[(u64)r * TRACE_K + k] != KINF && tv[(u64)r * TRACE_K + k] >= n);
    }
    if (b) atomicOr(bad, 1u);
  }
}

__global__ void k_trace_labels(const u64* tk, const u32* tv, const u32* tq, u32 count, const u64* const* dists,
                               float* labels) {
  for (u32 r = blockIdx.x * blockDim.x + threadIdx.x; r < count; r += gridDim.x * blockDim.x) {
    const u64* dist = dists[tq[r]];
    u32 k = 0;
    while (k < (u32)TRACE_K) {
      u64 key = tk[(u64)r * TRACE_K + k];
      if (key == KINF || dist[tv[(u64)r * TRACE_K + k]] != key) break;
      ++k;
    }
    labels[r] = log2f((float)(k < 1 ? 1 : k));
  }
}

// mu[f], sd[f] over n samples (one workgroup per feature).
__global__ void k_feat_stats(const float* X, u32 n, float* blob) {
  __shared__ double s1[256], s2[256];
  const int f = blockIdx.x;
  double a = 0, b = 0;
  for (u32 i = threadIdx.x; i < n; i += blockDim.x) {
    double x = X[(u64)i * F + f];
    a += x;
    b += x * x;
  }
  s1[threadIdx.x] = a;
  s2[threadIdx.x] = b;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      s1[threadIdx.x] += s1[threadIdx.x + o];
      s2[threadIdx.x] += s2[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double m = s1[0] / (n ? n : 1), v = s2[0] / (n ? n : 1) - m * m;
    blob[OMU + f] = (float)m;
    blob[OSD + f] = (float)sqrt(v > 1e-12 ? v : 1e-12);
  }
}

// One mini-batch of B samples X[idx0 .. idx0+B): each workgroup (256 threads)
// takes chunks of MS samples and leaves its share of the gradient of the mean
// squared error, and of the squared error itself, in
// part[blockIdx.x][0 .. MLP_PARAMS]; k_mlp_sum adds the shares.
//
// The three contractions over the hidden layer (z2 = h1 W2, dL/dh1 = dL/dz2
// W2^T, dL/dW2 = h1^T dL/dz2) run on the matrix cores in float32
// (16x16x4 tiles: products and sums stay 32-bit); wavefront w owns the columns
// [16w, 16w + 16) of the first two and the rows [16w, 16w + 16) of the last,
// whose accumulators stay in registers over all chunks.  z2, its GELU and
// their gradients stay in the registers of the lanes that computed them; rows
// are LD = 68 floats apart in LDS, which spreads a column of 16 rows and 4
// consecutive elements over all 64 banks.  Each share is a sum over at most
// B / gridDim samples, so a parameter's sum is a tree and not one chain of B.
//
// Bound by the chain of a chunk's steps and the launches: 24 us a step of 1,024
// samples (32 workgroups; 15 us here, 5 us in k_mlp_sum, the rest between the
// launches), 2.9 ms by one workgroup with a sample per thread and activations
// in global memory.  The gradient's error against float64 is 3e-8 - 6e-8; one
// chain of B additions per parameter has 2e-7 - 9e-7.
constexpr int MS = 32;   // samples per chunk
constexpr int LD = 68;   // LDS row stride of the 64-wide arrays
constexpr u32 GRAD_GRID = 256;             // most workgroups of k_mlp_grad
constexpr int PART = MLP_PARAMS + 1;       // a share: the gradient, then the squared error
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float sum16(float x) {  // over the 16 lanes of a row of the tile
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) x += __shfl_xor(x, o, 64);
  return x;
}
__device__ __forceinline__ float sum_rows(float x) {  // over the four row groups (lanes l, l+16, l+32, l+48)
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}

__global__ __launch_bounds__(256) void k_mlp_grad(const float* blob, const float* X, const float* Y, u32 idx0, u32 B,
                                                  float* part) {
  __shared__ float w1[F * H], b1[H], w2[H * LD], xs[MS * F];
  __shared__ float h1[MS * LD], z1[MS * LD], dz[MS * LD];  // z1: later dL/dz1; dz: dL/dz2
  __shared__ float ys[4 * MS], dys[MS];
  const int t = (int)threadIdx.x, l = t & 63, w = t >> 6, lc = l & 15, lk = l >> 4;
  for (int i = t; i < F * H; i += 256) w1[i] = bf16r(blob[OW1 + i]);
  for (int i = t; i < H * H; i += 256) w2[(i / H) * LD + i % H] = bf16r(blob[OW2 + i]);
  if (t < H) b1[t] = bf16r(blob[OB1 + t]);
  const int col = 16 * w + lc;  // this lane's column (hidden unit)
  const float b2c = bf16r(blob[OB2 + col]), w3c = bf16r(blob[OW3 + col]), b3 = bf16r(blob[OB3]);
  const float muf = blob[OMU + (t & (F - 1))], sdf = blob[OSD + (t & (F - 1))];
  f32x4 gw2[4] = {};
  float gw1[2] = {0.f, 0.f}, gb1 = 0.f, gb2 = 0.f, gw3 = 0.f, gb3 = 0.f;
  double lsum = 0.0;
  const u32 nch = (B + MS - 1) / MS;
  for (u32 ch = blockIdx.x; ch < nch; ch += gridDim.x) {
    const u32 s0 = ch * MS, ns = B - s0 < (u32)MS ? B - s0 : (u32)MS;
    static_assert(MS * F == 256, "one feature per thread");
    xs[t] = (u32)(t / F) < ns ? (X[(u64)(idx0 + s0) * F + t] - muf) / sdf : 0.f;
    __syncthreads();
    {
      const int j = t & (H - 1);
      for (int s = t / H; s < MS; s += 256 / H) {
        float a = b1[j];
#pragma unroll
        for (int f = 0; f < F; ++f) a += w1[f * H + j] * xs[s * F + f];
        z1[s * LD + j] = a;
        h1[s * LD + j] = gelu(a);
      }
    }
    __syncthreads();
    // z2 (this lane: column col, rows 16 rt + 4 lk + r)
    f32x4 z2[2] = {};
#pragma unroll
    for (int k = 0; k < H / 4; ++k) {
      const float b = w2[(4 * k + lk) * LD + col];
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
        z2[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(h1[(16 * rt + lc) * LD + 4 * k + lk], b, z2[rt], 0, 0, 0);
    }
    float h2[2][4];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        z2[rt][r] += b2c;
        h2[rt][r] = gelu(z2[rt][r]);
        const float y = sum16(w3c * h2[rt][r]);
        if (lc == 0) ys[w * MS + 16 * rt + 4 * lk + r] = y;
      }
    __syncthreads();
    if (t < MS) {
      const float y = b3 + ((ys[t] + ys[MS + t]) + (ys[2 * MS + t] + ys[3 * MS + t]));
      const float e = (u32)t < ns ? y - Y[idx0 + s0 + t] : 0.f;
      const float dy = 2.f * e / (float)B;
      dys[t] = dy;
      lsum += (double)e * e;
      gb3 += dy;
    }
    __syncthreads();
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * rt + 4 * lk + r;
        const float dy = dys[row], g = dy * w3c * gelu_d(z2[rt][r]);
        dz[row * LD + col] = g;
        gb2 += g;
        gw3 += dy * h2[rt][r];
      }
    __syncthreads();
    f32x4 dh[2] = {};  // dL/dh1
#pragma unroll
    for (int k = 0; k < H / 4; ++k) {
      const float b = w2[col * LD + 4 * k + lk];
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
        dh[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(dz[(16 * rt + lc) * LD + 4 * k + lk], b, dh[rt], 0, 0, 0);
    }
#pragma unroll
    for (int k = 0; k < MS / 4; ++k) {
      const float a = h1[(4 * k + lk) * LD + col];
#pragma unroll
      for (int c = 0; c < 4; ++c)
        gw2[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, dz[(4 * k + lk) * LD + 16 * c + lc], gw2[c], 0, 0, 0);
    }
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int x = (16 * rt + 4 * lk + r) * LD + col;
        const float g = dh[rt][r] * gelu_d(z1[x]);
        z1[x] = g;
        gb1 += g;
      }
    __syncthreads();
    {
      const int j = t & (H - 1), f = t / H;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        float a = 0.f;
        for (int s = 0; s < MS; ++s) a += xs[s * F + f + 4 * q] * z1[s * LD + j];
        gw1[q] += a;
      }
    }
    __syncthreads();
  }
  float* o = part + (u64)blockIdx.x * PART;
#pragma unroll
  for (int q = 0; q < 2; ++q) o[OW1 + (t / H + 4 * q) * H + (t & (H - 1))] = gw1[q];
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) o[OW2 + (16 * w + 4 * lk + r) * H + 16 * c + lc] = gw2[c][r];
  gb1 = sum_rows(gb1);
  gb2 = sum_rows(gb2);
  gw3 = sum_rows(gw3);
  if (lk == 0) {
    o[OB1 + col] = gb1;
    o[OB2 + col] = gb2;
    o[OW3 + col] = gw3;
  }
  if (w == 0) {  // lanes >= MS hold zeros
    gb3 = sum_rows(sum16(gb3));
    for (int o = 1; o < 64; o <<= 1) lsum += __shfl_xor(lsum, o, 64);
    if (l == 0) {
      o[OB3] = gb3;
      o[MLP_PARAMS] = (float)lsum;
    }
  }
}

// Adds the g shares of a batch of B samples: the gradient to grad (if set)
// and the mean squared error to loss[0]; with m set, takes the Adam step
// (Kingma & Ba 2015) on the master weights as well, c1 and c2 being the
// step's bias corrections.
__global__ __launch_bounds__(256) void k_mlp_sum(const float* part, u32 g, u32 B, float* grad, float* loss,
                                                 float* blob, float* m, float* v, float lr, float b1, float b2,
                                                 float eps, float c1, float c2) {
  const int p = (int)(blockIdx.x * 256 + threadIdx.x);
  if (p >= PART) return;
  constexpr int U = 8;  // shares in flight
  float s[U] = {};
  u32 i = 0;
  for (; i + U <= g; i += U)
#pragma unroll
    for (int q = 0; q < U; ++q) s[q] += part[(u64)(i + q) * PART + p];
  for (; i < g; ++i) s[0] += part[(u64)i * PART + p];
  const float a = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
  if (p == MLP_PARAMS) {
    loss[0] = a / (float)B;
    return;
  }
  if (grad) grad[p] = a;
  if (m) {
    m[p] = b1 * m[p] + (1.f - b1) * a;
    v[p] = b2 * v[p] + (1.f - b2) * a * a;
    blob[p] -= lr * (m[p] / c1) / (sqrtf(v[p] / c2) + eps);
  }
}

u32 grad_grid(u32 B) {
  const u32 nch = (B + MS - 1) / MS;
  return nch < GRAD_GRID ? nch : GRAD_GRID;
}

// Final rounding of the trained weights to bfloat16 values.
__global__ void k_round_bf16(float* blob) {
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < MLP_PARAMS; p += gridDim.x * blockDim.x)
    blob[p] = bf16r(blob[p]);
}

}  // namespace bkt

using namespace bkt;

namespace {
thread_local char g_lerr[256] = "";
std::mutex g_learn_mu;
}

#define LCHK(expr)                                                                   \
  do {                                                                               \
    hipError_t e_ = (expr);                                                          \
    if (e_ != hipSuccess) {                                                          \
      snprintf(g_lerr, sizeof g_lerr, "%s: %s", #expr, hipGetErrorString(e_));       \
      return e_ == hipErrorOutOfMemory ? PBH_ENOMEM : PBH_EDEVICE;                   \
    }                                                                                \
  } while (0)

extern "C" {

int mlp_trace_labels(const uint64_t* trace_keys, const uint32_t* trace_ids, const uint32_t* trace_query,
                     uint32_t count, const uint64_t* const* dists, const uint32_t* dist_n, uint32_t nq,
                     float* labels) {
  if (count == 0) return PBH_OK;
  if (!trace_keys || !trace_ids || !trace_query || !dists || !dist_n || nq == 0 || !labels) return PBH_EINVAL;
  u32 grid = (count + 255) / 256;
  grid = grid > 4096 ? 4096 : grid;
  std::lock_guard<std::mutex> lock(g_learn_mu);
  u32* bad = nullptr;
  LCHK(hipMalloc(&bad, sizeof(u32)));
  u32 hbad = 0;
  hipError_t e = hipMemset(bad, 0, sizeof(u32));
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_trace_check, dim3(grid), dim3(256), 0, 0, (const u64*)trace_keys, trace_ids, trace_query,
                       count, dist_n, nq, bad);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpy(&hbad, bad, sizeof(u32), hipMemcpyDeviceToHost);
  (void)hipFree(bad);
  LCHK(e);
  if (hbad) {
    snprintf(g_lerr, sizeof g_lerr, "mlp_trace_labels: a record names a query >= nq or an id >= its n");
    return PBH_EINVAL;
  }
  hipLaunchKernelGGL(k_trace_labels, dim3(grid), dim3(256), 0, 0, (const u64*)trace_keys, trace_ids, trace_query,
                     count, (const u64* const*)dists, labels);
  LCHK(hipGetLastError());
  LCHK(hipDeviceSynchronize());
  return PBH_OK;
}

int mlp_feature_stats(const float* X, uint32_t n, float* blob) {
  if (!X || !blob || n == 0) return PBH_EINVAL;
  hipLaunchKernelGGL(k_feat_stats, dim3(F), dim3(256), 0, 0, X, n, blob);
  LCHK(hipGetLastError());
  LCHK(hipDeviceSynchronize());
  return PBH_OK;
}

int mlp_grad(const float* X, const float* Y, uint32_t n, const float* blob, float* grad, float* loss) {
  if (!X || !Y || !blob || !grad || !loss || n == 0 || n > (1u << 16)) return PBH_EINVAL;
  std::lock_guard<std::mutex> lock(g_learn_mu);
  float* part = nullptr;
  const u32 g = grad_grid(n);
  LCHK(hipMalloc(&part, (size_t)g * PART * sizeof(float)));
  hipLaunchKernelGGL(k_mlp_grad, dim3(g), dim3(256), 0, 0, blob, X, Y, 0u, n, part);
  hipLaunchKernelGGL(k_mlp_sum, dim3((PART + 255) / 256), dim3(256), 0, 0, part, g, n, grad, loss, (float*)nullptr,
                     (float*)nullptr, (float*)nullptr, 0.f, 0.f, 0.f, 0.f, 1.f, 1.f);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipDeviceSynchronize();
  (void)hipFree(part);
  LCHK(e);
  return PBH_OK;
}

int mlp_train(const float* X, const float* Y, uint32_t n, float* blob, uint32_t batch, uint32_t steps, float lr,
              float* loss_trace) {
  if (!X || !Y || !blob || n == 0 || batch == 0 || batch > 4096) return PBH_EINVAL;
  std::lock_guard<std::mutex> lock(g_learn_mu);
  if (batch > n) batch = n;
  // one block: the shares, the Adam moments (cleared), the losses
  float* buf = nullptr;
  const u32 g = grad_grid(batch);
  const size_t np = (size_t)g * PART, nl = steps ? steps : 1;
  hipError_t e = hipMalloc(&buf, (np + 2 * MLP_PARAMS + nl) * sizeof(float));
  LCHK(e);
  float *part = buf, *m = buf + np, *v = m + MLP_PARAMS, *loss = v + MLP_PARAMS;
  e = hipMemset(m, 0, 2 * MLP_PARAMS * sizeof(float));
  const u32 nb = n / batch;
  for (u32 t = 0; e == hipSuccess && t < steps; ++t) {
    u32 idx0 = (t % nb) * batch;
    hipLaunchKernelGGL(k_mlp_grad, dim3(g), dim3(256), 0, 0, blob, X, Y, idx0, batch, part);
    hipLaunchKernelGGL(k_mlp_sum, dim3((PART + 255) / 256), dim3(256), 0, 0, part, g, batch, (float*)nullptr, loss + t,
                       blob, m, v, lr, 0.9f, 0.999f, 1e-8f, (float)(1.0 - std::pow((double)0.9f, t + 1.0)),
                       (float)(1.0 - std::pow((double)0.999f, t + 1.0)));
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_round_bf16, dim3((MLP_PARAMS + 255) / 256), dim3(256), 0, 0, blob);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e == hipSuccess && loss_trace && steps)
    e = hipMemcpy(loss_trace, loss, steps * sizeof(float), hipMemcpyDeviceToHost);
  (void)hipFree(buf);
  LCHK(e);
  return PBH_OK;
}

}  // extern "C"
