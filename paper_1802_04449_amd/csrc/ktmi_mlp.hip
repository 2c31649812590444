// ktmi_mlp.hip -- forward, gradient and Adam kernels of the learned root-solve
// guess (network in ktmi_mlp.hpp) and their C ABI.  Training runs on the GPU:
// forward (FP32, or BF16 for the 32x32 layer) and FP32 backward on the matrix
// cores; each wave sweeps a fixed set of 64-sample chunks into accumulators, its
// workgroup adds its four waves in order, then one kernel folds the workgroups in
// a fixed order (bitwise reproducible), then Adam.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "../../include/ktmi.h"
#include "ktmi_mlp.hpp"

namespace ktmi {

constexpr int kMlpBlock = 128;                 // samples per workgroup record (mlp_grid)
constexpr int kGradWaves = 4;                  // waves per workgroup of the gradient kernel
constexpr int kMlpGrid = 512;                  // workgroups of the gradient kernel (at most)
constexpr int kMlpSlots = kMlpNParam + 2;      // gradient sums, loss sum, sample count

__device__ __forceinline__ void load_w2bf(const float* __restrict__ prm, uint16_t* w2bf) {
  for (int k = threadIdx.x; k < kMlpH * kMlpH; k += blockDim.x)
    w2bf[k] = (uint16_t)to_bf16(prm[kOW2 + k]);
  __syncthreads();
}

__device__ __forceinline__ bool mlp_sample_ok(double E, double M, double emin) {
  return E >= emin && E < 1e300 && M >= 0.0 && M < 1e300;
}

// guess[i] for n samples (E, M); MODE 0 FP32, 1 BF16 matrix cores.  Samples
// with E < emin (or non-finite) get guess = E.
template <int MODE>
__global__ __launch_bounds__(256) void k_mlp_forward(const float* __restrict__ prm, int n,
                                                     const double* __restrict__ E,
                                                     const double* __restrict__ M, double emin,
                                                     double* __restrict__ guess) {
  __shared__ uint16_t w2bf[kMlpH * kMlpH];
  if (MODE == 1) load_w2bf(prm, w2bf);
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  const double e = s < n ? E[s] : 1.0, m = s < n ? M[s] : 0.0;
  const bool ok = s < n && mlp_sample_ok(e, m, emin);
  const double ee = ok ? e : 1.0, mm = ok ? m : 0.0;
  double g;
  if (MODE == 1) {
    g = mlp_guess_wave(prm, w2bf, ee, mm * mm);
  } else {
    g = mlp_guess_lane(prm, ee, mm * mm);
  }
  if (s < n) guess[s] = ok ? g : e;
}

// Unit held by accumulator register r of a 32 x 32 matrix-core result in half h = l / 32.
__device__ __forceinline__ constexpr int mlp_unit(int r, int h) {
  return 8 * (r >> 2) + 4 * h + (r & 3);
}

// Orders the wave's LDS writes before its reads by other lanes (LDS serves one wave's
// instructions in order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A wave's LDS: two 32 x 32 transposes (rows padded to 36: 16-byte aligned and free of
// bank conflicts both ways), the features and dz of its 64 samples.
struct GradLds {
  float X[kMlpH][36], Y[kMlpH][36];
  float F[4][64];
  float Dz[64];
};
static_assert(sizeof(GradLds) >= kMlpSlots * sizeof(float), "a wave's record fits its area");

// Gradient sums of the loss ((guess - e)/E)^2 over the samples with E >= emin,
// plus the loss sum and the sample count, per workgroup: part[block][slot].
//
// A wave takes 64 samples at a time: features and loss (FP64) once per lane, the
// network for two blocks of 32 samples on the matrix cores.  v_mfma_f32_32x32x2_f32
// (lane l holds A[l % 32][l / 32] and B[l / 32][l % 32], its results are rows
// mlp_unit(r, l / 32) of column l % 32) runs with units as rows and samples as columns,
// so every layer's result is the next one's B operand as it stands: step r contracts
// over the two units mlp_unit(r, 0) and mlp_unit(r, 1) that the lane halves hold.  Only
// the weight gradients, which contract over samples, need units and samples exchanged
// through LDS.  FP32 products and sums throughout (v_mfma_f32_32x32x8_bf16 for the
// 32 x 32 layer's forward in MODE 1).  Bound by FP32 matrix-core time (52 products of 64
// clocks per 32 samples, 42 us for 1e6 samples) next to about as much VALU work, at two
// waves per SIMD (256 registers, 11-20 spilled; one wave without the bound).  Kernel
// trace, gradient + fold: 8192 samples 206 -> 11.6 + 3.7 us (FP32), 1e6 3645 -> 84 + 12 us (BF16
// forward; its matrix cores busy 36% of the time); a whole Adam step without the profiler
// 187 -> 16 and 3370 -> 91 us.  One sample per lane with LDS sums over 128 samples, as it was,
// left the matrix cores idle and read 2 x 128 LDS values for each of the 1249 sums and chunk.
template <int MODE>
__global__ __launch_bounds__(64 * kGradWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mlp_grad(const float* __restrict__ prm, int n,
                                                             const double* __restrict__ E,
                                                             const double* __restrict__ M,
                                                             const double* __restrict__ eps,
                                                             double emin, float* __restrict__ part) {
  __shared__ GradLds lds[kGradWaves];
  const int l = threadIdx.x & 63, wave = threadIdx.x >> 6, half = l >> 5, c = l & 31;
  GradLds& w = lds[wave];
  // operands of the products: W2 for the forward (FP32 or BF16), W2^T for the backward,
  // W1 with b1 as a fifth feature, b2 as a last contraction step
  float wf[16], wb[16], w3[16];
  bf16x4 wf16[4];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int u = mlp_unit(r, half);
    wf[r] = prm[kOW2 + c * kMlpH + u];
    wb[r] = prm[kOW2 + u * kMlpH + c];
    w3[r] = prm[kOW3 + u];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int j = 0; j < 4; ++j) wf16[k][j] = (short)to_bf16(wf[4 * k + j]);
  const float w1a = prm[kOW1 + c * 4 + half], w1b = prm[kOW1 + c * 4 + 2 + half];
  const float one = half ? 0.0f : 1.0f;
  const float b1 = half ? 0.0f : prm[kOB1 + c], b2 = half ? 0.0f : prm[kOB2 + c];
  const float b3 = prm[kOB3];
  // accumulators: W2 as matrix-core results; of unit c over this half's samples: W1's
  // row, b1, b2, w3; of this lane's samples: b3, loss, count
  float gW2[16], gW1[4] = {0.0f, 0.0f, 0.0f, 0.0f}, gb1 = 0.0f, gb2 = 0.0f, gw3 = 0.0f;
  double gb3 = 0.0, loss = 0.0, cnt = 0.0;
#pragma unroll
  for (int r = 0; r < 16; ++r) gW2[r] = 0.0f;
  const int nchunk = (int)(((long)n + 63) / 64);
  for (int ch = blockIdx.x * kGradWaves + wave; ch < nchunk; ch += gridDim.x * kGradWaves) {
    const int s = ch * 64 + l;
    const double e = s < n ? E[s] : 1.0, m = s < n ? M[s] : 0.0;
    const bool ok = s < n && mlp_sample_ok(e, m, emin);
    const double ee = ok ? e : 1.0, mm = ok ? m : 0.0, target = ok ? eps[s] : 0.5;
    float f[4];
    double lo;
    mlp_features(ee, mm * mm, f, lo);
#pragma unroll
    for (int k = 0; k < 4; ++k) w.F[k][l] = f[k];
    wave_lds_sync();
    float h1[2][16], h2[2][16], zb[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      f32x16 a = {};
      a = __builtin_amdgcn_mfma_f32_32x32x2f32(b1, one, a, 0, 0, 0);
      a = __builtin_amdgcn_mfma_f32_32x32x2f32(w1a, w.F[half][32 * b + c], a, 0, 0, 0);
      a = __builtin_amdgcn_mfma_f32_32x32x2f32(w1b, w.F[2 + half][32 * b + c], a, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 16; ++r) h1[b][r] = mlp_tanh(a[r]);
      a = f32x16{};
      if (MODE == 1) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          bf16x4 h;
#pragma unroll
          for (int j = 0; j < 4; ++j) h[j] = (short)to_bf16(h1[b][4 * k + j]);
          a = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(wf16[k], h, a, 0, 0, 0);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          a = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[r], h1[b][r], a, 0, 0, 0);
      }
      a = __builtin_amdgcn_mfma_f32_32x32x2f32(b2, one, a, 0, 0, 0);
      float z = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        h2[b][r] = mlp_tanh(a[r]);
        z += w3[r] * h2[b][r];
      }
      zb[b] = b3 + (z + __shfl_xor(z, 32, 64));
    }
    // loss and its derivative in z of this lane's own sample (32 half + c)
    const double sg = 1.0 / (1.0 + exp(-(double)(half ? zb[1] : zb[0])));
    const double r = (ee - lo) / ee;
    const double t = ee > lo ? (target - lo) / (ee - lo) : 0.0;
    const double d = r * (sg - t);
    const float dz = ok ? (float)(2.0 * d * r * sg * (1.0 - sg)) : 0.0f;
    gb3 += dz;
    loss += ok ? d * d : 0.0;
    cnt += ok ? 1.0 : 0.0;
    w.Dz[l] = dz;
    wave_lds_sync();
    f32x16 aw = {};
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const float dzc = w.Dz[32 * b + c];
      f32x16 a = {};
#pragma unroll
      for (int r2 = 0; r2 < 16; ++r2) {
        const float d2 = dzc * w3[r2] * (1.0f - h2[b][r2] * h2[b][r2]);
        w.X[mlp_unit(r2, half)][c] = d2;
        w.Y[mlp_unit(r2, half)][c] = h1[b][r2];
        a = __builtin_amdgcn_mfma_f32_32x32x2f32(wb[r2], d2, a, 0, 0, 0);  // W2^T d2
      }
      wave_lds_sync();
      // dW2 += d2 h1^T, db2 += d2: unit c, samples 16 half + 0..15 of the block
      float x[16], y[16], sum = 0.0f;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        x[q] = w.X[c][16 * half + q];
        y[q] = w.Y[c][16 * half + q];
      }
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        aw = __builtin_amdgcn_mfma_f32_32x32x2f32(x[q], y[q], aw, 0, 0, 0);
        sum += x[q];
      }
      gb2 += sum;
      wave_lds_sync();
      // d1 = (W2^T d2)(1 - h1^2): dW1 += d1 f^T, db1 += d1; dw3 += dz h2
#pragma unroll
      for (int r2 = 0; r2 < 16; ++r2) {
        w.X[mlp_unit(r2, half)][c] = a[r2] * (1.0f - h1[b][r2] * h1[b][r2]);
        w.Y[mlp_unit(r2, half)][c] = h2[b][r2];
      }
      wave_lds_sync();
      float s1 = 0.0f, s3 = 0.0f, sw[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int sq = 32 * b + 16 * half + q;
        const float d1 = w.X[c][16 * half + q];
        s1 += d1;
        s3 += w.Dz[sq] * w.Y[c][16 * half + q];
#pragma unroll
        for (int k = 0; k < 4; ++k) sw[k] += d1 * w.F[k][sq];
      }
      gb1 += s1;
      gw3 += s3;
#pragma unroll
      for (int k = 0; k < 4; ++k) gW1[k] += sw[k];
      wave_lds_sync();
    }
#pragma unroll
    for (int r2 = 0; r2 < 16; ++r2) gW2[r2] += aw[r2];
  }
  // the wave's record in its own LDS area, then the workgroup's in wave order
  gb1 += __shfl_xor(gb1, 32, 64);
  gb2 += __shfl_xor(gb2, 32, 64);
  gw3 += __shfl_xor(gw3, 32, 64);
#pragma unroll
  for (int k = 0; k < 4; ++k) gW1[k] += __shfl_xor(gW1[k], 32, 64);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    gb3 += __shfl_xor(gb3, off, 64);
    loss += __shfl_xor(loss, off, 64);
    cnt += __shfl_xor(cnt, off, 64);
  }
  float* rec = (float*)&w;
#pragma unroll
  for (int r2 = 0; r2 < 16; ++r2) rec[kOW2 + mlp_unit(r2, half) * kMlpH + c] = gW2[r2];
  if (half == 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) rec[kOW1 + c * 4 + k] = gW1[k];
    rec[kOB1 + c] = gb1;
    rec[kOB2 + c] = gb2;
    rec[kOW3 + c] = gw3;
  }
  if (l == 0) {
    rec[kOB3] = (float)gb3;
    rec[kMlpNParam] = (float)loss;
    rec[kMlpNParam + 1] = (float)cnt;
  }
  __syncthreads();
  float* out = part + (size_t)blockIdx.x * kMlpSlots;
  for (int k = threadIdx.x; k < kMlpSlots; k += 64 * kGradWaves) {
    float a = ((const float*)&lds[0])[k];
#pragma unroll
    for (int v = 1; v < kGradWaves; ++v) a += ((const float*)&lds[v])[k];
    out[k] = a;
  }
}

// out[p] = (sum over workgroups of part[.][p]) / count; out[kMlpNParam] = mean loss,
// out[kMlpNParam + 1] = count.  A workgroup folds kFoldP slots: row r adds records
// r, r + kFoldRows, ... in order, then the rows are added in order (the count the same
// way), so the chain of dependent additions is 1 / kFoldRows of the records (512
// records: 138 us one after the other, 12 us so).
constexpr int kFoldP = 16, kFoldRows = 32;
__global__ __launch_bounds__(kFoldP* kFoldRows) void k_mlp_fold(const float* __restrict__ part,
                                                                int nblk, float* __restrict__ out) {
  __shared__ double sh[kFoldRows][kFoldP + 1];
  const int q = threadIdx.x % kFoldP, row = threadIdx.x / kFoldP;
  const int p = blockIdx.x * kFoldP + q;
  double acc = 0.0, cnt = 0.0;
  for (int b = row; b < nblk; b += kFoldRows) {
    const float* rec = part + (size_t)b * kMlpSlots;
    acc += p < kMlpSlots ? rec[p] : 0.0f;
    if (q == 0) cnt += rec[kMlpNParam + 1];
  }
  sh[row][q] = acc;
  if (q == 0) sh[row][kFoldP] = cnt;
  __syncthreads();
  if (row != 0 || p >= kMlpSlots) return;
  acc = cnt = 0.0;
  for (int r = 0; r < kFoldRows; ++r) {
    acc += sh[r][q];
    cnt += sh[r][kFoldP];
  }
  out[p] = p == kMlpNParam + 1 ? (float)cnt : (cnt > 0.0 ? (float)(acc / cnt) : 0.0f);
}

// Adam (Kingma & Ba): bias-corrected first and second moments, t from 1.
__global__ void k_mlp_adam(float* __restrict__ prm, const float* __restrict__ g,
                           float* __restrict__ m, float* __restrict__ v, float c1, float c2,
                           float lr, float b1, float b2, float epsilon) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= kMlpNParam) return;
  const float gp = g[p];
  const float mp = b1 * m[p] + (1.0f - b1) * gp;
  const float vp = b2 * v[p] + (1.0f - b2) * gp * gp;
  m[p] = mp;
  v[p] = vp;
  prm[p] -= lr * (mp / c1) / (sqrtf(vp / c2) + epsilon);
}

// Records (workgroups of the gradient kernel) of n samples: one per kMlpBlock samples.
static int mlp_grid(int n) {
  const int nchunk = (int)(((long)n + kMlpBlock - 1) / kMlpBlock);
  return nchunk < kMlpGrid ? nchunk : kMlpGrid;
}

// Largest sample count: the gradient kernel indexes samples with 32-bit ints
// (chunk * kMlpBlock + thread), which stay below 2^31 up to this n.
constexpr int kMlpMaxSamples = 0x7fffffff - kMlpBlock;

// Scratch of ktmi_mlp_grad_noalloc: the partial sums of the gradient kernel's
// workgroups (at most kMlpGrid records of kMlpSlots floats, 2.56 MB).  One copy
// per GPU, held until the process ends.  Its name is a host-side stand-in in
// host code: kernels get the device address from hipGetSymbolAddress.
constexpr size_t kMlpScratchFloats = (size_t)kMlpGrid * kMlpSlots;
static __device__ __align__(256) float scratch[kMlpScratchFloats];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static float* g_scratch_ptr[kMaxDevices];  // device address of scratch on each GPU

// Device address of scratch on the current GPU, looked up once per device.
static int scratch_on_current_device(float** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return KTMI_EHIP;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return KTMI_EHIP;
    g_scratch_ptr[dev] = (float*)p;
  }
  *out = g_scratch_ptr[dev];
  return KTMI_OK;
}

// Gradient kernel, then the fixed-order fold of its workgroups, into out.
static int launch_mlp_grad(const float* params, int n, const double* E, const double* M,
                           const double* eps, double emin, int mode, float* out, float* part,
                           hipStream_t s) {
  // four waves of 64 samples per workgroup: a record per 256 samples, at most mlp_grid(n)
  // (all kMlpGrid records from 131 000 samples on)
  const int nblk = std::min(mlp_grid(n), (int)(((long)n + 64 * kGradWaves - 1) / (64 * kGradWaves)));
  const dim3 grid(nblk), block(64 * kGradWaves);
  if (mode == KTMI_MLP_BF16)
    hipLaunchKernelGGL(k_mlp_grad<1>, grid, block, 0, s, params, n, E, M, eps, emin, part);
  else
    hipLaunchKernelGGL(k_mlp_grad<0>, grid, block, 0, s, params, n, E, M, eps, emin, part);
  hipLaunchKernelGGL(k_mlp_fold, dim3((kMlpSlots + kFoldP - 1) / kFoldP), dim3(kFoldP * kFoldRows),
                     0, s, part, nblk, out);
  return hipGetLastError() == hipSuccess ? KTMI_OK : KTMI_EHIP;
}

}  // namespace ktmi

using namespace ktmi;

extern "C" {

int ktmi_mlp_nparam(void) { return kMlpNParam; }

int ktmi_mlp_forward(const float* params, int n, const double* E, const double* M, double emin,
                     double* guess, int mode, void* stream) {
  if (!params || n < 0 || (n && (!E || !M || !guess)) || (mode != KTMI_MLP_FP32 &&
                                                         mode != KTMI_MLP_BF16))
    return KTMI_EINVAL;
  if (n == 0) return KTMI_OK;
  const dim3 grid((n + 255) / 256), block(256);
  hipStream_t s = (hipStream_t)stream;
  if (mode == KTMI_MLP_BF16)
    hipLaunchKernelGGL(k_mlp_forward<1>, grid, block, 0, s, params, n, E, M, emin, guess);
  else
    hipLaunchKernelGGL(k_mlp_forward<0>, grid, block, 0, s, params, n, E, M, emin, guess);
  return hipGetLastError() == hipSuccess ? KTMI_OK : KTMI_EHIP;
}

size_t ktmi_mlp_grad_workspace_bytes(int n) {
  if (n < 1) return 0;
  return (size_t)mlp_grid(n) * kMlpSlots * sizeof(float);
}

int ktmi_mlp_grad(const float* params, int n, const double* E, const double* M, const double* eps,
                  double emin, int mode, float* out, void* ws, size_t bytes, void* stream) {
  if (!params || n < 1 || !E || !M || !eps || !out || !ws ||
      (mode != KTMI_MLP_FP32 && mode != KTMI_MLP_BF16))
    return KTMI_EINVAL;
  if (n > kMlpMaxSamples || bytes < ktmi_mlp_grad_workspace_bytes(n)) return KTMI_EINVAL;
  return launch_mlp_grad(params, n, E, M, eps, emin, mode, out, (float*)ws, (hipStream_t)stream);
}

int ktmi_mlp_grad_noalloc(const float* params, int n, const double* E, const double* M,
                          const double* eps, double emin, int mode, float* out, void* stream) {
  if (!params || n < 1 || n > kMlpMaxSamples || !E || !M || !eps || !out ||
      (mode != KTMI_MLP_FP32 && mode != KTMI_MLP_BF16))
    return KTMI_EINVAL;
  // every sample count fits: the kernel never runs more than kMlpGrid workgroups
  if ((size_t)mlp_grid(n) * kMlpSlots > kMlpScratchFloats) return KTMI_EINVAL;
  float* part = nullptr;
  const int rc = scratch_on_current_device(&part);
  if (rc != KTMI_OK) return rc;
  return launch_mlp_grad(params, n, E, M, eps, emin, mode, out, part, (hipStream_t)stream);
}

int ktmi_mlp_adam(float* params, const float* grad, float* m, float* v, int t, float lr, float b1,
                  float b2, float epsilon, void* stream) {
  if (!params || !grad || !m || !v || t < 1 || !(lr > 0.0f) || !(b1 >= 0.0f && b1 < 1.0f) ||
      !(b2 >= 0.0f && b2 < 1.0f) || !(epsilon > 0.0f))
    return KTMI_EINVAL;
  const float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
  hipLaunchKernelGGL(k_mlp_adam, dim3((kMlpNParam + 255) / 256), dim3(256), 0,
                     (hipStream_t)stream, params, grad, m, v, c1, c2, lr, b1, b2, epsilon);
  return hipGetLastError() == hipSuccess ? KTMI_OK : KTMI_EHIP;
}

}  // extern "C"
