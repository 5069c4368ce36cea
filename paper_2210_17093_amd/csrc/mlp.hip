// Learned warm start of the qsGW iteration: per-state features, a
// 16 -> 128 -> 128 -> 1 GELU network (FP32 master weights) with its forward
// pass, MSE gradient and Adam update, and the shifted, re-sorted starting
// orbitals.  The 128-wide layers run on the FP32 matrix-core GEMM engine; the
// rest are element-wise kernels and fixed-order reductions (deterministic).
#include "internal.hpp"

#include <algorithm>

namespace {

constexpr int kIn = 16, kHid = 128;
constexpr int64_t kOffW1 = 0, kOffB1 = kOffW1 + kHid * kIn, kOffW2 = kOffB1 + kHid,
                  kOffB2 = kOffW2 + kHid * kHid, kOffW3 = kOffB2 + kHid, kOffB3 = kOffW3 + kHid,
                  kNParams = kOffB3 + 1;
static_assert(kNParams == QSGW_MLP_NPARAMS, "parameter layout");

__device__ __forceinline__ float gelu(float z) {
  return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
}
__device__ __forceinline__ float gelu_grad(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) +
         z * 0.39894228040143268f * expf(-0.5f * z * z);
}

// Z = v + b[n] (kept for the backward pass), A = gelu(Z).
struct EpiBiasGelu {
  const float* b;
  float* Z;
  float* A;
  int64_t ld;
  __device__ __forceinline__ void operator()(int64_t, int64_t, int64_t m, int64_t n, double v,
                                             bool) const {
    const float z = (float)v + b[n];
    if (Z) Z[m * ld + n] = z;
    A[m * ld + n] = gelu(z);
  }
};

// dZ = v * gelu'(Z)
struct EpiGeluGrad {
  const float* Z;
  float* dZ;
  int64_t ld;
  __device__ __forceinline__ void operator()(int64_t, int64_t, int64_t m, int64_t n, double v,
                                             bool) const {
    dZ[m * ld + n] = (float)v * gelu_grad(Z[m * ld + n]);
  }
};

// Output layer, one wave per row: y = A2 . w3 + b3.
__device__ __forceinline__ float mlp_row_out(float a0, float a1, float w0, float w1, float b3) {
  float acc = a0 * w0 + a1 * w1;
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  return acc + b3;  // (lane 0)
}
__global__ void k_mlp_out(const float* A2, const float* w3, const float* b3, int64_t n, float* y) {
  const int64_t row = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= n) return;
  const float out = mlp_row_out(A2[row * kHid + lane], A2[row * kHid + lane + 64], w3[lane],
                                w3[lane + 64], b3[0]);
  if (lane == 0) y[row] = out;
}

// Output layer of a training step and everything its rows feed in one pass
// (each wave kOutRows / 4 rows, lane l columns l and l + 64):
//   y = A2 . w3 + b3, dy = 2 (y - t) / n, dZ2[b][j] = dy[b] w3[j] gelu'(Z2[b][j]),
// and this workgroup's share of the column sums, in FP64:
//   part[g] = [ sum dZ2 (128) | sum A2 dy (128) | sum dy (1) | sum (y - t)^2 (1) ].
// Bound by the launch and the row loads (6 MB at n = 4096).  32 rows a
// workgroup put 128 of them on the chip at the training minibatch of 4096; with
// one thread walking 1024 rows of a column the four column sums of a step took
// 0.92 ms, this kernel with its k_sum_cols takes about 20 us.
constexpr int kOutRows = 32;
constexpr int kOutCols = 2 * kHid + 2;
__global__ __launch_bounds__(256) void k_mlp_out_grad(const float* __restrict__ A2,
                                                      const float* __restrict__ Z2,
                                                      const float* __restrict__ w3,
                                                      const float* __restrict__ b3, int64_t n,
                                                      const float* __restrict__ t,
                                                      float* __restrict__ dZ2,
                                                      double* __restrict__ part) {
  constexpr int RW = kOutRows / 4;
  __shared__ double red[4][kOutCols];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * kOutRows + wave * RW;
  const float w0 = w3[lane], w1 = w3[lane + 64], b = b3[0];
  double s2[2] = {0.0, 0.0}, s3[2] = {0.0, 0.0}, sd = 0.0, sq = 0.0;
#pragma unroll
  for (int u = 0; u < RW; ++u) {
    const int64_t row = r0 + u;
    if (row >= n) break;  // (uniform over the wave)
    const float a0 = A2[row * kHid + lane], a1 = A2[row * kHid + lane + 64];
    const float z0 = Z2[row * kHid + lane], z1 = Z2[row * kHid + lane + 64];
    const float r = __shfl(mlp_row_out(a0, a1, w0, w1, b), 0, 64) - t[row];
    const float dy = 2.0f * r / (float)n;
    const float d0 = dy * w0 * gelu_grad(z0), d1 = dy * w1 * gelu_grad(z1);
    dZ2[row * kHid + lane] = d0;
    dZ2[row * kHid + lane + 64] = d1;
    s2[0] += (double)d0;
    s2[1] += (double)d1;
    s3[0] += (double)a0 * (double)dy;
    s3[1] += (double)a1 * (double)dy;
    sd += (double)dy;
    sq += (double)r * (double)r;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    red[wave][lane + 64 * h] = s2[h];
    red[wave][kHid + lane + 64 * h] = s3[h];
  }
  if (lane == 0) {
    red[wave][2 * kHid] = sd;
    red[wave][2 * kHid + 1] = sq;
  }
  __syncthreads();
  for (int c = threadIdx.x; c < kOutCols; c += 256)
    part[(int64_t)blockIdx.x * kOutCols + c] = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
}

// Column sums of a [n][128] matrix over rows [g R, (g + 1) R): part[g][col]
// (FP64), two row lanes per column.
constexpr int kColRows = 32;
__global__ __launch_bounds__(256) void k_col_partial(const float* __restrict__ A, int64_t n,
                                                     double* __restrict__ part) {
  __shared__ double red[kHid];
  const int c = threadIdx.x & (kHid - 1), h = threadIdx.x / kHid;
  const int64_t r0 = (int64_t)blockIdx.x * kColRows + h * (kColRows / 2);
  double s = 0.0;
#pragma unroll
  for (int u = 0; u < kColRows / 2; ++u)
    if (r0 + u < n) s += (double)A[(r0 + u) * kHid + c];
  if (h) red[c] = s;
  __syncthreads();
  if (!h) part[(int64_t)blockIdx.x * kHid + c] = s + red[c];
}

// out[i] (float) = sum_g part[g][i] of short rows and many groups (16 columns a
// workgroup, 16 group lanes each, fixed order); with `loss`, column len holds
// the squared errors and *loss = their sum / n.
__global__ __launch_bounds__(256) void k_sum_cols(const double* __restrict__ part, int64_t ng,
                                                  int ld, int len, float* __restrict__ out,
                                                  int64_t n, double* __restrict__ loss) {
  __shared__ double red[16][17];
  const int cl = threadIdx.x & 15, gl = threadIdx.x >> 4;
  const int i = blockIdx.x * 16 + cl;
  double s = 0.0;
  if (i < ld)
#pragma unroll 8
    for (int64_t g = gl; g < ng; g += 16) s += part[g * ld + i];
  red[gl][cl] = s;
  __syncthreads();
  if (gl == 0 && i < ld) {
    s = 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) s += red[u][cl];
    if (i < len)
      out[i] = (float)s;
    else if (loss)
      *loss = s / (double)n;
  }
}

// out[i] (float) = sum_z part[z][i] (fixed order)
__global__ void k_sum_parts(const double* part, int64_t nz, int64_t len, float* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= len) return;
  double s = 0.0;
#pragma unroll 8
  for (int64_t z = 0; z < nz; ++z) s += part[z * len + i];
  out[i] = (float)s;
}

// Adam (beta1 0.9, beta2 0.999, eps 1e-8) with bias correction for step t >= 1.
__global__ void k_adam(float* p, float* m, float* v, const float* g, int64_t len, float lr,
                       float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= len) return;
  const float gi = g[i];
  const float mi = 0.9f * m[i] + 0.1f * gi;
  const float vi = 0.999f * v[i] + 0.001f * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
}

// BF16 inference of the whole network, one workgroup (4 waves) per 64 rows,
// 16 rows per wave.  Every matrix operand is rounded to BF16 (nearest even):
// X, W1, the first hidden activations, W2, the second hidden activations and
// w3; products on v_mfma_f32_16x16x32_bf16 (layer 1's k = 16 padded to 32
// with zeros) with FP32 accumulation; biases and GELU in FP32; the output
// layer is an FP32 dot product of the BF16 values.  Fragments: lane l holds
// k = 8 (l / 16) .. + 7 of row l % 16 (A) or column l % 16 (B); accumulator
// element q of lane l is row 4 (l / 16) + q, column l % 16.
constexpr int kBfPitch = kHid + 8;  // LDS row pitch (272 bytes: 16-byte aligned rows)
__global__ __launch_bounds__(256) void k_mlp_forward_bf16(const float* __restrict__ P, int64_t n,
                                                          const float* __restrict__ X,
                                                          float* __restrict__ y) {
  __shared__ __attribute__((aligned(16))) __bf16 W2s[kHid * kBfPitch];
  __shared__ __attribute__((aligned(16))) __bf16 W1s[kHid * 40];
  __shared__ __attribute__((aligned(16))) __bf16 Hs[4][16 * kBfPitch];
  __shared__ float w3s[kHid];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int e = tid; e < kHid * kHid; e += 256)
    W2s[(e / kHid) * kBfPitch + (e % kHid)] = (__bf16)P[kOffW2 + e];
  for (int e = tid; e < kHid * 32; e += 256) {
    const int j = e / 32, k = e % 32;
    W1s[j * 40 + k] = k < kIn ? (__bf16)P[kOffW1 + j * kIn + k] : (__bf16)0.0f;
  }
  if (tid < kHid) w3s[tid] = (float)(__bf16)P[kOffW3 + tid];
  __syncthreads();
  const int64_t r0 = (int64_t)blockIdx.x * 64 + wave * 16;
  const int rl = lane & 15, kg = lane >> 4;
  // layer 1: A = X rows (k 0..15, zeros beyond)
  bf16x8 a;
  {
    const int64_t row = r0 + rl;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = 8 * kg + j;
      a[j] = (row < n && k < kIn) ? (__bf16)X[row * kIn + k] : (__bf16)0.0f;
    }
  }
  __bf16* H = Hs[wave];
#pragma unroll
  for (int jt = 0; jt < kHid / 16; ++jt) {
    const int col = jt * 16 + rl;
    const bf16x8 b = *reinterpret_cast<const bf16x8*>(&W1s[col * 40 + 8 * kg]);
    f32x4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    const float bias = P[kOffB1 + col];
#pragma unroll
    for (int q = 0; q < 4; ++q) H[(4 * kg + q) * kBfPitch + col] = (__bf16)gelu(acc[q] + bias);
  }
  __syncthreads();
  // layer 2 and the output layer
  float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int jt = 0; jt < kHid / 16; ++jt) {
    const int col = jt * 16 + rl;
    f32x4 acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < kHid / 32; ++ks) {
      const bf16x8 ha = *reinterpret_cast<const bf16x8*>(&H[rl * kBfPitch + ks * 32 + 8 * kg]);
      const bf16x8 wb = *reinterpret_cast<const bf16x8*>(&W2s[col * kBfPitch + ks * 32 + 8 * kg]);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ha, wb, acc, 0, 0, 0);
    }
    const float bias = P[kOffB2 + col];
#pragma unroll
    for (int q = 0; q < 4; ++q) part[q] += (float)(__bf16)gelu(acc[q] + bias) * w3s[col];
  }
  // sum over the 16 lanes of a row group (the columns), fixed pattern
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) part[q] += __shfl_xor(part[q], off, 64);
  if (rl == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t row = r0 + 4 * kg + q;
      if (row < n) y[row] = part[q] + P[kOffB3];
    }
  }
}

// Per-state features of the first iteration (see qsgw.h), standardized as
// (f - mean) / scale when mean is given.
__global__ void k_mlp_features(int64_t nbf, int64_t nocc, const double* eps, const double* diag,
                               const float* mean, const float* scale, float* X) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= nbf) return;
  const double e = eps[m], homo = eps[nocc - 1], lumo = eps[nocc];
  const double re = diag[m * 4 + 0], im = diag[m * 4 + 1], der = diag[m * 4 + 2],
               sx = diag[m * 4 + 3];
  const double z = 1.0 / (1.0 - der);
  double f[kIn];
  f[0] = e;
  f[1] = sx;
  f[2] = re;
  f[3] = der;
  f[4] = (double)nocc / (double)nbf;
  f[5] = lumo - homo;
  f[6] = im;
  f[7] = z;
  f[8] = m < nocc ? 1.0 : 0.0;
  f[9] = e - homo;
  f[10] = e - lumo;
  f[11] = (double)nbf / 120.0;
  f[12] = (double)m / (double)nbf;
  f[13] = z * re;
  f[14] = fabs(der) > 1.0 ? 1.0 : 0.0;
  f[15] = 1.0;
#pragma unroll
  for (int q = 0; q < kIn; ++q) {
    float x = (float)f[q];
    if (mean) x = (x - mean[q]) / scale[q];
    X[m * kIn + q] = x;
  }
}

// Warm start: e'_m = eps0_m + delta_m, stably sorted; perm[r] = state of rank r.
__global__ void k_warm_rank(int64_t nbf, const double* eps0, const float* delta, double* eps,
                            int64_t* perm) {
  for (int64_t m = threadIdx.x; m < nbf; m += blockDim.x) {
    const double em = eps0[m] + (double)delta[m];
    int64_t r = 0;
    for (int64_t j = 0; j < nbf; ++j) {
      const double ej = eps0[j] + (double)delta[j];
      r += (ej < em || (ej == em && j < m)) ? 1 : 0;
    }
    eps[r] = em;
    perm[r] = m;
  }
}

// C[:, r] = C0[:, perm[r]]
__global__ void k_warm_permute(int64_t nbf, const double* C0, const int64_t* perm, double* C) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nbf * nbf) return;
  const int64_t row = idx / nbf, r = idx - row * nbf;
  C[idx] = C0[row * nbf + perm[r]];
}

struct MlpBuffers {
  float *Z1, *A1, *Z2, *A2, *dZ2, *dZ1, *grad;
  double *part, *opart, *cpart;
};

// nz = 0: inference buffers only.
int mlp_buffers(qsgw_ctx* c, int64_t n, int64_t nz, MlpBuffers* b) {
  float* f = nullptr;
  double* d = nullptr;
  const int64_t og = (n + kOutRows - 1) / kOutRows, cg = (n + kColRows - 1) / kColRows;
  const size_t nf = (size_t)(6 * n * kHid + kNParams + 64);
  const size_t ndd = (size_t)(nz > 0 ? nz * kHid * kHid + og * kOutCols + cg * kHid : 1);
  CHECK(ws_get(c, W_MLP_F32, nf, &f));
  CHECK(ws_get(c, W_MLP_F64, ndd, &d));
  b->Z1 = f;
  b->A1 = b->Z1 + n * kHid;
  b->Z2 = b->A1 + n * kHid;
  b->A2 = b->Z2 + n * kHid;
  b->dZ2 = b->A2 + n * kHid;
  b->dZ1 = b->dZ2 + n * kHid;
  b->grad = b->dZ1 + n * kHid;
  b->part = d;  // (dW1 reuses it after dW2)
  b->opart = b->part + nz * kHid * kHid;
  b->cpart = b->opart + og * kOutCols;
  return QSGW_OK;
}

// Forward through both hidden layers into the buffers.
int mlp_hidden(qsgw_ctx* c, const float* P, int64_t n, const float* X, MlpBuffers& b, bool keepZ) {
  CHECK((gemm_t<float, 64, 64, false>(
      c, "mlp layer 1", Strided<true, float>{X, kIn, 1, 0, n},
      Strided<true, float>{P + kOffW1, kIn, 1, 0, kHid},
      EpiBiasGelu{P + kOffB1, keepZ ? b.Z1 : nullptr, b.A1, kHid}, n, kHid, kIn, 1)));
  CHECK((gemm_t<float, 64, 64, false>(
      c, "mlp layer 2", Strided<true, float>{b.A1, kHid, 1, 0, n},
      Strided<true, float>{P + kOffW2, kHid, 1, 0, kHid},
      EpiBiasGelu{P + kOffB2, keepZ ? b.Z2 : nullptr, b.A2, kHid}, n, kHid, kHid, 1)));
  return QSGW_OK;
}

int check_n(qsgw_ctx* c, int64_t n) {
  if (n < 1 || n > (1LL << 26)) return fail(c, QSGW_ERR_INVALID_ARG, "need 1 <= n <= 2^26 states");
  return QSGW_OK;
}

}  // namespace

extern "C" {

int qsgw_mlp_forward(qsgw_ctx* c, const float* params, int64_t n, const float* X, float* y) {
  if (!c) return QSGW_ERR_INVALID_ARG;
  CHECK(check_n(c, n));
  if (!params || !X || !y) return fail(c, QSGW_ERR_INVALID_ARG, "null pointer");
  CHECK(check_finite(c, "qsgw_mlp_forward",
                     {fin32(params, kNParams, "params"), fin32(X, n * kIn, "X")}));
  MlpBuffers b;
  CHECK(mlp_buffers(c, n, 0, &b));
  CHECK(mlp_hidden(c, params, n, X, b, false));
  hipLaunchKernelGGL(k_mlp_out, dim3(blocks_for(n, 4)), dim3(256), 0, c->stream, b.A2,
                     params + kOffW3, params + kOffB3, n, y);
  return launch_check(c, "k_mlp_out");
}

int qsgw_mlp_forward_bf16(qsgw_ctx* c, const float* params, int64_t n, const float* X, float* y) {
  if (!c) return QSGW_ERR_INVALID_ARG;
  CHECK(check_n(c, n));
  if (!params || !X || !y) return fail(c, QSGW_ERR_INVALID_ARG, "null pointer");
  CHECK(check_finite(c, "qsgw_mlp_forward_bf16",
                     {fin32(params, kNParams, "params"), fin32(X, n * kIn, "X")}));
  hipLaunchKernelGGL(k_mlp_forward_bf16, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, c->stream,
                     params, n, X, y);
  return launch_check(c, "k_mlp_forward_bf16");
}

int qsgw_mlp_train_step(qsgw_ctx* c, float* params, float* adam_m, float* adam_v, int64_t step,
                        double lr, int64_t n, const float* X, const float* target, float* grad,
                        double* loss) {
  if (!c) return QSGW_ERR_INVALID_ARG;
  CHECK(check_n(c, n));
  if (!params || !adam_m || !adam_v || !X || !target)
    return fail(c, QSGW_ERR_INVALID_ARG, "null pointer");
  if (step < 1) return fail(c, QSGW_ERR_INVALID_ARG, "Adam steps count from 1");
  if (!(lr >= 0.0) || !isfinite(lr)) return fail(c, QSGW_ERR_INVALID_ARG, "need a finite lr >= 0");
  CHECK(check_finite(c, "qsgw_mlp_train_step",
                     {fin32(params, kNParams, "params"), fin32(adam_m, kNParams, "adam_m"),
                      fin32(adam_v, kNParams, "adam_v"), fin32(X, n * kIn, "X"),
                      fin32(target, n, "target")}));
  // weight gradients reduce over the batch: split K = n into 32 chunks (the
  // two products have 4 and 2 output tiles), of 128 to 512 rows: below 128 the
  // partial sums cost more than the chunk, above 512 the chunk is the chain
  // (n = 4096, dW2: 27.9 us at 512 rows, 8 chunks)
  const int64_t chunk = n <= 32 * 128 ? 128 : (n >= 32 * 512 ? 512 : (n + 31) / 32);
  const SplitPlan sp = split_plan(n, (n + chunk - 1) / chunk);
  const int64_t og = (n + kOutRows - 1) / kOutRows, cg = (n + kColRows - 1) / kColRows;
  MlpBuffers b;
  CHECK(mlp_buffers(c, n, sp.nz, &b));
  CHECK(mlp_hidden(c, params, n, X, b, true));
  float* g = grad ? grad : b.grad;
  // output layer: dZ2, and db2, dw3 = A2^T dy, db3 = sum dy (adjacent in the
  // parameter layout) with the loss
  static_assert(kOffW3 == kOffB2 + kHid && kOffB3 == kOffW3 + kHid, "parameter layout");
  hipLaunchKernelGGL(k_mlp_out_grad, dim3((unsigned)og), dim3(256), 0, c->stream, b.A2, b.Z2,
                     params + kOffW3, params + kOffB3, n, target, b.dZ2, b.opart);
  CHECK(launch_check(c, "k_mlp_out_grad"));
  hipLaunchKernelGGL(k_sum_cols, dim3((kOutCols + 15) / 16), dim3(256), 0, c->stream, b.opart, og,
                     kOutCols, 2 * kHid + 1, g + kOffB2, n, loss);
  // layer 2: dW2[i][j] = sum_b dZ2[b][i] A1[b][j]
  CHECK((gemm_t<float, 64, 64, false>(
      c, "mlp dW2", Strided<false, float>{b.dZ2, 1, kHid, 0, kHid},
      Strided<false, float>{b.A1, 1, kHid, 0, kHid},
      EpiStore{b.part, kHid, 0, kHid * kHid, 1.0}, kHid, kHid, n, 1, sp)));
  hipLaunchKernelGGL(k_sum_parts, dim3(blocks_for(kHid * kHid)), dim3(256), 0, c->stream, b.part,
                     sp.nz, (int64_t)(kHid * kHid), g + kOffW2);
  // dZ1 = (dZ2 W2) * gelu'(Z1)
  CHECK((gemm_t<float, 64, 64, false>(
      c, "mlp dA1", Strided<true, float>{b.dZ2, kHid, 1, 0, n},
      Strided<false, float>{params + kOffW2, 1, kHid, 0, kHid}, EpiGeluGrad{b.Z1, b.dZ1, kHid}, n,
      kHid, kHid, 1)));
  // layer 1: dW1[i][q] = sum_b dZ1[b][i] X[b][q], db1 = colsum dZ1
  CHECK((gemm_t<float, 64, 64, false>(
      c, "mlp dW1", Strided<false, float>{b.dZ1, 1, kHid, 0, kHid},
      Strided<false, float>{X, 1, kIn, 0, kIn}, EpiStore{b.part, kIn, 0, kHid * kIn, 1.0}, kHid,
      kIn, n, 1, sp)));
  hipLaunchKernelGGL(k_sum_parts, dim3(blocks_for(kHid * kIn)), dim3(256), 0, c->stream, b.part,
                     sp.nz, (int64_t)(kHid * kIn), g + kOffW1);
  hipLaunchKernelGGL(k_col_partial, dim3((unsigned)cg), dim3(256), 0, c->stream, b.dZ1, n, b.cpart);
  hipLaunchKernelGGL(k_sum_cols, dim3((kHid + 15) / 16), dim3(256), 0, c->stream, b.cpart, cg,
                     kHid, kHid, g + kOffB1, n, (double*)nullptr);
  CHECK(launch_check(c, "mlp gradient"));
  const float c1 = 1.0f - powf(0.9f, (float)step), c2 = 1.0f - powf(0.999f, (float)step);
  hipLaunchKernelGGL(k_adam, dim3(blocks_for(kNParams)), dim3(256), 0, c->stream, params, adam_m,
                     adam_v, g, kNParams, (float)lr, c1, c2);
  return launch_check(c, "k_adam");
}

int qsgw_mlp_features(qsgw_ctx* c, int64_t nbf, int64_t nocc, const double* eps, const double* diag,
                      const float* mean, const float* scale, float* X) {
  if (!c) return QSGW_ERR_INVALID_ARG;
  if (!(nocc > 0 && nocc < nbf)) return fail(c, QSGW_ERR_INVALID_ARG, "need 0 < nocc < nbf");
  if (!eps || !diag || !X || (!mean) != (!scale))
    return fail(c, QSGW_ERR_INVALID_ARG, "null pointer (mean and scale go together)");
  CHECK(check_finite(c, "qsgw_mlp_features",
                     {fin(eps, nbf, "eps"), fin(diag, 4 * nbf, "diag"), fin32(mean, kIn, "mean"),
                      fin32(scale, kIn, "scale")}));
  hipLaunchKernelGGL(k_mlp_features, dim3(blocks_for(nbf)), dim3(256), 0, c->stream, nbf, nocc, eps,
                     diag, mean, scale, X);
  return launch_check(c, "k_mlp_features");
}

int qsgw_warm_start(qsgw_ctx* c, int64_t nbf, const double* eps0, const double* C0,
                    const float* delta, double* eps, double* C) {
  if (!c) return QSGW_ERR_INVALID_ARG;
  if (nbf < 1 || nbf > 46340) return fail(c, QSGW_ERR_INVALID_ARG, "bad nbf");
  if (!eps0 || !C0 || !delta || !eps || !C) return fail(c, QSGW_ERR_INVALID_ARG, "null pointer");
  if (eps == eps0 || C == C0) return fail(c, QSGW_ERR_INVALID_ARG, "outputs must not alias inputs");
  CHECK(check_finite(c, "qsgw_warm_start", {fin(eps0, nbf, "eps0"), fin(C0, nbf * nbf, "C0"),
                                            fin32(delta, nbf, "delta")}));
  int64_t* perm = nullptr;
  CHECK(ws_get(c, W_MLP_PERM, (size_t)nbf, &perm));
  hipLaunchKernelGGL(k_warm_rank, dim3(1), dim3(1024), 0, c->stream, nbf, eps0, delta, eps, perm);
  hipLaunchKernelGGL(k_warm_permute, dim3(blocks_for(nbf * nbf)), dim3(256), 0, c->stream, nbf, C0,
                     perm, C);
  return launch_check(c, "warm start");
}

}  // extern "C"
