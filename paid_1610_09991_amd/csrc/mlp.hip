// mlp.hip -- the subdivision-density model of the learned seeding: model
// features of each container, and the FP32 kernels of a 7 -> 128 -> 128 ->
// 128 -> 256 perceptron (GELU on the hidden layers): forward, backward with the
// mean squared error, Adam.  Training and inference share the same kernels.
//
// The model predicts, per cell of a 16 x 16 grid over the zone, log2(1 + n)
// with n the number of leaves the converged adaptive tree has in that cell.
// It works in a reduced frame: the integrand at transfer momentum l equals
// the integrand at l - 2 pi e_x moved by pi e_x in p (both energies are
// 2 pi periodic), and the dispersion is invariant under the square's point
// group, so l is reduced to [-pi, pi)^2 and then to the wedge
// 0 <= l_y <= l_x, and each container cell is read from the matching model
// cell.  None of this is in the paper; the adaptive loop of Alg. 2 still
// decides every split that the seed does not and the termination.
#include <math.h>

#include "launch.h"

namespace paid {

namespace {

__device__ inline float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ inline float gelu_d(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) +
         z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// ------------------------------------------------------------------ matrix-core pieces
// FP32 products on the matrix cores (16 x 16 x 4, FP32 in, FP32 accumulation).
// Lane (kk, m) = (lane >> 4, lane & 15) holds A[m][k] and B[k][m] of the step's
// four k, and result register i is row 4 kk + i, column m.  The order of k is
// free: quarter kk takes k = kk K/4 + s at step s, so that a lane's operands of
// consecutive steps are consecutive in memory (16-byte loads).  Fixed orders
// throughout: results do not depend on the launch.
//
// A workgroup of eight waves takes 16 RT samples through all layers, with the
// activations in LDS: one launch for the whole pass, no activations in global
// memory.  Each wave owns 16 of the 128 columns of a layer (32 of the 256
// outputs), reads their weights once from L2 into registers and uses them for
// RT row tiles.  One product kernel per layer instead (64 x 64 tiles, scalar
// FMAs, activations through memory and a device allocation per call) took 108
// us of kernels and 168 us a call for 23,040 samples (now 64 and 74), and a
// training step of 256 samples 17 launches of 8-16 workgroups each, 516 us a
// call with its Adam step (now three launches, 62 us).
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));  // caller's arrays: 4-byte aligned

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kHidLd = kMlpHid + 4, kOutLd = kMlpOut + 4;  // LDS leading dimensions (bank spread)
static_assert(kMlpHid == 16 * kWaves, "a wave owns 16 hidden columns");

__device__ inline f4 mfma4(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// acc[t] = X W^T for the wave's 16 columns n0.. : X [16 RT][K] in LDS (leading
// dimension ld), W [..][K] row-major, K a multiple of 16
template <int RT, int K>
__device__ inline void mul_wt(const float *X, int ld, const float *W, int n0, f4 (&acc)[RT]) {
  const int lane = threadIdx.x & 63, m = lane & 15, kk = lane >> 4;
  constexpr int Q = K / 16;  // float4 per quarter
  f4 b[Q];
  const f4u *w = reinterpret_cast<const f4u *>(W + (long)(n0 + m) * K + kk * (K / 4));
#pragma unroll
  for (int s = 0; s < Q; ++s) b[s] = w[s];
#pragma unroll
  for (int t = 0; t < RT; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < Q; ++s)
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const f4 x = *reinterpret_cast<const f4 *>(X + (16 * t + m) * ld + kk * (K / 4) + 4 * s);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[t] = mfma4(x[i], b[s][i], acc[t]);
    }
}

// acc[t] = X W for the wave's 16 columns n0.. : X [16 RT][K] in LDS, W [K][128]
template <int RT, int K>
__device__ inline void mul_w(const float *X, int ld, const float *W, int n0, f4 (&acc)[RT]) {
  const int lane = threadIdx.x & 63, m = lane & 15, kk = lane >> 4;
  constexpr int C = 8;  // float4 of X a chunk: 32 weights in flight
  const float *w = W + (long)kk * (K / 4) * kMlpHid + n0 + m;
#pragma unroll
  for (int t = 0; t < RT; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int s0 = 0; s0 < K / 16; s0 += C) {
    float b[4 * C];
#pragma unroll
    for (int s = 0; s < 4 * C; ++s) b[s] = w[(long)(4 * s0 + s) * kMlpHid];
#pragma unroll
    for (int s = 0; s < C; ++s)
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const f4 x = *reinterpret_cast<const f4 *>(X + (16 * t + m) * ld + kk * (K / 4) + 4 * (s0 + s));
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[t] = mfma4(x[i], b[4 * s + i], acc[t]);
      }
  }
}

// The hidden layers of 16 RT samples from r0 on: the last hidden activations
// end in X[0] (LDS, [16 RT][kHidLd] each of two buffers).  TRAIN: also gelu' of
// the pre-activations into G[l] (LDS) and the activations into a.A[l] (global).
template <int RT, bool TRAIN>
__device__ void hidden_layers(const MlpLayout &L, const float *w, const float *x, int n, long r0, float *X0,
                              float *X1, float *G, const MlpAct &a) {
  constexpr int R = 16 * RT;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6, m = lane & 15, kk = lane >> 4, n0 = 16 * wv;
  auto put = [&](int l, float *Y, int row, int col, float z) {
    const float y = gelu(z);
    Y[row * kHidLd + col] = y;
    if (TRAIN) {
      G[(l * R + row) * kHidLd + col] = gelu_d(z);
      if (r0 + row < n) a.A[l][(r0 + row) * kMlpHid + col] = y;
    }
  };
  // 7 inputs: scalar FMAs, a column per thread, every fourth row (their
  // samples through X1, which nothing uses yet)
  for (int e = t; e < R * kMlpIn; e += kThreads) X1[e] = r0 * kMlpIn + e < (long)n * kMlpIn ? x[r0 * kMlpIn + e] : 0.f;
  __syncthreads();
  {
    const int col = t & (kMlpHid - 1);
    float wr[kMlpIn];
#pragma unroll
    for (int k = 0; k < kMlpIn; ++k) wr[k] = w[L.w[0] + (long)col * kMlpIn + k];
    const float b = w[L.b[0] + col];
    for (int row = t / kMlpHid; row < R; row += kThreads / kMlpHid) {
      float z = 0.f;
#pragma unroll
      for (int k = 0; k < kMlpIn; ++k) z = fmaf(X1[row * kMlpIn + k], wr[k], z);
      put(0, X0, row, col, z + b);
    }
  }
  __syncthreads();
#pragma unroll
  for (int l = 1; l < 3; ++l) {
    const float *X = (l == 1) ? X0 : X1;
    float *Y = (l == 1) ? X1 : X0;
    f4 acc[RT];
    mul_wt<RT, kMlpHid>(X, kHidLd, w + L.w[l], n0, acc);
    const float b = w[L.b[l] + n0 + m];
#pragma unroll
    for (int q = 0; q < RT; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) put(l, Y, 16 * q + 4 * kk + i, n0 + m, acc[q][i] + b);
    __syncthreads();
  }
}

template <int RT>
__global__ void __launch_bounds__(kThreads) k_forward(MlpLayout L, const float *__restrict__ w,
                                                      const float *__restrict__ x, int n, float *__restrict__ y) {
  constexpr int R = 16 * RT;
  __shared__ __align__(16) float X[2][R * kHidLd];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, m = lane & 15, kk = lane >> 4;
  const long r0 = (long)blockIdx.x * R;
  hidden_layers<RT, false>(L, w, x, n, r0, X[0], X[1], nullptr, MlpAct{});
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int n0 = 32 * wv + 16 * c;
    f4 acc[RT];
    mul_wt<RT, kMlpHid>(X[0], kHidLd, w + L.w[3], n0, acc);
    const float b = w[L.b[3] + n0 + m];
#pragma unroll
    for (int q = 0; q < RT; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const long row = r0 + 16 * q + 4 * kk + i;
        if (row < n) y[row * kMlpOut + n0 + m] = acc[q][i] + b;
      }
  }
}

// Forward pass, squared error and the backward pass down to every layer's
// delta, of 16 samples a workgroup: activations, deltas (global, for the
// weight gradients) and the workgroup's sum of squares (FP64, fixed order).
__global__ void __launch_bounds__(kThreads) k_deltas(MlpLayout L, const float *__restrict__ w,
                                                     const float *__restrict__ x, const float *__restrict__ y, int n,
                                                     MlpAct a) {
  constexpr int R = 16;
  __shared__ __align__(16) float X[2][R * kHidLd];
  __shared__ __align__(16) float G[3 * R * kHidLd];
  __shared__ __align__(16) float O[R * kOutLd];
  __shared__ double sq[kThreads];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6, m = lane & 15, kk = lane >> 4;
  const long r0 = (long)blockIdx.x * R;
  hidden_layers<1, true>(L, w, x, n, r0, X[0], X[1], G, a);
  // outputs: dY = 2 (yhat - y) / (n 256)
  const float sc = (float)(2.0 / ((double)n * kMlpOut));
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int n0 = 32 * wv + 16 * c;
    f4 acc[1];
    mul_wt<1, kMlpHid>(X[0], kHidLd, w + L.w[3], n0, acc);
    const float b = w[L.b[3] + n0 + m];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 4 * kk + i;
      float d = 0.f;
      if (r0 + row < n) {
        const float e = (acc[0][i] + b) - y[(r0 + row) * kMlpOut + n0 + m];
        d = sc * e;
        s += (double)e * (double)e;
        a.dY[(r0 + row) * kMlpOut + n0 + m] = d;
      }
      O[row * kOutLd + n0 + m] = d;
    }
  }
  sq[t] = s;
  __syncthreads();
  for (int o = kThreads / 2; o > 0; o >>= 1) {
    if (t < o) sq[t] += sq[t + o];
    __syncthreads();
  }
  if (t == 0) a.part[blockIdx.x] = sq[0];
  // deltas of the hidden layers: D_l = (D_{l+1} W_{l+1}) gelu'(Z_l)
#pragma unroll
  for (int l = 2; l >= 0; --l) {
    f4 acc[1];
    if (l == 2)
      mul_w<1, kMlpOut>(O, kOutLd, w + L.w[3], 16 * wv, acc);
    else
      mul_w<1, kMlpHid>(l == 1 ? X[0] : X[1], kHidLd, w + L.w[l + 1], 16 * wv, acc);
    float *D = l == 1 ? X[1] : X[0];
    if (l == 2) __syncthreads();  // (X[0] held the forward pass's last activations)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 4 * kk + i, col = 16 * wv + m;
      const float d = acc[0][i] * G[(l * R + row) * kHidLd + col];
      D[row * kHidLd + col] = d;
      if (r0 + row < n) a.D[l][(r0 + row) * kMlpHid + col] = d;
    }
    __syncthreads();
  }
}

// Weight and bias gradients gW[o][i] = sum_r d[r][o] X[r][i], gb[o] = sum_r
// d[r][o]: a workgroup per 32 x 32 tile of one layer's weights, its eight waves
// take an eighth of the samples each, and the parts are added in wave order.
// The first workgroup also adds up the loss.
constexpr int kGradTiles[4] = {4, 16, 16, 32};  // tiles of each layer: (out / 32) (in / 32)
constexpr int kGradBlocks = 4 + 16 + 16 + 32;

__global__ void __launch_bounds__(kThreads) k_grads(MlpLayout L, const float *__restrict__ x, int n, MlpAct a,
                                                    float *__restrict__ grad, int parts, double *loss,
                                                    const int *step) {
  __shared__ float S[kWaves][32 * 33 + 32];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6, m = lane & 15, kk = lane >> 4;
  int l = 0, tile = blockIdx.x;
  while (tile >= kGradTiles[l]) tile -= kGradTiles[l++];
  const int ni = L.ni[l], no = L.no[l], it = (ni + 31) / 32;
  const int o0 = 32 * (tile / it), i0 = 32 * (tile % it);
  const float *d = l == 3 ? a.dY : a.D[l], *X = l == 0 ? x : a.A[l - 1];
  const int per = ((n + kWaves - 1) / kWaves + 3) & ~3;
  const int ra = wv * per, rb = ra + per < n ? ra + per : n;
  f4 acc[2][2];
  float bs[2] = {0.f, 0.f};
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q) acc[p][q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int r = ra; r < rb; r += 4) {
    const long row = r + kk;
    const bool in = row < rb;
    float da[2], xb[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      da[p] = in ? d[row * no + o0 + 16 * p + m] : 0.f;
      xb[p] = (in && i0 + 16 * p + m < ni) ? X[row * ni + i0 + 16 * p + m] : 0.f;
      bs[p] += da[p];
    }
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int q = 0; q < 2; ++q) acc[p][q] = mfma4(da[p], xb[q], acc[p][q]);
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) S[wv][(16 * p + 4 * kk + i) * 33 + 16 * q + m] = acc[p][q][i];
    float b = bs[p];  // over the four rows of a step: lanes m, m + 16, m + 32, m + 48
    b += __shfl_xor(b, 16, 64);
    b += __shfl_xor(b, 32, 64);
    if (kk == 0) S[wv][32 * 33 + 16 * p + m] = b;
  }
  __syncthreads();
  for (int e = t; e < 32 * 32; e += kThreads) {
    const int o = e >> 5, i = e & 31;
    float s = S[0][o * 33 + i];
    for (int v = 1; v < kWaves; ++v) s += S[v][o * 33 + i];
    if (i0 + i < ni) grad[L.w[l] + (long)(o0 + o) * ni + i0 + i] = s;
  }
  if (i0 == 0 && t < 32) {
    float s = S[0][32 * 33 + t];
    for (int v = 1; v < kWaves; ++v) s += S[v][32 * 33 + t];
    grad[L.b[l] + o0 + t] = s;
  }
  if (blockIdx.x == 0 && wv == kWaves - 1 && loss) {
    double s = 0.0;
    for (int p = lane; p < parts; p += 64) s += a.part[p];
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) loss[step ? *step : 0] = s / ((double)n * kMlpOut);
  }
}

// Adam (beta1 0.9, beta2 0.999, eps 1e-8) with cosine decay of the rate from
// lr0 to lr1 over `steps`; the step t (from 1) is *tdev + 1 when tdev is set
__global__ void k_adam(float *w, const float *g, float *m, float *v, long np, int t_host,
                       const int *tdev, float lr0, float lr1, int steps) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= np) return;
  const int t = tdev ? *tdev + 1 : t_host;
  double lr = lr0;
  if (steps > 0) lr = lr1 + 0.5 * (lr0 - lr1) * (1.0 + cos(3.14159265358979323846 * (double)(t - 1) / steps));
  const float c1 = (float)(1.0 - pow(0.9, (double)t)), c2 = (float)(1.0 - pow(0.999, (double)t));
  float gi = g[i];
  float mi = 0.9f * m[i] + 0.1f * gi;
  float vi = 0.999f * v[i] + 0.001f * gi * gi;
  m[i] = mi;
  v[i] = vi;
  w[i] -= (float)lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
}

__global__ void k_gather(const float *X, const float *Y, const int *idx, const int *step, int bs,
                         float *Xb, float *Yb) {
  const int r = blockIdx.x, t = threadIdx.x;
  const long src = idx[(long)(*step) * bs + r];
  if (t < kMlpIn) Xb[(long)r * kMlpIn + t] = X[src * kMlpIn + t];
  Yb[(long)r * kMlpOut + t] = Y[src * kMlpOut + t];
}

__global__ void k_count(int *c) {
  if (threadIdx.x == 0) *c += 1;
}

// features and fold of every container (same container order as the setup)
__global__ void k_seed_features(const Entry *entries, const double *q, int n_ctr, int n_q, int n_ch,
                                int ch_first, float *X, int *fold) {
  int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n_ctr) return;
  int ich = c % n_ch, iq = (c / n_ch) % n_q, ip = c / (n_ch * n_q);
  const Entry e = entries[ip];
  const int ch = (n_ch == 2) ? ich : ch_first;
  const double pi = 3.14159265358979323846;
  double lx = q[2 * iq], ly = q[2 * iq + 1];
  double nx = floor((lx + pi) / (2.0 * pi)), ny = floor((ly + pi) / (2.0 * pi));
  double rx = lx - 2.0 * pi * nx, ry = ly - 2.0 * pi * ny;
  int hx = ((long long)nx) & 1, hy = ((long long)ny) & 1;
  int mx = rx < 0.0, my = ry < 0.0;
  double ax = fabs(rx), ay = fabs(ry);
  int sw = ay > ax;
  float *x = X + (long)c * kMlpIn;
  x[0] = (float)((sw ? ay : ax) / pi);
  x[1] = (float)((sw ? ax : ay) / pi);
  x[2] = (float)(e.mu / e.t);
  x[3] = (float)log10(e.T / e.t);
  x[4] = (float)(e.tp / e.t);
  x[5] = (float)log10(e.Om / e.t);
  x[6] = ch == 1 ? 1.0f : -1.0f;
  fold[c] = hx | (hy << 1) | (mx << 2) | (my << 3) | (sw << 4);
}

}  // namespace

// ------------------------------------------------------------------ host side
hipError_t launch_seed_features(const Entry *entries, const double *q, int n_ctr, int n_q, int n_ch,
                                int ch_first, float *X, int *fold, hipStream_t s) {
  if (n_ctr == 0) return hipSuccess;
  hipLaunchKernelGGL(k_seed_features, dim3((n_ctr + 255) / 256), dim3(256), 0, s, entries, q, n_ctr,
                     n_q, n_ch, ch_first, X, fold);
  return hipGetLastError();
}

// Parameter layout: per layer l, W_l [out][in] row-major, then b_l [out].
MlpLayout mlp_layout() {
  MlpLayout L;
  const int dims[5] = {kMlpIn, kMlpHid, kMlpHid, kMlpHid, kMlpOut};
  long off = 0;
  for (int l = 0; l < 4; ++l) {
    L.ni[l] = dims[l];
    L.no[l] = dims[l + 1];
    L.w[l] = off;
    off += (long)dims[l + 1] * dims[l];
    L.b[l] = off;
    off += dims[l + 1];
  }
  L.total = off;
  return L;
}

// 16 samples a workgroup fill the chip up to 4,096 samples; above that 32,
// which read the weights (268 KB from L2) half as often
hipError_t mlp_forward(const float *w, const float *x, int n, float *y, hipStream_t s) {
  const MlpLayout L = mlp_layout();
  if (n <= 4096)
    hipLaunchKernelGGL(k_forward<1>, dim3((n + 15) / 16), dim3(kThreads), 0, s, L, w, x, n, y);
  else
    hipLaunchKernelGGL(k_forward<2>, dim3((n + 31) / 32), dim3(kThreads), 0, s, L, w, x, n, y);
  return hipGetLastError();
}

hipError_t mlp_loss_grad(const float *w, const float *x, const float *y, int n, const MlpAct &a, float *grad,
                         double *loss, const int *step, hipStream_t s) {
  const MlpLayout L = mlp_layout();
  const int blocks = (n + 15) / 16;
  hipLaunchKernelGGL(k_deltas, dim3(blocks), dim3(kThreads), 0, s, L, w, x, y, n, a);
  hipLaunchKernelGGL(k_grads, dim3(kGradBlocks), dim3(kThreads), 0, s, L, x, n, a, grad, blocks, loss, step);
  return hipGetLastError();
}

hipError_t mlp_adam(float *w, const float *g, float *m, float *v, long np, int t, const int *tdev,
                    float lr0, float lr1, int steps, hipStream_t s) {
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s, w, g, m, v, np, t,
                     tdev, lr0, lr1, steps);
  return hipGetLastError();
}

hipError_t mlp_gather(const float *X, const float *Y, const int *idx, const int *step, int bs,
                      float *Xb, float *Yb, hipStream_t s) {
  hipLaunchKernelGGL(k_gather, dim3(bs), dim3(kMlpOut), 0, s, X, Y, idx, step, bs, Xb, Yb);
  return hipGetLastError();
}

hipError_t mlp_count(int *c, hipStream_t s) {
  hipLaunchKernelGGL(k_count, dim3(1), dim3(64), 0, s, c);
  return hipGetLastError();
}

// ------------------------------------------------------------------ fixed working memory
// Working memory of the loss-and-gradient entry point that allocates
// nothing: the per-sample buffers of kNoAllocMaxN samples (activations, deltas,
// output deltas), the workgroups' sums of squares and the FP64 loss.  Every
// element a call reads is written earlier in the same call, so nothing has
// to start at zero.  Each device holds its own copy of the array at its own
// address; host code must use that address (from hipGetSymbolAddress), never
// the array's name, which on the host is only a stand-in.
static __device__ __align__(256) float scratch[kNoAllocFloats];

hipError_t noalloc_scratch_address(float **ptr) {
  void *p = nullptr;
  hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  *ptr = static_cast<float *>(p);
  return hipSuccess;
}

}  // namespace paid
