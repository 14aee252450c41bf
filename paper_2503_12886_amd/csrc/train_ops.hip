// The small dense pieces of the training step around the renderer: the
// weight MLP psi = F(theta) (Eq. 2) forward/backward, and Adam with
// per-attribute learning rates (Sec. A.3).
#include "gbr_internal.h"

namespace gbr {

// ---------------------------------------------------------------- MLP forward
// One workgroup per frame runs the three layers back to back: the layer's
// input vector sits in LDS, each wave forms 16 output units at a time (4 of
// the short last layer), lanes over the input.  Weight rows are read
// coalesced at a uniform row address and one lane offset, so the loads cost no
// vector arithmetic, and the units' sums over the wave are taken together:
// each halving step of the butterfly (partners 32, 16, 8, 4, 2, 1 apart, the
// same pairs as one butterfly per unit) folds two units' registers into one,
// 32 operations for 16 units where 16 separate butterflies take 96 lane
// exchanges.  When the weights of all three layers fit the registers (inputs
// up to 64, hidden layers up to 256) every load is issued before the first
// product, so that one load latency precedes the layers instead of three.
// Bound by latency and one CU's issue: a frame's workgroup 14.3 -> 6.9 us
// at 56-256-256-20 (2000 -> 400 vector operations a wave).  Pre-activations
// are kept (z1, z2 for the backward; the ReLU of a layer is applied when the
// next layer reads them).
constexpr int kMlpThreads = 1024;
constexpr int kMlpWaves = kMlpThreads / 64;
constexpr int kMlpMaxIn = 1024;
constexpr int kMlpRows = 16, kMlpRowsOut = 4;   // units a wave forms together: hidden layers, last layer

// x <- the two registers' sums over partners 32 (16) lanes apart: x's in the
// lower half (even rows), y's in the upper (odd rows).
__device__ __forceinline__ float fold32(float x, float y) {
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(x), "+v"(y));
  return x + y;
}
__device__ __forceinline__ float fold16(float x, float y) {
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(x), "+v"(y));
  return x + y;
}
// The same 8 (4) lanes apart inside the rows of 16: bank-masked DPP adds in
// place, with the two wait states that DPP reads need before and after.
__device__ __forceinline__ float fold8(float x, float y) {
  asm volatile("s_nop 1\n\t"
               "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
               "v_add_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xc\n\ts_nop 1"
               : "+v"(x) : "v"(y));
  return x;
}
__device__ __forceinline__ float fold4(float x, float y) {
  asm volatile("s_nop 1\n\t"
               "v_add_f32_dpp %0, %0, %0 row_shl:4 row_mask:0xf bank_mask:0x5\n\t"
               "v_add_f32_dpp %0, %1, %1 row_shr:4 row_mask:0xf bank_mask:0xa\n\ts_nop 1"
               : "+v"(x) : "v"(y));
  return x;
}

// The sums over the wave of R values a lane: lane l returns value l R / 64's.
__device__ __forceinline__ float wave_sums(float (&s)[16]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) s[i] = fold32(s[i], s[i + 8]);
#pragma unroll
  for (int i = 0; i < 4; ++i) s[i] = fold16(s[i], s[i + 4]);
#pragma unroll
  for (int i = 0; i < 2; ++i) s[i] = fold8(s[i], s[i + 2]);
  float x = fold4(s[0], s[1]);
  x += dpp_mov<0x4e, 0xf, 0xf, false>(x);
  return x + dpp_mov<0xb1, 0xf, 0xf, false>(x);
}
__device__ __forceinline__ float wave_sums(float (&s)[4]) {
  float x = fold16(fold32(s[0], s[2]), fold32(s[1], s[3]));
  x += dpp_mov<0x128, 0xf, 0xf, false>(x);   // row_ror:8
  x += dpp_mov<0x124, 0xf, 0xf, false>(x);   // row_ror:4 (the row has period 8 by now)
  x += dpp_mov<0x4e, 0xf, 0xf, false>(x);
  return x + dpp_mov<0xb1, 0xf, 0xf, false>(x);
}

// Weights of units [j0, j0 + R) at inputs c0 + lane + 64 t, t < T4 (units and
// inputs clamped into range; the inputs' values are zeroed past n_in).  j0 is
// wave-uniform.
template <int R, int T4>
__device__ __forceinline__ void mlp_weights(const float* __restrict__ W, int n_in, int n_out, int j0, int c0,
                                            float (&wv)[R][T4]) {
  const int lane = threadIdx.x & 63;
  uint32_t c[T4];                          // byte offsets (32 bits: the loads take them beside a scalar row address)
#pragma unroll
  for (int t = 0; t < T4; ++t) c[t] = 4u * (uint32_t)min(c0 + 64 * t + lane, n_in - 1);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const char* row = reinterpret_cast<const char*>(W + (int64_t)min(j0 + r, n_out - 1) * n_in);
#pragma unroll
    for (int t = 0; t < T4; ++t) wv[r][t] = *reinterpret_cast<const float*>(row + c[t]);
  }
}

template <int R, int T4>
__device__ __forceinline__ void mlp_products(const float (&wv)[R][T4], const float* in, int n_in, int c0, bool relu_in,
                                             float (&s)[R]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int t = 0; t < T4; ++t) {
    const int c = c0 + 64 * t + lane;
    const float v = in[min(c, n_in - 1)];
    const float x = c < n_in ? (relu_in ? fmaxf(v, 0.0f) : v) : 0.0f;
#pragma unroll
    for (int r = 0; r < R; ++r) s[r] = __builtin_fmaf(wv[r][t], x, s[r]);
  }
}

// Where a layer's units go: memory, LDS, float64 in memory (null: not there).
struct MlpOut {
  float* g;
  float* l;
  double* d;
};

// out[j0 + i] = bias + the sums, i < R
template <int R>
__device__ __forceinline__ void mlp_store(float (&s)[R], const float* __restrict__ bias, int n_out, int j0,
                                          MlpOut out) {
  const int lane = threadIdx.x & 63;
  const float tot = wave_sums(s);
  const int j = j0 + lane * R / 64;
  if (lane % (64 / R) == 0 && j < n_out) {
    const float v = tot + bias[j];
    if (out.g) out.g[j] = v;
    if (out.l) out.l[j] = v;
    if (out.d) out.d[j] = (double)v;
  }
}

// out[j] = bias[j] + sum_c W[j][c] act(in[c]) for j < n_out; act = ReLU when relu_in.
template <int R>
__device__ __forceinline__ void mlp_layer(const float* __restrict__ W, const float* __restrict__ bias,
                                          const float* in, int n_in, int n_out, bool relu_in, MlpOut out) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int j0 = w * R; j0 < n_out; j0 += kMlpWaves * R) {
    float s[R];
#pragma unroll
    for (int r = 0; r < R; ++r) s[r] = 0.0f;
    for (int c0 = 0; c0 < n_in; c0 += 256) {
      float wv[R][4];
      mlp_weights(W, n_in, n_out, j0, c0, wv);
      mlp_products(wv, in, n_in, c0, relu_in, s);
    }
    mlp_store(s, bias, n_out, j0, out);
  }
}

// One frame's three layers.  z1, z2 (may be null): its pre-activations; psi64
// (may be null): its outputs as float64.  HELD: inputs up to 64 and hidden
// layers up to 256 (a block of rows per wave): the three layers' weights are
// read at once.
template <bool HELD>
__device__ __forceinline__ void mlp_frame(const float* __restrict__ params, const float* __restrict__ theta, int d_in,
                                          int hidden, int K, float* __restrict__ psi, float* __restrict__ z1,
                                          float* __restrict__ z2, double* __restrict__ psi64) {
  __shared__ float xa[kMlpMaxIn], xb[kMlpMaxIn];
  const float* W1 = params;
  const float* b1 = W1 + (int64_t)hidden * d_in;
  const float* W2 = b1 + hidden;
  const float* b2 = W2 + (int64_t)hidden * hidden;
  const float* W3 = b2 + hidden;
  const float* b3 = W3 + (int64_t)K * hidden;
  if constexpr (HELD) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j0 = w * kMlpRows, k0 = w * kMlpRowsOut;
    const float th = (int)threadIdx.x < d_in ? theta[threadIdx.x] : 0.0f;
    float w1[kMlpRows][1], w2[kMlpRows][4], w3[kMlpRowsOut][4];
    mlp_weights(W1, d_in, hidden, j0, 0, w1);
    mlp_weights(W2, hidden, hidden, j0, 0, w2);
    mlp_weights(W3, hidden, K, k0, 0, w3);
    __builtin_amdgcn_sched_barrier(0);      // every load before the layers
    if ((int)threadIdx.x < d_in) xa[threadIdx.x] = th;
    __syncthreads();
    float s[kMlpRows], so[kMlpRowsOut];
#pragma unroll
    for (int r = 0; r < kMlpRows; ++r) s[r] = 0.0f;
    mlp_products(w1, xa, d_in, 0, false, s);
    mlp_store(s, b1, hidden, j0, MlpOut{z1, xb, nullptr});
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kMlpRows; ++r) s[r] = 0.0f;
    mlp_products(w2, xb, hidden, 0, true, s);
    mlp_store(s, b2, hidden, j0, MlpOut{z2, xa, nullptr});
    __syncthreads();
    if (k0 < K) {
#pragma unroll
      for (int r = 0; r < kMlpRowsOut; ++r) so[r] = 0.0f;
      mlp_products(w3, xa, hidden, 0, true, so);
      mlp_store(so, b3, K, k0, MlpOut{psi, nullptr, psi64});
    }
  } else {
    for (int t = threadIdx.x; t < d_in; t += kMlpThreads) xa[t] = theta[t];
    __syncthreads();
    mlp_layer<kMlpRows>(W1, b1, xa, d_in, hidden, false, MlpOut{z1, xb, nullptr});
    __syncthreads();
    mlp_layer<kMlpRows>(W2, b2, xb, hidden, hidden, true, MlpOut{z2, xa, nullptr});
    __syncthreads();
    mlp_layer<kMlpRowsOut>(W3, b3, xa, hidden, K, true, MlpOut{psi, nullptr, psi64});
  }
}

template <bool HELD>
__global__ __launch_bounds__(kMlpThreads) void mlp_fwd_kernel(const float* __restrict__ params,
                                                              const float* __restrict__ theta, int d_in, int hidden,
                                                              int K, float* __restrict__ psi, float* __restrict__ z1,
                                                              float* __restrict__ z2) {
  const int64_t b = blockIdx.x;
  mlp_frame<HELD>(params, theta + b * d_in, d_in, hidden, K, psi + b * K, z1 + b * hidden, z2 + b * hidden, nullptr);
}

// The MLPs of several models (gbr_drive): a workgroup per frame of all of them,
// which also leaves the frame's row of the blend's weight table.  A model at a
// time has one CU or a few at work and each launch's gap: 8 models of one
// frame, 56-256-256-20, 8 x 9.4 us -> 12.2.
template <bool HELD>
__global__ __launch_bounds__(kMlpThreads) void mlp_drive_kernel(DriveTable t, int d_in, int hidden) {
  const int gi = t.group_of(t.frame0, blockIdx.x);
  const DriveGroup& g = t.g[gi];
  const int64_t b = blockIdx.x - t.frame0[gi];
  double* w64 = t.w64 + (int64_t)blockIdx.x * kBlendW64Stride;
  const int k = threadIdx.x;
  if (k == 0 || (k > g.K && k < kBlendW64Stride)) w64[k] = k == 0 ? 1.0 : 0.0;   // the implicit 1 of slice 0
  mlp_frame<HELD>(g.mlp, g.theta + b * d_in, d_in, hidden, g.K, g.psi + b * g.K, nullptr, nullptr, w64 + 1);
}

static bool mlp_held(int d_in, int hidden, int K) {
  return d_in <= 64 && hidden <= kMlpWaves * kMlpRows && K <= kMlpWaves * kMlpRowsOut;
}

void launch_mlp_drive(const DriveTable& t, int d_in, int hidden, hipStream_t s) {
  // (K <= 63 always fits)
  if (mlp_held(d_in, hidden, kBlendW64Stride - 1))
    hipLaunchKernelGGL(mlp_drive_kernel<true>, dim3(t.frames), dim3(kMlpThreads), 0, s, t, d_in, hidden);
  else
    hipLaunchKernelGGL(mlp_drive_kernel<false>, dim3(t.frames), dim3(kMlpThreads), 0, s, t, d_in, hidden);
}

void launch_mlp_fwd(const float* params, const float* theta, int B, int d_in, int hidden, int K, float* psi,
                    float* z1, float* z2, hipStream_t s) {
  if (B == 0) return;
  if (mlp_held(d_in, hidden, K))
    hipLaunchKernelGGL(mlp_fwd_kernel<true>, dim3(B), dim3(kMlpThreads), 0, s, params, theta, d_in, hidden, K, psi, z1,
                       z2);
  else
    hipLaunchKernelGGL(mlp_fwd_kernel<false>, dim3(B), dim3(kMlpThreads), 0, s, params, theta, d_in, hidden, K, psi,
                       z1, z2);
}

// ---------------------------------------------------------------- MLP backward
// dz2 = (W3^T dpsi) * [z2 > 0], then dz1 = (W2^T dz2) * [z1 > 0].  Each frame
// takes kActParts workgroups: every one forms the whole of dz2 (K x hidden
// terms; the first one stores it) and its own part of dz1's units.  A unit's
// sum is split over as many threads as the workgroup has for it (weight rows
// read coalesced across units, each thread's loads in flight together), and
// the pieces are added in order.  Then one thread per parameter sums over the
// frames in frame order.
constexpr int kActParts = 4;

// dz[i] = [z[i] > 0] * sum_k W[k][i] g[k] for i in [i0, i1) (g in LDS; dz to
// dz_l (LDS, indexed by i) when non-null and to dz_g (global) when non-null).
__device__ __forceinline__ void mlp_act_back(const float* __restrict__ W, const float* g, int n_g, int n_x, int i0,
                                             int i1, const float* __restrict__ z, float* part, float* dz_l,
                                             float* __restrict__ dz_g) {
  const int nu = i1 - i0;                                          // units, <= kMlpThreads
  const int split = min(16, max(1, kMlpThreads / max(nu, 1)));     // threads per unit
  const int per = (n_g + split - 1) / split;
  const int t = (int)threadIdx.x;
  if (nu > 0 && t < nu * split) {
    const int i = i0 + t % nu, qk = t / nu;
    const int k0 = qk * per, k1 = min(n_g, k0 + per);
    // 16 steps at a time, every weight load issued first (index clamped into
    // range); steps past k1 add 0 * w, which leaves the sum as it is
    float s = 0.0f;
    for (int kb = k0; kb < k1; kb += 16) {
      float wv[16], gv[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int k = min(kb + u, k1 - 1);
        wv[u] = W[(int64_t)k * n_x + i];
        gv[u] = kb + u < k1 ? g[k] : 0.0f;
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) s = __builtin_fmaf(wv[u], gv[u], s);
    }
    part[qk * kMlpMaxIn + (i - i0)] = s;
  }
  __syncthreads();
  for (int u = t; u < nu; u += kMlpThreads) {
    float v = 0.0f;
    for (int qk = 0; qk < split; ++qk) v += part[qk * kMlpMaxIn + u];
    const int i = i0 + u;
    v = z[i] > 0.0f ? v : 0.0f;
    if (dz_l) dz_l[i] = v;
    if (dz_g) dz_g[i] = v;
  }
  __syncthreads();
}

__global__ __launch_bounds__(kMlpThreads) void mlp_bwd_act_kernel(const float* __restrict__ W2,
                                                                  const float* __restrict__ W3,
                                                                  const float* __restrict__ dpsi,
                                                                  const float* __restrict__ z1,
                                                                  const float* __restrict__ z2, int hidden, int K,
                                                                  float* __restrict__ dz1, float* __restrict__ dz2) {
  __shared__ float part[16 * kMlpMaxIn];
  __shared__ float gk[kMlpMaxIn], gh[kMlpMaxIn];
  const int b = blockIdx.x, q = blockIdx.y;
  for (int k = threadIdx.x; k < K; k += kMlpThreads) gk[k] = dpsi[(int64_t)b * K + k];
  __syncthreads();
  mlp_act_back(W3, gk, K, hidden, 0, hidden, z2 + (int64_t)b * hidden, part, gh,
               q == 0 ? dz2 + (int64_t)b * hidden : nullptr);
  const int per = (hidden + kActParts - 1) / kActParts;
  const int i0 = min(hidden, q * per), i1 = min(hidden, i0 + per);
  mlp_act_back(W2, gh, hidden, hidden, i0, i1, z1 + (int64_t)b * hidden, part, nullptr, dz1 + (int64_t)b * hidden);
}

// sum over frames b of x[b xs] * act(y[b ys]) (y absent: of x[b xs]), in frame
// order, one rounding per step; frames are read 16 at a time (index clamped
// into range) so that their loads are in flight together, and the steps past
// the last frame add exact zeros (0 * 0), which leave the sum as it is.
template <bool HAS_Y, bool RELU_Y>
__device__ __forceinline__ float frame_sum(int B, const float* x, int64_t xs, const float* y, int64_t ys) {
  float s = 0.0f;
  for (int b0 = 0; b0 < B; b0 += 16) {
    float xv[16], yv[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int64_t b = min(b0 + u, B - 1);
      const bool in = b0 + u < B;
      const float xl = x[b * xs], yl = HAS_Y ? y[b * ys] : 1.0f;
      xv[u] = in ? xl : 0.0f;
      yv[u] = in ? (RELU_Y ? fmaxf(yl, 0.0f) : yl) : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) s = HAS_Y ? __builtin_fmaf(xv[u], yv[u], s) : s + xv[u];
  }
  return s;
}

__global__ __launch_bounds__(256) void mlp_bwd_param_kernel(const float* __restrict__ theta,
                                                            const float* __restrict__ z1,
                                                            const float* __restrict__ z2,
                                                            const float* __restrict__ dz1,
                                                            const float* __restrict__ dz2,
                                                            const float* __restrict__ dpsi, int B, int d_in,
                                                            int hidden, int K, float* __restrict__ dP) {
  const int64_t n1 = (int64_t)hidden * d_in, n2 = (int64_t)hidden * hidden, n3 = (int64_t)K * hidden;
  const int64_t total = n1 + hidden + n2 + hidden + n3 + K;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  float s;
  int64_t r = i;
  if (r < n1) {                                    // W1[j][c] = sum_b dz1[b][j] theta[b][c]
    const int j = (int)(r / d_in), c = (int)(r % d_in);
    s = frame_sum<true, false>(B, dz1 + j, hidden, theta + c, d_in);
  } else if ((r -= n1) < hidden) {                 // b1
    s = frame_sum<false, false>(B, dz1 + r, hidden, nullptr, 0);
  } else if ((r -= hidden) < n2) {                 // W2[j][c] = sum_b dz2[b][j] relu(z1[b][c])
    const int j = (int)(r / hidden), c = (int)(r % hidden);
    s = frame_sum<true, true>(B, dz2 + j, hidden, z1 + c, hidden);
  } else if ((r -= n2) < hidden) {                 // b2
    s = frame_sum<false, false>(B, dz2 + r, hidden, nullptr, 0);
  } else if ((r -= hidden) < n3) {                 // W3[k][c] = sum_b dpsi[b][k] relu(z2[b][c])
    const int k = (int)(r / hidden), c = (int)(r % hidden);
    s = frame_sum<true, true>(B, dpsi + k, K, z2 + c, hidden);
  } else {                                         // b3
    r -= n3;
    s = frame_sum<false, false>(B, dpsi + r, K, nullptr, 0);
  }
  dP[i] = s;
}

void launch_mlp_bwd(const float* params, const float* theta, const float* z1, const float* z2, const float* dpsi,
                    int B, int d_in, int hidden, int K, float* dz1, float* dz2, float* dparams, hipStream_t s) {
  if (B == 0) return;
  const float* W2 = params + (int64_t)hidden * d_in + hidden;
  const float* W3 = W2 + (int64_t)hidden * hidden + hidden;
  hipLaunchKernelGGL(mlp_bwd_act_kernel, dim3(B, kActParts), dim3(kMlpThreads), 0, s, W2, W3, dpsi, z1, z2, hidden,
                     K, dz1, dz2);
  const int64_t total = (int64_t)hidden * d_in + hidden + (int64_t)hidden * hidden + hidden + (int64_t)K * hidden + K;
  hipLaunchKernelGGL(mlp_bwd_param_kernel, dim3(div_up(total, 256)), dim3(256), 0, s, theta, z1, z2, dz1, dz2, dpsi,
                     B, d_in, hidden, K, dparams);
}

// ---------------------------------------------------------------- Adam
__global__ void adam_tick_kernel(StatusDev* status, int group, float b1, float b2, float* bc) {
  if (status->overflow) return;
  const int t = ++status->adam_step[group];
  bc[0] = (float)(1.0 - pow((double)b1, (double)t));
  bc[1] = (float)(1.0 - pow((double)b2, (double)t));
}

__global__ __launch_bounds__(256) void adam_kernel(const StatusDev* status, const float* __restrict__ bc,
                                                   float* __restrict__ p, const float* __restrict__ g,
                                                   float* __restrict__ m, float* __restrict__ v, int64_t n,
                                                   int64_t split, LrTable lr, float b1, float b2, float eps) {
  if (status->overflow) return;
  const float c1 = bc[0], c2 = bc[1];
  const float rc1 = 1.0f / c1, rsc2 = 1.0f / sqrtf(c2);
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const float rate = lr.v[(i >= split ? 16 : 0) + (int)(i & 15)];
    adam_update(p[i], m[i], v[i], g[i], rate, b1, b2, rc1, rsc2, eps);
  }
}

void launch_adam_tick(StatusDev* status, int group, float b1, float b2, hipStream_t s) {
  hipLaunchKernelGGL(adam_tick_kernel, dim3(1), dim3(1), 0, s, status, group, b1, b2, &status->adam_bc[group][0]);
}

void launch_adam(StatusDev* status, int group, float* p, const float* g, float* m, float* v, int64_t n,
                 int64_t split, const float* lr_table_host, float b1, float b2, float eps, hipStream_t s) {
  LrTable lr;
  for (int i = 0; i < 32; ++i) lr.v[i] = lr_table_host[i];
  launch_adam_tick(status, group, b1, b2, s);
  if (n == 0) return;
  const unsigned nb = (unsigned)std::min<int64_t>(div_up(n, 256), 8192);
  hipLaunchKernelGGL(adam_kernel, dim3(nb), dim3(256), 0, s, status, &status->adam_bc[group][0], p, g, m, v, n, split, lr,
                     b1, b2, eps);
}

}  // namespace gbr
