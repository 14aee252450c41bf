// Linear blending of Gaussian blendshapes (Eq. 1) and its adjoint.
//
// Forward:  raw[b][n][f] = sum_{k=0..K} w~[b][k] * bases[k][n][f],  w~[b][0] = 1,
//           w~[b][k] = weights[b][k-1].
// Adjoint:  dbases[k][n][f] = sum_b w~[b][k] draw[b][n][f]       (contract over frames)
//           dweights[b][k-1] = sum_{n,f} bases[k][n][f] draw[b][n][f]
//                                                               (contract over N*16)
//
// The blend and dbases contract over at most K+1 = 64 slices or the batch's
// frames: short contractions whose cost is reading and writing the slices,
// so one thread owns one (Gaussian, feature) element, reads each of its
// inputs once (coalesced across the threads) and writes each output once.
// The blend accumulates in float64 in slice order and rounds once: the
// products of two float32 values are exact in float64, so each frame's
// result is the float64 sum rounded to float32 and does not depend on the
// batch it is blended in.  dweights contracts over N*16 elements into a
// B x K result: a long dense contraction, done on the matrix cores
// (v_mfma_f32_16x16x4f32) with per-wave partials reduced in a fixed order.
#include <algorithm>
#include <type_traits>

#include "gbr_internal.h"

namespace gbr {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kBlendThreads = 256;
constexpr int kFrameGroup = 16;        // frames whose weights are staged together

// Kernels that keep a value per slice in registers are instantiated for every
// multiple of 8 slices and launched at the smallest that holds K + 1: slices
// past K are read (clamped) and multiplied for nothing: of 100k Gaussians and
// 8 frames the blend of 41 slices took 74 us in a 64-slice kernel and takes 62
// in one of 48, 31 slices 69 -> 45 (of 32), 6 slices 26 -> 19 (of 8).
template <typename F>
static void with_slices(int K, F&& launch) {
  switch (K / 8) {                     // ceil((K + 1) / 8) = K / 8 + 1
    case 0: launch(std::integral_constant<int, 8>()); break;
    case 1: launch(std::integral_constant<int, 16>()); break;
    case 2: launch(std::integral_constant<int, 24>()); break;
    case 3: launch(std::integral_constant<int, 32>()); break;
    case 4: launch(std::integral_constant<int, 40>()); break;
    case 5: launch(std::integral_constant<int, 48>()); break;
    case 6: launch(std::integral_constant<int, 56>()); break;
    default: launch(std::integral_constant<int, 64>()); break;
  }
}

// ---------------------------------------------------------------- forward
// The frames' weights, as float64 with the implicit 1 of slice 0, are laid
// out once in a table that every thread reads at the same address (scalar
// loads: each weight reaches the multiply-adds as a scalar operand).
__global__ void blend_weights_f64_kernel(const float* __restrict__ weights, int K, double* __restrict__ w64) {
  const int b = blockIdx.x, k = threadIdx.x;   // slices past K get weight 0
  w64[(int64_t)b * kBlendW64Stride + k] = (k == 0) ? 1.0 : (k <= K ? (double)weights[(int64_t)b * K + (k - 1)] : 0.0);
}

template <int KM>   // KM >= K + 1: slice values kept in registers
__device__ __forceinline__ void blend_element(const float* __restrict__ bases, const double* __restrict__ w64, int B,
                                              int K, int64_t N, int64_t i, float* __restrict__ raw) {
  const int64_t L = N * kNF;
  if (i >= L) return;
  const bool pad = (i % kNF) >= 14;
  // every load is issued unconditionally (slice index clamped into range) so
  // that they are all in flight together; slices past K are then zeroed
  float x[KM];
#pragma unroll
  for (int k = 0; k < KM; ++k) x[k] = bases[(int64_t)min(k, K) * L + i];
  double v[KM];
#pragma unroll
  for (int k = 0; k < KM; ++k) v[k] = (k <= K) ? (double)x[k] : 0.0;
  for (int b = 0; b < B; ++b) {
    const double* w = w64 + (int64_t)b * kBlendW64Stride;
    double acc = v[0];
#pragma unroll
    for (int k = 1; k < KM; ++k) acc = __builtin_fma(w[k], v[k], acc);   // exact product, one rounding per step
    raw[(int64_t)b * L + i] = pad ? 0.0f : (float)acc;
  }
}

template <int KM>
__global__ __launch_bounds__(kBlendThreads) void blend_fwd_kernel(const float* __restrict__ bases,
                                                                   const double* __restrict__ w64, int B, int K,
                                                                   int64_t N, float* __restrict__ raw) {
  blend_element<KM>(bases, w64, B, K, N, (int64_t)blockIdx.x * kBlendThreads + threadIdx.x, raw);
}

// The blends of several models in one launch (gbr_drive), so that one fills
// the chip where the last one's workgroups run out: 8 models of 20k to 100k
// Gaussians and 21 slices, 146 us in eight launches -> 123.
template <int KM>
__global__ __launch_bounds__(kBlendThreads) void blend_drive_kernel(DriveTable t) {
  const int gi = t.group_of(t.block0, blockIdx.x);
  const DriveGroup& g = t.g[gi];
  blend_element<KM>(g.bases, t.w64 + (int64_t)t.frame0[gi] * kBlendW64Stride, g.B, g.K, g.N,
                    (int64_t)(blockIdx.x - t.block0[gi]) * kBlendThreads + threadIdx.x, g.raw);
}

int64_t blend_drive_blocks(int64_t N) { return N / (kBlendThreads / kNF) + (N % (kBlendThreads / kNF) != 0); }

// Models of one instance (slices in eights) share a launch, and those of fewer
// slices join it while the slices they would read and multiply for nothing cost
// less than a launch of their own: some 0.3 to 0.45 ns a workgroup and eight
// slices against 4 us.  8 models' MLPs and blends (us, in one launch / as here):
// K = 20 and one of 63, 60k Gaussians 220 / 164, 20k 82 / 59, 2k 18 / 18; K = 7,
// 15, ... 63, 60k 245 / 217, 20k 93 / 86, 2k 19 / 19 (43 in eight); K = 20 and 25
// in turn, 60k 144 / 147, 20k 47 / 47 (52 in two).
constexpr int64_t kDriveWaste = 12000;

void launch_blend_drive(const DriveTable& t, hipStream_t s) {
  int64_t blocks8[kBlendW64Stride / 8] = {};   // workgroups per instance
  for (int i = 0; i < t.groups; ++i) blocks8[t.g[i].K / 8] += blend_drive_blocks(t.g[i].N);
  for (int hi = kBlendW64Stride / 8 - 1; hi >= 0;) {
    int lo = hi;                        // the launch takes instances [lo, hi]
    if (blocks8[hi] > 0)
      for (int64_t waste = 0; lo > 0 && (waste += blocks8[lo - 1] * (hi - lo + 1)) <= kDriveWaste;) --lo;
    DriveTable u;                       // (block0 alone is searched: frame0 keeps the weight rows)
    int n = 0;
    u.blocks = 0;
    for (int i = 0; i < t.groups; ++i) {
      const int k8 = t.g[i].K / 8;
      if (k8 < lo || k8 > hi) continue;
      u.g[n] = t.g[i];
      u.frame0[n] = t.frame0[i];
      u.block0[n] = u.blocks;
      u.blocks += (uint32_t)blend_drive_blocks(t.g[i].N);
      ++n;
    }
    if (n > 0) {
      u.close(n, t.frames, t.w64);
      with_slices(8 * hi, [&](auto km) {
        hipLaunchKernelGGL(blend_drive_kernel<km()>, dim3(u.blocks), dim3(kBlendThreads), 0, s, u);
      });
    }
    hi = lo - 1;
  }
}

void launch_blend_fwd(const float* bases, const float* weights, int B, int K, int64_t N, float* raw, double* w64,
                      hipStream_t s) {
  if (N == 0 || B == 0) return;
  hipLaunchKernelGGL(blend_weights_f64_kernel, dim3(B), dim3(kBlendW64Stride), 0, s, weights, K, w64);
  const dim3 grid(div_up(N * kNF, kBlendThreads));
  with_slices(K, [&](auto km) {
    hipLaunchKernelGGL(blend_fwd_kernel<km()>, grid, dim3(kBlendThreads), 0, s, bases, w64, B, K, N, raw);
  });
}

// ---------------------------------------------------------------- adjoint: dbases
// One thread per (Gaussian, feature): the frames' draw values are read once
// per group of 16, every slice's sum is kept in a register and added over
// the groups in frame order.  dbases_element forms those sums; the plain
// adjoint writes them, the fused step feeds them to Adam (so both see the
// same gradient).  Every thread of the workgroup must call it (barriers).
template <int KM>
__device__ __forceinline__ void dbases_element(const float* __restrict__ draw, const float* __restrict__ weights,
                                               int B, int K, int64_t L, int64_t i, bool live,
                                               float (&wt)[KM][kFrameGroup], float (&acc)[KM]) {
#pragma unroll
  for (int k = 0; k < KM; ++k) acc[k] = 0.0f;
  for (int b0 = 0; b0 < B; b0 += kFrameGroup) {
    const int nb = min(kFrameGroup, B - b0);
    __syncthreads();
    for (int t = threadIdx.x; t < kFrameGroup * KM; t += kBlendThreads) {
      const int bb = t / KM, k = t % KM;
      float x = 0.0f;
      if (bb < nb && k <= K) x = (k == 0) ? 1.0f : weights[(int64_t)(b0 + bb) * K + (k - 1)];
      wt[k][bb] = x;
    }
    __syncthreads();
    if (!live) continue;
    float d[kFrameGroup];
#pragma unroll
    for (int bb = 0; bb < kFrameGroup; ++bb) d[bb] = draw[(int64_t)(b0 + min(bb, nb - 1)) * L + i];
#pragma unroll
    for (int bb = 0; bb < kFrameGroup; ++bb) d[bb] = (bb < nb) ? d[bb] : 0.0f;   // (weights past nb are 0 too)
#pragma unroll
    for (int k = 0; k < KM; ++k) {
      if (k <= K) {
        float s = 0.0f;
#pragma unroll
        for (int bb = 0; bb < kFrameGroup; ++bb) s = __builtin_fmaf(wt[k][bb], d[bb], s);
        acc[k] += s;
      }
    }
  }
}

template <int KM>
__global__ __launch_bounds__(kBlendThreads) void blend_dbases_kernel(const float* __restrict__ draw,
                                                                      const float* __restrict__ weights, int B,
                                                                      int K, int64_t N, float* __restrict__ dbases,
                                                                      int accumulate) {
  __shared__ float wt[KM][kFrameGroup];   // slice-major: a slice's 16 weights in 4 loads
  const int64_t L = N * kNF;
  const int64_t i = (int64_t)blockIdx.x * kBlendThreads + threadIdx.x;
  const bool live = i < L;
  const bool pad = (i % kNF) >= 14;
  float acc[KM];
  dbases_element<KM>(draw, weights, B, K, L, i, live, wt, acc);
  if (!live) return;
#pragma unroll
  for (int k = 0; k < KM; ++k) {
    if (k <= K) {
      float* dst = &dbases[(int64_t)k * L + i];
      const float v = pad ? 0.0f : acc[k];
      *dst = accumulate ? *dst + v : v;
    }
  }
}

// The Adam step on the bases with the blend adjoint's dbases formed on the
// fly: each thread's K+1 gradients go straight into the update of its
// elements, so dbases is neither written nor read back.  Element k*L + i
// takes the rate lr[(k > 0) * 16 + i % 16].  The whole grid returns on an
// overflowed pass (the flag is uniform), before any barrier.
template <int KM>
__global__ __launch_bounds__(kBlendThreads) void blend_adam_kernel(const float* __restrict__ draw,
                                                                    const float* __restrict__ weights, int B, int K,
                                                                    int64_t N, float* __restrict__ p,
                                                                    float* __restrict__ m, float* __restrict__ v,
                                                                    const StatusDev* status, int group, LrTable lr,
                                                                    float b1, float b2, float eps) {
  __shared__ float wt[KM][kFrameGroup];
  if (status->overflow) return;
  const int64_t L = N * kNF;
  const int64_t i = (int64_t)blockIdx.x * kBlendThreads + threadIdx.x;
  const bool live = i < L;
  const bool pad = (i % kNF) >= 14;
  float acc[KM];
  dbases_element<KM>(draw, weights, B, K, L, i, live, wt, acc);
  if (!live) return;
  const float rc1 = 1.0f / status->adam_bc[group][0], rsc2 = 1.0f / sqrtf(status->adam_bc[group][1]);
#pragma unroll
  for (int k = 0; k < KM; ++k) {
    if (k <= K) {
      const int64_t e = (int64_t)k * L + i;
      const float rate = lr.v[(k > 0 ? 16 : 0) + (int)(i & 15)];
      adam_update(p[e], m[e], v[e], pad ? 0.0f : acc[k], rate, b1, b2, rc1, rsc2, eps);
    }
  }
}

void launch_blend_adam(const float* draw, const float* weights, int B, int K, int64_t N, float* p, float* m, float* v,
                       StatusDev* status, int group, const float* lr_table_host, float b1, float b2, float eps,
                       hipStream_t s) {
  LrTable lr;
  for (int i = 0; i < 32; ++i) lr.v[i] = lr_table_host[i];
  launch_adam_tick(status, group, b1, b2, s);
  if (N == 0 || B == 0) return;
  const dim3 g1(div_up(N * kNF, kBlendThreads));
  // (past 32 slices one of 64: the sizes between take more registers, 119 to
  // 153 against 109, and at 100k x 40 the update 396 us against 347)
  with_slices(K < 32 ? K : kBlendW64Stride - 1, [&](auto km) {
    hipLaunchKernelGGL(blend_adam_kernel<km()>, g1, dim3(kBlendThreads), 0, s, draw, weights, B, K, N, p, m, v, status,
                       group, lr, b1, b2, eps);
  });
}

// ---------------------------------------------------------------- adjoint: dweights
// A wave covers the flattened elements of a span of the N*16 per-slice
// vectors in blocks of 16: lane (x, q) loads 4 consecutive elements (q-th
// quarter) of frame x's draw and of slice x's (and 16 + x's, ...) base; each
// of the 4 components feeds one 16x16x4 product per 16 frames and 16 slices,
// contracted over the 4 quarters.  The pad features (14, 15) are skipped.
// The workgroup's four waves are added in LDS and it writes one [B][K]
// partial.  Of larger inputs kDwBlocks workgroups run, each wave over several spans
// whose sums are added in span order, and the kernel is instantiated per 16
// frames and 16 slices: bound by reading draw and the bases once.  64 frames
// of 100k Gaussians x 20: 172 + 62 (reduction) -> 150 + 5 us, where a partial per
// wave of 256 elements (32 MB, re-read at a stride of a partial) and products
// of 64 x 64 for 64 x 20 had cost as much again as the reading.  (With twice the
// workgroups it takes 158 + 8, with as many spans for every wave 172.)
constexpr int kDwSpan = 256;
constexpr int kDwBlocks = 1024;

template <int BT, int KT, bool MULTI>   // MULTI: several spans per wave
__global__ __launch_bounds__(256) void blend_dweights_kernel(const float* __restrict__ draw,
                                                              const float* __restrict__ bases, int B, int K,
                                                              int64_t N, float* __restrict__ partials) {
  __shared__ float ws[4][256];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int x = lane & 15, q = lane >> 4;
  const int64_t L = N * kNF;
  const int64_t spans = (L + kDwSpan - 1) / kDwSpan;
  const f4 zero = {0.f, 0.f, 0.f, 0.f};
  f4 acc[BT][KT], sum[BT][KT];              // a span's products; the spans before it
#pragma unroll
  for (int i = 0; i < BT; ++i)
#pragma unroll
    for (int j = 0; j < KT; ++j) acc[i][j] = sum[i][j] = zero;
  // Blocks of 16 elements, G at a time: every load of a group is issued
  // before its products, and the products of out-of-range rows are taken on
  // zeros rather than branched around, so that the group's loads are in
  // flight together.  A span's last group may run past its blocks: those
  // re-read the span's last block and are zeroed.
  constexpr int G = BT + KT <= 4 ? 4 : BT + KT <= 6 ? 2 : 1;
  for (int64_t sp = (int64_t)blockIdx.x * 4 + w; sp < spans; sp += (int64_t)gridDim.x * 4) {
    const int64_t e_begin = sp * kDwSpan;
    const int nit = (int)((min(L, e_begin + kDwSpan) - e_begin) / 16);   // (uniform; L is a multiple of 16)
    for (int it0 = 0; it0 < nit; it0 += G) {
      f4 a[G][BT], bb[G][KT];
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const bool live = it0 + u < nit;
        const int64_t e = e_begin + (int64_t)min(it0 + u, nit - 1) * 16 + 4 * q;
        // unconditional loads (row and block clamped into range), masked afterwards
#pragma unroll
        for (int i = 0; i < BT; ++i) {
          const int b = 16 * i + x;
          a[u][i] = *reinterpret_cast<const f4*>(draw + (int64_t)min(b, B - 1) * L + e);
          if (!(live && b < B)) a[u][i] = zero;
        }
#pragma unroll
        for (int j = 0; j < KT; ++j) {
          const int k = 16 * j + x + 1;
          bb[u][j] = *reinterpret_cast<const f4*>(bases + (int64_t)min(k, K) * L + e);
          if (!(live && k <= K)) bb[u][j] = zero;
        }
        if (q == 3) {                          // features 14 and 15 are pads
#pragma unroll
          for (int i = 0; i < BT; ++i) { a[u][i][2] = 0.f; a[u][i][3] = 0.f; }
#pragma unroll
          for (int j = 0; j < KT; ++j) { bb[u][j][2] = 0.f; bb[u][j][3] = 0.f; }
        }
      }
      __builtin_amdgcn_sched_barrier(0);      // keep the group's loads ahead of its products
#pragma unroll
      for (int u = 0; u < G; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int i = 0; i < BT; ++i)
#pragma unroll
            for (int j = 0; j < KT; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][i][c], bb[u][j][c], acc[i][j], 0, 0, 0);
    }
    if (!MULTI) break;
#pragma unroll
    for (int i = 0; i < BT; ++i)
#pragma unroll
      for (int j = 0; j < KT; ++j) {
        sum[i][j] += acc[i][j];
        acc[i][j] = zero;
      }
  }
  // D layout of the f32 16x16x4 op: lane l, item r holds row 4(l/16) + r, column l%16.
  float* out = partials + (int64_t)blockIdx.x * B * K;
#pragma unroll
  for (int i = 0; i < BT; ++i)
#pragma unroll
    for (int j = 0; j < KT; ++j) {
      if (i + j) __syncthreads();
#pragma unroll
      for (int r = 0; r < 4; ++r) ws[w][(4 * q + r) * 16 + x] = MULTI ? sum[i][j][r] : acc[i][j][r];
      __syncthreads();
      const int o = threadIdx.x, b = 16 * i + (o >> 4), k = 16 * j + (o & 15);
      if (b < B && k < K) out[(int64_t)b * K + k] = ((ws[0][o] + ws[1][o]) + ws[2][o]) + ws[3][o];
    }
}

// A workgroup per 16 outputs, 64 partials side by side: a thread sums the
// partials of its output 64 apart, 16 at a time in a tree (their loads in
// flight together), then a fixed-shape tree over the 64.  16 consecutive
// outputs are read as one 64-byte line.
constexpr int kRedCols = 16, kRedRows = 64;

__global__ __launch_bounds__(kRedCols * kRedRows) void reduce_partials_kernel(const float* __restrict__ partials,
                                                                              int n_part, int BK,
                                                                              float* __restrict__ out,
                                                                              int accumulate) {
  __shared__ float sm[kRedRows][kRedCols + 1];
  const int c = threadIdx.x % kRedCols, r = threadIdx.x / kRedCols;
  const int i = blockIdx.x * kRedCols + c, ic = min(i, BK - 1);
  float s = 0.0f;
  for (int p0 = r; p0 < n_part; p0 += 16 * kRedRows) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int p = p0 + u * kRedRows;
      const float x = partials[(int64_t)min(p, n_part - 1) * BK + ic];
      v[u] = p < n_part ? x : 0.0f;
    }
#pragma unroll
    for (int d = 8; d > 0; d >>= 1)
#pragma unroll
      for (int u = 0; u < d; ++u) v[u] += v[u + d];
    s += v[0];
  }
  sm[r][c] = s;
  __syncthreads();
  for (int d = kRedRows / 2; d > 0; d >>= 1) {
    if (r < d) sm[r][c] += sm[r + d][c];
    __syncthreads();
  }
  if (r == 0 && i < BK) out[i] = accumulate ? out[i] + sm[0][c] : sm[0][c];
}

// Both counts are the entry points' limits on a shape and exceed what the launch
// writes, a partial per workgroup, at most kDwBlocks of them.
int64_t blend_bwd_partials(int B, int K, int64_t N) {
  const int64_t waves = (int64_t)div_up(N * kNF, 4 * kDwSpan) * 4;
  return waves * (int64_t)B * K;
}

int64_t blend_bwd_partials_used(int B, int K, int64_t N) {
  if (K == 0) return 0;
  const int64_t blocks = (int64_t)div_up(N * kNF, 4 * kDwSpan);
  const bool small = B <= 16 && K <= 32;
  return (small ? blocks : 4 * blocks) * (int64_t)B * K;
}

template <int BT, bool MULTI>
static void launch_dweights(int blocks, const float* draw, const float* bases, int B, int K, int64_t N,
                            float* partials, hipStream_t s) {
  const dim3 g(blocks), t(256);
#define GBR_DW(KT) \
  hipLaunchKernelGGL((blend_dweights_kernel<BT, KT, MULTI>), g, t, 0, s, draw, bases, B, K, N, partials)
  if (K <= 16) GBR_DW(1);
  else if (K <= 32) GBR_DW(2);
  else if (K <= 48) GBR_DW(3);
  else GBR_DW(4);
#undef GBR_DW
}

template <bool MULTI>
static void launch_dweights(int blocks, const float* draw, const float* bases, int B, int K, int64_t N,
                            float* partials, hipStream_t s) {
  if (B <= 16) launch_dweights<1, MULTI>(blocks, draw, bases, B, K, N, partials, s);
  else if (B <= 32) launch_dweights<2, MULTI>(blocks, draw, bases, B, K, N, partials, s);
  else if (B <= 48) launch_dweights<3, MULTI>(blocks, draw, bases, B, K, N, partials, s);
  else launch_dweights<4, MULTI>(blocks, draw, bases, B, K, N, partials, s);
}

void launch_blend_bwd(const float* draw, const float* bases, const float* weights, int B, int K, int64_t N,
                      float* dbases, float* dweights, float* partials, int64_t n_partials, int accumulate,
                      hipStream_t s) {
  if (N == 0 || B == 0) return;
  const dim3 g1(div_up(N * kNF, kBlendThreads));
  // (past 40 slices one of 64, as for the update below: at 100k Gaussians and 8
  // frames 43 slices 80 us so and 87 in an instance of 48, 55 slices 92 and 108
  // in one of 56; 39 slices 77 and 72 in one of 40, 31 slices 60 and 53)
  if (dbases)
    with_slices(K < 40 ? K : kBlendW64Stride - 1, [&](auto km) {
      hipLaunchKernelGGL(blend_dbases_kernel<km()>, g1, dim3(kBlendThreads), 0, s, draw, weights, B, K, N, dbases,
                         accumulate);
    });
  if (K == 0) return;
  // (one or two products a block: a few more workgroups than kDwBlocks still
  // finish sooner with a span each than some of their waves with two: 16 frames
  // of 80k x 31 44 -> 40 us, 66k 40 -> 37; with more products, 32 frames of 80k x
  // 20 67 -> 72, 64 of 97k x 8 102 -> 112)
  const int line = B <= 16 && K <= 32 ? kDwBlocks * 3 / 2 : kDwBlocks;
  const int all = div_up(N * kNF, 4 * kDwSpan), blocks = all > line ? kDwBlocks : all;
  if (all > blocks) launch_dweights<true>(blocks, draw, bases, B, K, N, partials, s);
  else launch_dweights<false>(blocks, draw, bases, B, K, N, partials, s);
  (void)n_partials;
  hipLaunchKernelGGL(reduce_partials_kernel, dim3(div_up(B * K, kRedCols)), dim3(kRedCols * kRedRows), 0, s, partials,
                     blocks, B * K, dweights, accumulate);
}

}  // namespace gbr
