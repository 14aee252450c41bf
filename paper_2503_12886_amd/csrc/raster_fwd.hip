// Forward half of the batch-parallel rasterizer (Sec. 3.2): preprocess of
// every (frame, Gaussian), tile binning, per-tile depth order and front-to-back
// compositing, for all frames of a batch with no host synchronisation.
#include "gbr_device.h"
#include "tangent_ops.h"

namespace gbr {

// ---------------------------------------------------------------- fills
__global__ void fill_u32_kernel(uint32_t* p, uint32_t v, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}
__global__ void fill_f32_kernel(float* p, float v, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}
void launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)std::min<int64_t>(div_up(n, 256), 4096)), dim3(256), 0, s, p, v, n);
}
void launch_fill_f32(float* p, float v, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(fill_f32_kernel, dim3((unsigned)std::min<int64_t>(div_up(n, 256), 4096)), dim3(256), 0, s, p, v, n);
}

// ---------------------------------------------------------------- exclusive scan (u32)
// out[k] = sum of in[0..k), out[n] = the grand total.  Two passes:
// per-block totals, then every block adds the totals of the blocks before it
// (read directly, summed in 64 bits) to its own rescan.  The grand total is
// published (and checked against a capacity) by the workgroup that writes
// out[n].  Integer sums, so the order does not matter for the result.  The
// depth buckets' scan (below) and one of this kind share a launch pair: the
// buckets' blocks come first in the grid.
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanBlock = kScanThreads * kScanItems;

__device__ __forceinline__ void publish_total(unsigned long long total, StatusDev* status, int64_t cap_check,
                                              unsigned long long* total_out) {
  if (total_out) *total_out = total;
  if (cap_check >= 0 && total > (unsigned long long)cap_check) status->overflow |= 1u;
}

__device__ __forceinline__ void scan_totals_block(const ScanJob& J, int blk, uint32_t* lw) {
  const uint32_t* __restrict__ in = J.in;
  const int64_t n = J.n;
  const int64_t base = (int64_t)blk * kScanBlock;
  // loads issued unconditionally (index clamped into range), then masked
  uint32_t v[kScanItems];
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t k = base + (int64_t)i * kScanThreads + threadIdx.x;
    v[i] = (n > 0) ? in[min(k, n - 1)] : 0u;
  }
  uint32_t s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) s += (base + (int64_t)i * kScanThreads + threadIdx.x < n) ? v[i] : 0u;
  uint32_t tot;
  block_excl_scan<kScanThreads>(s, lw, &tot);
  if (threadIdx.x == 0) J.block_sums[blk] = tot;
}

// The scan of the depth buckets: bkt_count holds a row of nbk counts per (frame,
// block of splats); a bucket's start is the number of splats in the buckets
// before it, and each block's offset in a bucket follows the blocks before
// it.  A workgroup takes kBktScan buckets, two to a thread, and reads every
// block's row of them (rows are contiguous, for the count and the scatter pass
// as well: with a bucket's blocks adjacent, each of those passes' accesses was
// a line of its own).  The totals lie in the tiles' bitmap rows, which are
// built later: at least 32 words a frame, where 16 are used.
constexpr int kBktScan = 2 * kScanThreads;

struct BucketPair {
  const uint32_t* row;       // the pair's counts in the first block's row
  int64_t out;               // and its index in the buckets; < 0: none
};
__device__ __forceinline__ BucketPair bucket_pair(const PassArgs& a, int blk) {
  const int64_t k = (int64_t)blk * kBktScan + 2 * threadIdx.x;   // (nbk is a power of two >= 64: a pair has one frame)
  if (k >= (int64_t)a.B * a.nbk) return BucketPair{a.bkt_count, -1};
  const int64_t b = k / a.nbk;
  return BucketPair{a.bkt_count + b * a.nblk * a.nbk + k % a.nbk, k};
}
__device__ __forceinline__ uint2 bucket_sums(const PassArgs& a, const BucketPair& P) {
  uint2 c = make_uint2(0u, 0u);
#pragma unroll 8
  for (int j = 0; j < a.nblk; ++j) {
    const uint2 v = *reinterpret_cast<const uint2*>(P.row + (int64_t)j * a.nbk);
    c.x += v.x;
    c.y += v.y;
  }
  return P.out < 0 ? make_uint2(0u, 0u) : c;
}

__global__ __launch_bounds__(kScanThreads) void order_totals_kernel(PassArgs a, ScanJob side, int nb0) {
  __shared__ uint32_t lw[kScanThreads / 64];
  if ((int)blockIdx.x >= nb0) return scan_totals_block(side, (int)blockIdx.x - nb0, lw);
  const uint2 c = bucket_sums(a, bucket_pair(a, (int)blockIdx.x));
  uint32_t tot;
  block_excl_scan<kScanThreads>(c.x + c.y, lw, &tot);
  if (threadIdx.x == 0) a.tbits[blockIdx.x] = tot;
}

__device__ __forceinline__ void bucket_apply_block(const PassArgs& a, int blk) {
  __shared__ uint32_t lw[kScanThreads / 64];
  __shared__ uint32_t wsum[kScanThreads / 64];
  const BucketPair P = bucket_pair(a, blk);
  const uint2 c = bucket_sums(a, P);
  uint32_t part = 0;
  for (int k = threadIdx.x; k < blk; k += kScanThreads) part += a.tbits[k];
  part = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(part), 63);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = part;
  const uint32_t ex = block_excl_scan<kScanThreads>(c.x + c.y, lw, nullptr);   // (orders wsum as well)
  if (P.out < 0) return;
  uint32_t x = ex + ((wsum[0] + wsum[1]) + (wsum[2] + wsum[3])), y = x + c.x;
  *reinterpret_cast<uint2*>(a.bkt_start + P.out) = make_uint2(x, y);
  if (P.out + 2 == (int64_t)a.B * a.nbk) a.bkt_start[P.out + 2] = y + c.y;
  uint32_t* out = a.bkt_moff + (P.row - a.bkt_count);
#pragma unroll 8
  for (int j = 0; j < a.nblk; ++j) {
    const uint2 v = *reinterpret_cast<const uint2*>(P.row + (int64_t)j * a.nbk);
    *reinterpret_cast<uint2*>(out + (int64_t)j * a.nbk) = make_uint2(x, y);
    x += v.x;
    y += v.y;
  }
}

__device__ __forceinline__ void scan_apply_block(const ScanJob& J, int blk, StatusDev* status) {
  __shared__ uint32_t tile[kScanBlock];
  __shared__ uint32_t lw[kScanThreads / 64];
  __shared__ unsigned long long wsum[kScanThreads / 64];
  const uint32_t* __restrict__ in = J.in;
  const uint32_t* __restrict__ block_sums = J.block_sums;
  uint32_t* __restrict__ out = J.out;
  const int64_t n = J.n;
  const int64_t base = (int64_t)blk * kScanBlock;
  uint32_t v[kScanItems];
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) v[i] = (n > 0) ? in[min(base + i * kScanThreads + threadIdx.x, n - 1)] : 0u;
  // this block's offset: the totals of the blocks before it
  unsigned long long part = 0;
  for (int k = threadIdx.x; k < blk; k += kScanThreads) part += block_sums[k];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = part;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int idx = i * kScanThreads + threadIdx.x;
    tile[idx] = (base + idx < n) ? v[i] : 0u;
  }
  __syncthreads();
  unsigned long long off = 0;
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w) off += wsum[w];
  uint32_t local[kScanItems];
  uint32_t s = 0;
  for (int i = 0; i < kScanItems; ++i) {
    local[i] = tile[threadIdx.x * kScanItems + i];
    s += local[i];
  }
  uint32_t ex = block_excl_scan<kScanThreads>(s, lw, nullptr);
  for (int i = 0; i < kScanItems; ++i) {
    tile[threadIdx.x * kScanItems + i] = ex;
    ex += local[i];
  }
  __syncthreads();
  for (int i = 0; i < kScanItems; ++i) {
    const int idx = i * kScanThreads + threadIdx.x;
    const int64_t k = base + idx;
    if (k < n) {
      const uint32_t val = (uint32_t)(off + tile[idx]);
      out[k] = val;
    }
  }
  // out[n] = grand total, written by the block that holds position n
  if (threadIdx.x == kScanThreads - 1 && base <= n && n < base + kScanBlock) {
    const unsigned long long total = off + ex;   // ex of the last thread: the block's running total
    out[n] = (uint32_t)total;
    publish_total(total, status, J.cap_check, J.total_out);
  }
}

__global__ __launch_bounds__(kScanThreads) void order_apply_kernel(PassArgs a, ScanJob side, int nb0) {
  if ((int)blockIdx.x >= nb0) scan_apply_block(side, (int)blockIdx.x - nb0, a.status);
  else bucket_apply_block(a, (int)blockIdx.x);
}

__global__ __launch_bounds__(kScanThreads) void scan_totals_kernel(ScanJob J) {
  __shared__ uint32_t lw[kScanThreads / 64];
  scan_totals_block(J, (int)blockIdx.x, lw);
}
__global__ __launch_bounds__(kScanThreads) void scan_apply_kernel(ScanJob J, StatusDev* status) {
  scan_apply_block(J, (int)blockIdx.x, status);
}

int64_t scan_scratch_words(int64_t n) { return div_up(n + 1, kScanBlock) + 1; }

void launch_scan(const ScanJob& J, StatusDev* status, hipStream_t s) {
  const int nb = (int)div_up(J.n + 1, kScanBlock);
  hipLaunchKernelGGL(scan_totals_kernel, dim3(nb), dim3(kScanThreads), 0, s, J);
  hipLaunchKernelGGL(scan_apply_kernel, dim3(nb), dim3(kScanThreads), 0, s, J, status);
}

void launch_bucket_scan(const PassArgs& a, const ScanJob& side, hipStream_t s) {
  const int nb0 = (int)div_up((int64_t)a.B * a.nbk, kBktScan);
  const dim3 grid(nb0 + (int)div_up(side.n + 1, kScanBlock));
  hipLaunchKernelGGL(order_totals_kernel, grid, dim3(kScanThreads), 0, s, a, side, nb0);
  hipLaunchKernelGGL(order_apply_kernel, grid, dim3(kScanThreads), 0, s, a, side, nb0);
}

// ---------------------------------------------------------------- preprocess
// One thread per (frame, Gaussian).  Activations and EWA projection in
// float64 (so that the integer decisions -- which pixels and tiles a Gaussian
// may reach, and its binary32 depth key -- are exactly reproducible), the
// per-pixel record rounded to float32.  Each block also reduces its splats'
// depth keys to a minimum and maximum, stored in the block's own slot (the
// depth passes take the frame's range, which scales the depth buckets, from
// those slots).  The pass's first kernel, it also clears the pass's counters
// (tile-class counts, overflow flag) in block (0, 0).
struct Projected {
  bool valid;
  double mx, my, A, Bq, C, o, tz;
  int x0, x1, y0, y1;
};

// v0, v1, v2: the first three float4 of a blended record (position,
// quaternion, log-scales, opacity logit, red).
__device__ __forceinline__ void project_gaussian(const float4 v0, const float4 v1, const float4 v2, const FrameDev& F,
                                                 Projected& p) {
  p.valid = false;
  const double mu0 = v0.x, mu1 = v0.y, mu2 = v0.z;
  const double tx = (double)F.R[0] * mu0 + (double)F.R[1] * mu1 + (double)F.R[2] * mu2 + (double)F.t[0];
  const double ty = (double)F.R[3] * mu0 + (double)F.R[4] * mu1 + (double)F.R[5] * mu2 + (double)F.t[1];
  const double tz = (double)F.R[6] * mu0 + (double)F.R[7] * mu1 + (double)F.R[8] * mu2 + (double)F.t[2];
  p.tz = tz;
  if (!(tz > (double)F.near_z)) return;
  double qw = v0.w, qx = v1.x, qy = v1.y, qz = v1.z;
  const double qinv = 1.0 / sqrt(qw * qw + qx * qx + qy * qy + qz * qz);
  qw *= qinv; qx *= qinv; qy *= qinv; qz *= qinv;
  const double s0 = exp((double)v1.w), s1 = exp((double)v2.x), s2 = exp((double)v2.y);
  p.o = 1.0 / (1.0 + exp(-(double)v2.z));
  // rotation of the unit quaternion, columns scaled: M = R(q) diag(s)
  const double M00 = (1.0 - 2.0 * (qy * qy + qz * qz)) * s0, M01 = 2.0 * (qx * qy - qw * qz) * s1,
               M02 = 2.0 * (qx * qz + qw * qy) * s2;
  const double M10 = 2.0 * (qx * qy + qw * qz) * s0, M11 = (1.0 - 2.0 * (qx * qx + qz * qz)) * s1,
               M12 = 2.0 * (qy * qz - qw * qx) * s2;
  const double M20 = 2.0 * (qx * qz - qw * qy) * s0, M21 = 2.0 * (qy * qz + qw * qx) * s1,
               M22 = (1.0 - 2.0 * (qx * qx + qy * qy)) * s2;
  // W = J Rcam, the 2x3 local affine map of the perspective projection
  const double iz = 1.0 / tz;
  const double jx = (double)F.fx * iz, jy = (double)F.fy * iz;
  const double ux = -jx * tx * iz, uy = -jy * ty * iz;
  double W0[3], W1[3];
  for (int j = 0; j < 3; ++j) {
    W0[j] = jx * (double)F.R[j] + ux * (double)F.R[6 + j];
    W1[j] = jy * (double)F.R[3 + j] + uy * (double)F.R[6 + j];
  }
  // V = W M;  Sigma2 = V V^T + lowpass I
  const double V00 = W0[0] * M00 + W0[1] * M10 + W0[2] * M20;
  const double V01 = W0[0] * M01 + W0[1] * M11 + W0[2] * M21;
  const double V02 = W0[0] * M02 + W0[1] * M12 + W0[2] * M22;
  const double V10 = W1[0] * M00 + W1[1] * M10 + W1[2] * M20;
  const double V11 = W1[0] * M01 + W1[1] * M11 + W1[2] * M21;
  const double V12 = W1[0] * M02 + W1[1] * M12 + W1[2] * M22;
  const double sa = V00 * V00 + V01 * V01 + V02 * V02 + kLowPass;
  const double sb = V00 * V10 + V01 * V11 + V02 * V12;
  const double sc = V10 * V10 + V11 * V11 + V12 * V12 + kLowPass;
  p.mx = (double)F.fx * tx * iz + (double)F.cx;
  p.my = (double)F.fy * ty * iz + (double)F.cy;
  const double det = sa * sc - sb * sb;
  if (!(det > 0.0)) return;
  p.A = sc / det; p.Bq = -sb / det; p.C = sa / det;
  // alpha >= 1/255 needs q <= 2 ln(255 o); axis-aligned half extents of that ellipse
  const double thr = 2.0 * log(255.0 * p.o);
  if (!(thr >= 0.0)) return;
  const double ex = sqrt(thr * sa) + kBoxPad, ey = sqrt(thr * sc) + kBoxPad;
  double fx0 = ceil(p.mx - ex - 0.5), fx1 = floor(p.mx + ex - 0.5);
  double fy0 = ceil(p.my - ey - 0.5), fy1 = floor(p.my + ey - 0.5);
  fx0 = fmax(fx0, 0.0); fy0 = fmax(fy0, 0.0);
  fx1 = fmin(fx1, (double)(F.W - 1)); fy1 = fmin(fy1, (double)(F.H - 1));
  if (fx0 > fx1 || fy0 > fy1) return;
  p.x0 = (int)fx0; p.x1 = (int)fx1; p.y0 = (int)fy0; p.y1 = (int)fy1;
  p.valid = true;
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, o, 64));
  return v;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o, 64));
  return v;
}

// The pass's frames: in device memory already, or in the kernel's arguments,
// from where the first workgroup stores them for the kernels that follow.
struct StoredFrames {
  __device__ __forceinline__ const FrameDev& at(const PassArgs& a, int b) const { return a.frames[b]; }
  __device__ __forceinline__ void store(const PassArgs&) const {}
};
struct ArgFrames {
  FrameDev f[kArgFrames];
  __device__ __forceinline__ const FrameDev& at(const PassArgs&, int b) const { return f[b]; }
  __device__ __forceinline__ void store(const PassArgs& a) const {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(f);
    uint32_t* dst = reinterpret_cast<uint32_t*>(const_cast<FrameDev*>(a.frames));
    for (int i = threadIdx.x; i < a.B * (int)(sizeof(FrameDev) / 4); i += 256) dst[i] = src[i];
  }
};
static_assert(sizeof(PassArgs) + sizeof(ArgFrames) + sizeof(void*) <= 4096, "a kernel's arguments take 4 KB");

template <typename Frames>
__global__ __launch_bounds__(256) void preprocess_kernel(PassArgs a, Frames frames, const float* __restrict__ raw) {
  __shared__ uint32_t wmin[4], wmax[4];
  const int b = blockIdx.y;
  const FrameDev& F = frames.at(a, b);
  const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.x == 0 && b == 0) {   // the pass's counters: this is its first kernel
    frames.store(a);
    if (threadIdx.x < 66) a.cls_cnt[threadIdx.x] = 0u;
    if (threadIdx.x == 0) { a.status->overflow = 0u; a.status->entries = 0ull; }
  }
  if ((int64_t)blockIdx.x * 256 >= F.gauss_count) return;   // uniform per block
  const int tsh = __ffs(a.tile) - 1;                         // tile is a power of two
  uint32_t dmin = 0xffffffffu, dmax = 0u;
  if (n < F.gauss_count) {
    const int64_t s = F.gauss_base + n;
    const float4* src = reinterpret_cast<const float4*>(raw + s * kNF);
    float4 v0 = src[0], v1 = src[1];
    const float4 col = src[2];              // log-scales 1-2, opacity logit, red
    const float4 col2 = src[3];             // green, blue
    if (a.tg.on) tangent_deform(a.tg, b, n, v0, v1, v0, v1);   // tangent space -> frame b's mesh
    Projected p;
    project_gaussian(v0, v1, col, F, p);
    float* rec = a.rec + s * kRecF;
    int4 r = make_int4(0, 0, -1, -1);
    uint32_t count = 0, key = 0xffffffffu;
    if (p.valid) {
      r = make_int4(p.x0 >> tsh, p.y0 >> tsh, p.x1 >> tsh, p.y1 >> tsh);
      count = (uint32_t)((r.z - r.x + 1) * (r.w - r.y + 1));
      const float4 r0 = make_float4((float)p.mx, (float)p.my, (float)(-0.5 * kLog2e * p.A), (float)(-kLog2e * p.Bq));
      const float4 r1 = make_float4((float)(-0.5 * kLog2e * p.C), (float)log2(p.o), col.w, col2.x);
      const float4 r2 = make_float4(col2.y, (float)p.tz,
                                    __uint_as_float((uint32_t)p.x0 | ((uint32_t)p.x1 << 16)),
                                    __uint_as_float((uint32_t)p.y0 | ((uint32_t)p.y1 << 16)));
      reinterpret_cast<float4*>(rec)[0] = r0;
      reinterpret_cast<float4*>(rec)[1] = r1;
      reinterpret_cast<float4*>(rec)[2] = r2;
      key = __float_as_uint(r2.y);
      dmin = key; dmax = key;
    } else {
      reinterpret_cast<float4*>(rec)[2] = make_float4(0.0f, (float)p.tz, 0.0f, 0.0f);
    }
    a.rect[s] = r;
    a.cnt[s] = count;
    a.dkey[s] = key;
  }
  // the block's depth range (wave reductions), stored in its own slot: the
  // depth passes reduce the frame's slots, so nothing is cleared or merged
  dmin = wave_min_u32(dmin);
  dmax = wave_max_u32(dmax);
  if ((threadIdx.x & 63) == 0) { wmin[threadIdx.x >> 6] = dmin; wmax[threadIdx.x >> 6] = dmax; }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t* mm = a.blk_mm + 2 * (F.gauss_base / 256 + b + blockIdx.x);
    mm[0] = min(min(wmin[0], wmin[1]), min(wmin[2], wmin[3]));
    mm[1] = max(max(wmax[0], wmax[1]), max(wmax[2], wmax[3]));
  }
}

bool launch_preprocess(const PassArgs& a, const FrameDev* host_frames, const float* raw, int64_t max_frame_splats,
                       hipStream_t s) {
  if (a.B == 0 || max_frame_splats == 0) return false;
  const dim3 grid(div_up(max_frame_splats, 256), a.B);
  if (host_frames) {
    ArgFrames f;
    for (int b = 0; b < kArgFrames; ++b) f.f[b] = host_frames[b < a.B ? b : 0];
    hipLaunchKernelGGL(preprocess_kernel<ArgFrames>, grid, dim3(256), 0, s, a, f, raw);
  } else {
    hipLaunchKernelGGL(preprocess_kernel<StoredFrames>, grid, dim3(256), 0, s, a, StoredFrames(), raw);
  }
  return true;
}

// ---------------------------------------------------------------- binning
// A tile's list is the set of frame-local depth ranks of the splats that
// overlap it.  Each tile owns a row of bitmap_words words (bit r = rank r);
// reading a row's set bits in ascending order gives the tile's list in depth
// order, so no entry array is scattered or sorted.  Rows are cut into
// segments of seg_words words, and the set bits of every segment are counted
// once (seg_cnt): the tile's entry count is their sum, and the compositing
// places each segment in the tile's order from those counts alone, reading
// only the segments it consumes.
//
// Rows are built by rank: workgroup j of a frame takes the splats of ranks
// [32 SW j, 32 SW (j + 1)), which own segment j (words [SW j, SW (j + 1)))
// of every row.  Each splat ORs its bit into an LDS copy of those SW words
// for every tile of its rect; the workgroup then stores the bit count of
// every tile's segment and the segments that have set bits.  Every count is
// written by exactly one workgroup, and a segment whose count is zero is
// never read (its words keep whatever an earlier pass left there), so
// nothing needs clearing and rows of empty tiles cost no stores.
// In LDS a tile's segment takes SW + 1 words: the lanes of a half-wave OR
// into the same word offset of their (scattered) tiles, and with a stride of
// SW words those tiles would share a couple of banks; an odd stride spreads
// them over all of them.  Frames with more tiles than the LDS copy holds set
// the bits in memory with atomics after clearing the rows, and count the
// segments in a second pass.
constexpr int kRowBuildWords = 2048 * 9;     // LDS words (72 KB): 2048 tiles at SW = 8, 1084 at SW = 16

int bitmap_seg_words(int max_frame_tiles, int64_t row_words) {
  int sw = (int64_t)max_frame_tiles * 17 <= kRowBuildWords ? 16 : 8;
  while (row_words / sw > kMaxRowSegs) sw *= 2;
  return sw;
}

template <int SW>
__global__ __launch_bounds__(32 * SW) void bitmap_rows_kernel(PassArgs a, int per) {
  constexpr int NT = 32 * SW;                 // one thread per rank of the segment
  constexpr int ST = SW + 1;                  // LDS words per tile
  __shared__ __align__(16) uint32_t words[kRowBuildWords];
  int b, seg;
  if (!frame_block(a, per, b, seg)) return;
  const FrameDev& F = a.frames[b];
  const uint32_t vbase = a.bkt_start[b * a.nbk];
  const uint32_t nv = a.bkt_start[(b + 1) * a.nbk] - vbase;
  const uint32_t r0 = seg * (uint32_t)NT;
  if (r0 >= nv || a.status->overflow) return;
  const int nw4 = F.n_tiles * (SW / 4);
  const int nz4 = (F.n_tiles * ST + 3) / 4;   // <= kRowBuildWords / 4 (a multiple of 4 words)
  uint4* w4 = reinterpret_cast<uint4*>(words);
  for (int q = threadIdx.x; q < nz4; q += NT) w4[q] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  const uint32_t r = r0 + threadIdx.x;
  if (r < nv) {
    const uint32_t s = a.depth_sorted[vbase + r];
    const int4 rc = a.rect[s];
    const uint32_t bit = 1u << (r & 31u);
    const int wl = (int)((r >> 5) & (SW - 1));
    for (int ty = rc.y; ty <= rc.w; ++ty)
      for (int tx = rc.x; tx <= rc.z; ++tx) atomicOr(&words[(ty * F.ntx + tx) * ST + wl], bit);
  }
  __syncthreads();
  // every tile's bit count, also kept in its segment's pad word
  uint16_t* cnt = a.seg_cnt + (int64_t)F.tile_base * a.seg_stride + seg;
  for (int t = threadIdx.x; t < F.n_tiles; t += NT) {
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < SW; ++k) c += __popc(words[t * ST + k]);
    cnt[(int64_t)t * a.seg_stride] = (uint16_t)c;
    words[t * ST + SW] = c;
  }
  __syncthreads();
  // the segments with set bits (16-byte stores; rows and segments are 64-byte aligned)
  uint32_t* rows = a.tbits + (int64_t)F.tile_base * a.bitmap_words + (int64_t)seg * SW;
  for (int q = threadIdx.x; q < nw4; q += NT) {
    const int t = q / (SW / 4), k = q % (SW / 4);
    const uint32_t* src = words + t * ST + 4 * k;
    if (words[t * ST + SW] == 0u) continue;
    reinterpret_cast<uint4*>(rows + (int64_t)t * a.bitmap_words)[k] = make_uint4(src[0], src[1], src[2], src[3]);
  }
}

__global__ __launch_bounds__(256) void bitmap_rows_atomic_kernel(PassArgs a) {
  const int b = blockIdx.y;
  const FrameDev& F = a.frames[b];
  const uint32_t vbase = a.bkt_start[b * a.nbk];
  const uint32_t nv = a.bkt_start[(b + 1) * a.nbk] - vbase;
  const uint32_t r = blockIdx.x * 256u + threadIdx.x;
  if (r >= nv || a.status->overflow) return;
  const uint32_t s = a.depth_sorted[vbase + r];
  const int4 rc = a.rect[s];
  const uint32_t bit = 1u << (r & 31u);
  uint32_t* base = a.tbits + (int64_t)F.tile_base * a.bitmap_words + (r >> 5);
  for (int ty = rc.y; ty <= rc.w; ++ty)
    for (int tx = rc.x; tx <= rc.z; ++tx) atomicOr(base + (int64_t)(ty * F.ntx + tx) * a.bitmap_words, bit);
}

// Bit counts of the segments of rows set in memory: a thread per (tile, segment).
__global__ __launch_bounds__(256) void seg_count_kernel(PassArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)a.n_tiles * a.seg_stride || a.status->overflow) return;
  const int64_t g = i / a.seg_stride;
  const int sg = (int)(i % a.seg_stride);
  const uint4* src = reinterpret_cast<const uint4*>(a.tbits + g * a.bitmap_words + (int64_t)sg * a.seg_words);
  uint32_t c = 0;
  for (int k = 0; k < a.seg_words / 4; ++k) {
    const uint4 v = src[k];
    c += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
  }
  a.seg_cnt[i] = (uint16_t)c;
}

void launch_bitmap_rows(const PassArgs& a, int64_t max_frame_splats, int max_frame_tiles, hipStream_t s) {
  if (a.B == 0 || max_frame_splats == 0) return;
  const bool in_lds = (int64_t)max_frame_tiles * (a.seg_words + 1) <= kRowBuildWords;
  const int per = (int)div_up(max_frame_splats, 32 * a.seg_words);
  if (in_lds && a.seg_words == 32) {
    hipLaunchKernelGGL(bitmap_rows_kernel<32>, frame_grid(a, per), dim3(1024), 0, s, a, per);
  } else if (in_lds && a.seg_words == 16) {
    hipLaunchKernelGGL(bitmap_rows_kernel<16>, frame_grid(a, per), dim3(512), 0, s, a, per);
  } else if (in_lds && a.seg_words == 8) {
    hipLaunchKernelGGL(bitmap_rows_kernel<8>, frame_grid(a, per), dim3(256), 0, s, a, per);
  } else {
    launch_fill_u32(a.tbits, 0u, (int64_t)a.n_tiles * a.bitmap_words, s);
    hipLaunchKernelGGL(bitmap_rows_atomic_kernel, dim3(div_up(max_frame_splats, 256), a.B), dim3(256), 0, s, a);
    hipLaunchKernelGGL(seg_count_kernel, dim3(div_up((int64_t)a.n_tiles * a.seg_stride, 256)), dim3(256), 0, s, a);
  }
}

// A tile's entry count is the sum of its row's segment counts: one wave per
// tile, lanes over the segments.  The first 128 counts are read (clamped to
// the row) before the frame's segment count is known, which only masks
// them, so that their loads overlap the frame lookup.
__global__ __launch_bounds__(256) void tile_count_kernel(PassArgs a) {
  // (the wave's tile, declared uniform so that the frame lookup runs on scalar loads)
  const int g = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (g >= a.n_tiles) return;
  const int lane = threadIdx.x & 63;
  const uint16_t* sc = a.seg_cnt + (int64_t)g * a.seg_stride;
  const uint32_t last = (uint32_t)a.seg_stride - 1u;
  const uint32_t v0 = sc[min((uint32_t)lane, last)], v1 = sc[min((uint32_t)lane + 64u, last)];
  const int b = frame_of_tile(a.frames, a.B, g);
  const uint32_t nv = a.bkt_start[(b + 1) * a.nbk] - a.bkt_start[b * a.nbk];
  const uint32_t nseg = ((nv + 31) / 32 + a.seg_words - 1) / a.seg_words;
  uint32_t c = ((uint32_t)lane < nseg ? v0 : 0u) + ((uint32_t)lane + 64u < nseg ? v1 : 0u);
  for (uint32_t q = lane + 128; q < nseg; q += 64) c += sc[q];
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
  if (lane == 0) a.tile_count[g] = c;
}

void launch_tile_count(const PassArgs& a, hipStream_t s) {
  if (a.n_tiles == 0) return;
  hipLaunchKernelGGL(tile_count_kernel, dim3(div_up(a.n_tiles, 4)), dim3(256), 0, s, a);
}

// ---------------------------------------------------------------- tile classes
// Forward: work = list length; backward: entries the forward pass used (also
// written out as the tile's last used position).  A workgroup of 1024 tiles
// counts its tiles per class in LDS, reserves one range per class in the
// class lists (33 global atomics), and writes its tiles there.  The forward
// classification needs only the tile counts, so it runs in the tile scan's
// first launch (workgroups after the scan's, 4 tiles per thread).
template <int NTH>
__device__ __forceinline__ void classify_block(const PassArgs& a, int blk, bool backward, uint32_t* cnt,
                                               uint32_t* base) {
  constexpr int PER = 1024 / NTH;   // tiles per thread
  if (threadIdx.x < 33) cnt[threadIdx.x] = 0u;
  __syncthreads();
  int c[PER];
  uint32_t slot[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int g = blk * 1024 + k * NTH + (int)threadIdx.x;
    c[k] = -1;
    slot[k] = 0;
    if (g < a.n_tiles) {
      uint32_t work;
      if (backward) {                     // the tile's last used position: the largest of its quadrants'
        const uint4 ql = reinterpret_cast<const uint4*>(a.qlast)[g];
        work = max(max(ql.x, ql.y), max(ql.z, ql.w));
        a.tile_last[g] = work;
      } else {
        work = a.tile_count[g];
      }
      c[k] = work_class(work);
      slot[k] = atomicAdd(&cnt[c[k]], 1u);
    }
  }
  __syncthreads();
  uint32_t* gcnt = a.cls_cnt + (backward ? 33 : 0);
  if (threadIdx.x < 33) base[threadIdx.x] = cnt[threadIdx.x] ? atomicAdd(&gcnt[threadIdx.x], cnt[threadIdx.x]) : 0u;
  __syncthreads();
  uint32_t* lists = backward ? a.order_bwd : a.order_fwd;
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (c[k] >= 0) lists[(int64_t)c[k] * a.n_tiles + base[c[k]] + slot[k]] = (uint32_t)(blk * 1024 + k * NTH + threadIdx.x);
}

__global__ __launch_bounds__(1024) void classify_tiles_kernel(PassArgs a, int backward) {
  __shared__ uint32_t cnt[33], base[33];
  classify_block<1024>(a, (int)blockIdx.x, backward != 0, cnt, base);
}

void launch_classify_tiles(const PassArgs& a, bool backward, hipStream_t s) {
  if (a.n_tiles == 0) return;
  hipLaunchKernelGGL(classify_tiles_kernel, dim3(div_up(a.n_tiles, 1024)), dim3(1024), 0, s, a, backward ? 1 : 0);
}

// The tile scan's totals pass (workgroups [0, nb)) and the forward
// classification (the rest, 1024 tiles each) in one launch.
__global__ __launch_bounds__(kScanThreads) void tile_totals_classify_kernel(ScanJob J, int nb0, PassArgs a) {
  __shared__ uint32_t lw[kScanThreads / 64];
  __shared__ uint32_t cnt[33], base[33];
  if ((int)blockIdx.x < nb0) scan_totals_block(J, (int)blockIdx.x, lw);
  else classify_block<kScanThreads>(a, (int)blockIdx.x - nb0, false, cnt, base);
}

// The same for fewer than kScanBlock tiles, whose scan is one block's: both in
// a launch, 3.5 + 3.0 -> 3.2 us for 1024 tiles, 4.5 + 4.8 -> 4.8 for 3360.
__global__ __launch_bounds__(kScanThreads) void tile_scan_classify_kernel(ScanJob J, PassArgs a) {
  __shared__ uint32_t cnt[33], base[33];
  if (blockIdx.x == 0) scan_apply_block(J, 0, a.status);
  else classify_block<kScanThreads>(a, (int)blockIdx.x - 1, false, cnt, base);
}

void launch_tile_scan_classify(const PassArgs& a, uint32_t* block_sums, int64_t cap_check,
                               unsigned long long* total_out, hipStream_t s) {
  const ScanJob J{a.tile_count, a.tile_start, a.n_tiles, block_sums, cap_check, total_out};
  const int nb0 = (int)div_up((int64_t)a.n_tiles + 1, kScanBlock);
  const int ncls = a.n_tiles > 0 ? div_up(a.n_tiles, 1024) : 0;
  if (nb0 == 1) {                             // one block: no totals to wait for
    hipLaunchKernelGGL(tile_scan_classify_kernel, dim3(1 + ncls), dim3(kScanThreads), 0, s, J, a);
    return;
  }
  hipLaunchKernelGGL(tile_totals_classify_kernel, dim3(nb0 + ncls), dim3(kScanThreads), 0, s, J, nb0, a);
  hipLaunchKernelGGL(scan_apply_kernel, dim3(nb0), dim3(kScanThreads), 0, s, J, a.status);
}

// ---------------------------------------------------------------- complete lists
// The whole sorted list of every tile, from its bitmap row: each thread owns
// a run of words, a block prefix count places its set bits, which it writes
// as splat indices (rank -> splat through the frame's depth order).  The
// forward pass orders each tile only as far as it composites; this pass
// completes the lists on request.
__global__ __launch_bounds__(256) void tile_lists_kernel(PassArgs a) {
  __shared__ uint32_t lw[4];
  if (a.status->overflow) return;
  const int g = blockIdx.x;
  const uint32_t start = a.tile_start[g];
  if (a.tile_start[g + 1] == start) return;
  const int b = frame_of_tile(a.frames, a.B, g);
  const uint32_t vbase = a.bkt_start[b * a.nbk];
  const uint32_t nv = a.bkt_start[(b + 1) * a.nbk] - vbase;
  const uint32_t W = (nv + 31) / 32;
  const uint32_t* row = a.tbits + (int64_t)g * a.bitmap_words;
  const uint16_t* segc = a.seg_cnt + (int64_t)g * a.seg_stride;
  const uint32_t sh = (uint32_t)__ffs(a.seg_words) - 1u;
  // the words of a segment with no set bits are not stored: read as zero
  auto word = [&](uint32_t w) { return segc[w >> sh] ? row[w] : 0u; };
  const uint32_t wpt = (W + 255) / 256;
  const uint32_t w0 = min(W, threadIdx.x * wpt), w1 = min(W, w0 + wpt);
  uint32_t c = 0;
  for (uint32_t w = w0; w < w1; ++w) c += __popc(word(w));
  uint32_t out = start + block_excl_scan<256>(c, lw, nullptr);
  for (uint32_t w = w0; w < w1; ++w) {
    uint32_t bits = word(w);
    while (bits) {
      const uint32_t bit = __ffs(bits) - 1u;
      bits &= bits - 1u;
      a.sorted[out++] = a.depth_sorted[vbase + w * 32u + bit];
    }
  }
}

void launch_tile_lists(const PassArgs& a, hipStream_t s) {
  if (a.n_tiles == 0) return;
  hipLaunchKernelGGL(tile_lists_kernel, dim3(a.n_tiles), dim3(256), 0, s, a);
}

// ---------------------------------------------------------------- compositing
// (pixels to threads: TileMap)
template <int T> using TileShape = TileMap<T>;

// Whether a splat's alpha >= 1/255 region may reach the rectangle
// [x0, x1] x [y0, y1] of pixel centres: the maximum of the concave power
// ca dx^2 + cb dx dy + cc dy^2 over the rectangle against
// -log2(255) - log2(o), less a margin of 0.01 that keeps the test
// conservative under float32 rounding (at that margin alpha is 0.7 % below
// the threshold).  The power grows along the way from any point to the mean,
// so its maximum lies on an edge that faces the mean (or at the mean, when
// the rectangle holds it): the edge at the rectangle's nearest x and the one
// at its nearest y are searched, each at its own best point (an error of
// that point only lowers the value to second order, so an approximate
// reciprocal will do).  The comparison keeps a NaN.  A splat that cannot
// reach a pixel is never taken there, so skipping it changes nothing.
__device__ __forceinline__ bool strip_reach(float4 r0, float4 r1, float x0, float x1, float y0, float y1) {
  const float ca = r0.z, cb = r0.w, cc = r1.x;
  x0 -= r0.x; x1 -= r0.x; y0 -= r0.y; y1 -= r0.y;
  const float xe = __builtin_amdgcn_fmed3f(0.0f, x0, x1), ye = __builtin_amdgcn_fmed3f(0.0f, y0, y1);
  const float h = -0.5f * cb;
  const float ya = __builtin_amdgcn_fmed3f(h * __builtin_amdgcn_rcpf(cc) * xe, y0, y1);
  const float xb = __builtin_amdgcn_fmed3f(h * __builtin_amdgcn_rcpf(ca) * ye, x0, x1);
  const float pa = (ca * xe + cb * ya) * xe + cc * ya * ya;
  const float pb = (ca * xb + cb * ye) * xb + cc * ye * ye;
  const float thr = -kLog2_255 - r1.y - 0.01f;
  return !(pa < thr) || !(pb < thr);
}

// The rectangle of the pixel centres of the lanes in M, the quadrant's first
// at (qx0, qy0): lanes are 8 per row, so a column runs if any of its 8 lanes
// does, a row if its byte of the wave mask is nonzero.
template <int PXW>
__device__ __forceinline__ void running_rect(unsigned long long M, float qx0, float qy0, float& sx0, float& sx1,
                                             float& sy0, float& sy1) {
  unsigned long long cm8 = M | (M >> 32);
  cm8 |= cm8 >> 16;
  cm8 |= cm8 >> 8;
  cm8 &= 0xffull;
  unsigned long long rm = M | (M >> 4);
  rm |= rm >> 2;
  rm |= rm >> 1;
  rm &= 0x0101010101010101ull;
  const int c0l = __ffsll((long long)cm8) - 1, c1l = 63 - __clzll((long long)cm8);
  const int r0l = (__ffsll((long long)rm) - 1) >> 3, r1l = (63 - __clzll((long long)rm)) >> 3;
  sx0 = qx0 + (float)(c0l * PXW);
  sx1 = qx0 + (float)(c1l * PXW + PXW - 1);
  sy0 = qy0 + (float)(r0l * PXW);
  sy1 = qy0 + (float)(r1l * PXW + PXW - 1);
}

// alpha of a splat at a pixel, bit-identical wherever it is evaluated:
// power = ca dx^2 + cb dx dy + cc dy^2 (= -q/2 in log2 units) plus lo =
// log2(opacity), clamped at lo (q >= 0), and alpha = 2^power = o 2^(-q/2 log2 e).
// The clamp is one v_min_f32 (min(power, lo) for every non-NaN power);
// written as such because fminf would first canonicalise lo, one more
// instruction per (entry, pixel).
__device__ __forceinline__ float splat_alpha(float4 r0, float cc, float lo, float px, float py, float& dx, float& dy,
                                             float& pw_raw) {
#pragma clang fp contract(off)
  dx = px - r0.x;
  dy = py - r0.y;
  float pw = __builtin_fmaf(r0.z * dx, dx, lo);
  pw = __builtin_fmaf(r0.w * dx, dy, pw);
  pw = __builtin_fmaf(cc * dy, dy, pw);
  pw_raw = pw;
  float pc;
  asm("v_min_f32 %0, %1, %2" : "=v"(pc) : "v"(pw), "v"(lo));
  return __builtin_amdgcn_exp2f(pc);
}

// The front-to-back step of an entry at a pixel: w is its alpha, or -0 where
// that is below 1/255 (the entry is skipped, Te passes unchanged).
// T (1 - alpha) < 1e-4 stops the pixel before this entry (Te -> -T); a stopped
// pixel has Te <= 0, so its tn <= 0 stops it again (Te kept: -|Te|) and it
// takes nothing.  Returns minus the entry's weight: negative where it is
// taken, else +0, so that its sign is the pixel's bit, which goes to took.
__device__ __forceinline__ float fold_step(float w, float& Te, uint32_t& took) {
  const float tn = __builtin_fmaf(-w, Te, Te);   // T (1 - alpha), rounded once
  const bool stop = tn < kTMin;
  const float nw = stop ? 0.0f : -w * Te;
  Te = stop ? -fabsf(Te) : tn;                   // one select with source modifiers
  took = __builtin_amdgcn_alignbit(took, __float_as_uint(nw), 31);
  return nw;
}

// Four staged candidates, in the nine 16-byte words that the wave reads them
// in (every lane the same): mean and conic's first two terms of each; (cc, lo)
// of each, lo = log2 opacity; colours.  The reads cost the LDS unit 5.7 cycles
// a word of 16 bytes, 4.7 of 8 and 11.3 of 12, shared by a CU's waves, which
// is as much as the blending takes of the vector units.
struct __align__(16) FwdGroup {
  static constexpr int N = 4;
  float4 v[9];
  __device__ __forceinline__ void put(int u, float4 q0, float4 q1, float qb) {
    float* f = reinterpret_cast<float*>(v);
    v[u] = q0;
    *reinterpret_cast<float2*>(f + 16 + 2 * u) = make_float2(q1.x, q1.y);
    f[24 + 3 * u] = q1.z; f[25 + 3 * u] = q1.w; f[26 + 3 * u] = qb;
  }
  __device__ __forceinline__ void pad(int u) {
    float* f = reinterpret_cast<float*>(v);
    f[17 + 2 * u] = -1e30f;
    f[24 + 3 * u] = 0.f; f[25 + 3 * u] = 0.f; f[26 + 3 * u] = 0.f;
  }
};

// One wave per (tile, quadrant): each wave composites its quadrant's pixels
// on its own, with no barrier shared with the other quadrants of the tile,
// and stops as soon as its own pixels have stopped.
//
// The tile's list is a stream of depth ranks, the set bits of its bitmap row
// in ascending order, produced 64 positions at a time: the row's segments
// with set bits are found 64 segments at a time from their counts, their
// words read 64 at a time (a word per lane, the next 64 read ahead), and
// each word's bits are emitted once, as positions are asked for.  Three
// batches are in flight: while batch i is composited, the records of batch
// i + 1 and the splat indices of batch i + 2 are on their way, so that the
// chain segment counts -> words -> rank -> splat -> record costs its four
// load latencies once per tile and not once per batch.
//
// The entries of a batch whose alpha >= 1/255 region may reach the wave's
// running pixels are compacted into LDS in list order (a lane tests an
// entry); the compositing then walks that dense array 4 at a time with a
// uniform counter.  Per (entry, pixel) the front-to-back step is written on
// the pixel's signed transmittance Te (its transmittance while it runs; once
// it has stopped, minus the transmittance at the stop), so every decision is
// a vector compare and select; which entries a pixel took is kept in a word a
// lane, from which the wave's mask and the pixel's last position follow once
// in 32 entries.  Entries behind the wave's stop are not
// composited; at most two batches of them are read.  The consumed part of the
// sorted list is written out for the backward pass (the quadrant waves of a
// tile write identical values), with a 64-bit mask per batch of the entries
// that the quadrant took and the quadrant's last used position.  The quadrant
// waves of a tile get block indices of the same residue mod 8, so that they
// run on one XCD and share its L2.
//
// Measured (us, against a batch read through its four latencies in turn, the
// words of straddling segments read and emitted twice): one 512 x 512 frame
// of 50k Gaussians 117 -> 84, 16 of them 223 -> 218, 10 mesh-bound frames 353
// -> 275, 64 uneven frames of 100k 1044 -> 980.  With the clamp in the power,
// the takes as sign bits per lane (they were a wave mask, a select and two
// scalar operations an entry) and four entries in nine words (three, in eight
// reads of 8 or 16 bytes): 84 -> 78, 217 -> 209, 267 -> 256, 960 -> 960.  16
// frames issue 110 million vector instructions, 185 us of the 209.  Three
// entries at a time, 72 registers and 7 waves a SIMD: 84, 207, 270, 1009.
// Waves of long lists at a raised issue priority: slower.
constexpr int kFwdBatch = 64;
constexpr uint32_t kFwdRing = 256;   // a power of two >= 64 + 32: a whole word fits behind a batch

// The stream of a tile's depth ranks (see the compositing below), run by one wave.
struct RankStream {
  const uint32_t* row;
  const uint16_t* segc;
  const uint32_t* sorted;               // the frame's splats in depth order
  uint32_t* list;                       // LDS [kFwdRing]: ranks ahead of the batch, by position mod the ring's size
  uint32_t* segs;                       // LDS [64]: the window's segments that have set bits
  uint32_t SW, sh, nv, nseg, total;
  uint32_t wseg = 0, wcnt = 0;          // next window: its first segment, this lane's segment's count
  uint32_t nov = 0, kov = 0;            // segments with set bits in the window, and how many were read
  uint32_t bits = 0, wrank = 0, winc = 0;   // this lane's word: bits not emitted, rank of bit 0, inclusive count
  uint32_t wtot = 0, wdone = 0;         // (uniform) set bits of the 64 words held, and how many of them are emitted
  uint32_t bend = 0;                    // (uniform) position after the emitted ones
  uint32_t nbits = 0, nrank = 0;        // the next 64 words
  bool nmore = false;                   // (uniform) there are any
  int lane;

  __device__ __forceinline__ RankStream(const PassArgs& a, int g, int b, uint32_t n, uint32_t* ring, uint32_t* sg,
                                        int ln)
      : row(a.tbits + (int64_t)g * a.bitmap_words), segc(a.seg_cnt + (int64_t)g * a.seg_stride), list(ring), segs(sg),
        SW((uint32_t)a.seg_words), sh((uint32_t)__ffs(a.seg_words) - 1u), total(n), lane(ln) {
    const uint32_t vbase = a.bkt_start[b * a.nbk];
    nv = a.bkt_start[(b + 1) * a.nbk] - vbase;
    sorted = a.depth_sorted + vbase;
    nseg = ((nv + 31) / 32 + SW - 1) / SW;
  }
  __device__ __forceinline__ void start() {
    wcnt = segc[min((uint32_t)lane, nseg - 1u)];
    read_words();
  }
  // issues the load of the next 64 words
  __device__ __forceinline__ void read_words() {
    while (kov >= nov && wseg < nseg) {
      const uint32_t sg = wseg + (uint32_t)lane;
      const bool ne = sg < nseg && wcnt != 0u;
      const unsigned long long om = __ballot(ne);
      wave_sync();
      if (ne) segs[lanes_below(om)] = sg;
      wave_sync();
      nov = (uint32_t)__popcll(om);
      kov = 0;
      wseg += 64u;
      wcnt = segc[min(wseg + (uint32_t)lane, nseg - 1u)];
    }
    const uint32_t k = kov + ((uint32_t)lane >> sh);
    const bool have = k < nov;
    const uint32_t wq = have ? segs[k & 63u] * SW + ((uint32_t)lane & (SW - 1u)) : 0u;
    const uint32_t w = row[wq];
    nbits = have ? w : 0u;
    nrank = wq * 32u;
    nmore = kov < nov;
    kov += 64u >> sh;
  }
  // the splats of positions [c0, c0 + 64) (lanes past the list's end: some splat of the frame)
  __device__ __forceinline__ uint32_t read_splats(uint32_t c0) {
    if (c0 >= total) return 0u;
    const uint32_t c1 = min(c0 + (uint32_t)kFwdBatch, total);
    while (bend < c1) {
      if (wdone == wtot) {
        if (!nmore) break;
        bits = nbits;
        wrank = nrank;
        winc = wave_incl_scan(__popc(bits));
        wtot = (uint32_t)__builtin_amdgcn_readlane((int)winc, 63);
        wdone = 0;
        read_words();
      }
      // the words that end within the ring (positions from c0 on are in use): all of them, but for dense rows
      const int space = (int)(c0 + kFwdRing - bend);
      const unsigned long long fit = __ballot((int)(winc - wdone) <= space);   // lane 0 on; never empty
      const uint32_t upto = (uint32_t)__builtin_amdgcn_readlane((int)winc, 63 - __clzll((long long)fit));
      if ((int)(winc - wdone) <= space) {
        uint32_t at = bend + winc - wdone - __popc(bits);
        while (bits != 0u) {
          list[at & (kFwdRing - 1u)] = wrank + (uint32_t)__builtin_ctz(bits);
          bits &= bits - 1u;
          ++at;
        }
      }
      bend += upto - wdone;
      wdone = upto;
    }
    wave_sync();
    const uint32_t rk = list[(c0 + (uint32_t)lane) & (kFwdRing - 1u)];
    wave_sync();
    return sorted[min(rk, nv - 1u)];   // (every rank is written)
  }
};

template <int T>
__global__ __launch_bounds__(64, T == 32 ? 1 : 6) void composite_fwd_kernel(PassArgs a, float* __restrict__ images) {
  using S = TileShape<T>;
  constexpr int NQ = S::NW;             // quadrants per tile
  constexpr int U = FwdGroup::N;        // entries evaluated together (independent alphas)
  constexpr int kTook = 32 / U * U;     // entries whose takes a lane holds in a word
  __shared__ FwdGroup sg[(kFwdBatch + U - 1) / U + 2];   // the batch's candidates
  __shared__ uint32_t pos[kFwdBatch];       // and the position after each
  __shared__ uint32_t list[kFwdRing];       // ranks ahead of the batch, by position mod the ring's size
  __shared__ uint32_t segs[64];             // the window's segments that have set bits
  if (a.status->overflow) return;
  const int lane = threadIdx.x;
  int r = blockIdx.x, q = 0;
  if (NQ > 1) {
    const int grp = blockIdx.x / (8 * NQ), within = blockIdx.x % (8 * NQ);
    q = within / 8;
    r = grp * 8 + within % 8;
  }
  const int g = tile_of_rank(a.cls_cnt, a.order_fwd, a.n_tiles, r);
  if (g < 0) return;
  const int b = frame_of_tile(a.frames, a.B, g);
  const FrameDev& F = a.frames[b];
  const int lt = g - F.tile_base;
  const int tx = lt % F.ntx, ty = lt / F.ntx;
  const uint32_t start = a.tile_start[g], total = a.tile_start[g + 1] - start;
  const int vt = q * 64 + lane;         // this lane's thread index in the tile's pixel map
  const int lx0 = S::lx0(vt), ly0 = S::ly0(vt);
  // Te: transmittance while the pixel runs; once it has stopped, minus the
  // transmittance at the stop (-0 outside the frame).  last: list position
  // after the last entry taken
  float Te[S::PX], C0[S::PX], C1[S::PX], C2[S::PX], pxf[S::PX], pyf[S::PX];
  uint32_t last[S::PX];
  bool inside[S::PX];
  bool mine = false;
#pragma unroll
  for (int p = 0; p < S::PX; ++p) {
    const int px = tx * T + lx0 + (p % S::PXW), py = ty * T + ly0 + (p / S::PXW);
    pxf[p] = (float)px + 0.5f;
    pyf[p] = (float)py + 0.5f;
    inside[p] = px < F.W && py < F.H;
    Te[p] = inside[p] ? 1.0f : 0.0f;
    C0[p] = C1[p] = C2[p] = 0.0f; last[p] = 0;
    mine |= inside[p];
  }
  // the wave's quadrant origin (pixel centre of its first lane's first pixel);
  // entries are culled against the rectangle of its pixels still running
  static_assert(S::LPR == 8, "the live-rectangle fold assumes 8 lanes per quadrant row");
  const float qx0 = (float)(tx * T + S::qx(vt) * S::QW) + 0.5f;
  const float qy0 = (float)(ty * T + S::qy(vt) * S::QW) + 0.5f;
  bool live = total > 0 && __ballot(mine) != 0ull;

  RankStream stream(a, g, b, total, list, segs, lane);
  uint32_t sp0 = 0, sp1 = 0;            // splats of this batch and the next
  float4 q0 = make_float4(0.f, 0.f, 0.f, 0.f), q1 = q0;   // this batch's records
  float qb = 0.f;
  if (live) {
    stream.start();
    sp0 = stream.read_splats(0);
    const float4* rec = reinterpret_cast<const float4*>(a.rec + (int64_t)sp0 * kRecF);
    q0 = rec[0]; q1 = rec[1]; qb = rec[2].x;
    sp1 = stream.read_splats(kFwdBatch);
  }
  for (uint32_t c0 = 0; live && c0 < total; c0 += kFwdBatch) {
    const int n = (int)min((uint32_t)kFwdBatch, total - c0);
    // ---- the rectangle of the pixel centres still running ----
    bool run = false;
#pragma unroll
    for (int p = 0; p < S::PX; ++p) run |= Te[p] > 0.0f;
    float sx0, sx1, sy0, sy1;
    running_rect<S::PXW>(__ballot(run), qx0, qy0, sx0, sx1, sy0, sy1);
    // ---- the batch's candidates compacted in list order ----
    if (lane < n) a.sorted[start + c0 + lane] = sp0;
    const bool cand = lane < n && strip_reach(q0, q1, sx0, sx1, sy0, sy1);
    const unsigned long long cmk = __ballot(cand);
    const int ncand = __popcll(cmk);      // (uniform)
    const int kslot = (int)lanes_below(cmk);   // this lane's candidate slot, if its entry is one
    if (cand) {
      sg[kslot / U].put(kslot % U, q0, q1, qb);
      pos[kslot] = c0 + (uint32_t)lane + 1u;
    }
    // padding entries: opacity 0 (log2 -1e30), never taken; their colour 0
    // (the mean and conic may be anything: min(power, -1e30) = -1e30)
    if (lane < U) sg[(ncand + lane) / U].pad((ncand + lane) % U);
    wave_sync();
    // ---- the batches behind this one: records of the first, indices of the second ----
    const float4* rec = reinterpret_cast<const float4*>(a.rec + (int64_t)sp1 * kRecF);
    q0 = rec[0]; q1 = rec[1]; qb = rec[2].x;
    sp0 = sp1;
    sp1 = stream.read_splats(c0 + 2 * kFwdBatch);
    // ---- compositing: the candidates in list order, U at a time; a group's
    // conics are read while the group before it is blended, its colours while
    // its alphas are formed ----
    unsigned long long tookm = 0ull;      // (uniform) bit k: some pixel took candidate k
    float4 r0[U], r1a = sg[0].v[U], r1b = sg[0].v[U + 1];
#pragma unroll
    for (int u = 0; u < U; ++u) r0[u] = sg[0].v[u];
    const FwdGroup* grp = sg;
    for (int k0 = 0; live && k0 < ncand; k0 += kTook) {
      const int k1 = min(ncand, k0 + kTook);
      uint32_t took[S::PX];               // bit k - 1 - j: the pixel took candidate j of [k0, k)
#pragma unroll
      for (int p = 0; p < S::PX; ++p) took[p] = 0u;
      int k = k0;
      do {
        const float4 ca = grp->v[U + 2], cb = grp->v[U + 3], cd = grp->v[U + 4];
        const float cr[U] = {ca.x, ca.w, cb.z, cd.y}, cg[U] = {ca.y, cb.x, cb.w, cd.z}, cl[U] = {ca.z, cb.y, cd.x, cd.w};
        const float cc[U] = {r1a.x, r1a.z, r1b.x, r1b.z}, lo[U] = {r1a.y, r1a.w, r1b.y, r1b.w};
        float al[S::PX][U];
#pragma unroll
        for (int p = 0; p < S::PX; ++p)
#pragma unroll
          for (int u = 0; u < U; ++u) al[p][u] = clamped_alpha(r0[u], cc[u], lo[u], pxf[p], pyf[p]);
        __builtin_amdgcn_sched_barrier(0);
        ++grp;
#pragma unroll
        for (int u = 0; u < U; ++u) r0[u] = grp->v[u];
        r1a = grp->v[U];
        r1b = grp->v[U + 1];
        k += U;
        bool run = false;
#pragma unroll
        for (int p = 0; p < S::PX; ++p) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const float nw = fold_step(al[p][u] >= kAlphaMin ? al[p][u] : -0.0f, Te[p], took[p]);
            C0[p] = __builtin_fmaf(-nw, cr[u], C0[p]);
            C1[p] = __builtin_fmaf(-nw, cg[u], C1[p]);
            C2[p] = __builtin_fmaf(-nw, cl[u], C2[p]);
          }
          run |= Te[p] > 0.0f;
        }
        live = __builtin_amdgcn_ballot_w64(run) != 0ull;
      } while (k < (live ? k1 : 0));
      uint32_t any = 0u;
#pragma unroll
      for (int p = 0; p < S::PX; ++p) {
        if (took[p] != 0u) last[p] = pos[k - 1 - __builtin_ctz(took[p])];
        any |= took[p];
      }
      tookm |= (unsigned long long)(__builtin_bitreverse32(wave_or(any)) >> (32 - (k - k0))) << k0;
    }
    // the entries of the batch that the quadrant took
    const unsigned long long taken = __ballot(cand && ((tookm >> kslot) & 1ull));
    if (lane == 0) a.qmask[4 * ((int64_t)(start >> 6) + g + (c0 >> 6)) + q] = taken;
    wave_sync();                          // the candidates' slots are rewritten by the next batch
  }
  uint32_t my_last = 0;
#pragma unroll
  for (int p = 0; p < S::PX; ++p) {
    if (inside[p]) {
      const int px = (int)pxf[p], py = (int)pyf[p];
      const int64_t pix = (int64_t)py * F.W + px;
      const int64_t hw = (int64_t)F.W * F.H;
      float* img = images + F.pix_base * 3;
      const float Tfin = fabsf(Te[p]);
      img[pix] = C0[p] + Tfin * F.bg[0];
      img[hw + pix] = C1[p] + Tfin * F.bg[1];
      img[2 * hw + pix] = C2[p] + Tfin * F.bg[2];
      a.n_iter[F.pix_base + pix] = last[p];
      a.t_final[F.pix_base + pix] = Tfin;
      my_last = max(my_last, last[p]);
    }
  }
  my_last = wave_max_u32(my_last);
  if (lane < 4 && (lane == q || NQ == 1)) a.qlast[g * 4 + lane] = lane == q ? my_last : 0u;
}

// The same for few tiles (launch_composite_fwd), a workgroup of three waves to
// each quadrant: a lone wave issues an instruction every four cycles or so,
// whatever it is, and the longest list's instructions are the pass's time; the
// chip has room for more waves, so a quadrant's walk is made a pipeline of
// three parts, near enough equal for a batch of 20 candidates.  One wave reads the list and stages a batch's
// candidates, at most kStepMax of them a step; one forms the alphas of the
// step before at the quadrant's pixels, to LDS; one folds those of the step
// before that.  A barrier ends a step.  The entries are culled against the
// pixels that ran two steps earlier: no fewer than run now, so only entries
// that nothing takes are added.  Every alpha and every fold is the one-wave
// kernel's operation on the same values.
//
// One 512 x 512 frame of 50k Gaussians 78 -> 57 us, of 200k 169 -> 107, one
// 128 x 128 frame of 2k 35 -> 29.  With at most 16 or 24 candidates a step
// (less LDS, more workgroups in flight): 62, 61 for the first.
constexpr int kStepMax = 32;

struct FwdStep {
  unsigned long long cand;              // the batch's candidates
  uint32_t c0;                          // the batch's first position
  uint32_t n;                           // candidates of this step
  uint32_t first;                       // the batch's candidates before them
  uint32_t ends;                        // bit 0: the batch ends with this step, bit 1: the list does
};

// a value that all lanes hold, to the scalar unit
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ unsigned long long uniform(unsigned long long x) {
  return (unsigned long long)uniform((uint32_t)(x >> 32)) << 32 | uniform((uint32_t)x);
}

template <int T>
__global__ __launch_bounds__(192) void composite_fwd_split_kernel(PassArgs a, float* __restrict__ images) {
  using S = TileShape<T>;
  static_assert(S::PX == 1, "a pixel to a lane");
  constexpr int NQ = S::NW;
  constexpr int U = FwdGroup::N;        // entries taken together
  __shared__ FwdGroup sg[3][kStepMax / U + 1];
  __shared__ uint32_t pos[3][kStepMax];
  __shared__ float alpha[(2 * kStepMax + U) * 64];   // two steps' (and what is read past the second)
  __shared__ FwdStep info[3];
  __shared__ unsigned long long running[2];
  __shared__ uint32_t list[kFwdRing];
  __shared__ uint32_t segs[64];
  if (a.status->overflow) return;
  const int lane = threadIdx.x & 63, role = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int r = blockIdx.x, q = 0;
  if (NQ > 1) {
    const int grp = blockIdx.x / (8 * NQ), within = blockIdx.x % (8 * NQ);
    q = within / 8;
    r = grp * 8 + within % 8;
  }
  const int g = tile_of_rank(a.cls_cnt, a.order_fwd, a.n_tiles, r);
  if (g < 0) return;
  const int b = frame_of_tile(a.frames, a.B, g);
  const FrameDev& F = a.frames[b];
  const int lt = g - F.tile_base;
  const int tx = lt % F.ntx, ty = lt / F.ntx;
  const uint32_t start = a.tile_start[g], total = a.tile_start[g + 1] - start;
  const int vt = q * 64 + lane;
  const int px = tx * T + S::lx0(vt), py = ty * T + S::ly0(vt);
  const float pxf = (float)px + 0.5f, pyf = (float)py + 0.5f;
  const bool inside = px < F.W && py < F.H;
  const unsigned long long all = __ballot(inside);
  float Te = inside ? 1.0f : 0.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f;   // (the fold's)
  uint32_t last = 0;
  if (total > 0 && all != 0ull) {       // (uniform over the workgroup)
    if (threadIdx.x < 3) info[threadIdx.x] = FwdStep{0ull, 0u, 0u, 0u, 0u};
    if (threadIdx.x < 2) running[threadIdx.x] = all;
    __syncthreads();
    int st = 0;                         // step mod 3
    if (role == 2) {
      RankStream stream(a, g, b, total, list, segs, lane);
      stream.start();
      const float qx0 = (float)(tx * T + S::qx(vt) * S::QW) + 0.5f;
      const float qy0 = (float)(ty * T + S::qy(vt) * S::QW) + 0.5f;
      uint32_t c0 = 0, i = 0;           // this batch, this step
      unsigned long long M = all;
      // splats of this batch and the two behind it
      uint32_t sp0 = stream.read_splats(0), sp1 = stream.read_splats(kFwdBatch);
      uint32_t sp2 = stream.read_splats(2 * kFwdBatch);
      auto record = [&](uint32_t sp, float4& q0, float4& q1, float& qb) {
        const float4* rec = reinterpret_cast<const float4*>(a.rec + (int64_t)sp * kRecF);
        q0 = rec[0]; q1 = rec[1]; qb = rec[2].x;
      };
      // the steps of a batch whose records are q; q is left with those of the
      // batch after the next, so that every load has a step or more to arrive.
      // Returns whether the pipeline has ended.
      auto batch = [&](float4& q0, float4& q1, float& qb) -> bool {
        unsigned long long cmk = 0ull;
        if (c0 < total) {
          const int n = (int)min((uint32_t)kFwdBatch, total - c0);
          float sx0, sx1, sy0, sy1;
          running_rect<1>(M, qx0, qy0, sx0, sx1, sy0, sy1);
          if (lane < n) a.sorted[start + c0 + lane] = sp0;
          cmk = __ballot(lane < n && strip_reach(q0, q1, sx0, sx1, sy0, sy1));
        }
        const uint32_t ncand = (uint32_t)__popcll(cmk), kslot = lanes_below(cmk);
        const bool cand = (cmk >> lane) & 1ull;
        for (uint32_t done = 0;; done += kStepMax) {
          const uint32_t nst = min(ncand - done, (uint32_t)kStepMax);
          const bool whole = done + nst == ncand;
          const uint32_t k = kslot - done;
          if (cand && k < nst) {
            sg[st][k / U].put(k % U, q0, q1, qb);
            pos[st][k] = c0 + (uint32_t)lane + 1u;
          }
          if (lane < U) sg[st][(nst + lane) / U].pad((nst + lane) % U);
          if (lane == 0)
            info[st] = FwdStep{cmk, c0, nst, done,
                               c0 < total && whole ? 1u | (c0 + kFwdBatch >= total ? 2u : 0u) : 0u};
          if (whole) {
            sp0 = sp1;
            const uint32_t sp = sp2;
            sp1 = sp2;
            sp2 = stream.read_splats(c0 + 3 * kFwdBatch);
            record(sp, q0, q1, qb);
            c0 += c0 < total ? kFwdBatch : 0u;
          }
          st = st == 2 ? 0 : st + 1;
          __syncthreads();
          M = uniform(running[i++ & 1u]);
          if (M == 0ull) return true;
          if (whole) return false;
        }
      };
      float4 qa0, qa1, qb0, qb1;
      float qa2, qb2;
      record(sp0, qa0, qa1, qa2);
      record(sp1, qb0, qb1, qb2);
      while (!batch(qa0, qa1, qa2) && !batch(qb0, qb1, qb2)) {
      }
    } else if (role == 1) {
      st = 2;
      for (uint32_t i = 0;; ++i) {
        const int n = uniform(info[st].n);
        const FwdGroup* in = sg[st];
        float* out = alpha + (i & 1u) * (kStepMax * 64) + lane;
        float4 r0[U], r1a = in->v[U], r1b = in->v[U + 1];
#pragma unroll
        for (int u = 0; u < U; ++u) r0[u] = in->v[u];
        for (int k = 0; k < n; k += U) {
          const float cc[U] = {r1a.x, r1a.z, r1b.x, r1b.z}, lo[U] = {r1a.y, r1a.w, r1b.y, r1b.w};
          float al[U];
#pragma unroll
          for (int u = 0; u < U; ++u) al[u] = clamped_alpha(r0[u], cc[u], lo[u], pxf, pyf);
          __builtin_amdgcn_sched_barrier(0);
          ++in;
#pragma unroll
          for (int u = 0; u < U; ++u) r0[u] = in->v[u];
          r1a = in->v[U];
          r1b = in->v[U + 1];
#pragma unroll
          for (int u = 0; u < U; ++u) out[(k + u) * 64] = (al[u] >= kAlphaMin) ? al[u] : -0.0f;
        }
        st = st == 2 ? 0 : st + 1;
        __syncthreads();
        if (uniform(running[i & 1u]) == 0ull) break;
      }
    } else {
      st = 1;
      unsigned long long tookm = 0ull;  // bit k: some pixel took the batch's candidate k
      for (uint32_t i = 0;; ++i) {
        const int n = uniform(info[st].n);
        const uint32_t first = uniform(info[st].first), ends = uniform(info[st].ends);
        const FwdGroup* in = sg[st];
        const float* w = alpha + (~i & 1u) * (kStepMax * 64) + lane;
        unsigned long long M = __ballot(Te > 0.0f);
        uint32_t took = 0u;             // bit k - 1 - j: the pixel took the step's candidate j
        int k = 0;
        float wu[U];
        float4 ca = in->v[U + 2], cb = in->v[U + 3], cd = in->v[U + 4];
#pragma unroll
        for (int u = 0; u < U; ++u) wu[u] = w[u * 64];
        while (k < n && M != 0ull) {
          const float cr[U] = {ca.x, ca.w, cb.z, cd.y}, cg[U] = {ca.y, cb.x, cb.w, cd.z}, cl[U] = {ca.z, cb.y, cd.x, cd.w};
          float nw[U];
#pragma unroll
          for (int u = 0; u < U; ++u) nw[u] = fold_step(wu[u], Te, took);
          k += U;
          w += U * 64;
#pragma unroll
          for (int u = 0; u < U; ++u) wu[u] = w[u * 64];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            C0 = __builtin_fmaf(-nw[u], cr[u], C0);
            C1 = __builtin_fmaf(-nw[u], cg[u], C1);
            C2 = __builtin_fmaf(-nw[u], cl[u], C2);
          }
          ++in;
          ca = in->v[U + 2]; cb = in->v[U + 3]; cd = in->v[U + 4];
          M = __builtin_amdgcn_ballot_w64(Te > 0.0f);
        }
        if (k > 0) {
          if (took != 0u) last = pos[st][k - 1 - __builtin_ctz(took)];
          tookm |= (unsigned long long)(__builtin_bitreverse32(wave_or(took)) >> (32 - k)) << first;
        }
        if ((ends & 1u) || (M == 0ull && n > 0)) {
          const unsigned long long cmk = info[st].cand;
          const int kslot = (int)lanes_below(cmk);
          const unsigned long long taken = __ballot(((cmk >> lane) & 1ull) && ((tookm >> kslot) & 1ull));
          if (lane == 0) a.qmask[4 * ((int64_t)(start >> 6) + g + (info[st].c0 >> 6)) + q] = taken;
          tookm = 0ull;
        }
        if (lane == 0) running[i & 1u] = (ends & 2u) ? 0ull : M;
        st = st == 2 ? 0 : st + 1;
        __syncthreads();
        if (uniform(running[i & 1u]) == 0ull) break;
      }
    }
  }
  if (role != 0) return;
  if (inside) {
    const int64_t pix = (int64_t)py * F.W + px;
    const int64_t hw = (int64_t)F.W * F.H;
    float* img = images + F.pix_base * 3;
    const float Tfin = fabsf(Te);
    img[pix] = C0 + Tfin * F.bg[0];
    img[hw + pix] = C1 + Tfin * F.bg[1];
    img[2 * hw + pix] = C2 + Tfin * F.bg[2];
    a.n_iter[F.pix_base + pix] = last;
    a.t_final[F.pix_base + pix] = Tfin;
  }
  last = wave_max_u32(last);
  if (lane < 4 && (lane == q || NQ == 1)) a.qlast[g * 4 + lane] = lane == q ? last : 0u;
}

constexpr int kSplitTiles = 1280;

void launch_composite_fwd(const PassArgs& a, float* images, hipStream_t s) {
  if (a.n_tiles == 0) return;
  const int nq = a.tile == 8 ? 1 : 4;
  const dim3 grid(nq == 1 ? a.n_tiles : div_up(a.n_tiles, 8) * 8 * nq);
  // Past some 1300 tiles the chip is full of waves and the pipeline's barriers
  // and LDS traffic cost more than its shorter chains save; below 8 splats a
  // tile there is no chain to shorten.  One wave / three waves (us): 50k splats
  // on 1024 tiles 74 / 51, on 1536 65 / 65, on 2048 79 / 68 but 20k 48 / 56,
  // 150k on 3072 85 / 100, 60k on 1250 58 / 49; on 1024 tiles 10k 33 / 30,
  // 5k 24 / 26, 4k 30 / 30.
  if (a.tile == 16 && a.n_tiles <= kSplitTiles && a.n_splats >= 8 * (int64_t)a.n_tiles) {
    hipLaunchKernelGGL(composite_fwd_split_kernel<16>, grid, dim3(192), 0, s, a, images);
    return;
  }
  if (a.tile == 8) hipLaunchKernelGGL(composite_fwd_kernel<8>, grid, dim3(64), 0, s, a, images);
  else if (a.tile == 16) hipLaunchKernelGGL(composite_fwd_kernel<16>, grid, dim3(64), 0, s, a, images);
  else hipLaunchKernelGGL(composite_fwd_kernel<32>, grid, dim3(64), 0, s, a, images);
}

// Contributors per pixel, on request: the entries before the pixel's stop
// position whose alpha reaches 1/255 (every such entry was taken, nothing
// after the stop was).  Reads the complete per-tile lists; a workgroup per
// tile, a thread per pixel.  Diagnostic only, not part of a pass.
__global__ __launch_bounds__(256) void count_contrib_kernel(PassArgs a) {
  const int g = blockIdx.x;
  if (a.status->overflow || g >= a.n_tiles) return;
  const int b = frame_of_tile(a.frames, a.B, g);
  const FrameDev& F = a.frames[b];
  const int T = a.tile;
  const int lt = g - F.tile_base;
  const int tx = lt % F.ntx, ty = lt / F.ntx;
  const uint32_t start = a.tile_start[g];
  for (int q = threadIdx.x; q < T * T; q += 256) {
    const int px = tx * T + q % T, py = ty * T + q / T;
    if (px >= F.W || py >= F.H) continue;
    const int64_t pix = F.pix_base + (int64_t)py * F.W + px;
    const uint32_t nit = a.n_iter[pix];
    uint32_t c = 0;
    for (uint32_t i = 0; i < nit; ++i) {
      const float4* rec = reinterpret_cast<const float4*>(a.rec + (int64_t)a.sorted[start + i] * kRecF);
      float dx, dy, pwr;
      const float al = splat_alpha(rec[0], rec[1].x, rec[1].y, (float)px + 0.5f, (float)py + 0.5f, dx, dy, pwr);
      c += al >= kAlphaMin ? 1u : 0u;
    }
    a.n_contrib[pix] = c;
  }
}

void launch_count_contrib(const PassArgs& a, hipStream_t s) {
  if (a.n_tiles == 0) return;
  hipLaunchKernelGGL(count_contrib_kernel, dim3(a.n_tiles), dim3(256), 0, s, a);
}

}  // namespace gbr
