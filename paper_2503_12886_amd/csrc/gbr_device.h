// Wave- and block-level building blocks shared by the kernels: prefix scans
// and the stable ballot-ranked LSD radix pass.
#pragma once

#include "gbr_internal.h"

namespace gbr {

// The workgroup's frame and its place among the frame's `per` in a grid of
// frame_grid(a, per); false: no frame.  With by_xcd, frame b's workgroups are those whose
// index is b mod 8, so that they run on one XCD: the keys that a frame's
// blocks scatter, and the splats' rectangles that are gathered in depth order,
// stay in its L2 instead of passing through all eight.  64 frames of 100k
// splats: scatter pass 80 -> 43 us, bitmap rows 153 -> 149; 16 of 50k: 13 -> 10,
// 31 -> 27.  (The ranking gains nothing: 42 -> 45.)
__device__ __forceinline__ bool frame_block(const PassArgs& a, int per, int& b, int& blk) {
  b = blockIdx.y;
  blk = blockIdx.x;
  if (!a.by_xcd) return true;
  const int i = blk / 8;
  b = i / per * 8 + blk % 8;
  blk = i % per;
  return b < a.B;
}

// Inclusive scan across the wave by DPP adds: four shifts inside the rows of
// 16 lanes, then the rows' totals carried on (lane 15 of rows 0 and 2 into
// rows 1 and 3, lane 31 into rows 2 and 3).  Six VALU adds; by lane shuffles
// each step is an LDS round trip.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_add_u32(uint32_t x) {
  return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v = dpp_add_u32<0x111, 0xf>(v);   // row_shr:1
  v = dpp_add_u32<0x112, 0xf>(v);
  v = dpp_add_u32<0x114, 0xf>(v);
  v = dpp_add_u32<0x118, 0xf>(v);
  v = dpp_add_u32<0x142, 0xa>(v);   // row_bcast:15
  return dpp_add_u32<0x143, 0xc>(v);   // row_bcast:31
}

template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_u32(uint32_t v) {
  return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
// The OR of a value over the wave's lanes, on the scalar unit.
__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
  v = dpp_or_u32<0x111, 0xf>(v);   // row_shr:1
  v = dpp_or_u32<0x112, 0xf>(v);
  v = dpp_or_u32<0x114, 0xf>(v);
  v = dpp_or_u32<0x118, 0xf>(v);
  v = dpp_or_u32<0x142, 0xa>(v);   // row_bcast:15
  v = dpp_or_u32<0x143, 0xc>(v);   // row_bcast:31
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Orders the wave's LDS accesses across its lanes (they execute in program
// order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// min(alpha, 0.99) of a splat at a pixel, bit-identical in the forward and the
// backward pass: power = ca dx^2 + cb dx dy + cc dy^2 (r0.z, r0.w, cc) plus
// lo = log2 opacity, clamped at lo, and alpha = 2^power.  v_exp_f32 gives 0.99f itself at kAlphaMaxLog2
// (and some 45 float32 to either side), no more below and no less above, so the
// clamp goes to the power, where it is an operand of the minimum that is
// taken anyway.
constexpr float kAlphaMaxLog2 = -0.014499555f;
__device__ __forceinline__ float clamped_alpha(float4 r0, float cc, float lo, float px, float py) {
#pragma clang fp contract(off)
  const float dx = px - r0.x, dy = py - r0.y;
  float pw = __builtin_fmaf(r0.z * dx, dx, lo);
  pw = __builtin_fmaf(r0.w * dx, dy, pw);
  pw = __builtin_fmaf(cc * dy, dy, pw);
  float pc;
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(pc) : "v"(pw), "v"(lo), "s"(kAlphaMaxLog2));
  return __builtin_amdgcn_exp2f(pc);
}

// Exclusive scan of one value per thread across a block of NT threads.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* lds_waves, uint32_t* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  constexpr int NW = NT / 64;
  uint32_t inc = wave_incl_scan(v);
  if (lane == 63) lds_waves[w] = inc;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    uint32_t x = lds_waves[i];
    if (i < w) off += x;
    tot += x;
  }
  __syncthreads();
  if (total) *total = tot;
  return off + inc - v;
}


// Stable LSD radix pass (8-bit digit at `shift`) of n 64-bit keys from src to
// dst by a block of kSortThreads threads.  Wave w owns a contiguous segment of
// the keys, so (wave, step, lane) order is key order and equal digits keep
// their relative order; the rank of a key among equal digits in its step is
// found with ballots over the digit's bits.  src/dst may be LDS or global.
constexpr int kSortThreads = 256;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortCap = 8192;

__device__ __forceinline__ unsigned long long digit_peers(uint32_t d, bool valid) {
  unsigned long long peers = __ballot(valid);
#pragma unroll
  for (int bit = 0; bit < 8; ++bit) {
    const bool on = (d >> bit) & 1u;
    const unsigned long long m = __ballot(on);
    peers &= on ? m : ~m;
  }
  return peers;
}

template <typename SrcT, typename DstT>
__device__ __forceinline__ void radix_pass(SrcT src, DstT dst, int n, int shift, uint32_t* hist,
                                           uint32_t* lds_waves) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int seg = ((n + kSortThreads - 1) / kSortThreads) * 64;
  const int lo = w * seg, hi = min(n, lo + seg);
  for (int i = threadIdx.x; i < kSortWaves * 256; i += kSortThreads) hist[i] = 0u;
  __syncthreads();
  for (int base = lo; base < hi; base += 64) {
    const int k = base + lane;
    const bool valid = k < hi;
    const uint32_t d = valid ? (uint32_t)(src[k] >> shift) & 255u : 0u;
    const unsigned long long peers = digit_peers(d, valid);
    if (valid && lanes_below(peers) == 0) hist[w * 256 + d] += (uint32_t)__popcll(peers);
  }
  __syncthreads();
  // offsets in (digit, wave) order
  uint32_t tot = 0;
  if (threadIdx.x < 256) {
    for (int ww = 0; ww < kSortWaves; ++ww) {
      const uint32_t c = hist[ww * 256 + threadIdx.x];
      hist[ww * 256 + threadIdx.x] = tot;
      tot += c;
    }
  }
  __syncthreads();
  const uint32_t dbase = block_excl_scan<kSortThreads>(threadIdx.x < 256 ? tot : 0u, lds_waves, nullptr);
  if (threadIdx.x < 256)
    for (int ww = 0; ww < kSortWaves; ++ww) hist[ww * 256 + threadIdx.x] += dbase;
  __syncthreads();
  for (int base = lo; base < hi; base += 64) {
    const int k = base + lane;
    const bool valid = k < hi;
    const unsigned long long key = valid ? src[k] : 0ull;
    const uint32_t d = (uint32_t)(key >> shift) & 255u;
    const unsigned long long peers = digit_peers(d, valid);
    const uint32_t below = lanes_below(peers);
    uint32_t at = 0;
    if (valid) at = hist[w * 256 + d];
    if (valid) dst[at + below] = key;
    if (valid && below == 0) hist[w * 256 + d] = at + (uint32_t)__popcll(peers);
  }
  __syncthreads();
}


}  // namespace gbr
