// Backward half of the batch-parallel rasterizer: per-tile reverse traversal
// of the compositing recurrence, per-entry partial gradients reduced across
// the tile's pixels without atomics, a fixed-order gather per splat, and the
// adjoint of activation + EWA projection.  Also the photometric loss.
#include "gbr_device.h"
#include "tangent_ops.h"

namespace gbr {

template <int T> using TileShapeB = TileMap<T>;

// Must stay bit-identical to the forward kernel's alpha: power = ca dx^2 +
// cb dx dy + cc dy^2 + lo (lo = log2 opacity), alpha = 2^min(power, lo).
// The clamp is one v_min_f32 (min(power, lo) for every non-NaN power);
// written as such because fminf would first canonicalise lo, one more
// instruction per (entry, pixel).
__device__ __forceinline__ float splat_alpha_b(float4 r0, float4 r1, float px, float py, float& dx, float& dy) {
#pragma clang fp contract(off)
  dx = px - r0.x;
  dy = py - r0.y;
  float pw = __builtin_fmaf(r0.z * dx, dx, r1.y);
  pw = __builtin_fmaf(r0.w * dx, dy, pw);
  pw = __builtin_fmaf(r1.x * dy, dy, pw);
  float pc;
  asm("v_min_f32 %0, %1, %2" : "=v"(pc) : "v"(pw), "v"(r1.y));
  return __builtin_amdgcn_exp2f(pc);
}

// Per-entry partial, summed over the tile's pixels, in units of t = alpha *
// dL/dalpha (the gradient with respect to the power is t ln 2):
//   (sum t dx, sum t dy, sum t dx^2, sum t dx dy, sum t dy^2, sum t,
//    d r, d g, d b)
// with (dx, dy) the pixel's offset from the mean.  The splat's gradients
// follow once per splat, after the sums: the power's coefficients ca, cb, cc
// get ln 2 times the three second moments, the mean -ln 2 (2 ca, cb; cb,
// 2 cc) times the first moments, the opacity logit (1 - o) sum t.  Along the
// traversal each lane keeps only the transmittance and <colour behind,
// dL/dout>.
// The power passes its gradient also where rounding lifts it above log2 o and
// it is clamped there: the quadratic form is never negative, so the clamp
// removes an error and no dependence.  (With no gradient from those pixels,
// splats thousands of pixels long, whose conic is indefinite in binary32, had
// 1 to 20 % of the terms' magnitude wrong in the long scale's gradient, and
// 0.1 % with it.)
// A wave's sum over its lanes is taken in a fixed order; the block then adds
// its waves in order and writes the entry's partial, by emission slot, only
// if some pixel contributed; a byte flag marks it.

// Folds one entry into a lane's back-to-front state (transmittance in front
// of the entry, colour behind it) and returns its partial in acc.  Lanes
// whose pixel did not take the entry add exact zeros and keep their state.
template <int PX>
__device__ __forceinline__ void entry_grad(const float4 r0, const float4 r1, const float cbl, const uint32_t li,
                                           const float* pxf, const float* pyf, const uint32_t* nit, float* T_,
                                           float* SG, const float* G0, const float* G1, const float* G2,
                                           float* acc) {
#pragma unroll
  for (int p = 0; p < PX; ++p) {
    float dx, dy;
    const float a0 = splat_alpha_b(r0, r1, pxf[p], pyf[p], dx, dy);
    const bool take = li < nit[p] && a0 >= kAlphaMin;
    // an untaken entry folds with alpha 0: 1/(1 - 0) = 1 exactly, so the
    // transmittance passes through unchanged and the weight is 0
    const float al = take ? fminf(a0, kAlphaMax) : 0.0f;
    const float inv = __builtin_amdgcn_rcpf(1.0f - al);
    const float Ti = T_[p] * inv;                     // transmittance in front of this entry
    const float wgt = al * Ti;
    const float cg = r1.z * G0[p] + r1.w * G1[p] + cbl * G2[p];   // <colour, dL/dout>
    const float dal = Ti * cg - SG[p] * inv;          // d out / d alpha
    SG[p] += wgt * cg;                                // <colour behind, dL/dout>
    T_[p] = Ti;
    // min(0.99, .) passes the gradient only below the clamp
    const float t = (take && a0 < kAlphaMax) ? a0 * dal : 0.0f;
    const float p1 = t * dx, p2 = t * dy;
    const float v[9] = {p1, p2, p1 * dx, p1 * dy, p2 * dy, t, wgt * G0[p], wgt * G1[p], wgt * G2[p]};
    // the first pixel assigns (adding it to 0 would cost an instruction per value)
#pragma unroll
    for (int c = 0; c < 9; ++c) acc[c] = (p == 0) ? v[c] : acc[c] + v[c];
  }
}

// The sums over the 16 lanes of each row of 9 values, transposed into one
// register: at each halving step two registers are paired, each lane keeping
// one of the two values and adding its partner's copy of it (partners by
// row_ror:8, row_half_mirror, quad_perm xor 2, then xor 1), so 21 VALU
// operations replace 36 in-row shifts.  Lane i of a row ends with the row's
// total of value 8 when i is odd, else of value 4 i1 + 2 i2 + i3 (i1, i2, i3
// the bits 1 to 3 of i); every lane's total covers each of the 16 lanes once.
// In the first two steps the two halves of a pair are whole DPP banks (4
// lanes), so each half is one DPP add that writes only its banks, in place
// (inline assembly: two wait states before DPP reads of VALU results);
// the last two steps select between the registers.
template <int CTRL>
__device__ __forceinline__ float pair_fold(float x, float y, bool hi) {
  const float z = hi ? y : x, w = hi ? x : y;
  return z + dpp_mov<CTRL, 0xf, 0xf, false>(w);
}
#define GBR_BANK_PAIR(ctrl, x, y, mx, my)                                                    \
  "v_add_f32_dpp %" #x ", %" #x ", %" #x " " ctrl " row_mask:0xf bank_mask:" mx "\n\t"     \
  "v_add_f32_dpp %" #x ", %" #y ", %" #y " " ctrl " row_mask:0xf bank_mask:" my "\n\t"
__device__ __forceinline__ float rows_transposed9(const float (&v)[9], int lane) {
  constexpr int kQuadXor2 = 0x4e, kQuadXor1 = 0xb1;
  float a0 = v[0], a1 = v[2], a2 = v[4], a3 = v[6], a4 = v[8];
  // partners 8 apart: the first value in lanes 0-7 (banks 0, 1), the second in 8-15
  asm volatile("s_nop 1\n\t"
               GBR_BANK_PAIR("row_ror:8", 0, 5, "0x3", "0xc") GBR_BANK_PAIR("row_ror:8", 1, 6, "0x3", "0xc")
               GBR_BANK_PAIR("row_ror:8", 2, 7, "0x3", "0xc") GBR_BANK_PAIR("row_ror:8", 3, 8, "0x3", "0xc")
               "v_add_f32_dpp %4, %4, %4 row_ror:8 row_mask:0xf bank_mask:0xf"
               : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3), "+v"(a4)
               : "v"(v[1]), "v"(v[3]), "v"(v[5]), "v"(v[7]));
  // partners mirrored inside 8 lanes: the first value in banks 0 and 2, the second in 1 and 3
  asm volatile("s_nop 1\n\t"
               GBR_BANK_PAIR("row_half_mirror", 0, 3, "0x5", "0xa") GBR_BANK_PAIR("row_half_mirror", 1, 4, "0x5", "0xa")
               "v_add_f32_dpp %2, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xf\n\ts_nop 1"
               : "+v"(a0), "+v"(a2), "+v"(a4)
               : "v"(a1), "v"(a3));
  const bool b1 = lane & 2, b0 = lane & 1;
  const float d0 = pair_fold<kQuadXor2>(a0, a2, b1);
  const float d1 = a4 + dpp_mov<kQuadXor2, 0xf, 0xf, false>(a4);
  return pair_fold<kQuadXor1>(d0, d1, b0);
}
#undef GBR_BANK_PAIR

// Adds rows 0 and 1, and rows 2 and 3, lane by lane (each half-wave's two
// rows end with the same sums): a lane swap of the register with its copy.
__device__ __forceinline__ float row_pair_sum(float x) {
  float y = x;
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(x), "+v"(y));
  return x + y;
}

// Tiles of 32 pixels: four pixels per lane.  The lane's own sums over its
// pixels come first, so the cross-lane sums are shared by four pixels and
// stay on the vector unit; CHUNK positions are staged between two barriers.
template <int CHUNK>
__global__ __launch_bounds__(TileShapeB<32>::NT) void composite_bwd32_kernel(PassArgs a,
                                                                             const float* __restrict__ dimages) {
  constexpr int T = 32;
  static_assert(CHUNK <= 256, "a group's chunk positions are packed one byte each");
  using S = TileShapeB<T>;
  constexpr int U = 4;                      // entries folded per step (independent alphas)
  __shared__ float4 s0[CHUNK];
  __shared__ float4 s1[CHUNK];
  __shared__ float4 s2[CHUNK];             // .x only: 16-byte slots share the LDS address of s0 and s1
  __shared__ float red[CHUNK][S::NW][9];
  __shared__ uint32_t wany[CHUNK];         // byte w: wave w wrote red[i][w]
  __shared__ uint32_t sid[CHUNK];
  if (a.status->overflow) return;
  const int g = tile_of_rank(a.cls_cnt + 33, a.order_bwd, a.n_tiles, blockIdx.x);
  if (g < 0) return;
  const uint32_t L = a.tile_last[g];
  if (L == 0) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t Lw = a.qlast[g * 4 + w];    // this wave's quadrant took nothing at or past Lw
  const int b = frame_of_tile(a.frames, a.B, g);
  const FrameDev& F = a.frames[b];
  const int lt = g - F.tile_base;
  const int tx = lt % F.ntx, ty = lt / F.ntx;
  const uint32_t start = a.tile_start[g];
  const int lx0 = S::lx0(threadIdx.x), ly0 = S::ly0(threadIdx.x);
  float T_[S::PX], SG[S::PX], G0[S::PX], G1[S::PX], G2[S::PX];
  uint32_t nit[S::PX];
  float pxf[S::PX], pyf[S::PX];
  const float* img_g = dimages + F.pix_base * 3;
  const int64_t hw = (int64_t)F.W * F.H;
#pragma unroll
  for (int p = 0; p < S::PX; ++p) {
    const int px = tx * T + lx0 + (p % S::PXW), py = ty * T + ly0 + (p / S::PXW);
    pxf[p] = (float)px + 0.5f;
    pyf[p] = (float)py + 0.5f;
    nit[p] = 0; T_[p] = 1.0f; SG[p] = 0.0f; G0[p] = G1[p] = G2[p] = 0.0f;
    if (px < F.W && py < F.H) {
      const int64_t pix = (int64_t)py * F.W + px;
      nit[p] = a.n_iter[F.pix_base + pix];
      T_[p] = a.t_final[F.pix_base + pix];
      G0[p] = img_g[pix]; G1[p] = img_g[hw + pix]; G2[p] = img_g[2 * hw + pix];
      // <colour behind the current entry, dL/dout>, starts at <T_end * background, dL/dout>
      SG[p] = T_[p] * (F.bg[0] * G0[p] + F.bg[1] * G1[p] + F.bg[2] * G2[p]);
    }
  }
  uint8_t* wany8 = reinterpret_cast<uint8_t*>(wany);
  const unsigned long long* qmask = a.qmask + 4 * ((int64_t)(start >> 6) + g) + w;
  for (int cbeg = (int)((L - 1) / CHUNK) * CHUNK; cbeg >= 0; cbeg -= CHUNK) {
    const int n = min(CHUNK, (int)L - cbeg);
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += S::NT) {
      const uint32_t sp = a.sorted[start + cbeg + i];
      const float4* rec = reinterpret_cast<const float4*>(a.rec + (int64_t)sp * kRecF);
      s0[i] = rec[0]; s1[i] = rec[1]; s2[i] = make_float4(rec[2].x, 0.0f, 0.0f, 0.0f);
      sid[i] = sp;
      wany[i] = 0u;
    }
    __syncthreads();
    // Entries this wave's pixels took in the forward pass (its contribution
    // mask bit), visited back to front in groups of 4.  A pixel takes an
    // entry here exactly when it took it in the forward pass (the same alpha
    // bits, the same stop position), so every visited entry has a
    // contributing pixel in the wave and its partial is written unchecked.
    for (int gb = (n - 1) & ~63; gb >= 0; gb -= 64) {
      unsigned long long m = (uint32_t)(cbeg + gb) < Lw ? qmask[4 * (int64_t)((cbeg + gb) >> 6)] : 0ull;
      while (m) {
        int e[U];
        int cnt = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          e[u] = -1;
          if (m) {
            const int hb = 63 - __clzll((long long)m);
            m &= ~(1ull << hb);
            e[u] = gb + hb;
            ++cnt;
          }
        }
        if (cnt <= 2) {
          // a short group (the tail of a chunk): two entries, one lane-swap
          // fold (entry 0 in lanes 0-31, entry 1 in 32-63), the transposed
          // row sums, then each half-wave's two rows added
          float acc2[2][9];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int i = e[u] < 0 ? e[0] : e[u];
            const uint32_t li = e[u] < 0 ? 0xffffffffu : (uint32_t)(cbeg + i);
            entry_grad<S::PX>(s0[i], s1[i], s2[i].x, li, pxf, pyf, nit, T_, SG, G0, G1, G2, acc2[u]);
          }
          fold32x9(acc2[0], acc2[1]);
          const float tot = row_pair_sum(rows_transposed9(acc2[0], lane));
          const int li = lane & 15;
          if ((lane & 16) == 0 && ((li & 1) == 0 || li == 1)) {   // rows 0 and 2, one lane per value
            const int u = lane >> 5;
            const int eu = u == 0 ? e[0] : e[1];
            const int c = (li & 1) ? 8 : (((li >> 1) & 1) << 2) | (((li >> 2) & 1) << 1) | ((li >> 3) & 1);
            if (u < cnt) {
              red[eu][w][c] = tot;
              if (li == 1) wany8[eu * 4 + w] = 1;
            }
          }
          continue;
        }
        float acc[U][9];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          // an absent entry is folded as an untaken one (zeros, state kept)
          const int i = e[u] < 0 ? e[0] : e[u];
          const uint32_t li = e[u] < 0 ? 0xffffffffu : (uint32_t)(cbeg + i);
          entry_grad<S::PX>(s0[i], s1[i], s2[i].x, li, pxf, pyf, nit, T_, SG, G0, G1, G2, acc[u]);
        }
        // Sums of the 4 x 9 partials over the wave's 64 lanes, in a fixed
        // order: fold lanes 32 apart (entries 0|1 and 2|3 into one register
        // per value), then 16 apart (all four entries of a value in one
        // register, a row each: row r holds entry (r >> 1) | ((r & 1) << 1)),
        // then the transposed in-row sums, which leave each of the entry's 9
        // totals in its own lane of the row.
        fold32x9(acc[0], acc[1]);
        fold32x9(acc[2], acc[3]);
        fold16x9(acc[0], acc[2]);
        const float tot = rows_transposed9(acc[0], lane);
        // the group's chunk positions (< CHUNK <= 256), one byte each, so that
        // a lane picks its row's entry with one shift
        const uint32_t epack = (uint32_t)(e[0] & 0xff) | ((uint32_t)(e[1] & 0xff) << 8) |
                               ((uint32_t)(e[2] & 0xff) << 16) | ((uint32_t)(e[3] & 0xff) << 24);
        const int li = lane & 15;
        if ((li & 1) == 0 || li == 1) {   // one lane per value of the row
          const int r = lane >> 4, u = (r >> 1) | ((r & 1) << 1);
          const int eu = (int)((epack >> (8 * u)) & 0xffu);
          const int c = (li & 1) ? 8 : (((li >> 1) & 1) << 2) | (((li >> 2) & 1) << 1) | ((li >> 3) & 1);
          if (u < cnt) {
            red[eu][w][c] = tot;
            if (li == 1) wany8[eu * 4 + w] = 1;
          }
        }
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += S::NT) {
      const uint32_t wa = wany[i];
      if (wa == 0u) continue;
      float v[9];   // -0 + x is x for every x, so the first wave's add folds away
#pragma unroll
      for (int c = 0; c < 9; ++c) v[c] = -0.0f;
#pragma unroll
      for (int ww = 0; ww < S::NW; ++ww) {
        if (!((wa >> (8 * ww)) & 0xffu)) continue;
#pragma unroll
        for (int c = 0; c < 9; ++c) v[c] += red[i][ww][c];
      }
      // emission slot: the splat's offset + row-major index of this tile in its rect
      const uint32_t sp = sid[i];
      const int4 r = a.rect[sp];
      const uint32_t e = a.soff[sp] + (uint32_t)((ty - r.y) * (r.z - r.x + 1) + (tx - r.x));
      float4* dst = reinterpret_cast<float4*>(a.part + (int64_t)e * kPartF);
      dst[0] = make_float4(v[0], v[1], v[2], v[3]);
      dst[1] = make_float4(v[4], v[5], v[6], v[7]);
      dst[2] = make_float4(v[8], 0.0f, 0.0f, 0.0f);
      a.part_flag[e] = 1;
    }
  }
}

// One workgroup per tile, a wave per quadrant, one pixel per lane (tiles of 8
// and 16 pixels).  The list is walked back to front in batches of 64
// positions (those of the forward pass, whose 64-bit masks say which entries
// each quadrant took); a wave visits the entries its quadrant took.  A pixel
// takes an entry here exactly when it took it in the forward pass (the same
// alpha bits, the same stop position), so every visited entry has a
// contributing pixel in the wave and its partial is written unchecked.
//
// Per visited entry a lane forms two numbers, t and the blending weight; the
// entry's nine sums over the pixels are t's products with 1, dx, dy, dx^2,
// dx dy, dy^2 (the pixel's offset from the mean) and the weight's with the
// pixel's three image gradients.  The sums are taken 8 entries at a time with
// the roles of the lanes exchanged: the two numbers go to LDS a row of 64
// pixels per entry, and lane 8 e + y reads back the 8 pixels of row y of entry
// e, sums them along x in registers (dx from the entry's mean; the image
// gradients of its 8 pixels stay in registers), forms the y moments of its
// sums (dy is one number for the row), and 20 more operations add the 8 lanes'
// nine sums: 12 vector operations a visit where nine products and the
// cross-lane sums of each entry took 27.  (Moments about the quadrant's
// centre, moved to the mean once per (tile, entry), take 9 operations, the powers
// of x being literals, but the move cancels where the splat is smaller than its
// distance from the centre: for the smallest splats, sigma 0.55 pixels, the
// second moments carry 80 u sum |t| dx^2 where these carry 0.6.)
// (As a product on the matrix cores, 16 v_mfma_f32_16x16x4f32 per 8 entries,
// the sums cost as much: 6 and 3 of its 16 columns are used, and the vector
// unit stands still meanwhile.)
//
// Records, emission slots and masks of the next batch are read while one is
// worked on (a batch's chain sorted -> record is two load latencies, and a
// frame rendered alone is bound by its longest tile's walk).
// Measured (us, against nine products and lane swaps per entry, the masks as
// bytes per entry, records read between two barriers): 16 frames of 512 x 512
// and 50k Gaussians 402 -> 302, 10 mesh-bound ones 638 -> 405, 64 uneven
// frames of 100k 1285 -> 1080, five of 333 x 500 166 -> 117, one of 128 x 128
// 88 -> 56.  With alpha / (1 - alpha) in place of 1 / (1 - alpha), the clamp
// in the power, and the rows' reads contiguous (below): 304 -> 294, 404 -> 391,
// 1090 -> 1065, 118 -> 114, 56 -> 54.  With the moments about the mean instead of
// the quadrant's centre, and a t of 0 whatever the state: 292 -> 301, 388 -> 408,
// 1054 -> 1080, 113 -> 119, 54 -> 57.  Bound by instruction issue: 148M vector
// operations (204M at first), 80 % of the slots, 5 waves a SIMD by LDS.
// A row of 64 pixels in LDS: the halves of the quadrant's rows (4 pixels, 16
// bytes) in order of (half, row), so that the 8 lanes of an entry read 128
// bytes in one piece.  The bank conflicts that are left (a quarter of the LDS
// cycles: rows a multiple of the banks apart, the lower half of a write's lanes
// in 16 banks) cost nothing: without any of them 294 as well.
constexpr int kBwdRow = 64;

// One entry folded into a lane's back-to-front state (transmittance in front
// of the entry, colour behind it), in two parts.  A lane whose pixel did not
// take the entry folds alpha / (1 - alpha) = 0: its state passes through
// unchanged, the weight is 0 and so is t, whatever the state (a product in which
// 0 times anything is 0, or a gradient that is not finite at this pixel would
// reach entries that it did not take).
struct EntryAlpha {
  float q, qt, cg;       // alpha / (1 - alpha), the same with 0 where the alpha is clamped, <colour, dL/dout>
};
__device__ __forceinline__ EntryAlpha entry_alpha(float al, bool before_stop, const float4 r1, float cbl, float G0,
                                                  float G1, float G2) {
  EntryAlpha x;
  const float q = al * __builtin_amdgcn_rcpf(1.0f - al);
  x.q = before_stop && al >= kAlphaMin ? q : 0.0f;
  x.cg = r1.z * G0 + r1.w * G1 + cbl * G2;
  x.qt = al < kAlphaMax ? x.q : 0.0f;               // min(0.99, .) passes the gradient only below the clamp
  return x;
}
__device__ __forceinline__ void entry_fold(const EntryAlpha& x, float& T_, float& SG, float& t, float& wgt) {
  const float d = T_ * x.cg - SG;                   // (1 - alpha) d out / d alpha
  wgt = x.q * T_;                                   // alpha times the transmittance in front of the entry
  SG += wgt * x.cg;                                 // <colour behind, dL/dout>
  T_ += wgt;
  asm("v_mul_legacy_f32 %0, %1, %2" : "=v"(t) : "v"(x.qt), "v"(d));   // q d, 0 for q = 0
}

// The highest set bit of a wave-uniform mask, cleared there (64: none).
__device__ __forceinline__ uint32_t pop_highest(unsigned long long& m) {
  int z;
  asm("s_flbit_i32_b64 %0, %1" : "=s"(z) : "s"(m));   // -1 for 0
  const uint32_t e = (uint32_t)(63 - z);
  asm("s_bitset0_b64 %0, %1" : "+s"(m) : "s"(e));     // (64 clears bit 0 of 0)
  return e;
}

// The sums over the 8 lanes of each group of 9 values: lane i of a group
// returns the total of value 4 i0 + 2 i1 + i2 (its bits), and the ninth's in
// `last`.  Partners by row_half_mirror (whole DPP banks: one bank-masked add
// in place per value, two wait states before and after for the DPP reads),
// then 2 and 1 lanes apart.
#define GBR_BANK_PAIR(x, y)                                                                        \
  "v_add_f32_dpp %" #x ", %" #x ", %" #x " row_half_mirror row_mask:0xf bank_mask:0x5\n\t"     \
  "v_add_f32_dpp %" #x ", %" #y ", %" #y " row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
__device__ __forceinline__ float octets_transposed9(const float (&v)[9], int lane, float& last) {
  constexpr int kQuadXor2 = 0x4e, kQuadXor1 = 0xb1;
  float a0 = v[0], a1 = v[2], a2 = v[4], a3 = v[6], a4 = v[8];
  asm volatile("s_nop 1\n\t" GBR_BANK_PAIR(0, 5) GBR_BANK_PAIR(1, 6) GBR_BANK_PAIR(2, 7) GBR_BANK_PAIR(3, 8)
               "v_add_f32_dpp %4, %4, %4 row_half_mirror row_mask:0xf bank_mask:0xf\n\ts_nop 1"
               : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3), "+v"(a4)
               : "v"(v[1]), "v"(v[3]), "v"(v[5]), "v"(v[7]));
  const bool b1 = lane & 2, b0 = lane & 1;
  const float d0 = pair_fold<kQuadXor2>(a0, a1, b1), d1 = pair_fold<kQuadXor2>(a2, a3, b1);
  a4 += dpp_mov<kQuadXor2, 0xf, 0xf, false>(a4);
  last = a4 + dpp_mov<kQuadXor1, 0xf, 0xf, false>(a4);
  return pair_fold<kQuadXor1>(d0, d1, b0);
}
#undef GBR_BANK_PAIR

// (tiles of 8: 9.8 KB of LDS a wave leave room for 4 a SIMD)
template <int T>
__global__ __launch_bounds__(TileShapeB<T>::NT, T == 8 ? 4 : 5) void composite_bwd_kernel(
    PassArgs a, const float* __restrict__ dimages) {
  using S = TileShapeB<T>;
  static_assert(S::PX == 1 && S::QW == 8, "a pixel per lane, quadrants of 8 x 8");
  constexpr int NW = S::NW;
  __shared__ float4 st[3][65];              // mx my ca cb | cc lo r g | b; row 64: an entry that is never taken
  __shared__ uint32_t slot[64];             // emission slot
  __shared__ float red[65][NW][9];          // a wave's sums of an entry; row 64 takes what a short group leaves over
  __shared__ __align__(16) float tb[NW][16 * kBwdRow];
  if (a.status->overflow) return;
  const int g = tile_of_rank(a.cls_cnt + 33, a.order_bwd, a.n_tiles, blockIdx.x);
  if (g < 0) return;
  const uint32_t L = a.tile_last[g];
  if (L == 0) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = frame_of_tile(a.frames, a.B, g);
  const FrameDev& F = a.frames[b];
  const int lt = g - F.tile_base;
  const int tx = lt % F.ntx, ty = lt / F.ntx;
  const uint32_t start = a.tile_start[g];
  const int px = tx * T + S::lx0(threadIdx.x), py = ty * T + S::ly0(threadIdx.x);
  const float pxf = (float)px + 0.5f, pyf = (float)py + 0.5f;
  uint32_t nit = 0;
  float T_ = 1.0f, SG = 0.0f, G0 = 0.0f, G1 = 0.0f, G2 = 0.0f;
  if (px < F.W && py < F.H) {
    const float* img_g = dimages + F.pix_base * 3;
    const int64_t hw = (int64_t)F.W * F.H, pix = (int64_t)py * F.W + px;
    nit = a.n_iter[F.pix_base + pix];
    T_ = a.t_final[F.pix_base + pix];
    G0 = img_g[pix]; G1 = img_g[hw + pix]; G2 = img_g[2 * hw + pix];
    // <colour behind the current entry, dL/dout>, starts at <T_end * background, dL/dout>
    SG = T_ * (F.bg[0] * G0 + F.bg[1] * G1 + F.bg[2] * G2);
  }
  // the lane's part of the sums: a row of entry lane / 8 of a group, its pixel
  // centres at (qx[k], qy); the image gradients of that row's pixels
  const int q0x = tx * T + (w & 1) * 8, q0y = ty * T + (w >> 1) * 8;   // (w = 0 in tiles of 8)
  const float qy = (float)(q0y + (lane & 7)) + 0.5f;
  float qx[8];                              // (uniform: scalar registers)
#pragma unroll
  for (int k = 0; k < 8; ++k)
    qx[k] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int((float)(q0x + k) + 0.5f)));
  float* tw = tb[w];
  const float* twr = tw + (lane >> 3) * kBwdRow + (lane & 7) * 4;
  const int cell = (lane & 4) * 8 + (lane >> 3) * 4 + (lane & 3);
  const int value = 4 * (lane & 1) + (lane & 2) + ((lane >> 2) & 1);   // which of the sums the lane ends with
  float gx[8][3];
  if (threadIdx.x < 3) st[threadIdx.x][64] = make_float4(0.0f, threadIdx.x == 1 ? -1e30f : 0.0f, 0.0f, 0.0f);
  {
    tw[cell] = G0; tw[kBwdRow + cell] = G1; tw[2 * kBwdRow + cell] = G2;
    wave_sync();
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int k = 0; k < 8; ++k) gx[k][c] = tw[c * kBwdRow + (k & 4) * 8 + (lane & 7) * 4 + (k & 3)];
    wave_sync();
  }
  // this lane's part of a batch's write-out: a quadrant's sums of one entry
  const int oi = w * (64 / NW) + lane / NW, oq = lane % NW;
  const uint32_t oql = a.qlast[g * 4 + oq];   // quadrant oq took nothing at or past it (its masks end there)
  const unsigned long long* qmask = a.qmask + 4 * ((int64_t)(start >> 6) + g) + oq;
  const uint32_t* srt = a.sorted + start;

  // a batch's records and slots, on their way from memory (a lane per entry;
  // four waves read a piece each: a third of the record, or the slot)
  float4 p0, p1, p2;
  uint32_t pslot = 0, sp = 0;
  auto read_batch = [&](uint32_t s) {
    const float4* rec = reinterpret_cast<const float4*>(a.rec + (int64_t)s * kRecF);
    if (NW == 1 || w < 3) p0 = rec[NW == 1 ? 0 : w];
    if (NW == 1) { p1 = rec[1]; p2 = rec[2]; }
    if (NW == 1 || w == 3) {   // the splat's offset + row-major index of this tile in its rect
      const int4 r = a.rect[s];
      pslot = a.soff[s] + (uint32_t)((ty - r.y) * (r.z - r.x + 1) + (tx - r.x));
    }
  };
  const uint32_t cl = (L - 1u) & ~63u;      // the last batch
  read_batch(srt[min(cl + (uint32_t)lane, L - 1u)]);   // (lanes past the last used position: its last entry)
  unsigned long long nmask = qmask[4 * (int64_t)(cl >> 6)];   // quadrant oq's mask of the batch
  if (cl > 0) sp = srt[cl - 64u + (uint32_t)lane];
  for (uint32_t c0 = cl;; c0 -= 64u) {
    // ---- the batch's records to LDS; the next ones on their way ----
    if (NW == 1 || w < 3) st[NW == 1 ? 0 : w][lane] = p0;
    if (NW == 1) { st[1][lane] = p1; st[2][lane] = p2; }
    if (NW == 1 || w == 3) slot[lane] = pslot;
    const unsigned long long omask = c0 < oql ? nmask : 0ull;
    unsigned long long m;
    __syncthreads();
    if (c0 > 0) {
      nmask = qmask[4 * (int64_t)((c0 >> 6) - 1u)];
      read_batch(sp);
      if (c0 > 64u) sp = srt[c0 - 128u + (uint32_t)lane];
    }
    m = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(omask >> 32), w) << 32) |
        (uint32_t)__builtin_amdgcn_readlane((int)omask, w);   // lane w holds quadrant w's
    const bool obit = (omask >> oi) & 1ull;
    bool any = obit;                        // some quadrant took the entry
    if (NW == 4) {
      int x = obit ? 1 : 0;
      x |= __builtin_amdgcn_update_dpp(0, x, 0xb1, 0xf, 0xf, false);   // quad_perm: lanes 1 apart, then 2 apart
      x |= __builtin_amdgcn_update_dpp(0, x, 0x4e, 0xf, 0xf, false);
      any = x != 0;
    }
    const uint32_t oslot = slot[oi];
    // ---- the quadrant's entries, back to front, in groups of 8 ----
    while (m) {
      uint32_t elo = 0x40404040u, ehi = 0x40404040u;   // the group's positions, a byte each (64: no entry)
#pragma unroll
      for (int h = 0; h < 4; ++h) {         // a pair of entries
        if (m) {
          const uint32_t ea = pop_highest(m), eb = pop_highest(m);   // (eb = 64: none left)
          const uint32_t pair = ea | (eb << 8);
          uint32_t& eh = h < 2 ? elo : ehi;
          eh = (h & 1) ? (eh & 0xffffu) | (pair << 16) : 0x40400000u | pair;
          const float4 a0 = st[0][ea], a1 = st[1][ea], b0 = st[0][eb], b1 = st[1][eb];
          const float a2 = st[2][ea].x, b2 = st[2][eb].x;
          float ta, wa, tc, wc;
          const float aa = clamped_alpha(a0, a1.x, a1.y, pxf, pyf);
          const float ab = clamped_alpha(b0, b1.x, b1.y, pxf, pyf);
          const EntryAlpha xa = entry_alpha(aa, c0 + ea < nit, a1, a2, G0, G1, G2);
          const EntryAlpha xb = entry_alpha(ab, c0 + eb < nit, b1, b2, G0, G1, G2);
          entry_fold(xa, T_, SG, ta, wa);
          entry_fold(xb, T_, SG, tc, wc);
          tw[(2 * h) * kBwdRow + cell] = ta;
          tw[(2 * h + 1) * kBwdRow + cell] = tc;
          tw[(8 + 2 * h) * kBwdRow + cell] = wa;
          tw[(9 + 2 * h) * kBwdRow + cell] = wc;
        }
      }
      wave_sync();
      // the row's 8 pixels (a short group's unwritten rows only spoil their own sums)
      const uint32_t e = ((lane & 32 ? ehi : elo) >> (lane & 24)) & 0xffu;
      const float2 mean = *reinterpret_cast<const float2*>(&st[0][e]);
      float t[8], wg[8];
#pragma unroll
      for (int k = 0; k < 8; k += 4) {
        float4 x = *reinterpret_cast<const float4*>(twr + 8 * k);
        float4 y = *reinterpret_cast<const float4*>(twr + 8 * kBwdRow + 8 * k);
        asm("" : "+v"(x.x), "+v"(x.y), "+v"(x.z), "+v"(x.w));   // (as one read of 16 bytes)
        t[k] = x.x; t[k + 1] = x.y; t[k + 2] = x.z; t[k + 3] = x.w;
        wg[k] = y.x; wg[k + 1] = y.y; wg[k + 2] = y.z; wg[k + 3] = y.w;
      }
      wave_sync();
      float v[9];
      {
        float p[8], m2 = 0.0f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float dx = qx[k] - mean.x;
          p[k] = t[k] * dx;
          m2 = k == 0 ? p[0] * dx : __builtin_fmaf(p[k], dx, m2);
        }
        const float dy = qy - mean.y;
        v[5] = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
        v[0] = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
        v[2] = m2;
        v[1] = dy * v[5];
        v[3] = dy * v[0];
        v[4] = dy * v[1];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          v[6 + c] = wg[0] * gx[0][c];
#pragma unroll
          for (int k = 1; k < 8; ++k) v[6 + c] = __builtin_fmaf(wg[k], gx[k][c], v[6 + c]);
        }
      }
      float ninth;
      const float tot = octets_transposed9(v, lane, ninth);
      red[e][w][value] = tot;
      if ((lane & 7) == 0) red[e][w][8] = ninth;
    }
    __syncthreads();
    // ---- the batch's partials: the quadrants' sums added in order ----
    if (any) {
      float v[9];
#pragma unroll
      for (int c = 0; c < 9; ++c) v[c] = obit ? red[oi][oq][c] : 0.0f;
      if (NW == 4) {                        // (an entry's four lanes take this branch together)
#pragma unroll
        for (int c = 0; c < 9; ++c) {
          v[c] += dpp_mov<0xb1, 0xf, 0xf, false>(v[c]);
          v[c] += dpp_mov<0x4e, 0xf, 0xf, false>(v[c]);
        }
      }
      float4* dst = reinterpret_cast<float4*>(a.part + (int64_t)oslot * kPartF);
      if (NW == 1 || oq == 0) dst[0] = make_float4(v[0], v[1], v[2], v[3]);
      if (NW == 1 || oq == 1) dst[1] = make_float4(v[4], v[5], v[6], v[7]);
      if (NW == 1 || oq == 2) dst[2] = make_float4(v[8], 0.0f, 0.0f, 0.0f);
      if (NW == 1 || oq == 3) a.part_flag[oslot] = 1;
    }
    if (c0 == 0) break;
  }
}

void launch_composite_bwd(const PassArgs& a, const float* dimages, const float* images, int chunk, hipStream_t s) {
  (void)images;
  if (a.n_tiles == 0) return;
  const dim3 grid(a.n_tiles);
  if (a.tile == 8) {
    hipLaunchKernelGGL(composite_bwd_kernel<8>, grid, dim3(TileShapeB<8>::NT), 0, s, a, dimages);
  } else if (a.tile == 16) {
    hipLaunchKernelGGL(composite_bwd_kernel<16>, grid, dim3(TileShapeB<16>::NT), 0, s, a, dimages);
  } else {
    const dim3 nt(TileShapeB<32>::NT);
    if (chunk == 64) hipLaunchKernelGGL(composite_bwd32_kernel<64>, grid, nt, 0, s, a, dimages);
    else if (chunk == 128) hipLaunchKernelGGL(composite_bwd32_kernel<128>, grid, nt, 0, s, a, dimages);
    else hipLaunchKernelGGL(composite_bwd32_kernel<256>, grid, nt, 0, s, a, dimages);
  }
}

// ---------------------------------------------------------------- gather + projection adjoint
// A splat's entries' partials are summed in row-major tile order (unflagged
// entries -- no contributing pixel, or past the tile's last used position --
// are zero), each flag read is reset to 0 for the next pass, and the 9 sums
// are chained back through the conic, the EWA projection and the activations
// in float64 into the splat's draw row.
//
// Batches of kTwoPassSplats splats or more do it in two passes.  The gather
// writes every splat's sums to its row and lists the splats with a flagged
// entry, a list per workgroup: most splats lie behind the ones that stop the
// pixels and have none (half to four fifths of those measured).  The adjoint,
// a wave per list, rewrites the listed splats' rows.  The entries of a wave's
// 64 splats are one run of emission slots, which the wave gathers together:
// flags 16 to a lane (1024 entries a window); the flagged entries listed in
// LDS; their 48-byte partials fetched by three lanes each, 21 to a load, and
// added from LDS by the splat's lane; the rows written as one run.  With a
// thread reading its own splat's flags, partials and row, five times as many
// memory instructions are issued, most of their lanes idle or on lines of
// their own, and their issue bounds the pass.  Smaller batches keep that form,
// one launch: the second launch's latencies cost more than it saves.
// Measured, one launch against two (us): 100k splats 18 / 22, 150k 15 / 21,
// 500k 47 / 44, 600k (half of them listed) 89 / 80, 800k 76 / 64, 6.4M
// 361 / 287.  A gradient written over the Gaussians themselves takes one launch:
// two would overwrite them with the sums before the adjoint reads them.
constexpr int64_t kTwoPassSplats = 500000;

// Flag bytes (0 or 1) of 4 entries -> 4 bits.
__device__ __forceinline__ uint32_t flag_nibble(uint32_t w) {
  return (w & 1u) | ((w >> 7) & 2u) | ((w >> 14) & 4u) | ((w >> 21) & 8u);
}

constexpr int kGatherThreads = 256;       // splats per list: the projection's workgroups
constexpr int kGatherWindow = 1024;       // entries whose flags a wave reads at once
constexpr int kGatherStage = 63;          // partials a wave stages at once: three rounds of 21

struct GatherWave {
  float4 stage[64 * 4];                   // partials (3 to an entry), then the draw rows
  uint16_t hit[kGatherWindow];            // the window's flagged entries, from its first slot
  uint16_t bits[64];                      // the flags of each lane's 16 entries
  uint16_t before[64];                    // and the flagged entries before them
};

__global__ __launch_bounds__(kGatherThreads) void gather_sums_kernel(PassArgs a, float* __restrict__ draw) {
  __shared__ GatherWave gw[kGatherThreads / 64];
  __shared__ uint32_t wn[kGatherThreads / 64];
  const int b = blockIdx.y;
  const FrameDev& F = a.frames[b];
  const int64_t n0 = (int64_t)blockIdx.x * kGatherThreads;
  if (n0 >= F.gauss_count) return;          // (uniform)
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  GatherWave& G = gw[w];
  const int64_t nw = n0 + w * 64;           // the wave's first splat
  const int rows = (int)min((int64_t)64, F.gauss_count - nw);   // (may be negative: nothing to do)
  const int64_t s = F.gauss_base + min(nw + lane, F.gauss_count - 1);
  const uint32_t ovf = a.status->overflow;
  const uint32_t off = a.soff[s], cnt = lane < rows ? a.cnt[s] : 0u;
  float acc[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k] = 0.0f;
  bool any = false;
  if (rows > 0 && !ovf) {
    const uint32_t first = __builtin_amdgcn_readlane((int)off, 0);
    const uint32_t end = __builtin_amdgcn_readlane((int)(off + cnt), rows - 1);
    for (uint32_t e0 = first & ~15u; e0 < end; e0 += kGatherWindow) {
      // ---- the window's flags: 16 to a lane, read and cleared ----
      const uint32_t el = e0 + 16u * (uint32_t)lane;
      uint32_t m = 0u;
      if (el < end) {
        uint4* fl = reinterpret_cast<uint4*>(a.part_flag + el);   // (padded by 64 bytes past the capacity)
        const uint4 x = *fl;
        m = flag_nibble(x.x) | flag_nibble(x.y) << 4 | flag_nibble(x.z) << 8 | flag_nibble(x.w) << 12;
        // only this wave's entries; the others' flags stay
        const uint32_t lo = first > el ? first - el : 0u, hi = min(end - el, 16u);
        m &= ((1u << hi) - 1u) & ~((1u << lo) - 1u);
        if (m != 0u) {
          if (lo == 0u && hi == 16u) {
            *fl = make_uint4(0u, 0u, 0u, 0u);
          } else {
            for (uint32_t r = m; r != 0u; r &= r - 1u) a.part_flag[el + (uint32_t)__builtin_ctz(r)] = 0;
          }
        }
      }
      const uint32_t c = __popc(m), inc = wave_incl_scan(c);
      const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
      if (total == 0u) continue;
      wave_sync();
      G.bits[lane] = (uint16_t)m;
      G.before[lane] = (uint16_t)(inc - c);
      uint32_t at = inc - c;
      for (uint32_t r = m; r != 0u; r &= r - 1u) G.hit[at++] = (uint16_t)(16 * lane + __builtin_ctz(r));
      wave_sync();
      // ---- this splat's flagged entries: [h0, h1) of the window's ----
      auto place = [&](uint32_t e) -> uint32_t {   // flagged entries before slot e
        if (e <= e0) return 0u;
        const uint32_t d = e - e0;
        if (d >= (uint32_t)kGatherWindow) return total;
        return G.before[d >> 4] + (uint32_t)__popc(G.bits[d >> 4] & ((1u << (d & 15u)) - 1u));
      };
      const uint32_t h0 = place(off), h1 = cnt ? place(off + cnt) : h0;
      any |= h1 > h0;
      // ---- their partials, staged and added in slot order; a round's are
      // on their way while the round before is added ----
      auto piece = [&](uint32_t g0, int j) -> float4 {   // piece t % 3 of entry g0 + t / 3, t = 63 j + lane
        const uint32_t t = (uint32_t)(63 * j + min(lane, 62)), r = min(g0 + t / 3u, total - 1u);
        return reinterpret_cast<const float4*>(a.part + (int64_t)(e0 + G.hit[r]) * kPartF)[t % 3u];
      };
      float4 x0 = piece(0, 0), x1 = piece(0, 1), x2 = piece(0, 2);
      for (uint32_t g0 = 0; g0 < total; g0 += kGatherStage) {
        wave_sync();
        if (lane < 63) {
          G.stage[lane] = x0;
          G.stage[63 + lane] = x1;
          G.stage[126 + lane] = x2;
        }
        wave_sync();
        const uint32_t g1 = g0 + kGatherStage;
        if (g1 < total) { x0 = piece(g1, 0); x1 = piece(g1, 1); x2 = piece(g1, 2); }
        const uint32_t hb = min(max(h0, g0), g1), he = min(max(h1, g0), g1);
        for (uint32_t h = hb; h < he; ++h) {
          const float4* q = G.stage + 3u * (h - g0);
          const float4 q0 = q[0], q1 = q[1];
          acc[0] += q0.x; acc[1] += q0.y; acc[2] += q0.z; acc[3] += q0.w;
          acc[4] += q1.x; acc[5] += q1.y; acc[6] += q1.z; acc[7] += q1.w;
          acc[8] += q[2].x;
        }
      }
    }
  }
  // ---- the draw rows, a contiguous run of memory ----
  wave_sync();
  G.stage[4 * lane] = make_float4(acc[0], acc[1], acc[2], acc[3]);
  G.stage[4 * lane + 1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
  G.stage[4 * lane + 2] = make_float4(acc[8], 0.f, 0.f, 0.f);
  G.stage[4 * lane + 3] = make_float4(0.f, 0.f, 0.f, 0.f);
  wave_sync();
  if (rows > 0) {
    float4* out = reinterpret_cast<float4*>(draw + (F.gauss_base + nw) * kNF);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (64 * j + lane < 4 * rows) out[64 * j + lane] = G.stage[64 * j + lane];
  }
  // ---- the workgroup's splats with a gradient, in order ----
  const unsigned long long m = __ballot(any);
  if (lane == 0) wn[w] = (uint32_t)__popcll(m);
  __syncthreads();
  uint32_t at = lanes_below(m);
  for (int i = 0; i < w; ++i) at += wn[i];
  if (any) a.hits[F.gauss_base + n0 + at] = (uint32_t)(nw + lane);
  if (threadIdx.x == kGatherThreads - 1)
    a.blk_mm[2 * (F.gauss_base / kGatherThreads + b + blockIdx.x)] = at + (any ? 1u : 0u);
}

constexpr int kAdjThreads = 64;

// The adjoint of frame b's splat n: v0, v1, v2 the first three float4 of its
// blended record, acc its sums.
__device__ __forceinline__ void splat_adjoint(const PassArgs& a, const FrameDev& F, int b, int64_t n, float4 v0,
                                              float4 v1, const float4 v2, const float (&acc)[9],
                                              float* __restrict__ draw) {
  float4* out = reinterpret_cast<float4*>(draw + (F.gauss_base + n) * kNF);

  // ---- recompute the forward quantities (float64) ----
  if (a.tg.on) tangent_deform(a.tg, b, n, v0, v1, v0, v1);   // as the forward pass did
  const float gp[11] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w, v2.x, v2.y, v2.z};
  const double mu0 = gp[0], mu1 = gp[1], mu2 = gp[2];
  double R[9], tcam[3];
  for (int i = 0; i < 9; ++i) R[i] = F.R[i];
  for (int i = 0; i < 3; ++i) tcam[i] = R[3 * i] * mu0 + R[3 * i + 1] * mu1 + R[3 * i + 2] * mu2 + (double)F.t[i];
  const double tx = tcam[0], ty = tcam[1], tz = tcam[2];
  const double qraw[4] = {gp[3], gp[4], gp[5], gp[6]};
  const double qn2 = qraw[0] * qraw[0] + qraw[1] * qraw[1] + qraw[2] * qraw[2] + qraw[3] * qraw[3];
  const double qlen = sqrt(qn2);
  const double qw = qraw[0] / qlen, qx = qraw[1] / qlen, qy = qraw[2] / qlen, qz = qraw[3] / qlen;
  const double sc[3] = {exp((double)gp[7]), exp((double)gp[8]), exp((double)gp[9])};
  const double o = 1.0 / (1.0 + exp(-(double)gp[10]));
  double Rq[9];
  Rq[0] = 1.0 - 2.0 * (qy * qy + qz * qz); Rq[1] = 2.0 * (qx * qy - qw * qz); Rq[2] = 2.0 * (qx * qz + qw * qy);
  Rq[3] = 2.0 * (qx * qy + qw * qz); Rq[4] = 1.0 - 2.0 * (qx * qx + qz * qz); Rq[5] = 2.0 * (qy * qz - qw * qx);
  Rq[6] = 2.0 * (qx * qz - qw * qy); Rq[7] = 2.0 * (qy * qz + qw * qx); Rq[8] = 1.0 - 2.0 * (qx * qx + qy * qy);
  double M[9];
  for (int i = 0; i < 3; ++i)
    for (int k = 0; k < 3; ++k) M[3 * i + k] = Rq[3 * i + k] * sc[k];
  const double iz = 1.0 / tz;
  const double fx = F.fx, fy = F.fy;
  const double jx = fx * iz, jy = fy * iz, ux = -fx * tx * iz * iz, uy = -fy * ty * iz * iz;
  double Wm[6];
  for (int k = 0; k < 3; ++k) {
    Wm[k] = jx * R[k] + ux * R[6 + k];
    Wm[3 + k] = jy * R[3 + k] + uy * R[6 + k];
  }
  double V[6];
  for (int i = 0; i < 2; ++i)
    for (int k = 0; k < 3; ++k) V[3 * i + k] = Wm[3 * i] * M[k] + Wm[3 * i + 1] * M[3 + k] + Wm[3 * i + 2] * M[6 + k];
  const double sa = V[0] * V[0] + V[1] * V[1] + V[2] * V[2] + kLowPass;
  const double sb = V[0] * V[3] + V[1] * V[4] + V[2] * V[5];
  const double scc = V[3] * V[3] + V[4] * V[4] + V[5] * V[5] + kLowPass;
  const double det = sa * scc - sb * sb;
  const double QA = scc / det, QB = -sb / det, QC = sa / det;

  // ---- record-space gradient -> conic coefficients of q = A dx^2 + 2B dx dy + C dy^2 ----
  // dL/dpower = ln 2 * alpha * dL/dalpha, so the moments of t carry a factor ln 2
  double am[5];
  for (int k = 0; k < 5; ++k) am[k] = (double)acc[k] * kLn2;
  const double dA = am[2] * (-0.5 * kLog2e);
  const double dB = am[3] * (-kLog2e);      // cb = -log2e * B  (coefficient of dx dy is 2B)
  const double dC = am[4] * (-0.5 * kLog2e);
  // conic -> Sigma2 (symmetric):  dS = -Q dQ Q with dQ = [[dA, dB/2], [dB/2, dC]]
  const double h = 0.5 * dB;
  const double t00 = QA * dA + QB * h, t01 = QA * h + QB * dC;
  const double t10 = QB * dA + QC * h, t11 = QB * h + QC * dC;
  const double g00 = -(t00 * QA + t01 * QB);
  const double g01 = -(t00 * QB + t01 * QC);
  const double g11 = -(t10 * QB + t11 * QC);
  // Sigma2 = V V^T + c I:  dV = 2 G V
  double dV[6];
  for (int k = 0; k < 3; ++k) {
    dV[k] = 2.0 * (g00 * V[k] + g01 * V[3 + k]);
    dV[3 + k] = 2.0 * (g01 * V[k] + g11 * V[3 + k]);
  }
  // V = W M:  dW = dV M^T,  dM = W^T dV
  double dW[6], dM[9];
  for (int i = 0; i < 2; ++i)
    for (int k = 0; k < 3; ++k)
      dW[3 * i + k] = dV[3 * i] * M[3 * k] + dV[3 * i + 1] * M[3 * k + 1] + dV[3 * i + 2] * M[3 * k + 2];
  for (int i = 0; i < 3; ++i)
    for (int k = 0; k < 3; ++k) dM[3 * i + k] = Wm[i] * dV[k] + Wm[3 + i] * dV[3 + k];
  // W rows: jx R0 + ux R2, jy R1 + uy R2  ->  d(jx), d(ux), d(jy), d(uy)
  double djx = 0, dux = 0, djy = 0, duy = 0;
  for (int k = 0; k < 3; ++k) {
    djx += dW[k] * R[k]; dux += dW[k] * R[6 + k];
    djy += dW[3 + k] * R[3 + k]; duy += dW[3 + k] * R[6 + k];
  }
  // jx = fx/tz, ux = -fx tx/tz^2, jy = fy/tz, uy = -fy ty/tz^2; mean = (fx tx/tz + cx, fy ty/tz + cy)
  // mean: d power / d mean = -(2 ca dx + cb dy, cb dx + 2 cc dy), summed as (sum dpw dx, sum dpw dy)
  const double ca = -0.5 * kLog2e * QA, cbq = -kLog2e * QB, cc = -0.5 * kLog2e * QC;
  const double dmx = -(2.0 * ca * am[0] + cbq * am[1]);
  const double dmy = -(cbq * am[0] + 2.0 * cc * am[1]);
  double dtx = dux * (-fx * iz * iz) + dmx * fx * iz;
  double dty = duy * (-fy * iz * iz) + dmy * fy * iz;
  double dtz = djx * (-fx * iz * iz) + dux * (2.0 * fx * tx * iz * iz * iz) + djy * (-fy * iz * iz) +
               duy * (2.0 * fy * ty * iz * iz * iz) - dmx * fx * tx * iz * iz - dmy * fy * ty * iz * iz;
  float res[16];
  for (int k = 0; k < 3; ++k) res[k] = (float)(R[k] * dtx + R[3 + k] * dty + R[6 + k] * dtz);
  // M = Rq diag(s):  dRq = dM diag(s),  ds_k = sum_i dM_ik Rq_ik
  double dRq[9], ds[3];
  for (int k = 0; k < 3; ++k) {
    ds[k] = dM[k] * Rq[k] + dM[3 + k] * Rq[3 + k] + dM[6 + k] * Rq[6 + k];
    for (int i = 0; i < 3; ++i) dRq[3 * i + k] = dM[3 * i + k] * sc[k];
  }
  // d Rq / d (w, x, y, z) of the unit quaternion
  double dq[4];
  dq[0] = 2.0 * (qz * (dRq[3] - dRq[1]) + qy * (dRq[2] - dRq[6]) + qx * (dRq[7] - dRq[5]));
  dq[1] = 2.0 * (qy * (dRq[1] + dRq[3]) + qz * (dRq[2] + dRq[6]) + qw * (dRq[7] - dRq[5]) - 2.0 * qx * (dRq[4] + dRq[8]));
  dq[2] = 2.0 * (qx * (dRq[1] + dRq[3]) + qw * (dRq[2] - dRq[6]) + qz * (dRq[5] + dRq[7]) - 2.0 * qy * (dRq[0] + dRq[8]));
  dq[3] = 2.0 * (qw * (dRq[3] - dRq[1]) + qx * (dRq[2] + dRq[6]) + qy * (dRq[5] + dRq[7]) - 2.0 * qz * (dRq[0] + dRq[4]));
  const double dotq = qw * dq[0] + qx * dq[1] + qy * dq[2] + qz * dq[3];
  const double qh[4] = {qw, qx, qy, qz};
  for (int k = 0; k < 4; ++k) res[3 + k] = (float)((dq[k] - qh[k] * dotq) / qlen);
  for (int k = 0; k < 3; ++k) res[7 + k] = (float)(ds[k] * sc[k]);
  // alpha = 2^(... + log2 o), o = sigmoid(logit):  dL/dlogit = (1 - o) * sum alpha dL/dalpha
  res[10] = (float)((double)acc[5] * (1.0 - o));
  res[11] = acc[6]; res[12] = acc[7]; res[13] = acc[8];
  res[14] = 0.0f; res[15] = 0.0f;
  float4 o0 = make_float4(res[0], res[1], res[2], res[3]);
  float4 o1 = make_float4(res[4], res[5], res[6], res[7]);
  if (a.tg.on) tangent_adjoint(tangent_frame(a.tg, b, n), o0, o1, o0, o1);   // back to tangent space
  out[0] = o0;
  out[1] = o1;
  out[2] = make_float4(res[8], res[9], res[10], res[11]);
  out[3] = make_float4(res[12], res[13], res[14], res[15]);
}

// A wave per list (a wave per 64 of its splats costs more in empty waves than
// the longer lists' second rounds); the frame is the grid's y index, so its
// camera is read at uniform addresses.
__global__ __launch_bounds__(kAdjThreads, 3) void proj_adjoint_kernel(PassArgs a, const float* __restrict__ raw,
                                                                      float* __restrict__ draw) {
  const int b = blockIdx.y;
  const FrameDev& F = a.frames[b];
  const int64_t n0 = (int64_t)blockIdx.x * kGatherThreads;
  if (n0 >= F.gauss_count) return;
  const uint32_t count = a.blk_mm[2 * (F.gauss_base / kGatherThreads + b + blockIdx.x)];
  for (uint32_t i = threadIdx.x; i < count; i += kAdjThreads) {
    const int64_t n = a.hits[F.gauss_base + n0 + i], s = F.gauss_base + n;
    const float4* g = reinterpret_cast<const float4*>(draw + s * kNF);
    const float4* src = reinterpret_cast<const float4*>(raw + s * kNF);
    const float4 g0 = g[0], g1 = g[1], g2 = g[2], v0 = src[0], v1 = src[1], v2 = src[2];
    const float acc[9] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w, g2.x};
    splat_adjoint(a, F, b, n, v0, v1, v2, acc, draw);
  }
}

// The one-launch form, a thread per splat.
// The 9 sums of a splat over its c entries from off on (acc zeroed by the caller).
__device__ __forceinline__ void gather_splat_sums(const PassArgs& a, uint32_t off, uint32_t c, float (&acc)[9]) {
  const uint32_t end = off + c;
  const uint32_t* fw = reinterpret_cast<const uint32_t*>(a.part_flag);   // padded by 64 bytes past the capacity
  // windows of 64 entries starting at a multiple of 16: the 16 flag words
  // are read as four aligned 16-byte loads and turned into a bit mask of
  // the flagged entries, whose partials are then read 4 at a time (all 4
  // in flight together)
  for (uint32_t e0 = off & ~15u; e0 < end; e0 += 64) {
    uint32_t w[16];
    const uint4* fq = reinterpret_cast<const uint4*>(fw + (e0 >> 2));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint4 x = fq[k];
      w[4 * k] = x.x; w[4 * k + 1] = x.y; w[4 * k + 2] = x.z; w[4 * k + 3] = x.w;
    }
    unsigned long long m = 0ull;
#pragma unroll
    for (int k = 0; k < 16; ++k) m |= (unsigned long long)flag_nibble(w[k]) << (4 * k);
    // keep [off, end) only
    const uint32_t lo = off > e0 ? off - e0 : 0u;
    const uint32_t hi = end - e0 < 64u ? end - e0 : 64u;
    m &= (hi >= 64u ? ~0ull : ((1ull << hi) - 1ull)) & ~((1ull << lo) - 1ull);
    while (m) {
      uint32_t e[4];
      bool v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        v[u] = m != 0ull;
        e[u] = v[u] ? e0 + (uint32_t)(__ffsll((long long)m) - 1) : off;   // off: in range, unused
        m &= m - 1ull;
      }
      float4 q[4][3];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float4* src = reinterpret_cast<const float4*>(a.part + (int64_t)e[u] * kPartF);
        q[u][0] = src[0]; q[u][1] = src[1]; q[u][2] = src[2];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (!v[u]) continue;
        // the flag goes back to 0 for the next pass (only this splat's
        // flags are written; neighbours mask this entry out of their windows)
        a.part_flag[e[u]] = 0;
        acc[0] += q[u][0].x; acc[1] += q[u][0].y; acc[2] += q[u][0].z; acc[3] += q[u][0].w;
        acc[4] += q[u][1].x; acc[5] += q[u][1].y; acc[6] += q[u][1].z; acc[7] += q[u][1].w;
        acc[8] += q[u][2].x;
      }
    }
  }
}

// A workgroup per (frame, 64 of its splats): the frame is the grid's y
// index, so its camera is read at uniform addresses.  One-wave workgroups
// let the chip's last round of waves be filled finely (the splats' gathers
// differ in length).
__global__ __launch_bounds__(kAdjThreads) void gather_adjoint_kernel(PassArgs a, const float* __restrict__ raw,
                                                                   float* __restrict__ draw) {
  const int b = blockIdx.y;
  const FrameDev& F = a.frames[b];
  const int64_t n = (int64_t)blockIdx.x * kAdjThreads + threadIdx.x;
  if (n >= F.gauss_count) return;
  const int64_t s = F.gauss_base + n;
  float4* out = reinterpret_cast<float4*>(draw + s * kNF);
  // the overflow flag, the count, the entry offset and the splat's blended
  // Gaussian are read together, so that one load latency precedes the
  // gather instead of three
  const uint32_t ovf = a.status->overflow, c = a.cnt[s], off = a.soff[s];
  const float4* src = reinterpret_cast<const float4*>(raw + s * kNF);
  float4 v0 = src[0], v1 = src[1];
  const float4 v2 = src[2];
  // (an empty use before the branch, or the compiler sinks the last two
  // loads past it and waits for the count first)
  asm volatile("" ::"v"(ovf), "v"(off), "v"(v0.x), "v"(v0.y), "v"(v0.z), "v"(v0.w), "v"(v1.x), "v"(v1.y), "v"(v1.z),
               "v"(v1.w), "v"(v2.x), "v"(v2.y), "v"(v2.z));
  if (ovf || c == 0) {
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    out[0] = z; out[1] = z; out[2] = z; out[3] = z;
    return;
  }
  float acc[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k] = 0.0f;
  gather_splat_sums(a, off, c, acc);
  splat_adjoint(a, F, b, n, v0, v1, v2, acc, draw);
}

// ---------------------------------------------------------------- colour initialisation (Eq. 3)
// draw_i / draw_1: the colour adjoint of the last render under the target
// images and under all-ones images, i.e. per (frame, Gaussian) the sums of
// w_p I_p and of w_p over the pixels (w_p the Gaussian's compositing weight).
// A thread per Gaussian: if not yet initialised, the first frame whose
// weight exceeds delta sets the base colour to their ratio.
__global__ __launch_bounds__(256) void color_init_apply_kernel(const float* __restrict__ draw_i,
                                                               const float* __restrict__ draw_1, int B, int64_t N,
                                                               float delta, float* __restrict__ bases,
                                                               uint8_t* __restrict__ done) {
  const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (n >= N || done[n]) return;
  for (int b = 0; b < B; ++b) {
    const int64_t r = ((int64_t)b * N + n) * kNF;
    const float w = draw_1[r + 11];
    if (w > delta) {
      bases[n * kNF + 11] = draw_i[r + 11] / w;
      bases[n * kNF + 12] = draw_i[r + 12] / w;
      bases[n * kNF + 13] = draw_i[r + 13] / w;
      done[n] = 1;
      return;
    }
  }
}

void launch_color_init_apply(const float* draw_i, const float* draw_1, int B, int64_t N, float delta, float* bases,
                             uint8_t* done, hipStream_t s) {
  if (N == 0) return;
  hipLaunchKernelGGL(color_init_apply_kernel, dim3(div_up(N, 256)), dim3(256), 0, s, draw_i, draw_1, B, N, delta,
                     bases, done);
}

void launch_gather_bwd(const PassArgs& a, const float* raw, float* draw, int64_t max_frame_splats, hipStream_t s) {
  if (a.n_splats == 0 || max_frame_splats == 0) return;
  if (a.n_splats < kTwoPassSplats || draw == raw) {
    hipLaunchKernelGGL(gather_adjoint_kernel, dim3(div_up(max_frame_splats, kAdjThreads), a.B), dim3(kAdjThreads), 0, s,
                       a, raw, draw);
    return;
  }
  const dim3 grid(div_up(max_frame_splats, kGatherThreads), a.B);
  hipLaunchKernelGGL(gather_sums_kernel, grid, dim3(kGatherThreads), 0, s, a, draw);
  hipLaunchKernelGGL(proj_adjoint_kernel, grid, dim3(kAdjThreads), 0, s, a, raw, draw);
}

// ---------------------------------------------------------------- loss
// kind 1: mean |x - y| (Sec. 3.2 L1 colour loss), kind 2: mean (x - y)^2.
// Per-block float64 partial sums, then one block sums them in order.
constexpr int kLossThreads = 256;
constexpr int kLossPerBlock = kLossThreads * 16;

__global__ __launch_bounds__(kLossThreads) void loss_kernel(const float* __restrict__ x, const float* __restrict__ y,
                                                             int64_t n, int kind, float* __restrict__ dx,
                                                             double* __restrict__ partials,
                                                             const StatusDev* status) {
  __shared__ double sm[kLossThreads];
  const int64_t base = (int64_t)blockIdx.x * kLossPerBlock;
  const float inv = 1.0f / (float)n;
  // loads issued unconditionally (index clamped into range, n >= 1), then masked
  float xv[16], yv[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int64_t k = min(base + (int64_t)i * kLossThreads + threadIdx.x, n - 1);
    xv[i] = x[k];
    yv[i] = y[k];
  }
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int64_t k = base + (int64_t)i * kLossThreads + threadIdx.x;
    if (k < n) {
      const float d = xv[i] - yv[i];
      if (kind == 1) {
        s += fabs((double)d);
        dx[k] = (d > 0.0f ? inv : (d < 0.0f ? -inv : 0.0f));
      } else {
        s += (double)d * (double)d;
        dx[k] = 2.0f * d * inv;
      }
    }
  }
  sm[threadIdx.x] = s;
  __syncthreads();
  for (int w = kLossThreads / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) sm[threadIdx.x] += sm[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partials[blockIdx.x] = sm[0];
  (void)status;
}

// Thread t adds partials t, t + 256, ... in order (16 loads in flight at a
// time; a missing one adds 0), then a fixed tree over the threads.
__global__ void loss_final_kernel(const double* __restrict__ partials, int nb, int64_t n, StatusDev* status) {
  __shared__ double sm[256];
  double s = 0.0;
  for (int i0 = threadIdx.x; i0 < nb; i0 += 16 * 256) {
    double v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int i = i0 + j * 256;
      v[j] = i < nb ? partials[i] : 0.0;
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) s += v[j];
  }
  sm[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) sm[threadIdx.x] += sm[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) status->loss = (float)(sm[0] / (double)n);
}

int64_t loss_partials(int64_t n_floats) { return div_up(n_floats, kLossPerBlock); }

void launch_loss(const PassArgs& a, const float* images, const float* targets, int kind, float* dimages,
                 float* partials, int64_t n_partials, hipStream_t s) {
  const int64_t n = a.n_pixels * 3;
  if (n == 0) return;
  const int nb = div_up(n, kLossPerBlock);
  (void)n_partials;
  double* part = reinterpret_cast<double*>(partials);
  hipLaunchKernelGGL(loss_kernel, dim3(nb), dim3(kLossThreads), 0, s, images, targets, n, kind, dimages, part,
                     a.status);
  hipLaunchKernelGGL(loss_final_kernel, dim3(1), dim3(256), 0, s, part, nb, n, a.status);
}

}  // namespace gbr
