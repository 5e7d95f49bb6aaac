// Device kernels of the differentiable soft-argmin head (gfx950, wave64).
//
// The head keeps the cost and the cross-based aggregation of the paper
// (Eq. 3-5, 7-8) in floating point so that the disparity is a smooth
// function of the images and of the two cost weights; the census strings
// and the cross arms (Sec. III-B, III-C) are the integer path's, taken of the
// quantised images and frozen.
//
//   forward   k_soft_prep   RGB float -> float half image, and the uint8 half
//                           image of the quantised RGB (for k_feat)
//             k_feat        census and arms (shared with the integer path),
//                           and the padded pixel planes {float half image, census}
//             k_soft_size   1 / |S(x,y)|, the cross-region pixel count
//             k_soft_agg    cost C = (1 - e^{-255|dI|/lambda_AD}) +
//                           (1 - e^{-H/lambda_census}), CA over the cross
//                           region, and the softmax sums over a d-chunk
//             k_soft_merge  d_hat = sum d e_d / sum e_d, log2 sum e_d
//             (with the weights saved, k_soft_agg also writes every e_d)
//   backward  k_soft_bprep  per-pixel constants of dL/dCA
//             k_soft_agg    the aggregate again, where the forward saved neither
//                           it nor the weights
//             k_soft_tcolw  dL/dCA from either, and the transposed vertical
//                           window sums (integer difference arrays over bands
//                           of output rows, LDS atomics)
//             k_soft_tr     transposed horizontal window sums back to dL/dC
//                           then dC/d(dI), dC/d(lambda) per
//                           pixel, summed over the slab into the half-image
//                           gradients
//             k_soft_gright dL/d(right half image) from the strips' partials
//             k_soft_gfull  transposed downscale and gray: dL/d(RGB)
//             k_soft_lam    fixed-order sum of the lambda partials
//   loss      k_l1_*        mean |2 d_hat - GT(2x,2y)| over non-occluded
//                           pixels, per pair, averaged over the batch
//
// Aggregation runs on costs in fixed point (C * 2^k rounded, k chosen per
// plan so that every cross-region sum stays below 2^31): the row and column
// prefix sums then wrap modulo 2^32 and every window difference is the exact
// sum of the rounded costs, whatever the prefix magnitude.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hip.h"

namespace stereo_dev {
// Internal linkage: each source of the library that launches a kernel
// carries its own copy (no relocatable device code).
namespace {

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// ----------------------------------------------------------- k_soft_prep
// One thread per half-res pixel of one image (img = 2 pair + {0 left, 1 right}).
// Float path: gray = (77 R + 150 G + 29 B) / 256, half = mean of the 3x3 block
// at (2x, 2y), borders clamped.  Integer path: each channel quantised to
// floor(255 v + 1/2) in float32 (product and sum rounded separately), clamped
// to 0..255, then the integer gray and (sum + 4) / 9 as in k_prep.
// The workgroup's 64 x 4 half-res pixels cover 9 x 130 full-res pixels
// (rows 2 y0 - 1 .. 2 y0 + 7, columns 2 x0 - 1 .. 2 x0 + 128, clamped): each
// of them is loaded once (coalesced 12-byte loads, all five of a thread
// issued together) and its two grays go to LDS; each half-res pixel then sums
// its block there in the order (row, column).
// grid: (ceil(X/64), ceil(Y/4), 2n), block (64, 4).
constexpr int kPrepTW = 130, kPrepTH = 9, kPrepTN = kPrepTW * kPrepTH;
constexpr int kPrepLoads = (kPrepTN + 255) / 256;

__global__ void __launch_bounds__(256) k_soft_prep(const float* __restrict__ left,
                                                   const float* __restrict__ right, int W, int H,
                                                   int X, int Y, float* __restrict__ half_f,
                                                   uint8_t* __restrict__ half_u8) {
  __shared__ float s_f[kPrepTH][kPrepTW];
  __shared__ int s_i[kPrepTH][kPrepTW];
  const int t = threadIdx.y * 64 + threadIdx.x;
  const int x0 = blockIdx.x * 64, y0 = blockIdx.y * 4, img = blockIdx.z;
  const float* rgb = ((img & 1) ? right : left) + (size_t)(img >> 1) * H * W * 3;
  float pr[kPrepLoads][3];
  int ti[kPrepLoads];
#pragma unroll
  for (int k = 0; k < kPrepLoads; ++k) {
    ti[k] = min(t + 256 * k, kPrepTN - 1);  // past the tile: repeats its last pixel
    const int r = ti[k] / kPrepTW, c = ti[k] - r * kPrepTW;
    const float* p = rgb + ((size_t)clampi(2 * y0 - 1 + r, 0, H - 1) * W +
                            clampi(2 * x0 - 1 + c, 0, W - 1)) * 3;
    pr[k][0] = p[0];
    pr[k][1] = p[1];
    pr[k][2] = p[2];
  }
#pragma unroll
  for (int k = 0; k < kPrepLoads; ++k) {
    const float r = pr[k][0], g = pr[k][1], b = pr[k][2];
    int q[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float v = floorf(__fadd_rn(__fmul_rn(255.f, pr[k][c]), 0.5f));
      q[c] = (int)fminf(fmaxf(v, 0.f), 255.f);
    }
    const int row = ti[k] / kPrepTW, col = ti[k] - row * kPrepTW;
    s_f[row][col] = (77.f * r + 150.f * g + 29.f * b) * (1.f / 256.f);
    s_i[row][col] = (77 * q[0] + 150 * q[1] + 29 * q[2] + 128) >> 8;
  }
  __syncthreads();
  const int lx = threadIdx.x, ly = threadIdx.y, x = x0 + lx, y = y0 + ly;
  if (x >= X || y >= Y) return;
  float sf = 0.f;
  int si = 0;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      sf += s_f[2 * ly + j][2 * lx + i];
      si += s_i[2 * ly + j][2 * lx + i];
    }
  }
  const size_t o = (size_t)img * X * Y + (size_t)y * X + x;
  half_f[o] = sf * (1.f / 9.f);
  half_u8[o] = (uint8_t)((si + 4) / 9);
}

// ----------------------------------------------------------- k_soft_size
// 1 / |S(x,y)| for the left image of each pair: |S| = sum over s in
// [-M, N] of (m + n + 1) at (x, y + s) (Eq. 7-8 applied to a unit cost).
// One workgroup = 64 columns x kSizeRows rows.  The row supports m + n + 1
// (at most 63: arm_x <= 31) of the tile rows y0 - arm_y + r, r < 144,
// are summed down each column: wave w loads the rows 9 w .. 9 w + 8 together
// (rows clamped into the image; a window never reaches a clamped row) and
// keeps their running sum, the waves' totals give each wave its offset, and
// the exclusive column prefix P (16 bits: at most 144 x 63) goes to LDS, so
// a window is P[t + N + 1] - P[t - M], t the tile row of y.
// grid: (ceil(X/64), ceil(Y/kSizeRows), n), block (64, kSizeRows).
constexpr int kSizeRows = 16, kSizeMaxArm = 63, kSizeSeg = 9;
static_assert(kSizeRows * kSizeSeg >= kSizeRows + 2 * kSizeMaxArm, "tile rows");

__global__ void __launch_bounds__(64 * kSizeRows) k_soft_size(const uint32_t* __restrict__ arms,
                                                             int X, int Y, int XA, int arm_y,
                                                             float* __restrict__ inv_size) {
  __shared__ uint16_t s_p[kSizeRows * kSizeSeg + 1][64];
  __shared__ uint16_t s_t[kSizeRows][64];
  const int x0 = blockIdx.x * 64, y0 = blockIdx.y * kSizeRows, pair = blockIdx.z;
  const int lx = threadIdx.x, ly = threadIdx.y, x = x0 + lx;  // x < XA: zero padding past X
  const uint32_t* a = arms + (size_t)(2 * pair) * Y * XA;
  const int y = y0 + ly;
  uint32_t c = a[(size_t)min(y, Y - 1) * XA + x];
  uint32_t v[kSizeSeg];
#pragma unroll
  for (int k = 0; k < kSizeSeg; ++k)
    v[k] = a[(size_t)clampi(y0 - arm_y + kSizeSeg * ly + k, 0, Y - 1) * XA + x];
  // the pixel's own arms stay loaded with the tile's (not after the barriers)
  __asm__ volatile("" : "+v"(c));
  uint32_t run = 0, loc[kSizeSeg];
#pragma unroll
  for (int k = 0; k < kSizeSeg; ++k) {
    run += (v[k] & 255u) + ((v[k] >> 8) & 255u) + 1u;
    loc[k] = run;
  }
  s_t[ly][lx] = (uint16_t)run;
  __syncthreads();
  uint32_t off = 0;
#pragma unroll
  for (int l = 0; l < kSizeRows; ++l) off += l < ly ? (uint32_t)s_t[l][lx] : 0u;
#pragma unroll
  for (int k = 0; k < kSizeSeg; ++k) s_p[kSizeSeg * ly + k + 1][lx] = (uint16_t)(off + loc[k]);
  if (ly == 0) s_p[0][lx] = 0;
  __syncthreads();
  if (x >= X || y >= Y) return;
  const int M = (c >> 16) & 255, N = c >> 24, t = ly + arm_y;  // tile row of y
  const int sum = (int)s_p[t + N + 1][lx] - (int)s_p[t - M][lx];
  inv_size[(size_t)pair * X * Y + (size_t)y * X + x] = 1.f / (float)sum;
}

// ------------------------------------------------------------ k_soft_agg
struct SoftArgs {
  const uint2* sp;          // [2n][Y][XS] padded pixel planes
  const uint32_t* arms;     // [2n][Y][XA]
  const float* lam;         // device [2]: lambda_AD, lambda_census
  const float* inv_size;    // [n][Y][X]
  float2* part;             // [n][nchunk][Y][X] {sum e, sum d e}, or NULL
  float* wts;               // [..][n][Y][XW] e_d, plane 0 = disparity wlo, or NULL
  float* wts2;              // the same, for the disparities from wsplit on
  int ca;                   // wts and wts2 take CA in place of e_d
  int X, Y, XS, pads, XA, XW, arm_x, arm_y;
  int nbands, dlo, dhi, wlo, wsplit, nstrips, ngroups, npair;
  int csize, nchunk;        // d-chunk size; chunks = ceil((dhi - dlo) / csize), the last the remainder
  float fx;                 // fixed-point scale 2^k of the costs
  float zc;                 // 2^-k log2(e) / tau: CA_int * inv_size * zc = mean / tau in log2 units
  uint32_t sp_bytes, arms_bytes;
};

// Blocks are dealt to the 8 XCDs in turn (block id mod 8): block `id` of
// `count` takes item (id mod 8) * ceil(count / 8) + id / 8, so that
// neighbouring items, which read the same rows, run on one XCD and find each
// other's halo in its L2.  The launch has 8 * ceil(count / 8) blocks; the items
// past the last one are none.
__device__ __forceinline__ int xcd_item(int id, int count) {
  return (id & (kXcds - 1)) * ((count + kXcds - 1) / kXcds) + id / kXcds;
}

constexpr int kXcdQueues = 4;  // workgroup dispatch queues per XCD (position mod 4)

// Position j of an XCD's workgroup sequence -> (local group, d-chunk), for
// nloc groups of nchunk chunks each, nfull of them full-size and, when
// nchunk > nfull, one shorter remainder chunk.  Workgroup j waits in the
// XCD's dispatch queue j % kXcdQueues for a CU of that queue.  The remainder
// chunks take the last positions of one queue, T-1, T-1-4, ... (T = nloc *
// nchunk), so that the workgroups past the first round follow short ones
// there; where that does not fit they simply come last.
__device__ __forceinline__ void chunk_at(int j, int nloc, int nfull, int nchunk, int& local,
                                         int& chunk) {
  const int T = nloc * nchunk;
  if (nchunk == nfull) {
    local = j / nfull;
    chunk = j - local * nfull;
  } else if (kXcdQueues * (nloc - 1) > T - 1) {
    local = j < nloc * nfull ? j / nfull : j - nloc * nfull;
    chunk = j < nloc * nfull ? j - local * nfull : nfull;
  } else {
    const int q = T - 1 - j;  // remainder chunks at q = 0, 4, ..., 4 (nloc - 1)
    if (q % kXcdQueues == 0 && q / kXcdQueues < nloc) {
      local = nloc - 1 - q / kXcdQueues;
      chunk = nfull;
    } else {
      const int i = j - max(0, nloc - (q / kXcdQueues + 1));  // full chunks before j
      local = i / nfull;
      chunk = i - local * nfull;
    }
  }
}

// LDS bytes of k_soft_agg beside the plane: row buffers and the census table.
constexpr int kAggRowBytes = kWaves * 128 * 4 + 32;
// Most rows of the plane (the zero row beside them).
constexpr int kAggRows = (kLdsBytes - kAggRowBytes) / 256 - 1;

// One workgroup = one 64-column strip x one band of rows x one pair x one
// chunk of disparities; 16 waves, the layout of k_match with one base (row
// pass with a DPP wave scan, column sums in registers until the segment offsets
// are known, plane, window differences).  The cost of a column c at disparity d:
//   c - d >= 0: C = (2 - exp(-255 |L(c) - R(c-d)| / lambda_AD)) - exp(-H / lambda_census)
//   c - d <  0: C = 2
// taken to fixed point.  Output rows of a thread: o0 + wave + 16 k, k < KMAX.
// e = 2^{-CA mean / tau (log2 units)}; its sums e and d e per output pixel over
// the chunk go to part, every e to wts (each where given).
// A wave's segment has at most SEG rows (their sums stay in registers).
// The row sums are in registers, with two barriers a disparity (one for the
// segments' totals, one for the plane) in place of three and a second pass over
// the plane.  4 pairs of 718x496, 73 disparities: 440 us before, 366 us now (24 of
// it from weight rows of whole 128-byte lines).  Counters there: vector
// instructions issue in 58% of the SIMDs' cycles at most (four clocks each; an
// exponential 8, some of the others 2), the LDS is active in 22%, a wave waits in
// 44% of its cycles: with four waves a SIMD it is the waiting that is left.
// grid: ceil(groups / 8) * 8 * nchunk workgroups (1-D), block 1024.
template <int KMAX, int SEG>
__global__ void __launch_bounds__(kThreads) k_soft_agg(SoftArgs a) {
  extern __shared__ __align__(16) uint8_t s_agg[];
  auto s_row = reinterpret_cast<uint32_t(*)[128]>(s_agg);
  float* s_ex = reinterpret_cast<float*>(s_agg + kWaves * 128 * 4);
  const uint32_t ex0 = lds_addr(s_ex);
  uint32_t* s_plane = reinterpret_cast<uint32_t*>(s_agg + kAggRowBytes);  // row 0 = zeros

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int X = a.X, Y = a.Y;
  const int wg = blockIdx.x, xcd = wg & (kXcds - 1), j = wg / kXcds;
  int local, chunk;
  chunk_at(j, (a.ngroups + kXcds - 1) / kXcds, (a.dhi - a.dlo) / a.csize, a.nchunk, local, chunk);
  int group = local * kXcds + xcd;
  if (group >= a.ngroups) return;
  const int strip = group % a.nstrips;
  group /= a.nstrips;
  const int band = group % a.nbands;
  const int pair = group / a.nbands;
  const int x0 = strip * kTX;
  const int ob = (Y + a.nbands - 1) / a.nbands;
  const int y0 = band * ob, y1 = min(Y, y0 + ob);
  const int ya = max(0, y0 - a.arm_y), yb = min(Y, y1 + a.arm_y);
  const int nb = yb - ya, o0 = y0 - ya, o1 = y1 - ya;
  const int d0 = a.dlo + chunk * a.csize, d1 = min(a.dhi, d0 + a.csize);
  const int hx = (a.arm_x + 2) & ~1, e0 = x0 - hx;
  const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(a.sp, a.sp_bytes);
  const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(a.arms, a.arms_bytes);
  const uint32_t img_l = (uint32_t)(2 * pair);
  const uint32_t sprow = (uint32_t)a.XS * 8u, armrow = (uint32_t)a.XA * 4u;
  const float lam_ad = a.lam[0], lam_c = a.lam[1];
  // e^{-255 |dI| / lambda_AD} = 2^{-|dI| k2}
  const float k2 = 255.f * 1.4426950408889634f / lam_ad;
  if (t < 8) s_ex[t] = t < 7 ? fast_exp2(-(float)t * 1.4426950408889634f / lam_c) : 0.f;
  if (t < 64) s_plane[t] = 0u;

  const int x = x0 + lane;
  // rows of the band in segments of whole row pairs (the row pass takes its
  // rows in pairs), one per wave in order, the pairs split as evenly as
  // possible: the waves of each SIMD (wave mod 4) then share the rows evenly
  const int nbat = (nb + 1) / 2, bq = nbat / kWaves, br = nbat % kWaves;
  const int r0 = min(nb, 2 * (wave * bq + min(wave, br)));
  const int r1 = min(nb, r0 + 2 * (bq + (wave < br)));

  static_assert(KMAX % 2 == 0 && SEG % kRowBatch == 0, "rows go in pairs");
  uint32_t marm[KMAX / 2];
  float se[KMAX], sde[KMAX], isz[KMAX];
#pragma unroll
  for (int k = 0; k < KMAX; ++k) {
    const int r = o0 + wave + k * kWaves;
    const bool in = x < X && r < o1;
    // no branch around the load (rows past the band read its last row and are
    // masked by a wave-uniform select; columns past X read the zero padding)
    const uint32_t v = a.arms[((size_t)img_l * Y + ya + min(r, o1 - 1)) * a.XA + x] >> 16;
    const uint32_t mn = r < o1 ? v : 0u;
    if (k & 1) marm[k / 2] |= mn << 16;
    else marm[k / 2] = mn;
    se[k] = 0.f;
    sde[k] = 0.f;
    // unconditional load at a clamped pixel, then a select (as above)
    const float iv = a.inv_size[((size_t)pair * Y + ya + min(r, o1 - 1)) * X + min(x, X - 1)];
    isz[k] = in ? iv * a.zc : 0.f;
  }
  const float fx = a.fx;
  __syncthreads();

  // cost of a pair of pixels in fixed point (the columns without a match apart)
  auto cost = [&](uint32_t lv, uint32_t lc, uint32_t rv, uint32_t rc) -> uint32_t {
    const float di = fabsf(__uint_as_float(lv) - __uint_as_float(rv));
    const float ex = __uint_as_float(lds_read(__builtin_popcount(lc ^ rc) + ex0));
    const float cf = (2.f - fast_exp2(-di * k2)) - ex;
    return (uint32_t)(cf * fx + 0.5f);
  };
  const uint32_t cout = (uint32_t)(2.f * fx + 0.5f);

  for (int d = d0; d < d1; ++d) {
    // per-lane addresses formed anew for each disparity (see k_match)
    uint32_t ln = (uint32_t)lane;
    __asm__ volatile("" : "+v"(ln));
    // byte offset of this lane's first column pair in a padded row
    const uint32_t vb = (uint32_t)(a.pads + e0) * 8u + ln * 16u;
    const uint32_t vo = vb - (uint32_t)(d * 8), vx = ((uint32_t)x0 + ln) * 4u;
    uint32_t wrow = lds_addr(s_row[wave]) + ln * 8u;
    uint32_t ent = lds_addr(s_row[wave]) + (uint32_t)hx * 4u + ln * 4u;
    __asm__ volatile("" : "+v"(ent), "+v"(wrow));
    const bool edge = e0 < d;  // the strip holds columns without a match (wave-uniform)
    const bool out0 = e0 + 2 * (int)ln < d, out1 = e0 + 2 * (int)ln + 1 < d;
    // scalar byte offsets of the row to load next (rows past the segment's end
    // are the next one's, or the band's last row again)
    const uint32_t yl = img_l * (uint32_t)Y + (uint32_t)(ya + r0);
    uint32_t sl = yl * sprow, sa = yl * armrow;
    const uint32_t other = (uint32_t)Y * sprow;  // the right image's rows follow the left one's
    int rn = r0;
    __asm__ volatile("" : "+s"(sl), "+s"(sa), "+s"(rn));
    struct RowIn { u32x4 L, R; };
    auto load_batch = [&](RowIn (&in)[kRowBatch], uint32_t (&am)[kRowBatch]) {
#pragma unroll
      for (int i = 0; i < kRowBatch; ++i) {
        in[i].L = __builtin_amdgcn_raw_buffer_load_b128(rs, vb, sl, 0);
        in[i].R = __builtin_amdgcn_raw_buffer_load_b128(rs, vo, sl + other, 0);
        am[i] = __builtin_amdgcn_raw_buffer_load_b32(ra, vx, sa, 0);
        ++rn;
        sl += rn < nb ? sprow : 0u;
        sa += rn < nb ? armrow : 0u;
      }
    };
    uint32_t run[SEG], tot = 0;
    RowIn in[kRowBatch];
    uint32_t am[2][kRowBatch];
    if (r0 < r1) load_batch(in, am[0]);
    static_while<SEG / kRowBatch>([&](auto Q) {
      constexpr int q = decltype(Q)::value;
      const int r = r0 + q * kRowBatch;
      if (r >= r1) return false;
      // a falling priority keeps the waves of a SIMD abreast (see k_match)
      if constexpr (q == 0) __builtin_amdgcn_s_setprio(2);
      if constexpr (q == SEG / 6) __builtin_amdgcn_s_setprio(1);
      if constexpr (q == SEG / 3) __builtin_amdgcn_s_setprio(0);
      uint32_t c1[kRowBatch], pr[kRowBatch];
#pragma unroll
      for (int i = 0; i < kRowBatch; ++i) {
        pr[i] = cost(in[i].L.x, in[i].L.y, in[i].R.x, in[i].R.y);
        c1[i] = cost(in[i].L.z, in[i].L.w, in[i].R.z, in[i].R.w);
      }
      // the pixels are used up: the next batch's take their registers
      // (unconditional, so that the waits do not depend on a branch)
      load_batch(in, am[(q + 1) & 1]);
      if (edge) {
#pragma unroll
        for (int i = 0; i < kRowBatch; ++i) {
          pr[i] = out0 ? cout : pr[i];
          c1[i] = out1 ? cout : c1[i];
        }
      }
#pragma unroll
      for (int i = 0; i < kRowBatch; ++i) pr[i] += c1[i];
      wave_scan_incl_n(pr);
#pragma unroll
      for (int i = 0; i < kRowBatch; ++i) {
        lds_write2(wrow, pr[i] - c1[i], pr[i]);
        WAVE_LDS_ORDER();
        const uint32_t m = am[q & 1][i] & 255u, n = (am[q & 1][i] >> 8) & 255u;
        tot += lds_read(ent + n * 4u) - lds_read(ent - m * 4u - 4u);
        WAVE_LDS_ORDER();
        run[q * kRowBatch + i] = tot;
      }
      return true;
    });
    // the wave's total goes to its own row buffer (see k_match)
    s_row[wave][ln] = tot;
    __syncthreads();
    __builtin_amdgcn_s_setprio(3);
    uint32_t off = 0;
    int s0 = 0;
#pragma unroll
    for (int n = kWaves / 2; n > 0; n >>= 1)
      if (wave & n) {
        uint32_t v[8];
#pragma unroll
        for (int s = 0; s < n; ++s) v[s] = s_row[s0 + s][ln];
#pragma unroll
        for (int s = 0; s < n; ++s) off += v[s];
        s0 += n;
      }
    uint32_t* pw = s_plane + (r0 + 1) * 64 + ln;
    int nrows = r1 - r0;
    __asm__ volatile("" : "+s"(nrows));
    static_while<SEG>([&](auto K) {
      constexpr int k = decltype(K)::value;
      if (k >= nrows) return false;
      pw[k * 64] = run[k] + off;
      return true;
    });
    __syncthreads();
    // window differences of this wave's output rows, two slot pairs at a time,
    // the reads of the next ones in flight
    const float fd = (float)d;
    const uint32_t fin = lds_addr(s_plane) + (uint32_t)((o0 + wave + 1) * 64) * 4u + ln * 4u;
    uint32_t kpermM = 0x020c000cu;
    __asm__ volatile("" : "+v"(kpermM));
    // rows of the weight plane of d
    float* wd = a.wts ? (d < a.wsplit ? a.wts : a.wts2) +
                            (((size_t)(d - a.wlo) * a.npair + pair) * Y + ya + o0 + wave) * a.XW + x0
                      : nullptr;
    if (x < X) {
      uint32_t wh[2][kWinGroup][2], wl[2][kWinGroup][2];
      auto window_reads = [&](auto G) {
        constexpr int g = decltype(G)::value;
#pragma unroll
        for (int i = 0; i < kWinGroup; ++i) {
          const int jp = g * kWinGroup + i;
          if (jp >= KMAX / 2) continue;
          uint32_t nw, mw;  // N and M of two rows in bits 8..15 of the halves: byte offsets
          __asm__ volatile("v_and_b32 %0, 0xff00ff00, %1" : "=v"(nw) : "v"(marm[jp]));
          __asm__ volatile("v_perm_b32 %0, 0, %1, %2" : "=v"(mw) : "v"(marm[jp]), "v"(kpermM));
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const uint32_t kb = (uint32_t)((2 * jp + e) * kWaves * 64 * 4);
            wh[g & 1][i][e] = lds_read((fin + (e ? nw >> 16 : nw & 0xffffu)) + kb);
            wl[g & 1][i][e] = lds_read((fin - (e ? mw >> 16 : mw & 0xffffu)) + kb - 256u);
          }
        }
      };
      constexpr int kGroups = (KMAX / 2 + kWinGroup - 1) / kWinGroup;
      window_reads(std::integral_constant<int, 0>{});
      static_for<kGroups>([&](auto G) {
        constexpr int g = decltype(G)::value;
        if constexpr (g + 1 < kGroups) window_reads(std::integral_constant<int, g + 1>{});
        WAVE_LDS_ORDER();  // those reads are issued before this group is waited for
#pragma unroll
        for (int i = 0; i < kWinGroup; ++i)
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int k = 2 * (g * kWinGroup + i) + e;
            if (k >= KMAX) continue;
            const uint32_t ca = wh[g & 1][i][e] - wl[g & 1][i][e];
            const float ev = fast_exp2(-(float)ca * isz[k]);
            se[k] += ev;
            sde[k] += fd * ev;
            if (wd && o0 + wave + k * kWaves < o1)
              wd[(size_t)k * kWaves * a.XW + ln] = a.ca ? (float)ca : ev;
          }
      });
    }
  }

  if (a.part && x < X) {
    float2* out = a.part + (size_t)(pair * a.nchunk + chunk) * X * Y;
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
      const int r = o0 + wave + k * kWaves;
      if (r < o1) out[(size_t)(ya + r) * X + x] = make_float2(se[k], sde[k]);
    }
  }
}

// ---------------------------------------------------------- k_soft_merge
// Sums the chunk partials in chunk order: d_hat = sum d e / sum e and
// lse2 = log2 sum e.  grid: (ceil(X*Y/256), n), block 256.
__global__ void __launch_bounds__(256) k_soft_merge(const float2* __restrict__ part, int nchunk,
                                                    int npix, float* __restrict__ dhat,
                                                    float* __restrict__ lse2) {
  const int i = blockIdx.x * 256 + threadIdx.x, pair = blockIdx.y;
  if (i >= npix) return;
  const float2* p = part + (size_t)pair * nchunk * npix + i;
  float s = 0.f, sd = 0.f;
  // loads in groups of 8 in flight, sums in chunk order
  for (int c0 = 0; c0 < nchunk; c0 += 8) {
    float2 v[8];
#pragma unroll
    for (int g = 0; g < 8; ++g) v[g] = p[(size_t)min(c0 + g, nchunk - 1) * npix];
#pragma unroll
    for (int g = 0; g < 8; ++g)
      if (c0 + g < nchunk) {
        s += v[g].x;
        sd += v[g].y;
      }
  }
  dhat[(size_t)pair * npix + i] = sd / s;
  lse2[(size_t)pair * npix + i] = __log2f(s);
}

// ---------------------------------------------------------- k_soft_bprep
// Per-pixel constants of the adjoint: w = zc / |S| (log2-unit mean per
// fixed-point aggregate), lse2, d_hat and A = -g_dhat / (tau |S|), so that
// dL/dCA(d) = A p_d (d - d_hat) with p_d = 2^{-CA w - lse2}.
// grid: (ceil(X*Y/256), n), block 256.
__global__ void __launch_bounds__(256) k_soft_bprep(const float* __restrict__ inv_size,
                                                    const float* __restrict__ lse2,
                                                    const float* __restrict__ dhat,
                                                    const float* __restrict__ g_dhat, int npix,
                                                    float zc, float inv_tau,
                                                    float4* __restrict__ pc) {
  const int i = blockIdx.x * 256 + threadIdx.x, pair = blockIdx.y;
  if (i >= npix) return;
  const size_t o = (size_t)pair * npix + i;
  const float is = inv_size[o];
  pc[o] = make_float4(is * zc, lse2[o], dhat[o], -g_dhat[o] * is * inv_tau);
}

// ------------------------------------------------------------ k_soft_tcolw
// Transpose of the vertical window sum (Eq. 8) with dL/dCA formed on the fly
// from the softmax weights e_d = 2^{-CA(d) w} of the forward:
//   dL/dCA(x,y,d) = A p_d (d - d_hat),  p_d = e_d 2^{-lse2}
//   CA(x,y) = sum_{s=-M(x,y)}^{N(x,y)} CA_x(x,y+s)  gives
//   dL/dCA_x(x,y') = sum of dL/dCA(x,y) over the y whose window holds y'
// (A, lse2 and d_hat from k_soft_bprep's constants).  A block takes a
// 64-column strip, a band of B output rows (tcol_band) and a range of
// disparities of one pair.  The band's rows y' in [Y0, Y0 + B) can only be
// reached from sources y in [Y0 - arm_y, Y0 + B + arm_y); each source's window,
// clipped to the band, becomes a difference array (+g at its first row, -g
// after its last) and a prefix down the column gives the sums.  The difference
// array is integer fixed point with a per-column scale 2^k, k = 23 - e where
// 2^(e-1) <= the column's largest |g| < 2^e: each term is at most 2^23 and a sum
// of at most 2 arm_y + 1 <= 127 terms at most 2^30, so LDS integer atomics give
// exact sums in any order (the result does not depend on scheduling) and each
// term is rounded to 2^(e-24), the float resolution of the column's largest
// value.  Thread (wave w, lane l) holds, over the range, the constants of
// column x0 + l at the source rows Y0 - arm_y + w + 16 i and the difference rows
// their windows start and end at.
// A disparity passes through four stages: A its terms and the column's largest
// (LDS atomic maximum), B the scatter, C each wave's prefix over its output rows,
// D the offsets of the waves above and the stores.  Between two barriers every
// wave does B of one disparity, D and C of the two before it and A of the next,
// on three difference arrays in turn: one barrier a disparity instead of three.
// Close to the memory rate (0.97 GB at 4.4 TB/s, halo rows included, where a copy
// reaches 5.2 to 5.8); the LDS, with 24 atomics a thread and disparity, is active
// in 21% of the cycles and vector instructions issue in 46% at most.  4 pairs of
// 718x496, 73 disparities: 264 us with three barriers, 246 with one, 217 with rows
// of whole 128-byte lines.  CA = true takes saved CA: at 4 pairs of 960x540 and
// 128 disparities, where the backward computed CA again and summed its planes one
// by one, forward and backward together took 3.60 ms and take 2.14 (this kernel
// 0.60).
// grid: strips * bands * n * ndg rounded up to 8 (1-D, xcd_item), block 1024;
// disparity group g of ndg covers [dlo + g nd / ndg, dlo + (g + 1) nd / ndg).
constexpr int kTcolBand = 128;
__host__ __device__ constexpr int tcol_band(int arm_y) { return arm_y <= 31 ? kTcolBand : kTcolBand / 2; }
constexpr int kTcwWaves = 16;
constexpr int kTcwSrc = 12;  // source rows per thread: B + 2 arm_y <= 16 * 12
static_assert(tcol_band(31) + 2 * 31 <= kTcwWaves * kTcwSrc &&
                  tcol_band(63) + 2 * 63 <= kTcwWaves * kTcwSrc, "k_soft_tcolw source rows");

struct TcwArgs {
  const float* wts;         // [..][n][Y][XW] e_d or CA, plane 0 = disparity wlo
  const float4* pc;         // [n][Y][X] constants (k_soft_bprep)
  const uint32_t* arms;     // [2n][Y][XA]
  float* gcax;              // [nds][n][Y][XW] dL/dCA_x
  uint32_t wts_bytes;
  int X, Y, XA, XW, arm_y, npair, dlo, dhi, wlo, ndg;
};

// Exponent e with 2^(e-1) <= v < 2^e of the bits of a float v >= 0 (frexp's;
// denormals too); 0 for v = 0.
__device__ __forceinline__ int float_exp(uint32_t bits) {
  const int be = (int)(bits >> 23);
  return be > 0 ? be - 126 : (bits ? -117 - (int)__builtin_clz(bits) : 0);
}

template <bool CA>
__global__ void __launch_bounds__(64 * kTcwWaves) k_soft_tcolw(TcwArgs a) {
  constexpr int RPW = kTcolBand / kTcwWaves;  // output rows per wave, at most
  __shared__ __align__(16) int s_d[3][kTcolBand + 1][64];  // row B: ends behind the band
  __shared__ int s_tot[2][kTcwWaves][64];
  __shared__ uint32_t s_max[3][64];  // largest |g| of the column
  __shared__ float s_w[CA ? kTcwSrc : 1][64 * kTcwWaves];  // w of the sources (each thread's own)
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int X = a.X, Y = a.Y, B = tcol_band(a.arm_y);
  // the bands of a strip are neighbours (they share their halo rows)
  const int nstrips = (X + 63) / 64, nbands = (Y + B - 1) / B;
  const int item = xcd_item(blockIdx.x, nstrips * nbands * a.npair * a.ndg);
  if (item >= nstrips * nbands * a.npair * a.ndg) return;
  const int x = item / nbands % nstrips * 64 + lane, Y0 = item % nbands * B;
  const int pair = item / (nbands * nstrips) % a.npair, dg = item / (nbands * nstrips * a.npair);
  const int nd = a.dhi - a.dlo;
  const int d0 = a.dlo + dg * nd / a.ndg, n = a.dlo + (dg + 1) * nd / a.ndg - d0;
  const int Y1 = min(Y, Y0 + B);
  const bool xv = x < X;
  const int xc = min(x, X - 1);
  const size_t plane = (size_t)a.XW * Y;
  const int ys = max(0, Y0 - a.arm_y), ye = min(Y, Y1 + a.arm_y);
  // source row of slot i (wave-uniform), clamped into the sources
  auto src_row = [&](int i) { return min(ys + wave + kTcwWaves * i, ye - 1); };
  // constants of the source rows (loads at clamped rows; a row outside the
  // sources or a column past X gets A = 0, so it adds nothing; one whose window
  // misses the band counts for the scale and adds q - q to row 0)
  float cA[kTcwSrc], cS[kTcwSrc], cD[kTcwSrc];
  // byte offsets (256 a row) of the difference rows lo and hi + 1 of two
  // sources, in the 16-bit halves
  uint32_t cLo[kTcwSrc / 2], cHi[kTcwSrc / 2];
#pragma unroll
  for (int i = 0; i < kTcwSrc; ++i) {
    const int y = src_row(i);
    const float4 q = a.pc[((size_t)pair * Y + y) * X + xc];
    const uint32_t am = a.arms[((size_t)(2 * pair) * Y + y) * a.XA + xc];
    const int lo = max(y - (int)((am >> 16) & 255u), Y0), hi = min(y + (int)(am >> 24), Y1 - 1);
    cA[i] = xv && ys + wave + kTcwWaves * i < ye ? q.w : 0.f;
    cS[i] = CA ? -q.y : fast_exp2(-q.y);
    if (CA) s_w[i][t] = q.x;
    cD[i] = q.z;
    const bool in = lo <= hi;
    const uint32_t el = in ? (uint32_t)(lo - Y0) << 8 : 0u, eh = in ? (uint32_t)(hi + 1 - Y0) << 8 : 0u;
    if (i & 1) {
      cLo[i / 2] |= el << 16;
      cHi[i / 2] |= eh << 16;
    } else {
      cLo[i / 2] = el;
      cHi[i / 2] = eh;
    }
  }
  // weight loads: the lane's column in the vector offset, the row and plane
  // (wave-uniform) in the scalar one
  const __amdgpu_buffer_rsrc_t rw = buffer_rsrc(a.wts, a.wts_bytes);
  const uint32_t vcol = (uint32_t)xc * 4u;
  float w[kTcwSrc], g[kTcwSrc];
  auto load_w = [&](int k) {  // past the range: the last one again
    const uint32_t sp =
        (uint32_t)(((size_t)(d0 + min(k, n - 1) - a.wlo) * a.npair + pair) * plane * 4);
#pragma unroll
    for (int i = 0; i < kTcwSrc; ++i)
      w[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
          rw, vcol, sp + (uint32_t)src_row(i) * (uint32_t)a.XW * 4u, 0));
  };
  auto stage_a = [&](int k, uint32_t* mx) {
    const float fd = (float)(d0 + k);
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < kTcwSrc; ++i) {
      const float p = CA ? fast_exp2(fmaf(-w[i], s_w[i][t], cS[i])) : w[i] * cS[i];
      g[i] = cA[i] * p * (fd - cD[i]);
      m = fmaxf(m, fabsf(g[i]));
    }
    // the bit order of floats >= 0 is that of their values
    (void)__hip_atomic_fetch_max(mx + lane, __float_as_uint(m), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto zero = [&](int (*dst)[64]) {
    for (int i = t; i < (B + 1) * 16; i += 64 * kTcwWaves)
      reinterpret_cast<u32x4*>(&dst[0][0])[i] = u32x4{0u, 0u, 0u, 0u};
  };
  // output rows Y0 + r0 .. of this wave, and the lane's place in a row
  const int rpw = B / kTcwWaves, r0 = wave * rpw;
  const size_t dstride = (size_t)a.npair * plane;
  float* gout = a.gcax + ((size_t)(d0 - a.dlo) * a.npair + pair) * plane + (size_t)(Y0 + r0) * a.XW + x;
  if (n <= 0) return;  // block-uniform
  load_w(0);
  if (t < 192) (&s_max[0][0])[t] = 0u;
  zero(s_d[0]);
  __syncthreads();
  stage_a(0, s_max[0]);
  load_w(1);
  __syncthreads();
  int loc[RPW];
  uint32_t mC = 0, mD = 0;  // column maxima of the disparities in stages C and D
  int b0 = 0, b1 = 2, b2 = 1;  // difference arrays of stage B, C, and the one to clear
  for (int k = 0; k < n + 2; ++k) {
    uint32_t mB = 0;
    if (k < n) {  // B
      mB = s_max[b0][lane];
      const float up = mB ? ldexpf(1.f, 23 - float_exp(mB)) : 0.f;
      char* col = reinterpret_cast<char*>(&s_d[b0][0][lane]);
#pragma unroll
      for (int i = 0; i < kTcwSrc; ++i) {
        const int q = (int)rintf(g[i] * up);
        const uint32_t lo = i & 1 ? cLo[i / 2] >> 16 : cLo[i / 2] & 0xffffu;
        const uint32_t hi = i & 1 ? cHi[i / 2] >> 16 : cHi[i / 2] & 0xffffu;
        (void)__hip_atomic_fetch_add(reinterpret_cast<int*>(col + lo), q, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_WORKGROUP);
        (void)__hip_atomic_fetch_sub(reinterpret_cast<int*>(col + hi), q, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    if (k + 1 < n) {  // A of the next disparity
      stage_a(k + 1, s_max[b2]);
      load_w(k + 2);
      zero(s_d[b2]);
    }
    if (k >= 2) {  // D
      int off = 0, s0 = 0;
      // the totals above: the wave's number as 8 + 4 + 2 + 1, groups of reads
      // in flight together
#pragma unroll
      for (int m = kTcwWaves / 2; m > 0; m >>= 1)
        if (wave & m) {
          int v[8];
#pragma unroll
          for (int s = 0; s < m; ++s) v[s] = s_tot[k & 1][s0 + s][lane];
#pragma unroll
          for (int s = 0; s < m; ++s) off += v[s];
          s0 += m;
        }
      if (xv) {
        const float down = mD ? ldexpf(1.f, float_exp(mD) - 23) : 0.f;
        float* o = gout + (size_t)(k - 2) * dstride;
#pragma unroll
        for (int i = 0; i < RPW; ++i)
          if (i < rpw && Y0 + r0 + i < Y1) o[(size_t)i * a.XW] = (float)(loc[i] + off) * down;
      }
    }
    if (k >= 1 && k <= n) {  // C
      int run = 0;
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        if (i < rpw) run += s_d[b1][r0 + i][lane];
        loc[i] = run;
      }
      s_tot[(k - 1) & 1][wave][lane] = run;
      if (t < 64) s_max[b1][t] = 0u;  // for the disparity two further
    }
    mD = mC;
    mC = mB;
    const int nb = b2;
    b2 = b1;
    b1 = b0;
    b0 = nb;
    __syncthreads();
  }
}

// ------------------------------------------------------------- k_soft_tr
// Transpose of the horizontal window sum (Eq. 7), then the cost derivatives
// there, summed over a slab of disparities into the half-image gradients.
//   CA_x(x,y) = sum_{t=-m}^{n} C(x+t,y)  gives
//   dL/dC(c,y,d) = sum over the x with x - m(x) <= c <= x + n(x) of
//                  dL/dCA_x(x,y,d):
// for a row, a product of the [disparity][x] matrix with the 0/1 matrix
// [x][c] of the row's arms, which is the same for every disparity.  Then with
// dI = L(x,y) - R(x-d,y), a = 255 |dI|, E = e^{-a/lambda_AD}:
//   t = dL/dC * dC/d(dI) = dL/dC * (255 / lambda_AD) E sign(dI)
//   dL/dL(x,y)        += t       dL/dR(x-d,y) -= t
//   dL/dlambda_AD     += dL/dC * (-E a / lambda_AD^2)
//   dL/dlambda_census += dL/dC * (-e^{-H/lambda_census} H / lambda_census^2)
// for x - d >= 0 (the constant cost of x - d < 0 has no derivative).
// A wave takes 64 columns of one row.  The 0/1 matrix of the 128 source columns
// x0 - 32 .. x0 + 95 (every column whose window reaches the strip, arm_x <= 31)
// is built once, in registers, and the matrix cores form 16 disparities x 64
// columns at a time (v_mfma_i32_16x16x64_i8: four groups of 16 columns, two
// tiles of 64 sources).  The terms are integer fixed point with a scale
// 2^(23 - e) per row and disparity, 2^(e-1) <= the largest |g| of the 128
// sources < 2^e, each as three bytes: the sums of up to 63 terms stay below 2^30
// and are exact, so the only rounding is that of a term to 2^(e-24).  (The lower
// two bytes u are unsigned; the instruction's are signed, so u - 128 goes in and
// 128 times the number of a column's sources is added.  Three bf16 terms of a
// float are exact too, but the bf16 instruction's accumulation is biased:
// dL/dlambda, a sum of millions of cancelling terms, lost three digits.)
// The sums go through the wave's LDS tile, so that a lane takes the derivatives
// of one column at the disparities in order: dL/dlambda cancels so far that its
// float sums keep their digits only in a fixed order of additions.  The left
// gradient of the column stays in a register; the right one, of column x - d,
// is in the neighbouring lane at the next disparity: one lane shift, and the
// values of a disparity go to an LDS row that ends with each entry's last one,
// then to the strip's partial row, which k_soft_gright sums over the strips.
// A block takes 4 rows of a strip.
// Vector arithmetic first (about 43 instructions a column and disparity, 16 of
// them for the derivatives: issued in up to 76% of the SIMDs' cycles; three waves a
// SIMD, waiting in 40% of theirs).  4 pairs of 718x496, 73
// disparities: 242 us as a scan and scatter of difference arrays in LDS, 197 now;
// at 960x540 and 128 disparities 557 and 445.
// grid: strips * ceil(Y / 4) * n rounded up to 8 (1-D, xcd_item), block 256.
struct TrArgs {
  const float* gcax;        // [nds][n][Y][XW] dL/dCA_x
  const uint32_t* arms;     // [2n][Y][XA]
  const uint2* sp;          // [2n][Y][XS] padded pixel planes
  const float* lam;         // device [2]
  float* g_half;            // [2n][Y][X] half-image gradients (left ones written or added here)
  float* gr_part;           // [n][strips][Y][WP] -dL/dR partials of this slab
  float2* lam_part;         // one {d/dlambda_AD, d/dlambda_census} per workgroup
  int X, Y, XS, pads, XA, XW, npair, dlo, dhi, nstrips, WP;
  int first;                // first slab: the left gradients are written, not added
};

constexpr int kTrMaxWP = 64 + 127;  // 64 columns + a slab of up to 128 disparities
constexpr int kTrD = 16;            // disparities of a tile
constexpr int kTrRows = 4;          // rows of a block, one a wave
constexpr int kTrPitch = 68;        // of an LDS tile: the four quarters' rows in different banks
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// Four bytes by selector: 0..3 take a byte of lo, 4..7 one of hi, 12 zero.
__device__ __forceinline__ uint32_t perm8(uint32_t hi, uint32_t lo, uint32_t sel) {
  return __builtin_amdgcn_perm(hi, lo, sel);
}

// -1, 0 or 1 by the sign of the integer v.
__device__ __forceinline__ int sign_int(uint32_t v) {
  int r;
  __asm__("v_med3_i32 %0, %1, -1, 1" : "=v"(r) : "v"(v));
  return r;
}
// max(m, |a|, |b|)
__device__ __forceinline__ float max3_abs(float m, float a, float b) {
  __asm__("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(m) : "v"(m), "v"(a), "v"(b));
  return m;
}

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) k_soft_tr(TrArgs a) {
  __shared__ uint2 s_r[4][kTrMaxWP];
  __shared__ float s_gr[4][kTrMaxWP];
  __shared__ float s_g[4][kTrD][kTrPitch];
  __shared__ __align__(16) float s_dn[4][kTrD];  // per wave: scales of a tile's disparities
  __shared__ float s_hc[4][8];  // per wave: the census term of dC/dlambda_census by h
  __shared__ float2 s_red[4];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int nbands = (a.Y + kTrRows - 1) / kTrRows, count = a.nstrips * nbands * a.npair;
  const int item = xcd_item(blockIdx.x, count);
  if (item >= count) return;
  const int strip = item % a.nstrips, y = item / a.nstrips % nbands * kTrRows + wave;
  const int pair = item / (a.nstrips * nbands);
  const int X = a.X, Y = a.Y;
  const int l16 = lane & 15, quarter = lane >> 4;
  float pa = 0.f, pcs = 0.f;
  if (y < Y) {
    const int x0 = strip * 64, x = x0 + lane;
    const uint2* spl = a.sp + ((size_t)(2 * pair) * Y + y) * a.XS + a.pads;
    const uint2* spr = spl + (size_t)Y * a.XS;
    const uint32_t* arm = a.arms + ((size_t)(2 * pair) * Y + y) * a.XA;
    const float* grow = a.gcax + ((size_t)pair * Y + y) * a.XW;
    const size_t dstride = (size_t)a.npair * Y * a.XW;
    const bool ends = x0 < 32 || x0 + 96 > X;  // some sources lie outside the image
    // the sources of a tile of 16 disparities: source tile k, this lane's
    // disparity (past the slab the last one again; its rows are not used) and its
    // 16 columns x0 - 32 + 64 k + 16 quarter + j
    float4 v[2][4];
    auto load_tile = [&](int dt) {
      const int dl = min(dt + l16, a.dhi - 1) - a.dlo;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        // (a group that reaches past X ends in the row's padding)
        const int xs = x0 - 32 + 64 * k + 16 * quarter;
        const float* gp = grow + (size_t)dl * dstride + min(max(xs, 0), (X - 1) & ~15);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[k][j] = reinterpret_cast<const float4*>(gp)[j];
      }
    };
    load_tile(a.dlo);
    // right pixels of columns x0 - dhi + 1 .. x0 + 63 - dlo (the plane's padding
    // reads zero outside the image)
    const int wd = 64 + (a.dhi - a.dlo) - 1;
    for (int i = lane; i < wd; i += 64) s_r[wave][i] = spr[x0 - a.dhi + 1 + i];
    const float lam_ad = a.lam[0], lam_c = a.lam[1];
    const float k2 = 255.f * 1.4426950408889634f / lam_ad;
    const float kt = 255.f / lam_ad, ka = 1.f / (lam_ad * lam_ad), kc = 1.f / (lam_c * lam_c);
    const float l2c = 1.4426950408889634f / lam_c;
    // -e^{-h/lambda_census} h / lambda_census^2 for h = 0..6, one copy per wave
    // (a wave's LDS accesses are served in order: no barrier)
    if (lane < 7)
      s_hc[wave][lane] = -fast_exp2(-(float)lane * l2c) * (float)lane * kc;
    WAVE_LDS_ORDER();
    const uint32_t hc0 = lds_addr(s_hc[wave]);
    uint2 lp = spl[x];
    lp.x = __float_as_uint(__uint_as_float(lp.x) + 0.f);  // (-0 - 0 would be -0)
    // the 0/1 matrix: of source tile k, this lane's 16 sources against its column
    // of group n, one byte each.  A source x holds column c when v = c - x + m
    // and m + n - v are both >= 0; two sources a word, in 16 bits, where the sign
    // byte of either is 0xff or 0.  Sources left of the image or past
    // the rows of arms hold none; those between X and there have no arms.
    uint32_t bm[4][2][4];
    int k128[4] = {0, 0, 0, 0};  // the number of the column's sources, then 128 times it
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int xs = x0 - 32 + 64 * k + 16 * quarter;  // first of the 16
      const uint4* ap = reinterpret_cast<const uint4*>(arm + min(max(xs, 0), a.XA - 16));
      const uint32_t rel = (uint32_t)(x0 + l16 - xs) & 0xffffu;  // c - x of source 0, group 0
      const u16x2 rel2 = {(uint16_t)rel, (uint16_t)rel};
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const uint4 w4 = ap[jj];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          // m and m + n of sources 4 jj + 2 i, + 1
          const uint32_t wa = i ? w4.z : w4.x, wb = i ? w4.w : w4.y;
          const u16x2 m = __builtin_bit_cast(u16x2, perm8(wb, wa, 0x0c040c00u));
          u16x2 l = m + __builtin_bit_cast(u16x2, perm8(wb, wa, 0x0c050c01u));
          l = (uint32_t)xs < (uint32_t)a.XA ? l : u16x2{0xff80, 0xff80};  // -128: below every v
          const u16x2 v0 = rel2 + m - u16x2{(uint16_t)(4 * jj + 2 * i), (uint16_t)(4 * jj + 2 * i + 1)};
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const u16x2 v2 = v0 + u16x2{(uint16_t)(16 * n), (uint16_t)(16 * n)};
            const uint32_t miss = __builtin_bit_cast(uint32_t, v2) | __builtin_bit_cast(uint32_t, l - v2);
            if (i == 0) {
              bm[n][k][jj] = miss;
            } else {
              const uint32_t b = ~perm8(miss, bm[n][k][jj], 0x07050301u) & 0x01010101u;
              bm[n][k][jj] = b;
              k128[n] += __builtin_popcount(b);
            }
          }
        }
      }
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      k128[n] += __shfl_xor(k128[n], 16);
      k128[n] = 128 * (k128[n] + __shfl_xor(k128[n], 32));
    }
    float gl = 0.f, gr = 0.f;
    for (int dt = a.dlo; dt < a.dhi; dt += kTrD) {
      // scale of this lane's disparity, from its 32 values and the other quarters'
      float mx = 0.f;
      if (ends) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          int xs = x0 - 32 + 64 * k + 16 * quarter;
          __asm__ volatile("" : "+v"(xs));  // keeps this a branch
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            v[k][j].x = (uint32_t)(xs + 4 * j) < (uint32_t)X ? v[k][j].x : 0.f;
            v[k][j].y = (uint32_t)(xs + 4 * j + 1) < (uint32_t)X ? v[k][j].y : 0.f;
            v[k][j].z = (uint32_t)(xs + 4 * j + 2) < (uint32_t)X ? v[k][j].z : 0.f;
            v[k][j].w = (uint32_t)(xs + 4 * j + 3) < (uint32_t)X ? v[k][j].w : 0.f;
          }
        }
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          mx = max3_abs(max3_abs(mx, v[k][j].x, v[k][j].y), v[k][j].z, v[k][j].w);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      // (the smallest terms' scale stays finite)
      const uint32_t mb = __float_as_uint(mx);
      const int ex = max(float_exp(mb), -100);
      // a mantissa of ones would round to 2^23, one more than three bytes hold: such
      // values are taken as the float below, 2^23 - 1 units (as near as 2^23 is)
      const bool ones = (mb & 0x7fffffu) == 0x7fffffu;
      if (__any(ones)) {
        const float lim = __uint_as_float(ones ? mb - 1u : mb);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            v[k][j].x = fminf(fmaxf(v[k][j].x, -lim), lim);
            v[k][j].y = fminf(fmaxf(v[k][j].y, -lim), lim);
            v[k][j].z = fminf(fmaxf(v[k][j].z, -lim), lim);
            v[k][j].w = fminf(fmaxf(v[k][j].w, -lim), lim);
          }
      }
      const float up = mb ? ldexpf(1.f, 23 - ex) : 0.f;
      if (lane < kTrD) s_dn[wave][lane] = mb ? ldexpf(1.f, ex - 23) : 0.f;
      // the terms' bytes, the lower two less 128
      uint32_t dig[3][2][4];
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float f[4] = {v[k][j].x, v[k][j].y, v[k][j].z, v[k][j].w};
          uint32_t q[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) q[i] = (uint32_t)(int)rintf(f[i] * up);
          const uint32_t l01 = perm8(q[1], q[0], 0x05010400u), l23 = perm8(q[3], q[2], 0x05010400u);
          const uint32_t h01 = perm8(q[1], q[0], 0x0c0c0602u), h23 = perm8(q[3], q[2], 0x06020c0cu);
          dig[0][k][j] = perm8(l23, l01, 0x05040100u) ^ 0x80808080u;
          dig[1][k][j] = perm8(l23, l01, 0x07060302u) ^ 0x80808080u;
          dig[2][k][j] = h01 | h23;
        }
      i32x4 acc[4] = {};
      auto frag = [](const uint32_t (&u)[4]) {
        return i32x4{(int)u[0], (int)u[1], (int)u[2], (int)u[3]};
      };
#pragma unroll
      for (int g = 2; g >= 0; --g) {
        if (g < 2) {
#pragma unroll
          for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[n][i] = (acc[n][i] << 8) + k128[n];
        }
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int n = 0; n < 4; ++n)
            acc[n] = __builtin_amdgcn_mfma_i32_16x16x64_i8(frag(dig[g][k]), frag(bm[n][k]), acc[n], 0, 0, 0);
      }
      if (dt + kTrD < a.dhi) load_tile(dt + kTrD);  // in flight through the derivatives
      WAVE_LDS_ORDER();
      const float4 dn4 = *reinterpret_cast<const float4*>(&s_dn[wave][4 * quarter]);
      const float dn[4] = {dn4.x, dn4.y, dn4.z, dn4.w};
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int n = 0; n < 4; ++n)
          s_g[wave][4 * quarter + r][16 * n + l16] = (float)acc[n][r] * dn[r];
      WAVE_LDS_ORDER();
      // columns without a match and columns past X add nothing: only in the
      // strips left of the disparity and in the last strip
      const bool edge = x0 < dt + kTrD - 1 || x0 + 64 > X;
      const int ib = lane + (a.dhi - 1 - dt);  // LDS entry of column x - dt
      const int nr = min(kTrD, a.dhi - dt);
      static_while<kTrD>([&](auto R) {
        constexpr int r = decltype(R)::value;
        if (r >= nr) return false;
        float gc = s_g[wave][r][lane];
        if (edge) {
          int xx = x;
          __asm__ volatile("" : "+v"(xx));  // keeps this a branch
          gc = xx >= dt + r && xx < X ? gc : 0.f;
        }
        const uint2 rp = s_r[wave][ib - r];
        const float di = __uint_as_float(lp.x) - __uint_as_float(rp.x), ad = fabsf(di);
        const float E = fast_exp2(-ad * k2);
        const float tv = (float)sign_int(__float_as_uint(di)) * (gc * E);
        gl += tv;
        gr = tv + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(gr), 0x138, 0xf, 0xf, true));
        s_gr[wave][ib - r] = gr;
        pa = fmaf(gc, __fmul_rn(__fmul_rn(__fmul_rn(E, -255.f), ad), ka), pa);
        pcs = fmaf(gc, __uint_as_float(lds_read(__builtin_popcount(lp.y ^ rp.y) + hc0)), pcs);
        return true;
      });
      WAVE_LDS_ORDER();
    }
    // left gradients: each pixel has one owner (so the first slab writes every
    // one); slabs run one after another
    if (x < X) {
      float* g = a.g_half + ((size_t)(2 * pair) * Y + y) * X + x;
      *g = a.first ? kt * gl : *g + kt * gl;
    }
    // right partials of this strip: columns x0 - dhi + 1 .. x0 + 63 - dlo
    float* gp = a.gr_part + (((size_t)pair * a.nstrips + strip) * Y + y) * a.WP;
    for (int c = lane; c < wd; c += 64) gp[c] = -kt * s_gr[wave][c];
  }
  // fixed-order reduction of the lambda partials over the workgroup
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    pa += __shfl_down(pa, o);
    pcs += __shfl_down(pcs, o);
  }
  if (lane == 0) s_red[wave] = make_float2(pa, pcs);
  __syncthreads();
  if (t == 0) {
    float2 s = s_red[0];
    for (int w = 1; w < 4; ++w) { s.x += s_red[w].x; s.y += s_red[w].y; }
    a.lam_part[item] = s;
  }
}

// --------------------------------------------------------- k_soft_gright
// dL/dR(x,y) over a slab [dlo, dhi): the partials of the strips s whose
// columns x + d (d in the slab) reach, floor((x + dlo) / 64) ..
// floor((x + dhi - 1) / 64), summed in strip order, written to g_half for the
// first slab and added to it for the others.
// grid: (ceil(X/256), Y, n), block 256.
__global__ void __launch_bounds__(256) k_soft_gright(const float* __restrict__ gr_part, int nstrips,
                                                     int WP, int dlo, int dhi, int X, int Y,
                                                     int first, float* __restrict__ g_half) {
  const int x = blockIdx.x * 256 + threadIdx.x, y = blockIdx.y, pair = blockIdx.z;
  if (x >= X) return;
  const int s0 = (x + dlo) / 64, s1 = min(nstrips - 1, (x + dhi - 1) / 64);
  float acc = 0.f;
  for (int s = s0; s <= s1; ++s) {
    const int c = x - (s * 64 - dhi + 1);  // in 0 .. WP - 1 for the strips reached
    acc += gr_part[(((size_t)pair * nstrips + s) * Y + y) * WP + c];
  }
  float* g = g_half + ((size_t)(2 * pair + 1) * Y + y) * X + x;
  *g = first ? acc : *g + acc;
}

// ---------------------------------------------------------- k_soft_gfull
// dL/d(RGB) from dL/d(half image): a full-res pixel (u, v) receives g/9 from
// every half-res pixel whose clamped 3x3 block holds it, once per block cell
// that lands on it, times the channel's gray weight (77, 150, 29) / 256.
// Along each axis those pixels are among p >> 1 and (p + 1) >> 1 (the latter
// only for odd p inside the image), with weight #{j in -1..1 :
// clamp(2 q + j) = p}: the four loads are unconditional (indices clamped, a
// repeated index gets weight 0).
// grid: (ceil(W/256), H, 2n), block 256.
__device__ __forceinline__ int gfull_weight(int q, int p, int lim) {
  int w = 0;
#pragma unroll
  for (int j = -1; j <= 1; ++j) w += clampi(2 * q + j, 0, lim - 1) == p;
  return w;
}

__global__ void __launch_bounds__(256) k_soft_gfull(const float* __restrict__ g_half, int W, int H,
                                                    int X, int Y, float* __restrict__ g_left,
                                                    float* __restrict__ g_right) {
  const int u = blockIdx.x * 256 + threadIdx.x, v = blockIdx.y, img = blockIdx.z;
  if (u >= W) return;
  const float* gh = g_half + (size_t)img * X * Y;
  const int ya = v >> 1, yb = min((v + 1) >> 1, Y - 1);
  const int xa = u >> 1, xb = min((u + 1) >> 1, X - 1);
  const float g00 = gh[(size_t)ya * X + xa], g01 = gh[(size_t)ya * X + xb];
  const float g10 = gh[(size_t)yb * X + xa], g11 = gh[(size_t)yb * X + xb];
  const float wya = (float)gfull_weight(ya, v, H), wyb = yb != ya ? (float)gfull_weight(yb, v, H) : 0.f;
  const float wxa = (float)gfull_weight(xa, u, W), wxb = xb != xa ? (float)gfull_weight(xb, u, W) : 0.f;
  const float acc = (wya * (wxa * g00 + wxb * g01) + wyb * (wxa * g10 + wxb * g11)) *
                    (1.f / (9.f * 256.f));
  float* out = ((img & 1) ? g_right : g_left) + ((size_t)(img >> 1) * H * W + (size_t)v * W + u) * 3;
  out[0] = 77.f * acc;
  out[1] = 150.f * acc;
  out[2] = 29.f * acc;
}

// ------------------------------------------------------------ k_soft_lam
// Sum of the per-workgroup lambda partials in a fixed order: thread t sums
// entries t + 1024 j into four accumulators (j mod 4), then a tree.
// grid: 1, block 1024.
__global__ void __launch_bounds__(1024) k_soft_lam(const float2* __restrict__ part, int count,
                                                   float* __restrict__ g_lam) {
  __shared__ float2 s[1024];
  const int t = threadIdx.x;
  float2 acc[4] = {};
  int i = t, j = 0;
  for (; i + 3 * 1024 < count; i += 4 * 1024) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float2 v = part[i + u * 1024];
      acc[u].x += v.x;
      acc[u].y += v.y;
    }
  }
  for (; i < count; i += 1024, ++j) {
    const float2 v = part[i];
    acc[j & 3].x += v.x;
    acc[j & 3].y += v.y;
  }
  s[t] = make_float2((acc[0].x + acc[1].x) + (acc[2].x + acc[3].x),
                     (acc[0].y + acc[1].y) + (acc[2].y + acc[3].y));
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if (t < o) {
      s[t].x += s[t + o].x;
      s[t].y += s[t + o].y;
    }
    __syncthreads();
  }
  if (t == 0) {
    g_lam[0] = s[0].x;
    g_lam[1] = s[0].y;
  }
}

// ----------------------------------------------------------- k_fill_f32
__global__ void k_fill_f32(float* __restrict__ p, size_t n, float v) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// ---------------------------------------------------------------- k_l1_*
// L = (1/n) sum over pairs of mean over {(x,y): nonocc(2x,2y)} of
// |2 d_hat(x,y) - GT(2x,2y)|; dL/dd_hat = 2 sign(2 d_hat - GT) / (n count)
// there (sign(0) = 0), 0 elsewhere.
// k_l1_partial grid: (nblk, n), block 256; partial sums per block.  Block b
// takes the rows b, b + nblk, ...; each thread four columns of a row at a
// time, their loads issued together (columns past X clamped, then not
// counted); a fixed-order reduction over the block.
__global__ void __launch_bounds__(256) k_l1_partial(const float* __restrict__ dhat,
                                                    const int16_t* __restrict__ gt,
                                                    const uint8_t* __restrict__ nonocc, int W,
                                                    int H, int X, int Y,
                                                    float2* __restrict__ part) {
  __shared__ float2 s[4];
  const int t = threadIdx.x, pair = blockIdx.y;
  const int npix = X * Y;
  float sum = 0.f, cnt = 0.f;
  for (int y = blockIdx.x; y < Y; y += gridDim.x) {
    const size_t fr = (size_t)pair * H * W + (size_t)(2 * y) * W;
    const float* dr = dhat + (size_t)pair * npix + (size_t)y * X;
    for (int x0 = 0; x0 < X; x0 += 4 * 256) {
      float dv[4];
      int gv[4];
      uint32_t mv[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int x = min(x0 + t + 256 * k, X - 1);
        dv[k] = dr[x];
        gv[k] = gt[fr + 2 * x];
        mv[k] = nonocc[fr + 2 * x];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool use = x0 + t + 256 * k < X && mv[k] != 0u;
        sum += use ? fabsf(2.f * dv[k] - (float)gv[k]) : 0.f;
        cnt += use ? 1.f : 0.f;
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    sum += __shfl_xor(sum, o, 64);
    cnt += __shfl_xor(cnt, o, 64);
  }
  if ((t & 63) == 0) s[t >> 6] = make_float2(sum, cnt);
  __syncthreads();
  if (t == 0) {
    float2 r = s[0];
    for (int w = 1; w < 4; ++w) {
      r.x += s[w].x;
      r.y += s[w].y;
    }
    part[(size_t)pair * gridDim.x + blockIdx.x] = r;
  }
}

// k_l1_final grid: 1, block 256: loss and the per-pair counts.  Wave w takes
// the pairs w, w + 4, ...: lane b sums the blocks b, b + 64, ... of a pair,
// then a butterfly over the lanes; the per-pair means are summed in pair
// order (a fixed order: the result does not depend on scheduling).
__global__ void __launch_bounds__(256) k_l1_final(const float2* __restrict__ part, int nblk,
                                                  int npair, float* __restrict__ loss,
                                                  float* __restrict__ counts) {
  __shared__ float s_mean[64];  // npair <= 64
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int p = wave; p < npair; p += 4) {
    float s = 0.f, c = 0.f;
#pragma unroll 4
    for (int b = lane; b < nblk; b += 64) {
      const float2 v = part[(size_t)p * nblk + b];
      s += v.x;
      c += v.y;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      s += __shfl_xor(s, o, 64);
      c += __shfl_xor(c, o, 64);
    }
    if (lane == 0) {
      counts[p] = c;
      s_mean[p] = s / fmaxf(c, 1.f);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float total = 0.f;
    for (int p = 0; p < npair; ++p) total += s_mean[p];
    *loss = total / (float)npair;
  }
}

// k_l1_grad grid: (ceil(X*Y/256), n), block 256.
__global__ void __launch_bounds__(256) k_l1_grad(const float* __restrict__ dhat,
                                                 const int16_t* __restrict__ gt,
                                                 const uint8_t* __restrict__ nonocc,
                                                 const float* __restrict__ counts,
                                                 const float* __restrict__ gscale, int W, int H,
                                                 int X, int Y, int npair,
                                                 float* __restrict__ g_dhat) {
  const int i = blockIdx.x * 256 + threadIdx.x, pair = blockIdx.y;
  const int npix = X * Y;
  if (i >= npix) return;
  const int y = i / X, x = i - y * X;
  const size_t f = (size_t)pair * H * W + (size_t)(2 * y) * W + 2 * x;
  // all loads issued together, the mask applied after
  const uint8_t m = nonocc[f];
  const float dv = dhat[(size_t)pair * npix + i], gv = (float)gt[f];
  const float cnt = counts[pair], sc = gscale ? *gscale : 1.f;
  const float r = 2.f * dv - gv;
  const float sg = r > 0.f ? 1.f : (r < 0.f ? -1.f : 0.f);
  float g = 2.f * sg / (fmaxf(cnt, 1.f) * (float)npair);
  if (gscale) g *= sc;
  g_dhat[(size_t)pair * npix + i] = m ? g : 0.f;
}

}  // namespace
}  // namespace stereo_dev
