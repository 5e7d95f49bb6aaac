// Device kernels of the stereo path (gfx950, wave64).
//
// Pipeline per pair (Sec. IV, Step1-8), all integer arithmetic:
//   k_prep     RGB -> gray -> 3x3 mean at even coordinates    (Sec. III-A, Eq. 2)
//   k_feat     mini-census + cross arms of both half images    (Sec. III-B, III-C)
//   k_match    cost, x- and y-aggregation and WTA, fused: the  (Eq. 3-9)
//              cost volume never leaves the chip
//   k_wta      combine the d-chunk minima                       (Eq. 9)
//   k_refine   cross-check, 3x3 median and bilateral filling    (Eq. 10, Sec. III-E, Eq. 11)
//   k_upscale  bilateral x / linear y upscale to full res      (Step8)
//   k_post     the last three in one, for small frames
//   k_gray_full  the full-resolution mode's first step          (Sec. V)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "common.h"

namespace stereo_dev {
// Internal linkage: each source of the library that launches a kernel
// carries its own copy (no relocatable device code).
namespace {

constexpr int kTX = 64;           // k_match strip width = one wave
constexpr int kWaves = 16;        // k_match workgroup = 16 waves
constexpr int kThreads = kWaves * 64;
constexpr int kLdsBytes = 163840; // LDS per workgroup on gfx950
constexpr int kXcds = 8;          // accelerator complex dies, each with its own L2
constexpr int kWinGroup = 2;      // k_match slot pairs whose window reads go together
constexpr int kRowBatch = 2;      // k_match rows whose lookups and scans interleave

__device__ __forceinline__ int iabs(int v) { return v < 0 ? -v : v; }
__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }
__device__ __forceinline__ int gray_of(const uint8_t* p) {
  return (77 * p[0] + 150 * p[1] + 29 * p[2] + 128) >> 8;
}

// ---------------------------------------------------------------- k_prep
// One workgroup = 64 x 8 half-res pixels of one image.  The gray values of
// the full-res rows 2 y0 - 1 .. 2 y0 + 15 and columns 2 x0 - 4 .. 2 x0 + 131
// (borders clamped) go to LDS; each thread then forms the rounded-half-up
// mean of the 3x3 block centred on (2x, 2y) for two output rows.  Where the
// tile's columns lie inside the image, rows start 4-byte aligned (W a
// multiple of 4, aligned base) and a thread reads 4 RGB pixels as three
// aligned words; each gray is then one byte-align and one 4-byte dot product.
// Elsewhere each pixel is read bytewise with clamped coordinates.
// grid: (ceil(X/64), ceil(Y/8), 2 * npair), block (64, 4).
constexpr int kPrepRows = 8;

__global__ void __launch_bounds__(256) k_prep(PairPtrs pp, int W, int H, int X, int Y,
                                              uint8_t* __restrict__ half) {
  constexpr int TR = 2 * kPrepRows + 1, TC = 136, TG = TC / 4;  // TG groups of 4 pixels a row
  constexpr uint32_t kGrayW = 77u | 150u << 8 | 29u << 16;      // gray weights per byte
  __shared__ __align__(4) uint8_t g[TR + 1][TC];  // row TR takes the stores of idle items
  const int x0 = blockIdx.x * 64, y0 = blockIdx.y * kPrepRows, img = blockIdx.z;
  const int pair = img >> 1;
  const uint8_t* rgb = (img & 1) ? pp.right[pair] : pp.left[pair];
  const int t = threadIdx.y * 64 + threadIdx.x, cb = 2 * x0 - 4;  // tile column 0
  const bool words = (W & 3) == 0 && (reinterpret_cast<uintptr_t>(rgb) & 3u) == 0 && cb >= 0 &&
                     cb + TC <= W;
  constexpr int NG = (TR * TG + 255) / 256;  // groups of 4 pixels per thread
  if (words) {
    uint32_t w[NG][3];
#pragma unroll
    for (int k = 0; k < NG; ++k) {  // all loads first; groups past the tile repeat its last
      const int gi = min(t + 256 * k, TR * TG - 1), r = gi / TG, c = 4 * (gi - r * TG);
      const uint32_t* q = reinterpret_cast<const uint32_t*>(
          rgb + ((size_t)clampi(2 * y0 - 1 + r, 0, H - 1) * W + cb + c) * 3);
      w[k][0] = q[0];
      w[k][1] = q[1];
      w[k][2] = q[2];
    }
#pragma unroll
    for (int k = 0; k < NG; ++k) {  // no branch, so no load is sunk next to its use
      const int gi = t + 256 * k;
      const int r = gi < TR * TG ? gi / TG : TR, c = gi < TR * TG ? 4 * (gi - r * TG) : 0;
      // pixel i's bytes start at byte 3i of the 12
      const uint32_t p0 = w[k][0], p1 = __builtin_amdgcn_alignbyte(w[k][1], w[k][0], 3),
                     p2 = __builtin_amdgcn_alignbyte(w[k][2], w[k][1], 2),
                     p3 = __builtin_amdgcn_alignbyte(w[k][2], w[k][2], 1);
      const uint32_t g0 = __builtin_amdgcn_udot4(p0 & 0xffffffu, kGrayW, 128u, false) >> 8;
      const uint32_t g1 = __builtin_amdgcn_udot4(p1 & 0xffffffu, kGrayW, 128u, false) >> 8;
      const uint32_t g2 = __builtin_amdgcn_udot4(p2 & 0xffffffu, kGrayW, 128u, false) >> 8;
      const uint32_t g3 = __builtin_amdgcn_udot4(p3 & 0xffffffu, kGrayW, 128u, false) >> 8;
      *reinterpret_cast<uint32_t*>(&g[r][c]) = g0 | g1 << 8 | g2 << 16 | g3 << 24;
    }
  } else {
    constexpr int NP = (TR * TC + 255) / 256;  // pixels per thread
    uint32_t px[NP][3];
#pragma unroll
    for (int k = 0; k < NP; ++k) {  // all loads first, clamped into the image
      const int pi = min(t + 256 * k, TR * TC - 1), r = pi / TC, c = pi - r * TC;
      const uint8_t* q = rgb + ((size_t)clampi(2 * y0 - 1 + r, 0, H - 1) * W +
                                clampi(cb + c, 0, W - 1)) * 3;
      px[k][0] = q[0];
      px[k][1] = q[1];
      px[k][2] = q[2];
    }
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int pi = t + 256 * k;
      const int r = pi < TR * TC ? pi / TC : TR, c = pi < TR * TC ? pi - r * TC : 0;
      g[r][c] = (uint8_t)((77 * px[k][0] + 150 * px[k][1] + 29 * px[k][2] + 128) >> 8);
    }
  }
  __syncthreads();
  const int lx = threadIdx.x, x = x0 + lx;
  if (x >= X) return;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int ly = threadIdx.y + 4 * k, y = y0 + ly;
    if (y >= Y) break;
    int s = 0;
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int i = 0; i < 3; ++i) s += g[2 * ly + j][2 * lx + 3 + i];
    half[(size_t)img * X * Y + (size_t)y * X + x] = (uint8_t)((s + 4) / 9);
  }
}

// ---------------------------------------------------------------- k_feat
// Packed half-res pixels.  The differentiable head takes {the float half
// image value's bits, census string in each of the four bytes} (8 bytes; the
// bit count of an xor of two such words is the byte offset of the distance in a
// table of floats).  k_match takes gray in
// bits 0..7 and the census string in bits 8..13 (16 bits), two pixels per
// 32-bit load; that plane is stored twice, the second copy one pixel to the
// right, so that the pair of pixels starting at any column is one aligned
// word of one of the copies (half the bytes per row of the 32-bit form, which
// k_match's row loads are bound by).
constexpr int kFeatRows = 16;    // output rows per k_feat workgroup (one pixel per thread)
constexpr int kMaxArm = 127;
constexpr uint32_t kCensus4 = 0x01010101u;  // a census string (6 bits) to four bytes

// Length of one arm of a pixel of value c: the number of steps t = 1, 2, ...
// along the axis, taken without a break, whose pixel satisfies |I - c| < delta,
// at most lim.  p points at the pixel in an LDS tile and STRIDE is the tile
// distance of one step (negative for the left / upper arm).  Steps are tested
// in chunks of up to 32 into a bitmask of the steps that fail, step t of a
// chunk in bit t-1, built from the farthest step down; the chunk's run is the
// number of trailing zeros.  A test is two VALU ops: v_sad_u16 forms
// |v - c| + 2^31 - delta, whose bit 31 is [|v - c| >= delta], and
// v_alignbit_b32 shifts that bit into the mask.  A chunk's loads are all
// issued before its first test.  The last chunk tests the cap rounded up to a
// multiple of 8 steps (a wave-uniform choice among four unrolled forms): the
// steps past the cap only set bits above it, which lim (<= cap) cuts off, and
// the tile holds kArmPad spare pixels for them.
constexpr int kArmPad = 7;

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// Run of passing steps 1..N (N <= 32) from the pixel at LDS address p, bias =
// 2^31 - delta.  The reads have constant offsets above the lowest address.
template <int STRIDE, int N>
__device__ __forceinline__ int arm_run(uint32_t p, uint32_t c, uint32_t bias) {
  uint32_t lo = STRIDE > 0 ? p + STRIDE : p + N * STRIDE;
  // (the reads of different N are not the same to the compiler, which would
  // share them and extend each byte apart from its read)
  __asm__ volatile("" : "+v"(lo));
  // one byte load per step (merged into wide loads, each byte would take
  // one more VALU op to extract; the compiler barrier keeps them apart)
  uint32_t v[N];
#pragma unroll
  for (int t = 1; t <= N; ++t) {
    v[t - 1] = *(const __attribute__((address_space(3))) uint8_t*)(uintptr_t)(
        lo + (uint32_t)(STRIDE > 0 ? (t - 1) * STRIDE : (t - N) * STRIDE));
    __asm__ volatile("" ::: "memory");
  }
  // the bits above N - 1 start as failures, so a chunk of fewer than 32
  // steps ends its run at N at most
  uint32_t m = 0xffffffffu;
#pragma unroll
  for (int t = N; t >= 1; --t)
    m = __builtin_amdgcn_alignbit(m, __builtin_amdgcn_sad_u16(v[t - 1], c, bias), 31);
  __asm__ volatile("; %1 steps" : "+v"(m) : "n"(N));  // (nor are the tests)
  return m == 0u ? 32 : __builtin_ctz(m);
}

template <int STRIDE>
__device__ __forceinline__ int arm_len(uint32_t p, int c, int delta, int cap, int lim) {
  if (delta <= 0 || cap <= 0) return 0;
  const uint32_t bias = 0x80000000u - (uint32_t)delta;
  const uint32_t cu = (uint32_t)c;
  int len = 0;
  bool alive = true;
  for (; cap > 32; cap -= 32, p += 32 * STRIDE) {
    const int run = arm_run<STRIDE, 32>(p, cu, bias);
    len += alive ? run : 0;
    alive = alive && run == 32;
  }
  int run;
  switch ((cap + 7) >> 3) {
    case 1: run = arm_run<STRIDE, 8>(p, cu, bias); break;
    case 2: run = arm_run<STRIDE, 16>(p, cu, bias); break;
    case 3: run = arm_run<STRIDE, 24>(p, cu, bias); break;
    default: run = arm_run<STRIDE, 32>(p, cu, bias); break;
  }
  len += alive ? run : 0;
  return min(len, lim);
}

// One workgroup = 64 columns x kFeatRows rows of one image, one pixel per
// thread.  Two LDS tiles of the half image (borders clamped): rows y0-1 ..
// y0+kFeatRows over the columns reachable by the horizontal arms and the
// census, and rows y0-arm_y .. y0+kFeatRows-1+arm_y over the 64 columns for
// the vertical arms, each with kArmPad spare pixels past the arms.
//   census: 6 neighbours in three rows, bit k = [neighbour < centre]
//   arms  : contiguous pixels with |I - I(centre)| < delta, capped per side
//           and at the image border; packed m | n<<8 | M<<16 | N<<24
// Pixels go to sp ({bits of half_f at the pixel (an unpadded [Y][X] plane per
// image), kCensus4 * census}, may be NULL) and to the two copies of pk16 (gray | census
// << 8, may be NULL; the second copy copy16 elements after the first, one
// pixel to the right); pitch XP, column x at pad + x.
// xoff (may be NULL) takes, for k_match's row pass, the distances in bytes
// from column x's entry in a wave's row buffer to the row-prefix entries that
// bound CA_x (Eq. 7) there: 4 (m + 1) down in bits 0..15 and 4 n up in bits
// 16..31; pitch XA like arms.
// Two workgroups share a CU only while a wave holds at most 80 SGPRs; the
// waves-per-EU bound keeps the compiler under that (above it the kernel took
// a fifth longer).
// Vector arithmetic first: 2 instructions a step tested (228 a pixel at caps 21
// and 31) of about 350, nearly all of the kinds that take four clocks; they issue
// in 78% of the SIMDs' cycles, and the LDS is active in 60%.  A wave is one row,
// so that row addresses are scalar, and every step's read is one instruction
// (both together took 515).  16 images of 960x540: 118 us before, 100 now; 2 of
// 718x496: 14.7 and 13.3.
// grid: (ceil(X/64), ceil(Y/kFeatRows), 2 * npair), block (64, kFeatRows).
__global__ void __launch_bounds__(64 * kFeatRows) __attribute__((amdgpu_waves_per_eu(8)))
k_feat(const uint8_t* __restrict__ half, int X, int Y, int delta, int arm_x_l, int arm_x_r,
       int arm_y, int XP, int pad, int XA, const float* __restrict__ half_f,
       uint2* __restrict__ sp, uint32_t* __restrict__ arms, uint32_t* __restrict__ xoff,
       uint16_t* __restrict__ pk16, size_t copy16) {
  constexpr int TXW = 64 + 2 * (kMaxArm + kArmPad);
  __shared__ uint8_t tx[kFeatRows + 2][TXW];
  __shared__ uint8_t ty[kFeatRows + 2 * (kMaxArm + kArmPad)][64];
  const int x0 = blockIdx.x * 64, y0 = blockIdx.y * kFeatRows, img = blockIdx.z;
  const int ly = __builtin_amdgcn_readfirstlane((int)threadIdx.y);  // a wave is a row
  const uint8_t* h = half + (size_t)img * X * Y;
  // horizontal cap of this image (the two images may differ, Sec. V)
  const int arm_x = (img & 1) ? arm_x_r : arm_x_l;
  // tile margins: the arms plus the spare steps (at least the census's 2)
  const int hx = arm_x + kArmPad, wx = 64 + 2 * hx;
  const int my = arm_y + kArmPad, hy = kFeatRows + 2 * my;
  // Tile loads: the loads of both tiles' first batches are issued before
  // the first store (one load, wait and store after another was bound by
  // memory latency); larger caps take more batches.  Rows and columns past a
  // tile's end are clamped to its last one: such a load and store repeat a
  // valid one with the same value.
  {
    const int r0 = ly, r1 = min(r0 + kFeatRows, kFeatRows + 1);
    const uint8_t* s0 = h + (size_t)clampi(y0 - 1 + r0, 0, Y - 1) * X;
    const uint8_t* s1 = h + (size_t)clampi(y0 - 1 + r1, 0, Y - 1) * X;
    const uint8_t* sc = h + clampi(x0 + (int)threadIdx.x, 0, X - 1);
    // tx: rows r0, r1 and columns c0 + lane, c0 + 64 + lane
    auto load_x = [&](int c0, int* cc, uint8_t* v) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        cc[k] = min(c0 + 64 * k + (int)threadIdx.x, wx - 1);
        const int gx = clampi(x0 - hx + cc[k], 0, X - 1);
        v[2 * k] = s0[gx];
        v[2 * k + 1] = s1[gx];
      }
    };
    auto store_x = [&](const int* cc, const uint8_t* v) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        tx[r0][cc[k]] = v[2 * k];
        tx[r1][cc[k]] = v[2 * k + 1];
      }
    };
    // ty: rows (j0 + j) * kFeatRows + r0, j < 8, of column lane
    auto load_y = [&](int j0, int* rr, uint8_t* v) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        rr[j] = min((j0 + j) * kFeatRows + r0, hy - 1);
        v[j] = sc[(size_t)clampi(y0 - my + rr[j], 0, Y - 1) * X];
      }
    };
    auto store_y = [&](const int* rr, const uint8_t* v) {
#pragma unroll
      for (int j = 0; j < 8; ++j) ty[rr[j]][threadIdx.x] = v[j];
    };
    int cc[2], rr[8];
    uint8_t vx[4], vy[8];
    load_x(0, cc, vx);
    load_y(0, rr, vy);
    store_x(cc, vx);
    store_y(rr, vy);
    for (int c0 = 128; c0 < wx; c0 += 128) {
      load_x(c0, cc, vx);
      store_x(cc, vx);
    }
    for (int j0 = 8; j0 * kFeatRows < hy; j0 += 8) {
      load_y(j0, rr, vy);
      store_y(rr, vy);
    }
  }
  __syncthreads();
  const int lx = threadIdx.x, x = x0 + lx, y = y0 + ly;
  const bool inside = x < X && y < Y;
  uint32_t p16 = 0;
  if (inside) {
    const uint8_t* row = &tx[ly + 1][hx + lx];   // row[i] = I(x + i, y)
    const int c = row[0];
    int bits = 0;
    bits |= (tx[ly][hx + lx - 1] < c) << 0;
    bits |= (tx[ly][hx + lx + 1] < c) << 1;
    bits |= (row[-2] < c) << 2;
    bits |= (row[2] < c) << 3;
    bits |= (tx[ly + 2][hx + lx - 1] < c) << 4;
    bits |= (tx[ly + 2][hx + lx + 1] < c) << 5;
    const uint32_t rowa = lds_addr(row), cola = lds_addr(&ty[ly + my][lx]);
    const int m = arm_len<-1>(rowa, c, delta, arm_x, min(arm_x, x));
    const int n = arm_len<1>(rowa, c, delta, arm_x, min(arm_x, X - 1 - x));
    const int M = arm_len<-64>(cola, c, delta, arm_y, min(arm_y, y));
    const int N = arm_len<64>(cola, c, delta, arm_y, min(arm_y, Y - 1 - y));
    if (sp)
      sp[((size_t)img * Y + y) * XP + pad + x] =
          make_uint2(__float_as_uint(half_f[((size_t)img * Y + y) * X + x]), (uint32_t)bits * kCensus4);
    arms[((size_t)img * Y + y) * XA + x] =
        (uint32_t)m | ((uint32_t)n << 8) | ((uint32_t)M << 16) | ((uint32_t)N << 24);
    if (xoff)
      xoff[((size_t)img * Y + y) * XA + x] = 4u * ((uint32_t)m + 1u) | 4u * (uint32_t)n << 16;
    p16 = (uint32_t)c | (uint32_t)bits << 8;
  }
  if (pk16) {
    // pairs (x, x + 1) as aligned words: copy 0 from the even columns, copy 1
    // (one column to the right) from the odd ones, the pixel x + 1 from the
    // next lane (one wave is one row of the tile); the copy-1 pair across two
    // workgroups (lane 63 here, lane 0 of the next) is written in halves
    const uint32_t nb = (uint32_t)__shfl_down((int)p16, 1, 64);
    if (inside) {
      uint16_t* q = pk16 + ((size_t)img * Y + y) * XP + pad + x;
      if ((lx & 1) == 0) {
        *reinterpret_cast<uint32_t*>(q) = p16 | nb << 16;
        if (lx == 0) q[copy16 + 1] = (uint16_t)p16;
      } else if (lx != 63) {
        *reinterpret_cast<uint32_t*>(q + copy16 + 1) = p16 | nb << 16;
      } else {
        q[copy16 + 1] = (uint16_t)p16;
      }
    }
  }
}

// ---------------------------------------------------------------- k_match
// Inclusive prefix sums over the 64 lanes of a wave of N values (DPP row shifts
// inside rows of 16 lanes, then row broadcasts across rows), step by step in turn:
// each DPP step waits two slots for the value it reads, which the other values'
// steps fill.
template <int N>
__device__ __forceinline__ void wave_scan_incl_n(uint32_t (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += __builtin_amdgcn_update_dpp(0u, v[i], 0x111, 0xf, 0xf, false);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += __builtin_amdgcn_update_dpp(0u, v[i], 0x112, 0xf, 0xf, false);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += __builtin_amdgcn_update_dpp(0u, v[i], 0x114, 0xf, 0xf, false);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += __builtin_amdgcn_update_dpp(0u, v[i], 0x118, 0xf, 0xf, false);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += __builtin_amdgcn_update_dpp(0u, v[i], 0x142, 0xa, 0xf, false);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += __builtin_amdgcn_update_dpp(0u, v[i], 0x143, 0xc, 0xf, false);
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// LDS words by their byte address.
typedef const __attribute__((address_space(3))) uint32_t* lds_cptr;
__device__ __forceinline__ uint32_t lds_read(uint32_t addr) { return *(lds_cptr)(uintptr_t)addr; }
__device__ __forceinline__ void lds_write2(uint32_t addr, uint32_t v0, uint32_t v1) {
  *(__attribute__((address_space(3))) u32x2*)(uintptr_t)addr = u32x2{v0, v1};
}

// Keeps the compiler from moving LDS accesses of one wave across this point;
// the LDS itself serves the accesses of a wave in issue order.
#define WAVE_LDS_ORDER() __asm__ volatile("" ::: "memory")

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes,
                                           0x00020000);
}

// cost table [h][signed brightness difference + 256], h = census distance
// 0..6: 7 rows of 511 entries.  The row pitch, 530 entries = 265 words, is 9
// banks mod 64: entries of rows 1..6 apart land 9, 18, ..., 54 banks apart,
// so lookups of neighbouring pixels (census distances a row or two apart,
// brightness differences a few entries apart) rarely share a bank.
constexpr int kTabPitch = 530;
constexpr int kTabRows = 7;
constexpr int kTab = kTabRows * kTabPitch;

// Values the device cost table is built from: the tables of Eq. 4 (AD) and
// Eq. 5 (census) in fixed point, computed on the host in double.
struct TabArgs {
  uint16_t ad[256];
  uint16_t mc[7];
};

// Set-up of a plan's device state, ordered on the plan's stream (no memset
// node, so it may be captured in a graph): clears nzero words at zero (the
// padding of the pixel and arm planes must read 0; the kernels write the
// image part) and writes the cost table, entry (h, 256 + diff) = LUT_AD[|diff|]
// + LUT_MC[h]; column 0 and the pitch's spare columns 0.
// grid: any, block 256.
__global__ void __launch_bounds__(256) k_plan_init(uint32_t* __restrict__ zero, size_t nzero,
                                                   uint16_t* __restrict__ tab, TabArgs t) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nzero; i += stride)
    zero[i] = 0u;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < (size_t)kTab; i += stride) {
    const int h = (int)i / kTabPitch, col = (int)i - h * kTabPitch;
    const int a = col < 256 ? 256 - col : col - 256;
    // columns 1..511 hold differences -255..255; column 0 (a difference of
    // -256) and the spare columns are never read
    tab[i] = (col == 0 || col > 511) ? (uint16_t)0 : (uint16_t)(t.ad[a] + t.mc[h]);
  }
}

// Bytes of k_match's static LDS: the cost table.
constexpr int kMatchTabBytes = ((kTab * 2 + 15) / 16) * 16;

// Bytes of k_match's dynamic LDS block with NS sub-passes, a plane of NB bases
// and `rows` rows (plane row 0 is the zero row): row buffers and the plane,
// whose rows hold 64 words per base.
__host__ __device__ constexpr int match_lds_bytes(int ns, int nbase, int rows) {
  return kWaves * ns * 128 * 4 + rows * nbase * 256;
}

// Plane rows (zero row included) that fit beside NS sub-passes of 128
// row-buffer columns.
__host__ __device__ constexpr int match_plane_rows(int ns, int nbase) {
  return (kLdsBytes - kMatchTabBytes - kWaves * ns * 128 * 4) / (nbase * 256);
}

// Rows behind the pixel and arm planes that k_match's row loads may touch: the
// missing second row of an odd segment and the next batch's two.
constexpr int kMatchSlackRows = 3;

// Most band rows per wave, and so most rows of a band over 16: what the plane
// holds with one sub-pass (288 rows of both bases, 576 of one).
__host__ __device__ constexpr int match_seg_rows(int nbase) { return 36 / nbase; }

// Columns left of a strip in k_match's row buffer: the window's entry
// x - m - 1, rounded up to even (column pairs).
__host__ __device__ constexpr int match_halo(int arm_cap) { return (arm_cap + 2) & ~1; }

// How far the right-based strip, moved by d, may lie left (lo) or right (hi)
// of the left-based one so that the windows of both still fall inside the
// 128 NS row-buffer columns; arm = the larger horizontal cap.  The d-chunks
// hold at most lo + hi + 1 disparities.
__host__ __device__ constexpr int match_slack_lo(int arm) { return match_halo(arm) - (arm + 1); }
__host__ __device__ constexpr int match_slack_hi(int ns, int arm) {
  return 128 * ns - match_halo(arm) - 64 - arm;
}

// Column offset of the right-based strip of a chunk that ends at disparity
// dlast: right strip start = left strip start - offset, the smallest offset
// that keeps d - offset <= hi.
__host__ __device__ constexpr int match_delta(int dlast, int hi) { return dlast > hi ? dlast - hi : 0; }

// The workgroups of a k_match launch: one per (strip, band, base with NB = 1,
// pair, d-chunk) that has an output column.  Every chunk has the nfull strips
// that start left of X; a chunk whose right-based strips are moved far enough
// (delta > x0 - X) has up to kMatchExtra more at the right.  Items are numbered
// by strip, so that neighbours read the same image rows: first those of the
// full strips, `units` (bands x bases x pairs) x nfull x nchunk, chunk fastest,
// then per extra strip units x (chunks it has).  Workgroups are dealt to the 8
// XCDs in turn (id mod 8); XCD k takes the items k * per .. (k + 1) * per - 1, so
// that a strip's rows stay in one XCD's L2 and every XCD has as many.
constexpr int kMatchExtra = 9;  // D <= 512, 64 columns a strip, and the last strip's ragged end

struct MatchGrid {
  int nfull, units, total, per;
  int nextra;                  // extra strips in use
  int first[kMatchExtra];      // first chunk of each extra strip
};

struct MatchArgs {
  const uint16_t* pk;     // [2][2*npair][Y][XP]  padded: gray | census << 8, two copies
  const uint32_t* arms;   // [2*npair][Y][XA]  zero past column X
  const uint32_t* xoff;   // [2*npair][Y][XA]  row-buffer distances (k_feat), zero past column X
  const uint16_t* tab;    // [kTabRows][kTabPitch]
  uint32_t* keys;         // [npair][nchunk][2][nk]  (min CA) << dbits | argmin d
  int X, Y, XP, pad, XA, nk, arm, arm_y;  // arm: the larger horizontal cap
  int cmax;               // cost of a match outside the other image
  int dbits;              // key = CA << dbits | d
  int nbands, dlo, dhi;
  int nchunk;             // d-chunks, of sizes that differ by one at most
  MatchGrid grid;
  uint32_t pk_bytes, arms_bytes;  // sizes of the pk (both copies) and arms buffers, slack rows included
  uint32_t copy_bytes;    // bytes from the first pk copy to the second
  // debug planes (pair 0, the single disparity dlo; used by the DBG variant)
  uint16_t* dbg_cost;
  uint32_t* dbg_cax;
  uint32_t* dbg_ca;
  int dbg_base;
};

// f(integral_constant 0), ..., f(integral_constant N - 1)
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// f(integral_constant 0), f(integral_constant 1), ... while f returns true
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_while(F&& f) {
  if constexpr (I < N) {
    if (f(std::integral_constant<int, I>{})) static_while<N, I + 1>(f);
  }
}

// acc + |hi - lo| (hi >= lo): one instruction
__device__ __forceinline__ uint32_t add_diff(uint32_t hi, uint32_t lo, uint32_t acc) {
  uint32_t r;
  __asm__("v_sad_u32 %0, %1, %2, %3" : "=v"(r) : "v"(hi), "v"(lo), "v"(acc));
  return r;
}

// One workgroup = one 64-column strip x one band of rows x one chunk of
// disparities; 16 waves.
// NB = 2 takes both base images: the cost C(c, d) of left column c against
// right column c - d serves both (Eq. 6: C^R(x') = C^L(x' + d)), so a row is
// evaluated and scanned once for 64 left-based columns x = x0 + lane and 64
// right-based ones x' = x0 - delta + lane; delta (match_delta) keeps the
// columns x' + d of every d of the chunk inside the row buffer.
// NB = 1 takes one base (columns x0 + lane; for the right one the images
// change places: cost(R(x), L(x + d)) is C^L(x + d) term for term): its plane
// holds twice the rows, for vertical arms so long that the halo rows of the
// lower bands cost more than the shared evaluation saves.
// For each d of the chunk:
//   row pass   : each wave takes a segment of the band's rows; every lane
//                evaluates the cost (Eq. 3-5, one lookup in a table indexed by
//                census distance and signed brightness difference) of two
//                adjacent columns of the 128 NS starting at x0 - hx, an inclusive
//                wave scan gives the row prefix P, and CA_x = P[x+n] - P[x-m-1]
//                (Eq. 7) of each base is added to running column sums, which
//                stay in registers row by row;
//   column pass: the segments' totals, exchanged through the row buffers, give
//                each wave its offset, and the column prefix Q of the band
//                goes to the LDS plane;
//   window, WTA: CA = Q[y+N] - Q[y-M-1] (Eq. 8) for the band's output rows and
//                key = min(key, CA << dbits | d): the smallest d wins ties (Step5).
// Two barriers a disparity: the plane is written between them and read after
// the second, so one wave's window step overlaps another's next row pass.
// Neither VALU issue nor the LDS is full: counters at 8 x 960x540 half-res
// pixels, D = 128, show vector instructions in 57% of the SIMDs' cycles (3.4 clocks
// each on average: measured alone, 32-bit adds, logic, shifts and moves of two
// operands take 2, the DPP, SDWA and three-operand forms, bit counts and minima 4)
// and the LDS active in 60%; a wave waits in 31% of its cycles, and 160 KB of LDS
// leave four waves a SIMD.  51%, 53% and 37% at 718x496, D = 73; 70%, 63% and 25%
// at 1436x992, D = 145 with arms 41 and 61.  Against one base a workgroup with the plane
// written in the row pass and corrected by LDS atomics after a third barrier:
// 1747 -> 1242 us there, 92.7 -> 77.8 us at 718x496 D = 73, 709 -> 539 us at
// 1436x992 D = 145, 1159 -> 855 us at 1436x992 D = 145 with arms 41 and 61.
// Sums wrap modulo 2^32; every difference taken is a window sum below
// 2^(32 - dbits) (the parameter check), hence exact and room for d in the
// key's low dbits.  A band has at most 16 KMAX output rows and 16
// match_seg_rows(NB) rows in all.
// grid: 8 * grid.per workgroups (1-D), block 1024.
template <int NS, int NB, int KMAX, bool DBG>
__global__ void __launch_bounds__(kThreads) k_match(MatchArgs a) {
  // The cost table is the kernel's static LDS, at LDS address 0, so table
  // addresses fold into the read's offset field.  The rest is one dynamic
  // block carved at constant offsets, sized by the host to the plane rows the
  // plan reads (match_lds_bytes): LDS the plan does not need is left to the
  // kernels of other streams (the next frame's), which can then share the CU.
  constexpr int kOffRow = 0;
  constexpr int kOffPlane = kOffRow + kWaves * NS * 128 * 4;
  constexpr int kPitch = NB * 64;  // words of a plane row
  constexpr int kSegRows = match_seg_rows(NB);
  __shared__ __align__(16) uint16_t s_tab[kMatchTabBytes / 2];
  extern __shared__ __align__(16) uint8_t s_lds[];
  auto s_row = reinterpret_cast<uint32_t(*)[NS * 128]>(s_lds + kOffRow);
  uint32_t* s_plane = reinterpret_cast<uint32_t*>(s_lds + kOffPlane);  // row 0 = zeros

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);  // uniform: row offsets stay scalar
  const int X = a.X, Y = a.Y;
  int item = (blockIdx.x & (kXcds - 1)) * a.grid.per + blockIdx.x / kXcds;
  if (blockIdx.x / kXcds >= a.grid.per || item >= a.grid.total) return;  // padding workgroup
  int strip, unit, chunk;
  if (item < a.grid.nfull * a.grid.units * a.nchunk) {
    chunk = item % a.nchunk;
    item /= a.nchunk;
    strip = item % a.grid.nfull;
    unit = item / a.grid.nfull;
  } else {
    item -= a.grid.nfull * a.grid.units * a.nchunk;
    int e = 0, n = a.nchunk - a.grid.first[0];
    while (item >= a.grid.units * n) {
      item -= a.grid.units * n;
      ++e;
      n = a.nchunk - a.grid.first[e];
    }
    strip = a.grid.nfull + e;
    unit = item / n;
    chunk = a.grid.first[e] + item - unit * n;
  }
  const int band = unit % a.nbands;
  unit /= a.nbands;
  const int base = NB == 2 ? 0 : unit & 1, pair = NB == 2 ? unit : unit >> 1;
  const int nd = a.dhi - a.dlo;
  const int d0 = a.dlo + chunk * nd / a.nchunk, d1 = a.dlo + (chunk + 1) * nd / a.nchunk;
  const int x0 = strip * kTX, delta = NB == 2 ? match_delta(d1 - 1, match_slack_hi(NS, a.arm)) : 0;
  const int ob = (Y + a.nbands - 1) / a.nbands;
  const int y0 = band * ob, y1 = min(Y, y0 + ob);
  const int ya = max(0, y0 - a.arm_y), yb = min(Y, y1 + a.arm_y);
  const int nb = yb - ya, o0 = y0 - ya, o1 = y1 - ya;
  const int hx = match_halo(a.arm), e0 = x0 - hx;  // the row buffer starts at column e0 (even)
  // columns c of image img[0] against columns c + sgn d of the other one
  const int sgn = base ? 1 : -1;
  const __amdgpu_buffer_rsrc_t rb = buffer_rsrc(a.pk, a.pk_bytes);
  const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(a.xoff, a.arms_bytes);
  const uint32_t img[2] = {(uint32_t)(2 * pair + base), (uint32_t)(2 * pair + (base ^ 1))};
  const uint32_t pkrow = (uint32_t)a.XP * 2u, armrow = (uint32_t)a.XA * 4u;
  const bool dbg = DBG && pair == 0 && (NB == 2 || base == a.dbg_base);
  (void)dbg;

  for (int i = t; i < kTab; i += kThreads) s_tab[i] = a.tab[i];
  if (t < kPitch) s_plane[t] = 0u;

  // output columns of the lane, per base: outside the image a clamped column
  // is read and nothing stored
  int xo[NB];
  uint32_t vx[NB];
#pragma unroll
  for (int h = 0; h < NB; ++h) {
    xo[h] = x0 + lane - (h ? delta : 0);
    vx[h] = (uint32_t)min(max(xo[h], 0), a.XA - 1) * 4u;
  }
  // rows of the band in segments of whole row pairs (the row pass takes its
  // rows in pairs), one per wave in order, the pairs split as evenly as
  // possible: the waves of each SIMD (wave mod 4) then share the rows evenly
  const int nbat = (nb + 1) / 2, bq = nbat / kWaves, br = nbat % kWaves;
  const int r0 = min(nb, 2 * (wave * bq + min(wave, br)));
  const int r1 = min(nb, r0 + 2 * (bq + (wave < br)));

  // Output rows of this thread: r = o0 + wave + 16 k, k < KMAX; slot k NB + h
  // is row k of base h.  marm packs per slot NB times the vertical arms M, N
  // (<= 127), one byte each, two slots a word: a plane row is 256 NB bytes,
  // so such an arm in bits 8..15 of a 16-bit half is its offset.  Rows outside
  // the band or columns outside the image get M = N = 0; their keys are never
  // stored.
  constexpr int kSlots = KMAX * NB;
  static_assert(kSlots % 2 == 0, "slots go in pairs");
  uint32_t key[kSlots], marm[kSlots / 2];
#pragma unroll
  for (int u = 0; u < kSlots; ++u) {
    const int k = u / NB, h = u % NB;
    key[u] = 0xffffffffu;
    const int r = o0 + wave + k * kWaves;
    // no branch around the load (a branch made every load wait for the one
    // before): rows past the band read its last row and are masked by a
    // wave-uniform select; columns past X read the plane's zero padding
    const uint32_t v = a.arms[((size_t)img[h] * Y + ya + min(r, o1 - 1)) * a.XA + vx[h] / 4u] >> 16;
    const uint32_t mn = r < o1 ? v * NB : 0u;  // arms <= 127: no bit crosses a byte
    if (u & 1) marm[u / 2] |= mn << 16;
    else marm[u / 2] = mn;
  }
  __syncthreads();

  const char* tb = reinterpret_cast<const char*>(s_tab) + 512;
  // cost of pixel J of a pair word: entry (h, 256 + diff) at byte offset
  // h * 2 * kTabPitch + 2 * diff + 512; the census distance h is the popcount
  // of the xor of the census bytes (one SDWA xor)
  auto cost = [&](uint32_t b, uint32_t o, auto J) -> uint32_t {
    uint32_t hw;
    if constexpr (decltype(J)::value == 0)
      __asm__("v_xor_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 "
              "src1_sel:BYTE_1" : "=v"(hw) : "v"(b), "v"(o));
    else
      __asm__("v_xor_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 "
              "src1_sel:BYTE_3" : "=v"(hw) : "v"(b), "v"(o));
    constexpr int sh = decltype(J)::value * 16;
    const uint32_t h = __builtin_popcount(hw);
    const int df = (int)((b >> sh) & 255u) - (int)((o >> sh) & 255u);
    const int e = (int)h * (2 * kTabPitch) + df + df;
    return *reinterpret_cast<const uint16_t*>(tb + e);
  };
  using J0 = std::integral_constant<int, 0>;
  using J1 = std::integral_constant<int, 1>;

  for (int d = d0; d < d1; ++d) {
    // Per-lane addresses are formed anew for each disparity from the lane
    // number, one instruction each: held over the loop they would take the
    // registers of the row sums (the asm statement hides that they are the same).
    uint32_t ln = (uint32_t)lane;
    __asm__ volatile("" : "+v"(ln));
    // byte offset of this lane's first column pair inside a padded pk row
    const uint32_t vb = (uint32_t)(a.pad + e0) * 2u + ln * 4u;
    // LDS addresses of the lane's pair in the wave's row buffer and of the
    // entry of column x0 + lane
    uint32_t wrow = lds_addr(s_row[wave]) + ln * 8u;
    const uint32_t ent0 = lds_addr(s_row[wave]) + (uint32_t)hx * 4u + ln * 4u;
    // a pair of other-image pixels starting at an odd column is an aligned
    // word of the second copy (the parity of the column is that of d)
    const uint32_t odd = (uint32_t)d & 1u;
    const uint32_t vo = vb + (uint32_t)(sgn * d * 2) + 2u * odd;
    const uint32_t ocopy = odd ? a.copy_bytes : 0u;
    // the entry of each base's output column: the right-based column x' is
    // left column x' + d
    uint32_t ent[NB];
    ent[0] = ent0;
    if constexpr (NB == 2) ent[1] = ent0 + (uint32_t)((d - delta) * 4);
    // held as they are: taken apart again, they would cost an add at each use
    __asm__ volatile("" : "+v"(ent[0]), "+v"(ent[NB - 1]), "+v"(wrow));
    // columns without a match cost C_max (the x - d < 0 / x + d >= X
    // convention): selected after the lookup, in the strips that hold such
    // columns only (wave-uniform).  Both bases: c < d and c >= X; one base:
    // the other image's column outside it.
    const int lo = NB == 2 ? d : (base ? -d : d), hi = NB == 2 ? X : (base ? X - d : X + d);
    const bool edge = e0 < lo || e0 + 128 * NS > hi;
    bool out[NS][2];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int c = e0 + s * 128 + 2 * (int)ln + jj;
        out[s][jj] = c < lo || c >= hi;
      }
    // ---- row pass over this wave's rows r0..r1-1, kRowBatch rows at a time
    // (their lookups and scans interleave), the loads of the next batch in flight.
    struct RowIn { uint32_t b[NS], o[NS], am[NB]; };
    // scalar byte offsets of the row to load next, stepped row by row (rows
    // past the segment's end belong to the next one, or to the kMatchSlackRows
    // rows behind the planes; their sums are not stored).  The asm statement
    // keeps the compiler from holding the offsets of all rows over the d loop.
    const uint32_t yi[2] = {img[0] * (uint32_t)Y + (uint32_t)(ya + r0), img[1] * (uint32_t)Y + (uint32_t)(ya + r0)};
    uint32_t sb = yi[0] * pkrow, so = yi[1] * pkrow + ocopy;
    uint32_t sa[2] = {yi[0] * armrow, yi[1] * armrow};
    __asm__ volatile("" : "+s"(sb), "+s"(so), "+s"(sa[0]), "+s"(sa[1]));
    auto load_batch = [&](RowIn (&in)[kRowBatch]) {
#pragma unroll
      for (int i = 0; i < kRowBatch; ++i) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          in[i].b[s] = __builtin_amdgcn_raw_buffer_load_b32(rb, vb + s * 256, sb, 0);
          in[i].o[s] = __builtin_amdgcn_raw_buffer_load_b32(rb, vo + s * 256, so, 0);
        }
#pragma unroll
        for (int h = 0; h < NB; ++h)
          in[i].am[h] = __builtin_amdgcn_raw_buffer_load_b32(ra, vx[h], sa[h], 0);
        sb += pkrow;
        so += pkrow;
        sa[0] += armrow;
        if constexpr (NB == 2) sa[1] += armrow;
      }
    };
    uint32_t run[kSegRows][NB], tot[NB] = {};
    RowIn in[2][kRowBatch];  // two buffer sets, used in turn
    if (r0 < r1) load_batch(in[0]);
    auto batch = [&](auto Q) {
      constexpr int q = decltype(Q)::value;
      const int r = r0 + q * kRowBatch;
      if (r >= r1) return false;
      // the waves of a SIMD issue oldest first: a falling priority keeps them
      // abreast, so that the last one does not run its rows alone
      if constexpr (q == 0) __builtin_amdgcn_s_setprio(2);
      if constexpr (q == kSegRows / 6) __builtin_amdgcn_s_setprio(1);
      if constexpr (q == kSegRows / 3) __builtin_amdgcn_s_setprio(0);
      // loaded unconditionally, so that the waits for this batch do not depend
      // on the next one's loads
      load_batch(in[(q + 1) & 1]);
      const RowIn (&cur)[kRowBatch] = in[q & 1];
      uint32_t c0[kRowBatch][NS], c1[kRowBatch][NS], pr[kRowBatch * NS];
#pragma unroll
      for (int i = 0; i < kRowBatch; ++i)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          c0[i][s] = cost(cur[i].b[s], cur[i].o[s], J0{});
          c1[i][s] = cost(cur[i].b[s], cur[i].o[s], J1{});
        }
      if (edge) {
#pragma unroll
        for (int i = 0; i < kRowBatch; ++i)
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            c0[i][s] = out[s][0] ? (uint32_t)a.cmax : c0[i][s];
            c1[i][s] = out[s][1] ? (uint32_t)a.cmax : c1[i][s];
          }
      }
#pragma unroll
      for (int i = 0; i < kRowBatch; ++i)
#pragma unroll
        for (int s = 0; s < NS; ++s) pr[i * NS + s] = c0[i][s] + c1[i][s];
      wave_scan_incl_n(pr);
#pragma unroll
      for (int i = 0; i < kRowBatch; ++i) {
        uint32_t carry = 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const uint32_t p = pr[i * NS + s] + carry;
          if (NS > 1) carry = __builtin_amdgcn_readlane(p, 63);
          lds_write2(wrow + s * 512, p - c1[i][s], p);
        }
        WAVE_LDS_ORDER();
        // CA_x of each base; am: byte distances of the entries x + n (high
        // half, up) and x - m - 1 (low half, down) from the column's own entry
        uint32_t ph[NB], pl[NB];
#pragma unroll
        for (int h = 0; h < NB; ++h) {
          ph[h] = lds_read(ent[h] + (cur[i].am[h] >> 16));
          pl[h] = lds_read(ent[h] - (cur[i].am[h] & 0xffffu));
        }
        WAVE_LDS_ORDER();
#pragma unroll
        for (int h = 0; h < NB; ++h) {
          tot[h] = add_diff(ph[h], pl[h], tot[h]);
          run[q * kRowBatch + i][h] = tot[h];
        }
        if constexpr (DBG) {
          const int y = ya + r + i;
          if (dbg && r + i < r1 && y >= y0 && y < y1) {
#pragma unroll
            for (int h = 0; h < NB; ++h)
              if ((NB == 1 || h == a.dbg_base) && xo[h] >= 0 && xo[h] < X)
                a.dbg_cax[(size_t)y * X + xo[h]] = ph[h] - pl[h];
            // the strip's columns of the wanted base: left column c is column
            // c - d of the right base
            const bool rb2 = NB == 2 && a.dbg_base;
            const int s0 = rb2 ? x0 - delta : x0;
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
              for (int jj = 0; jj < 2; ++jj) {
                const int c = e0 + s * 128 + 2 * lane + jj - (rb2 ? d : 0);
                if (c >= max(s0, 0) && c < min(s0 + kTX, X))
                  a.dbg_cost[(size_t)y * X + c] = (uint16_t)(jj ? c1[i][s] : c0[i][s]);
              }
          }
        }
      }
      return true;
    };
    static_while<kSegRows / kRowBatch>(batch);
    // ---- column pass.  The wave's totals go to its own row buffer (its rows
    // are done, and no other wave reads it before the barrier).  Only the
    // band's last rows can be an odd segment, whose total holds a row past the
    // end: no segment follows it, so that total is not used.
#pragma unroll
    for (int h = 0; h < NB; ++h) s_row[wave][NB * ln + h] = tot[h];
    __syncthreads();
    __builtin_amdgcn_s_setprio(3);
    uint32_t off[NB] = {};
    // the wave's own number as 8 + 4 + 2 + 1: groups of reads in flight together
    int s0 = 0;
#pragma unroll
    for (int n = kWaves / 2; n > 0; n >>= 1)
      if (wave & n) {
        uint32_t v[8][NB];
#pragma unroll
        for (int s = 0; s < n; ++s)
#pragma unroll
          for (int h = 0; h < NB; ++h) v[s][h] = s_row[s0 + s][NB * ln + h];
#pragma unroll
        for (int s = 0; s < n; ++s)
#pragma unroll
          for (int h = 0; h < NB; ++h) off[h] += v[s][h];
        s0 += n;
      }
    uint32_t* pw = s_plane + (r0 + 1) * kPitch + ln;
    // counted anew: the row pass's tests are not kept for these
    int nrows = r1 - r0;
    __asm__ volatile("" : "+s"(nrows));
    static_while<kSegRows>([&](auto K) {
      constexpr int k = decltype(K)::value;
      if (k >= nrows) return false;
#pragma unroll
      for (int h = 0; h < NB; ++h) pw[k * kPitch + h * 64] = run[k][h] + off[h];
      return true;
    });
    __syncthreads();
    // ---- vertical window and WTA for this wave's output rows, kWinGroup slot
    // pairs at a time, the reads of the next group in flight
    // byte offset in the plane of (band row o0 + wave, lane); plane row = band
    // row + 1
    const uint32_t fin_b = (uint32_t)((o0 + wave + 1) * kPitch) * 4u + ln * 4u;
    // the key shift lives in a VGPR, so that shift-and-or with the scalar d
    // is one instruction (one scalar operand per vector instruction)
    uint32_t vdbits = (uint32_t)a.dbits;
    // byte selector of v_perm: bytes 0 and 2 of marm (M of two slots) to bytes
    // 1 and 3, zeros to bytes 0 and 2
    uint32_t kpermM = 0x020c000cu;
    __asm__ volatile("" : "+v"(vdbits), "+v"(kpermM));
    uint32_t wh[2][kWinGroup][2], wl[2][kWinGroup][2];
    auto window_reads = [&](auto G) {
      constexpr int g = decltype(G)::value;
#pragma unroll
      for (int i = 0; i < kWinGroup; ++i) {
        constexpr int jp0 = g * kWinGroup;
        const int jp = jp0 + i;
        if (jp >= kSlots / 2) continue;
        // byte offsets of plane rows +N and -(M+1) from the output rows of two
        // slots (16-bit halves): nw holds N, mw holds M; each read address is
        // then one SDWA add or subtract.  Volatile asm keeps them inside the d
        // loop (hoisted, they would need kSlots VGPRs).
        uint32_t nw, mw;
        __asm__ volatile("v_and_b32 %0, 0xff00ff00, %1" : "=v"(nw) : "v"(marm[jp]));
        __asm__ volatile("v_perm_b32 %0, 0, %1, %2" : "=v"(mw) : "v"(marm[jp]), "v"(kpermM));
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          // rows +N and -(M+1) of the slot's output row (plane row 0 at least:
          // M never reaches above the band); the slot's constant part becomes
          // the reads' immediate offset
          const int u = 2 * jp + e, k = u / NB, h = u % NB;
          const uint8_t* row = s_lds + kOffPlane + k * kWaves * kPitch * 4 + h * 256 + fin_b;
          const uint32_t on = e ? nw >> 16 : nw & 0xffffu, om = e ? mw >> 16 : mw & 0xffffu;
          wh[g & 1][i][e] = *reinterpret_cast<const uint32_t*>(row + on);
          wl[g & 1][i][e] = *reinterpret_cast<const uint32_t*>(row - kPitch * 4 - om);
        }
      }
    };
    constexpr int kWinGroups = (kSlots / 2 + kWinGroup - 1) / kWinGroup;
    window_reads(std::integral_constant<int, 0>{});
    static_for<kWinGroups>([&](auto G) {
      constexpr int g = decltype(G)::value;
      if constexpr (g + 1 < kWinGroups) window_reads(std::integral_constant<int, g + 1>{});
      WAVE_LDS_ORDER();  // those reads are issued before this group is waited for
#pragma unroll
      for (int i = 0; i < kWinGroup; ++i)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int u = 2 * (g * kWinGroup + i) + e;
          if (u >= kSlots) continue;
          const uint32_t kv = ((wh[g & 1][i][e] - wl[g & 1][i][e]) << vdbits) | (uint32_t)d;
          key[u] = kv < key[u] ? kv : key[u];
        }
    });
  }

  int nout = o1 - o0 - wave;  // output rows left for this wave, from row k = 0
  __asm__ volatile("" : "+v"(nout));  // recompute the row tests here
#pragma unroll
  for (int h = 0; h < NB; ++h) {
    const int x = xo[h];
    if (x < 0 || x >= X) continue;
    uint32_t* kp = a.keys + ((size_t)(pair * a.nchunk + chunk) * 2 + (NB == 2 ? h : base)) * a.nk;
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
      const int r = o0 + wave + k * kWaves;
      if (k * kWaves < nout) {
        kp[(size_t)(ya + r) * X + x] = key[k * NB + h];
        // a debug run covers the single disparity dlo, so the key holds CA
        if (DBG && dbg && (NB == 1 || h == a.dbg_base))
          a.dbg_ca[(size_t)(ya + r) * X + x] = key[k * NB + h] >> a.dbits;
      }
    }
  }
}

// ----------------------------------------------------------------- k_wta
// Minimum key over the d-chunks for both bases: D = key & (2^dbits - 1)
// (Eq. 9; the key order makes the smallest d win ties), and the minimum
// aggregate key >> dbits when mincost != NULL.  Four pixels per thread; planes have the
// padded stride nk (a multiple of 64 pixels).
// grid: (ceil(nk / 1024), npair), block 256.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int16_t i16x4 __attribute__((ext_vector_type(4)));

// Minimum keys of four pixels over the chunks; kp the first chunk's, planes
// stride words apart.  Loads in groups of kWtaGroup chunks (of NB bases, stride / 2
// apart) in flight together; a group running past the last chunk reloads the
// last one, which leaves the minimum unchanged.
constexpr int kWtaGroup = 8;
template <int NB>
__device__ __forceinline__ void min_keys(const uint32_t* kp, int nchunk, size_t stride, u32x4 (&mb)[NB]) {
#pragma unroll
  for (int b = 0; b < NB; ++b) mb[b] = u32x4{0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu};
  for (int c0 = 0; c0 < nchunk; c0 += kWtaGroup) {
    u32x4 v[kWtaGroup][NB];
#pragma unroll
    for (int g = 0; g < kWtaGroup; ++g) {
      const int c = min(c0 + g, nchunk - 1);
#pragma unroll
      for (int b = 0; b < NB; ++b)
        __builtin_memcpy(&v[g][b], kp + (size_t)c * stride + (size_t)b * (stride / 2), 16);
    }
#pragma unroll
    for (int g = 0; g < kWtaGroup; ++g)
#pragma unroll
      for (int b = 0; b < NB; ++b) mb[b] = __builtin_elementwise_min(mb[b], v[g][b]);
  }
}

__global__ void __launch_bounds__(256) k_wta(const uint32_t* __restrict__ keys, int nchunk,
                                             int nk, int dbits, int16_t* __restrict__ disp,
                                             uint32_t* __restrict__ mincost) {
  const int i = (blockIdx.x * 256 + threadIdx.x) * 4;
  const int pair = blockIdx.y;
  if (i >= nk) return;
  const uint32_t* kp = keys + (size_t)pair * nchunk * 2 * nk + i;
  u32x4 mb[2];
  min_keys<2>(kp, nchunk, 2 * (size_t)nk, mb);
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const u32x4 m = mb[b];
    const size_t o = (size_t)(2 * pair + b) * nk + i;
    const uint32_t dm = (1u << dbits) - 1u;
    *reinterpret_cast<i16x4*>(disp + o) =
        i16x4{(int16_t)(m.x & dm), (int16_t)(m.y & dm), (int16_t)(m.z & dm), (int16_t)(m.w & dm)};
    if (mincost)
      *reinterpret_cast<u32x4*>(mincost + o) =
          u32x4{m.x >> dbits, m.y >> dbits, m.z >> dbits, m.w >> dbits};
  }
}

// -------------------------------------------------------------- k_refine
// One workgroup per half-res row.  GCP(x) = [x - k >= 0 and D^R(x - k) = k],
// k = D^L(x) (Eq. 10); M = 3x3 median of D^L (borders clamped); GCPs keep M;
// a non-GCP takes the nearest GCPs left (x-i) and right (x+j): linear
// interpolation from M(x-i) toward M(x+j), rounded half up, when they differ
// by at most T, else the side of strictly closer brightness (the right one on
// a tie) (Sec. III-E).  One side only: copy it; none: 0.  fill_mode 1 and 2
// are the two simpler fills Sec. III-E describes first: the GCP closer in
// distance (the right one at equal distance), or the smaller disparity.
// The rows are staged in LDS, the GCP flags of the row become a bit array
// (one wave ballot per 64 columns), and each non-GCP finds its nearest GCPs
// by bit search in that array.  The values go to filled (may be NULL) and, in
// full-resolution mode, where they are the map, to the output (as a kernel of
// its own that copy took 5 us at 1436x992).
// grid: (Y, npair), block 256.
__device__ __forceinline__ int floor_div_pos(int n, int d) {  // d > 0
  return n >= 0 ? n / d : -((-n + d - 1) / d);
}

__device__ __forceinline__ int median9(int* v) {
  // 19-comparator median-of-9 selection network (Paeth, Graphics Gems;
  // exhaustively checked on all 0/1 inputs by the test suite's CPU twin)
#define CS(i, j) { int lo = min(v[i], v[j]); int hi = max(v[i], v[j]); v[i] = lo; v[j] = hi; }
  CS(1, 2) CS(4, 5) CS(7, 8) CS(0, 1) CS(3, 4) CS(6, 7) CS(1, 2) CS(4, 5) CS(7, 8)
  CS(0, 3) CS(5, 8) CS(4, 7) CS(3, 6) CS(1, 4) CS(2, 5) CS(4, 7) CS(4, 2) CS(6, 4)
  CS(4, 2)
#undef CS
  return v[4];
}

// Value of column x of a row of X (bit x of gm set: a GCP), its medians med and
// grays h.
__device__ __forceinline__ int fill_value(const uint64_t* gm, const int16_t* med, const uint8_t* h,
                                          int x, int X, int T, int fill_mode) {
  const int wx = x >> 6, bx = x & 63, nw = (X + 63) >> 6;
  if ((gm[wx] >> bx) & 1ull) return med[x];
  int w = wx, xl = -1, xr = X;
  uint64_t mk = gm[w] & ((1ull << bx) - 1ull);            // columns < x
  while (mk == 0ull && w > 0) mk = gm[--w];
  if (mk) xl = w * 64 + 63 - __builtin_clzll(mk);
  w = wx;
  mk = bx == 63 ? 0ull : gm[w] & (~0ull << (bx + 1));     // columns > x
  while (mk == 0ull && w + 1 < nw) mk = gm[++w];
  if (mk) xr = w * 64 + __builtin_ctzll(mk);
  if (xl >= 0 && xr < X) {
    const int i = x - xl, j = xr - x, dla = med[xl], drb = med[xr];
    if (fill_mode == 1) return i < j ? dla : drb;
    if (fill_mode == 2) return min(dla, drb);
    if (iabs(dla - drb) <= T) return dla + floor_div_pos(2 * i * (drb - dla) + (i + j), 2 * (i + j));
    return iabs(h[xl] - h[x]) < iabs(h[xr] - h[x]) ? dla : drb;
  }
  return xl >= 0 ? med[xl] : xr < X ? med[xr] : 0;
}

// LDS bytes of a workgroup, by the row's width: with 45 kB for every width (4096
// columns) a CU held 12 waves.  8 pairs of 960x540 31.6 us before, 23.4 now; one of
// 1436x992 14.0 and 12.0; 718x496, where the grid does not fill the CUs, 6.1 and 6.3.
inline unsigned refine_lds(int X) { return (unsigned)((X + 63) / 64) * (8 + 64 * 11); }

__global__ void __launch_bounds__(256) k_refine(const int16_t* __restrict__ disp, int nk,
                                                const uint16_t* __restrict__ pk, int XP, int pad,
                                                int X, int Y, int T, int fill_mode,
                                                uint8_t* __restrict__ gcp_out,
                                                int16_t* __restrict__ med_out,
                                                int16_t* __restrict__ filled, PairPtrs pp,
                                                int full) {
  extern __shared__ uint64_t s_ref[];           // refine_lds(X) bytes, rows of P columns
  const int P = (X + 63) & ~63;
  uint64_t* s_gm = s_ref;                       // GCP flag of column x in bit x % 64 of word x / 64
  int16_t* s_d = reinterpret_cast<int16_t*>(s_gm + P / 64);  // 4 rows: D^L y-1, y, y+1 (clamped), D^R y
  int16_t* s_med = s_d + 4 * P;
  uint8_t* s_h = reinterpret_cast<uint8_t*>(s_med + P);      // left gray of row y
  const int y = blockIdx.x, pair = blockIdx.y, t = threadIdx.x;
  const size_t plane = (size_t)X * Y;
  const int16_t* dl = disp + (size_t)(2 * pair) * nk;
  const int16_t* dr = disp + (size_t)(2 * pair + 1) * nk;
  const uint16_t* pkr = pk + ((size_t)(2 * pair) * Y + y) * XP + pad;
  const size_t rm = (size_t)max(y - 1, 0) * X, r0 = (size_t)y * X, rp = (size_t)min(y + 1, Y - 1) * X;
  // stage the rows: four columns per thread and round, all loads of a round
  // issued before its stores (clamped columns load a valid value, not stored)
  for (int xb = 0; xb < X; xb += 1024) {
    int16_t a[4][4];
    uint32_t hp[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int x = min(xb + t + 256 * i, X - 1);
      a[i][0] = dl[rm + x];
      a[i][1] = dl[r0 + x];
      a[i][2] = dl[rp + x];
      a[i][3] = dr[r0 + x];
      hp[i] = pkr[x];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int x = xb + t + 256 * i;
      if (x < X) {
#pragma unroll
        for (int q = 0; q < 4; ++q) s_d[q * P + x] = a[i][q];
        s_h[x] = (uint8_t)hp[i];
      }
    }
  }
  __syncthreads();
  // cross-check and median; the GCP flags of 64 consecutive columns are one
  // wave's ballot
  for (int xb = 0; xb < X; xb += 256) {
    const int x = xb + t;
    bool g = false;
    if (x < X) {
      const int xm = max(x - 1, 0), xp = min(x + 1, X - 1);
      const int16_t *d1 = s_d + P, *d2 = d1 + P;
      int v[9] = {s_d[xm], s_d[x], s_d[xp], d1[xm], d1[x], d1[xp], d2[xm], d2[x], d2[xp]};
      const int k = v[4];
      g = x - k >= 0 && d2[P + x - k] == k;
      const int m = median9(v);
      s_med[x] = (int16_t)m;
      if (gcp_out) gcp_out[(size_t)pair * plane + r0 + x] = (uint8_t)g;
      if (med_out) med_out[(size_t)pair * plane + r0 + x] = (int16_t)m;
    }
    const uint64_t bal = __ballot(g);
    if ((t & 63) == 0 && x < X) s_gm[x >> 6] = bal;  // (words of the row only)
  }
  __syncthreads();
  // fill: the nearest GCPs left and right from the bit array
  for (int x = t; x < X; x += 256) {
    const int16_t v = (int16_t)fill_value(s_gm, s_med, s_h, x, X, T, fill_mode);
    if (filled) filled[(size_t)pair * plane + r0 + x] = v;
    if (full) pp.out[pair][r0 + x] = v;
  }
}

// ------------------------------------------------------------ k_gray_full
// Full-resolution mode (the method on the original images, Sec. V): the
// "half" image is the gray image itself.  grid: (ceil(W/256), H, 2 npair),
// block 256.
__global__ void __launch_bounds__(256) k_gray_full(PairPtrs pp, int W, int H,
                                                   uint8_t* __restrict__ half) {
  const int x = blockIdx.x * 256 + threadIdx.x, y = blockIdx.y, img = blockIdx.z;
  if (x >= W) return;
  const uint8_t* rgb = (img & 1) ? pp.right[img >> 1] : pp.left[img >> 1];
  half[(size_t)img * W * H + (size_t)y * W + x] = (uint8_t)gray_of(rgb + ((size_t)y * W + x) * 3);
}

// ------------------------------------------------------------- k_upscale
// One thread per 2x2 block of full-res output pixels (Step8).  Along x: even
// columns take 2 D+(x); an odd column between D+(x) and D+(x+1) takes their
// sum (the doubled midpoint) when they differ by at most T, else the doubled
// value of the side whose full-res gray is strictly closer (the right one on
// a tie); a last odd column copies.  Along y: odd rows are the rounded-up
// mean of the two neighbouring upscaled rows; a last odd row copies.
// grid: (ceil(X/64), ceil(Y/4), npair), block (64, 4).
// odd column between upscaled values 2*dlv and 2*drv; g0, g1, g2 are the
// full-res grays left of, at and right of it
__device__ __forceinline__ int up_odd(int dlv, int drv, const uint8_t* rgb_row, int xo, int T) {
  if (iabs(dlv - drv) <= T) return dlv + drv;
  const int g0 = gray_of(rgb_row + (xo - 1) * 3), g1 = gray_of(rgb_row + xo * 3),
            g2 = gray_of(rgb_row + (xo + 1) * 3);
  return iabs(g0 - g1) < iabs(g2 - g1) ? 2 * dlv : 2 * drv;
}

// Output pixels of half-res pixel (x, y); f0 and f1 are the filled rows y and
// y + 1.
__device__ __forceinline__ void up_block(const int16_t* f0, const int16_t* f1, const uint8_t* rgb,
                                         int16_t* out, int x, int y, int W, int H, int X, int Y, int T) {
  const int xo = 2 * x, yo = 2 * y;
  const bool hasr = x + 1 < X, hasd = y + 1 < Y;
  const int a = f0[x], b = hasr ? f0[x + 1] : a;
  // upscaled row y at columns 2x and 2x+1
  const int u0 = 2 * a;
  const int u1 = hasr ? up_odd(a, b, rgb + (size_t)yo * W * 3, xo + 1, T) : 2 * a;
  const bool odd_col = xo + 1 < W;
  out[(size_t)yo * W + xo] = (int16_t)u0;
  if (odd_col) out[(size_t)yo * W + xo + 1] = (int16_t)u1;
  if (yo + 1 < H) {
    int v0 = u0, v1 = u1;
    if (hasd) {
      const int c = f1[x], e = hasr ? f1[x + 1] : c;
      const int w0 = 2 * c;
      const int w1 = hasr ? up_odd(c, e, rgb + (size_t)(yo + 2) * W * 3, xo + 1, T) : 2 * c;
      v0 = (u0 + w0 + 1) >> 1;
      v1 = (u1 + w1 + 1) >> 1;
    }
    out[(size_t)(yo + 1) * W + xo] = (int16_t)v0;
    if (odd_col) out[(size_t)(yo + 1) * W + xo + 1] = (int16_t)v1;
  }
}

__global__ void __launch_bounds__(256) k_upscale(PairPtrs pp, const int16_t* __restrict__ filled,
                                                 int W, int H, int X, int Y, int T) {
  const int x = blockIdx.x * 64 + threadIdx.x;
  const int y = blockIdx.y * 4 + threadIdx.y;
  const int pair = blockIdx.z;
  if (x >= X || y >= Y) return;
  const int16_t* f = filled + ((size_t)pair * Y + y) * X;
  up_block(f, f + X, pp.left[pair], pp.out[pair], x, y, W, H, X, Y, T);
}

// ---------------------------------------------------------------- k_post
// k_wta, k_refine and k_upscale in one: a workgroup takes kPostRows half-res rows
// y0 .. of a pair, which need the filled rows y0 .. y0 + kPostRows, their medians
// D^L one row further on either side and their cross-check D^R, all in LDS.
// The rows that two workgroups need are reduced by both (8 rows of keys for
// every 2, where k_wta reads 4), so this pays while launches and latency count
// (kPostMaxPixels): 320x240 28.8 us a frame with three kernels, 23.7 with one;
// 640x480 45.2 and 41.8; 1237x823 84.1 and 83.5; 1436x992 105.4 and 105.2;
// 2872x1984 597 and 605; 8 pairs of 1920x1080 1466 and 1501.  1 or 4 rows, or 512
// threads, took 0.2 to 5 us more at all of the first four.
// grid: (ceil(Y / kPostRows), npair), block kPostThreads.
constexpr int kPostRows = 2, kPostThreads = 1024, kPostMaxX = 2048, kPostMaxPixels = 1 << 18;

__global__ void __launch_bounds__(kPostThreads) k_post(PairPtrs pp, const uint32_t* __restrict__ keys,
                                                       int nchunk, int nk, int dbits,
                                                       const uint16_t* __restrict__ pk, int XP, int pad,
                                                       int W, int H, int X, int Y, int T, int fill_mode) {
  constexpr int NF = kPostRows + 1, NL = NF + 2;  // filled rows, rows of D^L
  __shared__ int16_t s_d[NL + NF][kPostMaxX];     // D^L rows y0 - 1 .. (clamped), D^R rows y0 ..
  __shared__ int16_t s_med[NF][kPostMaxX];
  __shared__ uint8_t s_h[NF][kPostMaxX];
  __shared__ uint64_t s_gm[NF][kPostMaxX / 64];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int y0 = blockIdx.x * kPostRows, pair = blockIdx.y;
  const uint32_t dm = (1u << dbits) - 1u;
  // minima of four columns a thread (the last four again where X is no multiple)
  const int nq = (X + 3) / 4;
  const uint32_t* kp = keys + (size_t)pair * nchunk * 2 * nk;
  for (int i = t; i < (NL + NF) * nq; i += kPostThreads) {
    const int j = i / nq, x = min(4 * (i - j * nq), X - 4);
    const int y = j < NL ? clampi(y0 - 1 + j, 0, Y - 1) : min(y0 + j - NL, Y - 1);
    u32x4 m[1];
    min_keys<1>(kp + (j < NL ? 0 : nk) + (size_t)y * X + x, nchunk, 2 * (size_t)nk, m);
    s_d[j][x] = (int16_t)(m[0].x & dm);
    s_d[j][x + 1] = (int16_t)(m[0].y & dm);
    s_d[j][x + 2] = (int16_t)(m[0].z & dm);
    s_d[j][x + 3] = (int16_t)(m[0].w & dm);
  }
  const int nw = (X + 63) >> 6;
  for (int i = wave; i < NF * nw; i += kPostThreads / 64) {
    const int j = i / nw, x = (i - j * nw) * 64 + lane;
    if (x < X)
      s_h[j][x] = (uint8_t)pk[((size_t)(2 * pair) * Y + min(y0 + j, Y - 1)) * XP + pad + x];
  }
  __syncthreads();
  for (int i = wave; i < NF * nw; i += kPostThreads / 64) {
    const int j = i / nw, w = i - j * nw, x = w * 64 + lane;
    bool g = false;
    if (x < X) {
      const int xm = max(x - 1, 0), xp = min(x + 1, X - 1);
      int v[9] = {s_d[j][xm],     s_d[j][x],     s_d[j][xp],     s_d[j + 1][xm], s_d[j + 1][x],
                  s_d[j + 1][xp], s_d[j + 2][xm], s_d[j + 2][x], s_d[j + 2][xp]};
      const int k = v[4];
      g = x - k >= 0 && s_d[NL + j][x - k] == k;
      s_med[j][x] = (int16_t)median9(v);
    }
    const uint64_t bal = __ballot(g);
    if (lane == 0) s_gm[j][w] = bal;
  }
  __syncthreads();
  // the filled rows take the place of D^L's first ones
  for (int i = wave; i < NF * nw; i += kPostThreads / 64) {
    const int j = i / nw, x = (i - j * nw) * 64 + lane;
    if (x < X) s_d[j][x] = (int16_t)fill_value(s_gm[j], s_med[j], s_h[j], x, X, T, fill_mode);
  }
  __syncthreads();
  for (int i = wave; i < kPostRows * nw; i += kPostThreads / 64) {
    const int r = i / nw, x = (i - r * nw) * 64 + lane, y = y0 + r;
    if (x < X && y < Y) up_block(s_d[r], s_d[r + 1], pp.left[pair], pp.out[pair], x, y, W, H, X, Y, T);
  }
}

}  // namespace
}  // namespace stereo_dev
