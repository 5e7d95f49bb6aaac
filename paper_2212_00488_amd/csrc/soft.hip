// Host side of the soft-argmin head: plans, launch sequences and the C
// interface declared in include/stereo.h (stereo_soft_*).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "context.h"
#include "kernels.hip.h"
#include "soft.hip.h"
#include "stereo.h"

using namespace stereo_dev;

namespace stereo_host {

constexpr int kSoftMaxPairs = 64;
// The weight planes of all disparities of a plan and its dL/dCA_x planes: at most
// this many bytes each, so that 32-bit offsets reach every weight (k_soft_tcolw).
constexpr size_t kPlanesMost = (size_t(1) << 32) - 1;
// A slab's weight and dL/dCA_x planes, where the caller sets no slab.
constexpr size_t kSlabBudget = size_t(1) << 30;

struct SoftPlan {
  int n = 0, W = 0, H = 0, Dmax = 0, X = 0, Y = 0, D = 0;
  stereo_soft_params p{};
  int kmax = 8, nstrips = 0, nbands = 0, rows = 0;
  int csize = 1, nchunk = 0;   // k_soft_agg d-chunk size and forward chunk count
  int XS = 0, pads = 0, XA = 0;
  int XW = 0;          // row pitch of the weight and dL/dCA_x planes: whole 128-byte lines
  int fxk = 18;        // fixed-point bits of the costs
  int nds = 1;         // disparities per backward slab, and of the plan's own weight planes
  bool ca = false;     // a forward saves CA, not e_d (several slabs)
  size_t lam_count = 0;
  size_t bytes = 0;
  void* block = nullptr;
  float* half_f = nullptr;     // [2n][Y][X]
  uint8_t* half_u8 = nullptr;  // [2n][Y][X]
  uint32_t* arms = nullptr;    // [2n][Y][XA]
  uint2* sp = nullptr;         // [2n][Y][XS] padded {half value, census}
  float* inv_size = nullptr;   // [n][Y][X]
  float2* part = nullptr;      // [n][nchunk][Y][X]
  float4* pc = nullptr;        // [n][Y][X]
  float* wts = nullptr;        // [nds][n][Y][XW] e_d or CA
  // The weight planes of the disparities from nds on, an allocation of their own:
  // made by the first call that uses them (a forward that saves its weights, a
  // backward) where the scratch has room, and given back when it is wanted for
  // something else; without them a backward computes CA again, slab by slab.
  float* rest = nullptr;       // [D - nds][n][Y][XW]
  size_t rest_bytes = 0;       // of rest while it is there
  bool rest_captured = false;  // a captured graph uses rest: never given back
  uint64_t rest_retry = 0;     // after a failed allocation: not tried before this tick
  float* gcax = nullptr;       // [nds][n][Y][XW] dL/dCA_x
  float* gr_part = nullptr;    // [n][nstrips][Y][WP] right-gradient partials of a slab
  int WP = 0;                  // 64 + nds - 1 columns per partial row
  float* g_half = nullptr;     // [2n][Y][X]
  float2* lam_part = nullptr;  // [lam_count]
  // images of the last feature pass on this plan (STEREO_SOFT_F_REUSE_FEATURES)
  const float* feat_left = nullptr;
  const float* feat_right = nullptr;
  // inputs of the last forward, when it saved its weights e_d in the weight
  // planes (STEREO_SOFT_F_SAVE_WEIGHTS, planes of all D); any other forward, a
  // backward that recomputes the weights and the loss of rest clear wts_valid
  bool wts_valid = false;
  const float* wts_left = nullptr;
  const float* wts_right = nullptr;
  const float* wts_lam = nullptr;
  uint64_t last_use = 0, prev_use = 0;  // ticks of the last two calls
  hipStream_t owner = nullptr; // the stream the plan serves (plans are never shared
                               // between streams, so calls on two streams may overlap)
};

void free_soft_plans(std::vector<SoftPlan*>& plans) {
  for (SoftPlan* pl : plans) {
    if (pl->block) (void)hipFree(pl->block);
    if (pl->rest) (void)hipFree(pl->rest);
    delete pl;
  }
  plans.clear();
}

// Plans are shared by calls whose parameters differ in flags only.
bool same_soft(const stereo_soft_params& a, const stereo_soft_params& b) {
  return a.tau == b.tau && a.color_delta == b.color_delta && a.arm_x == b.arm_x &&
         a.arm_y == b.arm_y && a.slab == b.slab;
}

int soft_checks(stereo_ctx* c, int n, int W, int H, int Dmax, const stereo_soft_params* params,
                stereo_soft_params* p) {
  if (n < 1 || n > kSoftMaxPairs) return fail(c, STEREO_EINVAL, "n %d outside 1..%d", n, kSoftMaxPairs);
  if (W < 2 || H < 2 || W > STEREO_MAX_SIDE || H > STEREO_MAX_SIDE)
    return fail(c, STEREO_EINVAL, "image size %dx%d outside 2..%d", W, H, STEREO_MAX_SIDE);
  if (Dmax < 1 || Dmax > W || Dmax > STEREO_MAX_DMAX)
    return fail(c, STEREO_EINVAL, "Dmax %d outside 1..min(W=%d, %d)", Dmax, W, STEREO_MAX_DMAX);
  if (params) {
    if (params->size != sizeof(stereo_soft_params))
      return fail(c, STEREO_EINVAL, "params.size %u != %zu", params->size, sizeof(stereo_soft_params));
    *p = *params;
  } else {
    stereo_soft_default_params(p);
  }
  // exp2 of -mean / tau (log2 units) stays a normal float down to tau = 0.025
  if (!(p->tau >= 0.025f) || !std::isfinite(p->tau))
    return fail(c, STEREO_EINVAL, "tau must be finite and >= 0.025");
  if (p->color_delta < 0 || p->color_delta > 256)
    return fail(c, STEREO_EINVAL, "color_delta %d outside 0..256", p->color_delta);
  if (p->arm_x < 0 || p->arm_x > 31 || p->arm_y < 0 || p->arm_y > 63)
    return fail(c, STEREO_EINVAL, "soft head arm caps: arm_x in 0..31, arm_y in 0..63");
  if (p->slab < 0) return fail(c, STEREO_EINVAL, "slab must be >= 0");
  if (p->flags & ~(STEREO_SOFT_F_REUSE_FEATURES | STEREO_SOFT_F_SAVE_WEIGHTS))
    return fail(c, STEREO_EINVAL, "unknown flags");
  return 0;
}

// Modelled k_soft_agg time, in units of one disparity of one workgroup, for
// d-chunks of cs disparities: each XCD's workgroups, in order of their positions
// (chunk_at), go to dispatch queue (position % kXcdQueues), where each takes
// the CU of that queue that frees first; a workgroup costs its disparities
// plus ovh units of set-up and drain (arms, |S|, chunk sums).  The queue
// structure (4 queues of 8 CUs per XCD, filled in turn) is what timings of such
// placements showed on a kernel of this layout: a workgroup past the first round
// waits for a CU of its own queue, not for the first CU to free.
double agg_makespan(int groups, int D, int cs, int cus_per_xcd, double ovh) {
  const int nfull = D / cs, rem = D - nfull * cs, nchunk = nfull + (rem > 0);
  const int nloc = (groups + kXcds - 1) / kXcds, T = nloc * nchunk;
  const int per_q = std::max(1, cus_per_xcd / kXcdQueues);
  const bool stacked = nchunk != nfull && kXcdQueues * (nloc - 1) <= T - 1;
  double worst = 0.0;
  std::vector<double> cu((size_t)kXcdQueues * per_q);
  for (int x = 0; x < kXcds && x < groups; ++x) {
    std::fill(cu.begin(), cu.end(), 0.0);
    for (int j = 0; j < T; ++j) {
      int local, chunk;
      const int q = T - 1 - j;
      if (stacked && q % kXcdQueues == 0 && q / kXcdQueues < nloc) {
        local = nloc - 1 - q / kXcdQueues;
        chunk = nfull;
      } else if (stacked) {
        const int i = j - std::max(0, nloc - (q / kXcdQueues + 1));
        local = i / nfull;
        chunk = i - local * nfull;
      } else {
        local = j < nloc * nfull ? j / nfull : j - nloc * nfull;
        chunk = j < nloc * nfull ? j - local * nfull : nfull;
      }
      if (local * kXcds + x >= groups) continue;  // padding workgroup
      double* qb = cu.data() + (size_t)(j % kXcdQueues) * per_q;
      *std::min_element(qb, qb + per_q) += ovh + (chunk < nfull ? cs : rem);
    }
    worst = std::max(worst, *std::max_element(cu.begin(), cu.end()));
  }
  return worst;
}

// Chunk size with the shortest modelled time among ceil(D / n), n = 1..64,
// at most 16 workgroups per CU.  A workgroup's fixed cost (set-up, drain and
// the first disparity's cold reads) is taken as one disparity over
// kSetupRows band rows, a value fitted to an earlier kernel of this layout.  The
// forward at every chunk size of nine shapes: the pick is the fastest at 320x240,
// 640x480, 800x600, 1237x823 and 1436x992, 2% from it with 4 pairs of 1436x992 (15
// disparities, 396 us; 10, 389), 6% at 2872x1984 (19, 727 us; 12, 686), and 10%
// and 14% at 1920x1080 Dmax 256 (1 pair: 26, 244 us; 8, 222.  4 pairs: 32, 897 us;
// 16, 783).
constexpr double kSetupRows = 300.0;

int best_chunk_size(int groups, int D, int rows, int num_cu) {
  const int cus = std::max(1, num_cu / kXcds);
  const double ovh = kSetupRows / std::max(1, rows);
  int best = D;
  double best_t = 1e300;
  for (int n = 1; n <= std::min(D, 64); ++n) {
    const int cs = (D + n - 1) / n;
    if ((long)groups * ((D + cs - 1) / cs) > 16L * num_cu) break;
    const double t = agg_makespan(groups, D, cs, cus, ovh);
    if (t < best_t - 1e-9) {  // ties keep the larger chunks (fewer workgroups)
      best_t = t;
      best = cs;
    }
  }
  return best;
}

// Shape and launch geometry of a plan (host side only).
void soft_geometry(SoftPlan& pl, int num_cu) {
  const stereo_soft_params& p = pl.p;
  pl.X = (pl.W + 1) / 2; pl.Y = (pl.H + 1) / 2; pl.D = (pl.Dmax + 1) / 2;
  const int X = pl.X, Y = pl.Y, D = pl.D;
  // fixed point: (2 arm_x + 1)(2 arm_y + 1) costs of at most 2 stay below 2^31
  const double cells = (2.0 * p.arm_x + 1) * (2.0 * p.arm_y + 1);
  pl.fxk = (int)std::floor(std::log2(2147483648.0 / (2.0 * cells + 1.0)));
  pl.fxk = std::min(pl.fxk, 22);
  // k_soft_agg: one row-buffer pass (arm_x <= 31), bands whose output rows
  // fit 16 per thread and whose rows fit the plane
  int nb = 1, km = 8;
  for (;; ++nb) {
    const int ob = (Y + nb - 1) / nb;
    const int per = (ob + kWaves - 1) / kWaves;
    if (per > 16) continue;
    km = per <= 8 ? 8 : 16;
    const int rows = nb == 1 ? Y : ob + 2 * p.arm_y;
    const int o0max = nb == 1 ? 0 : p.arm_y;
    if (rows <= kAggRows && o0max + kWaves * km <= kAggRows) break;
  }
  pl.nbands = nb;
  pl.kmax = km;
  pl.rows = nb == 1 ? Y : std::min(Y, (Y + nb - 1) / nb + 2 * p.arm_y);
  pl.nstrips = (X + kTX - 1) / kTX;
  pl.XA = pl.nstrips * kTX;
  pl.XW = (X + 31) & ~31;
  // row loads reach x0 - hx - d .. x0 - hx + 127 for every strip x0
  pl.pads = ((128 + D + 2) + 1) & ~1;
  pl.XS = (pl.pads + pl.XA + 128 + 2 + 1) & ~1;
  const int groups = pl.nstrips * pl.nbands * pl.n;
  pl.csize = best_chunk_size(groups, D, pl.rows, num_cu);
  pl.nchunk = (D + pl.csize - 1) / pl.csize;
}

// Device bytes of a plan with weight planes and slabs of nds disparities.
size_t soft_bytes(const SoftPlan& pl, int nds) {
  auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
  const size_t n = pl.n, nimg = 2 * n, Y = pl.Y, npix = (size_t)pl.X * Y, nplane = (size_t)pl.XW * Y;
  const size_t nslab = (pl.D + nds - 1) / nds;
  return al(nimg * npix * 4) + al(nimg * npix) + al(nimg * Y * pl.XA * 4) +
         al(nimg * Y * pl.XS * 8) + al(n * npix * 4) + al(n * pl.nchunk * npix * 8) +
         al(n * npix * 16) + 2 * al(nds * n * nplane * 4) +
         al(nimg * npix * 4) + al(nslab * n * pl.nstrips * ((Y + kTrRows - 1) / kTrRows) * 8) +
         al(n * pl.nstrips * Y * (64 + nds - 1) * 4);
}

// Whether the weight planes may hold all disparities: the caller sets no slab and
// every weight can be addressed.
bool all_weights_allowed(const SoftPlan& pl) {
  return pl.p.slab == 0 && (size_t)pl.D * pl.n * pl.XW * pl.Y * 4 <= kPlanesMost;
}

// The slabs of a plan, the preferred one first: that of kSlabBudget, or the
// caller's (at most 128 disparities: k_soft_tr's LDS rows of right gradients).
// The others, half as large each, for where the cap or the device does not hold
// the scratch.
std::vector<int> soft_slabs(const SoftPlan& pl) {
  const size_t npix = (size_t)pl.X * pl.Y, nplane = (size_t)pl.XW * pl.Y, n = pl.n;
  const int D = pl.D, slab = pl.p.slab;
  const size_t budget = std::max<size_t>(1, kSlabBudget / (2 * n * npix * 4));
  int nds = std::min(slab > 0 ? std::min(slab, D) : (int)std::min<size_t>(D, budget), kTrMaxWP - 63);
  nds = (int)std::max<size_t>(1, std::min<size_t>(nds, kPlanesMost / (n * nplane * 4)));
  std::vector<int> v{nds};
  while (v.back() > 1) v.push_back((v.back() + 1) / 2);
  return v;
}

// A plan of the geometry geo with slabs of nds: its device memory, and its set-up
// enqueued on s.
int make_soft_plan(stereo_ctx* c, const SoftPlan& geo, int nds, hipStream_t s, SoftPlan** out) {
  const size_t bytes = soft_bytes(geo, nds);
  if (c->mem_cap && c->used + bytes > c->mem_cap)
    return fail(c, STEREO_ENOMEM, "soft plan needs %zu bytes, cap %zu, in use %zu", bytes,
                c->mem_cap, c->used);
  void* block = nullptr;
  hipError_t e = hipMalloc(&block, bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return fail(c, STEREO_ENOMEM, "hipMalloc(%zu): %s", bytes, hipGetErrorString(e));
  }
  SoftPlan* pl = new SoftPlan(geo);
  const int n = pl->n, Y = pl->Y, D = pl->D;
  const size_t npix = (size_t)pl->X * Y, nplane = (size_t)pl->XW * Y, nimg = 2 * (size_t)n;
  pl->block = block;
  pl->nds = nds;
  pl->WP = 64 + nds - 1;
  pl->lam_count = (size_t)((D + nds - 1) / nds) * n * pl->nstrips * ((Y + kTrRows - 1) / kTrRows);
  pl->bytes = bytes;
  char* cur = static_cast<char*>(pl->block);
  pl->half_f = carve<float>(cur, nimg * npix);
  pl->half_u8 = carve<uint8_t>(cur, nimg * npix);
  pl->arms = carve<uint32_t>(cur, nimg * Y * pl->XA);
  pl->sp = carve<uint2>(cur, nimg * Y * pl->XS);
  pl->inv_size = carve<float>(cur, n * npix);
  pl->part = carve<float2>(cur, (size_t)n * pl->nchunk * npix);
  pl->pc = carve<float4>(cur, n * npix);
  pl->wts = carve<float>(cur, (size_t)nds * n * nplane);
  pl->gcax = carve<float>(cur, (size_t)nds * n * nplane);
  pl->g_half = carve<float>(cur, nimg * npix);
  pl->lam_part = carve<float2>(cur, pl->lam_count);
  pl->gr_part = carve<float>(cur, (size_t)n * pl->nstrips * Y * pl->WP);
  // zero padding of the arm and pixel planes (kernels write the image part),
  // ordered on the plan's stream: no other stream is stalled
  hipLaunchKernelGGL(k_fill_f32, dim3(1024), dim3(256), 0, s, reinterpret_cast<float*>(pl->arms),
                     nimg * Y * pl->XA, 0.f);
  hipLaunchKernelGGL(k_fill_f32, dim3(1024), dim3(256), 0, s, reinterpret_cast<float*>(pl->sp),
                     nimg * Y * pl->XS * 2, 0.f);
  e = hipGetLastError();
  if (e != hipSuccess) {
    (void)hipFree(pl->block);
    delete pl;
    return fail(c, STEREO_EHIP, "soft plan initialisation: %s", hipGetErrorString(e));
  }
  c->used += bytes;
  *out = pl;
  return 0;
}

// Gives back the further weight planes of a plan (after the device has finished
// with them).
void drop_rest(stereo_ctx* c, SoftPlan& pl) {
  (void)hipDeviceSynchronize();
  (void)hipFree(pl.rest);
  c->used -= pl.rest_bytes;
  pl.rest = nullptr;
  pl.rest_bytes = 0;
  pl.wts_valid = false;
}

// Gives back the further weight planes of the least recently used plan that has
// some and was last used before the tick; false when there is none.
bool drop_one_rest(stereo_ctx* c, uint64_t before) {
  SoftPlan* lru = nullptr;
  for (SoftPlan* pl : c->soft_plans)
    if (pl->rest && !pl->rest_captured && pl->last_use < before &&
        (!lru || pl->last_use < lru->last_use))
      lru = pl;
  if (lru) drop_rest(c, *lru);
  return lru != nullptr;
}

size_t soft_optional_bytes(const stereo_ctx* c) {
  size_t b = 0;
  for (const SoftPlan* pl : c->soft_plans)
    if (!pl->rest_captured) b += pl->rest_bytes;
  return b;
}

bool drop_soft_optional(stereo_ctx* c) { return drop_one_rest(c, UINT64_MAX); }

// Whether the plan's weight planes hold all D disparities, for a call on s that
// would use them: those beyond a slab are allocated now if need be, where the
// scratch has room with the further planes given back of the plans not used
// since the tick `idle` (two shapes in turn do not take them from each other in
// every call).  Nothing is allocated while s is captured.
bool hold_all_weights(stereo_ctx* c, SoftPlan& pl, uint64_t idle, hipStream_t s) {
  if (pl.nds >= pl.D) return true;
  if (!pl.rest && (!all_weights_allowed(pl) || c->tick < pl.rest_retry)) return false;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  const bool capturing =
      hipStreamIsCapturing(s, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  if (pl.rest) {
    pl.rest_captured |= capturing;
    return true;
  }
  if (capturing) return false;
  const size_t bytes = (size_t)(pl.D - pl.nds) * pl.n * pl.XW * pl.Y * 4;
  bool failed = false;
  do {
    if (c->mem_cap && c->used + bytes > c->mem_cap) continue;
    void* block = nullptr;
    failed = hipMalloc(&block, bytes) != hipSuccess;
    if (!failed) {
      pl.rest = static_cast<float*>(block);
      pl.rest_bytes = bytes;
      c->used += bytes;
      return true;
    }
    (void)hipGetLastError();
  } while (drop_one_rest(c, idle));
  if (failed) pl.rest_retry = c->tick + 64;
  return false;
}

// Gives up the least recently used soft plan (after the device has finished with
// it); false when there is none.
bool evict_one_soft(stereo_ctx* c) {
  if (c->soft_plans.empty()) return false;
  const auto lru = std::min_element(c->soft_plans.begin(), c->soft_plans.end(),
                                    [](SoftPlan* a, SoftPlan* b) { return a->last_use < b->last_use; });
  std::vector<SoftPlan*> one{*lru};
  c->soft_plans.erase(lru);
  (void)hipDeviceSynchronize();
  c->used -= one[0]->bytes + one[0]->rest_bytes;
  free_soft_plans(one);
  return true;
}

// make_soft_plan, with the further weight planes of other soft plans given back,
// then those plans given up, while the scratch does not hold it.  A cap that
// would not hold it with all of them gone is left as it is.
int make_soft_plan_evicting(stereo_ctx* c, const SoftPlan& geo, int nds, hipStream_t s,
                            SoftPlan** out) {
  const size_t bytes = soft_bytes(geo, nds);
  size_t kept = c->used;
  for (const SoftPlan* pl : c->soft_plans) kept -= pl->bytes + pl->rest_bytes;
  if (c->mem_cap && kept + bytes > c->mem_cap)
    return fail(c, STEREO_ENOMEM, "soft plan needs %zu bytes, cap %zu, in use %zu", bytes,
                c->mem_cap, c->used);
  int rc = make_soft_plan(c, geo, nds, s, out);
  while (rc == STEREO_ENOMEM && (drop_soft_optional(c) || evict_one_soft(c)))
    rc = make_soft_plan(c, geo, nds, s, out);
  return rc;
}

int get_soft_plan(stereo_ctx* c, int n, int W, int H, int Dmax, const stereo_soft_params& p,
                  hipStream_t s, SoftPlan** out) {
  for (SoftPlan* pl : c->soft_plans)
    if (pl->n == n && pl->W == W && pl->H == H && pl->Dmax == Dmax && pl->owner == s &&
        same_soft(pl->p, p)) {
      pl->prev_use = pl->last_use;
      pl->last_use = ++c->tick;
      *out = pl;
      return 0;
    }
  SoftPlan geo, *pl = nullptr;
  geo.n = n; geo.W = W; geo.H = H; geo.Dmax = Dmax; geo.p = p;
  soft_geometry(geo, c->num_cu);
  // k_soft_agg addresses the pixel and arm planes through 32-bit buffer
  // offsets
  const size_t rows = (size_t)2 * n * geo.Y;
  if (rows * geo.XS * 8 >= (size_t(1) << 32) || rows * geo.XA * 4 >= (size_t(1) << 32))
    return fail(c, STEREO_EINVAL, "%d pairs of %dx%d exceed the 4 GiB pixel or arm planes of the "
                "soft head; pass fewer pairs per call", n, W, H);
  const std::vector<int> slabs = soft_slabs(geo);
  // One slab saves e_d; the terms of several are formed from CA itself, p_d =
  // 2^{-CA w - log2 sum e} in one rounding of the exponent, as they are when the
  // planes are computed again.
  geo.ca = slabs[0] < geo.D;
  int rc = STEREO_ENOMEM;
  for (int nds : slabs) {
    rc = make_soft_plan_evicting(c, geo, nds, s, &pl);
    if (rc != STEREO_ENOMEM) break;
  }
  if (rc) return rc;
  c->err.clear();
  pl->last_use = ++c->tick;
  pl->owner = s;
  c->soft_plans.push_back(pl);
  *out = pl;
  return 0;
}

// Features shared by forward and backward: float and uint8 half images,
// census and arms (k_feat of the integer path, which also writes the padded
// pixel planes), 1/|S|.
void soft_features(SoftPlan& pl, const float* left, const float* right, hipStream_t s) {
  pl.feat_left = left;
  pl.feat_right = right;
  const int X = pl.X, Y = pl.Y, n2 = 2 * pl.n;
  hipLaunchKernelGGL(k_soft_prep, dim3((X + 63) / 64, (Y + 3) / 4, n2), dim3(64, 4), 0, s, left,
                     right, pl.W, pl.H, X, Y, pl.half_f, pl.half_u8);
  hipLaunchKernelGGL(k_feat, dim3((X + 63) / 64, (Y + kFeatRows - 1) / kFeatRows, n2),
                     dim3(64, kFeatRows), 0, s, pl.half_u8, X, Y, pl.p.color_delta, pl.p.arm_x,
                     pl.p.arm_x, pl.p.arm_y, pl.XS, pl.pads, pl.XA, pl.half_f, pl.sp, pl.arms,
                     nullptr, nullptr, 0);
  hipLaunchKernelGGL(k_soft_size, dim3((X + 63) / 64, (Y + kSizeRows - 1) / kSizeRows, pl.n),
                     dim3(64, kSizeRows), 0, s, pl.arms, X, Y, pl.XA, pl.p.arm_y, pl.inv_size);
}

SoftArgs soft_args(const SoftPlan& pl, const float* lambdas, int dlo, int dhi, int csize) {
  SoftArgs a{};
  a.sp = pl.sp; a.arms = pl.arms; a.lam = lambdas; a.inv_size = pl.inv_size;
  a.X = pl.X; a.Y = pl.Y; a.XS = pl.XS; a.pads = pl.pads; a.XA = pl.XA; a.XW = pl.XW;
  a.arm_x = pl.p.arm_x; a.arm_y = pl.p.arm_y;
  a.nbands = pl.nbands; a.dlo = dlo; a.dhi = dhi;
  a.csize = std::max(1, std::min(csize, dhi - dlo));
  a.nchunk = (dhi - dlo + a.csize - 1) / a.csize;
  a.nstrips = pl.nstrips; a.ngroups = pl.nstrips * pl.nbands * pl.n; a.npair = pl.n;
  a.fx = std::ldexp(1.0f, pl.fxk);
  a.zc = (float)(std::ldexp(1.0, -pl.fxk) * 1.4426950408889634 / pl.p.tau);
  a.sp_bytes = (uint32_t)((size_t)2 * pl.n * pl.Y * pl.XS * 8);
  a.arms_bytes = (uint32_t)((size_t)2 * pl.n * pl.Y * pl.XA * 4);
  return a;
}

// k_soft_agg's weights of all disparities, in the plan's own planes and the rest.
void all_weights(const SoftPlan& pl, SoftArgs& a) {
  a.wts = pl.wts;
  // plane 0 of the rest is disparity nds
  a.wts2 = reinterpret_cast<float*>(reinterpret_cast<uintptr_t>(pl.rest) -
                                    (size_t)pl.nds * pl.n * pl.XW * pl.Y * sizeof(float));
  a.wlo = 0;
  a.wsplit = pl.nds;
}

// Most rows of a k_soft_agg band: the first and the last band have one halo.
int agg_rows(const SoftPlan& pl) {
  const int ob = (pl.Y + pl.nbands - 1) / pl.nbands;
  return pl.nbands == 1 ? pl.Y : std::min(pl.Y, ob + (pl.nbands == 2 ? 1 : 2) * pl.p.arm_y);
}

template <int KMAX, int SEG>
void launch_soft_agg_k(const SoftPlan& pl, const SoftArgs& a, hipStream_t s) {
  dim3 grid((unsigned)(((a.ngroups + kXcds - 1) / kXcds) * kXcds * a.nchunk));
  // the plane rows the band writes, or its window step reads
  const int o0max = pl.nbands == 1 ? 0 : pl.p.arm_y;
  const size_t lds = kAggRowBytes + (size_t)(std::max(agg_rows(pl), o0max + kWaves * KMAX) + 1) * 256;
  static const hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void*>(&k_soft_agg<KMAX, SEG>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
  (void)attr;  // were it refused, the launch fails and its error is reported
  hipLaunchKernelGGL((k_soft_agg<KMAX, SEG>), grid, dim3(kThreads), lds, s, a);
}

void launch_soft_agg(const SoftPlan& pl, const SoftArgs& a, hipStream_t s) {
  // rows of a wave's segment (whole pairs): 254 at most with 128 output rows,
  // 382 with 256
  const int seg = 2 * (((agg_rows(pl) + 1) / 2 + kWaves - 1) / kWaves);
  if (pl.kmax == 8) launch_soft_agg_k<8, 16>(pl, a, s);
  else if (seg <= 18) launch_soft_agg_k<16, 18>(pl, a, s);
  else launch_soft_agg_k<16, 24>(pl, a, s);
}

int soft_prologue(stereo_ctx* c, int n, int W, int H, int Dmax, const stereo_soft_params* params,
                  hipStream_t s, SoftPlan** pl, uint32_t* flags = nullptr) {
  stereo_soft_params p;
  int rc = soft_checks(c, n, W, H, Dmax, params, &p);
  if (rc) return rc;
  if (flags) *flags = p.flags;
  HIP_TRY(c, hipSetDevice(c->device));
  return get_soft_plan(c, n, W, H, Dmax, p, s, pl);
}

constexpr int kL1Blocks = 256;  // partial-sum blocks per pair

// L1 scratch of the context for the stream s: partials [kSoftMaxPairs][kL1Blocks],
// counts [kSoftMaxPairs], loss [1]; one block per stream (made on first use),
// so losses on two streams never share partial sums.
int l1_scratch(stereo_ctx* c, hipStream_t s, float2** part, float** counts, float** loss) {
  void* block = nullptr;
  for (const auto& b : c->l1_blocks)
    if (b.first == s) block = b.second;
  if (!block) {
    const size_t bytes = (size_t)kSoftMaxPairs * (kL1Blocks * 8 + 4) + 1024;
    hipError_t e = hipMalloc(&block, bytes);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return fail(c, STEREO_ENOMEM, "hipMalloc(%zu): %s", bytes, hipGetErrorString(e));
    }
    c->l1_blocks.emplace_back(s, block);
  }
  char* cur = static_cast<char*>(block);
  *part = carve<float2>(cur, (size_t)kSoftMaxPairs * kL1Blocks);
  *counts = carve<float>(cur, kSoftMaxPairs);
  *loss = carve<float>(cur, 1);
  return 0;
}

int l1_checks(stereo_ctx* c, int n, int W, int H) {
  if (n < 1 || n > kSoftMaxPairs) return fail(c, STEREO_EINVAL, "n %d outside 1..%d", n, kSoftMaxPairs);
  if (W < 2 || H < 2 || W > STEREO_MAX_SIDE || H > STEREO_MAX_SIDE)
    return fail(c, STEREO_EINVAL, "image size %dx%d outside 2..%d", W, H, STEREO_MAX_SIDE);
  HIP_TRY(c, hipSetDevice(c->device));
  return 0;
}

void l1_reduce(int n, int W, int H, const float* d_hat, const int16_t* gt, const uint8_t* nonocc,
               float2* part, float* counts, float* loss, hipStream_t s) {
  const int X = (W + 1) / 2, Y = (H + 1) / 2;
  hipLaunchKernelGGL(k_l1_partial, dim3(kL1Blocks, n), dim3(256), 0, s, d_hat, gt, nonocc, W, H,
                     X, Y, part);
  hipLaunchKernelGGL(k_l1_final, dim3(1), dim3(256), 0, s, part, kL1Blocks, n, loss, counts);
}

}  // namespace stereo_host

using namespace stereo_host;

extern "C" {

void stereo_soft_default_params(stereo_soft_params* p) {
  if (!p) return;
  std::memset(p, 0, sizeof *p);
  p->size = sizeof(stereo_soft_params);
  p->tau = 0.1f;
  p->color_delta = 13;
  p->arm_x = 21;
  p->arm_y = 31;
  p->slab = 0;
  p->flags = 0;
}

int stereo_soft_forward(stereo_ctx* c, const float* left, const float* right, int n, int W, int H,
                        int Dmax, const float* lambdas, const stereo_soft_params* params,
                        float* d_hat, float* lse2, hipStream_t stream) {
  if (!c) return STEREO_EINVAL;
  c->err.clear();
  if (!left || !right || !lambdas || !d_hat || !lse2) return fail(c, STEREO_EINVAL, "null pointer");
  SoftPlan* pl = nullptr;
  uint32_t flags = 0;
  int rc = soft_prologue(c, n, W, H, Dmax, params, stream, &pl, &flags);
  if (rc) return rc;
  soft_features(*pl, left, right, stream);
  SoftArgs a = soft_args(*pl, lambdas, 0, pl->D, pl->csize);
  a.part = pl->part;
  a.ca = pl->ca;
  pl->wts_valid = (flags & STEREO_SOFT_F_SAVE_WEIGHTS) &&
                  hold_all_weights(c, *pl, pl->prev_use, stream);
  if (pl->wts_valid) {
    all_weights(*pl, a);
    pl->wts_left = left;
    pl->wts_right = right;
    pl->wts_lam = lambdas;
  }
  launch_soft_agg(*pl, a, stream);
  const int npix = pl->X * pl->Y;
  hipLaunchKernelGGL(k_soft_merge, dim3((npix + 255) / 256, pl->n), dim3(256), 0, stream, pl->part,
                     pl->nchunk, npix, d_hat, lse2);
  return launch_status(c);
}

int stereo_soft_backward(stereo_ctx* c, const float* left, const float* right, int n, int W,
                         int H, int Dmax, const float* lambdas, const stereo_soft_params* params,
                         const float* d_hat, const float* lse2, const float* g_dhat,
                         float* g_left, float* g_right, float* g_lambdas, hipStream_t stream) {
  if (!c) return STEREO_EINVAL;
  c->err.clear();
  if (!left || !right || !lambdas || !d_hat || !lse2 || !g_dhat || !g_left || !g_right ||
      !g_lambdas)
    return fail(c, STEREO_EINVAL, "null pointer");
  SoftPlan* pl = nullptr;
  uint32_t flags = 0;
  int rc = soft_prologue(c, n, W, H, Dmax, params, stream, &pl, &flags);
  if (rc) return rc;
  const int X = pl->X, Y = pl->Y, npix = X * Y;
  const bool reuse = (flags & STEREO_SOFT_F_REUSE_FEATURES) != 0;
  if (!reuse || pl->feat_left != left || pl->feat_right != right)
    soft_features(*pl, left, right, stream);
  // the forward's weights of these inputs are on the plan, or are computed again
  const bool saved = reuse && pl->wts_valid && pl->wts_left == left && pl->wts_right == right &&
                     pl->wts_lam == lambdas;
  const float zc = (float)(std::ldexp(1.0, -pl->fxk) * 1.4426950408889634 / pl->p.tau);
  hipLaunchKernelGGL(k_soft_bprep, dim3((npix + 255) / 256, pl->n), dim3(256), 0, stream,
                     pl->inv_size, lse2, d_hat, g_dhat, npix, zc, 1.f / pl->p.tau, pl->pc);
  const int groups = pl->nstrips * pl->nbands * pl->n;
  const int tb = tcol_band(pl->p.arm_y);
  const int base = pl->nstrips * ((Y + tb - 1) / tb) * pl->n;
  // weight planes of all D: computed once (no other plan's are given back for it)
  const bool whole = hold_all_weights(c, *pl, 0, stream);
  if (!saved) pl->wts_valid = false;  // the planes are overwritten below
  auto weights = [&](int dlo, int dhi) {
    SoftArgs a = soft_args(*pl, lambdas, dlo, dhi,
                           best_chunk_size(groups, dhi - dlo, pl->rows, c->num_cu));
    if (whole) {
      all_weights(*pl, a);
    } else {
      a.wts = pl->wts;
      a.wlo = dlo;
      a.wsplit = dhi;
    }
    a.ca = 1;
    launch_soft_agg(*pl, a, stream);
  };
  if (!saved && whole) weights(0, pl->D);
  int slab = 0;
  const int lam_slab = pl->nstrips * ((Y + kTrRows - 1) / kTrRows) * pl->n;
  for (int dlo = 0; dlo < pl->D; dlo += pl->nds, ++slab) {
    const int dhi = std::min(pl->D, dlo + pl->nds);
    if (!saved && !whole) weights(dlo, dhi);
    TcwArgs tc{};
    const bool further = whole && dlo > 0;  // this slab's weights are in the rest
    tc.wts = further ? pl->rest : pl->wts; tc.wlo = further ? pl->nds : dlo;
    tc.wts_bytes = (uint32_t)(further ? pl->rest_bytes : (size_t)pl->nds * pl->n * pl->XW * Y * 4);
    tc.pc = pl->pc; tc.arms = pl->arms; tc.gcax = pl->gcax;
    tc.X = X; tc.Y = Y; tc.XA = pl->XA; tc.XW = pl->XW; tc.arm_y = pl->p.arm_y; tc.npair = pl->n;
    tc.dlo = dlo; tc.dhi = dhi;
    // disparity groups so that the grid fills the CUs about three blocks deep
    // (each group reloads the per-pixel constants: at 4 x 718x496, 4 groups
    // ran faster than 3 or 6)
    tc.ndg = std::max(1, std::min(dhi - dlo, (3 * c->num_cu + base - 1) / base));
    const dim3 tg((unsigned)((base * tc.ndg + kXcds - 1) / kXcds * kXcds));
    if (saved && !pl->ca) hipLaunchKernelGGL(k_soft_tcolw<false>, tg, dim3(64 * kTcwWaves), 0, stream, tc);
    else hipLaunchKernelGGL(k_soft_tcolw<true>, tg, dim3(64 * kTcwWaves), 0, stream, tc);
    TrArgs ta{};
    ta.gcax = pl->gcax; ta.arms = pl->arms; ta.sp = pl->sp; ta.lam = lambdas;
    ta.g_half = pl->g_half; ta.gr_part = pl->gr_part;
    ta.lam_part = pl->lam_part + (size_t)slab * lam_slab;
    ta.X = X; ta.Y = Y; ta.XS = pl->XS; ta.pads = pl->pads; ta.XA = pl->XA; ta.XW = pl->XW;
    ta.npair = pl->n; ta.dlo = dlo; ta.dhi = dhi; ta.WP = pl->WP;
    ta.nstrips = pl->nstrips;
    ta.first = dlo == 0;  // the first slab writes every half-image gradient
    hipLaunchKernelGGL(k_soft_tr, dim3((unsigned)((lam_slab + kXcds - 1) / kXcds * kXcds)), dim3(256), 0,
                       stream, ta);
    hipLaunchKernelGGL(k_soft_gright, dim3((X + 255) / 256, Y, pl->n), dim3(256), 0, stream,
                       pl->gr_part, pl->nstrips, pl->WP, dlo, dhi, X, Y, (int)(dlo == 0),
                       pl->g_half);
  }
  hipLaunchKernelGGL(k_soft_gfull, dim3((W + 255) / 256, H, 2 * pl->n), dim3(256), 0, stream,
                     pl->g_half, W, H, X, Y, g_left, g_right);
  hipLaunchKernelGGL(k_soft_lam, dim3(1), dim3(1024), 0, stream, pl->lam_part, slab * lam_slab,
                     g_lambdas);
  return launch_status(c);
}

int stereo_soft_l1_loss(stereo_ctx* c, const float* d_hat, const int16_t* gt,
                        const uint8_t* nonocc, int n, int W, int H, float* loss,
                        hipStream_t stream) {
  if (!c) return STEREO_EINVAL;
  c->err.clear();
  if (!d_hat || !gt || !nonocc || !loss) return fail(c, STEREO_EINVAL, "null pointer");
  int rc = l1_checks(c, n, W, H);
  if (rc) return rc;
  float2* part;
  float *counts, *scratch_loss;
  rc = l1_scratch(c, stream, &part, &counts, &scratch_loss);
  if (rc) return rc;
  l1_reduce(n, W, H, d_hat, gt, nonocc, part, counts, loss, stream);
  return launch_status(c);
}

int stereo_soft_l1_grad(stereo_ctx* c, const float* d_hat, const int16_t* gt,
                        const uint8_t* nonocc, int n, int W, int H, const float* gscale,
                        float* g_dhat, hipStream_t stream) {
  if (!c) return STEREO_EINVAL;
  c->err.clear();
  if (!d_hat || !gt || !nonocc || !g_dhat) return fail(c, STEREO_EINVAL, "null pointer");
  int rc = l1_checks(c, n, W, H);
  if (rc) return rc;
  float2* part;
  float *counts, *scratch_loss;
  rc = l1_scratch(c, stream, &part, &counts, &scratch_loss);
  if (rc) return rc;
  l1_reduce(n, W, H, d_hat, gt, nonocc, part, counts, scratch_loss, stream);
  const int X = (W + 1) / 2, Y = (H + 1) / 2, npix = X * Y;
  hipLaunchKernelGGL(k_l1_grad, dim3((npix + 255) / 256, n), dim3(256), 0, stream, d_hat, gt,
                     nonocc, counts, gscale, W, H, X, Y, n, g_dhat);
  return launch_status(c);
}

}  // extern "C"
