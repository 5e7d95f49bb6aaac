// Host side of the stereo library: context, per-shape plans, launches and
// the C interface declared in include/stereo.h.
#include "stereo.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "context.h"
#include "kernels.hip.h"
#include "pipeline.h"

using namespace stereo_dev;

// Fixed scratch of stereo_disparity_noalloc: one array per device, allocated
// when the code object is loaded on that device and held until the process
// ends.  Host code never uses its name as an address: the device address of
// each device's copy comes from hipGetSymbolAddress (noalloc_scratch_of).
constexpr size_t kNoallocBytes = size_t(STEREO_NOALLOC_MAX_BYTES);
static __device__ __align__(256) uint8_t scratch[kNoallocBytes];

namespace stereo_host {

// Device address of `scratch` on `device` (the current device), looked up
// once per device; null with *err set when the lookup failed.
void* noalloc_scratch_of(int device, std::string* err) {
  static std::mutex mu;
  static std::vector<void*> addr;
  static std::vector<std::string> why;
  std::lock_guard<std::mutex> lock(mu);
  if ((size_t)device >= addr.size()) {
    addr.resize(device + 1, nullptr);
    why.resize(device + 1);
  }
  if (!addr[device] && why[device].empty()) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e == hipSuccess && ptr) {
      addr[device] = ptr;
    } else {
      (void)hipGetLastError();
      why[device] = std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e);
    }
  }
  *err = why[device];
  return addr[device];
}

// Cost tables of Eq. 4 and Eq. 5 in fixed point: S(1 - exp(-t)) rounded half
// up, with t = (a / 255) / lambda_AD for brightness difference a and
// t = h / lambda_MC for census Hamming distance h.
void build_tables(const stereo_params& p, uint16_t ad[256], uint16_t mc[7]) {
  const double S = p.cost_scale, lad = p.lambda_ad, lmc = p.lambda_mc;
  for (int a = 0; a < 256; ++a) ad[a] = (uint16_t)std::floor(S * (1.0 - std::exp(-(a / 255.0) / lad)) + 0.5);
  for (int h = 0; h < 7; ++h) mc[h] = (uint16_t)std::floor(S * (1.0 - std::exp(-h / lmc)) + 0.5);
}


bool same_params(const stereo_params& a, const stereo_params& b) {
  return a.lambda_ad == b.lambda_ad && a.lambda_mc == b.lambda_mc && a.cost_scale == b.cost_scale &&
         a.color_delta == b.color_delta && a.arm_x == b.arm_x && a.arm_y == b.arm_y &&
         a.fill_T == b.fill_T && a.arm_x_r == b.arm_x_r && a.fill_mode == b.fill_mode &&
         (a.flags & STEREO_F_FULL_RES) == (b.flags & STEREO_F_FULL_RES);
}

bool full_res(const stereo_params& p) { return (p.flags & STEREO_F_FULL_RES) != 0; }

// Bits of the disparity field of the winner-take-all keys: enough for D - 1.
int key_dbits(int D) {
  int b = 1;
  while ((1 << b) < D) ++b;
  return b;
}

}  // namespace stereo_host

namespace stereo_host {

// Checks p for a search range of D disparities (D >= 1); resolves arm_x_r.
int check_params(stereo_ctx* c, stereo_params& p, int D) {
  if (p.size != sizeof(stereo_params))
    return fail(c, STEREO_EINVAL, "params.size %u != %zu", p.size, sizeof(stereo_params));
  if (!(p.lambda_ad > 0.f) || !std::isfinite(p.lambda_ad) || !(p.lambda_mc > 0.f) ||
      !std::isfinite(p.lambda_mc))
    return fail(c, STEREO_EINVAL, "lambda_ad and lambda_mc must be finite and > 0");
  if (p.cost_scale < 1 || p.cost_scale > 1024)
    return fail(c, STEREO_EINVAL, "cost_scale %d outside 1..1024", p.cost_scale);
  if (p.color_delta < 0 || p.color_delta > 256)
    return fail(c, STEREO_EINVAL, "color_delta %d outside 0..256", p.color_delta);
  if (p.arm_x_r == -1) p.arm_x_r = p.arm_x;
  if (p.arm_x < 0 || p.arm_x > 127 || p.arm_y < 0 || p.arm_y > 127 || p.arm_x_r < 0 ||
      p.arm_x_r > 127)
    return fail(c, STEREO_EINVAL, "arm caps must be in 0..127 (arm_x_r: -1 or 0..127)");
  if (p.fill_mode < 0 || p.fill_mode > 2) return fail(c, STEREO_EINVAL, "fill_mode %d outside 0..2", p.fill_mode);
  if (p.fill_T < 0 || p.fill_T > 1023) return fail(c, STEREO_EINVAL, "fill_T outside 0..1023");
  uint16_t ad[256], mc[7];
  build_tables(p, ad, mc);
  const double cmax = (double)ad[255] + mc[6];
  const int ax = std::max(p.arm_x, p.arm_x_r), dbits = key_dbits(D);
  const double bound = (2.0 * ax + 1) * (2.0 * p.arm_y + 1) * cmax;
  if (bound >= std::ldexp(1.0, 32 - dbits))
    return fail(c, STEREO_EINVAL,
                "(2 arm_x + 1)(2 arm_y + 1) C_max = %.0f must be < 2^%d for D = %d "
                "(lower cost_scale or the arm caps)", bound, 32 - dbits, D);
  return 0;
}

void free_plan(Plan* pl) {
  if (!pl) return;
  if (pl->block) (void)hipFree(pl->block);
  if (pl->dbg_block) (void)hipFree(pl->dbg_block);
  delete pl;
}


// KMAX (output rows per k_match thread and base) of the instance for `rows`
// of them with nbase bases; -1 when there is none.
int match_kmax(int rows, int nbase) {
  if (nbase == 2) {
    for (int s : {4, 8, 12, 16, 18})
      if (rows <= s) return s;
  } else {
    for (int s : {16, 36})
      if (rows <= s) return s;
  }
  return -1;
}

// Row bands of k_match with nbase bases a workgroup, nb at least.  The rows of
// a band (halos included; the first and the last band have one) fit the plane
// and the segment sums, and its window step, which reads plane rows up to
// o0 + 16 KMAX (padding rows included, o0 <= arm_y is the top halo), stays in
// the plane.
struct Bands {
  int n, kmax, rows, out;  // bands, KMAX, most rows of a band, its output rows
  long total;              // rows of all bands
};

Bands match_bands(int Y, int arm_y, int ns, int nbase, int nb) {
  const int pr = match_plane_rows(ns, nbase);
  for (;; ++nb) {
    const int ob = (Y + nb - 1) / nb, km = match_kmax((ob + kWaves - 1) / kWaves, nbase);
    if (km < 0 || ob * (nb - 1) >= Y) continue;
    int rows = 0;
    long total = 0;
    for (int b = 0; b < nb; ++b) {
      const int r = std::min(Y, std::min(Y, (b + 1) * ob) + arm_y) - std::max(0, b * ob - arm_y);
      rows = std::max(rows, r);
      total += r;
    }
    const int o0max = nb == 1 ? 0 : arm_y;
    if (rows <= kWaves * match_seg_rows(nbase) && rows + 1 <= pr && o0max + kWaves * km + 1 <= pr)
      return Bands{nb, km, rows, ob, total};
  }
}

// Whether bands of both bases exist at all: one output row between two halos,
// and the window step of the smallest instance below one.
bool bands_exist(int arm_y, int ns) {
  const int pr = match_plane_rows(ns, 2);
  return arm_y + kWaves * match_kmax(1, 2) + 1 <= pr && 2 * arm_y + 2 <= pr &&
         2 * arm_y + 1 <= kWaves * match_seg_rows(2);
}

// The workgroups of D disparities in nchunk chunks (kernels.hip.h, MatchGrid).
MatchGrid match_grid(const Plan& pl, int npair, int D0, int D1, int nchunk) {
  MatchGrid g{};
  g.nfull = (pl.X + kTX - 1) / kTX;
  g.units = pl.nbands * npair * (3 - pl.nbase);
  g.total = g.nfull * g.units * nchunk;
  if (pl.nbase == 2) {
    const int hi = match_slack_hi(pl.ns, std::max(pl.p.arm_x, pl.p.arm_x_r)), nd = D1 - D0;
    for (int s = g.nfull; g.nextra < kMatchExtra; ++s) {
      int c = 0;  // first chunk whose right-based strip s starts left of X
      while (c < nchunk && s * kTX - match_delta(D0 + (c + 1) * nd / nchunk - 1, hi) >= pl.X) ++c;
      if (c == nchunk) break;
      g.first[g.nextra++] = c;
      g.total += g.units * (nchunk - c);
    }
  }
  g.per = (g.total + kXcds - 1) / kXcds;
  return g;
}

// Modelled k_match time, in units of one band row of one disparity: every XCD
// has g.per workgroups for its CUs (in rounds, since they are nearly equal),
// each its set-up and drain (cost table, arms, key stores), and per disparity
// the rows and the output rows' window step; then k_wta's pass over the keys.
// The weights are fitted to timings of every chunk count with 1 to 8 bands at
// 320x240, 640x480, 800x600, 1237x823, 1436x992 (also at full resolution with
// arms 41 and 61), 2872x1984 and 4 x 1920x1080: the pick is within 4% of the
// fastest k_match at each (a unit is about 19 ns).
double match_time(const Plan& pl, const Bands& b, const MatchGrid& g, int nchunk, int num_cu) {
  constexpr double kSetup = 300.0, kWindow = 0.7, kKeys = 0.85e-4;
  const int cus = std::max(1, num_cu / kXcds), size = (pl.D + nchunk - 1) / nchunk;
  const int rounds = (g.per + cus - 1) / cus;
  return rounds * (kSetup + size * (b.rows + kWindow * b.out)) +
         kKeys * nchunk * pl.npair * pl.X * pl.Y;
}

// Launch geometry: bands keep the k_match LDS plane, the segment sums and the
// key registers within bounds; d-chunks, and more bands than needed, raise
// the workgroup count to fill the CUs.  nbase: 2 both bases a workgroup where
// that is the better form, 1 one base.  forced_nchunk: the number of chunks (at
// least as many as the strips need), or 0 for the modelled one.
void plan_geometry(Plan& pl, int num_cu, int forced_nchunk, int nbase) {
  const int arm = std::max(pl.p.arm_x, pl.p.arm_x_r), arm_y = pl.p.arm_y;
  // Both bases in one workgroup, with the fewest 128-column sub-passes that
  // leave their strips room for chunks of kMinChunk disparities, unless the
  // halo rows of the lower bands outweigh the shared evaluation: the two
  // forms' instructions per band row are about 26 and 2 x 23
  constexpr int kMinChunk = 6;
  constexpr double kBothRows = 1.7;  // rows of both bases that cost as much as two of one base
  const int ns1 = (66 + 2 * arm + 127) / 128;
  auto cap_of = [&](int ns) { return match_slack_lo(arm) + match_slack_hi(ns, arm) + 1; };
  int ns2 = 1;
  while (ns2 < 3 && (match_slack_hi(ns2, arm) < 0 || cap_of(ns2) < std::min(kMinChunk, pl.D))) ++ns2;
  pl.nbase = 1;
  pl.ns = ns1;
  pl.ccap = pl.D;
  const Bands one = match_bands(pl.Y, arm_y, ns1, 1, 1);
  if (nbase == 2 && bands_exist(arm_y, ns2) &&
      (double)match_bands(pl.Y, arm_y, ns2, 2, 1).total * ns2 <= kBothRows * one.total * ns1) {
    pl.nbase = 2;
    pl.ns = ns2;
    pl.ccap = cap_of(ns2);
  }
  // bands and d-chunks with the shortest modelled time (ties keep the fewer
  // bands and the larger chunks)
  double best_t = 1e300;
  constexpr int kMoreBands = 6;
  int nb = 1, best_nb = 1;
  for (int k = 0; k < kMoreBands && nb <= pl.Y; ++k, ++nb) {
    const Bands b = match_bands(pl.Y, arm_y, pl.ns, pl.nbase, nb);
    nb = pl.nbands = b.n;
    int n0 = (pl.D + pl.ccap - 1) / pl.ccap, n1 = std::min(pl.D, std::max(n0, 64));
    if (forced_nchunk > 0) n0 = n1 = std::max(n0, forced_nchunk);
    for (int n = n0; n <= n1; ++n) {
      const MatchGrid g = match_grid(pl, pl.npair, 0, pl.D, n);
      if (g.total > 16L * num_cu && best_t < 1e300) break;
      const double t = match_time(pl, b, g, n, num_cu);
      if (t < best_t - 1e-9) {
        best_t = t;
        best_nb = b.n;
        pl.kmax = b.kmax;
        pl.brows = b.rows;
        pl.nchunk = n;
        pl.model_t = t;
      }
    }
  }
  pl.nbands = best_nb;
  pl.csize = (pl.D + pl.nchunk - 1) / pl.nchunk;
  // pk padding covers every column a k_match lane loads: x0 - hx - D at the
  // left, x0 - hx + 128 NS + D (one base; both: x0 - hx + 128 NS with x0 <
  // X + D) at the right, one more in the shifted copy; pad and the pitch are
  // even, so the pair of columns from an even column is an aligned 32-bit word
  pl.pad = ((128 * pl.ns + pl.D + 2) + 3) & ~3;
  pl.XP = (pl.X + 2 * pl.pad + 63) & ~63;
  pl.XA = (pl.X + kTX - 1) / kTX * kTX;
}

// The number of d-chunks stereo_autotune chose for this shape and parameters, or 0.
int tuned_nchunk(const stereo_ctx* c, int W, int H, int Dmax, int npair, const stereo_params& p) {
  for (const Tuned& t : c->tuned)
    if (t.W == W && t.H == H && t.Dmax == Dmax && t.npair == npair && same_params(t.p, p))
      return t.nchunk;
  return 0;
}

// Device bytes of a plan's block and of its pixel (pk, both copies) and arm
// planes, for the geometry already in pl.
struct PlanBytes {
  size_t total, pk, arms;  // arms: each of the arms and xoff planes
};

PlanBytes plan_bytes(const Plan& pl) {
  auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
  const size_t n = (size_t)pl.X * pl.Y, npair = pl.npair;
  const size_t npk = (size_t)2 * npair * pl.Y * pl.XP;
  const size_t nar = (size_t)2 * npair * pl.Y * pl.XA;
  const size_t nk = pl.nk;
  PlanBytes b;
  b.pk = 2 * npk * 2;
  b.arms = nar * 4;
  b.total = al(2 * npair * n) + al(b.pk) + 2 * al(b.arms) + al(kTab * 2) +
            al((size_t)npair * pl.nchunk * 2 * nk * 4) + al(2 * npair * nk * 2) +
            al(2 * npair * nk * 4) + al(npair * n) + al(npair * n * 2) + al(npair * n * 2);
  return b;
}

// Launch geometries of a shape, the first the preferred one: both bases a
// workgroup or one base (whose chunks may hold all disparities), the chunks of
// the shortest modelled time or as few as the strips allow (fewer keys).
struct Form {
  int nbase;
  bool fewest_chunks;
};
constexpr Form kForms[] = {{2, false}, {2, true}, {1, false}, {1, true}};

// Shape, tables and launch geometry of a plan (host side only, no device
// memory); rejects shapes whose pixel or arm planes the kernels' 32-bit
// buffer offsets cannot address.
int plan_setup(stereo_ctx* c, Plan& pl, int W, int H, int Dmax, const stereo_params& p,
               int npair, const Form& form) {
  pl.W = W; pl.H = H; pl.Dmax = Dmax; pl.npair = npair;
  if (full_res(p)) {
    pl.X = W; pl.Y = H; pl.D = Dmax;
  } else {
    pl.X = (W + 1) / 2; pl.Y = (H + 1) / 2; pl.D = (Dmax + 1) / 2;
  }
  pl.dbits = key_dbits(pl.D);
  pl.p = p;
  build_tables(p, pl.lut_ad, pl.lut_mc);
  pl.cmax = pl.lut_ad[255] + pl.lut_mc[6];
  plan_geometry(pl, c->num_cu,
                form.fewest_chunks ? 1 : tuned_nchunk(c, W, H, Dmax, npair, p), form.nbase);
  pl.nk = (int)(((size_t)pl.X * pl.Y + 63) & ~size_t(63));
  const PlanBytes b = plan_bytes(pl);
  if (b.pk >= (size_t(1) << 32) || b.arms >= (size_t(1) << 32))
    return fail(c, STEREO_EINVAL, "%d pairs of %dx%d exceed the 4 GiB pixel or arm planes", npair,
                W, H);
  return 0;
}

// Carves the planes of pl from the device block at base and enqueues their
// set-up on stream s: padding cleared, cost table written (k_plan_init).
void plan_carve_and_init(Plan& pl, void* base, hipStream_t s) {
  const size_t n = (size_t)pl.X * pl.Y, npair = pl.npair, nk = pl.nk;
  const PlanBytes b = plan_bytes(pl);
  char* cur = static_cast<char*>(base);
  pl.half = carve<uint8_t>(cur, 2 * npair * n);
  pl.pk = carve<uint16_t>(cur, b.pk / 2);
  pl.arms = carve<uint32_t>(cur, b.arms / 4);
  pl.xoff = carve<uint32_t>(cur, b.arms / 4);
  pl.tab = carve<uint16_t>(cur, kTab);
  pl.keys = carve<uint32_t>(cur, npair * pl.nchunk * 2 * nk);
  pl.disp = carve<int16_t>(cur, 2 * npair * nk);
  pl.mincost = carve<uint32_t>(cur, 2 * npair * nk);
  pl.gcp = carve<uint8_t>(cur, npair * n);
  pl.med = carve<int16_t>(cur, npair * n);
  pl.filled = carve<int16_t>(cur, npair * n);
  TabArgs t{};
  for (int i = 0; i < 256; ++i) t.ad[i] = pl.lut_ad[i];
  for (int i = 0; i < 7; ++i) t.mc[i] = pl.lut_mc[i];
  // pk, arms and xoff are adjacent in the block: one cleared range covers them
  const size_t nzero = (size_t)(reinterpret_cast<char*>(pl.xoff) + b.arms -
                                reinterpret_cast<char*>(pl.pk)) / 4;
  const unsigned blocks = (unsigned)std::min<size_t>(2048, (nzero + 1023) / 1024 + 1);
  hipLaunchKernelGGL(k_plan_init, dim3(blocks), dim3(256), 0, s,
                     reinterpret_cast<uint32_t*>(pl.pk), nzero, pl.tab, t);
}

// The geometries to take where the scratch does not hold the preferred one
// (`first`): the other forms in order of modelled time, each needing less scratch
// than every one before it (at 1436x992 Dmax 145 the forms take 45.9, 28.8, 31.7
// and 20.3 MB at 4224, 4829, 7240 and 15157 units: the third is none of these).
std::vector<Plan> smaller_forms(stereo_ctx* c, const Plan& first) {
  std::vector<Plan> all, out;
  const std::string err = c->err;  // a form that is refused is left out
  for (const Form& form : kForms) {
    Plan pl;
    if (&form != kForms && !plan_setup(c, pl, first.W, first.H, first.Dmax, first.p, first.npair, form))
      all.push_back(pl);
  }
  c->err = err;
  std::sort(all.begin(), all.end(), [](const Plan& a, const Plan& b) { return a.model_t < b.model_t; });
  size_t least = plan_bytes(first).total;
  for (const Plan& pl : all)
    if (plan_bytes(pl).total < least) {
      least = plan_bytes(pl).total;
      out.push_back(pl);
    }
  return out;
}

// A plan of the geometry geo: its device memory, and its set-up enqueued on s.
int make_plan(stereo_ctx* c, const Plan& geo, hipStream_t s, Plan** out) {
  const size_t bytes = plan_bytes(geo).total;
  if (c->mem_cap && c->used + bytes > c->mem_cap)
    return fail(c, STEREO_ENOMEM, "plan needs %zu bytes, cap %zu, in use %zu", bytes, c->mem_cap,
                c->used);
  void* block = nullptr;
  hipError_t e = hipMalloc(&block, bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return fail(c, STEREO_ENOMEM, "hipMalloc(%zu): %s", bytes, hipGetErrorString(e));
  }
  Plan* pl = new Plan(geo);
  pl->block = block;
  pl->bytes = bytes;
  // set-up on the stream the plan serves: later work on that stream follows
  // it, and no other stream or slot is stalled
  plan_carve_and_init(*pl, pl->block, s);
  e = hipGetLastError();
  if (e != hipSuccess) {
    free_plan(pl);
    return fail(c, STEREO_EHIP, "plan initialisation: %s", hipGetErrorString(e));
  }
  c->used += bytes;
  *out = pl;
  return 0;
}

// Plans that may be given up for another: not the one whose intermediates are
// kept nor those a captured graph still launches into.
bool evictable(const stereo_ctx* c, const Plan* pl) {
  return pl != c->last && pl->pins == 0 && !pl->captured;
}

// Gives up the least recently used plan that may be (after the device has
// finished with it); false when there is none.
bool evict_one(stereo_ctx* c) {
  Plan* lru = nullptr;
  for (Plan* pl : c->plans)
    if (evictable(c, pl) && (!lru || pl->last_use < lru->last_use)) lru = pl;
  if (!lru) return false;
  (void)hipDeviceSynchronize();
  drop_plan(c, lru);
  return true;
}

// make_plan, with the soft head's optional planes given back, then idle plans
// given up, while the scratch does not hold it.  A cap that would not hold it
// with all of them gone is left as it is.
int make_plan_evicting(stereo_ctx* c, const Plan& geo, hipStream_t s, Plan** out) {
  const size_t bytes = plan_bytes(geo).total;
  size_t kept = c->used - soft_optional_bytes(c);
  for (const Plan* pl : c->plans)
    if (evictable(c, pl)) kept -= pl->bytes;
  if (c->mem_cap && kept + bytes > c->mem_cap)
    return fail(c, STEREO_ENOMEM, "plan needs %zu bytes, cap %zu, in use %zu", bytes, c->mem_cap,
                c->used);
  int rc = make_plan(c, geo, s, out);
  while (rc == STEREO_ENOMEM && (drop_soft_optional(c) || evict_one(c))) rc = make_plan(c, geo, s, out);
  return rc;
}

int get_plan(stereo_ctx* c, int W, int H, int Dmax, const stereo_params& p, int npair,
             const void* owner, hipStream_t s, Plan** out, bool smaller) {
  for (Plan* pl : c->plans)
    if (pl->W == W && pl->H == H && pl->Dmax == Dmax && pl->npair >= npair && pl->owner == owner &&
        same_params(pl->p, p)) {
      pl->last_use = ++c->tick;
      *out = pl;
      return 0;
    }
  // a new plan needs an allocation, which a stream under graph capture
  // cannot make
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone)
    return fail(c, STEREO_EINVAL,
                "no scratch yet for %dx%d Dmax %d on this stream: make one call outside the "
                "graph capture first (or use stereo_disparity_noalloc)", W, H, Dmax);
  (void)hipGetLastError();
  // the preferred form, idle plans given up for it; where the scratch does not
  // hold it even so, the fastest of the smaller ones that it does
  Plan geo, *pl = nullptr;
  int rc = plan_setup(c, geo, W, H, Dmax, p, npair, kForms[0]);
  if (rc) return rc;
  rc = make_plan_evicting(c, geo, s, &pl);
  if (rc == STEREO_ENOMEM && smaller)
    for (const Plan& g : smaller_forms(c, geo)) {
      rc = make_plan_evicting(c, g, s, &pl);
      if (rc != STEREO_ENOMEM) break;
    }
  if (rc) return rc;
  c->err.clear();
  pl->last_use = ++c->tick;
  pl->owner = owner;
  c->plans.push_back(pl);
  *out = pl;
  return 0;
}

void drop_plan(stereo_ctx* c, Plan* pl) {
  for (size_t i = 0; i < c->plans.size(); ++i)
    if (c->plans[i] == pl) {
      if (c->last == pl) c->last = nullptr;
      c->used -= pl->bytes;
      free_plan(pl);
      c->plans.erase(c->plans.begin() + i);
      return;
    }
}

// Frees every plan of (W, H, Dmax, p), whatever its owner (after the device
// has finished with them), so that the next call makes it again.
int evict_shape(stereo_ctx* c, int W, int H, int Dmax, const stereo_params& p) {
  for (const Plan* pl : c->plans)
    if (pl->W == W && pl->H == H && pl->Dmax == Dmax && same_params(pl->p, p) &&
        (pl->pins > 0 || pl->captured))
      return fail(c, STEREO_EINVAL, "a captured graph uses the scratch of %dx%d Dmax %d; tune "
                  "before capturing", W, H, Dmax);
  HIP_TRY(c, hipDeviceSynchronize());
  for (size_t i = 0; i < c->plans.size();) {
    Plan* pl = c->plans[i];
    if (pl->W == W && pl->H == H && pl->Dmax == Dmax && same_params(pl->p, p)) {
      if (c->last == pl) c->last = nullptr;
      c->used -= pl->bytes;
      free_plan(pl);
      c->plans.erase(c->plans.begin() + i);
    } else {
      ++i;
    }
  }
  return 0;
}

void set_tuned(stereo_ctx* c, int W, int H, int Dmax, int npair, const stereo_params& p,
               int nchunk) {
  for (Tuned& t : c->tuned)
    if (t.W == W && t.H == H && t.Dmax == Dmax && t.npair == npair && same_params(t.p, p)) {
      t.nchunk = nchunk;
      return;
    }
  c->tuned.push_back(Tuned{W, H, Dmax, npair, p, nchunk});
}

MatchArgs match_args(const Plan& pl, int npair, int dlo, int dhi, int nchunk) {
  MatchArgs a{};
  a.pk = pl.pk; a.arms = pl.arms; a.xoff = pl.xoff; a.tab = pl.tab; a.keys = pl.keys;
  a.X = pl.X; a.Y = pl.Y; a.XP = pl.XP; a.pad = pl.pad; a.XA = pl.XA; a.nk = pl.nk;
  a.arm = std::max(pl.p.arm_x, pl.p.arm_x_r); a.arm_y = pl.p.arm_y; a.dbits = pl.dbits;
  a.cmax = pl.cmax;
  a.copy_bytes = (uint32_t)((size_t)2 * pl.npair * pl.Y * pl.XP * 2);
  // the slack rows are the planes that follow in the plan's block, which are
  // always longer (carved in this order: pk, arms, xoff, tab, keys, ...)
  const PlanBytes b = plan_bytes(pl);
  auto bound = [](size_t n) { return (uint32_t)std::min(n, (size_t(1) << 32) - 1); };
  a.pk_bytes = bound(b.pk + (size_t)kMatchSlackRows * pl.XP * 2);
  a.arms_bytes = bound(b.arms + (size_t)kMatchSlackRows * pl.XA * 4);
  a.nbands = pl.nbands; a.dlo = dlo; a.dhi = dhi;
  a.nchunk = nchunk;
  a.grid = match_grid(pl, npair, dlo, dhi, nchunk);
  return a;
}

// k_match with KMAX = KM: its LDS block holds the plane rows the plan's
// bands write (band rows + 1) or its window step reads (o0 + 16 KMAX + 1),
// whichever is more; the rest of the CU's LDS stays free for other streams.
template <int NS, int NB, int KM>
void launch_match_km(const Plan& pl, const MatchArgs& a, dim3 grid, hipStream_t s) {
  const int o0max = pl.nbands == 1 ? 0 : pl.p.arm_y;
  const size_t lds = (size_t)match_lds_bytes(NS, NB, std::max(pl.brows, o0max + kWaves * KM) + 1);
  // dynamic LDS beyond the default limit needs the attribute (set once per
  // instance); were it refused, the launch below fails and run() reports
  // that launch's error
  auto allow = [](const void* f) {
    return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes - kMatchTabBytes);
  };
  if (a.dbg_cost) {
    static const hipError_t attr = allow(reinterpret_cast<const void*>(&k_match<NS, NB, KM, true>));
    (void)attr;
    hipLaunchKernelGGL((k_match<NS, NB, KM, true>), grid, dim3(kThreads), lds, s, a);
  } else {
    static const hipError_t attr = allow(reinterpret_cast<const void*>(&k_match<NS, NB, KM, false>));
    (void)attr;
    hipLaunchKernelGGL((k_match<NS, NB, KM, false>), grid, dim3(kThreads), lds, s, a);
  }
}

template <int NS>
void launch_match_k(const Plan& pl, const MatchArgs& a, dim3 grid, hipStream_t s) {
  if (pl.nbase == 1) {
    if (pl.kmax == 16) launch_match_km<NS, 1, 16>(pl, a, grid, s);
    else launch_match_km<NS, 1, 36>(pl, a, grid, s);
    return;
  }
  switch (pl.kmax) {
    case 4: launch_match_km<NS, 2, 4>(pl, a, grid, s); break;
    case 8: launch_match_km<NS, 2, 8>(pl, a, grid, s); break;
    case 12: launch_match_km<NS, 2, 12>(pl, a, grid, s); break;
    case 16: launch_match_km<NS, 2, 16>(pl, a, grid, s); break;
    default: launch_match_km<NS, 2, 18>(pl, a, grid, s); break;
  }
}

void launch_match(const Plan& pl, const MatchArgs& a, hipStream_t s) {
  dim3 grid((unsigned)(kXcds * a.grid.per));
  switch (pl.ns) {
    case 1: launch_match_k<1>(pl, a, grid, s); break;
    case 2: launch_match_k<2>(pl, a, grid, s); break;
    default: launch_match_k<3>(pl, a, grid, s); break;
  }
}

// Events of the next timed call (created on first use, reused after reset).
int timing_events(stereo_ctx* c, hipEvent_t** ev) {
  const size_t per = STEREO_NUM_STAGES + 1, need = (size_t)(c->timed_calls + 1) * per;
  while (c->events.size() < need) {
    hipEvent_t e;
    HIP_TRY(c, hipEventCreate(&e));
    c->events.push_back(e);
  }
  *ev = &c->events[(size_t)c->timed_calls * per];
  return 0;
}

int launch_status(stereo_ctx* c) {
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : fail(c, STEREO_EHIP, "kernel launch: %s", hipGetErrorString(e));
}

// The whole path for npair pairs already checked against the plan.
int run(stereo_ctx* c, Plan& pl, const PairPtrs& pp, int npair, bool keep, bool timed,
        hipStream_t s) {
  const int X = pl.X, Y = pl.Y;
  hipEvent_t* ev = nullptr;
  if (timed) {
    int rc = timing_events(c, &ev);
    if (rc) return rc;
  }
  auto mark = [&](int i) { if (ev) (void)hipEventRecord(ev[i], s); };
  dim3 b2(64, 4);
  const bool full = full_res(pl.p);
  mark(0);
  if (full)
    hipLaunchKernelGGL(k_gray_full, dim3((X + 255) / 256, Y, 2 * npair), dim3(256), 0, s, pp, X, Y,
                       pl.half);
  else
    hipLaunchKernelGGL(k_prep, dim3((X + 63) / 64, (Y + kPrepRows - 1) / kPrepRows, 2 * npair),
                       b2, 0, s, pp, pl.W, pl.H, X, Y, pl.half);
  mark(1);
  hipLaunchKernelGGL(k_feat, dim3((X + 63) / 64, (Y + kFeatRows - 1) / kFeatRows, 2 * npair),
                     dim3(64, kFeatRows), 0,
                     s, pl.half, X, Y, pl.p.color_delta, pl.p.arm_x, pl.p.arm_x_r, pl.p.arm_y,
                     pl.XP, pl.pad, pl.XA, nullptr, nullptr, pl.arms, pl.xoff, pl.pk,
                     (size_t)2 * pl.npair * Y * pl.XP);
  mark(2);
  launch_match(pl, match_args(pl, npair, 0, pl.D, pl.nchunk), s);
  mark(3);
  // one kernel for the rest of small frames (stage times and kept planes need the
  // three; rows of fewer than 4 columns do not fill its loads)
  if (!full && !keep && !timed && X >= 4 && X <= kPostMaxX && (size_t)npair * X * Y <= kPostMaxPixels) {
    hipLaunchKernelGGL(k_post, dim3((Y + kPostRows - 1) / kPostRows, npair), dim3(kPostThreads), 0, s, pp,
                       pl.keys, pl.nchunk, pl.nk, pl.dbits, pl.pk, pl.XP, pl.pad, pl.W, pl.H, X, Y,
                       pl.p.fill_T, pl.p.fill_mode);
    return launch_status(c);
  }
  hipLaunchKernelGGL(k_wta, dim3((pl.nk + 1023) / 1024, npair), dim3(256), 0, s, pl.keys,
                     pl.nchunk, pl.nk, pl.dbits, pl.disp, keep ? pl.mincost : nullptr);
  mark(4);
  hipLaunchKernelGGL(k_refine, dim3(Y, npair), dim3(256), refine_lds(X), s, pl.disp, pl.nk, pl.pk, pl.XP,
                     pl.pad, X, Y, pl.p.fill_T, pl.p.fill_mode, keep ? pl.gcp : nullptr,
                     keep ? pl.med : nullptr, full && !keep ? nullptr : pl.filled, pp, (int)full);
  mark(5);
  if (!full)
    hipLaunchKernelGGL(k_upscale, dim3((X + 63) / 64, (Y + 3) / 4, npair), b2, 0, s, pp,
                       pl.filled, pl.W, pl.H, X, Y, pl.p.fill_T);
  mark(6);
  if (int rc = launch_status(c)) return rc;
  if (timed) ++c->timed_calls;
  return 0;
}

int common_checks(stereo_ctx* c, int W, int H, int Dmax, const stereo_params* params,
                  stereo_params* p) {
  if (W < 2 || H < 2 || W > STEREO_MAX_SIDE || H > STEREO_MAX_SIDE)
    return fail(c, STEREO_EINVAL, "image size %dx%d outside 2..%d", W, H, STEREO_MAX_SIDE);
  if (Dmax < 1 || Dmax > W || Dmax > STEREO_MAX_DMAX)
    return fail(c, STEREO_EINVAL, "Dmax %d outside 1..min(W=%d, %d)", Dmax, W, STEREO_MAX_DMAX);
  if (params) {
    if (params->size != sizeof(stereo_params))
      return fail(c, STEREO_EINVAL, "params.size %u != %zu", params->size, sizeof(stereo_params));
    *p = *params;
  } else {
    stereo_default_params(p);
  }
  const bool full = (p->flags & STEREO_F_FULL_RES) != 0;
  if (full && W > STEREO_MAX_SIDE / 2)
    return fail(c, STEREO_EINVAL, "full-resolution mode needs W <= %d", STEREO_MAX_SIDE / 2);
  return check_params(c, *p, full ? Dmax : (Dmax + 1) / 2);
}

}  // namespace stereo_host

using namespace stereo_host;

extern "C" {

void stereo_default_params(stereo_params* p) {
  if (!p) return;
  std::memset(p, 0, sizeof *p);
  p->size = sizeof(stereo_params);
  p->lambda_ad = 0.3f;
  p->lambda_mc = 2.3f;
  p->cost_scale = 1024;
  p->color_delta = 13;
  p->arm_x = 21;
  p->arm_y = 31;
  p->fill_T = 3;
  p->flags = 0;
  p->arm_x_r = -1;
  p->fill_mode = 0;
}

int stereo_create(stereo_ctx** out, int device, size_t mem_cap) {
  if (!out) return STEREO_EINVAL;
  *out = nullptr;
  int n = 0;
  if (hipGetDeviceCount(&n) != hipSuccess || device < 0 || device >= n) {
    (void)hipGetLastError();
    return STEREO_EINVAL;
  }
  if (hipSetDevice(device) != hipSuccess) return STEREO_EHIP;
  stereo_ctx* c = new stereo_ctx();
  c->device = device;
  c->mem_cap = mem_cap;
  int cu = 0;
  if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess &&
      cu > 0)
    c->num_cu = cu;
  // the device's fixed scratch array, for stereo_disparity_noalloc
  c->noalloc_scratch = noalloc_scratch_of(device, &c->noalloc_err);
  *out = c;
  return 0;
}

void stereo_destroy(stereo_ctx* c) {
  if (!c) return;
  (void)hipSetDevice(c->device);
  for (hipEvent_t e : c->events) (void)hipEventDestroy(e);
  for (Plan* pl : c->plans) free_plan(pl);
  free_soft_plans(c->soft_plans);
  for (auto& b : c->l1_blocks) (void)hipFree(b.second);
  delete c;
}

const char* stereo_last_error(const stereo_ctx* c) { return c ? c->err.c_str() : "null context"; }

int stereo_disparity_batch(stereo_ctx* c, const uint8_t* const* left, const uint8_t* const* right,
                           int n, int W, int H, int Dmax, const stereo_params* params,
                           int16_t* const* out_disp, hipStream_t stream) {
  if (!c) return STEREO_EINVAL;
  c->err.clear();
  if (!left || !right || !out_disp || n < 1) return fail(c, STEREO_EINVAL, "null pointer or n < 1");
  for (int i = 0; i < n; ++i)
    if (!left[i] || !right[i] || !out_disp[i]) return fail(c, STEREO_EINVAL, "null image pointer %d", i);
  stereo_params p;
  int rc = common_checks(c, W, H, Dmax, params, &p);
  if (rc) return rc;
  HIP_TRY(c, hipSetDevice(c->device));
  const bool keep = (p.flags & STEREO_F_KEEP_INTERMEDIATES) != 0;
  const int per = std::min(n, kMaxPairs);
  Plan* pl = nullptr;
  rc = get_plan(c, W, H, Dmax, p, per, stream, stream, &pl);
  if (rc) return rc;
  // a graph captured from this call launches into the plan's memory later:
  // the plan is never evicted for another (it is freed by stereo_destroy)
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone)
    pl->captured = true;
  (void)hipGetLastError();
  // where planes are kept, those of pair 0: its launch comes last, since every
  // launch uses the same scratch
  const int ngroups = (n + kMaxPairs - 1) / kMaxPairs;
  for (int g = 0; g < ngroups; ++g) {
    const int i0 = (keep ? (g + 1) % ngroups : g) * kMaxPairs, m = std::min(kMaxPairs, n - i0);
    PairPtrs pp{};
    for (int i = 0; i < m; ++i) {
      pp.left[i] = left[i0 + i];
      pp.right[i] = right[i0 + i];
      pp.out[i] = out_disp[i0 + i];
    }
    rc = run(c, *pl, pp, m, keep && i0 == 0, (p.flags & STEREO_F_STAGE_TIMING) != 0, stream);
    if (rc) return rc;
  }
  if (keep) c->last = pl;
  return 0;
}

int stereo_autotune(stereo_ctx* c, const uint8_t* const* left, const uint8_t* const* right, int n,
                    int W, int H, int Dmax, const stereo_params* params, int* chosen,
                    int* sizes, float* times_ms, int max_times, hipStream_t stream) {
  if (!c) return STEREO_EINVAL;
  c->err.clear();
  if (!left || !right || n < 1) return fail(c, STEREO_EINVAL, "null pointer or n < 1");
  const int m = std::min(n, kMaxPairs);
  for (int i = 0; i < m; ++i)
    if (!left[i] || !right[i]) return fail(c, STEREO_EINVAL, "null image pointer %d", i);
  stereo_params p;
  int rc = common_checks(c, W, H, Dmax, params, &p);
  if (rc) return rc;
  p.flags &= ~(STEREO_F_KEEP_INTERMEDIATES | STEREO_F_STAGE_TIMING);
  HIP_TRY(c, hipSetDevice(c->device));
  // the modelled default, then the sizes ceil(D / k), k = 1 .. min(D, 32), that the
  // strips of both bases allow, each as the fewest chunks of that size
  Plan probe{};
  probe.W = W; probe.H = H; probe.Dmax = Dmax; probe.npair = m; probe.p = p;
  probe.X = full_res(p) ? W : (W + 1) / 2;
  probe.Y = full_res(p) ? H : (H + 1) / 2;
  probe.D = full_res(p) ? Dmax : (Dmax + 1) / 2;
  plan_geometry(probe, c->num_cu, 0, 2);
  std::vector<int> cand{probe.nchunk}, cand_size{probe.csize};
  for (int k = 1; k <= std::min(probe.D, 32); ++k) {
    const int cs = (probe.D + k - 1) / k;
    if (cs > probe.ccap || std::find(cand_size.begin(), cand_size.end(), cs) != cand_size.end()) continue;
    cand_size.push_back(cs);
    cand.push_back((probe.D + cs - 1) / cs);
  }
  // scratch output maps for the trial runs
  int16_t* outs = nullptr;
  HIP_TRY(c, hipMalloc(&outs, (size_t)m * W * H * 2));
  PairPtrs pp{};
  for (int i = 0; i < m; ++i) {
    pp.left[i] = left[i];
    pp.right[i] = right[i];
    pp.out[i] = outs + (size_t)i * W * H;
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  const int before = tuned_nchunk(c, W, H, Dmax, m, p);
  // candidates that ran: where the scratch holds a smaller form only, several
  // have the same launch, which is timed once
  struct Trial { int nbase, ns, nbands, nchunk, csize; };
  std::vector<Trial> ran;
  int best = 0, best_size = 0;
  float best_ms = 1e30f;
  hipError_t he = hipEventCreate(&e0);
  if (he == hipSuccess) he = hipEventCreate(&e1);
  for (size_t k = 0; k < cand.size() && he == hipSuccess && rc == 0; ++k) {
    set_tuned(c, W, H, Dmax, m, p, cand[k]);
    rc = evict_shape(c, W, H, Dmax, p);
    Plan* pl = nullptr;
    if (!rc) rc = get_plan(c, W, H, Dmax, p, m, stream, stream, &pl);
    if (rc) break;
    const Trial now{pl->nbase, pl->ns, pl->nbands, pl->nchunk, pl->csize};
    if (std::any_of(ran.begin(), ran.end(), [&](const Trial& t) {
          return t.nbase == now.nbase && t.ns == now.ns && t.nbands == now.nbands && t.nchunk == now.nchunk;
        }))
      continue;
    rc = run(c, *pl, pp, m, false, false, stream);  // warm
    constexpr int kReps = 5;
    if (!rc) he = hipEventRecord(e0, stream);
    for (int r = 0; r < kReps && !rc && he == hipSuccess; ++r) rc = run(c, *pl, pp, m, false, false, stream);
    if (!rc && he == hipSuccess) he = hipEventRecord(e1, stream);
    if (!rc && he == hipSuccess) he = hipEventSynchronize(e1);
    float ms = 0.f;
    if (!rc && he == hipSuccess) he = hipEventElapsedTime(&ms, e0, e1);
    if (rc || he != hipSuccess) break;
    ms /= kReps;
    if ((int)ran.size() < max_times) {
      if (sizes) sizes[ran.size()] = now.csize;
      if (times_ms) times_ms[ran.size()] = ms;
    }
    ran.push_back(now);
    if (ms < best_ms) {
      best_ms = ms;
      best = cand[k];
      best_size = now.csize;
    }
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipDeviceSynchronize();
  (void)hipFree(outs);
  if (!rc && he != hipSuccess) rc = fail(c, STEREO_EHIP, "autotune: %s", hipGetErrorString(he));
  // a call that failed leaves what was chosen before
  set_tuned(c, W, H, Dmax, m, p, rc ? before : best);
  const std::string err = c->err;
  const int rc2 = evict_shape(c, W, H, Dmax, p);
  if (rc) c->err = err;
  if (rc) return rc;
  if (rc2) return rc2;
  if (chosen) *chosen = best_size;
  if (max_times > (int)ran.size()) {
    if (sizes) sizes[ran.size()] = 0;
    if (times_ms) times_ms[ran.size()] = -1.f;
  }
  return 0;
}

int stereo_disparity(stereo_ctx* c, const uint8_t* left, const uint8_t* right, int W, int H,
                     int Dmax, const stereo_params* params, int16_t* out_disp, hipStream_t stream) {
  if (!c) return STEREO_EINVAL;
  return stereo_disparity_batch(c, &left, &right, 1, W, H, Dmax, params, &out_disp, stream);
}

int stereo_disparity_noalloc(stereo_ctx* c, const uint8_t* left, const uint8_t* right, int W,
                             int H, int Dmax, const stereo_params* params, int16_t* out_disp,
                             hipStream_t stream) {
  if (!c) return STEREO_EINVAL;
  c->err.clear();
  if (!left || !right || !out_disp) return fail(c, STEREO_EINVAL, "null pointer");
  stereo_params p;
  int rc = common_checks(c, W, H, Dmax, params, &p);
  if (rc) return rc;
  if (p.flags & (STEREO_F_KEEP_INTERMEDIATES | STEREO_F_STAGE_TIMING))
    return fail(c, STEREO_EINVAL, "stereo_disparity_noalloc takes neither "
                "STEREO_F_KEEP_INTERMEDIATES nor STEREO_F_STAGE_TIMING");
  if (!c->noalloc_scratch)
    return fail(c, STEREO_EHIP, "no fixed scratch on device %d: %s", c->device,
                c->noalloc_err.c_str());
  // the plan lives on the stack and its memory is the fixed array: geometry
  // and tables are host arithmetic, the set-up (padding cleared, cost table
  // written) is a kernel on the caller's stream
  Plan pl{};
  rc = plan_setup(c, pl, W, H, Dmax, p, 1, kForms[0]);
  if (rc) return rc;
  if (plan_bytes(pl).total > kNoallocBytes)
    for (const Plan& g : smaller_forms(c, pl)) {
      pl = g;
      if (plan_bytes(pl).total <= kNoallocBytes) break;
    }
  const size_t bytes = plan_bytes(pl).total;
  if (bytes > kNoallocBytes)
    return fail(c, STEREO_EINVAL, "%dx%d Dmax %d needs %zu bytes of scratch; the fixed array "
                "holds %zu (use stereo_disparity)", W, H, Dmax, bytes, kNoallocBytes);
  HIP_TRY(c, hipSetDevice(c->device));
  (void)hipGetLastError();
  plan_carve_and_init(pl, c->noalloc_scratch, stream);
  PairPtrs pp{};
  pp.left[0] = left;
  pp.right[0] = right;
  pp.out[0] = out_disp;
  return run(c, pl, pp, 1, false, false, stream);
}

int stereo_stage_times(stereo_ctx* c, double* ms, int* calls, int reset) {
  if (!c) return STEREO_EINVAL;
  c->err.clear();
  if (!ms) return fail(c, STEREO_EINVAL, "null ms");
  HIP_TRY(c, hipSetDevice(c->device));
  for (int i = 0; i < STEREO_NUM_STAGES; ++i) ms[i] = 0.0;
  const size_t per = STEREO_NUM_STAGES + 1;
  for (int k = 0; k < c->timed_calls; ++k) {
    hipEvent_t* ev = &c->events[(size_t)k * per];
    HIP_TRY(c, hipEventSynchronize(ev[STEREO_NUM_STAGES]));
    for (int i = 0; i < STEREO_NUM_STAGES; ++i) {
      float t = 0.f;
      HIP_TRY(c, hipEventElapsedTime(&t, ev[i], ev[i + 1]));
      ms[i] += t;
    }
  }
  if (calls) *calls = c->timed_calls;
  if (reset) c->timed_calls = 0;
  return 0;
}

int stereo_get_intermediate(stereo_ctx* c, int which, int d, void* dst, size_t bytes,
                            hipStream_t stream) {
  if (!c) return STEREO_EINVAL;
  c->err.clear();
  Plan* pl = c->last;
  if (!pl) return fail(c, STEREO_EINVAL, "no call with STEREO_F_KEEP_INTERMEDIATES yet");
  if (!dst) return fail(c, STEREO_EINVAL, "null destination");
  HIP_TRY(c, hipSetDevice(c->device));
  const size_t n = (size_t)pl->X * pl->Y;
  auto need = [&](size_t b) { return bytes >= b; };
  switch (which) {
    case STEREO_I_LUT: {
      if (!need(263 * 2)) break;
      std::memcpy(dst, pl->lut_ad, 256 * 2);
      std::memcpy(static_cast<char*>(dst) + 512, pl->lut_mc, 7 * 2);
      return 0;
    }
    case STEREO_I_HALF_L: case STEREO_I_HALF_R: case STEREO_I_CENSUS_L: case STEREO_I_CENSUS_R: {
      if (!need(n)) break;
      const int img = (which == STEREO_I_HALF_R || which == STEREO_I_CENSUS_R) ? 1 : 0;
      std::vector<uint16_t> tmp(n);
      HIP_TRY(c, hipStreamSynchronize(stream));
      HIP_TRY(c, hipMemcpy2D(tmp.data(), (size_t)pl->X * 2,
                             pl->pk + (size_t)img * pl->Y * pl->XP + pl->pad, (size_t)pl->XP * 2,
                             (size_t)pl->X * 2, pl->Y, hipMemcpyDeviceToHost));
      const bool census = which == STEREO_I_CENSUS_L || which == STEREO_I_CENSUS_R;
      uint8_t* o = static_cast<uint8_t*>(dst);
      for (size_t i = 0; i < n; ++i) o[i] = census ? (uint8_t)(tmp[i] >> 8) : (uint8_t)tmp[i];
      return 0;
    }
    case STEREO_I_ARMS_L: case STEREO_I_ARMS_R: {
      if (!need(4 * n)) break;
      const int img = which == STEREO_I_ARMS_R ? 1 : 0;
      HIP_TRY(c, hipStreamSynchronize(stream));
      HIP_TRY(c, hipMemcpy2D(dst, (size_t)pl->X * 4, pl->arms + (size_t)img * pl->Y * pl->XA,
                             (size_t)pl->XA * 4, (size_t)pl->X * 4, pl->Y, hipMemcpyDeviceToHost));
      return 0;
    }
    case STEREO_I_COST_L_D: case STEREO_I_COST_R_D: case STEREO_I_CAX_L_D: case STEREO_I_CAX_R_D:
    case STEREO_I_CA_L_D: case STEREO_I_CA_R_D: {
      const bool cost = which == STEREO_I_COST_L_D || which == STEREO_I_COST_R_D;
      if (!need(cost ? 2 * n : 4 * n)) break;
      if (d < 0 || d >= pl->D) return fail(c, STEREO_EINVAL, "d %d outside 0..%d", d, pl->D - 1);
      if (!pl->dbg_block) {
        const size_t b = ((2 * n + 255) & ~size_t(255)) + 2 * ((4 * n + 255) & ~size_t(255));
        hipError_t e = hipMalloc(&pl->dbg_block, b);
        if (e != hipSuccess) {
          (void)hipGetLastError();
          return fail(c, STEREO_ENOMEM, "debug planes: %s", hipGetErrorString(e));
        }
        char* cur = static_cast<char*>(pl->dbg_block);
        pl->dbg_cost = carve<uint16_t>(cur, n);
        pl->dbg_cax = carve<uint32_t>(cur, n);
        pl->dbg_ca = carve<uint32_t>(cur, n);
      }
      // one-disparity run of the fused kernel on pair 0 with the debug planes
      // of the wanted base on; it overwrites the first d-chunk keys only
      MatchArgs a = match_args(*pl, 1, d, d + 1, 1);
      a.dbg_cost = pl->dbg_cost; a.dbg_cax = pl->dbg_cax; a.dbg_ca = pl->dbg_ca;
      a.dbg_base = (which == STEREO_I_COST_R_D || which == STEREO_I_CAX_R_D ||
                    which == STEREO_I_CA_R_D) ? 1 : 0;
      launch_match(*pl, a, stream);
      HIP_TRY(c, hipGetLastError());
      HIP_TRY(c, hipStreamSynchronize(stream));
      const void* src = cost ? (const void*)pl->dbg_cost
                      : (which == STEREO_I_CAX_L_D || which == STEREO_I_CAX_R_D)
                            ? (const void*)pl->dbg_cax : (const void*)pl->dbg_ca;
      HIP_TRY(c, hipMemcpy(dst, src, cost ? 2 * n : 4 * n, hipMemcpyDeviceToHost));
      return 0;
    }
    case STEREO_I_MINCOST_L: case STEREO_I_MINCOST_R: {
      if (!need(4 * n)) break;
      HIP_TRY(c, hipStreamSynchronize(stream));
      HIP_TRY(c, hipMemcpy(dst, pl->mincost + (which == STEREO_I_MINCOST_R ? pl->nk : 0), 4 * n,
                           hipMemcpyDeviceToHost));
      return 0;
    }
    case STEREO_I_DISP_L: case STEREO_I_DISP_R: {
      if (!need(2 * n)) break;
      HIP_TRY(c, hipStreamSynchronize(stream));
      HIP_TRY(c, hipMemcpy(dst, pl->disp + (which == STEREO_I_DISP_R ? pl->nk : 0), 2 * n,
                           hipMemcpyDeviceToHost));
      return 0;
    }
    case STEREO_I_GCP: {
      if (!need(n)) break;
      HIP_TRY(c, hipStreamSynchronize(stream));
      HIP_TRY(c, hipMemcpy(dst, pl->gcp, n, hipMemcpyDeviceToHost));
      return 0;
    }
    case STEREO_I_MEDIAN: case STEREO_I_FILLED: {
      if (!need(2 * n)) break;
      HIP_TRY(c, hipStreamSynchronize(stream));
      HIP_TRY(c, hipMemcpy(dst, which == STEREO_I_MEDIAN ? pl->med : pl->filled, 2 * n,
                           hipMemcpyDeviceToHost));
      return 0;
    }
    default:
      return fail(c, STEREO_EINVAL, "unknown intermediate %d", which);
  }
  return fail(c, STEREO_EINVAL, "destination of %zu bytes too small for intermediate %d", bytes,
              which);
}

}  // extern "C"
