// C ABI, candidates: chi-square and gradient, batched L-BFGS refinement, and the
// downhill simplex along lines, all on candidates' own maps and light curves.

#include "host.h"

#include <mutex>

using namespace morse;
using namespace morse::host;

// Scratch of the allocation-free entry point (morse_chi2_grad_noalloc): one array per
// GPU, held until the process ends.  Host code uses its device address from
// hipGetSymbolAddress (kept per device), never the array's name.
constexpr size_t kNoallocScratchBytes = (size_t)128 << 20;
static __device__ __align__(256) char scratch[kNoallocScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
char* g_scratch_ptr[kMaxScratchDevices] = {};
}  // namespace

namespace morse {
namespace host {
// Called by morse_ctx_create with `device` current (and again, cached, by the entry
// point).
int noalloc_scratch(int device, char** out) {
  if (device < 0 || device >= kMaxScratchDevices)
    return fail(nullptr, MORSE_EUNSUPPORTED, "device %d: at most %d devices", device,
                kMaxScratchDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return fail(nullptr, MORSE_EHIP, "hipGetSymbolAddress(scratch) on device %d: %s", device,
                  hipGetErrorString(e));
    g_scratch_ptr[device] = static_cast<char*>(p);
  }
  *out = g_scratch_ptr[device];
  return MORSE_OK;
}
}  // namespace host
}  // namespace morse

namespace {

int plan_candidates(morse_ctx* ctx, const morse_map_view* maps, int32_t n_maps,
                    const morse_lightcurves* lcs, int64_t n, Plan& pl, size_t& i_sums,
                    size_t& i_wF, size_t& i_quad) {
  if (!maps || n_maps <= 0) return fail(ctx, MORSE_EINVAL, "need n_maps >= 1 maps");
  int rc;
  for (int i = 0; i < n_maps; ++i) {
    if (!maps[i].d_map) return fail(ctx, MORSE_EINVAL, "map %d: d_map is NULL", i);
    if ((rc = check_window(ctx, &maps[i].window, "map window"))) return rc;
  }
  if ((rc = check_lightcurves(ctx, lcs))) return rc;
  if (n < 0) return fail(ctx, MORSE_EINVAL, "n < 0");
  if ((rc = check_quad_size(ctx, maps, n_maps))) return rc;
  i_sums = pl.add(24 * (size_t)lcs->n_events);
  i_wF = pl.add(8 * (size_t)lcs->h_offsets[lcs->n_events]);
  i_quad = pl.add(quad_region_bytes(maps, n_maps));
  return MORSE_OK;
}

hipError_t prepare_candidates(const LcView& lc, int32_t ne, const MapC* d_maps, const std::vector<MapC>& hm,
                              hipStream_t st) {
  PrepArgs p{};
  p.lc = lc;
  p.n_events = ne;
  p.maps = d_maps;
  p.n_maps = (int32_t)hm.size();
  return launch_prep(p, hm.data(), st);
}

// Host metadata of the candidate entry points (event offsets, reference times, map
// table) lives in its own device buffer, put there only when it changes, so calls that
// alternate with searches need not put it again.
int setup_candidates(morse_ctx* ctx, const morse_map_view* maps, int32_t n_maps,
                     const morse_lightcurves* lcs, const Plan& pl, size_t i_sums, size_t i_wF,
                     size_t i_quad, LcView& lc, MapC*& d_maps, std::vector<MapC>& hm) {
  int rc;
  const int32_t ne = lcs->n_events;
  hm.resize(n_maps);
  for (int i = 0; i < n_maps; ++i) hm[i] = make_mapc(maps[i].d_map, maps[i].window);
  assign_quads(hm, pl.ptr(ctx, i_quad));
  MetaBlock mb;
  const size_t o_off = mb.add(lcs->h_offsets, 8 * (size_t)(ne + 1)),
               o_tref = mb.add(lcs->h_t_ref, 8 * (size_t)ne),
               o_maps = mb.add(hm.data(), sizeof(MapC) * n_maps);  // with the packed cells' addresses
  Hasher key;
  key.pod(ne);
  key.pod(n_maps);
  key.bytes(mb.bytes.data(), mb.bytes.size());
  char* meta;
  if ((rc = put_meta(ctx, ctx->cmeta, mb.bytes, key.h, &meta))) return rc;
  int64_t* d_off = (int64_t*)(meta + o_off);
  double* d_tref = (double*)(meta + o_tref);
  d_maps = (MapC*)(meta + o_maps);
  lc.t = lcs->d_t;
  lc.w = lcs->d_weight;
  lc.F = lcs->d_flux;
  lc.wFc = (double*)pl.ptr(ctx, i_wF);
  lc.off = d_off;
  lc.sums = (double*)pl.ptr(ctx, i_sums);
  lc.t_ref = d_tref;
  lc.sorted = nullptr;
  HIP_TRY(ctx, prepare_candidates(lc, ne, d_maps, hm, ctx->stream));
  return MORSE_OK;
}
}  // namespace

namespace {
// Refinements of many candidates on maps larger than the last-level cache evaluate all of them
// round by round: neighbours in the order then sample the same stretch of a map at the
// same time, which workgroups that run their candidates' rounds on their own soon do not.
// 50 rounds of 262,144 candidates on 64 maps of 64 MiB: 158 ms by round, 174 to 195 in one launch.
bool refine_by_round(int64_t n, bool beyond_cache) { return n >= 32768 && beyond_cache; }

// Four candidates a workgroup share one update's time, but wait for one another, and one after
// the other they sample different stretches of a map: short light curves, of which the update is
// the larger part, gain sooner.  Milliseconds with one and with four, 12 rounds (15 on 16 maps):
//   20 events x 300 points on a map of 256^2   3000: 0.34 / 0.35,  6144: 0.53 / 0.42,  16,384: 1.20 / 0.82
//   1 event x 1000 points, 4 maps of 2048^2    4096: 0.74 / 0.72,  6144: 0.99 / 0.86,  16,384: 2.14 / 1.79
//   8 ragged events of about 2000 points, 512^2  8192: 1.02 / 1.11,  12,288: 1.45 / 1.42,  16,384: 1.90 / 1.69
//   20 events x 3000 points, 4 maps of 2048^2  8192: 1.69 / 1.63,  12,288: 2.41 / 2.51,  16,384: 3.10 / 2.94
//   16 maps of 2048^2, which the cache does not hold, 16,384 candidates: 3.39 / 3.94
bool refine_by_four(int64_t n, int64_t mean_points, bool beyond_cache) {
  return n >= (mean_points <= 1024 ? 6144 : 16384) && !beyond_cache;
}
}  // namespace

extern "C" {


int morse_line_simplex(morse_ctx* ctx, const morse_map_view* maps, int32_t n_maps,
                       const morse_lightcurves* lcs, int32_t event, const double* d_lines,
                       int64_t n_lines, const double* d_start, const morse_simplex_opts* opts,
                       double* d_chi2, double* d_t0, double* d_tE, int32_t* d_iters,
                       int32_t* d_evals) {
  if (!ctx) return fail(nullptr, MORSE_EINVAL, "ctx is NULL");
  int rc;
  Plan pl;
  size_t i_sums, i_wF, i_quad;
  if ((rc = plan_candidates(ctx, maps, n_maps, lcs, n_lines, pl, i_sums, i_wF, i_quad))) return rc;
  if (event < 0 || event >= lcs->n_events) return fail(ctx, MORSE_EINVAL, "event %d out of range", event);
  if (!opts) return fail(ctx, MORSE_EINVAL, "opts is NULL");
  if (opts->max_iter < 0) return fail(ctx, MORSE_EINVAL, "max_iter < 0");
  if (!(std::isfinite(opts->step_t0) && std::isfinite(opts->step_ln_tE) && std::isfinite(opts->ftol) &&
        opts->ftol >= 0.0))
    return fail(ctx, MORSE_EINVAL, "steps and ftol must be finite, ftol >= 0");
  if (n_lines == 0) return MORSE_OK;
  if (!d_lines || !d_start || !d_chi2 || !d_t0 || !d_tE || !d_iters)
    return fail(ctx, MORSE_EINVAL, "NULL device array");
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  // start order: lines by descending largest sample on the first map (the filter's
  // sampling of the line across the window)
  const morse_grid2d& w0 = maps[0].window;
  const double R = 0.5 * std::sqrt(w0.wx * w0.wx + w0.wy * w0.wy);
  const double ns64 = std::ceil(2.0 * R * std::max(w0.nx / w0.wx, w0.ny / w0.wy)) + 1.0;
  const bool ordered = ns64 <= 1.0e7 && n_lines <= INT32_MAX;
  const size_t i_key = pl.add(ordered ? 4 * (size_t)n_lines : 0),
               i_hist = pl.add(ordered ? 4 * (size_t)kSimplexPrioBins : 0),
               i_order = pl.add(ordered ? 4 * (size_t)n_lines : 0);
  if ((rc = reserve(ctx, pl.total()))) return rc;
  SimplexArgs a{};
  MapC* d_maps;
  std::vector<MapC> hm;
  if ((rc = setup_candidates(ctx, maps, n_maps, lcs, pl, i_sums, i_wF, i_quad, a.lc, d_maps, hm))) return rc;
  a.maps = d_maps;
  a.n_maps = n_maps;
  a.event = event;
  a.n_points = (int32_t)(lcs->h_offsets[event + 1] - lcs->h_offsets[event]);
  a.lines = d_lines;
  a.n_lines = n_lines;
  a.start = d_start;
  a.d_t0 = opts->step_t0;
  a.d_ln_tE = opts->step_ln_tE;
  a.ftol = opts->ftol;
  a.max_iter = opts->max_iter;
  a.chi2 = d_chi2;
  a.t0 = d_t0;
  a.tE = d_tE;
  a.iters = d_iters;
  a.evals = d_evals;
  if (ordered) {
    HIP_TRY(ctx, launch_simplex_order(a, w0.cx, w0.cy, R, (int32_t)ns64, (float)(2.0 * R / (ns64 - 1.0)),
                                      (uint32_t*)pl.ptr(ctx, i_key), (uint32_t*)pl.ptr(ctx, i_hist),
                                      (int32_t*)pl.ptr(ctx, i_order), ctx->stream));
    a.order = (const int32_t*)pl.ptr(ctx, i_order);
  }
  HIP_TRY(ctx, launch_line_simplex(a, ctx->stream));
  return MORSE_OK;
}

int morse_chi2_grad(morse_ctx* ctx, const morse_map_view* maps, int32_t n_maps,
                    const morse_lightcurves* lcs, int64_t n, const double* d_params,
                    const int32_t* d_event, const int32_t* d_map_index, double* d_chi2,
                    double* d_grad, double* d_fs, double* d_fb) {
  if (!ctx) return fail(nullptr, MORSE_EINVAL, "ctx is NULL");
  int rc;
  Plan pl;
  size_t i_sums, i_wF, i_quad;
  if ((rc = plan_candidates(ctx, maps, n_maps, lcs, n, pl, i_sums, i_wF, i_quad))) return rc;
  if (n > 0 && (!d_params || !d_event || !d_map_index))
    return fail(ctx, MORSE_EINVAL, "d_params / d_event / d_map_index is NULL");
  if (n > INT32_MAX) return fail(ctx, MORSE_ERANGE, "more than 2^31 - 1 candidates");
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  const bool ordered = order_helps(n, n_maps, lcs->n_events);
  const size_t i_order = pl.add(ordered ? 4 * (size_t)n : 0), i_key = pl.add(ordered ? 4 * (size_t)n : 0),
               i_tc = pl.add(ordered ? sizeof(TrajC) * (size_t)n : 0),
               i_hist = pl.add(ordered ? 4 * (size_t)order_bins(n_maps, lcs->n_events) : 0);
  if ((rc = reserve(ctx, pl.total()))) return rc;
  GradArgs a{};
  MapC* d_maps;
  std::vector<MapC> hm;
  if ((rc = setup_candidates(ctx, maps, n_maps, lcs, pl, i_sums, i_wF, i_quad, a.lc, d_maps, hm))) return rc;
  a.n = n;
  a.tc = ordered ? (TrajC*)pl.ptr(ctx, i_tc) : nullptr;
  a.params = d_params;
  a.event = d_event;
  a.mapidx = d_map_index;
  a.maps = d_maps;
  a.n_events = lcs->n_events;
  a.n_maps = n_maps;
  a.chi2 = d_chi2;
  a.grad = d_grad;
  a.fs = d_fs;
  a.fb = d_fb;
  if (ordered) {
    int32_t* order = (int32_t*)pl.ptr(ctx, i_order);
    HIP_TRY(ctx, launch_cand_order(a, hm.data(), (uint32_t*)pl.ptr(ctx, i_key), (uint32_t*)pl.ptr(ctx, i_hist), order,
                                   ctx->stream));
    a.order = order;
  }
  LaunchTimer tm{ctx, MORSE_KERNEL_GRADIENT};
  HIP_TRY(ctx, tm.begin(ctx->stream));
  HIP_TRY(ctx, launch_chi2_grad(a, ctx->stream));
  HIP_TRY(ctx, tm.end(ctx->stream));
  return MORSE_OK;
}

int morse_chi2_grad_noalloc(morse_ctx* ctx, const morse_map_view* maps, int32_t n_maps,
                            const morse_lightcurves* lcs, int64_t n, const double* d_params,
                            const int32_t* d_event, const int32_t* d_map_index, double* d_chi2,
                            double* d_grad, double* d_fs, double* d_fb) {
  if (!ctx) return fail(nullptr, MORSE_EINVAL, "ctx is NULL");
  int rc;
  Plan pl;
  size_t i_sums, i_wF, i_quad;
  if ((rc = plan_candidates(ctx, maps, n_maps, lcs, n, pl, i_sums, i_wF, i_quad))) return rc;
  if (n > 0 && (!d_params || !d_event || !d_map_index))
    return fail(ctx, MORSE_EINVAL, "d_params / d_event / d_map_index is NULL");
  const int32_t ne = lcs->n_events;
  const size_t b_off = (8 * (size_t)(ne + 1) + 255) & ~size_t(255);
  const size_t b_tref = (8 * (size_t)ne + 255) & ~size_t(255);
  const size_t i_meta = pl.add(b_off + b_tref + sizeof(MapC) * n_maps);
  const size_t i_tc = pl.add((sizeof(TrajC) + 8) * (size_t)n);  // the stated limit counts 40 bytes a candidate for them
  const size_t i_order = pl.add(4 * (size_t)n), i_key = pl.add(4 * (size_t)n),
               i_hist = pl.add(4 * (size_t)order_bins(n_maps, ne));
  if (pl.total() > kNoallocScratchBytes)
    return fail(ctx, MORSE_ERANGE,
                "needs %.1f MiB of scratch; the allocation-free entry point holds %zu MiB "
                "(packed maps, light-curve preparation and candidate constants)",
                pl.total() / 1048576.0, kNoallocScratchBytes >> 20);
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  char* base = nullptr;
  if ((rc = noalloc_scratch(ctx->device, &base))) return fail(ctx, rc, "%s", morse_last_error(nullptr));
  // metadata: event offsets | reference times | map table, put on every call (the array keeps
  // whatever the last call on this GPU left in it)
  std::vector<MapC> hm(n_maps);
  for (int i = 0; i < n_maps; ++i) hm[i] = make_mapc(maps[i].d_map, maps[i].window);
  assign_quads(hm, pl.ptr_at(base, i_quad));
  char* meta = pl.ptr_at(base, i_meta);
  MapC* d_maps = (MapC*)(meta + b_off + b_tref);
  std::vector<char> block(b_off + b_tref + sizeof(MapC) * n_maps);
  std::memcpy(block.data(), lcs->h_offsets, 8 * (size_t)(ne + 1));
  std::memcpy(block.data() + b_off, lcs->h_t_ref, 8 * (size_t)ne);
  std::memcpy(block.data() + b_off + b_tref, hm.data(), sizeof(MapC) * n_maps);
  // 20,000 events: 146 us copied, 365 by value in 90 launches; 1000 events (16 KiB): 58 and 52
  if ((rc = put_now(ctx, meta, block))) return rc;
  GradArgs a{};
  a.lc.t = lcs->d_t;
  a.lc.w = lcs->d_weight;
  a.lc.F = lcs->d_flux;
  a.lc.wFc = (double*)pl.ptr_at(base, i_wF);
  a.lc.off = (const int64_t*)meta;
  a.lc.sums = (double*)pl.ptr_at(base, i_sums);
  a.lc.t_ref = (const double*)(meta + b_off);
  HIP_TRY(ctx, prepare_candidates(a.lc, ne, d_maps, hm, ctx->stream));
  a.n = n;
  a.params = d_params;
  a.event = d_event;
  a.mapidx = d_map_index;
  a.maps = d_maps;
  a.n_events = ne;
  a.n_maps = n_maps;
  a.chi2 = d_chi2;
  a.grad = d_grad;
  a.fs = d_fs;
  a.fb = d_fb;
  if (order_helps(n, n_maps, ne)) {
    int32_t* order = (int32_t*)pl.ptr_at(base, i_order);
    a.tc = (TrajC*)pl.ptr_at(base, i_tc);
    HIP_TRY(ctx, launch_cand_order(a, hm.data(), (uint32_t*)pl.ptr_at(base, i_key), (uint32_t*)pl.ptr_at(base, i_hist),
                                   order, ctx->stream));
    a.order = order;
  }
  HIP_TRY(ctx, launch_chi2_grad(a, ctx->stream));
  return MORSE_OK;
}

int morse_refine(morse_ctx* ctx, const morse_map_view* maps, int32_t n_maps,
                 const morse_lightcurves* lcs, int64_t n, double* d_params,
                 const int32_t* d_event, const int32_t* d_map_index,
                 const morse_lbfgs_opts* opts, double* d_chi2_out, double* d_chi2_init) {
  if (!ctx) return fail(nullptr, MORSE_EINVAL, "ctx is NULL");
  if (!opts) return fail(ctx, MORSE_EINVAL, "opts is NULL");
  if (opts->steps < 0 || opts->steps > 100000 || opts->history < 1 || opts->history > 16 ||
      opts->max_ls < 1 || !(opts->c1 > 0 && opts->c1 < 1) || !(opts->shrink > 0 && opts->shrink < 1))
    return fail(ctx, MORSE_EINVAL, "invalid L-BFGS options");
  int rc;
  Plan pl;
  size_t i_sums, i_wF, i_quad;
  if ((rc = plan_candidates(ctx, maps, n_maps, lcs, n, pl, i_sums, i_wF, i_quad))) return rc;
  if (n > 0 && (!d_params || !d_event || !d_map_index || !d_chi2_out))
    return fail(ctx, MORSE_EINVAL, "d_params / d_event / d_map_index / d_chi2_out is NULL");
  if (n == 0) return MORSE_OK;
  if (n > INT32_MAX) return fail(ctx, MORSE_ERANGE, "more than 2^31 - 1 candidates");
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  // One launch runs up to 1024 rounds, so that none lasts long; timed, each round is a launch.
  const int32_t span = timed(ctx, MORSE_KERNEL_GRADIENT) ? 1 : 1024;
  const bool ordered = order_helps(n, n_maps, lcs->n_events);
  std::vector<MapC> sizes(n_maps);
  for (int i = 0; i < n_maps; ++i) sizes[i] = make_mapc(maps[i].d_map, maps[i].window);
  const bool beyond_cache = maps_exceed_cache(sizes.data(), n_maps);
  const bool split = refine_by_round(n, beyond_cache),
             four = refine_by_four(n, lcs->h_offsets[lcs->n_events] / lcs->n_events, beyond_cache);
  const size_t i_order = pl.add(ordered ? 4 * (size_t)n : 0), i_key = pl.add(ordered ? 4 * (size_t)n : 0),
               i_hist = pl.add(ordered ? 4 * (size_t)order_bins(n_maps, lcs->n_events) : 0),
               i_state = pl.add(split || opts->steps >= span ? sizeof(RefineState) * (size_t)n : 0);
  if ((rc = reserve(ctx, pl.total()))) return rc;
  GradArgs a{};
  MapC* d_maps;
  std::vector<MapC> hm;
  if ((rc = setup_candidates(ctx, maps, n_maps, lcs, pl, i_sums, i_wF, i_quad, a.lc, d_maps, hm))) return rc;
  a.n = n;
  a.event = d_event;
  a.mapidx = d_map_index;
  a.maps = d_maps;
  a.n_events = lcs->n_events;
  a.n_maps = n_maps;
  if (ordered) {
    int32_t* order = (int32_t*)pl.ptr(ctx, i_order);
    HIP_TRY(ctx, launch_cand_order(a, hm.data(), (uint32_t*)pl.ptr(ctx, i_key), (uint32_t*)pl.ptr(ctx, i_hist), order,
                                   ctx->stream));
    a.order = order;
  }
  RefineArgs s{};
  s.params = d_params;
  s.chi2_out = d_chi2_out;
  s.chi2_init = d_chi2_init;
  s.state = (RefineState*)pl.ptr(ctx, i_state);
  s.m = opts->history;
  s.max_ls = opts->max_ls;
  s.c1 = opts->c1;
  s.shrink = opts->shrink;
  s.steps = opts->steps;
  if (split) {
    HIP_TRY(ctx, launch_round_start(a, s, ctx->stream));
    for (int32_t r = 0; r <= opts->steps; ++r) {
      LaunchTimer tm{ctx, MORSE_KERNEL_GRADIENT};
      HIP_TRY(ctx, tm.begin(ctx->stream));
      HIP_TRY(ctx, launch_round_eval(a, s, ctx->stream));
      HIP_TRY(ctx, tm.end(ctx->stream));
      HIP_TRY(ctx, launch_round_update(a, s, r, ctx->stream));
    }
    return MORSE_OK;
  }
  for (s.r0 = 0; s.r0 <= opts->steps; s.r0 = s.r1) {
    s.r1 = std::min(s.r0 + span, opts->steps + 1);
    LaunchTimer tm{ctx, MORSE_KERNEL_GRADIENT};
    HIP_TRY(ctx, tm.begin(ctx->stream));
    HIP_TRY(ctx, launch_refine(a, s, four, ctx->stream));
    HIP_TRY(ctx, tm.end(ctx->stream));
  }
  return MORSE_OK;
}

}  // extern "C"
