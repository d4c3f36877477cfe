// C ABI, trajectory search: plain and batched (one scoring launch) searches,
// best-per-map and top-k selection, the autotuner of the batched shape and its cache,
// and candidate lists from the top-k.

#include "host.h"

using namespace morse;
using namespace morse::host;

namespace {

struct TuneCfg {
  int traj_per_item;
  int waves_per_block;
  int tu;
};
// Candidate shapes of the batched search tried by the autotuner (saved caches name them by
// index: a change of the table or of what makes a shape fast raises the version in
// shape_class).  traj_per_item = trajectories per wavefront, tu = trajectories scored together
// by one wavefront (sharing light-curve loads).
constexpr TuneCfg kTune[] = {
    {8, 4, 2},  {8, 4, 1},  {16, 4, 2}, {8, 8, 2},  {32, 8, 2}, {4, 4, 2},  {16, 8, 4},
    {8, 2, 2},  {16, 4, 4}, {32, 8, 1}, {8, 2, 1},  {64, 4, 4}, {32, 8, 4}, {16, 2, 4},
    {8, 8, 4},  {4, 8, 4},  {4, 4, 4},  {4, 2, 4},  {4, 1, 4},  {2, 4, 2},  {2, 2, 2},
    {1, 4, 1},  {1, 2, 1},
};
constexpr int kShapeMany = 17, kShapeSome = 19, kShapeFew = 21;
// The shape before tuning, by the number of trajectories to score (over all events and
// maps).  A few leave the chip part empty, and one trajectory a wavefront with four chunks
// in flight is over soonest; many are scored with the fewest instructions, four a
// wavefront.  Measured on one map, us for TU = 1 / 2 / 4: 1024 trajectories x 1000 points
// 15.6 / 17.6 / 22.6, 4096 x 1000 23.7 / 23.2 / 27.6, 16384 x 1000 52 / 46 / 49, 32768 x 1000
// 89 / 70 / 65; 1024 x 6000 31 / 47 / 72, 16384 x 6000 173 / 130 / 119.  The length of the light
// curves is not asked for: with long ones four a wavefront pay from fewer trajectories on than
// the rule gives them (the last figures: 130 where the autotuner finds 119).
int default_shape(int64_t n) { return n <= 4096 ? kShapeFew : n <= 16384 ? kShapeSome : kShapeMany; }
constexpr int kNumTune = sizeof(kTune) / sizeof(kTune[0]);
// k_search_batched is compiled for at most 512 lanes (8 wavefronts) per workgroup and
// instantiated for TU = 1, 2 and 4; a shape outside that would not launch.
constexpr bool tune_shapes_valid() {
  for (const TuneCfg& c : kTune)
    if (c.waves_per_block < 1 || c.waves_per_block > 8 || c.traj_per_item < 1 || !(c.tu == 1 || c.tu == 2 || c.tu == 4))
      return false;
  return true;
}
static_assert(tune_shapes_valid(), "a batched-search shape the kernel cannot launch");
constexpr bool tune_shapes_differ() {
  for (int i = 0; i < kNumTune; ++i)
    for (int j = 0; j < i; ++j)
      if (kTune[i].traj_per_item == kTune[j].traj_per_item && kTune[i].waves_per_block == kTune[j].waves_per_block &&
          kTune[i].tu == kTune[j].tu)
        return false;
  return true;
}
static_assert(tune_shapes_differ(), "a shape listed twice is timed twice");
static_assert(kTune[kShapeMany].tu == 4 && kTune[kShapeSome].tu == 2 && kTune[kShapeFew].tu == 1, "default shapes");


}  // namespace

// =============================================================================
// Search planning shared by search / autotune.
namespace {

struct SearchPlan {
  int64_t n_traj = 0;
  int32_t n_events = 0, n_maps = 0;
  int64_t n_pts = 0;
  TrajC* tc = nullptr;
  MapC* d_maps = nullptr;
  std::vector<MapC> h_maps;
  LcView lc{};
  double* chi2 = nullptr;  // output or workspace
  char* select = nullptr;  // workspace of the selections
  SelectScratch sel{};
  int num_cu = 256;
  double* axes = nullptr;
  // trajectory lists: scoring order of the batched kernel and its counting-sort counters
  int32_t* perm = nullptr;
  uint32_t* perm_key = nullptr;
  uint32_t* perm_hist = nullptr;
  int32_t perm_lists = 0;
};

int validate_search(morse_ctx* ctx, const morse_map_view* maps, int32_t n_maps,
                    const morse_lightcurves* lcs, const morse_trajectories* trajs) {
  int rc;
  if (!maps || n_maps <= 0) return fail(ctx, MORSE_EINVAL, "need n_maps >= 1 maps");
  for (int i = 0; i < n_maps; ++i) {
    if (!maps[i].d_map) return fail(ctx, MORSE_EINVAL, "map %d: d_map is NULL", i);
    if ((rc = check_window(ctx, &maps[i].window, "map window"))) return rc;
  }
  if ((rc = check_lightcurves(ctx, lcs))) return rc;
  if (!trajs) return fail(ctx, MORSE_EINVAL, "trajs is NULL");
  if (trajs->kind == MORSE_TRAJ_GRID) {
    if (trajs->n_u0 <= 0 || trajs->n_alpha <= 0 || trajs->n_t0 <= 0 || trajs->n_tE <= 0 ||
        !trajs->h_u0 || !trajs->h_alpha || !trajs->h_t0 || !trajs->h_tE)
      return fail(ctx, MORSE_EINVAL, "grid trajectories: empty axis or NULL array");
    for (int i = 0; i < trajs->n_tE; ++i)
      if (!(trajs->h_tE[i] > 0 && std::isfinite(trajs->h_tE[i])))
        return fail(ctx, MORSE_EINVAL, "grid trajectories: tE must be finite and > 0");
    for (int i = 0; i < trajs->n_u0; ++i)
      if (!std::isfinite(trajs->h_u0[i])) return fail(ctx, MORSE_EINVAL, "grid: u0 not finite");
    for (int i = 0; i < trajs->n_alpha; ++i)
      if (!std::isfinite(trajs->h_alpha[i])) return fail(ctx, MORSE_EINVAL, "grid: alpha not finite");
    for (int i = 0; i < trajs->n_t0; ++i)
      if (!std::isfinite(trajs->h_t0[i])) return fail(ctx, MORSE_EINVAL, "grid: t0 not finite");
  } else if (trajs->kind == MORSE_TRAJ_LIST) {
    if (trajs->n <= 0 || !trajs->d_params) return fail(ctx, MORSE_EINVAL, "list trajectories: n <= 0 or NULL");
  } else {
    return fail(ctx, MORSE_EINVAL, "unknown trajectory kind %d", trajs->kind);
  }
  return MORSE_OK;
}

int64_t traj_count(const morse_trajectories* t) {
  return t->kind == MORSE_TRAJ_GRID ? (int64_t)t->n_u0 * t->n_alpha * t->n_t0 * t->n_tE : t->n;
}

// Reserve the workspace and upload the host metadata of a search into its own buffer
// (skipped when the same metadata is already resident).  Enqueues nothing else.
int plan_search(morse_ctx* ctx, const morse_map_view* maps, int32_t n_maps,
                const morse_lightcurves* lcs, const morse_trajectories* trajs,
                const morse_search_out* out, SearchPlan& sp) {
  int rc;
  sp.n_traj = traj_count(trajs);
  sp.n_events = lcs->n_events;
  sp.n_maps = n_maps;
  sp.n_pts = lcs->h_offsets[lcs->n_events];
  const int64_t n_tc = (trajs->kind == MORSE_TRAJ_LIST && !trajs->shared)
                           ? sp.n_traj * lcs->n_events
                           : sp.n_traj;
  const int64_t n_out = (int64_t)sp.n_events * n_maps * sp.n_traj;
  const int32_t k = out->top_k;
  const bool best = out->d_best_chi2 || out->d_best_idx;
  const bool need_chi2 = !out->d_chi2 && (best || k > 0);
  const int n_axes = trajs->kind == MORSE_TRAJ_GRID
                         ? trajs->n_u0 + trajs->n_alpha + trajs->n_t0 + trajs->n_tE
                         : 0;
  if ((rc = check_quad_size(ctx, maps, n_maps))) return rc;
  // lists are scored in an order grouped by direction (one counting sort per list)
  sp.perm_lists = (trajs->kind == MORSE_TRAJ_LIST && sp.n_traj > 0) ? (int32_t)(n_tc / sp.n_traj) : 0;
  if ((int64_t)sp.perm_lists * kPermBins > kPermBinsMax || n_tc > INT32_MAX) sp.perm_lists = 0;
  sp.sel = select_scratch(best ? (int64_t)sp.n_events * n_maps : 0, sp.n_traj, k > 0 ? sp.n_events : 0,
                          (int64_t)n_maps * sp.n_traj, k, ctx->num_cu);
  Plan pl;
  const size_t i_quad = pl.add(quad_region_bytes(maps, n_maps)),
               i_sums = pl.add(24 * (size_t)sp.n_events), i_sorted = pl.add(4 * (size_t)sp.n_events),
               i_wF = pl.add(8 * (size_t)sp.n_pts), i_tc = pl.add(sizeof(TrajC) * (size_t)n_tc),
               i_chi = pl.add(need_chi2 ? 8 * (size_t)n_out : 0),
               i_sel = pl.add(sp.sel.bytes),
               i_perm = pl.add(sp.perm_lists ? 4 * (size_t)n_tc : 0),
               i_pk = pl.add(sp.perm_lists ? 4 * (size_t)n_tc : 0),
               i_ph = pl.add(4 * (size_t)sp.perm_lists * kPermBins);
  if ((rc = reserve(ctx, pl.total()))) return rc;
  if (sp.perm_lists) {
    sp.perm = (int32_t*)pl.ptr(ctx, i_perm);
    sp.perm_key = (uint32_t*)pl.ptr(ctx, i_pk);
    sp.perm_hist = (uint32_t*)pl.ptr(ctx, i_ph);
  }
  double* d_sums = (double*)pl.ptr(ctx, i_sums);
  double* d_wF = (double*)pl.ptr(ctx, i_wF);
  sp.tc = (TrajC*)pl.ptr(ctx, i_tc);
  sp.chi2 = out->d_chi2 ? out->d_chi2 : (double*)pl.ptr(ctx, i_chi);
  sp.select = pl.ptr(ctx, i_sel);
  sp.num_cu = ctx->num_cu;
  sp.h_maps.resize(n_maps);
  for (int i = 0; i < n_maps; ++i) sp.h_maps[i] = make_mapc(maps[i].d_map, maps[i].window);
  assign_quads(sp.h_maps, pl.ptr(ctx, i_quad));
  // metadata buffer: offsets | reference times | map table | grid axes
  MetaBlock mb;
  const size_t o_off = mb.add(lcs->h_offsets, 8 * (size_t)(sp.n_events + 1)),
               o_tref = mb.add(lcs->h_t_ref, 8 * (size_t)sp.n_events),
               o_maps = mb.add(sp.h_maps.data(), sizeof(MapC) * n_maps);  // with the packed cells' addresses
  const size_t o_axes = mb.bytes.size();
  if (n_axes) {
    mb.add(trajs->h_u0, 8 * (size_t)trajs->n_u0, 8);
    mb.add(trajs->h_alpha, 8 * (size_t)trajs->n_alpha, 8);
    mb.add(trajs->h_t0, 8 * (size_t)trajs->n_t0, 8);
    mb.add(trajs->h_tE, 8 * (size_t)trajs->n_tE, 8);
  }
  Hasher key;
  key.bytes(mb.bytes.data(), mb.bytes.size());
  char* meta;
  if ((rc = put_meta(ctx, ctx->smeta, mb.bytes, key.h, &meta))) return rc;
  int64_t* d_off = (int64_t*)(meta + o_off);
  double* d_tref = (double*)(meta + o_tref);
  sp.d_maps = (MapC*)(meta + o_maps);
  sp.axes = n_axes ? (double*)(meta + o_axes) : nullptr;
  sp.lc.t = lcs->d_t;
  sp.lc.w = lcs->d_weight;
  sp.lc.F = lcs->d_flux;
  sp.lc.wFc = d_wF;
  sp.lc.off = d_off;
  sp.lc.sums = d_sums;
  sp.lc.t_ref = d_tref;
  sp.lc.sorted = (uint32_t*)pl.ptr(ctx, i_sorted);
  return MORSE_OK;
}

// Preparation (light-curve sums, trajectory constants, map packing, zeroed counters).
hipError_t enqueue_prep(const SearchPlan& sp, const morse_trajectories* trajs, hipStream_t st) {
  PrepArgs a{};
  a.lc = sp.lc;
  a.n_events = sp.n_events;
  a.n_traj = sp.n_traj;
  a.n = sp.n_traj;
  a.axes = sp.axes;
  if (trajs->kind == MORSE_TRAJ_GRID) {
    a.nu = trajs->n_u0;
    a.na = trajs->n_alpha;
    a.nt = trajs->n_t0;
    a.ne = trajs->n_tE;
  } else {
    a.params = trajs->d_params;
    if (!trajs->shared) a.n *= sp.n_events;
    a.key = sp.perm ? sp.perm_key : nullptr;
  }
  a.tc = sp.tc;
  a.zero = (uint32_t*)sp.select;
  a.n_zero = sp.sel.zero_bytes / 4;
  a.maps = sp.d_maps;
  a.n_maps = sp.n_maps;
  const hipError_t e = launch_prep(a, sp.h_maps.data(), st);
  if (e != hipSuccess || !sp.perm) return e;
  return launch_traj_perm(sp.perm_key, sp.n_traj, sp.perm_lists, sp.perm_hist, sp.perm, st);
}

hipError_t enqueue_select(const SearchPlan& sp, const morse_search_out* out, hipStream_t st) {
  hipError_t e = hipSuccess;
  if (out->d_best_chi2 || out->d_best_idx)
    e = launch_best(sp.chi2, (int64_t)sp.n_events * sp.n_maps, sp.n_traj, out->d_best_chi2,
                    out->d_best_idx, sp.select, sp.sel, sp.num_cu, st);
  if (e == hipSuccess && out->top_k > 0)
    e = launch_topk(sp.chi2, sp.n_events, (int64_t)sp.n_maps * sp.n_traj, out->top_k,
                    out->d_topk_chi2, out->d_topk_idx, sp.select, sp.sel, sp.num_cu, st);
  return e;
}

BatchedArgs batched_args(morse_ctx* ctx, const SearchPlan& sp, const morse_trajectories* trajs,
                         const morse_search_out* out, const TuneCfg& cfg) {
  BatchedArgs a;
  a.tc = sp.tc;
  a.n_traj = sp.n_traj;
  a.shared = (trajs->kind == MORSE_TRAJ_GRID || trajs->shared) ? 1 : 0;
  a.n_events = sp.n_events;
  a.n_maps = sp.n_maps;
  a.maps = sp.d_maps;
  a.lc = sp.lc;
  a.out.chi2 = sp.chi2;
  a.out.fs = out->d_fs;
  a.out.fb = out->d_fb;
  a.nu = a.na = a.nt = a.ne = 0;
  if (trajs->kind == MORSE_TRAJ_GRID) {
    a.nu = trajs->n_u0;
    a.na = trajs->n_alpha;
    a.nt = trajs->n_t0;
    a.ne = trajs->n_tE;
  }
  a.perm = sp.perm;
  a.traj_per_item = cfg.traj_per_item;
  a.waves_per_block = cfg.waves_per_block;
  a.tu = cfg.tu;
  a.centred = 1;
  for (const MapC& m : sp.h_maps) a.centred &= (m.sx == 0.0f && m.sy == 0.0f) ? 1 : 0;
  return a;
}

// Reads an autotune cache ({"class": index, ...}); false when the file cannot be read.
bool read_tune_cache(const char* path, std::map<std::string, int>& all) {
  std::ifstream in(path);
  if (!in) return false;
  std::string txt((std::istreambuf_iterator<char>(in)), std::istreambuf_iterator<char>());
  size_t p = 0;
  while ((p = txt.find('"', p)) != std::string::npos) {
    size_t q = txt.find('"', p + 1);
    if (q == std::string::npos) break;
    std::string k = txt.substr(p + 1, q - p - 1);
    size_t colon = txt.find(':', q);
    if (colon == std::string::npos) break;
    all[k] = std::atoi(txt.c_str() + colon + 1);
    p = txt.find_first_of(",}", colon);
    if (p == std::string::npos) break;
  }
  return true;
}

std::string shape_class(const SearchPlan& sp) {
  auto bucket = [](double v) { return (int)std::floor(std::log2(std::max(v, 1.0))); };
  std::ostringstream s;
  s << "gfx950|v4|maps" << bucket(sp.n_maps) << "|pts" << bucket((double)sp.n_pts / sp.n_events)
    << "|traj" << bucket((double)sp.n_traj) << "|ev" << bucket(sp.n_events);
  return s.str();
}

}  // namespace

extern "C" {


int morse_search(morse_ctx* ctx, const morse_map_view* maps, int32_t n_maps,
                 const morse_lightcurves* lcs, const morse_trajectories* trajs, int32_t mode,
                 morse_search_out* out) {
  if (!ctx) return fail(nullptr, MORSE_EINVAL, "ctx is NULL");
  if (!out) return fail(ctx, MORSE_EINVAL, "out is NULL");
  int rc;
  if ((rc = validate_search(ctx, maps, n_maps, lcs, trajs))) return rc;
  if (mode != MORSE_SEARCH_PLAIN && mode != MORSE_SEARCH_BATCHED)
    return fail(ctx, MORSE_EINVAL, "unknown search mode %d", mode);
  if (out->top_k < 0 || out->top_k > 4096)
    return fail(ctx, out->top_k < 0 ? MORSE_EINVAL : MORSE_EUNSUPPORTED, "top_k must be in [0, 4096]");
  if (out->top_k > 0 && (!out->d_topk_chi2 || !out->d_topk_idx))
    return fail(ctx, MORSE_EINVAL, "top_k > 0 needs d_topk_chi2 and d_topk_idx");
  if (out->top_k > 0 && ((double)n_maps * (double)traj_count(trajs) >= 4294967295.0 ||
                         lcs->n_events > 65535))
    return fail(ctx, MORSE_ERANGE, "top-k needs n_maps * n_traj < 2^32 and at most 65535 events");
  {
    const int64_t nt = traj_count(trajs);
    if ((double)nt * lcs->n_events * n_maps >= 9.0e18 ||
        (double)nt * lcs->n_events * n_maps >= 2147483647.0)
      return fail(ctx, MORSE_ERANGE, "too many (event, map, trajectory) items");
  }
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  SearchPlan sp;
  if ((rc = plan_search(ctx, maps, n_maps, lcs, trajs, out, sp))) return rc;

  if (mode == MORSE_SEARCH_PLAIN) {
    HIP_TRY(ctx, enqueue_prep(sp, trajs, ctx->stream));
    for (int32_t e = 0; e < sp.n_events; ++e) {
      const TrajC* tc = sp.tc + ((trajs->kind == MORSE_TRAJ_LIST && !trajs->shared) ? (int64_t)e * sp.n_traj : 0);
      for (int32_t m = 0; m < n_maps; ++m) {
        const int64_t base = ((int64_t)e * n_maps + m) * sp.n_traj;
        SearchOut so{sp.chi2 + base, out->d_fs ? out->d_fs + base : nullptr,
                     out->d_fb ? out->d_fb + base : nullptr};
        LaunchTimer tm{ctx, MORSE_KERNEL_SEARCH};
        HIP_TRY(ctx, tm.begin(ctx->stream));
        HIP_TRY(ctx, launch_search_plain(tc, sp.n_traj, sp.lc, e, lcs->h_offsets[e + 1] - lcs->h_offsets[e],
                                         sp.h_maps[m], so, 4, ctx->stream));
        HIP_TRY(ctx, tm.end(ctx->stream));
      }
    }
    HIP_TRY(ctx, enqueue_select(sp, out, ctx->stream));
    return MORSE_OK;
  }

  // batched: one scoring launch; with preparation and selection two (a grid, chi-squares alone) to
  // seventeen (lists, new metadata, the best of all and a long top-k) in all.
  // Launched one by one (3 us of the host each): 1024 trajectories with top-64 take 28 us a call,
  // from a captured graph of the same launches 45 us, and 80 to 300 where the graph has to be
  // captured again.
  auto it = ctx->tune.find(shape_class(sp));
  const int cfg_idx =
      it == ctx->tune.end() ? default_shape(sp.n_traj * sp.n_events * sp.n_maps) : it->second;
  const BatchedArgs a = batched_args(ctx, sp, trajs, out, kTune[cfg_idx]);
  HIP_TRY(ctx, enqueue_prep(sp, trajs, ctx->stream));
  LaunchTimer tm{ctx, MORSE_KERNEL_SEARCH};
  HIP_TRY(ctx, tm.begin(ctx->stream));
  HIP_TRY(ctx, launch_search_batched(a, ctx->stream));
  HIP_TRY(ctx, tm.end(ctx->stream));
  HIP_TRY(ctx, enqueue_select(sp, out, ctx->stream));
  return MORSE_OK;
}

int morse_autotune(morse_ctx* ctx, const morse_map_view* maps, int32_t n_maps,
                   const morse_lightcurves* lcs, const morse_trajectories* trajs,
                   const char* cache_path, int32_t* h_best_config) {
  if (!ctx) return fail(nullptr, MORSE_EINVAL, "ctx is NULL");
  int rc;
  if ((rc = validate_search(ctx, maps, n_maps, lcs, trajs))) return rc;
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  morse_search_out out{};
  SearchPlan sp;
  if ((rc = plan_search(ctx, maps, n_maps, lcs, trajs, &out, sp))) return rc;
  const std::string cls = shape_class(sp);
  // time each candidate on (at most) the first 16 events x 8 maps of the problem
  SearchPlan sub = sp;
  sub.n_events = std::min(sp.n_events, 16);
  sub.n_maps = std::min(sp.n_maps, 8);
  const size_t need = (size_t)sub.n_events * sub.n_maps * sp.n_traj * 8;
  double* scratch = nullptr;
  HIP_TRY(ctx, hipMalloc((void**)&scratch, need));
  sub.chi2 = scratch;
  hipError_t e = enqueue_prep(sp, trajs, ctx->stream);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (e == hipSuccess) e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  int best = 0;
  float best_ms = 1e30f;
  for (int c = 0; c < kNumTune && e == hipSuccess; ++c) {
    const BatchedArgs a = batched_args(ctx, sub, trajs, &out, kTune[c]);
    float ms = 0.0f;
    for (int rep = 0; rep < 2 && e == hipSuccess; ++rep) {
      e = hipEventRecord(e0, ctx->stream);
      if (e == hipSuccess) e = launch_search_batched(a, ctx->stream);
      if (e == hipSuccess) e = hipEventRecord(e1, ctx->stream);
      if (e == hipSuccess) e = hipEventSynchronize(e1);
      if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    }
    if (e == hipSuccess && ms < best_ms) {
      best_ms = ms;
      best = c;
    }
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipFree(scratch);
  if (e != hipSuccess) return fail(ctx, MORSE_EHIP, "autotune: %s", hipGetErrorString(e));
  ctx->tune[cls] = best;
  if (h_best_config) *h_best_config = best;
  if (cache_path) {
    // JSON object {"class": index, ...}: merge with the existing file
    std::map<std::string, int> all;
    read_tune_cache(cache_path, all);
    all[cls] = best;
    std::ofstream o(cache_path);
    o << "{";
    bool first = true;
    for (auto& kv : all) {
      o << (first ? "" : ", ") << "\"" << kv.first << "\": " << kv.second;
      first = false;
    }
    o << "}\n";
  }
  return MORSE_OK;
}

int morse_autotune_load(morse_ctx* ctx, const char* cache_path, int32_t* h_loaded) {
  if (!ctx) return fail(nullptr, MORSE_EINVAL, "ctx is NULL");
  if (!cache_path) return fail(ctx, MORSE_EINVAL, "cache_path is NULL");
  std::map<std::string, int> all;
  if (!read_tune_cache(cache_path, all))
    return fail(ctx, MORSE_EUNSUPPORTED, "cannot read autotune cache %s", cache_path);
  int32_t n = 0;
  for (const auto& kv : all) {
    if (kv.second < 0 || kv.second >= kNumTune) continue;
    ctx->tune[kv.first] = kv.second;
    ++n;
  }
  if (h_loaded) *h_loaded = n;
  return MORSE_OK;
}

int morse_candidates_from_topk(morse_ctx* ctx, const morse_trajectories* trajs, int32_t n_events,
                               int32_t n_maps, int32_t top_k, const int64_t* d_topk_idx,
                               double* d_params, int32_t* d_event, int32_t* d_map_index) {
  if (!ctx) return fail(nullptr, MORSE_EINVAL, "ctx is NULL");
  if (!trajs) return fail(ctx, MORSE_EINVAL, "trajs is NULL");
  if (n_events <= 0 || n_maps <= 0 || top_k <= 0)
    return fail(ctx, MORSE_EINVAL, "n_events, n_maps and top_k must be >= 1");
  if (!d_topk_idx || !d_params || !d_event || !d_map_index)
    return fail(ctx, MORSE_EINVAL, "NULL device pointer");
  const int64_t n_traj = traj_count(trajs);
  if (n_traj <= 0) return fail(ctx, MORSE_EINVAL, "empty trajectory set");
  if (trajs->kind == MORSE_TRAJ_LIST && !trajs->d_params)
    return fail(ctx, MORSE_EINVAL, "list trajectories: d_params is NULL");
  if (trajs->kind == MORSE_TRAJ_GRID &&
      (!trajs->h_u0 || !trajs->h_alpha || !trajs->h_t0 || !trajs->h_tE))
    return fail(ctx, MORSE_EINVAL, "grid trajectories: NULL axis");
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  const double* axes = nullptr;
  int rc;
  if (trajs->kind == MORSE_TRAJ_GRID) {
    MetaBlock mb;
    mb.add(trajs->h_u0, 8 * (size_t)trajs->n_u0, 8);
    mb.add(trajs->h_alpha, 8 * (size_t)trajs->n_alpha, 8);
    mb.add(trajs->h_t0, 8 * (size_t)trajs->n_t0, 8);
    mb.add(trajs->h_tE, 8 * (size_t)trajs->n_tE, 8);
    // the auxiliary buffer keeps the search's resident workspace intact
    if ((rc = reserve_aux(ctx, mb.bytes.size()))) return rc;
    double* d = (double*)ctx->aux.p;
    if ((rc = put_now(ctx, d, mb.bytes))) return rc;
    axes = d;
  }
  HIP_TRY(ctx, launch_candidates(axes, trajs->n_u0, trajs->n_alpha, trajs->n_t0, trajs->n_tE,
                                 trajs->d_params, trajs->shared, n_traj, n_events, n_maps, top_k,
                                 d_topk_idx, d_params, d_event, d_map_index, ctx->stream));
  return MORSE_OK;
}

}  // extern "C"
