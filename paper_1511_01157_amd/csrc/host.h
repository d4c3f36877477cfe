// Host-side helpers shared by the C ABI's source files (api_*.hip): the context
// structure behind the opaque morse_ctx, error reporting, workspace and metadata
// buffers, argument validation and map descriptors.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <chrono>
#include <complex>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <sstream>
#include <string>
#include <vector>

#include "internal.h"
#include "stack.h"
#include "lines.h"
#include "simplex.h"


// A device buffer that grows.
struct Buffer {
  char* p = nullptr;
  size_t size = 0;
  bool named = false;  // a captured call used it: the caller's graph holds its address
};

// A device buffer of host metadata with the key of what it holds (see put_meta).
struct MetaBuf : Buffer {
  uint64_t key = 0;
};

struct morse_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  int num_cu = 256;
  Buffer ws;
  // outgrown buffers that graphs still name, freed with the context
  std::vector<char*> retired;
  std::string err;
  // host metadata of the searches and of the candidate entry points, each in a device
  // buffer of its own (never in the shared workspace, which the other entry points
  // overwrite) and uploaded only when its key changes
  MetaBuf smeta, cmeta;
  // source-radius stacks: direct-sum taps, FFT twiddle tables and the transforms of
  // the profile pairs, each kept until a call needs different ones
  MetaBuf stack_taps, fft_tw, fft_spec;
  // critical points and their caustic images of the last finite-source call (key: s, q,
  // phases)
  MetaBuf fs_crit;
  // split of the last stack call's radii (key of its arguments): direct radii with
  // their tap counts (taps in stack_taps, in this order), FFT radii, widest FFT stencil
  struct StackSplit {
    uint64_t key = 0;
    std::vector<int> direct_k, fft_k;
    std::vector<int32_t> ntaps;
    std::vector<int32_t> reach;  // per direct radius: the largest |offset| along x, then y
    size_t w_bytes = 0;  // the tap offsets follow the weights at this byte offset
    int rmx = 0, rmy = 0;
  } stack_split;
  // autotune choices per shape class
  std::map<std::string, int> tune;
  // small auxiliary device buffer, separate from the workspace
  Buffer aux;
  // disk-convolution taps resident on the device, and what the host knows of them
  MetaBuf taps;
  struct DiskTaps {
    int32_t n = 0, rx = 0, ry = 0;  // number, and the largest |offset| along x and y
    size_t w_bytes = 0;             // the offsets follow the weights at this byte offset
    const char* p = nullptr;
    const float* w() const { return (const float*)p; }
    const int32_t* off() const { return (const int32_t*)(p + w_bytes); }
  } disk;
  // slots of the ray statistics (not used by captured calls)
  char* stat_slots = nullptr;
  // kernel timing: enabled families, pending event pairs, free events, totals
  uint32_t timing_mask = 0;
  struct Timed {
    int32_t kernel;
    hipEvent_t a, b;
  };
  std::vector<Timed> timed;
  std::vector<hipEvent_t> free_events;
  double time_ms[3] = {0.0, 0.0, 0.0};
  int64_t launches[3] = {0, 0, 0};
};

namespace morse {
namespace host {

// Message of the last error of this thread (returned by morse_last_error(NULL)).
extern thread_local std::string g_thread_error;


inline int fail(morse_ctx* ctx, int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  if (ctx) ctx->err = buf;
  g_thread_error = buf;
  return code;
}

#define HIP_TRY(ctx, expr)                                                                   \
  do {                                                                                       \
    hipError_t e_ = (expr);                                                                  \
    if (e_ != hipSuccess)                                                                    \
      return fail((ctx), MORSE_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_));         \
  } while (0)

// FNV-1a over raw bytes, for keys of uploaded metadata.
struct Hasher {
  uint64_t h = 1469598103934665603ull;
  void bytes(const void* p, size_t n) {
    const unsigned char* c = (const unsigned char*)p;
    for (size_t i = 0; i < n; ++i) {
      h ^= c[i];
      h *= 1099511628211ull;
    }
  }
  template <class T>
  void pod(const T& v) {
    bytes(&v, sizeof(T));
  }
};

// Folds the pending timing events into the totals (waits for them).
inline hipError_t resolve_timers(morse_ctx* ctx) {
  for (const auto& t : ctx->timed) {
    hipError_t e = hipEventSynchronize(t.b);
    float ms = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, t.a, t.b);
    if (e != hipSuccess) return e;
    ctx->time_ms[t.kernel] += ms;
    ctx->launches[t.kernel] += 1;
    ctx->free_events.push_back(t.a);
    ctx->free_events.push_back(t.b);
  }
  ctx->timed.clear();
  return hipSuccess;
}

inline hipError_t take_event(morse_ctx* ctx, hipEvent_t* e) {
  if (!ctx->free_events.empty()) {
    *e = ctx->free_events.back();
    ctx->free_events.pop_back();
    return hipSuccess;
  }
  return hipEventCreate(e);
}

inline bool timed(const morse_ctx* ctx, int32_t kernel) { return (ctx->timing_mask >> kernel) & 1u; }

// Brackets one launch of a kernel family with events on `st` when the family is timed.
struct LaunchTimer {
  morse_ctx* ctx;
  int32_t kernel;
  hipEvent_t a = nullptr;
  hipError_t begin(hipStream_t st) {
    if (!timed(ctx, kernel)) return hipSuccess;
    hipError_t e = take_event(ctx, &a);
    return e == hipSuccess ? hipEventRecord(a, st) : e;
  }
  hipError_t end(hipStream_t st) {
    if (!a) return hipSuccess;
    hipEvent_t b = nullptr;
    hipError_t e = take_event(ctx, &b);
    if (e == hipSuccess) e = hipEventRecord(b, st);
    if (e != hipSuccess) return e;
    ctx->timed.push_back({kernel, a, b});
    a = nullptr;
    // bound the pending list for callers that never read the totals
    return ctx->timed.size() >= 4096 ? resolve_timers(ctx) : hipSuccess;
  }
};

// Bump allocator over the context workspace: first collect sizes, then reserve.
struct Plan {
  std::vector<size_t> sizes;
  size_t add(size_t bytes) {
    sizes.push_back((bytes + 255) & ~size_t(255));
    return sizes.size() - 1;
  }
  size_t total() const {
    size_t t = 0;
    for (size_t s : sizes) t += s;
    return t;
  }
  char* ptr(morse_ctx* ctx, size_t id) const { return ptr_at(ctx->ws.p, id); }
  char* ptr_at(char* base, size_t id) const {
    size_t off = 0;
    for (size_t i = 0; i < id; ++i) off += sizes[i];
    return base + off;
  }
};

// Whether work on the context's stream is being captured.
inline bool capturing(morse_ctx* ctx) {
  hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(ctx->stream, &c) != hipSuccess) (void)hipGetLastError();
  return c != hipStreamCaptureStatusNone;
}

// Room for `bytes` in a buffer of the context, which becomes `want` bytes long when it has to
// grow (its contents are then lost).  A buffer that a captured call used may be written by that
// call's graph for as long as the context lives: it is not freed before, and nothing is
// allocated under a capture (the call is refused, with nothing enqueued).
inline int grow(morse_ctx* ctx, Buffer& b, size_t bytes, size_t want, const char* what) {
  const bool cap = capturing(ctx);
  if (bytes > b.size) {
    if (cap)
      return fail(ctx, MORSE_EUNSUPPORTED, "%s of %zu bytes cannot be allocated under capture: make a call of this size before it",
                  what, bytes);
    if (b.p && b.named) {
      ctx->retired.push_back(b.p);
    } else if (b.p) {
      HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
      (void)hipFree(b.p);
    }
    b = Buffer{};
    if (hipMalloc((void**)&b.p, want) != hipSuccess) {
      b.p = nullptr;
      return fail(ctx, MORSE_ENOMEM, "%s allocation of %zu bytes failed", what, want);
    }
    b.size = want;
  }
  b.named = b.named || cap;
  return MORSE_OK;
}

inline int reserve(morse_ctx* ctx, size_t bytes) {
  const size_t mib = size_t(1) << 20;
  return grow(ctx, ctx->ws, bytes, (std::max(bytes, mib) + mib - 1) & ~(mib - 1), "workspace");
}

inline int reserve_aux(morse_ctx* ctx, size_t bytes) {
  return grow(ctx, ctx->aux, bytes, std::max(bytes, size_t(1) << 16), "auxiliary");
}

// The largest |offset| along x and along y of a tap table (pairs dx, dy).
inline void tap_reach(const std::vector<int32_t>& off, int32_t& rx, int32_t& ry) {
  rx = ry = 0;
  for (size_t k = 0; k + 1 < off.size(); k += 2) {
    rx = std::max(rx, std::abs(off[k]));
    ry = std::max(ry, std::abs(off[k + 1]));
  }
}

// Grows a metadata buffer to at least `bytes` (its contents are then invalid).
inline int reserve_meta(morse_ctx* ctx, MetaBuf& mb, size_t bytes) {
  const char* before = mb.p;
  const int rc = grow(ctx, mb, bytes, bytes, "metadata");
  if (mb.p != before) mb.key = 0;
  return rc;
}

// Room for `bytes` of tables about to be made anew in a buffer that calls read without writing it:
// a graph that names it goes on reading the old ones.
inline int renew_meta(morse_ctx* ctx, MetaBuf& mb, size_t bytes) {
  if (capturing(ctx))
    return fail(ctx, MORSE_EUNSUPPORTED, "tables cannot be made under capture: make the same call before it");
  if (mb.named) {
    ctx->retired.push_back(mb.p);
    mb = MetaBuf{};
  }
  mb.key = 0;
  return reserve_meta(ctx, mb, bytes);
}

inline int upload(morse_ctx* ctx, void* dst, const void* src, size_t bytes) {
  if (!bytes) return MORSE_OK;
  HIP_TRY(ctx, hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, ctx->stream));
  return MORSE_OK;
}

// Puts src (which may go when this returns) at dst.  A captured call takes it along by value.
inline int put_now(morse_ctx* ctx, void* dst, const std::vector<char>& src) {
  if (src.size() <= kPutMax || capturing(ctx)) {
    HIP_TRY(ctx, launch_put(dst, src.data(), src.size(), ctx->stream));
    return MORSE_OK;
  }
  const int rc = upload(ctx, dst, src.data(), src.size());
  if (rc) return rc;
  HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  return MORSE_OK;
}

// Puts src on the device in one half of mb, at *at: ordinary calls use the first, where what a
// call put stays for the next with the same key; captured calls the second, which their graphs
// write on every replay without ordinary calls having to know.
inline int put_meta(morse_ctx* ctx, MetaBuf& mb, const std::vector<char>& src, uint64_t key, char** at) {
  const int rc = reserve_meta(ctx, mb, 2 * ((src.size() + 255) & ~size_t(255)));
  if (rc) return rc;
  if (capturing(ctx)) {
    *at = mb.p + mb.size / 2;
    return put_now(ctx, *at, src);
  }
  *at = mb.p;
  if (mb.key == key) return MORSE_OK;
  mb.key = 0;
  const int e = put_now(ctx, *at, src);
  if (e == MORSE_OK) mb.key = key;
  return e;
}

// Host metadata laid out in one block; sizes are rounded up to a multiple of `unit` bytes.
struct MetaBlock {
  std::vector<char> bytes;
  size_t add(const void* p, size_t n, size_t unit = 16) {
    const size_t at = bytes.size();
    bytes.resize(at + (n + unit - 1) / unit * unit);
    if (n) std::memcpy(bytes.data() + at, p, n);
    return at;
  }
};

inline bool grid_ok(const morse_grid2d* g) {
  return g && std::isfinite(g->cx) && std::isfinite(g->cy) && std::isfinite(g->wx) &&
         std::isfinite(g->wy) && g->wx > 0 && g->wy > 0 && g->nx >= 2 && g->ny >= 2 &&
         (g->nx % 2) == 0 && (g->ny % 2) == 0;
}

inline int check_lens(morse_ctx* ctx, double s, double q) {
  if (!(std::isfinite(s) && s > 0)) return fail(ctx, MORSE_EINVAL, "s must be finite and > 0");
  if (!(q >= 0.0 && q <= 1.0)) return fail(ctx, MORSE_EINVAL, "q must lie in [0, 1]");
  return MORSE_OK;
}

inline int check_window(morse_ctx* ctx, const morse_grid2d* w, const char* what) {
  if (!grid_ok(w)) return fail(ctx, MORSE_EINVAL, "%s: invalid grid (even counts >= 2, finite widths > 0)", what);
  if (w->nx > 32768 || w->ny > 32768)
    return fail(ctx, MORSE_ERANGE, "%s: at most 32768 pixels per side", what);
  return MORSE_OK;
}

inline MapC make_mapc(const float* map, const morse_grid2d& w) {
  MapC m;
  m.map = map;
  m.mx = w.nx;
  m.my = w.ny;
  m.sx = (float)w.cx;
  m.sy = (float)w.cy;
  m.kx = (float)((double)w.nx / w.wx);
  m.ky = (float)((double)w.ny / w.wy);
  m.ox = (float)(w.nx / 2) - 0.5f;
  m.oy = (float)(w.ny / 2) - 0.5f;
  m.lx = (float)(w.nx - 1);
  m.ly = (float)(w.ny - 1);
  m.tiles_x = (uint32_t)((w.nx - 1 + 3) / 4);
  m.tiles_y = (uint32_t)((w.ny - 1 + 1) / 2);
  m.row = 8 * m.tiles_x - 2;
  m.cells = 8 * m.tiles_x * m.tiles_y;
  m.quad = nullptr;
  return m;
}

// Quad-packed maps live in one workspace region: per map quad_bytes rounded to 256.
inline size_t quad_region_bytes(const morse_map_view* maps, int32_t n_maps) {
  size_t t = 0;
  for (int i = 0; i < n_maps; ++i)
    t += (quad_bytes(maps[i].window.nx, maps[i].window.ny) + 255) & ~size_t(255);
  return t;
}

inline void assign_quads(std::vector<MapC>& hm, char* region) {
  for (auto& m : hm) {
    m.quad = (const Quad*)region;
    region += (quad_bytes(m.mx, m.my) + 255) & ~size_t(255);
  }
}

// Critical points of the binary lens at nphi equally spaced phases of the critical-curve
// quartic (4 per phase, phase-major; defined with the caustic geometry).
void critical_points(double s, double q, int32_t nphi, std::vector<std::complex<double>>& z);

// Device address of the allocation-free entry point's scratch array on `device`
// (looked up once per device, with that device current; defined beside the entry
// point).  Returns MORSE_OK and sets *out, or an error code.
int noalloc_scratch(int device, char** out);

// Light curves: arrays present, CSR offsets from 0, each event at least 3 and at most
// kMaxEventPoints points (the kernels address an event's FP64 arrays with 32-bit byte
// offsets from the event's base, 8 B x 2^28 < 2^32), finite reference times.
constexpr int64_t kMaxEventPoints = (int64_t)1 << 28;

inline int check_lightcurves(morse_ctx* ctx, const morse_lightcurves* lcs) {
  if (!lcs || lcs->n_events <= 0 || !lcs->h_offsets || !lcs->h_t_ref || !lcs->d_t || !lcs->d_flux ||
      !lcs->d_weight)
    return fail(ctx, MORSE_EINVAL, "light curves: missing arrays or n_events <= 0");
  if (lcs->h_offsets[0] != 0) return fail(ctx, MORSE_EINVAL, "light curves: offsets[0] must be 0");
  for (int e = 0; e < lcs->n_events; ++e) {
    const int64_t n = lcs->h_offsets[e + 1] - lcs->h_offsets[e];
    if (n < 3) return fail(ctx, MORSE_EINVAL, "event %d has %lld < 3 points", e, (long long)n);
    if (n > kMaxEventPoints)
      return fail(ctx, MORSE_ERANGE, "event %d has %lld points, more than 2^28", e, (long long)n);
    if (!std::isfinite(lcs->h_t_ref[e])) return fail(ctx, MORSE_EINVAL, "event %d: t_ref not finite", e);
  }
  return MORSE_OK;
}

inline int check_quad_size(morse_ctx* ctx, const morse_map_view* maps, int32_t n_maps) {
  for (int i = 0; i < n_maps; ++i)
    if (quad_bytes(maps[i].window.nx, maps[i].window.ny) >= ((size_t)1 << 32))
      return fail(ctx, MORSE_ERANGE, "map %d: %d x %d pixels exceed the 4 GiB packed-cell limit", i,
                  maps[i].window.nx, maps[i].window.ny);
  return MORSE_OK;
}


}  // namespace host
}  // namespace morse
