// Internal declarations of the gfx950 library: device-side data layouts, the
// per-sample arithmetic shared by the search and gradient kernels, and the host
// launchers each kernel file exports to the C ABI sources (api_*.hip).  Not part of the
// public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <map>
#include <string>
#include <vector>

#include "../../include/morse.h"

namespace morse {

constexpr int kWave = 64;  // CDNA wavefront width

// ---------------------------------------------------------------------------
// Ray shooting constants, each rounded once from FP64 to binary32 on the host.
struct RayParams {
  float m1, m2, x1, x2;  // lens masses and positions
  float cx, cy, hx, hy;  // lattice centre and spacing
  float sx, sy, kx, ky;  // window centre and pixels per Einstein radius
  int32_t nx, ny, mx, my;
  int32_t row0, row1;    // lattice rows [row0, row1)
};

// Per-trajectory constants: binary32 geometry rounded once from FP64, t0 kept FP64
// so each event subtracts its own reference time before rounding.
struct TrajC {
  double t0;
  float iE, ca, sa, bx, by, pad;
};
static_assert(sizeof(TrajC) == 32, "TrajC layout");

// A map as the sampling kernels see it.  The row-major pixel values `map` are packed
// once per call into `quad`: cell (i, j), 0 <= i < mx - 1, 0 <= j < my - 1, holds what a
// bilinear sample of it takes from the four pixel-centre values around it, the left ones
// and the steps to the right ones (A[j][i], A[j][i+1] - A[j][i], A[j+1][i], A[j+1][i+1] -
// A[j+1][i]), the steps rounded to binary32 as the blend rounds them, as one 16-byte Quad,
// and the cells are grouped in
// tiles of 4 (x) by 2 (y) cells, one 128-byte cache line each, tiles in row-major order,
// cells inside a tile column-major:
//   q(i, j) = (j / 2) 8 tiles_x + 2 i + j % 2 = (j / 2) (8 tiles_x - 2) + (2 i + j)
// (= 8 tile + 2 (i % 4) + j % 2, tile = (j / 2) tiles_x + i / 4), so the index is one
// shift-add, one shift and one 24-bit multiply-add.  A bilinear sample is then one aligned
// load, and the samples of a wavefront along a trajectory touch about 2.5x fewer
// cache lines than two row-major row loads.
struct alignas(16) Quad {
  float v00, e0, v01, e1;
};

struct MapC {
  const float* map;
  const Quad* quad;
  uint32_t tiles_x, tiles_y;
  uint32_t row;                  // 8 tiles_x - 2, the index step of two rows of cells
  uint32_t cells;                // packed cells, 8 tiles_x tiles_y
  int32_t mx, my;
  float sx, sy, kx, ky, ox, oy;  // grid coordinate g = (zeta - s) k + o
  float lx, ly;                  // on-map bound: g < M - 1
};
// Load of cell q: one buffer_load_dwordx4 with a structured index (stride 16) through a
// buffer resource over the map's packed cells.  The resource is uniform (scalar registers)
// and the index one 32-bit register that the load itself scales, so a sample needs no
// address arithmetic beyond the index, and an index outside the packed map reads zeros
// instead of faulting (the hardware range check).  Word 1: the base's high bits and the
// stride; word 2: the number of cells; word 3: data format 32 bits (bits 15-18 = 4).
typedef int rsrc4 __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
__device__ float4v struct_buffer_load_f4(rsrc4 rsrc, int index, int offset, int soffset,
                                         int aux) __asm("llvm.amdgcn.struct.buffer.load.v4f32");
typedef float float2v __attribute__((ext_vector_type(2)));
__device__ float2v struct_buffer_load_f2(rsrc4 rsrc, int index, int offset, int soffset,
                                         int aux) __asm("llvm.amdgcn.struct.buffer.load.v2f32");
constexpr int kBufferWord3 = 0x00020000;
__device__ __forceinline__ Quad ldq(const MapC& m, uint32_t q) {
  const uint64_t base = (uint64_t)m.quad;
  // tiles_x tiles_y 128 < 2^32: the host rejects larger packed maps
  const rsrc4 r = {(int)(uint32_t)base, (int)((uint32_t)(base >> 32) | ((uint32_t)sizeof(Quad) << 16)),
                   (int)m.cells, kBufferWord3};
  const float4v v = struct_buffer_load_f4(r, (int)q, 0, 0, 0);
  return Quad{v.x, v.y, v.z, v.w};
}

// Packed size of a map with mx x my pixels (bytes).
inline size_t quad_bytes(int32_t mx, int32_t my) {
  return (size_t)((mx - 1 + 3) / 4) * (size_t)((my - 1 + 1) / 2) * 128;
}

// Light curves after preparation: per point binary32 time offset, w and the
// centred weighted flux w (F - Fbar); per event S_w, the weighted mean Fbar and
// V = sum w (F - Fbar)^2.
struct LcView {
  const float* t;
  const double* w;
  const double* wFc;
  const double* F;
  const int64_t* off;   // device CSR offsets [n_events + 1]
  const uint32_t* sorted;  // [n_events] 1 where the event's times do not decrease, or nullptr
  const double* sums;   // [n_events][3]: S_w, Fbar, V
  const double* t_ref;  // [n_events]
};

// ---------------------------------------------------------------------------
// Sampling along a trajectory (binary32, no fused multiply-add: the library is
// compiled with -ffp-contract=off, so every operation below rounds on its own).
//   tau = (t - t0')*iE; zeta = tau (ca, sa) + (bx, by); g = (zeta - s) k + o;
//   bilinear between pixel-centre values inside [0, M-1), else the single-lens
//   magnification (uu + 2)/sqrt(uu (uu + 4)) about the barycentre.
struct Sample {
  float A;
  float tau, zx, zy;
  float fx, fy, e0, e1, ax0, ax1;
  bool on;
};

// Load base[i] through a uniform base pointer and a 32-bit element offset, so the
// backend can address with a scalar base plus one 32-bit VGPR offset.  The pointer is
// taken as global memory explicitly (a pointer rebuilt from scalar registers has lost
// its address space, and a generic pointer would compile to a slower flat load).
template <class T>
__device__ __forceinline__ T ldg(const T* __restrict__ base, uint32_t i) {
  typedef const __attribute__((address_space(1))) char gchar;
  typedef const __attribute__((address_space(1))) T gT;
  return *(gT*)((gchar*)base + (size_t)(i * (uint32_t)sizeof(T)));
}

// Index of packed cell (i, j); below 2^28 since the packed map is below 4 GiB, and both
// factors of the product fit 24 bits.  kFewest: the sum is kept as one shift-add, else the
// compiler takes a shift, a product and a three-way sum, which it can schedule more freely: the
// line simplex, bound by latency, takes 3% less with those (4000 lines x 300 points 4.54 and
// 4.43 ms), the others half a percent more.
template <bool kFewest = true>
__device__ __forceinline__ uint32_t cell_index(const MapC& m, uint32_t i, uint32_t j) {
  uint32_t s = (i << 1) + j;
  if (kFewest) asm("" : "+v"(s));
  return __umul24(j >> 1, m.row) + s;
}

// The blend of a cell (binary32, each operation rounded on its own).
__device__ __forceinline__ float blend(const Quad& q, float fx, float fy) {
  const float ax0 = q.v00 + fx * q.e0, ax1 = q.v01 + fx * q.e1;
  return ax0 + fy * (ax1 - ax0);
}

// Sampling in steps, so that the loads of several points can all be issued before
// any of them is used: locate (trajectory position, on-map test, cell), one 16-byte
// fetch of the cell (an off-map lane reads cell 0, and ignores it), then the blend.
// The arithmetic is that of sample_A / sample_full.
struct Loc {
  float tau, zx, zy, fx, fy;
  uint32_t q;  // index of the packed cell (0 off the map)
  bool on;
};

template <bool kFewest = true>
__device__ __forceinline__ Loc locate(const MapC& m, float tt, float t0p, float iE, float ca,
                                      float sa, float bx, float by) {
  Loc l;
  l.tau = (tt - t0p) * iE;
  l.zx = l.tau * ca + bx;
  l.zy = l.tau * sa + by;
  const float gx = ((l.zx - m.sx) * m.kx) + m.ox;
  const float gy = ((l.zy - m.sy) * m.ky) + m.oy;
  // On the map: 0 <= g < M - 1, tested on the bit patterns as unsigned integers (for
  // a positive bound L, bits(g) < bits(L) iff +0 <= g < L; negative values and NaN
  // have larger patterns).  Only g = -0 would differ, and g is a sum with the nonzero
  // constant o = M/2 - 1/2, which an IEEE sum never rounds to -0.
  l.on = ((unsigned)(__float_as_uint(gx) < __float_as_uint(m.lx)) &
          (unsigned)(__float_as_uint(gy) < __float_as_uint(m.ly))) != 0u;
  // on the map g >= 0, so truncation is the floor and fract(g) = g - floor(g) exactly
  l.fx = __builtin_amdgcn_fractf(gx);
  l.fy = __builtin_amdgcn_fractf(gy);
  l.q = l.on ? cell_index<kFewest>(m, (uint32_t)gx, (uint32_t)gy) : 0u;
  return l;
}

// Single-lens magnification about the barycentre, (uu + 2)/sqrt(uu (uu + 4)), with a
// correctly rounded binary32 square root and quotient.  A correctly rounded result is
// unique, so any exact method gives the same bits.  When uu lies in [2^-22, 2^12) on every
// active lane the short form runs: the hardware's reciprocal square root, the root
// corrected by its residual, the quotient by the same reciprocal corrected by its residual.
// Against the IEEE square root and division it was compared for every binary32 uu from
// 2^-62 to 2^31: it equals them throughout [1.3e-7, 8189] (53 values outside differ).
// 8 instructions, 17 before.  Elsewhere the general sequences run.
__device__ __forceinline__ float point_lens_A(float zx, float zy) {
  const float uu = zx * zx + zy * zy;
  const float p = uu + 2.0f, d = uu * (uu + 4.0f);
  constexpr uint32_t lo = 0x34800000u, hi = 0x45800000u;  // 2^-22, 2^12
  if (__builtin_amdgcn_ballot_w64(__float_as_uint(uu) - lo >= hi - lo) == 0) {
    const float y = __builtin_amdgcn_rsqf(d);
    float s = d * y;
    s = fmaf(fmaf(-s, s, d), 0.5f * y, s);
    const float q = p * y;
    return fmaf(fmaf(-s, q, p), y, q);
  }
  return p / sqrtf(d);
}

__device__ __forceinline__ float sample_A(const MapC& m, float tt, float t0p, float iE, float ca,
                                          float sa, float bx, float by) {
  const float tau = (tt - t0p) * iE;
  const float zx = tau * ca + bx;
  const float zy = tau * sa + by;
  const float gx = ((zx - m.sx) * m.kx) + m.ox;
  const float gy = ((zy - m.sy) * m.ky) + m.oy;
  if (gx >= 0.0f && gx < m.lx && gy >= 0.0f && gy < m.ly) {
    const float fi = floorf(gx);
    const float fj = floorf(gy);
    const float fx = gx - fi;
    const float fy = gy - fj;
    return blend(ldq(m, cell_index(m, (uint32_t)(int)fi, (uint32_t)(int)fj)), fx, fy);
  }
  const float uu = zx * zx + zy * zy;
  return (uu + 2.0f) / sqrtf(uu * (uu + 4.0f));
}

__device__ __forceinline__ Sample sample_full(const MapC& m, float tt, float t0p, float iE,
                                              float ca, float sa, float bx, float by) {
  Sample s;
  s.tau = (tt - t0p) * iE;
  s.zx = s.tau * ca + bx;
  s.zy = s.tau * sa + by;
  const float gx = ((s.zx - m.sx) * m.kx) + m.ox;
  const float gy = ((s.zy - m.sy) * m.ky) + m.oy;
  s.on = (gx >= 0.0f && gx < m.lx && gy >= 0.0f && gy < m.ly);
  if (s.on) {
    const float fi = floorf(gx);
    const float fj = floorf(gy);
    s.fx = gx - fi;
    s.fy = gy - fj;
    const Quad c = ldq(m, cell_index(m, (uint32_t)(int)fi, (uint32_t)(int)fj));
    s.e0 = c.e0;
    s.e1 = c.e1;
    s.ax0 = c.v00 + s.fx * s.e0;
    s.ax1 = c.v01 + s.fx * s.e1;
    s.A = s.ax0 + s.fy * (s.ax1 - s.ax0);
  } else {
    const float uu = s.zx * s.zx + s.zy * s.zy;
    s.A = (uu + 2.0f) / sqrtf(uu * (uu + 4.0f));
    s.fx = s.fy = s.e0 = s.e1 = s.ax0 = s.ax1 = 0.0f;
  }
  return s;
}

// A uniform value in a vector register of its own: an instruction whose operands are all
// vector registers (or inline constants) issues in half the time of one with a scalar
// operand (2.5 against 4.3 cycles per wavefront for a binary32 add or multiply).
__device__ __forceinline__ float in_vgpr(float s) {
  float v;
  asm("v_mov_b32 %0, %1" : "=v"(v) : "s"(s));
  return v;
}

// A value known to be the same on every lane, moved to scalar registers word by word
// (loads from memory the kernel also writes are vector loads, whose results the
// compiler would otherwise keep in vector registers).
template <class T>
__device__ __forceinline__ T uniform(const T& v) {
  static_assert(sizeof(T) % 4 == 0, "uniform() moves 32-bit words");
  T r;
  const int* src = reinterpret_cast<const int*>(&v);
  int* dst = reinterpret_cast<int*>(&r);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) dst[i] = __builtin_amdgcn_readfirstlane(src[i]);
  return r;
}

// Deterministic wavefront sum (butterfly over 64 lanes, same order on every lane).
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// Wavefront reduce-scatter of N FP64 values per lane.  Each halving step over lane
// bit MASK keeps ceil(N/2) slots: lanes with the bit set keep the upper half (padded
// with a zero), the others the lower half, each adding its partner's copy of the slots
// it keeps; six steps (MASK = 32 .. 1) exchange about N values in all, against 6 N for
// one butterfly per value.  Each value is summed over the same pairing tree as
// wave_sum (IEEE addition commutes), so the totals are bitwise those of wave_sum.  On
// return v[0] holds the total of original value `slot` when `valid`; every value
// appears on exactly one valid lane, rs_lane<N>(q).
template <int N, int MASK = 32>
__device__ __forceinline__ void reduce_scatter(double* v, int lane, int& slot, bool& valid) {
  if constexpr (MASK >= 1) {
    constexpr int H = (N + 1) / 2;
    const bool up = (lane & MASK) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const double lo = v[i];
      const double hi = (i + H < N) ? v[i + H] : 0.0;
      const double other = __shfl_xor(up ? lo : hi, MASK, kWave);
      v[i] = (up ? hi : lo) + other;
    }
    reduce_scatter<H, MASK / 2>(v, lane, slot, valid);
    slot += up ? H : 0;
    valid = valid && slot < N;
  }
}

// Lane that holds value q after reduce_scatter<N>.
template <int N>
constexpr int rs_lane(int q) {
  int lane = 0, n = N;
  for (int mask = 32; mask >= 1; mask >>= 1) {
    const int h = (n + 1) / 2;
    if (q >= h) {
      lane |= mask;
      q -= h;
    }
    n = h;
  }
  return lane;
}

__device__ __forceinline__ double read_lane(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Wavefront totals of N values, on every lane (bitwise wave_sum of each value).
template <int N>
__device__ __forceinline__ void wave_sums(double (&v)[N]) {
  int slot = 0;
  bool valid = true;
  reduce_scatter<N>(v, threadIdx.x & (kWave - 1), slot, valid);
  const double mine = v[0];
#pragma unroll
  for (int q = 0; q < N; ++q) v[q] = read_lane(mine, rs_lane<N>(q));
}

// Neumaier's compensated addition: s + c carries the sum, c the rounding errors.
__device__ __forceinline__ void neumaier_add(double& s, double& c, double v) {
  double t = s + v;
  if (fabs(s) >= fabs(v))
    c += (s - t) + v;
  else
    c += (v - t) + s;
  s = t;
}

// Profiled fit (Eqs. 5-6) in centred form.  With b = A - 1 and per-point
// wFc = w (F - Fbar), one pass gives B1 = sum w b, B2 = sum w b^2, C = sum b wFc.
// Then S_bb = B2 - B1^2/S_w equals det/S_w of the normal equations
// (det = S_AA S_w - S_A^2, S_AA = B2 + 2 B1 + S_w), and
//   F_s = C / S_bb,  F_b = Fbar - F_s (1 + B1/S_w),  chi2 = V - F_s C.
// Degenerate (det <= 1e-12 S_AA S_w, i.e. S_bb <= 1e-12 S_AA): F_s = 0, F_b = Fbar,
// chi2 = V.
//
// The sums are plain (uncompensated) FP64, so the one-pass chi2 comes with a worst-case
// error bound, and `recheck` is set when that bound exceeds 1e-8 chi2; the caller then
// sums w r^2 directly (Neumaier-compensated second pass).  Each of B1, B2, C is a
// recursive sum over one lane's points followed by a fixed reduction tree, so with n
// = the terms per lane + the tree depth + the roundings of one term (fit_terms), its
// error is at most n u sum|terms| (u = 2^-53; Higham, Accuracy and Stability of
// Numerical Algorithms, sec. 4.2), and by Cauchy-Schwarz sum|w b| <= sqrt(S_w B2),
// sum|b wFc| <= sqrt(B2 V).  Through chi2 = V - C^2/S_bb, with F_s^2 S_bb <= V and
// kappa = B2/S_bb >= 1 (V carries its own compensated error, u V):
//   |d chi2| <= u V (n (3 kappa + 2 sqrt(kappa)) + 6 kappa + 5).
// For noisy data chi2 is near the number of points and the bound stays far below the
// threshold; a near-perfect or ill-conditioned fit takes the second pass.
struct Fit {
  double Fs, Fb, chi2;
  bool degenerate, recheck;
};

// Terms per lane plus reduction depth for the bound above: np points over `lanes`
// lanes, a tree of at most 8 levels, at most 2 serial cross-wave additions and 2
// roundings per term.
__device__ __forceinline__ double fit_terms(int32_t np, int lanes) {
  return (double)((np + lanes - 1) / lanes + 12);
}

__device__ __forceinline__ Fit centred_fit(double Sw, double Fbar, double V, double B1, double B2,
                                           double C, double nterms) {
  Fit f;
  const double SAA = (B2 + 2.0 * B1) + Sw;
  const double Sbb = B2 - (B1 * B1) / Sw;
  f.degenerate = !(Sbb > 1e-12 * SAA);
  f.recheck = false;
  if (f.degenerate) {
    f.Fs = 0.0;
    f.Fb = Fbar;
    f.chi2 = V;
    return f;
  }
  f.Fs = C / Sbb;
  f.Fb = Fbar - f.Fs * (1.0 + B1 / Sw);
  f.chi2 = V - f.Fs * C;
  const double kappa = B2 / Sbb;
  const double bound = (nterms * (3.0 * kappa + 2.0 * sqrt(kappa)) + 6.0 * kappa + 5.0) * V;
  f.recheck = !(f.chi2 > 0.0) || (bound > 9.007199254740992e7 * f.chi2);  // 1e-8 / u
  return f;
}

// ---------------------------------------------------------------------------
// Host launchers (one per kernel family); all enqueue on `st` and return the
// first HIP error.
hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t st);
hipError_t launch_fill_u64(uint64_t* p, size_t n, uint64_t v, hipStream_t st);
// Exclusive prefix sum of nb uint32 counters in place (one workgroup; counting sorts).
hipError_t launch_scan_u32(uint32_t* v, int64_t nb, hipStream_t st);
// order[0 .. n): the items 0 .. n - 1 by ascending key (key < nbins; the order among
// equal keys is unspecified).  hist: nbins counters of workspace.
hipError_t launch_bucket_order(const uint32_t* key, int64_t n, int32_t nbins, uint32_t* hist,
                               int32_t* order, hipStream_t st);
// Shoots the rows of p into counts.  With `stats` (three totals that the call adds to),
// `slots` is workspace of 4 kStatSlots words: workgroup b adds to slot b % kStatSlots, which
// takes one atomic in 256 (of a 32768^2 lattice 260,000 fell on each of the three totals and
// doubled its time).  nullptr: the workgroups add to the totals themselves.
constexpr uint32_t kStatSlots = 256;  // a power of two
hipError_t launch_rayshoot(const RayParams& p, uint32_t* counts, unsigned long long* stats,
                           unsigned long long* slots, int num_cu, hipStream_t st);
// Normalisation + convolution of a counts map with ntaps taps whose offsets reach at
// most rx columns and ry rows from the pixel (rx = ry = 0: the single tap (0, 0);
// otherwise at most 16 each).
hipError_t launch_normalize_convolve(const uint32_t* counts, float* map, int32_t mx, int32_t my,
                                     const float* d_w, const int32_t* d_off, int32_t ntaps,
                                     int32_t rx, int32_t ry, float scale, uint32_t* d_maxc,
                                     hipStream_t st);
// The preparation of a search or of an evaluation of candidates, one launch: light curves
// (lc.wFc, lc.sums and, unless nullptr, lc.sorted: whether the event's times do not decrease),
// trajectory constants tc[n] from a grid's axes or from rows of params, with their sorting
// key (see launch_traj_perm) unless nullptr, zeroed words, packed maps (h_maps: the device
// table's entries, for the sizes).
struct PrepArgs {
  LcView lc;
  int32_t n_events;
  int64_t n, n_traj;         // trajectories in all (0: none) and in a list
  const double* axes;        // [u0 (nu) | alpha (na) | t0 (nt) | tE (ne)], or nullptr
  int32_t nu, na, nt, ne;
  const double* params;
  TrajC* tc;
  uint32_t* key;
  uint32_t* zero;
  uint64_t n_zero;
  const MapC* maps;
  int32_t n_maps;
  uint32_t event_blocks, traj_blocks, zero_blocks, pack_blocks;  // set by the launcher
};
hipError_t launch_prep(PrepArgs a, const MapC* h_maps, hipStream_t st);
// Copies host memory (a multiple of 4 bytes) to dst by value: when it returns, src may go, and
// the launches can be captured.  A copy from pageable memory and the wait for it take 60 us
// or more of the host, one of these launches 4; beyond kPutMax bytes the copy is as quick.
constexpr int kPutWords = 896;
constexpr size_t kPutMax = 4 * 4 * kPutWords;
hipError_t launch_put(void* dst, const void* src, size_t bytes, hipStream_t st);

struct SearchOut {
  double* chi2;
  double* fs;
  double* fb;
};

// Plain search: one launch for one (event, map); outputs for that segment.  n_points: of the event.
hipError_t launch_search_plain(const TrajC* tc, int64_t n_traj, LcView lc, int32_t event,
                               int64_t n_points, MapC map, SearchOut out, int waves_per_block, hipStream_t st);

// Batched search over (event, map, trajectory block) items, one launch.
struct BatchedArgs {
  const TrajC* tc;          // per event if !shared
  int64_t n_traj;
  int32_t shared;
  int32_t n_events, n_maps;
  const MapC* maps;         // device table [n_maps]
  LcView lc;
  SearchOut out;            // full [e][m][traj] arrays
  int32_t nu, na, nt, ne;   // product-grid axes (na = 0 for trajectory lists)
  int32_t traj_per_item;
  int32_t waves_per_block;
  uint32_t chunk;           // workgroups per chunk dealt to an XCD (set by the launcher)
  uint32_t rotate;          // 1: the XCDs change places with each deal (set by the launcher)
  uint32_t first;           // this launch's first workgroup (set by the launcher)
  int32_t tu;               // trajectories scored together per wavefront (1, 2 or 4)
  int32_t centred;          // every map's window is centred on (0, 0)
  const int32_t* perm;      // trajectory lists: [lists][n_traj] scoring order, or nullptr
};
// Scoring order of trajectory lists (n_lists lists of n_traj) from their keys:
// each list grouped by direction and speed, kPermDirs buckets of alpha by kPermSpeeds
// quarter octaves of tE, so that waves scoring at the same time follow nearby lines through
// the map and cross it at the same points of the light curve (a counting sort; the order within
// a bucket is unspecified and changes the schedule only); perm holds indices over all
// lists (list * n_traj + trajectory).  key: n_lists * n_traj words of workspace, hist:
// n_lists * kPermBins counters.  Lists with more than kPermBinsMax counters in all are
// not reordered by the caller.
constexpr int kPermDirs = 16, kPermSpeeds = 16;
constexpr int kPermBins = kPermDirs * kPermSpeeds;
constexpr int64_t kPermBinsMax = 1 << 22;
hipError_t launch_traj_perm(const uint32_t* key, int64_t n_traj, int32_t n_lists, uint32_t* hist,
                            int32_t* perm, hipStream_t st);
// Items per (map, event) of the batched search.
__host__ __device__ inline uint32_t search_blocks(uint32_t n_traj, int32_t traj_per_item, int32_t tu) {
  const uint32_t ng = (n_traj + tu - 1) / tu;
  const uint32_t gpi = traj_per_item > tu ? (uint32_t)(traj_per_item / tu) : 1u;
  return (ng + gpi - 1) / gpi;
}
hipError_t launch_search_batched(BatchedArgs a, hipStream_t st);

// Workspace of the selections below: byte offsets.  Its first zero_bytes are zero before the
// first of them runs.
struct SelectScratch {
  size_t zero_bytes, part, tk_state, tk_hist, tk_keys, tk_idx, bytes;
};
// n_best segments of best_len for launch_best, n_seg of seg_len for launch_topk (0: not used).
SelectScratch select_scratch(int64_t n_best, int64_t best_len, int64_t n_seg, int64_t seg_len, int32_t k,
                             int num_cu);
// Best (chi2, index) per segment of length seg_len; n_seg segments.
hipError_t launch_best(const double* chi2, int64_t n_seg, int64_t seg_len, double* best_chi2,
                       int64_t* best_idx, char* scratch, const SelectScratch& s, int num_cu,
                       hipStream_t st);
// Top-k per segment (k <= 4096).
hipError_t launch_topk(const double* chi2, int64_t n_seg, int64_t seg_len, int32_t k,
                       double* out_chi2, int64_t* out_idx, char* scratch, const SelectScratch& s,
                       int num_cu, hipStream_t st);

// Expand top-k flat indices (map * n_traj + traj) into parameter rows.
hipError_t launch_candidates(const double* axes, int32_t nu, int32_t na, int32_t nt, int32_t ne,
                             const double* list, int32_t shared, int64_t n_traj, int32_t n_events,
                             int32_t n_maps, int32_t k, const int64_t* idx, double* params,
                             int32_t* event, int32_t* mapidx, hipStream_t st);

// Gradient evaluation.
struct GradArgs {
  int64_t n;
  const double* params;     // natural [n][4]
  const int32_t* event;
  const int32_t* mapidx;
  const MapC* maps;
  int32_t n_events, n_maps;  // out-of-range event / map indices give NaN outputs
  LcView lc;
  double* chi2;
  double* grad;             // [n][4] or nullptr
  double* fs;
  double* fb;
  const int32_t* order;     // [n] the order in which candidates are evaluated, or nullptr
  TrajC* tc;                // [n] constants of params, written with the order's keys, or nullptr
  int32_t map_first;        // set by launch_cand_order
};
hipError_t launch_chi2_grad(const GradArgs& a, hipStream_t st);
// Evaluation order of candidates [0, a.n): by event, the longest light curve first, and map
// (h_maps: the device table's entries, for the sizes); by map and then so when the maps take more
// than the last-level cache (256 MiB); by map, then event with more than kRankedEvents events;
// by map alone when n_maps x n_events exceeds kOrderBinsMax.  Candidates evaluated at the same time then sample the same map.  Within a group the order is unspecified: it changes only
// the schedule, never a result.  key: workspace of a.n words; hist: of order_bins(a)
// counters.  With a.tc the candidates' constants are written too.
constexpr int64_t kOrderBinsMax = 1 << 20;
constexpr int32_t kRankedEvents = 1024;
inline int64_t order_bins(int32_t n_maps, int32_t n_events) {
  const int64_t both = (int64_t)n_maps * n_events;
  return both <= kOrderBinsMax ? both : n_maps;
}
hipError_t launch_cand_order(GradArgs a, const MapC* h_maps, uint32_t* key, uint32_t* hist, int32_t* order,
                             hipStream_t st);

// Candidates that the chip holds all at once (ten workgroups a CU), or that sample one map
// for one event, need no order.
inline bool order_helps(int64_t n, int32_t n_maps, int32_t n_events) {
  return n > 2048 && order_bins(n_maps, n_events) > 1;
}

// chi2, (F_s, F_b) and the gradient; G: the sums w r D that it is formed from.
struct Eval {
  double chi2, Fs, Fb;
  double G[5], g[4];
  int32_t direct, pad;  // whether the direct sums are needed
};
constexpr int kMaxHistory = 16;
// One candidate's L-BFGS state.
struct RefineState {
  double an[4];                  // anchor: the starting row
  double g[4], d[4], f, step;    // at the accepted point
  struct Pair {
    double s[4], y[4], r, alph;
  } pair[kMaxHistory];           // ring of nh pairs from head
  TrajC tc;                      // of the trial point
  double tE;
  Eval ev;                       // its evaluation
  float p[4], pt[4];             // accepted and trial point
  int32_t nh, head, nls, active;
};
struct RefineArgs {
  double* params;                // [n][4] in and out
  double* chi2_out;
  double* chi2_init;             // or nullptr
  RefineState* state;            // [n], only used when one launch does not run all rounds
  int32_t m, max_ls;             // m <= kMaxHistory
  double c1, shrink;
  int32_t steps;                 // rounds 0 .. steps
  int32_t r0, r1;                // rounds of this launch
};
hipError_t launch_refine(const GradArgs& a, const RefineArgs& s, bool four, hipStream_t st);
// Whether n_maps maps, packed, take more than the last-level cache.
bool maps_exceed_cache(const MapC* h_maps, int32_t n_maps);
// The same rounds as launches of their own (s.state set): start, then for each round 0 .. steps
// evaluation and update; the last update writes the results.
hipError_t launch_round_start(const GradArgs& a, const RefineArgs& s, hipStream_t st);
hipError_t launch_round_eval(const GradArgs& a, const RefineArgs& s, hipStream_t st);
hipError_t launch_round_update(const GradArgs& a, const RefineArgs& s, int32_t round, hipStream_t st);

}  // namespace morse
