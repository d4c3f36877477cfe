// Trajectory search on gfx950 (sec. 4.2 of McDougall & Albrow 2015: the chi-square of
// every trajectory through a map, sampled by bilinear interpolation; Eqs. 5-6: the flux
// is linear in the magnification, so (F_s, F_b) are profiled out by weighted least
// squares).
//
// Layout.  One wavefront scores TU neighbouring trajectories at a time: its 64 lanes
// stride over the light-curve points, a chunk of 64 at a time (time-ordered, so a chunk's
// samples are neighbouring map cells, and most chunks lie wholly on or wholly off the map;
// both kinds are known beforehand from their end points), each lane keeps FP64 partial
// sums of the normal equations in centred form (b = A - 1 against the mean-centred
// weighted flux) per trajectory, and a fixed-order reduction (bitwise the butterfly of
// each value) totals them.  S_w, the weighted mean flux and V = sum w (F - Fbar)^2
// depend only on the light curve and are computed once per event.  The 2x2 solve gives
// chi2 = V - F_s C in the same pass; when the rounding bound of that form exceeds 1e-8
// relative (ill-conditioned or near-perfect fits) the wave re-samples and sums
// w (F - F_s A - F_b)^2 directly.
//
// Plain mode launches one grid per (event, map), one trajectory per wavefront.  Batched
// mode launches one grid over the (map, event, trajectory group) items, dealt to the XCDs
// in chunks, so thousands of (event, map) pairs of uneven length share one launch; the
// per-trajectory arithmetic and reduction order are the same, so results are bitwise identical
// between the modes.

#include "internal.h"

#include <algorithm>
#include <cstring>

namespace morse {

namespace {

// ---------------------------------------------------------------------------
// Light-curve preparation, one workgroup per event: S_w and S_F with
// Neumaier-compensated partial sums combined by a fixed pairwise tree, Fbar = S_F/S_w, then
// wFc = w (F - Fbar) per point and V = sum w (F - Fbar)^2 the same way.

// Pairwise tree over the workgroup's Neumaier partials (sum, compensation) held in
// columns (2q, 2q + 1) of s_part, q < NQ, in a fixed order; every thread returns the
// totals.
template <int NQ>
__device__ __forceinline__ void tree_totals(double (*s_part)[4], double (&tot)[NQ]) {
  const int tid = threadIdx.x;
  for (int half = blockDim.x / 2; half >= 1; half >>= 1) {
    if (tid < half) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        double sm = s_part[tid][2 * q], c = s_part[tid][2 * q + 1];
        neumaier_add(sm, c, s_part[tid + half][2 * q]);
        s_part[tid][2 * q] = sm;
        s_part[tid][2 * q + 1] = c + s_part[tid + half][2 * q + 1];
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) tot[q] = s_part[0][2 * q] + s_part[0][2 * q + 1];
  __syncthreads();
}

// Light curve e (one workgroup of 256; see above).  Up to kLcKeep points a lane stay in
// registers from the first pass to the second; 0: the second reads them again.
template <int kLcKeep>
__device__ void lc_prep(const LcView& lc, double* wFc, double* sums, uint32_t* sorted, int32_t e,
                        double (*s_part)[4]) {
  const int64_t a = lc.off[e], b = lc.off[e + 1];
  const bool keep = kLcKeep > 0 && b - a <= kLcKeep * 256;  // uniform
  double kw[kLcKeep + 1], kF[kLcKeep + 1];
  double s0 = 0, c0 = 0, s1 = 0, c1 = 0;
  if (keep) {
#pragma unroll
    for (int q = 0; q < kLcKeep; ++q) {
      const int64_t i = a + threadIdx.x + 256 * q;
      kw[q] = kF[q] = 0.0;
      if (i < b) {
        kw[q] = lc.w[i];
        kF[q] = lc.F[i];
      }
    }
#pragma unroll
    for (int q = 0; q < kLcKeep; ++q)
      if (a + threadIdx.x + 256 * q < b) {
        neumaier_add(s0, c0, kw[q]);
        neumaier_add(s1, c1, kw[q] * kF[q]);
      }
  } else {
    for (int64_t i = a + threadIdx.x; i < b; i += 256) {
      const double wi = lc.w[i];
      neumaier_add(s0, c0, wi);
      neumaier_add(s1, c1, wi * lc.F[i]);
    }
  }
  s_part[threadIdx.x][0] = s0;
  s_part[threadIdx.x][1] = c0;
  s_part[threadIdx.x][2] = s1;
  s_part[threadIdx.x][3] = c1;
  __syncthreads();
  double t01[2];
  tree_totals<2>(s_part, t01);
  const double Sw = t01[0];
  const double Fbar = t01[1] / Sw;
  double s2 = 0, c2 = 0;
  auto second = [&](int64_t i, double wi, double Fi) {
    const double d = Fi - Fbar;
    const double wd = wi * d;
    wFc[i] = wd;
    neumaier_add(s2, c2, wd * d);
  };
  if (keep) {
#pragma unroll
    for (int q = 0; q < kLcKeep; ++q) {
      const int64_t i = a + threadIdx.x + 256 * q;
      if (i < b) second(i, kw[q], kF[q]);
    }
  } else {
    for (int64_t i = a + threadIdx.x; i < b; i += 256) second(i, lc.w[i], lc.F[i]);
  }
  s_part[threadIdx.x][0] = s2;
  s_part[threadIdx.x][1] = c2;
  __syncthreads();
  double t2[1];
  tree_totals<1>(s_part, t2);
  if (threadIdx.x == 0) {
    sums[3 * e] = Sw;
    sums[3 * e + 1] = Fbar;
    sums[3 * e + 2] = t2[0];
  }
  if (sorted) {  // false with a NaN time: no order holds
    int ok = 1;
    for (int64_t i = a + threadIdx.x; i + 1 < b; i += 256) ok &= lc.t[i] <= lc.t[i + 1] ? 1 : 0;
    ok = __syncthreads_and(ok);
    if (threadIdx.x == 0) sorted[e] = (uint32_t)ok;
  }
}

// Per-trajectory constants: FP64 trigonometry, rounded once to binary32.
__device__ __forceinline__ TrajC make_traj(double t0, double u0, double tE, double al) {
  double s, c;
  sincos(al, &s, &c);
  TrajC r;
  r.t0 = t0;
  r.iE = (float)(1.0 / tE);
  r.ca = (float)c;
  r.sa = (float)s;
  r.bx = (float)(-u0 * s);
  r.by = (float)(u0 * c);
  r.pad = 0.0f;
  return r;
}

// Scoring order of trajectory lists: each trajectory's (list, alpha, tE bucket) key, then
// the shared bucket sort (its order holds indices over all lists).  Neighbours then follow
// nearby lines at nearby speeds, so the chunks that lie on the map for one mostly do for
// all.  24 events x 8 maps x 16384 trajectories: 8.69 ms, 8.78 ms in 256 directions alone.
__device__ __forceinline__ uint32_t perm_key(const TrajC& c, int64_t i, int64_t n_traj) {
  const float a = atan2f(c.sa, c.ca);  // (-pi, pi]
  const float q = 4.0f * __log2f(c.iE);
  int b = 0, s = 0;
  if (!isnan(a)) b = min(max((int)((a + 3.14159265f) * (kPermDirs / 6.28318531f)), 0), kPermDirs - 1);
  if (fabsf(q) < 1e6f) s = (int)floorf(q) & (kPermSpeeds - 1);
  return (uint32_t)((i / n_traj) * kPermBins + (b * kPermSpeeds + s));
}

// Quad packing (layout in MapC) of cells q, q + stride, ...; cells beyond the map (tile
// padding) are zero and never sampled.
__device__ __forceinline__ void pack_quads(const MapC& m, uint32_t first, uint32_t stride) {
  Quad* out = const_cast<Quad*>(m.quad);
  for (uint64_t at = first; at < m.cells; at += stride) {
    const uint32_t q = (uint32_t)at;
    const uint32_t tile = q >> 3, r = q & 7u, tj = tile / m.tiles_x;
    const uint32_t i = (tile - tj * m.tiles_x) * 4 + (r >> 1), j = tj * 2 + (r & 1u);
    Quad v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (i + 1 < (uint32_t)m.mx && j + 1 < (uint32_t)m.my) {
      const float* row = m.map + (size_t)j * m.mx + i;
      v.v00 = row[0];
      v.e0 = row[1] - row[0];
      v.v01 = row[m.mx];
      v.e1 = row[m.mx + 1] - row[m.mx];
    }
    out[q] = v;
  }
}

// All the preparation of a call in one launch, its parts side by side: a workgroup per light
// curve (the longest chain, first), then the trajectory constants, the cleared counters and
// the packing.  One after another they were four launches of 4 to 12 us each.
// kLcKeep: with points kept in registers (96 in all) five wavefronts fit a SIMD, without seven.
template <int kLcKeep>
__global__ __launch_bounds__(256) void k_prep(PrepArgs a) {
  __shared__ double s_part[256][4];
  uint32_t block = blockIdx.x;
  if (block < a.event_blocks) {
    for (int32_t e = (int32_t)block; e < a.n_events; e += (int32_t)a.event_blocks)
      lc_prep<kLcKeep>(a.lc, const_cast<double*>(a.lc.wFc), const_cast<double*>(a.lc.sums),
              const_cast<uint32_t*>(a.lc.sorted), e, s_part);
    return;
  }
  block -= a.event_blocks;
  if (block < a.traj_blocks) {
    for (int64_t i = block * (int64_t)256 + threadIdx.x; i < a.n; i += (int64_t)a.traj_blocks * 256) {
      TrajC c;
      if (a.axes) {  // [u0 | alpha | t0 | tE]; index ((iu*na + ia)*nt + it)*ne + ie
        int64_t r = i;
        const int ie = (int)(r % a.ne);
        r /= a.ne;
        const int it = (int)(r % a.nt);
        r /= a.nt;
        const int ia = (int)(r % a.na), iu = (int)(r / a.na);
        c = make_traj(a.axes[a.nu + a.na + it], a.axes[iu], a.axes[a.nu + a.na + a.nt + ie], a.axes[a.nu + ia]);
      } else {
        const double* p = a.params + 4 * i;
        c = make_traj(p[0], p[1], p[2], p[3]);
      }
      a.tc[i] = c;
      if (a.key) a.key[i] = perm_key(c, i, a.n_traj);
    }
    return;
  }
  block -= a.traj_blocks;
  if (block < a.zero_blocks) {
    for (uint64_t i = block * (uint64_t)256 + threadIdx.x; i < a.n_zero; i += a.zero_blocks * (uint64_t)256)
      a.zero[i] = 0u;
    return;
  }
  block -= a.zero_blocks;
  pack_quads(uniform(a.maps[block / a.pack_blocks]), (block % a.pack_blocks) * 256u + threadIdx.x,
             a.pack_blocks * 256u);
}

// Host metadata by value: kPutWords words of kernel arguments a launch.
struct PutWords {
  uint32_t w[kPutWords];
};
__global__ __launch_bounds__(256) void k_put(uint32_t* dst, uint32_t n, PutWords v) {
  for (uint32_t i = threadIdx.x; i < n; i += 256) dst[i] = v.w[i];
}

// ---------------------------------------------------------------------------
// Score TU trajectories with one wavefront.  All lanes return the same values.
// Each lane takes the points lane, lane + 64, ... in order; every trajectory's sums see the
// points in the same order for any TU and C, and wave_sums reduces each over the butterfly
// tree, so the results do not depend on the shape.
//
// Chunks.  The position along a trajectory is a chain of binary32 operations each monotone
// in the point's time, so over points in time order the grid coordinates gx and gy are
// monotone, and a chunk of 64 points whose first and last point lie on the map lies on it
// as a whole; one whose ends lie beyond the same side lies off it.  Lane l looks at the
// ends of chunk l, and ballots give both sets for 64 chunks and all TU trajectories.  A
// chunk on the map for every trajectory takes the short form: no on-map test, no selected
// cell, no single-lens branch; a trajectory that a chunk misses takes the single-lens
// magnification and no cell.  Others, and events whose times are not in order, take the
// general form.  All forms give the same bits.
//
// C chunks at a time (the short form) with few trajectories per wavefront, so that TU C
// cells are in flight: a search too small to fill the chip waits for loads, not for issue.
//
// Bound: instruction issue (a vector instruction every 3.1 cycles per SIMD, 80% of the
// launch), then the cells' way from L2.  The short form takes 31 instructions per point and
// trajectory, 6 of them FP64; with the general form, the off-map chunks and the work per
// group 36 on a 64 x 64 x 16 x 8 grid x 3000 points (1.49 ms, 1.06e12 point-evaluations/s;
// 1.77 ms before, 2.09 ms with the former untuned shape, on the same card; 1.60 and 1.68 on two others) and
// 39 on 24 ragged events x 8 maps x 16384 random trajectories (8.7 ms for 9.2; untuned 11.1).
// Also measured: the constants in vector registers (1.79 ms on the grid: five wavefronts
// per SIMD for six), no cell loads at all 1.47 ms, and straight-line code for each of the
// 16 on/off patterns of four trajectories (1.49 and 8.72 ms: no faster).
struct TrajV {
  float t0p, iE, ca, sa, bx, by;
};
__device__ __forceinline__ TrajV traj_v(const TrajC& c, float t0p) {
  return TrajV{t0p, c.iE, c.ca, c.sa, c.bx, c.by};
}

// Grid coordinates at time tt.  kCentred: a window about (0, 0), where zeta - s = zeta.
struct MapV {
  float sx, sy, kx, ky, ox, oy;
};
struct GridPos {
  float tau, gx, gy;
};
template <bool kCentred>
__device__ __forceinline__ GridPos grid_pos(const MapV& m, const TrajV& c, float tt) {
  GridPos g;
  g.tau = (tt - c.t0p) * c.iE;
  const float zx = g.tau * c.ca + c.bx, zy = g.tau * c.sa + c.by;
  if constexpr (kCentred) {
    g.gx = (zx * m.kx) + m.ox;
    g.gy = (zy * m.ky) + m.oy;
  } else {
    g.gx = ((zx - m.sx) * m.kx) + m.ox;
    g.gy = ((zy - m.sy) * m.ky) + m.oy;
  }
  return g;
}

// 0 <= g < l as an unsigned compare of the bit patterns (see locate).
__device__ __forceinline__ uint64_t inside(float g, float l) {
  return __builtin_amdgcn_ballot_w64(__float_as_uint(g) < __float_as_uint(l));
}
// Both values below 0, or both at or beyond l.
__device__ __forceinline__ uint64_t beyond(float g0, float g1, float l) {
  return (__builtin_amdgcn_ballot_w64(g0 < 0.0f) & __builtin_amdgcn_ballot_w64(g1 < 0.0f)) |
         (__builtin_amdgcn_ballot_w64(g0 >= l) & __builtin_amdgcn_ballot_w64(g1 >= l));
}

constexpr int kSegChunks = 64;            // chunks classified at a time
constexpr int kSegPoints = kSegChunks * kWave;
constexpr int32_t kClassifyMin = 256;     // shorter light curves take the general form
constexpr int32_t kPlainShort = 768;      // plain mode: so do these (see launch_search_plain)

struct LcPtrs {
  const float* t;
  const double* w;
  const double* wFc;
  const double* F;
  int32_t np;
  uint32_t sorted;
  double Sw, Fbar, V;
};

// The result of trajectory lane % TU.
struct GroupFit {
  double chi2, Fs, Fb;
};

// kShort: a short light curve, all of it in the general form, its next chunk of times and weights
// loaded before the cells of this one are there.
template <int TU, int C, bool kCentred, bool kShort = false>
__device__ __forceinline__ GroupFit score_group(const MapC& m, const LcPtrs& lc, const TrajV (&c)[TU],
                                                int lane) {
  const MapV mv{m.sx, m.sy, m.kx, m.ky, m.ox, m.oy};
  const int32_t np = lc.np;
  double acc[3 * TU];  // (B1, B2, C) per trajectory
#pragma unroll
  for (int q = 0; q < 3 * TU; ++q) acc[q] = 0.0;
  auto add = [&](int v, float A, double wv, double fv) {
    const double b = (double)A - 1.0;
    const double wb = wv * b;
    acc[3 * v] += wb;
    acc[3 * v + 1] = fma(wb, b, acc[3 * v + 1]);
    acc[3 * v + 2] = fma(b, fv, acc[3 * v + 2]);
  };
  float ta = 0.0f;
  double wa = 0.0, fa = 0.0;
  auto load = [&](uint32_t i) {
    const uint32_t ii = min(i, (uint32_t)(np - 1));
    ta = ldg(lc.t, ii);
    wa = ldg(lc.w, ii);
    fa = ldg(lc.wFc, ii);
  };
  if (kShort) load((uint32_t)lane);
  for (int32_t base = 0; base < np; base += kSegPoints) {
    const int32_t nch = min((np - base + kWave - 1) / kWave, kSegChunks);
    uint64_t off[TU], fast = 0;  // chunks off the map per trajectory, on it for every one
#pragma unroll
    for (int v = 0; v < TU; ++v) off[v] = 0;
    if (!kShort && lc.sorted && np >= kClassifyMin) {  // uniform
      const int32_t i0 = min(base + lane * kWave, np - 1), i1 = min(base + lane * kWave + kWave - 1, np - 1);
      const float ta = ldg(lc.t, (uint32_t)i0), tb = ldg(lc.t, (uint32_t)i1);
      const int32_t full = min((np - base) / kWave, kSegChunks);  // chunks of 64 points
      fast = full >= 64 ? ~0ull : (1ull << full) - 1ull;
#pragma unroll
      for (int v = 0; v < TU; ++v) {
        const GridPos a = grid_pos<kCentred>(mv, c[v], ta), b = grid_pos<kCentred>(mv, c[v], tb);
        fast &= inside(a.gx, m.lx) & inside(a.gy, m.ly) & inside(b.gx, m.lx) & inside(b.gy, m.ly);
        off[v] = beyond(a.gx, b.gx, m.lx) | beyond(a.gy, b.gy, m.ly);
      }
    }
    for (int32_t k = 0; k < nch; ++k) {
      // the run of chunks from k on that lie on the map for every trajectory, C at a time
      const uint64_t rest = ~(fast >> k);
      const int32_t run = (rest ? __builtin_ctzll(rest) : kSegChunks) / C;
      uint32_t i = (uint32_t)(base + k * kWave + lane);
      for (int32_t r = 0; r < run; ++r, i += C * kWave) {
        float tt[C], fx[C][TU], fy[C][TU];
        double wv[C], fv[C];
        Quad cell[C][TU];
#pragma unroll
        for (int u = 0; u < C; ++u) tt[u] = ldg(lc.t, i + u * kWave);
#pragma unroll
        for (int u = 0; u < C; ++u) {
          wv[u] = ldg(lc.w, i + u * kWave);
          fv[u] = ldg(lc.wFc, i + u * kWave);
        }
#pragma unroll
        for (int u = 0; u < C; ++u)
#pragma unroll
          for (int v = 0; v < TU; ++v) {
            const GridPos g = grid_pos<kCentred>(mv, c[v], tt[u]);
            fx[u][v] = __builtin_amdgcn_fractf(g.gx);
            fy[u][v] = __builtin_amdgcn_fractf(g.gy);
            cell[u][v] = ldq(m, cell_index(m, (uint32_t)g.gx, (uint32_t)g.gy));
          }
#pragma unroll
        for (int u = 0; u < C; ++u)
#pragma unroll
          for (int v = 0; v < TU; ++v) add(v, blend(cell[u][v], fx[u][v], fy[u][v]), wv[u], fv[u]);
      }
      k += run * C;
      if (k >= nch) break;
      const bool act = i < (uint32_t)np;
      if (!kShort) load(i);
      const float tt = ta;
      const double wv = wa, fv = fa;
      if (kShort) load(i + kWave);
      float tau[TU], fx[TU], fy[TU];
      uint64_t on[TU];
      Quad cell[TU];
#pragma unroll
      for (int v = 0; v < TU; ++v) {
        on[v] = 0;
        cell[v] = Quad{0.0f, 0.0f, 0.0f, 0.0f};
        fx[v] = fy[v] = 0.0f;
        const GridPos g = grid_pos<kCentred>(mv, c[v], tt);
        tau[v] = g.tau;
        if (!((off[v] >> k) & 1)) {  // uniform
          on[v] = inside(g.gx, m.lx) & inside(g.gy, m.ly);
          fx[v] = __builtin_amdgcn_fractf(g.gx);
          fy[v] = __builtin_amdgcn_fractf(g.gy);
          const bool mine = __builtin_amdgcn_inverse_ballot_w64(on[v]);
          cell[v] = ldq(m, mine ? cell_index(m, (uint32_t)g.gx, (uint32_t)g.gy) : 0u);
        }
      }
#pragma unroll
      for (int v = 0; v < TU; ++v) {
        float A = 0.0f;
        if (on[v]) A = blend(cell[v], fx[v], fy[v]);  // uniform
        if (~on[v]) {
          // the source position again from tau: the same operations, so the same bits,
          // and no register held across the loads
          float tv = tau[v];
          asm volatile("" : "+v"(tv));
          const float P = point_lens_A(tv * c[v].ca + c[v].bx, tv * c[v].sa + c[v].by);
          A = __builtin_amdgcn_inverse_ballot_w64(on[v]) ? A : P;
        }
        if (act) add(v, A, wv, fv);
      }
    }
  }
  // Totals to the lanes that fit them: lane l takes trajectory l % TU, so one fit serves all.
  int slot = 0;
  bool valid = true;
  reduce_scatter<3 * TU>(acc, lane, slot, valid);
  double tot[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    uint32_t from = 0;  // lane of sum j of each trajectory, a byte each
#pragma unroll
    for (int v = 0; v < TU; ++v) from |= (uint32_t)rs_lane<3 * TU>(3 * v + j) << (8 * v);
    tot[j] = __shfl(acc[0], (int)((from >> (8 * (lane % TU))) & 63u), kWave);
  }
  const Fit f = centred_fit(lc.Sw, lc.Fbar, lc.V, tot[0], tot[1], tot[2], fit_terms(np, kWave));
  GroupFit out{f.chi2, f.Fs, f.Fb};
  const uint64_t again = __builtin_amdgcn_ballot_w64(f.recheck);
#pragma unroll
  for (int v = 0; v < TU; ++v)
    if ((again >> v) & 1) {  // uniform
      const double Fs = read_lane(f.Fs, v), Fb = read_lane(f.Fb, v);
      double q = 0.0, qc = 0.0;
      for (int32_t i = lane; i < np; i += kWave) {
        const double a = (double)sample_A(m, ldg(lc.t, (uint32_t)i), c[v].t0p, c[v].iE, c[v].ca,
                                          c[v].sa, c[v].bx, c[v].by);
        const double r = ldg(lc.F, (uint32_t)i) - Fs * a - Fb;
        neumaier_add(q, qc, (ldg(lc.w, (uint32_t)i) * r) * r);
      }
      const double x = wave_sum(q + qc);
      if (lane % TU == v) out.chi2 = x;
    }
  return out;
}

// Chunks taken at a time in the short form: four cells in flight for any TU.
template <int TU>
constexpr int kChunks = 4 / TU;

template <bool kCentred, bool kShort>
__global__ __launch_bounds__(256) void k_search_plain(const TrajC* __restrict__ tc, int64_t n_traj,
                                                      LcView lc, int32_t e, MapC m, SearchOut out) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wpb = blockDim.x / kWave;
  const int64_t nw = (int64_t)gridDim.x * wpb;
  const int64_t p0 = lc.off[e];
  const LcPtrs lp{lc.t + p0, lc.w + p0, lc.wFc + p0, lc.F + p0, (int32_t)(lc.off[e + 1] - p0),
                  lc.sorted ? lc.sorted[e] : 0u, lc.sums[3 * e], lc.sums[3 * e + 1], lc.sums[3 * e + 2]};
  const double tref = lc.t_ref[e];
  for (int64_t k = (int64_t)blockIdx.x * wpb + (threadIdx.x / kWave); k < n_traj; k += nw) {
    const TrajC tk = uniform(tc[k]);
    const TrajV c[1] = {traj_v(tk, (float)(tk.t0 - tref))};
    const GroupFit r = score_group<1, kShort ? 1 : kChunks<1>, kCentred, kShort>(m, lp, c, lane);
    if (lane == 0) {
      if (out.chi2) out.chi2[k] = r.chi2;
      if (out.fs) out.fs[k] = r.Fs;
      if (out.fb) out.fb[k] = r.Fb;
    }
  }
}

// Batched search: one launch over (map, event, trajectory group) items, one item per
// wavefront, so thousands of (event, map) pairs of uneven length share a launch and the
// hardware's dispatcher balances them.  Workgroups are dispatched to the 8 XCDs in turn, so
// blockIdx % 8 names the XCD; the items are cut into chunks of a.chunk workgroups, dealt to
// the XCDs in turn: an XCD works through neighbouring items (its L2 serves one compact part
// of the work), and the chunks spread events of different lengths over all XCDs.  (A
// persistent grid with one work queue per XCD spent 20 us on draining the queues, 65,000
// atomics on eight counters: 1024 trajectories x 1000 points took 24 us and take 15.6.)
// Trajectories are taken in groups of
// TU neighbours, scored together.  Item = (map * n_events + event) * n_blocks + b
// scores groups b, b + n_blocks, ... (traj_per_item / TU of them): the waves of an
// XCD running at the same time take neighbouring items, so they score neighbouring
// trajectories of the same map and light curve.  On a product grid the scoring order
// runs over (alpha, u0, tE, t0), t0 fastest, so neighbouring trajectories lie on
// the same line through the map, cross it at the same speed and share most of the chunks
// that lie on it (the (u0, alpha, t0, tE) index order of the outputs is unchanged);
// trajectory lists are scored in the order of `perm`, grouped by direction and speed, for
// the same reason.
// Trajectory index of scoring position p of event e (see k_search_batched).
__device__ __forceinline__ int32_t traj_of(const BatchedArgs& a, uint32_t p, int32_t e) {
  if (a.na <= 0) {
    if (!a.perm) return (int32_t)p;
    const int64_t base = a.shared ? 0 : (int64_t)e * a.n_traj;  // perm holds indices over all lists
    return (int32_t)((int64_t)uniform(a.perm[base + p]) - base);
  }
  const uint32_t it = p % (uint32_t)a.nt, r1 = p / (uint32_t)a.nt;
  const uint32_t ie = r1 % (uint32_t)a.ne, r2 = r1 / (uint32_t)a.ne;
  const uint32_t iu = r2 % (uint32_t)a.nu, ia = r2 / (uint32_t)a.nu;
  return (int32_t)(((iu * a.na + ia) * a.nt + it) * a.ne + ie);
}

// All counts are below 2^31 (the host checks n_traj x n_events x n_maps).
template <int TU, bool kCentred>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(6))) void k_search_batched(BatchedArgs a) {
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t n_traj = (uint32_t)a.n_traj;
  const uint32_t ng = (n_traj + TU - 1) / TU;
  const uint32_t nb = search_blocks(n_traj, a.traj_per_item, TU);
  const uint32_t block = a.first + blockIdx.x;
  const uint32_t xcd = block % 8u, j = block / 8u;
  const uint32_t deal = j / a.chunk, wg = (deal * 8u + (xcd + deal * a.rotate) % 8u) * a.chunk + j % a.chunk;
  // first-lane read: the item is provably wave-uniform, so everything derived from it
  // (indices, map and trajectory constants) stays in scalar registers
  const uint64_t item64 = (uint64_t)wg * (blockDim.x / kWave) +
                          (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (item64 < (uint64_t)nb * a.n_events * a.n_maps) {
    const uint32_t item = (uint32_t)item64;
    const uint32_t b = item % nb, me = item / nb;
    const int32_t e = (int32_t)(me % (uint32_t)a.n_events);
    const int32_t mi = (int32_t)(me / (uint32_t)a.n_events);
    const MapC m = uniform(a.maps[mi]);
    const int64_t p0 = uniform(a.lc.off[e]);
    const LcPtrs lp{a.lc.t + p0, a.lc.w + p0, a.lc.wFc + p0, a.lc.F + p0,
                    (int32_t)(uniform(a.lc.off[e + 1]) - p0), a.lc.sorted ? uniform(a.lc.sorted[e]) : 0u,
                    uniform(a.lc.sums[3 * e]), uniform(a.lc.sums[3 * e + 1]), uniform(a.lc.sums[3 * e + 2])};
    const double tref = uniform(a.lc.t_ref[e]);
    const TrajC* tc = a.tc + (a.shared ? 0 : (int64_t)e * a.n_traj);
    const int64_t obase = ((int64_t)e * a.n_maps + mi) * a.n_traj;
    for (uint32_t g = b; g < ng; g += nb) {
      TrajV c[TU];
      int32_t mine = 0;  // index of the trajectory whose result this lane holds
#pragma unroll
      for (int v = 0; v < TU; ++v) {  // a short last group repeats its last trajectory
        const int32_t k = traj_of(a, min(g * TU + v, n_traj - 1), e);
        const TrajC tk = uniform(tc[k]);
        c[v] = traj_v(tk, uniform((float)(tk.t0 - tref)));
        mine = lane % TU == v ? k : mine;
      }
      const GroupFit r = score_group<TU, kChunks<TU>, kCentred>(m, lp, c, lane);
      if (lane < TU && g * TU + lane < n_traj) {
        const int64_t o = obase + mine;
        if (a.out.chi2) a.out.chi2[o] = r.chi2;
        if (a.out.fs) a.out.fs[o] = r.Fs;
        if (a.out.fb) a.out.fb[o] = r.Fb;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Selection.  Keys order doubles totally: -0 is taken as +0, NaN after everything;
// ties broken by the index.
__device__ __forceinline__ uint64_t order_key(double x) {
  if (x != x) return ~0ull;
  if (x == 0.0) x = 0.0;
  const uint64_t b = (uint64_t)__double_as_longlong(x);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// (key, index) pairs in lexicographic order.
struct KeyIdx {
  uint64_t key;
  uint32_t idx;
};
__device__ __forceinline__ bool before(uint64_t ka, uint32_t ia, uint64_t kb, uint32_t ib) {
  return ka < kb || (ka == kb && ia < ib);
}
__device__ __forceinline__ void wave_first(KeyIdx& v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const uint64_t k = __shfl_xor(v.key, o, kWave);
    const uint32_t i = (uint32_t)__shfl_xor((int)v.idx, o, kWave);
    if (before(k, i, v.key, v.idx)) v = KeyIdx{k, i};
  }
}

// Whether this workgroup is the last of `n` to come here (one ticket counter, zero before;
// every thread returns the same).  What the workgroups passed on before by device-scope
// atomics (put_device, atomicAdd: they act at the coherence point, and each wave waits here
// until its own have) the last may read by device-scope loads (get_device).  A fence would
// also write back the whole L2, which the scores just filled: 512 workgroups 65 us, so 10.
__device__ __forceinline__ bool last_here(uint32_t* ticket, uint32_t n) {
  __shared__ uint32_t s_last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) s_last = atomicAdd(ticket, 1u) == n - 1 ? 1u : 0u;
  __syncthreads();
  return s_last != 0u;
}
template <class T>
__device__ __forceinline__ void put_device(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ T get_device(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Smallest (chi2, index) of segment blockIdx.y, gridDim.x workgroups a segment: each leaves its
// slice's first pair, the last takes the first of those.  (One workgroup a segment read a
// single segment of 524,288 in 0.71 ms, these 10 us.)
__global__ __launch_bounds__(256) void k_best(const double* __restrict__ chi2, int64_t seg_len,
                                              uint32_t* __restrict__ ticket, KeyIdx* __restrict__ part,
                                              double* __restrict__ best_chi2,
                                              int64_t* __restrict__ best_idx) {
  __shared__ KeyIdx s_first[4];
  const int64_t seg = blockIdx.y;
  const double* base = chi2 + seg * seg_len;
  KeyIdx v{~0ull, 0xffffffffu};
  const int64_t step = (int64_t)gridDim.x * 256;
  for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < seg_len; i += 4 * step) {
    double x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = i + q * step < seg_len ? base[i + q * step] : 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (i + q * step < seg_len) {
        const uint64_t k = order_key(x[q]);
        const uint32_t j = (uint32_t)(i + q * step);
        if (before(k, j, v.key, v.idx)) v = KeyIdx{k, j};
      }
  }
  auto block_first = [&]() {
    wave_first(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s_first[threadIdx.x >> 6] = v;
    __syncthreads();
    v = s_first[0];
#pragma unroll
    for (int q = 1; q < 4; ++q)
      if (before(s_first[q].key, s_first[q].idx, v.key, v.idx)) v = s_first[q];
  };
  block_first();
  if (gridDim.x > 1) {
    if (threadIdx.x == 0) {
      put_device(&part[seg * gridDim.x + blockIdx.x].key, v.key);
      put_device(&part[seg * gridDim.x + blockIdx.x].idx, v.idx);
    }
    if (!last_here(ticket + seg, gridDim.x)) return;
    v = KeyIdx{~0ull, 0xffffffffu};
    for (uint32_t q = threadIdx.x; q < gridDim.x; q += 256) {
      const KeyIdx* w = part + seg * gridDim.x + q;
      const uint64_t k = get_device(&w->key);
      const uint32_t j = get_device(&w->idx);
      if (before(k, j, v.key, v.idx)) v = KeyIdx{k, j};
    }
    block_first();
  }
  if (threadIdx.x == 0) {
    if (best_chi2) best_chi2[seg] = base[v.idx];
    if (best_idx) best_idx[seg] = (int64_t)v.idx;
  }
}

// Top-k per segment, the k smallest by (order_key(chi2), index).  A segment of at most TK_CAP
// values is put in order in LDS at once.  A longer one first goes through up to six passes
// of 11-bit digits: every workgroup histograms its slice in LDS and adds it to the
// segment's histogram, and the last of them scans the bins and fixes the next digit of
// the threshold.  As soon as the values below the threshold's bin and those in it fit the
// segment's list (mostly after two passes) the rest return at once: all of them are collected
// and put in order.  Where more values than that equal the threshold to the last bit, the
// first by index are taken, from the counts of each workgroup's slice (k_tk_ties).  The
// launches, not the values, are what this takes: one for a short segment, nine for a long
// one, where nine passes of two launches, set-up, collection and ranking made 21.  A whole
// search of 1024 trajectories 216 -> 85 us with it, one of 524,288 2.51 -> 1.70 ms.
constexpr int TK_BINS = 2048;
constexpr int TK_THREADS = 256;
constexpr int TK_MAXK = 4096;
constexpr int TK_PASSES = 6;
constexpr int TK_CAP = 2 * TK_MAXK;

struct TkState {    // cleared before the first pass
  uint64_t prefix;  // fixed high digits of the threshold key
  int32_t below;    // values below the prefix (at most k - 1)
  int32_t done;     // passes made when the candidates fit the list, 0 until then
  int32_t taken;    // collected
  uint32_t ticket[TK_PASSES + 1];
  int32_t pad[4];
};
static_assert(sizeof(TkState) == 64, "TkState layout");

// Bits 63..53, 52..42, 41..31, 30..20, 19..9, 8..0 of the key.
__device__ __forceinline__ int tk_shift(int pass) { return pass < 5 ? 53 - 11 * pass : 0; }

// One digit of bin `d` counted for the active lanes (LDS histogram): lanes that share the
// first active lane's bin, usually most in the exponent's digits, add once.
__device__ __forceinline__ void tk_count(uint32_t* h, uint32_t d, bool act) {
  const uint64_t m = __builtin_amdgcn_ballot_w64(act);
  if (m == 0) return;
  const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, __builtin_ctzll(m));
  const uint64_t same = __builtin_amdgcn_ballot_w64(act && d == d0);
  if ((threadIdx.x & (kWave - 1)) == __builtin_ctzll(m)) atomicAdd(&h[d0], (uint32_t)__popcll(same));
  if (act && d != d0) atomicAdd(&h[d], 1u);
}

// The bin in which the krem-th smallest (1-based) of the counts falls: digit, the counts
// before it and its own, on every thread.  NT threads, TK_BINS counts c(b).
template <int NT, class F>
__device__ __forceinline__ void tk_pick(F c, int64_t krem, uint32_t* s_wave, int32_t* s_out, int& digit,
                                        int64_t& less, int64_t& in) {
  constexpr int PER = TK_BINS / NT;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint32_t v[PER], part = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    v[q] = c(threadIdx.x * PER + q);
    part += v[q];
  }
  uint32_t incl = part;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t l = (uint32_t)__shfl_up((int)incl, o);
    if (lane >= o) incl += l;
  }
  if (lane == kWave - 1) s_wave[wave] = incl;
  __syncthreads();
  int64_t cum = (int64_t)incl - part;
  for (int w = 0; w < wave; ++w) cum += s_wave[w];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    if (cum < krem && krem <= cum + v[q]) {
      s_out[0] = threadIdx.x * PER + q;
      s_out[1] = (int32_t)cum;  // below krem <= 4096
      s_out[2] = (int32_t)v[q];
    }
    cum += v[q];
  }
  __syncthreads();
  digit = s_out[0];
  less = s_out[1];
  in = (uint32_t)s_out[2];
  __syncthreads();
}

__global__ __launch_bounds__(TK_THREADS) void k_tk_hist(const double* __restrict__ chi2, int64_t seg_len,
                                                        int32_t k, int32_t cap, TkState* __restrict__ st,
                                                        uint32_t* __restrict__ hist, int pass) {
  __shared__ uint32_t h[TK_BINS];
  __shared__ uint32_t s_wave[TK_THREADS / kWave];
  __shared__ int32_t s_out[3];
  const int64_t seg = blockIdx.y;
  if (st[seg].done) return;  // uniform per segment
  const uint64_t prefix = st[seg].prefix;
  const int64_t krem = (int64_t)k - st[seg].below;  // k <= seg_len: longer than TK_CAP
  const int shift = tk_shift(pass);
  const uint64_t mask = pass == 0 ? 0ull : ~0ull << tk_shift(pass - 1);
  const uint32_t digit = pass < 5 ? TK_BINS - 1 : 511u;
  for (int b = threadIdx.x; b < TK_BINS; b += TK_THREADS) h[b] = 0u;
  __syncthreads();
  const double* base = chi2 + seg * seg_len;
  const int64_t step = (int64_t)gridDim.x * TK_THREADS;
  const int64_t rounds = (seg_len + 4 * step - 1) / (4 * step);  // the same for every lane
  int64_t i = blockIdx.x * (int64_t)TK_THREADS + threadIdx.x;
  for (int64_t r = 0; r < rounds; ++r, i += 4 * step) {
    double x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = i + q * step < seg_len ? base[i + q * step] : 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint64_t key = order_key(x[q]);
      tk_count(h, (uint32_t)(key >> shift) & digit, i + q * step < seg_len && (key & mask) == prefix);
    }
  }
  __syncthreads();
  uint32_t* g = hist + seg * TK_BINS;
  for (int b = threadIdx.x; b < TK_BINS; b += TK_THREADS)
    if (h[b]) atomicAdd(&g[b], h[b]);
  if (!last_here(&st[seg].ticket[pass], gridDim.x)) return;
  int d;
  int64_t less, in;
  tk_pick<TK_THREADS>([&](int b) { return get_device(&g[b]); }, krem, s_wave, s_out, d, less, in);
  if (threadIdx.x == 0) {
    st[seg].prefix = prefix | ((uint64_t)d << shift);
    st[seg].below += (int32_t)less;
    if (st[seg].below + in <= cap) st[seg].done = pass + 1;
  }
  for (int b = threadIdx.x; b < TK_BINS; b += TK_THREADS) g[b] = 0u;  // for the next pass
}

// Slice of workgroup b of the segment, in index order over the workgroups: a multiple of the
// workgroup's size, so that its rounds are whole.
__device__ __forceinline__ int64_t tk_slice(int64_t seg_len) {
  const int64_t rounds = (seg_len + TK_THREADS - 1) / TK_THREADS;
  return (rounds + gridDim.x - 1) / gridDim.x * TK_THREADS;
}

// Where more values equal the threshold key than can be taken: how many lie in the slices
// before each workgroup's (at most TK_BINS of them), left in the segment's histogram.
__global__ __launch_bounds__(TK_THREADS) void k_tk_ties(const double* __restrict__ chi2, int64_t seg_len,
                                                        TkState* __restrict__ st, uint32_t* __restrict__ hist) {
  __shared__ uint32_t s_wave[TK_THREADS / kWave];
  const int64_t seg = blockIdx.y;
  if (st[seg].done) return;  // uniform per segment
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const uint64_t key = st[seg].prefix;
  const double* base = chi2 + seg * seg_len;
  const int64_t slice = tk_slice(seg_len), i0 = blockIdx.x * slice, i1 = min(i0 + slice, seg_len);
  uint32_t count = 0;
  for (int64_t i = i0 + tid; i < i1; i += TK_THREADS) count += order_key(base[i]) == key ? 1u : 0u;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) count += (uint32_t)__shfl_xor((int)count, o, kWave);
  if (lane == 0) s_wave[wave] = count;
  __syncthreads();
  uint32_t* g = hist + seg * TK_BINS;
  if (tid == 0) put_device(&g[blockIdx.x], s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3]);
  if (!last_here(&st[seg].ticket[TK_PASSES], gridDim.x)) return;
  uint32_t cum = 0;
  for (uint32_t b0 = 0; b0 < gridDim.x; b0 += TK_THREADS) {
    const uint32_t b = b0 + tid;
    const uint32_t v = b < gridDim.x ? get_device(&g[b]) : 0u;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t l = (uint32_t)__shfl_up((int)incl, o);
      if (lane >= o) incl += l;
    }
    __syncthreads();
    if (lane == kWave - 1) s_wave[wave] = incl;
    __syncthreads();
    uint32_t before_wave = 0, all = 0;
    for (int w = 0; w < TK_THREADS / kWave; ++w) {
      before_wave += w < wave ? s_wave[w] : 0u;
      all += s_wave[w];
    }
    if (b < gridDim.x) g[b] = cum + before_wave + incl - v;
    cum += all;
  }
}

// The values below the threshold's bin and, where the passes ended early, those in it;
// otherwise those below the threshold key and the first of those equal to it.
__global__ __launch_bounds__(TK_THREADS) void k_tk_collect(const double* __restrict__ chi2, int64_t seg_len,
                                                           int32_t k, int32_t cap, TkState* __restrict__ st,
                                                           const uint32_t* __restrict__ hist,
                                                           uint64_t* __restrict__ keys,
                                                           uint32_t* __restrict__ idx) {
  __shared__ uint32_t s_wave[TK_THREADS / kWave];
  __shared__ int32_t s_at;
  const int64_t seg = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const uint64_t prefix = st[seg].prefix;
  const int32_t done = st[seg].done;
  const double* base = chi2 + seg * seg_len;
  const int64_t slice = tk_slice(seg_len), i0 = blockIdx.x * slice, i1 = min(i0 + slice, seg_len);
  // inclusive sum over the workgroup's threads; `all` of them
  auto scan = [&](uint32_t v, uint32_t& all) {
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t l = (uint32_t)__shfl_up((int)v, o);
      if (lane >= o) v += l;
    }
    __syncthreads();
    if (lane == kWave - 1) s_wave[wave] = v;
    __syncthreads();
    all = 0;
    for (int w = 0; w < TK_THREADS / kWave; ++w) {
      v += w < wave ? s_wave[w] : 0u;
      all += s_wave[w];
    }
    return v;
  };
  const int shift = done ? tk_shift(done - 1) : 0;
  const uint64_t top = (prefix >> shift) + (done ? 1u : 0u);  // done: the whole bin
  int64_t ties = done ? 0 : hist[seg * TK_BINS + blockIdx.x];
  const int64_t krem = done ? 0 : (int64_t)k - st[seg].below;
  // two sweeps, counting and writing, with one claim of the list a workgroup in between
  // (a claim a wave of 256 values: 41 us on 524,288, the counter's atomics one after another)
  int at = 0;
  for (int sweep = 0; sweep < 2; ++sweep) {
    uint32_t count = 0;
    int64_t t = ties;
    for (int64_t r = i0; r < i1; r += 4 * TK_THREADS) {  // uniform
      double x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = r + q * TK_THREADS + tid < i1 ? base[r + q * TK_THREADS + tid] : 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t i = r + q * TK_THREADS + tid;
        const uint64_t key = order_key(x[q]);
        bool take = i < i1 && (key >> shift) < top;
        if (!done && t < krem) {  // uniform: the first ties by index
          uint32_t all;
          const uint32_t eq = i < i1 && key == prefix ? 1u : 0u;
          const uint32_t rank = scan(eq, all) - eq;
          take = take || (eq && t + rank < krem);
          t += all;
        }
        if (take && sweep == 1 && at < cap) {
          keys[seg * cap + at] = key;
          idx[seg * cap + at] = (uint32_t)i;
        }
        at += take ? 1 : 0;
        count += take ? 1u : 0u;
      }
    }
    if (sweep == 0) {
      uint32_t all;
      const uint32_t incl = scan(count, all);
      if (all == 0) return;
      if (tid == 0) s_at = atomicAdd(&st[seg].taken, (int32_t)all);
      __syncthreads();
      at = s_at + (int32_t)(incl - count);
    }
  }
}

// The first k of a segment's pairs (the whole segment, or the collected list; at most N), by
// rank: element e goes to position #{pairs before it} (the pairs are distinct, so the ranks
// are a permutation).  A workgroup ranks 64 elements; each of its sixteen waves counts over a
// sixteenth of the pairs, which it reads from LDS a pair at a time for all its lanes.
// Positions past the segment's length get index -1 and NaN.
template <int N>
__global__ __launch_bounds__(1024) void k_tk_rank(const double* __restrict__ chi2, int64_t seg_len, int32_t k,
                                                  int32_t cap, const TkState* __restrict__ st,
                                                  const uint64_t* __restrict__ keys,
                                                  const uint32_t* __restrict__ idx,
                                                  double* __restrict__ out_chi2, int64_t* __restrict__ out_idx) {
  __shared__ uint64_t lk[N];
  __shared__ uint32_t li[N];
  __shared__ uint32_t part[16][kWave];
  const int64_t seg = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = uniform(tid / kWave);
  const double* base = chi2 + seg * seg_len;
  const int m = st ? min(st[seg].taken, cap) : (int)seg_len;  // at most N
  for (int q = m + (int)blockIdx.x * 1024 + tid; q < k; q += (int)gridDim.x * 1024) {
    out_idx[seg * k + q] = -1;
    out_chi2[seg * k + q] = __longlong_as_double(0x7ff8000000000000ll);
  }
  const int e0 = blockIdx.x * kWave, e = e0 + lane;
  if (e0 >= m) return;  // uniform
  for (int q = tid; q < m; q += 1024) {
    lk[q] = st ? keys[seg * cap + q] : order_key(base[q]);
    li[q] = st ? idx[seg * cap + q] : (uint32_t)q;
  }
  __syncthreads();
  const uint64_t mk = e < m ? lk[e] : 0ull;
  const uint32_t mi = e < m ? li[e] : 0u;
  const int j1 = m * (wave + 1) / 16;
  uint32_t count = 0;
#pragma unroll 8
  for (int j = m * wave / 16; j < j1; ++j) count += before(lk[j], li[j], mk, mi) ? 1u : 0u;
  part[wave][lane] = count;
  __syncthreads();
  if (wave != 0 || e >= m) return;
  uint32_t rank = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) rank += part[w][lane];
  if (rank >= (uint32_t)k) return;
  const bool valid = (int64_t)mi < seg_len;
  out_idx[seg * k + rank] = valid ? (int64_t)mi : -1;
  out_chi2[seg * k + rank] = valid ? base[mi] : __longlong_as_double(0x7ff8000000000000ll);
}

// One workgroup of T a segment: its pairs (the whole segment, or the collected list; at most N)
// into LDS, a bitonic sort, the first k written.  Positions past the segment's length get
// index -1 and NaN.
template <int N, int T>
__global__ __launch_bounds__(T) void k_tk_sort(const double* __restrict__ chi2, int64_t seg_len, int32_t k,
                                               int32_t cap, const TkState* __restrict__ st,
                                               const uint64_t* __restrict__ keys,
                                               const uint32_t* __restrict__ idx,
                                               double* __restrict__ out_chi2, int64_t* __restrict__ out_idx) {
  __shared__ uint64_t lk[N];
  __shared__ uint32_t li[N];
  const int64_t seg = blockIdx.x;
  const int tid = threadIdx.x;
  const double* base = chi2 + seg * seg_len;
  const int m = st ? min(st[seg].taken, cap) : (int)seg_len;  // at most N
  int n = 2;
  while (n < m) n <<= 1;
  for (int q = tid; q < n; q += T) {
    const bool in = q < m;
    lk[q] = !in ? ~0ull : st ? keys[seg * cap + q] : order_key(base[q]);
    li[q] = !in ? 0xffffffffu : st ? idx[seg * cap + q] : (uint32_t)q;
  }
  __syncthreads();
  for (int size = 2; size <= n; size <<= 1)
    for (int j = size >> 1; j > 0; j >>= 1) {
      for (int p = tid; p < n / 2; p += T) {
        const int a = 2 * p - (p & (j - 1)), b = a + j;
        const uint64_t ka = lk[a], kb = lk[b];
        const uint32_t ia = li[a], ib = li[b];
        if (before(kb, ib, ka, ia) == ((a & size) == 0)) {
          lk[a] = kb;
          lk[b] = ka;
          li[a] = ib;
          li[b] = ia;
        }
      }
      __syncthreads();
    }
  for (int q = tid; q < k; q += T) {
    const bool valid = q < m && (int64_t)li[q] < seg_len;
    out_idx[seg * k + q] = valid ? (int64_t)li[q] : -1;
    out_chi2[seg * k + q] = valid ? base[li[q]] : __longlong_as_double(0x7ff8000000000000ll);
  }
}

// Top-k flat index -> (t0, u0, tE, alpha), event and map index.  axes != nullptr:
// product grid [u0 | alpha | t0 | tE]; else list rows (per event unless shared).
__global__ void k_candidates(const double* __restrict__ axes, int32_t nu, int32_t na, int32_t nt,
                             int32_t ne, const double* __restrict__ list, int32_t shared,
                             int64_t n_traj, int32_t n_events, int32_t n_maps, int32_t k,
                             const int64_t* __restrict__ idx, double* __restrict__ params,
                             int32_t* __restrict__ event, int32_t* __restrict__ mapidx) {
  const int64_t n = (int64_t)n_events * k;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t e = (int32_t)(i / k);
    int64_t f = idx[i];
    if (f < 0 || f >= (int64_t)n_maps * n_traj) f = 0;
    const int32_t m = (int32_t)(f / n_traj);
    const int64_t tj = f - (int64_t)m * n_traj;
    double* out = params + 4 * i;
    if (axes) {
      int64_t r = tj;
      const int ie = (int)(r % ne);
      r /= ne;
      const int it = (int)(r % nt);
      r /= nt;
      const int ia = (int)(r % na);
      const int iu = (int)(r / na);
      out[0] = axes[nu + na + it];
      out[1] = axes[iu];
      out[2] = axes[nu + na + nt + ie];
      out[3] = axes[nu + ia];
    } else {
      const double* p = list + 4 * ((shared ? 0 : (int64_t)e * n_traj) + tj);
      out[0] = p[0];
      out[1] = p[1];
      out[2] = p[2];
      out[3] = p[3];
    }
    event[i] = e;
    mapidx[i] = m;
  }
}

}  // namespace

hipError_t launch_candidates(const double* axes, int32_t nu, int32_t na, int32_t nt, int32_t ne,
                             const double* list, int32_t shared, int64_t n_traj, int32_t n_events,
                             int32_t n_maps, int32_t k, const int64_t* idx, double* params,
                             int32_t* event, int32_t* mapidx, hipStream_t st) {
  const int64_t n = (int64_t)n_events * k;
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_candidates, dim3((unsigned)blocks), dim3(256), 0, st, axes, nu, na, nt, ne,
                     list, shared, n_traj, n_events, n_maps, k, idx, params, event, mapidx);
  return hipGetLastError();
}

hipError_t launch_prep(PrepArgs a, const MapC* h_maps, hipStream_t st) {
  uint32_t most = 0;
  for (int32_t k = 0; k < a.n_maps; ++k) most = std::max(most, h_maps[k].cells);
  // a launch has fewer than 2^32 lanes; the parts stride over more than that
  auto blocks = [](uint64_t n, int64_t cap) { return (uint32_t)std::min<uint64_t>((n + 255) / 256, (uint64_t)cap); };
  a.event_blocks = (uint32_t)std::min(a.n_events, 1 << 20);
  a.traj_blocks = blocks((uint64_t)a.n, 65536);
  a.zero_blocks = blocks(a.n_zero, 4096);
  a.pack_blocks = std::max(1u, blocks(most, std::min<int64_t>(65536, (int64_t(1) << 23) / std::max(a.n_maps, 1))));
  const uint64_t all = (uint64_t)a.event_blocks + a.traj_blocks + a.zero_blocks + (uint64_t)a.pack_blocks * a.n_maps;
  if (all == 0) return hipSuccess;
  if (all >= 1u << 24) return hipErrorInvalidValue;
  // A few light curves are over soonest with one pass over memory (6 us for 8); where there is
  // enough of them, or of packing, to fill the chip, more wavefronts count: 24 maps of 1600^2
  // pixels 400 and 341 us, 200,000 light curves of 4 points 780 and 530
  uint64_t cells = 0;
  for (int32_t k = 0; k < a.n_maps; ++k) cells += h_maps[k].cells;
  if (cells < (1u << 22) && a.n_events <= 2048)
    hipLaunchKernelGGL(k_prep<16>, dim3((unsigned)all), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL(k_prep<0>, dim3((unsigned)all), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_put(void* dst, const void* src, size_t bytes, hipStream_t st) {
  if (bytes % 4) return hipErrorInvalidValue;
  for (size_t at = 0; at < bytes; at += sizeof(PutWords)) {
    PutWords v;
    const size_t n = std::min(bytes - at, sizeof(PutWords));
    std::memcpy(&v, (const char*)src + at, n);
    hipLaunchKernelGGL(k_put, dim3(1), dim3(256), 0, st, (uint32_t*)((char*)dst + at), (uint32_t)(n / 4), v);
  }
  return hipGetLastError();
}

hipError_t launch_traj_perm(const uint32_t* key, int64_t n_traj, int32_t n_lists, uint32_t* hist,
                            int32_t* perm, hipStream_t st) {
  const int64_t n = n_traj * n_lists, nb = (int64_t)n_lists * kPermBins;
  if (n <= 0) return hipSuccess;
  if (n > INT32_MAX || nb > kPermBinsMax) return hipErrorInvalidValue;
  return launch_bucket_order(key, n, (int32_t)nb, hist, perm, st);
}

hipError_t launch_search_plain(const TrajC* tc, int64_t n_traj, LcView lc, int32_t event,
                               int64_t n_points, MapC map, SearchOut out, int waves_per_block, hipStream_t st) {
  if (n_traj <= 0) return hipSuccess;
  const int threads = waves_per_block * kWave;
  int64_t blocks = (n_traj + waves_per_block - 1) / waves_per_block;
  if (blocks > 1 << 20) blocks = 1 << 20;
  // A launch reads its code anew, so that a few short light curves are over sooner with less of
  // it, though every chunk then takes the general form: 80 launches of 64 trajectories x 260
  // points 425 us (456 with the classification), x 500 513 (540), x 800 658 (658), x 1500 993 (948).
  const bool centred = map.sx == 0.0f && map.sy == 0.0f, is_short = n_points < kPlainShort;
  auto* kernel = is_short ? (centred ? k_search_plain<true, true> : k_search_plain<false, true>)
                          : (centred ? k_search_plain<true, false> : k_search_plain<false, false>);
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(threads), 0, st, tc, n_traj, lc, event, map, out);
  return hipGetLastError();
}

hipError_t launch_search_batched(BatchedArgs a, hipStream_t st) {
  if (a.waves_per_block < 1 || a.waves_per_block > 8 || a.n_traj <= 0) return hipErrorInvalidValue;
  const int64_t items = (int64_t)search_blocks((uint32_t)a.n_traj, a.traj_per_item, a.tu) * a.n_events * a.n_maps;
  const int64_t wgs = (items + a.waves_per_block - 1) / a.waves_per_block;
  // chunks of an eighth of one (map, event), so that all XCDs share every event evenly, 512
  // workgroups at most.  24 ragged events x 8 maps x 16384 trajectories: 8.75 ms at an eighth
  // (256), 10.6 at 32 (neighbours on different XCDs), 13.0 and 13.4 at 1024 and 4096 (an
  // event's parts on some XCDs only)
  const int64_t per = (search_blocks((uint32_t)a.n_traj, a.traj_per_item, a.tu) + a.waves_per_block - 1) / a.waves_per_block;
  a.chunk = (uint32_t)std::max<int64_t>(1, std::min<int64_t>(512, per / 8));
  // With chunks of an eighth an XCD would take the same directions of every event, whose cost
  // differs: it takes the next eighth with each deal.  20 events x 4 maps of 2048^2 x 32768
  // trajectories, 1000 points: 15.5 ms, 16.3 without; the ragged events above 8.5 and 8.6.  Events of
  // few workgroups rather find their cells again in the XCD's L2 (3000 trajectories, 300 points: 0.71
  // and 0.68); of many, every XCD has several parts of each.
  a.rotate = per >= 512 && per <= 4096 ? 1u : 0u;
  const int64_t deal = 8 * (int64_t)a.chunk;
  const int64_t blocks = (wgs + deal - 1) / deal * deal;
  if (blocks > INT32_MAX) return hipErrorInvalidValue;
  const dim3 block(a.waves_per_block * kWave);
  // a launch has fewer than 2^32 lanes: more workgroups take several, each of whole deals
  const int64_t most = (int64_t(1) << 31) / block.x / deal * deal;
  for (int64_t first = 0; first < blocks; first += most) {
    const dim3 grid((unsigned)std::min(most, blocks - first));
    a.first = (uint32_t)first;
    switch (a.tu * 2 + (a.centred ? 1 : 0)) {
      case 2: hipLaunchKernelGGL((k_search_batched<1, false>), grid, block, 0, st, a); break;
      case 3: hipLaunchKernelGGL((k_search_batched<1, true>), grid, block, 0, st, a); break;
      case 4: hipLaunchKernelGGL((k_search_batched<2, false>), grid, block, 0, st, a); break;
      case 5: hipLaunchKernelGGL((k_search_batched<2, true>), grid, block, 0, st, a); break;
      case 8: hipLaunchKernelGGL((k_search_batched<4, false>), grid, block, 0, st, a); break;
      case 9: hipLaunchKernelGGL((k_search_batched<4, true>), grid, block, 0, st, a); break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

namespace {
// Workgroups per segment: 1024 values each, about four a CU over all segments at most.
int64_t select_blocks(int64_t n_seg, int64_t seg_len, int num_cu) {
  const int64_t cap = std::max<int64_t>(1, std::min<int64_t>(TK_BINS, 4 * (int64_t)num_cu) / n_seg);
  return std::max<int64_t>(1, std::min((seg_len + 1023) / 1024, cap));
}
size_t al256(size_t b) { return (b + 255) & ~size_t(255); }
constexpr int64_t kRankSegs = 8;
int32_t tk_cap(int32_t k) { return std::min(std::max(2 * k, 512), TK_CAP); }
}  // namespace

SelectScratch select_scratch(int64_t n_best, int64_t best_len, int64_t n_seg, int64_t seg_len, int32_t k,
                             int num_cu) {
  SelectScratch s{};
  const int64_t p = n_best > 0 ? select_blocks(n_best, best_len, num_cu) : 1;
  const bool lists = k > 0 && seg_len > TK_CAP;
  // cleared: tickets of the best, then the states and histograms of the top-k
  s.tk_state = al256(p > 1 ? 4 * (size_t)n_best : 0);
  s.tk_hist = s.tk_state + (lists ? sizeof(TkState) * (size_t)n_seg : 0);
  s.zero_bytes = s.tk_hist + (lists ? 4 * (size_t)TK_BINS * n_seg : 0);
  s.part = al256(s.zero_bytes);
  s.tk_keys = s.part + al256(p > 1 ? sizeof(KeyIdx) * (size_t)(p * n_best) : 0);
  s.tk_idx = s.tk_keys + al256(lists ? 8 * (size_t)tk_cap(k) * n_seg : 0);
  s.bytes = s.tk_idx + al256(lists ? 4 * (size_t)tk_cap(k) * n_seg : 0);
  return s;
}

hipError_t launch_best(const double* chi2, int64_t n_seg, int64_t seg_len, double* best_chi2,
                       int64_t* best_idx, char* scratch, const SelectScratch& s, int num_cu,
                       hipStream_t st) {
  if (n_seg <= 0) return hipSuccess;
  if (seg_len <= 0) return hipErrorInvalidValue;
  const int64_t p = select_blocks(n_seg, seg_len, num_cu);
  for (int64_t s0 = 0; s0 < n_seg; s0 += 65535) {  // the grid's second dimension
    const int64_t n = std::min<int64_t>(65535, n_seg - s0);
    hipLaunchKernelGGL(k_best, dim3((unsigned)p, (unsigned)n), dim3(256), 0, st, chi2 + s0 * seg_len, seg_len,
                       (uint32_t*)scratch + s0, (KeyIdx*)(scratch + s.part) + s0 * p,
                       best_chi2 ? best_chi2 + s0 : nullptr, best_idx ? best_idx + s0 : nullptr);
  }
  return hipGetLastError();
}

hipError_t launch_topk(const double* chi2, int64_t n_seg, int64_t seg_len, int32_t k,
                       double* out_chi2, int64_t* out_idx, char* scratch, const SelectScratch& s,
                       int num_cu, hipStream_t st) {
  if (n_seg <= 0 || k <= 0) return hipSuccess;
  TkState* state = nullptr;
  uint64_t* keys = (uint64_t*)(scratch + s.tk_keys);
  uint32_t* idx = (uint32_t*)(scratch + s.tk_idx);
  const int32_t cap = tk_cap(k);
  int64_t sorted = seg_len;
  if (seg_len > TK_CAP) {
    state = (TkState*)(scratch + s.tk_state);
    uint32_t* hist = (uint32_t*)(scratch + s.tk_hist);
    const dim3 grid((unsigned)select_blocks(n_seg, seg_len, num_cu), (unsigned)n_seg), block(TK_THREADS);
    for (int pass = 0; pass < TK_PASSES; ++pass)
      hipLaunchKernelGGL(k_tk_hist, grid, block, 0, st, chi2, seg_len, k, cap, state, hist, pass);
    hipLaunchKernelGGL(k_tk_ties, grid, block, 0, st, chi2, seg_len, state, hist);
    hipLaunchKernelGGL(k_tk_collect, grid, block, 0, st, chi2, seg_len, k, cap, state, hist, keys, idx);
    sorted = cap;
  }
  // Ranks take m^2 comparisons spread over the chip, the sort m log^2 m on one CU a segment:
  // 23 against 118 us for 8192 pairs of one segment, 7 against 18 for 1024; the sort takes as
  // long for a segment on every CU, the ranks' time grows with the segments.
  const dim3 ranks((unsigned)((sorted + kWave - 1) / kWave), (unsigned)n_seg);
  if (n_seg <= kRankSegs && sorted <= 1024)
    hipLaunchKernelGGL(k_tk_rank<1024>, ranks, dim3(1024), 0, st, chi2, seg_len, k, cap, state, keys, idx,
                       out_chi2, out_idx);
  else if (n_seg <= kRankSegs)
    hipLaunchKernelGGL(k_tk_rank<TK_CAP>, ranks, dim3(1024), 0, st, chi2, seg_len, k, cap, state, keys, idx,
                       out_chi2, out_idx);
  else if (sorted <= 1024)
    hipLaunchKernelGGL((k_tk_sort<1024, 512>), dim3((unsigned)n_seg), dim3(512), 0, st, chi2, seg_len, k, cap,
                       state, keys, idx, out_chi2, out_idx);
  else
    hipLaunchKernelGGL((k_tk_sort<TK_CAP, 1024>), dim3((unsigned)n_seg), dim3(1024), 0, st, chi2, seg_len, k,
                       cap, state, keys, idx, out_chi2, out_idx);
  return hipGetLastError();
}

}  // namespace morse
