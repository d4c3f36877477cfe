// Gradient refinement of search candidates on gfx950.
//
// Chi-square gradient.  The profiled chi-square (Eqs. 5-6 of McDougall & Albrow 2015;
// sec. 4.2 bilinear map sampling) has (F_s, F_b) at their exact minimisers, so by the
// envelope theorem d chi2/d theta = -2 F_s sum w r dA/d theta with r = F - F_s A - F_b.
// One 128-lane workgroup per candidate (two wavefronts over the points, so a few
// thousand candidates still fill the chip) samples each point once and accumulates in
// FP64 the normal-equation sums with, for the directions D below, sum w D, sum w b D
// and sum w (F - Fbar) D; the fit then gives (F_s, F_b) and the sums
//   Gx = sum w r dA/dzx,  Gy = sum w r dA/dzy,
//   Gxt = sum w r tau dA/dzx,  Gyt = sum w r tau dA/dzy,
//   Ga = sum w r (zx dA/dzy - zy dA/dzx),
// from which, with zeta = tau (ca, sa) + u0 (-sa, ca) and tau = (t - t0)/tE,
//   d/dt0 = -2 F_s (-(ca Gx + sa Gy)/tE),  d/du0 = -2 F_s (-sa Gx + ca Gy),
//   d/dtE = -2 F_s (-(ca Gxt + sa Gyt)/tE), d/dalpha = -2 F_s Ga.
// dA/dzeta: on the map, k (e0 + fy (e1 - e0), ax1 - ax0) from the bilinear cell;
// off the map, A(u) = (u^2+2)/(u sqrt(u^2+4)) gives dA/du = -8/(u^2 (u^2+4)^(3/2)).
//
// L-BFGS.  A candidate's rounds depend on no other candidate, so one workgroup runs all of
// them: the evaluation on both wavefronts, then the update of the state machine (accept on
// the Armijo test or backtrack; two-loop recursion for the next direction) on one lane, its
// state (binary32 variables p, FP64 history) in LDS.  Of a round of a 2000-point candidate,
// 20 of 35 thousand cycles are the evaluation, bound by FP64 issue; the rest is the update, a
// chain of some hundred dependent FP64 operations during which the CU's other nine
// workgroups evaluate.  A call of 51 rounds for 8192 candidates on 8 ragged events (2000
// points) takes 3.08 ms, 3.95 as two launches a round on the same card; 64 candidates 0.96.  Where there
// are many, a workgroup takes four and updates them side by side (see refine_by_four).
#include "internal.h"

namespace morse {

namespace {

__device__ __forceinline__ double dot4(const double* a, const double* b) {
  return ((a[0] * b[0] + a[1] * b[1]) + a[2] * b[2]) + a[3] * b[3];
}

// Sum of NV FP64 values over each wavefront in a fixed order (a reduce-scatter), left in
// s_part; their sum in wave order is the workgroup's, wave_sum of it.
template <int NV>
__device__ __forceinline__ void leave_partials(double (&v)[NV], double* s_part) {
  static_assert(kWave == 64 && NV <= 64, "reduce-scatter assumes 64-lane wavefronts");
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  int slot = 0;
  bool valid = true;
  reduce_scatter<NV>(v, lane, slot, valid);
  if (valid) s_part[wave * NV + slot] = v[0];
}

// One workgroup (GRAD_THREADS lanes over the points) per candidate; thread k takes the
// points k, k + GRAD_THREADS, k + 2 GRAD_THREADS, ... in increasing order.
#ifndef MORSE_GRAD_THREADS
#define MORSE_GRAD_THREADS 128
#endif
constexpr int GRAD_THREADS = MORSE_GRAD_THREADS;

template <int NV>
__device__ __forceinline__ double wave_sum(const double* s_part, int q) {
  double t = s_part[q];
  for (int k = 1; k < GRAD_THREADS / kWave; ++k) t += s_part[k * NV + q];
  return t;
}


// dA/dzeta of one sample: on the map from the bilinear cell, off the map from the
// point-source magnification.
__device__ __forceinline__ void sample_dA(const Sample& sm, double kx, double ky, double& dAx,
                                          double& dAy) {
  if (sm.on) {
    const double e0 = (double)sm.e0, e1 = (double)sm.e1;
    dAx = kx * (e0 + (double)sm.fy * (e1 - e0));
    dAy = ky * ((double)sm.ax1 - (double)sm.ax0);
  } else {
    // dA/dzeta = dA/du zeta/u = -8 zeta / (u^2 (u^2+4) sqrt(u^2 (u^2+4)))
    const double zx = (double)sm.zx, zy = (double)sm.zy;
    const double u2 = zx * zx + zy * zy;
    const double pp = u2 * (u2 + 4.0);
    const double f = -8.0 / (pp * sqrt(pp));
    dAx = f * zx;
    dAy = f * zy;
  }
}

// Number of derivative directions D (dA/dzx, dA/dzy, tau dA/dzx, tau dA/dzy,
// zx dA/dzy - zy dA/dzx) and of one-pass sums (3 fit sums + 3 per direction).
constexpr int kDirs = 5;
constexpr int kSums = 3 + 3 * kDirs;

// One pass: with b = A - 1, wFc = w (F - Fbar) and c0 = B1/S_w the residual is
// r = (F - Fbar) - F_s (b - c0), so for every direction D
//   sum w r D = P_D - F_s (Q_D - c0 R_D),  P_D = sum wFc D, Q_D = sum w b D, R_D = sum w D,
// and chi2 = V - F_s C (the search's one-pass fit).  When the fit is degenerate or that
// chi2 is flagged as cancellation-prone, a second pass sums w r^2 and w r D directly
// with the residual formed point by point.
//
// grad_sums: the first pass on the trajectory tc, by the whole workgroup; fit_sums, on one
// lane a candidate: the fit; direct_sums, by the workgroup: the second pass; form_gradient,
// on the lane: the gradient.
// A candidate's event and map, loaded once for all its rounds.
struct Target {
  MapC m;
  const float* t;
  const double *w, *wFc, *F;
  int32_t np;
  double t_ref;
};
__device__ __forceinline__ Target target_of(const GradArgs& a, int32_t e, int32_t mi) {
  Target z;
  z.m = uniform(a.maps[mi]);
  const int64_t p0 = uniform(a.lc.off[e]);
  z.np = (int32_t)(uniform(a.lc.off[e + 1]) - p0);
  z.t = a.lc.t + p0;
  z.w = a.lc.w + p0;
  z.wFc = a.lc.wFc + p0;
  z.F = a.lc.F + p0;
  z.t_ref = uniform(a.lc.t_ref[e]);
  return z;
}

__device__ __forceinline__ void grad_sums(const Target& z, const TrajC& tc, double* s_part) {
  const int tid = threadIdx.x;
  const MapC& m = z.m;
  const float iE = tc.iE, ca = tc.ca, sa = tc.sa, bx = tc.bx, by = tc.by;
  const float t0p = (float)(tc.t0 - z.t_ref);
  const int32_t np = z.np;
  const float* t = z.t;
  const double* w = z.w;
  const double* wFc = z.wFc;
  const double kx = (double)m.kx, ky = (double)m.ky;

  // acc: B1, B2, C, then (R_D, Q_D, P_D) per direction
  double acc[kSums];
#pragma unroll
  for (int q = 0; q < kSums; ++q) acc[q] = 0.0;
  // The point at time tl: tau and the source position are recomputed from tl (the
  // same operations as locate, so the same bits) rather than kept live across the
  // gathers, which keeps the kernel within 96 VGPRs: five wavefronts per SIMD.
  auto add_point = [&](const Loc& l, float tl, const Quad& v, double wi, double wfc) {
    float tr = tl;
    asm volatile("" : "+v"(tr));  // opaque copy: the compiler cannot reuse locate's values
    const float ltau = (tr - t0p) * iE;
    const float lzx = ltau * ca + bx, lzy = ltau * sa + by;
    const float e0 = v.e0, e1 = v.e1;
    const float ax0 = v.v00 + l.fx * e0, ax1 = v.v01 + l.fx * e1;
    float A = ax0 + l.fy * (ax1 - ax0);
    double dAx = kx * ((double)e0 + (double)l.fy * ((double)e1 - (double)e0));
    double dAy = ky * ((double)ax1 - (double)ax0);
    if (!l.on) {
      A = point_lens_A(lzx, lzy);
      // dA/dzeta = dA/du zeta/u = -8 zeta / (u^2 (u^2+4) sqrt(u^2 (u^2+4)))
      const double zx = (double)lzx, zy = (double)lzy;
      const double u2 = zx * zx + zy * zy;
      const double pp = u2 * (u2 + 4.0);
      const double f = -8.0 / (pp * sqrt(pp));
      dAx = f * zx;
      dAy = f * zy;
    }
    const double b = (double)A - 1.0;
    const double wb = wi * b;
    acc[0] += wb;
    acc[1] = fma(wb, b, acc[1]);
    acc[2] = fma(b, wfc, acc[2]);
    const double tau = (double)ltau;
    const double D[kDirs] = {dAx, dAy, dAx * tau, dAy * tau,
                             (double)lzx * dAy - (double)lzy * dAx};
#pragma unroll
    for (int k = 0; k < kDirs; ++k) {
      acc[3 + 3 * k] = fma(wi, D[k], acc[3 + 3 * k]);
      acc[4 + 3 * k] = fma(wb, D[k], acc[4 + 3 * k]);
      acc[5 + 3 * k] = fma(wfc, D[k], acc[5 + 3 * k]);
    }
  };
  // Software pipeline over two register sets (a, b), so that nothing is copied between
  // iterations: while one point is added, the cell and weights of the next point and
  // the time of the one after are in flight.  Loads past the end are clamped to the
  // last point and never added.
  constexpr int32_t STEP = GRAD_THREADS;
  auto idx = [&](int32_t j) -> uint32_t { return (uint32_t)(j < np ? j : np - 1); };
  float tla = ldg(t, idx(tid));
  Loc la = locate(m, tla, t0p, iE, ca, sa, bx, by);
  Quad va = ldq(m, la.q);
  double wa = ldg(w, idx(tid)), fa = ldg(wFc, idx(tid));
  float ta = ldg(t, idx(tid + STEP));
  for (int32_t i0 = tid; i0 < np; i0 += 2 * STEP) {
    // set b: point i0 + STEP (time ta); time of i0 + 2 STEP
    const float tb = ldg(t, idx(i0 + 2 * STEP));
    const float tlb = ta;
    const Loc lb = locate(m, ta, t0p, iE, ca, sa, bx, by);
    const Quad vb = ldq(m, lb.q);
    const double wb = ldg(w, idx(i0 + STEP)), fb = ldg(wFc, idx(i0 + STEP));
    add_point(la, tla, va, wa, fa);
    // set a: point i0 + 2 STEP (time tb); time of i0 + 3 STEP
    ta = ldg(t, idx(i0 + 3 * STEP));
    tla = tb;
    la = locate(m, tb, t0p, iE, ca, sa, bx, by);
    va = ldq(m, la.q);
    wa = ldg(w, idx(i0 + 2 * STEP));
    fa = ldg(wFc, idx(i0 + 2 * STEP));
    if (i0 + STEP < np) add_point(lb, tlb, vb, wb, fb);
  }
  leave_partials<kSums>(acc, s_part);
}

__device__ void fit_sums(int32_t np, double Sw, double Fbar, double V, const double* s_part, Eval& out) {
  const double B1 = wave_sum<kSums>(s_part, 0);
  const Fit fit = centred_fit(Sw, Fbar, V, B1, wave_sum<kSums>(s_part, 1), wave_sum<kSums>(s_part, 2),
                              fit_terms(np, GRAD_THREADS));
  out.Fs = fit.Fs;
  out.Fb = fit.Fb;
  out.chi2 = fit.chi2;
  out.direct = fit.degenerate || fit.recheck ? 1 : 0;
  const double c0 = B1 / Sw;
#pragma unroll
  for (int k = 0; k < kDirs; ++k)
    out.G[k] = wave_sum<kSums>(s_part, 5 + 3 * k) -
               out.Fs * (wave_sum<kSums>(s_part, 4 + 3 * k) - c0 * wave_sum<kSums>(s_part, 3 + 3 * k));
}

// Direct sums of w r^2 and w r D, Neumaier-compensated per thread.
__device__ __forceinline__ void direct_sums(const Target& z, const TrajC& tc, double Fs, double Fb,
                                            double* s_part) {
  const MapC& m = z.m;
  const float iE = tc.iE, ca = tc.ca, sa = tc.sa, bx = tc.bx, by = tc.by;
  const float t0p = (float)(tc.t0 - z.t_ref);
  const double kx = (double)m.kx, ky = (double)m.ky;
  double n2[1 + kDirs], n2c[1 + kDirs];
#pragma unroll
  for (int q = 0; q <= kDirs; ++q) n2[q] = n2c[q] = 0.0;
  for (int32_t i = threadIdx.x; i < z.np; i += GRAD_THREADS) {
    const uint32_t u = (uint32_t)i;
    const Sample sm = sample_full(m, ldg(z.t, u), t0p, iE, ca, sa, bx, by);
    const double A = (double)sm.A;
    const double r = ldg(z.F, u) - Fs * A - Fb;
    const double wr = ldg(z.w, u) * r;
    double dAx, dAy;
    sample_dA(sm, kx, ky, dAx, dAy);
    const double tau = (double)sm.tau;
    neumaier_add(n2[0], n2c[0], wr * r);
    neumaier_add(n2[1], n2c[1], wr * dAx);
    neumaier_add(n2[2], n2c[2], wr * dAy);
    neumaier_add(n2[3], n2c[3], (wr * dAx) * tau);
    neumaier_add(n2[4], n2c[4], (wr * dAy) * tau);
    neumaier_add(n2[5], n2c[5], wr * ((double)sm.zx * dAy - (double)sm.zy * dAx));
  }
#pragma unroll
  for (int q = 0; q <= kDirs; ++q) n2[q] += n2c[q];
  leave_partials<1 + kDirs>(n2, s_part);
}

__device__ void take_direct(const double* s_part, Eval& out) {
  out.chi2 = wave_sum<1 + kDirs>(s_part, 0);
#pragma unroll
  for (int k = 0; k < kDirs; ++k) out.G[k] = wave_sum<1 + kDirs>(s_part, 1 + k);
}

// kScaled: the parameters are the L-BFGS variables about an anchor of time scale tE_anchor
// and the gradient is with respect to them.
template <bool kScaled>
__device__ void form_gradient(const TrajC& tc, double tE, double tE_anchor, Eval& out) {
  const double c64 = (double)tc.ca, s64 = (double)tc.sa;
  const double k2 = -2.0 * out.Fs;
  out.g[0] = k2 * (-(c64 * out.G[0] + s64 * out.G[1]) / tE);
  out.g[1] = k2 * (-s64 * out.G[0] + c64 * out.G[1]);
  out.g[2] = k2 * (-(c64 * out.G[2] + s64 * out.G[3]) / tE);
  out.g[3] = k2 * out.G[4];
  if (kScaled) {
    out.g[0] = out.g[0] * tE_anchor;
    out.g[2] = out.g[2] * tE;
  }
}

__device__ __forceinline__ void eval_nan(Eval& out) {
  out.direct = 0;
  out.chi2 = out.Fs = out.Fb = __longlong_as_double(0x7ff8000000000000ll);
  for (int q = 0; q < 4; ++q) out.g[q] = out.chi2;
}

__device__ __forceinline__ bool in_range(const GradArgs& a, int32_t e, int32_t mi) {
  return e >= 0 && e < a.n_events && mi >= 0 && mi < a.n_maps;
}

// Trajectory constants of natural parameters (t0, u0, tE, alpha), FP64 trigonometry
// rounded once.
__device__ __forceinline__ TrajC natural_traj(double t0, double u0, double tE, double al) {
  double sn, cs;
  sincos(al, &sn, &cs);
  TrajC r;
  r.t0 = t0;
  r.iE = (float)(1.0 / tE);
  r.ca = (float)cs;
  r.sa = (float)sn;
  r.bx = (float)(-u0 * sn);
  r.by = (float)(u0 * cs);
  r.pad = 0.0f;
  return r;
}

// Workgroups are dispatched to the 8 XCDs in turn (the grid is a multiple of 8), so
// slot s runs on XCD s % 8.  With an evaluation order, slot s takes the s-th candidate of
// it: the longest light curves start first, so that none ends long after the others, and
// the XCDs work through the same map at the same time.  (Chunks of 64 to 1024 neighbours a
// XCD: 3 to 40% slower, the lengths then differ over the XCDs.)  Without one, XCD x takes the contiguous
// candidate range [x per, (x + 1) per), so that neighbouring candidates (similar
// trajectories after a ranked selection) share its L2.
// kConsts: the trajectory constants come from a.tc, and the kernel fits 96 VGPRs (five wavefronts
// per SIMD).  Without, they are formed here, by a chain of FP64 operations on one lane before the
// first load of a cell, for which the compiler spills at 96 and gets 128: a few candidates, which
// leave the chip part empty, are over sooner so than with another launch.  A call for 100,000
// candidates on 4 maps of 2048^2, formed here with the spills and from a.tc: 20 events of 300 points
// 935 and 709 us, of 3000 points 1620 and 1399; for 1500 candidates (128 VGPRs, no a.tc) 160 and 143.
template <bool kConsts>
__global__ __launch_bounds__(GRAD_THREADS) __attribute__((amdgpu_waves_per_eu(kConsts ? 5 : 4))) void k_chi2_grad(GradArgs a) {
  __shared__ double s_part[GRAD_THREADS / kWave * kSums];
  __shared__ TrajC s_tc;
  __shared__ Eval ev;
  const int64_t per = (a.n + 7) / 8;
  for (int64_t slot = blockIdx.x; slot < 8 * per; slot += gridDim.x) {
    const int64_t pos = a.order ? slot : (slot % 8) * per + slot / 8;
    if (pos >= a.n) continue;
    const int64_t c = a.order ? (int64_t)uniform(a.order[pos]) : pos;
    const int32_t e = uniform(a.event[c]), mi = uniform(a.mapidx[c]);
    const double* p = a.params + 4 * c;
    __syncthreads();  // the last candidate's constants, sums and results have been read
    if (in_range(a, e, mi)) {  // uniform
      if (!kConsts) {
        if (threadIdx.x == 0) s_tc = natural_traj(p[0], p[1], p[2], p[3]);
        __syncthreads();
      }
      const TrajC tc = kConsts ? uniform(a.tc[c]) : uniform(s_tc);
      const Target z = target_of(a, e, mi);
      grad_sums(z, tc, s_part);
      __syncthreads();
      if (threadIdx.x == 0) fit_sums(z.np, a.lc.sums[3 * e], a.lc.sums[3 * e + 1], a.lc.sums[3 * e + 2], s_part, ev);
      __syncthreads();
      if (uniform(ev.direct)) {
        direct_sums(z, tc, uniform(ev.Fs), uniform(ev.Fb), s_part);
        __syncthreads();
        if (threadIdx.x == 0) take_direct(s_part, ev);
      }
      if (threadIdx.x == 0) form_gradient<false>(tc, p[2], 0.0, ev);
    } else if (threadIdx.x == 0) {
      eval_nan(ev);
    }
    if (threadIdx.x == 0) {
      if (a.chi2) a.chi2[c] = ev.chi2;
      if (a.grad)
        for (int q = 0; q < 4; ++q) a.grad[4 * c + q] = ev.g[q];
      if (a.fs) a.fs[c] = ev.Fs;
      if (a.fb) a.fb[c] = ev.Fb;
    }
  }
}

// New search direction at the accepted point (q.p, q.g) and the first trial along it; stops
// the candidate when the trial would not move it.  A pair is loaded while the one before it
// is worked on: the two loops are one chain of dependent operations.
__device__ void new_direction(RefineState& q, int m) {
  using Pair = RefineState::Pair;
  const int nh = q.nh;
  double r[4], d[4], qq[4];
  for (int k = 0; k < 4; ++k) qq[k] = q.g[k];
  double gamma;
  if (nh > 0) {
    const int last = q.head + nh - 1 < m ? q.head + nh - 1 : q.head + nh - 1 - m;  // the newest
    int i = last;
    Pair z = q.pair[i];
    gamma = dot4(z.s, z.y) / dot4(z.y, z.y);
#pragma unroll 2
    for (int h = nh; h > 0; --h) {
      const int j = i > 0 ? i - 1 : m - 1;
      const Pair next = q.pair[j];
      const double a = z.r * dot4(z.s, qq);
      q.pair[i].alph = a;
      for (int k = 0; k < 4; ++k) qq[k] = qq[k] - a * z.y[k];
      z = next;
      i = j;
    }
    i = q.head;
    z = q.pair[i];
    for (int k = 0; k < 4; ++k) r[k] = gamma * qq[k];
#pragma unroll 2
    for (int h = nh; h > 0; --h) {
      i = i + 1 < m ? i + 1 : 0;
      const Pair next = q.pair[i];
      const double b = z.r * dot4(z.y, r);
      for (int k = 0; k < 4; ++k) r[k] = r[k] + z.s[k] * (z.alph - b);
      z = next;
    }
  } else {
    const double gn = sqrt(dot4(q.g, q.g));
    gamma = gn > 0.0 ? 1e-2 / gn : 0.0;
    for (int k = 0; k < 4; ++k) r[k] = gamma * qq[k];
  }
  for (int k = 0; k < 4; ++k) d[k] = -r[k];
  const double gd = dot4(q.g, d);
  bool finite = true;
  for (int k = 0; k < 4; ++k) finite = finite && isfinite(d[k]);
  if (!(gd < 0.0) || !finite) {
    q.nh = 0;
    const double gn = sqrt(dot4(q.g, q.g));
    gamma = gn > 0.0 ? 1e-2 / gn : 0.0;
    for (int k = 0; k < 4; ++k) d[k] = -(gamma * q.g[k]);
  }
  q.step = 1.0;
  q.nls = 0;
  bool moved = false;
  for (int k = 0; k < 4; ++k) {
    q.d[k] = d[k];
    const float v = (float)((double)q.p[k] + 1.0 * d[k]);
    q.pt[k] = v;
    moved = moved || (v != q.p[k]);
  }
  if (!moved) q.active = 0;
}

// Whether sy > 1e-12 |s| |y|, from the squares ss and yy.  Far from the bound, and with no
// square out of range, the squares decide.
__device__ __forceinline__ bool curved(double sy, double ss, double yy) {
  const double p = ss * yy;
  if (sy > 1e-140 && p < 1e290 && sy * sy > 1e-23 * p) return true;
  return sy > 1e-12 * sqrt(ss) * sqrt(yy);
}

// One update of the state machine given the evaluation (ft, gt) at the trial point; the next
// trial point is then q.pt, unless the candidate was stopped.
__device__ void lbfgs_step(RefineState& q, const RefineArgs& s, bool first, double ft, const double* gt) {
  const int m = s.m;
  if (first) {
    q.nh = q.head = 0;
  } else {
    const double gd = dot4(q.g, q.d);
    const double t = q.step;
    if (!(isfinite(ft) && ft <= q.f + (s.c1 * t) * gd)) {
      q.nls += 1;
      if (q.nls >= s.max_ls) {
        q.active = 0;
        return;
      }
      const double tn = t * s.shrink;
      q.step = tn;
      for (int k = 0; k < 4; ++k) q.pt[k] = (float)((double)q.p[k] + tn * q.d[k]);
      return;
    }
    double sv[4], yv[4];
    for (int k = 0; k < 4; ++k) {
      sv[k] = (double)q.pt[k] - (double)q.p[k];
      yv[k] = gt[k] - q.g[k];
    }
    const double sy = dot4(sv, yv);
    if (curved(sy, dot4(sv, sv), dot4(yv, yv))) {
      const double rho = 1.0 / sy;
      if (q.nh == m) {  // full: drop the oldest pair
        q.head = q.head + 1 < m ? q.head + 1 : 0;
        q.nh = m - 1;
      }
      const int i = q.head + q.nh < m ? q.head + q.nh : q.head + q.nh - m;
      for (int k = 0; k < 4; ++k) {
        q.pair[i].s[k] = sv[k];
        q.pair[i].y[k] = yv[k];
      }
      q.pair[i].r = rho;
      q.nh += 1;
    }
  }
  for (int k = 0; k < 4; ++k) {
    q.p[k] = q.pt[k];
    q.g[k] = gt[k];
  }
  q.f = ft;
  new_direction(q, m);
}

// Natural parameters of the displacement p from the anchor.
__device__ __forceinline__ void natural(const RefineState& q, const float* p, double (&v)[4]) {
  v[0] = q.an[0] + (double)p[0] * q.an[2];
  v[1] = q.an[1] + (double)p[1];
  v[2] = q.an[2] * exp((double)p[2]);
  v[3] = q.an[3] + (double)p[3];
}

// Rounds [s.r0, s.r1) of every candidate, K of them a workgroup (neighbours in the order): it
// evaluates one after the other, then K lanes fit and update them side by side.  The first
// launch starts them (anchor = the candidate's row, p = 0, empty history), the one that ends
// with the last round writes them back; between launches their state is kept in s.state.
template <int K>
__global__ __launch_bounds__(GRAD_THREADS) __attribute__((amdgpu_waves_per_eu(5))) void k_refine(GradArgs a,
                                                                                            RefineArgs s) {
  __shared__ double s_part[K][GRAD_THREADS / kWave * kSums];
  __shared__ RefineState q[K];
  __shared__ int64_t s_c[K];
  constexpr int kWords = sizeof(RefineState) / 4;
  const int tid = threadIdx.x;
  const int64_t groups = (a.n + K - 1) / K, per = (groups + 7) / 8;
  for (int64_t slot = blockIdx.x; slot < 8 * per; slot += gridDim.x) {
    const int64_t group = a.order ? slot : (slot % 8) * per + slot / 8;
    if (group >= groups) continue;
    const int nk = (int)min((int64_t)K, a.n - group * K);
    __syncthreads();  // the last candidates are done with the state
    if (tid < nk) {
      const int64_t pos = group * K + tid;
      s_c[tid] = a.order ? (int64_t)a.order[pos] : pos;
    }
    __syncthreads();
    if (s.r0 > 0) {
      for (int k = 0; k < nk; ++k)
        for (int i = tid; i < kWords; i += GRAD_THREADS)
          ((uint32_t*)&q[k])[i] = ((const uint32_t*)(s.state + s_c[k]))[i];
    } else if (tid < nk) {
      RefineState& z = q[tid];
      for (int k = 0; k < 4; ++k) {
        z.an[k] = s.params[4 * s_c[tid] + k];
        z.p[k] = z.pt[k] = 0.0f;
      }
      z.nls = 0;
      z.active = 1;
    }
    // a lone candidate's event and map are loaded once for all its rounds
    const int64_t c0 = uniform(s_c[0]);
    const int32_t e0 = uniform(a.event[c0]), m0 = uniform(a.mapidx[c0]);
    const bool valid0 = in_range(a, e0, m0);
    const Target z0 = target_of(a, valid0 ? e0 : 0, valid0 ? m0 : 0);
    const double* sums0 = a.lc.sums + 3 * (valid0 ? e0 : 0);
    const double Sw0 = uniform(sums0[0]), Fbar0 = uniform(sums0[1]), V0 = uniform(sums0[2]);
    for (int32_t round = s.r0; round < s.r1; ++round) {
      __syncthreads();
      bool live = false;
      for (int k = 0; k < nk; ++k) live = live || uniform(q[k].active) != 0;
      if (!live) break;
      // the trials' constants (natural_traj of natural), half on each wavefront
      if (tid < nk) {
        RefineState& z = q[tid];
        const double tE = z.an[2] * exp((double)z.pt[2]);
        z.tc.t0 = z.an[0] + (double)z.pt[0] * z.an[2];
        z.tc.iE = (float)(1.0 / tE);
        z.tE = tE;
      } else if (tid >= kWave && tid < kWave + nk) {
        RefineState& z = q[tid - kWave];
        const double u0 = z.an[1] + (double)z.pt[1];
        double sn, cs;
        sincos(z.an[3] + (double)z.pt[3], &sn, &cs);
        z.tc.ca = (float)cs;
        z.tc.sa = (float)sn;
        z.tc.bx = (float)(-u0 * sn);
        z.tc.by = (float)(u0 * cs);
      }
      __syncthreads();
      if constexpr (K == 1) {
        if (valid0) grad_sums(z0, uniform(q[0].tc), s_part[0]);
      } else {
#pragma unroll 1
        for (int k = 0; k < nk; ++k) {
          const int64_t c = uniform(s_c[k]);
          const int32_t e = uniform(a.event[c]), mi = uniform(a.mapidx[c]);
          if (uniform(q[k].active) && in_range(a, e, mi)) grad_sums(target_of(a, e, mi), uniform(q[k].tc), s_part[k]);
        }
      }
      __syncthreads();
      if (K == 1 && tid == 0) {
        if (valid0)
          fit_sums(z0.np, Sw0, Fbar0, V0, s_part[0], q[0].ev);
        else
          eval_nan(q[0].ev);
      }
      if (K > 1 && tid < nk && q[tid].active) {
        const int32_t e = a.event[s_c[tid]];
        if (in_range(a, e, a.mapidx[s_c[tid]]))
          fit_sums((int32_t)(a.lc.off[e + 1] - a.lc.off[e]), a.lc.sums[3 * e], a.lc.sums[3 * e + 1],
                   a.lc.sums[3 * e + 2], s_part[tid], q[tid].ev);
        else
          eval_nan(q[tid].ev);
      }
      __syncthreads();
#pragma unroll 1
      for (int k = 0; k < nk; ++k)
        if (uniform(q[k].active) && uniform(q[k].ev.direct)) {
          const int64_t c = uniform(s_c[k]);
          direct_sums(target_of(a, uniform(a.event[c]), uniform(a.mapidx[c])), uniform(q[k].tc),
                      uniform(q[k].ev.Fs), uniform(q[k].ev.Fb), s_part[k]);
          __syncthreads();
          if (tid == k) take_direct(s_part[k], q[k].ev);
        }
      if (tid < nk && q[tid].active) {
        RefineState& z = q[tid];
        const int64_t c = s_c[tid];
        if (in_range(a, a.event[c], a.mapidx[c])) form_gradient<true>(z.tc, z.tE, z.an[2], z.ev);
        if (round == 0 && s.chi2_init) s.chi2_init[c] = z.ev.chi2;
        lbfgs_step(z, s, round == 0, z.ev.chi2, z.ev.g);
      }
    }
    __syncthreads();
    if (s.r1 <= s.steps) {
      for (int k = 0; k < nk; ++k)
        for (int i = tid; i < kWords; i += GRAD_THREADS)
          ((uint32_t*)(s.state + s_c[k]))[i] = ((const uint32_t*)&q[k])[i];
    } else if (tid < nk) {
      const RefineState& z = q[tid];
      double v[4];
      natural(z, z.p, v);
      for (int k = 0; k < 4; ++k) s.params[4 * s_c[tid] + k] = v[k];
      s.chi2_out[s_c[tid]] = z.f;
    }
  }
}

// The same rounds as launches of their own, for many candidates on maps larger than the
// last-level cache (see refine_by_round): start; evaluation, a workgroup per candidate, and
// update, a thread per candidate, in turn; write-back.  The state is s.state throughout.
__device__ __forceinline__ void next_trial(RefineState& z) {
  double v[4];
  natural(z, z.pt, v);
  z.tc = natural_traj(v[0], v[1], v[2], v[3]);
  z.tE = v[2];
}

__global__ __launch_bounds__(64) void k_round_start(RefineArgs s, int64_t n) {
  const int64_t c = blockIdx.x * (int64_t)64 + threadIdx.x;
  if (c >= n) return;
  RefineState& z = s.state[c];
  for (int k = 0; k < 4; ++k) {
    z.an[k] = s.params[4 * c + k];
    z.p[k] = z.pt[k] = 0.0f;
  }
  z.nls = 0;
  z.active = 1;
  next_trial(z);
}

__global__ __launch_bounds__(GRAD_THREADS) __attribute__((amdgpu_waves_per_eu(5))) void k_round_eval(GradArgs a,
                                                                                                RefineArgs s) {
  __shared__ double s_part[GRAD_THREADS / kWave * kSums];
  __shared__ Eval ev;
  const int64_t per = (a.n + 7) / 8;
  for (int64_t slot = blockIdx.x; slot < 8 * per; slot += gridDim.x) {
    const int64_t pos = a.order ? slot : (slot % 8) * per + slot / 8;
    if (pos >= a.n) continue;
    const int64_t c = a.order ? (int64_t)uniform(a.order[pos]) : pos;
    RefineState* q = s.state + c;
    if (!uniform(q->active)) continue;
    const int32_t e = uniform(a.event[c]), mi = uniform(a.mapidx[c]);
    __syncthreads();  // the last candidate's sums have been read
    if (in_range(a, e, mi)) {  // uniform
      const TrajC tc = uniform(q->tc);
      const Target z = target_of(a, e, mi);
      grad_sums(z, tc, s_part);
      __syncthreads();
      if (threadIdx.x == 0) fit_sums(z.np, a.lc.sums[3 * e], a.lc.sums[3 * e + 1], a.lc.sums[3 * e + 2], s_part, ev);
      __syncthreads();
      if (uniform(ev.direct)) {
        direct_sums(z, tc, uniform(ev.Fs), uniform(ev.Fb), s_part);
        __syncthreads();
        if (threadIdx.x == 0) take_direct(s_part, ev);
      }
      if (threadIdx.x == 0) form_gradient<true>(tc, q->tE, q->an[2], ev);
    } else if (threadIdx.x == 0) {
      eval_nan(ev);
    }
    if (threadIdx.x == 0) {
      q->ev.chi2 = ev.chi2;
      for (int k = 0; k < 4; ++k) q->ev.g[k] = ev.g[k];
    }
  }
}

__global__ __launch_bounds__(64) void k_round_update(RefineArgs s, int64_t n, int32_t round) {
  const int64_t c = blockIdx.x * (int64_t)64 + threadIdx.x;
  if (c >= n) return;
  RefineState& z = s.state[c];
  if (z.active) {
    double g[4];
    for (int k = 0; k < 4; ++k) g[k] = z.ev.g[k];
    if (round == 0 && s.chi2_init) s.chi2_init[c] = z.ev.chi2;
    lbfgs_step(z, s, round == 0, z.ev.chi2, g);
    if (z.active) next_trial(z);
  }
  if (round == s.steps) {
    double v[4];
    natural(z, z.p, v);
    for (int k = 0; k < 4; ++k) s.params[4 * c + k] = v[k];
    s.chi2_out[c] = z.f;
  }
}

}  // namespace

namespace {

// Evaluation order: each candidate's key, then the shared bucket sort.  Keys go by event, the
// longest light curves first, then by map; by map first where the maps do not all fit the
// last-level cache (see launch_cand_order); with many events, by map, then event.
__device__ __forceinline__ uint32_t order_key(const GradArgs& a, int64_t c, bool by_event) {
  const int32_t e = a.event[c], m = a.mapidx[c];
  if (e < 0 || e >= a.n_events || m < 0 || m >= a.n_maps) return 0u;  // NaN outputs anyway
  if (!by_event) return (uint32_t)m;
  if (a.n_events > kRankedEvents) return (uint32_t)m * (uint32_t)a.n_events + (uint32_t)e;
  const int64_t len = a.lc.off[e + 1] - a.lc.off[e];
  uint32_t rank = 0;
  for (int32_t k = 0; k < a.n_events; ++k) {
    const int64_t lk = a.lc.off[k + 1] - a.lc.off[k];
    rank += lk > len || (lk == len && k < e) ? 1u : 0u;
  }
  return a.map_first ? (uint32_t)m * (uint32_t)a.n_events + rank : rank * (uint32_t)a.n_maps + (uint32_t)m;
}

__global__ void k_order_keys(GradArgs a, bool by_event, uint32_t* key) {
  for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < a.n;
       c += (int64_t)gridDim.x * blockDim.x) {
    key[c] = order_key(a, c, by_event);
    if (a.tc) {
      const double* p = a.params + 4 * c;
      a.tc[c] = natural_traj(p[0], p[1], p[2], p[3]);
    }
  }
}

}  // namespace

bool maps_exceed_cache(const MapC* h_maps, int32_t n_maps) {
  uint64_t bytes = 0;
  for (int32_t k = 0; k < n_maps; ++k) bytes += (uint64_t)h_maps[k].cells * sizeof(Quad);
  return bytes > (uint64_t(256) << 20);
}

hipError_t launch_cand_order(GradArgs a, const MapC* h_maps, uint32_t* key, uint32_t* hist, int32_t* order,
                             hipStream_t st) {
  // 8192 candidates of 8 events on 8 maps of 16 MiB: 3.0 ms with the longest event first, 3.4 in
  // the order of the maps; on 64 maps of 64 MiB the events first sample 40 maps at a time.
  a.map_first = maps_exceed_cache(h_maps, a.n_maps) ? 1 : 0;
  if (a.n <= 0) return hipSuccess;
  if (a.n > INT32_MAX || a.n_maps <= 0 || a.n_events <= 0) return hipErrorInvalidValue;
  const int64_t nb = order_bins(a.n_maps, a.n_events);
  const bool by_event = nb == (int64_t)a.n_maps * a.n_events;
  int64_t blocks = (a.n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_order_keys, dim3((unsigned)blocks), dim3(256), 0, st, a, by_event, key);
  return launch_bucket_order(key, a.n, (int32_t)nb, hist, order, st);
}

namespace {
unsigned candidate_blocks(int64_t n) { return (unsigned)std::min<int64_t>(8 * ((n + 7) / 8), 1 << 20); }
}  // namespace

hipError_t launch_chi2_grad(const GradArgs& a, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(a.tc ? k_chi2_grad<true> : k_chi2_grad<false>, dim3(candidate_blocks(a.n)), dim3(GRAD_THREADS),
                     0, st, a);
  return hipGetLastError();
}

hipError_t launch_round_start(const GradArgs& a, const RefineArgs& s, hipStream_t st) {
  if (s.m < 1 || s.m > kMaxHistory) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_round_start, dim3((unsigned)((a.n + 63) / 64)), dim3(64), 0, st, s, a.n);
  return hipGetLastError();
}

hipError_t launch_round_eval(const GradArgs& a, const RefineArgs& s, hipStream_t st) {
  hipLaunchKernelGGL(k_round_eval, dim3(candidate_blocks(a.n)), dim3(GRAD_THREADS), 0, st, a, s);
  return hipGetLastError();
}

hipError_t launch_round_update(const GradArgs& a, const RefineArgs& s, int32_t round, hipStream_t st) {
  hipLaunchKernelGGL(k_round_update, dim3((unsigned)((a.n + 63) / 64)), dim3(64), 0, st, s, a.n, round);
  return hipGetLastError();
}

hipError_t launch_refine(const GradArgs& a, const RefineArgs& s, bool four, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  if (s.m < 1 || s.m > kMaxHistory) return hipErrorInvalidValue;
  if (four)
    hipLaunchKernelGGL(k_refine<4>, dim3(candidate_blocks((a.n + 3) / 4)), dim3(GRAD_THREADS), 0, st, a, s);
  else
    hipLaunchKernelGGL(k_refine<1>, dim3(candidate_blocks(a.n)), dim3(GRAD_THREADS), 0, st, a, s);
  return hipGetLastError();
}

}  // namespace morse
