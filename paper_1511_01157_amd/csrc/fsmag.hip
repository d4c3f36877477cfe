// Finite-source magnification by image-centred ray shooting on gfx950 (sec. 5 of
// McDougall & Albrow 2015: point source beyond 10 rho from the caustic, otherwise polar
// grids grown around the source's images and integrated with the source profile).
//
// Classification, one wavefront per source: the distance from the source centre to the
// nearest caustic point; far sources take the point-source magnification of their
// images (Eqs. 3-4, one thread each), near ones are listed.  Regions, one 256-lane
// workgroup per listed source: every lane solves the lens equation for one of the
// centre and n_b boundary points (the quintic of Eq. 2, FP64 Aberth-Ehrlich), the
// images and the critical points whose caustic image lies inside the source become
// seeds in polar coordinates about the centre of mass; the seeds are sorted in LDS
// (bitonic), cut into angular runs at gaps wider than `gap` and each run at radial
// gaps; every region grows until none of its sides maps inside the source (side samples
// spread over the lanes); overlapping regions merge.  Integration, one 256-lane
// workgroup per (source, region): the region is cut to its inside cells, up to n_shrink times,
// by its nodes alone, then integrated once, column by column (one lane per theta
// column, radial segments with the limb crossing linear in f = rho^2 - |zeta - zeta_s|^2 and the
// square-root edge of the limb-darkened profile integrated exactly); a last kernel adds each
// source's region integrals in region order.  All arithmetic is FP64.

#include "fsmag.h"

#include <climits>

namespace morse {

namespace {

constexpr int kFsThreads = 256;
constexpr int kSeedCap = 2048;   // seeds per source (a power of two for the sort)
constexpr int kRegionCap = kFsRegionCap;
constexpr int kCritSeeds = 512;  // critical-point seeds at most

__global__ void k_fill_u32_fs(uint32_t* p) {
  if (threadIdx.x == 0) *p = 0u;
}

struct cd {
  double x, y;
};
__device__ __forceinline__ cd cadd(cd a, cd b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cd csub(cd a, cd b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ cd cmul(cd a, cd b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ __forceinline__ cd cscale(cd a, double s) { return {a.x * s, a.y * s}; }
__device__ __forceinline__ double cabs2(cd a) { return fma(a.x, a.x, a.y * a.y); }
// |a|, for numbers whose squares stay in the FP64 range (positions, steps, residuals; the
// square of a step below 1e-154 vanishes, far under the last place of any root)
__device__ __forceinline__ double cabs(cd a) { return sqrt(cabs2(a)); }
// 1/x within one unit in the last place for |x| in [1e-300, 1e300] (0 and inf give NaN): the
// hardware's reciprocal and two Newton steps, 5 instructions for the 10 of an IEEE division
__device__ __forceinline__ double recip(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}
// a / b: directly as a conj(b) / |b|^2 while |b|^2 stays well inside the FP64 range,
// else scaled (Smith).
__device__ __forceinline__ cd cdivc(cd a, cd b) {
  const double n = b.x * b.x + b.y * b.y;
  if (n > 1e-280 && n < 1e280) {
    const double s = recip(n);
    return {(a.x * b.x + a.y * b.y) * s, (a.y * b.x - a.x * b.y) * s};
  }
  if (fabs(b.x) >= fabs(b.y)) {
    const double r = b.y / b.x, d = b.x + b.y * r;
    return {(a.x + a.y * r) / d, (a.y - a.x * r) / d};
  }
  const double r = b.x / b.y, d = b.x * r + b.y;
  return {(a.x * r + a.y) / d, (a.y * r - a.x) / d};
}
__device__ __forceinline__ cd crecip(cd b) { return cdivc(cd{1.0, 0.0}, b); }

struct Lens {
  double m1, m2, x1, x2;
};

// Eq. 2: zeta = z - m1/(conj z - x1) - m2/(conj z - x2).
__device__ __forceinline__ cd lens_eq(const Lens& L, cd z) {
  const cd w1 = {z.x - L.x1, -z.y}, w2 = {z.x - L.x2, -z.y};
  return csub(csub(z, cscale(crecip(w1), L.m1)), cscale(crecip(w2), L.m2));
}

// f = rho^2 - |zeta(z) - zs|^2 at z = r (cs, sn) by Eq. 2 (positive inside the source), each
// lens term written as m_k (z - x_k) / |z - x_k|^2, the conjugate's reciprocal; one
// reciprocal of |z - x1|^2 |z - x2|^2 serves both (the samples of the image-centred
// integration and the growth test; a sample on a lens gives NaN, which compares as outside).
__device__ __forceinline__ double source_f(const Lens& L, double r, double cs, double sn, cd zs, double rho2) {
  const double zy = r * sn, yy = zy * zy;
  const double d1 = fma(r, cs, -L.x1), d2 = fma(r, cs, -L.x2);
  const double r1 = fma(d1, d1, yy), r2 = fma(d2, d2, yy);
  const double y = recip(r1 * r2);
  const double a1 = (L.m1 * r2) * y, a2 = (L.m2 * r1) * y;
  const double ex = fma(-a2, d2, fma(-a1, d1, fma(r, cs, -zs.x)));
  const double ey = fma(-(a1 + a2), zy, zy - zs.y);
  return fma(-ex, ex, fma(-ey, ey, rho2));
}

// The quintic whose roots contain the images of zeta.  With Q = (z - x1)(z - x2) and
// P_k = (conj zeta - x_k) Q + m1 (z - x2) + m2 (z - x1) (so 1/(conj z - x_k) = Q/P_k on
// an image, from the conjugate of Eq. 2), Eq. 2 times P1 P2 reads
//   (z - zeta) P1 P2 - Q (m1 P2 + m2 P1) = 0.
// Coefficients ascending, a[0..5].
__device__ void quintic(const Lens& L, cd zeta, cd (&a)[6]) {
  const cd zb = {zeta.x, -zeta.y};
  const double q0 = L.x1 * L.x2, q1 = -(L.x1 + L.x2);  // Q = q0 + q1 z + z^2
  const double lin0 = -(L.m1 * L.x2 + L.m2 * L.x1), lin1 = L.m1 + L.m2;
  cd P1[3], P2[3];
  const cd c1 = {zb.x - L.x1, zb.y}, c2 = {zb.x - L.x2, zb.y};
  P1[0] = cadd(cscale(c1, q0), cd{lin0, 0.0});
  P1[1] = cadd(cscale(c1, q1), cd{lin1, 0.0});
  P1[2] = c1;
  P2[0] = cadd(cscale(c2, q0), cd{lin0, 0.0});
  P2[1] = cadd(cscale(c2, q1), cd{lin1, 0.0});
  P2[2] = c2;
  cd T[5] = {};
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) T[i + j] = cadd(T[i + j], cmul(P1[i], P2[j]));
  cd U[3];
  for (int i = 0; i < 3; ++i) U[i] = cadd(cscale(P2[i], L.m1), cscale(P1[i], L.m2));
  const double Q[3] = {q0, q1, 1.0};
  cd QU[5] = {};
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) QU[i + j] = cadd(QU[i + j], cscale(U[j], Q[i]));
  // (z - zeta) T
  a[0] = csub(cmul(cd{-zeta.x, -zeta.y}, T[0]), QU[0]);
  for (int k = 1; k < 5; ++k) a[k] = csub(csub(T[k - 1], cmul(zeta, T[k])), QU[k]);
  a[5] = T[4];
}

__device__ __forceinline__ void poly_eval(const cd (&a)[6], cd z, cd& p, cd& dp) {
  p = a[5];
  dp = {0.0, 0.0};
  for (int k = 4; k >= 0; --k) {
    dp = cadd(cmul(dp, z), p);
    p = cadd(cmul(p, z), a[k]);
  }
}

// Roots of the quintic: Aberth-Ehrlich from a circle (Cauchy bound) until the largest
// relative step is below 1e-14 or, below 1e-9, stops halving (the rounding floor of
// the polynomial's evaluation, which ill-conditioned roots never get under), then two
// Newton steps per root.
__device__ void quintic_roots(const cd (&a)[6], cd (&z)[5]) {
  const cd inv5 = crecip(a[5]);
  double rad = 0.0;
  for (int i = 0; i < 5; ++i) {  // hypot: a source beside a lens has a tiny a[5]
    const cd c = cmul(a[i], inv5);
    rad = fmax(rad, hypot(c.x, c.y));
  }
  rad = 1.0 + rad;
  for (int k = 0; k < 5; ++k) {
    double sn, cs;
    sincos(0.4 + 2.0 * M_PI * k / 5.0, &sn, &cs);
    z[k] = {rad * cs, rad * sn};
  }
  double prev = __builtin_inf();
  for (int it = 0; it < 200; ++it) {
    double moved = 0.0;
    for (int k = 0; k < 5; ++k) {
      cd p, dp;
      poly_eval(a, z[k], p, dp);
      if (p.x == 0.0 && p.y == 0.0) continue;
      const cd ratio = cdivc(p, dp);
      cd rep = {0.0, 0.0};
      for (int j = 0; j < 5; ++j)
        if (j != k) rep = cadd(rep, crecip(csub(z[k], z[j])));
      const cd step = cdivc(ratio, csub(cd{1.0, 0.0}, cmul(ratio, rep)));
      if (!(isfinite(step.x) && isfinite(step.y))) continue;
      z[k] = csub(z[k], step);
      moved = fmax(moved, cabs(step) / (1.0 + cabs(z[k])));
    }
    if (moved < 1e-14 || (moved < 1e-9 && moved >= 0.5 * prev)) break;
    prev = moved;
  }
  for (int k = 0; k < 5; ++k)
    for (int it = 0; it < 2; ++it) {
      cd p, dp;
      poly_eval(a, z[k], p, dp);
      if (dp.x != 0.0 || dp.y != 0.0) z[k] = csub(z[k], cdivc(p, dp));
    }
}

// Images of zeta: the 5 roots when all satisfy Eq. 2 to 1e-6 (1 + |zeta|), else the 3
// with the smallest residuals (ties: the lower root index) when at least 3 do, else
// those that do.  sel[k] marks the images among the roots z[k]; returns their number.
// Written without indexing by a runtime value, so the arrays stay in registers.
__device__ __forceinline__ int images_of(const Lens& L, cd zeta, cd (&z)[5], bool (&sel)[5]) {
  cd a[6];
  quintic(L, zeta, a);
  quintic_roots(a, z);
  double res[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const double r = cabs(csub(lens_eq(L, z[k]), zeta));
    res[k] = isfinite(r) ? r : __builtin_inf();
  }
  const double tol = 1e-6 * (1.0 + cabs(zeta));
  int nvalid = 0;
#pragma unroll
  for (int k = 0; k < 5; ++k) nvalid += res[k] < tol ? 1 : 0;
  const int nimg = nvalid >= 5 ? 5 : (nvalid >= 3 ? 3 : nvalid);
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    int rank = 0;
#pragma unroll
    for (int j = 0; j < 5; ++j) rank += (res[j] < res[k] || (res[j] == res[k] && j < k)) ? 1 : 0;
    sel[k] = rank < nimg;
  }
  return nimg;
}

__device__ double point_source_A(const Lens& L, cd zeta) {
  cd z[5];
  bool sel[5];
  images_of(L, zeta, z, sel);
  double A = 0.0;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const cd w1 = {z[k].x - L.x1, -z[k].y}, w2 = {z[k].x - L.x2, -z[k].y};
    const cd g = cadd(cscale(crecip(cmul(w1, w1)), L.m1), cscale(crecip(cmul(w2, w2)), L.m2));
    A += sel[k] ? fabs(1.0 / (1.0 - cabs2(g))) : 0.0;
  }
  return A;
}

// Critical points at a.n_crit / 4 equally spaced phases phi and their caustic images: the
// roots of m1 (z - x2)^2 + m2 (z - x1)^2 = e^{-i phi} (z - x1)^2 (z - x2)^2, four lanes per
// phase, one root each.  Aberth-Ehrlich from a circle (all four steps at once, the roots
// exchanged by shuffles) under the quintic's stopping rule, then two Newton steps.  A phase
// that has converged keeps its roots while the wavefront's others go on, so its result
// does not depend on them.  Bound: latency, about a dozen rounds of a serial chain; 1024
// phases 17 us, for 100 ms of continuation from phase to phase on the host (whose 1e-16
// test ill-conditioned roots never met).
__global__ __launch_bounds__(64) void k_fs_crit(Lens L, int32_t nphi, double* __restrict__ crit,
                                                double* __restrict__ caus) {
  const int32_t t = blockIdx.x * 64 + threadIdx.x;
  const int32_t ph = min(t >> 2, nphi - 1), k = t & 3;  // padding lanes repeat the last phase
  double es, ec;
  sincos(2.0 * M_PI * ph / nphi, &es, &ec);
  const cd e = {ec, -es};
  const double S = L.x1 + L.x2, P = L.x1 * L.x2;
  const cd c0 = csub(cd{L.m1 * L.x2 * L.x2 + L.m2 * L.x1 * L.x1, 0.0}, cscale(e, P * P));
  const cd c1 = cadd(cd{-2.0 * (L.m1 * L.x2 + L.m2 * L.x1), 0.0}, cscale(e, 2.0 * S * P));
  const cd c2 = csub(cd{L.m1 + L.m2, 0.0}, cscale(e, S * S + 2.0 * P));
  const cd c3 = cscale(e, 2.0 * S), c4 = {-e.x, -e.y};
  auto eval = [&](cd z, cd& p, cd& dp) {
    p = c4;
    dp = {0.0, 0.0};
    for (const cd& c : {c3, c2, c1, c0}) {
      dp = cadd(cmul(dp, z), p);
      p = cadd(cmul(p, z), c);
    }
  };
  const double rad = 1.0 + fmax(fmax(cabs(c0), cabs(c1)), fmax(cabs(c2), cabs(c3)));  // |c4| = 1
  double sn, cs;
  sincos(0.4 + 0.5 * M_PI * k, &sn, &cs);
  cd z = {rad * cs, rad * sn};
  double prev = __builtin_inf();
  bool done = false;
  for (int it = 0; it < 200; ++it) {
    cd p, dp, rep = {0.0, 0.0};
    eval(z, p, dp);
    const cd ratio = cdivc(p, dp);
#pragma unroll
    for (int o = 1; o < 4; ++o) {
      const cd w = {__shfl_xor(z.x, o), __shfl_xor(z.y, o)};
      rep = cadd(rep, crecip(csub(z, w)));
    }
    const cd step = cdivc(ratio, csub(cd{1.0, 0.0}, cmul(ratio, rep)));
    const bool go = !done && !(p.x == 0.0 && p.y == 0.0) && isfinite(step.x) && isfinite(step.y);
    if (go) z = csub(z, step);
    double moved = go ? cabs(step) / (1.0 + cabs(z)) : 0.0;
    moved = fmax(moved, __shfl_xor(moved, 1));
    moved = fmax(moved, __shfl_xor(moved, 2));
    done = done || moved < 1e-14 || (moved < 1e-9 && moved >= 0.5 * prev);
    prev = moved;
    if (__builtin_amdgcn_ballot_w64(!done) == 0) break;
  }
  for (int it = 0; it < 2; ++it) {
    cd p, dp;
    eval(z, p, dp);
    if (dp.x != 0.0 || dp.y != 0.0) z = csub(z, cdivc(p, dp));
  }
  if (t >= 4 * nphi) return;
  const cd zeta = lens_eq(L, z);
  crit[2 * t] = z.x;
  crit[2 * t + 1] = z.y;
  caus[2 * t] = zeta.x;
  caus[2 * t + 1] = zeta.y;
}

// One wavefront per source: the lanes share the caustic points and a butterfly minimum
// gives the distance.  Far sources are marked for the point-source kernel, near ones
// listed for the image-centred kernel.
__global__ __launch_bounds__(256) void k_fs_classify(FsArgs a) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
  for (int64_t i = blockIdx.x * (int64_t)(blockDim.x / kWave) + threadIdx.x / kWave; i < a.n;
       i += waves) {
    const cd zs = {a.zeta[2 * i], a.zeta[2 * i + 1]};
    double dmin = __builtin_inf();
    for (int32_t j = lane; j < a.n_crit; j += kWave) {
      const double d = cabs2(csub(cd{a.caus[2 * j], a.caus[2 * j + 1]}, zs));
      if (d < dmin) dmin = d;  // squares; NaN points (a massless companion) never win
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) dmin = fmin(dmin, __shfl_xor(dmin, off));
    if (lane == 0) {
      if (sqrt(dmin) > a.near * a.rho) {
        a.nreg[i] = -1;
      } else {
        a.nreg[i] = 0;
        const uint32_t slot = atomicAdd(a.near_count, 1u);
        a.near_list[slot] = (int32_t)i;
      }
    }
  }
}

// Point-source magnification of the sources marked far (one thread per source).
__global__ __launch_bounds__(256) void k_fs_point(FsArgs a) {
  const Lens L{a.m1, a.m2, a.x1, a.x2};
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= a.n || a.nreg[i] != -1) return;
  a.A[i] = point_source_A(L, cd{a.zeta[2 * i], a.zeta[2 * i + 1]});
}

// ---------------------------------------------------------------------------------
// Image-centred kernel.
struct Region {
  double r0, r1, t0, t1;
};

__device__ __forceinline__ bool is_ring(const Region& g) { return g.t1 - g.t0 >= 2.0 * M_PI; }

// Ascending bitonic sort of n = kSeedCap keys with a payload (all lanes).
__device__ void bitonic(double* key, double* v1, double* v2) {
  for (int k = 2; k <= kSeedCap; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < kSeedCap; i += kFsThreads) {
        const int l = i ^ j;
        if (l > i) {
          const bool up = (i & k) == 0;
          if ((key[i] > key[l]) == up) {
            double t = key[i];
            key[i] = key[l];
            key[l] = t;
            t = v1[i];
            v1[i] = v1[l];
            v1[l] = t;
            t = v2[i];
            v2[i] = v2[l];
            v2[l] = t;
          }
        }
      }
      __syncthreads();
    }
}

// numpy.linspace(a, b, n)[k]
__device__ __forceinline__ double linspace_at(double a, double b, int n, int k) {
  return k == n - 1 ? b : a + k * ((b - a) / (n - 1));
}

__device__ __forceinline__ bool theta_overlap(const Region& a, const Region& b) {
  if (is_ring(a) || is_ring(b)) return true;
  const double k = rint(((a.t0 + a.t1) - (b.t0 + b.t1)) / (4.0 * M_PI));
  const double b0 = b.t0 + 2.0 * M_PI * k, b1 = b.t1 + 2.0 * M_PI * k;
  return !(b1 < a.t0 || b0 > a.t1);
}

__device__ Region region_union(const Region& a, const Region& b) {
  Region u{fmin(a.r0, b.r0), fmax(a.r1, b.r1), -M_PI, M_PI};
  if (is_ring(a) || is_ring(b)) return u;
  const double k = rint(((a.t0 + a.t1) - (b.t0 + b.t1)) / (4.0 * M_PI));
  u.t0 = fmin(a.t0, b.t0 + 2.0 * M_PI * k);
  u.t1 = fmax(a.t1, b.t1 + 2.0 * M_PI * k);
  if (u.t1 - u.t0 >= 2.0 * M_PI) {
    u.t0 = -M_PI;
    u.t1 = M_PI;
  }
  return u;
}

constexpr int kPer = kSeedCap / kFsThreads;  // seeds per lane of the prefix counts

struct Shared {
  double key[kSeedCap], r[kSeedCap], th[kSeedCap];
  int run[kSeedCap];
  Region reg[kRegionCap];
  int ired[4][kFsThreads];
  int n_seed, n_reg, flag[4];
};

// Smallest v of the workgroup.
__device__ int block_min(int v, Shared& sh) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
  __syncthreads();
  if (threadIdx.x % kWave == 0) sh.ired[0][threadIdx.x / kWave] = v;
  __syncthreads();
  for (int w = 0; w < kFsThreads / kWave; ++w) v = min(v, sh.ired[0][w]);
  return v;
}

// Sum of v over the lanes before this one.
__device__ int block_prefix(int v, Shared& sh) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  int incl = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int l = __shfl_up(incl, o);
    if (lane >= o) incl += l;
  }
  __syncthreads();
  if (lane == kWave - 1) sh.ired[0][wave] = incl;
  __syncthreads();
  int before = incl - v;
  for (int w = 0; w < wave; ++w) before += sh.ired[0][w];
  return before;
}

// Range of (lo, hi) over the wavefront, on every lane.
__device__ __forceinline__ void wave_range(double& lo, double& hi) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o));
    hi = fmax(hi, __shfl_xor(hi, o));
  }
}

template <int NT>
struct IntShared {
  double red[NT / kWave];
  int ired[NT / kWave][4];
};

// Bounds of the nodes of a region's grid that lie inside the source (all NT lanes of the
// workgroup): box = {k0, k1, j0, j1}, k1 < 0 when none does.  A wavefront looks from both ends
// for its first and its last node inside on any of 64 columns, then in between only until
// both its outer columns are known to be inside.
template <int NT>
__device__ void inside_box(const FsArgs& a, const Lens& L, cd zs, const Region& g, IntShared<NT>& sh,
                           int (&box)[4]) {
  const double rho2 = a.rho * a.rho;
  const double dth = (g.t1 - g.t0) / a.n_theta, dr = (g.r1 - g.r0) / a.n_r;
  int k0 = 1 << 30, k1 = -1, j0 = 1 << 30, j1 = -1;
  const int lane = threadIdx.x % kWave;
  for (int jb = threadIdx.x - lane; jb < a.n_theta; jb += NT) {  // 64 columns, one a lane
    const bool act = jb + lane < a.n_theta;
    const int top = min(kWave, a.n_theta - jb) - 1;
    double sn, cs;
    sincos(g.t0 + (jb + lane + 0.5) * dth, &sn, &cs);
    // The columns that are inside at any of the nodes k, k + step, .. (eight side by side, those
    // past `end` left out); k becomes the first such node, or the next to look at.
    constexpr int kLook = 8;
    auto look = [&](int& k, int step, int end) -> uint64_t {
      uint64_t m[kLook], any = 0;
#pragma unroll
      for (int q = 0; q < kLook; ++q) {
        const int kq = k + q * step;
        m[q] = __builtin_amdgcn_ballot_w64(act && (end - kq) * step >= 0 &&
                                           source_f(L, g.r0 + kq * dr, cs, sn, zs, rho2) > 0.0);
        any |= m[q];
      }
      int to = kLook;
#pragma unroll
      for (int q = kLook - 1; q >= 0; --q) to = m[q] ? q : to;
      k += step * to;
      return any;
    };
    // up to the first node inside on any column, down to the last
    uint64_t seen = 0, below = 0;
    int first = 0, last = a.n_r;
    while (first <= a.n_r && seen == 0) seen = look(first, 1, a.n_r);
    if (seen == 0) continue;
    while (last > first && below == 0) below = look(last, -1, first);
    seen |= below;
    // the outermost columns inside at a node in between
    int lo = __builtin_ctzll(seen), hi = 63 - __builtin_clzll(seen);
    for (int k = first + 1; k < last && (lo > 0 || hi < top); k += kLook) {
      int at = k;
      seen |= look(at, 1, last - 1);
      lo = __builtin_ctzll(seen);
      hi = 63 - __builtin_clzll(seen);
    }
    k0 = min(k0, first);
    k1 = max(k1, last);
    j0 = min(j0, jb + lo);
    j1 = max(j1, jb + hi);
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    k0 = min(k0, __shfl_xor(k0, o));
    k1 = max(k1, __shfl_xor(k1, o));
    j0 = min(j0, __shfl_xor(j0, o));
    j1 = max(j1, __shfl_xor(j1, o));
  }
  if (threadIdx.x % kWave == 0) {
    int* w = sh.ired[threadIdx.x / kWave];
    w[0] = k0;
    w[1] = k1;
    w[2] = j0;
    w[3] = j1;
  }
  __syncthreads();
  for (int w = 0; w < NT / kWave; ++w) {
    k0 = min(k0, sh.ired[w][0]);
    k1 = max(k1, sh.ired[w][1]);
    j0 = min(j0, sh.ired[w][2]);
    j1 = max(j1, sh.ired[w][3]);
  }
  __syncthreads();
  box[0] = k0;
  box[1] = k1;
  box[2] = j0;
  box[3] = j1;
}

// Integral of the profile over one region (all NT lanes of the workgroup; a fixed order of
// the sums).  kLimb: a limb-darkened profile; without it the square roots drop out.
template <int NT, bool kLimb>
__device__ double integrate_region(const FsArgs& a, const Lens& L, cd zs, const Region& g, IntShared<NT>& sh) {
  const double rho2 = a.rho * a.rho;
  const double dth = (g.t1 - g.t0) / a.n_theta;
  const double dr = (g.r1 - g.r0) / a.n_r;
  const double c_ld = 1.5 * a.gamma / a.rho * (2.0 / 3.0);
  double acc = 0.0;
  for (int j = threadIdx.x; j < a.n_theta; j += NT) {
    double sn, cs;
    sincos(g.t0 + (j + 0.5) * dth, &sn, &cs);
    double col = 0.0, ra = g.r0;
    double fa = source_f(L, ra, cs, sn, zs, rho2);
    bool ina = fa > 0.0;
    double sa = kLimb && ina ? sqrt(fa) : 0.0;
    for (int k = 1; k <= a.n_r; ++k) {
      const double r = g.r0 + k * dr;
      const double f = source_f(L, r, cs, sn, zs, rho2);
      const bool inb = f > 0.0;
      double sb = 0.0;
      if (ina || inb) {
        if (kLimb && inb) sb = sqrt(f);
        // the inside part [lo, hi] of the segment, the limb where f (linear) is zero
        double lo = ra, hi = ra + dr;
        if (ina != inb) {
          const double rs = ra + dr * fa / (fa - f);
          lo = ina ? lo : rs;
          hi = inb ? hi : rs;
        }
        const double area = 0.5 * (lo + hi) * (hi - lo);
        col += (1.0 - a.gamma) * area;
        if (kLimb)  // mean of sqrt(f) over the part, f linear: 2/3 (fa + sa sb + fb) / (sa + sb)
          col += c_ld * area * (((sa * sa + sa * sb) + sb * sb) * recip(sa + sb));
      }
      fa = f;
      ra = r;
      sa = sb;
      ina = inb;
    }
    acc += col;
  }
  acc = wave_sum(acc);
  if (threadIdx.x % kWave == 0) sh.red[threadIdx.x / kWave] = acc;
  __syncthreads();
  acc = sh.red[0];
  for (int w = 1; w < NT / kWave; ++w) acc += sh.red[w];
  __syncthreads();
  return acc * dth;
}

// Regions of one source per workgroup.  Bound: latency, of the quintics (one per lane) and of
// the sorts; the runs, the radial parts and their bounds come from prefix counts and
// wavefront ranges (one lane walking the 1200 seeds three times took 0.5 of 0.87 ms for the
// 335 near epochs of a light curve, now 0.32 ms).
__global__ __launch_bounds__(kFsThreads) void k_fs_regions(FsArgs a) {
  __shared__ Shared sh;
  const Lens L{a.m1, a.m2, a.x1, a.x2};
  const int tid = threadIdx.x;
  const double two_pi = 2.0 * M_PI;
  for (int64_t item = blockIdx.x; item < a.n_items; item += gridDim.x) {
    const int64_t i = a.near_list[a.item0 + item];
    const cd zs = {a.zeta[2 * i], a.zeta[2 * i + 1]};
    if (tid == 0) sh.n_seed = 0;
    __syncthreads();
    // seeds: images of the centre (j = 0) and of the boundary points, then the
    // critical points whose caustic image lies inside the source
    for (int j = tid; j <= a.n_b; j += kFsThreads) {
      cd p = zs;
      if (j > 0) {
        double sn, cs;
        sincos(two_pi * ((j - 1) + 0.5) / a.n_b, &sn, &cs);
        p = {zs.x + a.rho * cs, zs.y + a.rho * sn};
      }
      cd z[5];
      bool sel[5];
      images_of(L, p, z, sel);
#pragma unroll
      for (int k = 0; k < 5; ++k)
        if (sel[k]) {
          const int slot = atomicAdd(&sh.n_seed, 1);
          if (slot < kSeedCap) {
            sh.r[slot] = cabs(z[k]);
            sh.th[slot] = atan2(z[k].y, z[k].x);
          }
        }
    }
    // at most kCritSeeds of them: those of every m-th phase, m the smallest stride
    // >= ceil(count / kCritSeeds) that keeps at most kCritSeeds
    int m = 1;
    for (int pass = 0;; ++pass) {
      int c = 0;
      for (int32_t j = tid; j < a.n_crit; j += kFsThreads)
        c += (((j >> 2) % m) == 0 && cabs(csub(cd{a.caus[2 * j], a.caus[2 * j + 1]}, zs)) < a.rho) ? 1 : 0;
      sh.ired[0][tid] = c;
      __syncthreads();
      for (int w = kFsThreads / 2; w > 0; w >>= 1) {
        if (tid < w) sh.ired[0][tid] += sh.ired[0][tid + w];
        __syncthreads();
      }
      const int count = sh.ired[0][0];
      __syncthreads();
      if (count <= kCritSeeds) break;
      m = pass == 0 ? (count + kCritSeeds - 1) / kCritSeeds : m + 1;
    }
    for (int32_t j = tid; j < a.n_crit; j += kFsThreads) {
      const cd c = {a.caus[2 * j], a.caus[2 * j + 1]};
      if (((j >> 2) % m) == 0 && cabs(csub(c, zs)) < a.rho) {
        const int slot = atomicAdd(&sh.n_seed, 1);
        if (slot < kSeedCap) {
          const cd z = {a.crit[2 * j], a.crit[2 * j + 1]};
          sh.r[slot] = cabs(z);
          sh.th[slot] = atan2(z.y, z.x);
        }
      }
    }
    __syncthreads();
    const int ns = sh.n_seed;
    if (ns > kSeedCap || ns == 0) {  // uniform
      if (tid == 0) {
        a.A[i] = __builtin_nan("");
        a.nreg[i] = -2;
        a.reg_count[item] = 0;
      }
      __syncthreads();
      continue;
    }
    // 1. seeds by angle
    for (int j = tid; j < kSeedCap; j += kFsThreads) sh.key[j] = j < ns ? sh.th[j] : __builtin_inf();
    __syncthreads();
    bitonic(sh.key, sh.r, sh.th);
    // 2. angular runs: cuts at gaps wider than `gap` (circularly); walking from the
    // seed after the first cut, run ids and angles unwrapped from each run's first seed.
    // Each lane takes kPer seeds in a row; prefix counts give the run ids.
    int first = INT_MAX;
    for (int j = tid; j < ns; j += kFsThreads) {
      const double nxt = j + 1 < ns ? sh.th[j + 1] : sh.th[0] + two_pi;
      const int cut = (nxt - sh.th[j] > a.gap) ? 1 : 0;  // cut after seed j
      sh.run[j] = cut;
      if (cut) first = min(first, j);
    }
    first = block_min(first, sh);
    if (first == INT_MAX) {  // no cut: one ring (uniform)
      double r0 = __builtin_inf(), r1 = -__builtin_inf();
      for (int j = tid; j < ns; j += kFsThreads) {
        r0 = fmin(r0, sh.r[j]);
        r1 = fmax(r1, sh.r[j]);
      }
      wave_range(r0, r1);
      __syncthreads();
      if (tid % kWave == 0) {  // sh.key's sorted angles are done with
        sh.key[2 * (tid / kWave)] = r0;
        sh.key[2 * (tid / kWave) + 1] = r1;
      }
      __syncthreads();
      if (tid == 0) {
        for (int w = 1; w < kFsThreads / kWave; ++w) {
          r0 = fmin(r0, sh.key[2 * w]);
          r1 = fmax(r1, sh.key[2 * w + 1]);
        }
        sh.reg[0] = Region{r0, r1, -M_PI, M_PI};
        sh.n_reg = 1;
      }
      __syncthreads();
    } else {
      const bool wraps = sh.run[ns - 1] == 0;  // the last seed's run goes on at seed 0
      int cuts[kPer], ids[kPer], mine = 0;
      for (int q = 0; q < kPer; ++q) {
        const int m = tid * kPer + q, j = (first + 1 + m) % ns;
        cuts[q] = m < ns ? sh.run[j] : 0;
        ids[q] = mine;
        mine += cuts[q];
      }
      const int before = block_prefix(mine, sh);
      // seeds before the first cut that follow seed 0 without a cut belong to the wrapped
      // run: their id is the last of the unwrapped part's
      if (tid == 0) sh.flag[1] = 0;
      __syncthreads();
      const int m_wrap = ns - 1 - first;  // m of seed 0
      for (int q = 0; q < kPer; ++q)
        if (tid * kPer + q == m_wrap) sh.flag[1] = before + ids[q];  // run id of seed 0
      __syncthreads();
      const int wrap_id = sh.flag[1];
      __syncthreads();
      for (int q = 0; q < kPer; ++q) {
        const int m = tid * kPer + q, j = (first + 1 + m) % ns;
        if (m < ns) {
          const int run = before + ids[q];
          if (wraps && m >= m_wrap && run == wrap_id) sh.th[j] += two_pi;
          sh.key[j] = run * 1.0e6 + sh.r[j];  // radii stay far below 1e6
        }
      }
      __syncthreads();
      // 3. seeds by (run, r); parts of a run split where the radius jumps
      bitonic(sh.key, sh.r, sh.th);
      int starts[kPer];
      mine = 0;
      for (int q = 0; q < kPer; ++q) {
        const int j = tid * kPer + q;
        const bool fresh = j < ns && (j == 0 || floor(sh.key[j] / 1.0e6) != floor(sh.key[j - 1] / 1.0e6) ||
                                      sh.r[j] - sh.r[j - 1] > fmax(a.gap * sh.r[j], 4.0 * a.rho));
        starts[q] = fresh ? 1 : 0;
        mine += starts[q];
      }
      int at = block_prefix(mine, sh);
      for (int q = 0; q < kPer; ++q)
        if (starts[q]) {
          if (at < kRegionCap) sh.run[at] = tid * kPer + q;  // the part's first seed
          ++at;
        }
      if (tid == kFsThreads - 1) sh.n_reg = min(at, kRegionCap + 1);
      __syncthreads();
      const int nr = min(sh.n_reg, kRegionCap);
      const bool over = sh.n_reg > kRegionCap;
      for (int g = tid / kWave; g < nr; g += kFsThreads / kWave) {  // a wavefront per part
        const int j0 = sh.run[g], j1 = g + 1 < nr || over ? sh.run[min(g + 1, nr - 1)] : ns;
        double t0 = __builtin_inf(), t1 = -__builtin_inf();
        for (int j = j0 + tid % kWave; j < j1; j += kWave) {
          t0 = fmin(t0, sh.th[j]);
          t1 = fmax(t1, sh.th[j]);
        }
        wave_range(t0, t1);
        if (tid % kWave == 0) sh.reg[g] = Region{sh.r[j0], sh.r[max(j1 - 1, j0)], t0, t1};
      }
      __syncthreads();
    }
    if (sh.n_reg > kRegionCap) {  // uniform
      if (tid == 0) {
        a.A[i] = __builtin_nan("");
        a.nreg[i] = -3;
        a.reg_count[item] = 0;
      }
      __syncthreads();
      continue;
    }
    // 4. padding: 10 % of the extent plus rho in r and rho / r1 in theta
    if (tid == 0) {
      for (int g = 0; g < sh.n_reg; ++g) {
        Region& R = sh.reg[g];
        const double dr = 0.1 * (R.r1 - R.r0) + a.rho;
        R.r0 = fmax(0.0, R.r0 - dr);
        R.r1 = R.r1 + dr;
        if (R.t1 - R.t0 < two_pi) {
          const double dt = 0.1 * (R.t1 - R.t0) + a.rho / fmax(R.r1, 1e-12);
          R.t0 -= dt;
          R.t1 += dt;
        }
        if (R.t1 - R.t0 >= two_pi) {
          R.t0 = -M_PI;
          R.t1 = M_PI;
        }
      }
    }
    __syncthreads();
    // 5. growth: a side with a sample inside the source moves out by a quarter extent
    for (int g = 0; g < sh.n_reg; ++g) {
      for (int it = 0; it < a.n_grow; ++it) {
        if (tid < 4) sh.flag[tid] = 0;
        __syncthreads();
        const Region R = sh.reg[g];
        const int sides = is_ring(R) ? 2 : 4;
        for (int t = tid; t < sides * a.n_side; t += kFsThreads) {
          const int side = t / a.n_side, k = t % a.n_side;
          double rr, tt;
          if (side < 2) {
            rr = side == 0 ? R.r0 : R.r1;
            tt = linspace_at(R.t0, R.t1, a.n_side, k);
          } else {
            rr = linspace_at(R.r0, R.r1, a.n_side, k);
            tt = side == 2 ? R.t0 : R.t1;
          }
          double sn, cs;
          sincos(tt, &sn, &cs);
          if (source_f(L, rr, cs, sn, zs, a.rho * a.rho) > 0.0) sh.flag[side] = 1;
        }
        __syncthreads();
        const int h0 = sh.flag[0], h1 = sh.flag[1], h2 = sh.flag[2], h3 = sh.flag[3];
        __syncthreads();
        if (!(h0 | h1 | h2 | h3)) break;
        if (tid == 0) {
          Region& W = sh.reg[g];
          const double dr = 0.25 * (W.r1 - W.r0), dt = 0.25 * (W.t1 - W.t0);
          if (h0) W.r0 = fmax(0.0, W.r0 - dr);
          if (h1) W.r1 = W.r1 + dr;
          if (h2) W.t0 = W.t0 - dt;
          if (h3) W.t1 = W.t1 + dt;
          if (W.t1 - W.t0 >= two_pi) {
            W.t0 = -M_PI;
            W.t1 = M_PI;
          }
        }
        __syncthreads();
      }
    }
    // 6. overlapping regions merge (first overlapping pair first, until none overlap)
    if (tid == 0) {
      bool changed = true;
      while (changed) {
        changed = false;
        for (int p = 0; p < sh.n_reg && !changed; ++p)
          for (int q = p + 1; q < sh.n_reg && !changed; ++q) {
            const Region& A = sh.reg[p];
            const Region& B = sh.reg[q];
            if (!(B.r1 < A.r0 || B.r0 > A.r1) && theta_overlap(A, B)) {
              sh.reg[p] = region_union(A, B);
              for (int m = q; m + 1 < sh.n_reg; ++m) sh.reg[m] = sh.reg[m + 1];
              --sh.n_reg;
              changed = true;
            }
          }
      }
    }
    __syncthreads();
    // 7. the regions and their work items for the integration kernel
    const int n_reg = sh.n_reg;
    if (tid < n_reg) {
      const Region R = sh.reg[tid];
      double* out = a.regs + 4 * (item * kFsRegionCap + tid);
      out[0] = R.r0;
      out[1] = R.r1;
      out[2] = R.t0;
      out[3] = R.t1;
    }
    if (tid == 0) {
      a.reg_count[item] = n_reg;
      sh.flag[0] = (int)atomicAdd(a.work_count, (uint32_t)n_reg);
    }
    __syncthreads();
    if (tid < n_reg) a.work[sh.flag[0] + tid] = (uint32_t)(item * kFsRegionCap + tid);
    __syncthreads();
  }
}

// 8. One workgroup per (source, region): up to n_shrink times the region is cut to its
// inside cells (plus one cell), then integrated.  Only the last grid's integral counts, so
// the earlier ones are searched for their inside nodes alone.
// Bound: FP64 issue, 26 FP64 operations and a reciprocal per node.  256 lanes a workgroup:
// all the regions of a light curve (about 1100 of 512 x 512 cells on 335 near epochs) are
// resident at once, where 512 lanes took a second, nearly empty round.  That curve: 1.3 ms,
// 1.5 with every node of every grid looked at, 3.7 before (two IEEE divisions a node, every
// grid integrated with two square roots and three divisions a segment, 512 lanes).
constexpr int kIntThreads = 256;
__global__ __launch_bounds__(kIntThreads) void k_fs_integrate(FsArgs a) {
  __shared__ IntShared<kIntThreads> sh;
  const Lens L{a.m1, a.m2, a.x1, a.x2};
  const uint32_t n_work = *a.work_count;
  for (uint32_t w = blockIdx.x; w < n_work; w += gridDim.x) {
    const uint32_t slot = a.work[w];
    const int64_t i = a.near_list[a.item0 + slot / kFsRegionCap];
    const cd zs = {a.zeta[2 * i], a.zeta[2 * i + 1]};
    const double* rg = a.regs + 4 * (int64_t)slot;
    Region R{rg[0], rg[1], rg[2], rg[3]};
    bool empty = false;
    for (int it = 0; it < a.n_shrink; ++it) {
      int box[4];
      inside_box<kIntThreads>(a, L, zs, R, sh, box);
      empty = box[1] < 0;
      if (empty) break;
      const double dr = (R.r1 - R.r0) / a.n_r;
      const int n0 = max(box[0] - 1, 0), n1 = min(box[1] + 1, a.n_r);
      Region N = {R.r0 + n0 * dr, R.r0 + n1 * dr, R.t0, R.t1};
      if (!is_ring(R)) {
        const double dth = (R.t1 - R.t0) / a.n_theta;
        N.t0 = R.t0 + max(box[2] - 1, 0) * dth;
        N.t1 = R.t0 + min(box[3] + 2, a.n_theta) * dth;
      }
      if (N.r0 == R.r0 && N.r1 == R.r1 && N.t0 == R.t0 && N.t1 == R.t1) break;
      R = N;
    }
    double val = 0.0;
    if (!empty)
      val = a.gamma > 0.0 ? integrate_region<kIntThreads, true>(a, L, zs, R, sh)
                          : integrate_region<kIntThreads, false>(a, L, zs, R, sh);
    if (threadIdx.x == 0) a.reg_val[slot] = val;
  }
}

// 9. Per source: the region integrals summed in region order (one thread per source).
__global__ __launch_bounds__(256) void k_fs_finish(FsArgs a) {
  const int64_t item = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (item >= a.n_items) return;
  const int32_t nr = a.reg_count[item];
  if (nr <= 0) return;  // a seed or region failure, already written
  const int64_t i = a.near_list[a.item0 + item];
  double total = 0.0;
  for (int g = 0; g < nr; ++g) total += a.reg_val[item * kFsRegionCap + g];
  a.A[i] = total / (M_PI * a.rho * a.rho);
  a.nreg[i] = nr;
}

// Source positions along a trajectory (FP64): tau = (t - t0)/tE,
// zeta = tau (cos a, sin a) + u0 (-sin a, cos a).
__global__ __launch_bounds__(256) void k_traj_positions(const double* t, int64_t n, double t0,
                                                        double u0, double tE, double ca, double sa,
                                                        double* zeta) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double tau = (t[i] - t0) / tE;
    zeta[2 * i] = tau * ca - u0 * sa;
    zeta[2 * i + 1] = tau * sa + u0 * ca;
  }
}

}  // namespace

hipError_t launch_traj_positions(const double* t, int64_t n, double t0, double u0, double tE,
                                 double alpha, double* zeta, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_traj_positions, dim3((unsigned)blocks), dim3(256), 0, st, t, n, t0, u0, tE,
                     cos(alpha), sin(alpha), zeta);
  return hipGetLastError();
}

hipError_t launch_fs_crit(double m1, double m2, double x1, double x2, int32_t nphi, double* crit,
                          double* caus, hipStream_t st) {
  if (nphi < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_fs_crit, dim3((unsigned)((4 * (int64_t)nphi + 63) / 64)), dim3(64), 0, st,
                     Lens{m1, m2, x1, x2}, nphi, crit, caus);
  return hipGetLastError();
}

hipError_t launch_fs_classify(const FsArgs& a, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u32_fs, dim3(1), dim3(64), 0, st, a.near_count);
  int64_t blocks = (a.n + 3) / 4;  // four sources (wavefronts) per workgroup
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_fs_classify, dim3((unsigned)blocks), dim3(256), 0, st, a);
  hipLaunchKernelGGL(k_fs_point, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_fs_images(const FsArgs& a, int32_t max_blocks, hipStream_t st) {
  if (a.n_items <= 0) return hipSuccess;
  if (a.n_b < 1 || a.n_side < 2 || a.n_r < 1 || a.n_theta < 1 || a.n_grow < 0 || a.n_shrink < 0 ||
      a.n_items > kFsBatch)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_fill_u32_fs, dim3(1), dim3(64), 0, st, a.work_count);
  const int64_t blocks = a.n_items < max_blocks ? a.n_items : max_blocks;
  hipLaunchKernelGGL(k_fs_regions, dim3((unsigned)blocks), dim3(kFsThreads), 0, st, a);
  hipLaunchKernelGGL(k_fs_integrate, dim3((unsigned)max_blocks), dim3(kIntThreads), 0, st, a);
  hipLaunchKernelGGL(k_fs_finish, dim3((unsigned)((a.n_items + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace morse
