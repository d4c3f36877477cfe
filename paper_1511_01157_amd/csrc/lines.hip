// Caustic-centred trajectory lines on gfx950: the minimum-magnification filter and the
// expansion of the kept lines into trajectory lists.
//
// Sec. 4.2 of McDougall & Albrow 2015 searches straight trajectories at radial distances
// from the caustic centres; sec. 4.3 first discards every trajectory whose magnification
// along its path, read from the point-source map, stays below the minimum that the
// light curve implies.  A line here is (u0, alpha, shift): the path tau (cos a, sin a) +
// u0 (-sin a, cos a), whose closest approach to its caustic centre is at tau = shift.
//
// Filter layout.  One wavefront per line, lanes over the samples, two chunks of 64 in
// flight: the line is sampled across the map window at spacing h <= 1 pixel, each sample with the
// search's value for a point (the same binary32 geometry and bilinear blend, the cell read
// from the map in tiles; the single-lens value off the map), and the largest value (NaN if any
// sample is NaN) decides.  The kept lines are then listed in ascending order by a stream compaction (one
// workgroup for a few thousand lines, else counts per block, one scan, scatter), so the
// result does not depend on the schedule.

#include "lines.h"

#include <algorithm>
#include <type_traits>

namespace morse {

namespace {

constexpr int kFilterThreads = 256;
constexpr int kCompactThreads = 256;
constexpr int kCompactPer = 4;  // flags per thread
constexpr int kCompactBlock = kCompactThreads * kCompactPer;

constexpr float kInf = __builtin_inff();

// lane j's value, the same in every lane (j uniform)
__device__ __forceinline__ float lane_at(float v, int32_t j) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
}

// Inclusive prefix minimum or maximum over the lanes of values that hold no NaN, by DPP: shifts
// of 1, 2, 4 and 8 lanes inside the rows of 16, then the last lane of each row (of each
// half) to the rows after it.  12 instructions without the LDS, where a scan of shuffles,
// compares and selects takes 30 and the LDS's latency six times.
template <bool kMin>
__device__ __forceinline__ float lane_prefix(float x) {
  auto step = [&](auto ctrl, auto rows) {
    const int none = __float_as_int(kMin ? kInf : -kInf);
    const float y = __int_as_float(__builtin_amdgcn_update_dpp(
        none, __float_as_int(x), decltype(ctrl)::value, decltype(rows)::value, 0xf, false));
    x = kMin ? (y < x ? y : x) : (y > x ? y : x);
  };
  using std::integral_constant;
  step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});  // row_shr:1
  step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
  step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
  step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
  step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});  // row_bcast:15, rows 1 and 3
  step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});  // row_bcast:31, rows 2 and 3
  return x;
}

// v of lane l - 1 (lane 0 takes first).
__device__ __forceinline__ float from_below(float v, float first) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(first), __float_as_int(v), 0x138, 0xf, 0xf, false));
}

// A line's path and samples.  Sample k sits at tau_k = lo + k h; the position and the
// blend are the search's (time origin 0, tE 1, which change nothing).
struct LinePath {
  float ca, sa, bx, by, lo;
};
__device__ __forceinline__ LinePath line_path(const LineFilterArgs& a, int64_t l) {
  const double u0 = a.lines[3 * l], al = a.lines[3 * l + 1];
  double sn, cn;
  sincos(al, &sn, &cn);
  LinePath p;
  p.ca = (float)cn;
  p.sa = (float)sn;
  p.bx = (float)(-u0 * sn);
  p.by = (float)(u0 * cn);
  p.lo = (float)((a.cxw * cn + a.cyw * sn) - a.half_diag);
  return p;
}

// Index of cell (i, j)'s first pixel; i, j < 2^15, where the products are i / 7 and j / 3.
__device__ __forceinline__ uint32_t tile_index(const TileMap& t, uint32_t i, uint32_t j) {
  const uint32_t ti = __umul24(i, 37450u) >> 18, tj = __umul24(j, 43691u) >> 17;
  return __umul24(tj, t.row) + (__umul24(ti, 25u) + ((j << 3) + i));
}
// The pixels (i, j), (i + 1, j) and (i, j + 1), (i + 1, j + 1) as a cell; an index outside the
// packed map reads zeros.
__device__ __forceinline__ Quad ld_tile(const TileMap& t, uint32_t q) {
  const uint64_t base = (uint64_t)t.p;
  const rsrc4 r = {(int)(uint32_t)base, (int)((uint32_t)(base >> 32) | (4u << 16)), (int)t.n, kBufferWord3};
  const float2v a = struct_buffer_load_f2(r, (int)q, 0, 0, 0), b = struct_buffer_load_f2(r, (int)q, 32, 0, 0);
  return Quad{a.x, a.y, b.x, b.y};  // right pixels, not yet steps
}

// Packs a map into its tiles (pixels beyond the map are zero and belong to no cell).
__global__ __launch_bounds__(256) void k_tile_pack(MapC m, TileMap t) {
  for (uint32_t q = blockIdx.x * 256u + threadIdx.x; q < t.n; q += gridDim.x * 256u) {
    const uint32_t tile = q >> 5, tj = tile / t.tiles_x, ti = tile - tj * t.tiles_x;
    const uint32_t i = 7 * ti + (q & 7u), j = 3 * tj + ((q >> 3) & 3u);
    const bool in = i < (uint32_t)m.mx && j < (uint32_t)m.my;
    const_cast<float*>(t.p)[q] = in ? m.map[(size_t)j * m.mx + i] : 0.0f;
  }
}

// Samples of C chunks of 64 from sample kf (this lane's, as a float: below 2^24, exact) on,
// their cells in flight together.  kCentred: a window about (0, 0).
template <int C, bool kCentred>
__device__ __forceinline__ void line_samples(const LineFilterArgs& a, const LinePath& p, float kf, float (&A)[C]) {
  const MapC& m = a.m;
  float zx[C], zy[C], fx[C], fy[C];
  uint64_t on[C];
  Quad cell[C];
#pragma unroll
  for (int u = 0; u < C; ++u) {
    const float tau = p.lo + (kf + (float)(u * kWave)) * a.h;
    zx[u] = tau * p.ca + p.bx;
    zy[u] = tau * p.sa + p.by;
    const float gx = ((kCentred ? zx[u] : zx[u] - m.sx) * m.kx) + m.ox;
    const float gy = ((kCentred ? zy[u] : zy[u] - m.sy) * m.ky) + m.oy;
    on[u] = __builtin_amdgcn_ballot_w64(__float_as_uint(gx) < __float_as_uint(m.lx)) &
            __builtin_amdgcn_ballot_w64(__float_as_uint(gy) < __float_as_uint(m.ly));
    fx[u] = __builtin_amdgcn_fractf(gx);
    fy[u] = __builtin_amdgcn_fractf(gy);
    const bool mine = __builtin_amdgcn_inverse_ballot_w64(on[u]);
    cell[u] = ld_tile(a.t, mine ? tile_index(a.t, (uint32_t)gx, (uint32_t)gy) : 0u);
  }
#pragma unroll
  for (int u = 0; u < C; ++u) {
    const Quad c = cell[u];
    A[u] = blend(Quad{c.v00, c.e0 - c.v00, c.v01, c.e1 - c.v01}, fx[u], fy[u]);
    if (~on[u]) {  // uniform
      const float P = point_lens_A(zx[u], zy[u]);
      A[u] = __builtin_amdgcn_inverse_ballot_w64(on[u]) ? A[u] : P;
    }
  }
}

// Largest of the lanes' samples; NaN when any sample was NaN.
__device__ __forceinline__ float line_best(float best, uint64_t nans) {
  return nans ? __builtin_nanf("") : lane_at(lane_prefix<false>(best), kWave - 1);
}

constexpr int kLineChunks = 2;  // chunks of samples in flight (1, 2, 4: the filter 158, 160, 159 us, the peaks 283, 271, 280)

// Filter, one wavefront per line.  Bound: the pixels' way from L2 and beyond (each line has
// its own direction, so an XCD's L2 sees the whole map), then instruction issue: 24,576
// lines x 2,898 samples of a 2048^2 map 0.16 ms = 4.5e11 samples/s.  From the search's 16-byte
// cells it takes 0.33 ms (2.4 GB beyond L2, 7 TB/s, L2 hits 23%), 0.285 with one chunk in
// flight, and the packing writes 67 MB in place of 26.
template <bool kCentred>
__global__ __launch_bounds__(kFilterThreads) void k_line_filter(LineFilterArgs a) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t waves = (int64_t)gridDim.x * (kFilterThreads / kWave);
  for (int64_t l = blockIdx.x * (int64_t)(kFilterThreads / kWave) + threadIdx.x / kWave; l < a.n;
       l += waves) {
    const LinePath p = line_path(a, l);
    float best = -kInf;
    uint64_t nans = 0;
    for (int32_t c0 = 0; c0 < a.ns; c0 += kLineChunks * kWave) {
      float A[kLineChunks];
      line_samples<kLineChunks, kCentred>(a, p, (float)(c0 + lane), A);
#pragma unroll
      for (int u = 0; u < kLineChunks; ++u) {
        const bool in = c0 + u * kWave + lane < a.ns;
        nans |= __builtin_amdgcn_ballot_w64(in && A[u] != A[u]);
        best = in && A[u] > best ? A[u] : best;
      }
    }
    best = line_best(best, nans);
    if (lane == 0) {
      a.best[l] = best;
      a.keep[l] = best >= a.amin ? 1 : 0;
    }
  }
}

// Peak library.  One wavefront per line (four per workgroup): each chunk of 64 samples is
// computed lane-parallel exactly as in the filter.  A peak is a rise above fl32(trough *
// up) followed by a fall below fl32(top * down); the first sample starts the first
// trough; equal maxima keep the first.  The rule is a left-to-right scan, but between
// two of its events (a rise, a fall) the state changes only by a running minimum (the
// trough) or a running maximum (the top and its index), so each chunk is taken one
// event at a time.  Where no sample left in the chunk lies below the trough (above the
// top) the trough (top) holds for all of them and one compare finds the next event; else
// a prefix minimum or maximum over the lanes gives every sample the trough or top the
// scan would hold before it.  The first lane whose sample rises or
// falls against that value (found by ballot) is the next event, and the scan resumes
// after it.  NaN samples neither lower the trough, raise the top nor trigger an event, as in
// the scan; a NaN first sample leaves the trough NaN and the line without peaks.
// The lines above, a noisy map: 0.27 ms; 0.45 ms before, with a scan of shuffles per event and
// the 16-byte cells.
template <bool kCentred>
__global__ __launch_bounds__(kFilterThreads) void k_line_peaks(LinePeakArgs a) {
  const LineFilterArgs& f = a.f;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t waves = (int64_t)gridDim.x * (kFilterThreads / kWave);
  const float nan = __builtin_nanf("");
  for (int64_t l = blockIdx.x * (int64_t)(kFilterThreads / kWave) + threadIdx.x / kWave; l < f.n;
       l += waves) {
    const LinePath p = line_path(f, l);
    float best = -kInf;
    uint64_t nans = 0;
    float trough = 0.0f, top = 0.0f;
    int32_t top_i = 0, count = 0;
    bool rising = false;
    for (int32_t b0 = 0; b0 < f.ns; b0 += kLineChunks * kWave) {
      float S[kLineChunks];
      line_samples<kLineChunks, kCentred>(f, p, (float)(b0 + lane), S);
#pragma unroll
      for (int u = 0; u < kLineChunks; ++u) {
        const int32_t c0 = b0 + u * kWave, nk = min(kWave, f.ns - c0);
        if (nk <= 0) break;
        const float A = S[u];
        const uint64_t in = nk < kWave ? (1ull << nk) - 1ull : ~0ull;
        uint64_t act = in & __builtin_amdgcn_ballot_w64(A == A);  // samples not yet scanned
        nans |= in & ~act;
        best = __builtin_amdgcn_inverse_ballot_w64(act) && A > best ? A : best;
        if (c0 == 0) {
          trough = lane_at(A, 0);
          act &= ~1ull;
        }
        while (act) {
          if (!rising) {
            if (trough != trough) break;  // no sample compares with a NaN trough
            uint64_t ev;
            float low = trough;
            if ((__builtin_amdgcn_ballot_w64(A < trough) & act) == 0) {
              ev = __builtin_amdgcn_ballot_w64(A > trough * a.up) & act;
            } else {
              const float q = lane_prefix<true>(__builtin_amdgcn_inverse_ballot_w64(act) ? A : kInf);
              float T = from_below(q, kInf);
              T = T < trough ? T : trough;  // the trough before this lane's sample
              ev = __builtin_amdgcn_ballot_w64(A >= T) & __builtin_amdgcn_ballot_w64(A > T * a.up) & act;
              low = lane_at(q, kWave - 1);
            }
            if (ev == 0) {
              if (low < trough) trough = low;
              break;
            }
            const int32_t j = __builtin_ctzll(ev);
            top = lane_at(A, j);
            top_i = c0 + j;
            rising = true;
            act &= ~1ull << j;
          } else {
            uint64_t ev;
            if ((__builtin_amdgcn_ballot_w64(A > top) & act) == 0) {
              ev = __builtin_amdgcn_ballot_w64(A < top * a.down) & act;
            } else {
              const float q = lane_prefix<false>(__builtin_amdgcn_inverse_ballot_w64(act) ? A : -kInf);
              float T = from_below(q, -kInf);
              T = T > top ? T : top;  // the top before this lane's sample
              ev = __builtin_amdgcn_ballot_w64(A <= T) & __builtin_amdgcn_ballot_w64(A < T * a.down) & act;
              // the samples before the event (all of them without one)
              const uint64_t before = ev ? act & ((1ull << __builtin_ctzll(ev)) - 1ull) : act;
              if (before) {
                const float mx = lane_at(q, 63 - __builtin_clzll(before));
                if (mx > top) {  // the first sample equal to the new maximum
                  const int32_t j = __builtin_ctzll(__builtin_amdgcn_ballot_w64(A == mx) & before);
                  top = lane_at(A, j);
                  top_i = c0 + j;
                }
              }
            }
            if (ev == 0) break;
            if (lane == 0 && count < a.kmax) {
              a.ptau[l * a.kmax + count] = p.lo + (float)top_i * f.h;
              a.pA[l * a.kmax + count] = top;
            }
            ++count;
            rising = false;
            const int32_t end = __builtin_ctzll(ev);
            trough = lane_at(A, end);
            act &= ~1ull << end;
          }
        }
      }
    }
    best = line_best(best, nans);
    for (int32_t j = count + lane; j < a.kmax; j += kWave) {
      a.ptau[l * a.kmax + j] = nan;
      a.pA[l * a.kmax + j] = nan;
    }
    if (lane == 0) {
      f.best[l] = best;
      a.npeaks[l] = count;
      f.keep[l] = (best >= f.amin && count >= a.min_peaks) ? 1 : 0;
    }
  }
}

// Eqs. 7-8 per line, in FP64: one observed time -> the highest peak (ties: the earlier)
// with the given tE; two -> the two highest, in tau order.  t0' = t0 + shift tE.
__global__ __launch_bounds__(256) void k_peak_starts(PeakStartArgs a) {
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < a.n;
       k += (int64_t)gridDim.x * blockDim.x) {
    const int64_t l = a.kept ? a.kept[k] : k;
    const int32_t np = min(a.npeaks[l], a.kmax);
    double s0 = __builtin_nan(""), s1 = __builtin_nan("");
    if (np >= a.n_tp) {
      const float* A = a.pA + l * a.kmax;
      const float* T = a.ptau + l * a.kmax;
      int32_t j1 = 0;  // highest
      for (int32_t j = 1; j < np; ++j)
        if (A[j] > A[j1]) j1 = j;
      const double shift = a.lines[3 * l + 2];
      double tE, t0;
      if (a.n_tp == 1) {
        tE = a.tE;
        t0 = a.tp1 - (double)T[j1] * tE;
      } else {
        int32_t j2 = -1;  // second highest
        for (int32_t j = 0; j < np; ++j)
          if (j != j1 && (j2 < 0 || A[j] > A[j2])) j2 = j;
        const int32_t lo = min(j1, j2), hi = max(j1, j2);
        const double m1 = (double)T[lo], m2 = (double)T[hi];
        tE = (a.tp2 - a.tp1) / (m2 - m1);
        t0 = a.tp1 - m1 * tE;
      }
      s0 = t0 + shift * tE;
      s1 = tE;
    }
    a.start[2 * k] = s0;
    a.start[2 * k + 1] = s1;
  }
}

// Block b counts the set flags of keep[b B, (b + 1) B).
__global__ __launch_bounds__(kCompactThreads) void k_compact_count(const uint8_t* keep, int64_t n,
                                                                   int64_t* counts) {
  __shared__ int s[kCompactThreads];
  const int64_t base = blockIdx.x * (int64_t)kCompactBlock + threadIdx.x * kCompactPer;
  int c = 0;
  for (int j = 0; j < kCompactPer; ++j)
    if (base + j < n) c += keep[base + j] ? 1 : 0;
  s[threadIdx.x] = c;
  __syncthreads();
  for (int w = kCompactThreads / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) counts[blockIdx.x] = s[0];
}

// Exclusive scan of the nb block counts in place (one workgroup, chunk by chunk); the
// total goes to *total.
__global__ __launch_bounds__(kCompactThreads) void k_compact_scan(int64_t* counts, int64_t nb,
                                                                  int64_t* total) {
  __shared__ int64_t s[kCompactThreads];
  int64_t carry = 0;
  for (int64_t c0 = 0; c0 < nb; c0 += kCompactThreads) {
    const int64_t i = c0 + threadIdx.x;
    const int64_t v = i < nb ? counts[i] : 0;
    s[threadIdx.x] = v;
    __syncthreads();
    for (int w = 1; w < kCompactThreads; w <<= 1) {  // inclusive Hillis-Steele scan
      const int64_t add = threadIdx.x >= w ? s[threadIdx.x - w] : 0;
      __syncthreads();
      s[threadIdx.x] += add;
      __syncthreads();
    }
    if (i < nb) counts[i] = carry + s[threadIdx.x] - v;
    carry += s[kCompactThreads - 1];
    __syncthreads();
  }
  if (threadIdx.x == 0) *total = carry;
}

// Block b writes the indices of its set flags from position offsets[b] on.
__global__ __launch_bounds__(kCompactThreads) void k_compact_scatter(const uint8_t* keep, int64_t n,
                                                                     const int64_t* offsets,
                                                                     int64_t* kept) {
  __shared__ int s[kCompactThreads];
  const int64_t base = blockIdx.x * (int64_t)kCompactBlock + threadIdx.x * kCompactPer;
  int c = 0;
  for (int j = 0; j < kCompactPer; ++j)
    if (base + j < n) c += keep[base + j] ? 1 : 0;
  s[threadIdx.x] = c;
  __syncthreads();
  for (int w = 1; w < kCompactThreads; w <<= 1) {
    const int add = threadIdx.x >= w ? s[threadIdx.x - w] : 0;
    __syncthreads();
    s[threadIdx.x] += add;
    __syncthreads();
  }
  int64_t pos = offsets[blockIdx.x] + s[threadIdx.x] - c;
  for (int j = 0; j < kCompactPer; ++j)
    if (base + j < n && keep[base + j]) kept[pos++] = base + j;
}

// The whole compaction in one workgroup, a tile of 16 flags per lane at a time (keep 16-byte
// aligned): one launch for three while a few tiles hold all lines.
constexpr int kOneThreads = 1024, kOneTile = 16 * kOneThreads;
__global__ __launch_bounds__(kOneThreads) void k_compact_one(const uint8_t* __restrict__ keep, int64_t n,
                                                             int64_t* __restrict__ kept,
                                                             int64_t* __restrict__ total) {
  __shared__ uint32_t s_wave[kOneThreads / kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  int64_t carry = 0;
  for (int64_t b0 = 0; b0 < n; b0 += kOneTile) {
    const int64_t i0 = b0 + 16 * (int64_t)threadIdx.x;
    uint32_t bits = 0;
    if (i0 + 16 <= n) {
      const uint4 v = *reinterpret_cast<const uint4*>(keep + i0);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int j = 0; j < 16; ++j) bits |= ((w[j / 4] >> (8 * (j % 4))) & 0xffu ? 1u : 0u) << j;
    } else {
      for (int j = 0; i0 + j < n; ++j) bits |= (keep[i0 + j] ? 1u : 0u) << j;
    }
    const uint32_t c = __popc(bits);
    uint32_t incl = c;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t l = __shfl_up(incl, o);
      if (lane >= o) incl += l;
    }
    if (lane == kWave - 1) s_wave[wave] = incl;
    __syncthreads();
    uint32_t before = incl - c, all = 0;
#pragma unroll
    for (int w = 0; w < kOneThreads / kWave; ++w) {
      before += w < wave ? s_wave[w] : 0u;
      all += s_wave[w];
    }
    __syncthreads();
    if (kept)
      for (int64_t pos = carry + before; bits; bits &= bits - 1) kept[pos++] = i0 + __builtin_ctz(bits);
    carry += all;
  }
  if (threadIdx.x == 0) *total = carry;
}

__global__ __launch_bounds__(256) void k_lines_traj(const double* lines, const int64_t* kept,
                                                    int64_t n_kept, const double* t0, int32_t n_t0,
                                                    const double* tE, int32_t n_tE,
                                                    double* params) {
  const int64_t per = (int64_t)n_t0 * n_tE;
  const int64_t total = n_kept * per;
  for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < total;
       j += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = j / per;
    const int32_t a = (int32_t)((j / n_tE) % n_t0), b = (int32_t)(j % n_tE);
    const int64_t l = kept ? kept[k] : k;
    const double u0 = lines[3 * l], al = lines[3 * l + 1], shift = lines[3 * l + 2];
    params[4 * j] = t0[a] - shift * tE[b];
    params[4 * j + 1] = u0;
    params[4 * j + 2] = tE[b];
    params[4 * j + 3] = al;
  }
}

}  // namespace

hipError_t launch_tile_pack(const MapC& m, const TileMap& t, hipStream_t st) {
  if (!m.map || !t.p || t.n == 0) return hipErrorInvalidValue;
  const uint32_t blocks = std::min<uint32_t>((t.n + 255) / 256, 65536);
  hipLaunchKernelGGL(k_tile_pack, dim3(blocks), dim3(256), 0, st, m, t);
  return hipGetLastError();
}

hipError_t launch_line_filter(const LineFilterArgs& a, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  if (!a.lines || !a.best || !a.keep || a.ns < 2 || !a.t.p) return hipErrorInvalidValue;
  const int64_t per_block = kFilterThreads / kWave;
  int64_t blocks = (a.n + per_block - 1) / per_block;
  if (blocks > (1 << 20)) blocks = 1 << 20;
  if (a.m.sx == 0.0f && a.m.sy == 0.0f)
    hipLaunchKernelGGL(k_line_filter<true>, dim3((unsigned)blocks), dim3(kFilterThreads), 0, st, a);
  else
    hipLaunchKernelGGL(k_line_filter<false>, dim3((unsigned)blocks), dim3(kFilterThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_line_peaks(const LinePeakArgs& a, hipStream_t st) {
  if (a.f.n <= 0) return hipSuccess;
  if (!a.f.lines || !a.f.best || !a.f.keep || !a.npeaks || !a.ptau || !a.pA || a.f.ns < 2 ||
      !a.f.t.p || a.kmax < 1)
    return hipErrorInvalidValue;
  const int64_t per_block = kFilterThreads / kWave;
  int64_t blocks = (a.f.n + per_block - 1) / per_block;
  if (blocks > (1 << 20)) blocks = 1 << 20;
  if (a.f.m.sx == 0.0f && a.f.m.sy == 0.0f)
    hipLaunchKernelGGL(k_line_peaks<true>, dim3((unsigned)blocks), dim3(kFilterThreads), 0, st, a);
  else
    hipLaunchKernelGGL(k_line_peaks<false>, dim3((unsigned)blocks), dim3(kFilterThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_peak_starts(const PeakStartArgs& a, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  int64_t blocks = (a.n + 255) / 256;
  if (blocks > (1 << 20)) blocks = 1 << 20;
  hipLaunchKernelGGL(k_peak_starts, dim3((unsigned)blocks), dim3(256), 0, st, a);
  return hipGetLastError();
}

size_t compact_scratch_elems(int64_t n) { return (size_t)((n + kCompactBlock - 1) / kCompactBlock) + 1; }

hipError_t launch_compact(const uint8_t* keep, int64_t n, int64_t* scratch, int64_t* kept,
                          int64_t* d_count, hipStream_t st) {
  if (n <= 0) return hipErrorInvalidValue;
  // up to eight tiles one workgroup takes the place of three launches (24,576 lines: 16 us
  // either way, and two launches less)
  if (n <= 8 * kOneTile && ((uintptr_t)keep % 16) == 0) {
    hipLaunchKernelGGL(k_compact_one, dim3(1), dim3(kOneThreads), 0, st, keep, n, kept, d_count);
    return hipGetLastError();
  }
  const int64_t nb = (n + kCompactBlock - 1) / kCompactBlock;
  if (nb > (int64_t)1 << 30) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_compact_count, dim3((unsigned)nb), dim3(kCompactThreads), 0, st, keep, n,
                     scratch);
  hipLaunchKernelGGL(k_compact_scan, dim3(1), dim3(kCompactThreads), 0, st, scratch, nb, d_count);
  if (kept)
    hipLaunchKernelGGL(k_compact_scatter, dim3((unsigned)nb), dim3(kCompactThreads), 0, st, keep,
                       n, scratch, kept);
  return hipGetLastError();
}

hipError_t launch_lines_to_traj(const double* lines, const int64_t* kept, int64_t n_kept,
                                const double* t0, int32_t n_t0, const double* tE, int32_t n_tE,
                                double* params, hipStream_t st) {
  const int64_t total = n_kept * (int64_t)n_t0 * n_tE;
  if (total <= 0) return hipSuccess;
  int64_t blocks = (total + 255) / 256;
  if (blocks > (1 << 20)) blocks = 1 << 20;
  hipLaunchKernelGGL(k_lines_traj, dim3((unsigned)blocks), dim3(256), 0, st, lines, kept, n_kept,
                     t0, n_t0, tE, n_tE, params);
  return hipGetLastError();
}

}  // namespace morse
