// Map build on gfx950: inverse ray shooting into LDS-privatised uint32 histogram
// tiles merged with global atomics, then normalisation + uniform-disk convolution.
//
// Method: ray-shooting magnification maps (the family cited in sec. 3 of McDougall &
// Albrow 2015) of the binary-lens equation Eq. 2 with the lens placement of sec. 4.1;
// finite-source maps by convolution with the source profile (sec. 4.1).
//
// Ray kernel layout.  A 256-thread workgroup owns a tile of the image-plane lattice, 16 A
// x 16 B rays, A B of them per thread.  Rays are generated from their indices (no input
// arrays).  Thread (tx, ty) of a 16 x 16 arrangement takes the A x B block of rays at
// (A tx, B ty), so the lanes of one instruction lie A rays apart in x and B in y, i.e. on
// different source pixels (a lattice has several rays a pixel), which keeps the LDS
// atomics of an instruction off a single address (64 lanes on one address take 128 cycles
// of the LDS, on different ones 4), and the terms of a column and of a row are computed
// once per thread.  On a coarse lattice (about a ray a pixel or fewer) the lanes take neighbouring
// rays instead, whose pixels differ anyway, so that the atomics of an instruction that go to
// memory share its lines.  A tile whose rays provably all miss the window is skipped (see
// tile_misses).  Pass 1 computes every ray's bin and the
// workgroup's bounding box of in-window bins.  If the box fits in the LDS tile
// (RS_CAP or RS_CAP_COARSE bins) the rays are counted with LDS atomics and the non-zero bins merged
// with one global atomic each; otherwise (tiles straddling a lens, whose rays scatter
// over the whole source plane) each ray goes to a global atomic directly.  Integer
// addition is order-free, so the counts are bit-identical whatever the schedule.
//
// Mirror pairs.  With both lenses on the x axis, a lattice centred on y = 0 with an
// even row count and a window centred on y = 0, the ray of row ny - 1 - j is the
// mirror image of the ray of row j: its y is exactly -y, and since binary32 rounding
// commutes with negation every step of Eq. 2 gives exactly the same x and the negated
// y, so its bin is (bx, 2h - 1 - by) by the symmetric bin rule (h = my / 2), unless
// its y offset in the window is +-0, when both rays fall in row h.  Rows that have
// their mirror row in the same call are then shot once, from the upper half, and each
// binned ray is counted in both bins (the +-0 rays twice in their own bin); the ray
// statistics count every shot ray twice.

#include <algorithm>

#include "internal.h"

#include <cmath>

namespace morse {

namespace {

constexpr int RS_THREADS = 256;
constexpr int RS_CAP = 4096, RS_CAP_COARSE = 6144;  // LDS histogram bins (16, 24 KiB)

// n words at p; quads: the first 4 quads of them lie on 16-byte boundaries and go 16 bytes a
// store (16 MiB: 13 us in words, 9 so).
__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* p, size_t n, size_t quads, uint32_t v) {
  const size_t first = blockIdx.x * (size_t)256 + threadIdx.x, step = gridDim.x * (size_t)256;
  for (size_t i = first; i < quads; i += step) reinterpret_cast<uint4*>(p)[i] = make_uint4(v, v, v, v);
  for (size_t i = 4 * quads + first; i < n; i += step) p[i] = v;
}

__global__ void k_fill_u64(uint64_t* p, size_t n, uint64_t v) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// m / r, correctly rounded, for m = 0 or m in [2^-40, 1] and r in [2^-40, 2^40]: Markstein's
// method (the reciprocal, one Newton step, two corrections of the quotient by its residual),
// without the range scaling and the fix-up of special cases that a general division adds and
// that change nothing in this range (8 instructions for 11).
__device__ __forceinline__ float div_in_range(float m, float r) {
  float y = __builtin_amdgcn_rcpf(r);
  y = fmaf(fmaf(-r, y, 1.0f), y, y);
  float q = m * y;
  q = fmaf(fmaf(-r, q, m), y, q);
  return fmaf(fmaf(-r, q, m), y, q);
}

// Whether every ray of the rectangle [xa, xb] x [ya, yb] misses the window.  A lens at x_k
// displaces a ray by m_k / |z - x_k| at most, so with d_k the distance of lens k from the
// rectangle zeta lies within D = sum m_k / d_k of z in x and in y.  The slack covers the
// roundings of the binary32 ray (each of its few operations is off by 2^-24 of a number
// no larger than |z| + D + |s|) and one pixel.  Where a ray's offset in pixels might overflow
// (`big` bounds it in Einstein radii) the tile is kept: such rays count as non-finite, not as
// outside.  kSafe rays cannot.
template <bool kSafe>
__device__ __forceinline__ bool tile_misses(const RayParams& p, float xa, float xb, float ya, float yb) {
  const float dy = fmaxf(fmaxf(ya, -yb), 0.0f);
  const float e1 = fmaxf(fmaxf(xa - p.x1, p.x1 - xb), 0.0f), e2 = fmaxf(fmaxf(xa - p.x2, p.x2 - xb), 0.0f);
  // the hardware's reciprocal square root and reciprocal, within 2^-22, inside the slack;
  // a rectangle that holds a lens gets inf, and is kept
  const float D = p.m1 * __builtin_amdgcn_rsqf(e1 * e1 + dy * dy) + p.m2 * __builtin_amdgcn_rsqf(e2 * e2 + dy * dy);
  const float big = fmaxf(fmaxf(fabsf(xa), fabsf(xb)), fmaxf(fabsf(ya), fabsf(yb))) + D +
                    fmaxf(fabsf(p.sx), fabsf(p.sy));
  if (!kSafe && !(big * fmaxf(p.kx, p.ky) < 0x1p126f)) return false;
  const float slack = D + 1e-4f * big;
  const float wx = ((float)(p.mx >> 1) + 1.0f) * (1.0001f * __builtin_amdgcn_rcpf(p.kx)) + slack;
  const float wy = ((float)(p.my >> 1) + 1.0f) * (1.0001f * __builtin_amdgcn_rcpf(p.ky)) + slack;
  return xa - p.sx > wx || xb - p.sx < -wx || ya - p.sy > wy || yb - p.sy < -wy;
}

typedef unsigned short us2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(us2, a), __builtin_bit_cast(us2, b)));
}
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(us2, a), __builtin_bit_cast(us2, b)));
}

// kMirror: rows of the upper half, each ray standing for itself and its mirror ray.
// kSafe: the host has shown that every r_k = |z - x_k|^2 of the rows lies in [2^-40, 2^40]
// (and the masses and scales in range), so the short division is exact and no ray is
// non-finite.  The general form divides as IEEE asks and counts non-finite rays.
//
// Bound: instruction issue.  32768^2 rays (lattice twice the window's width) in mirror
// pairs into 2048^2: 373 us = 2.9e12 lattice rays/s, 43% of the tiles kept, 66 VALU
// instructions per kept wavefront of rays at 3.4 cycles each; without the LDS atomics or
// the merges it takes 375 and 358 us.  Before: 1.03 ms (and 2.02 ms with the statistics,
// whose three addresses took 260,000 atomics each) at 104 instructions per wavefront of
// rays: no tile skipped, IEEE divisions with scalings, the lattice point, finiteness and
// range tested per ray, scalar operands.
template <bool kMirror, bool kSafe, int A, int B, bool kCoarse>
__global__ __launch_bounds__(RS_THREADS) void k_rayshoot(RayParams p, uint32_t* __restrict__ counts,
                                                         unsigned long long* __restrict__ stats,
                                                         uint32_t slot_mask) {
  constexpr int CAP = kCoarse ? RS_CAP_COARSE : RS_CAP;
  __shared__ uint32_t hist[CAP];
  __shared__ uint32_t s_box[RS_THREADS / kWave][2];
  __shared__ uint32_t s_stat[RS_THREADS / kWave][3];

  const int tid = threadIdx.x;
  const int tx = tid & 15;
  const int ty = tid >> 4;
  const int wave = tid >> 6;
  const int lane = tid & 63;
  const int x0 = blockIdx.x * (16 * A);
  const int y0 = p.row0 + blockIdx.y * (16 * B);
  auto row_of = [&](int b) { return kCoarse ? ty + 16 * b : ty * B + b; };
  auto lattice = [](float c, int i, int n, float h) { return c + ((float)(i - (n >> 1)) + 0.5f) * h; };

  const int x1 = min(x0 + 16 * A, p.nx) - 1, y1 = min(y0 + 16 * B, p.row1) - 1;  // last column, row
  const uint32_t shot = (uint32_t)(x1 - x0 + 1) * (uint32_t)(y1 - y0 + 1);
  constexpr uint32_t kRays = kMirror ? 2u : 1u;  // rays each shot ray stands for
  // slot of the statistics this workgroup adds to (few workgroups per address)
  unsigned long long* st = stats ? stats + 4 * ((blockIdx.x + blockIdx.y * gridDim.x) & slot_mask) : nullptr;
  if (tile_misses<kSafe>(p, lattice(p.cx, x0, p.nx, p.hx), lattice(p.cx, x1, p.nx, p.hx),
                  lattice(p.cy, y0, p.ny, p.hy), lattice(p.cy, y1, p.ny, p.hy))) {
    if (tid == 0 && st) atomicAdd(&st[0], (unsigned long long)(shot * kRays));
    return;
  }

  const float m1 = in_vgpr(p.m1), m2 = in_vgpr(p.m2), sx = in_vgpr(p.sx), sy = in_vgpr(p.sy),
              kx = in_vgpr(p.kx), ky = in_vgpr(p.ky);
  const int hx = p.mx >> 1, hy = p.my >> 1;
  const float fhx = in_vgpr((float)hx), fhy = in_vgpr((float)hy);
  const float nan = __builtin_nanf("");
  float y[B], yy[B];
#pragma unroll
  for (int b = 0; b < B; ++b) {
    const int j = y0 + row_of(b);
    y[b] = j < p.row1 ? lattice(p.cy, j, p.ny, p.hy) : nan;  // NaN rays are never in the window
    yy[b] = y[b] * y[b];
  }
  // packed bin (by << 16 | bx), all ones when the ray is not binned
  uint32_t bins[A * B];
  uint32_t lo = 0xffffffffu, hi = 0u;  // packed bounds of the binned rays
  uint32_t n_in = 0, n_nf = 0, n_zero = 0;  // per wavefront

#pragma unroll
  for (int a = 0; a < A; ++a) {
    const int i = x0 + (kCoarse ? tx + 16 * a : tx * A + a);
    const float x = i < p.nx ? lattice(p.cx, i, p.nx, p.hx) : nan;
    const float d1 = x - p.x1, d2 = x - p.x2;
    const float d1s = d1 * d1, d2s = d2 * d2;
    // the B rays of the column together: their chains overlap, and one branch serves all
    float vx[B], vy[B];
    uint64_t in[B], any = 0;
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const float r1 = d1s + yy[b], r2 = d2s + yy[b];
      const float a1 = kSafe ? div_in_range(m1, r1) : m1 / r1;
      const float a2 = kSafe ? div_in_range(m2, r2) : m2 / r2;
      const float zx = (x - a1 * d1) - a2 * d2;
      const float zy = (y[b] - a1 * y[b]) - a2 * y[b];
      vx[b] = (zx - sx) * kx;
      vy[b] = (zy - sy) * ky;
      // one ballot per compare: the mask that the compare itself writes
      in[b] = __builtin_amdgcn_ballot_w64(fabsf(vx[b]) < fhx) & __builtin_amdgcn_ballot_w64(fabsf(vy[b]) < fhy);
      any |= in[b];
      if (!kSafe) {  // a padding ray (i or j past the end) is no ray
        const bool ray = i < p.nx && y0 + row_of(b) < p.row1;
        n_nf += __popcll(__builtin_amdgcn_ballot_w64(ray && !(isfinite(vx[b]) && isfinite(vy[b]))));
      }
      bins[a * B + b] = 0xffffffffu;
    }
    if (any) {  // uniform
#pragma unroll
      for (int b = 0; b < B; ++b) {
        n_in += __popcll(in[b]);
        // symmetric bin rule: v >= 0 (also -0) -> h + floor(v), v < 0 -> h - 1 - floor(-v);
        // v + 0 turns -0 into +0, and -1 - f is the complement of f
        const int bx = hx + ((int)fabsf(vx[b]) ^ (__float_as_int(vx[b] + 0.0f) >> 31));
        const int by = hy + ((int)fabsf(vy[b]) ^ (__float_as_int(vy[b] + 0.0f) >> 31));
        const uint32_t packed = ((uint32_t)by << 16) | (uint32_t)bx;
        const uint64_t axis = __builtin_amdgcn_ballot_w64(vy[b] == 0.0f) & in[b];
        uint64_t binned = in[b];
        if (axis) {  // uniform, and rare: rays on the window's horizontal centre line
          n_zero += __popcll(axis);
          if (kMirror) {  // such a ray and its mirror share the bin (bx, h)
            if ((axis >> lane) & 1)
              atomicAdd(&counts[(size_t)by * (size_t)p.mx + (size_t)bx], 2u);
            binned &= ~axis;
          }
        }
        const bool mine = __builtin_amdgcn_inverse_ballot_w64(binned);
        bins[a * B + b] = mine ? packed : 0xffffffffu;
        lo = pk_min(lo, bins[a * B + b]);
        hi = pk_max(hi, mine ? packed : 0u);
      }
    }
  }

  // workgroup bounding box of binned rays and the ray statistics
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    lo = pk_min(lo, (uint32_t)__shfl_xor((int)lo, o, kWave));
    hi = pk_max(hi, (uint32_t)__shfl_xor((int)hi, o, kWave));
  }
  if (lane == 0) {
    s_box[wave][0] = lo;
    s_box[wave][1] = hi;
    s_stat[wave][0] = n_in;
    s_stat[wave][1] = n_nf;
    s_stat[wave][2] = n_zero;
  }
  __syncthreads();
  lo = 0xffffffffu;
  hi = 0u;
  uint32_t tot[3] = {0u, 0u, 0u};
#pragma unroll
  for (int k = 0; k < RS_THREADS / kWave; ++k) {
    lo = pk_min(lo, s_box[k][0]);
    hi = pk_max(hi, s_box[k][1]);
#pragma unroll
    for (int q = 0; q < 3; ++q) tot[q] += s_stat[k][q];
  }
  if (tid == 0 && st) {
    const uint32_t n_out = (shot - tot[0] - tot[1]) * kRays;
    if (n_out) atomicAdd(&st[0], (unsigned long long)n_out);
    if (tot[1]) atomicAdd(&st[1], (unsigned long long)(tot[1] * kRays));
    if (tot[2]) atomicAdd(&st[2], (unsigned long long)(tot[2] * kRays));
  }
  if (lo == 0xffffffffu) return;  // no ray of this tile landed in the window

  const int bxmin = lo & 0xffff, bymin = lo >> 16;
  const int rows = (int)(hi >> 16) - bymin + 1;
  const int pitch = (int)(hi & 0xffff) - bxmin + 1;
  const int area = rows * pitch;
  const int top = 2 * hy - 1;  // mirror row of by is top - by
  if (area <= CAP) {
    for (int k = tid; k < area; k += RS_THREADS) hist[k] = 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < A * B; ++k) {
      const uint32_t bin = bins[k] - lo;  // no borrow between the halves: both are at least lo's
      if (bins[k] != 0xffffffffu) atomicAdd(&hist[__umul24(bin >> 16, pitch) + (bin & 0xffff)], 1u);
    }
    __syncthreads();
    auto merge = [&](int r, int c) {
      const uint32_t v = hist[r * pitch + c];
      if (v) {
        atomicAdd(&counts[(size_t)(bymin + r) * (size_t)p.mx + (size_t)(bxmin + c)], v);
        if (kMirror)
          atomicAdd(&counts[(size_t)(top - (bymin + r)) * (size_t)p.mx + (size_t)(bxmin + c)], v);
      }
    };
    // 16 x 16 bins a round, without a division a bin; a box that leaves more than half of
    // those lanes idle (a few columns or rows: a window of 2 x 32768 pixels took 126 us for 102)
    // goes 256 bins in a row a round
    if (((rows + 15) >> 4) * ((pitch + 15) >> 4) <= 2 * ((area + RS_THREADS - 1) / RS_THREADS)) {
      for (int r = ty; r < rows; r += 16)
        for (int c = tx; c < pitch; c += 16) merge(r, c);
    } else {
      for (int k = tid; k < area; k += RS_THREADS) merge(k / pitch, k % pitch);
    }
  } else {
#pragma unroll
    for (int k = 0; k < A * B; ++k) {
      if (bins[k] != 0xffffffffu) {
        const int bx = bins[k] & 0xffff;
        const int by = bins[k] >> 16;
        atomicAdd(&counts[(size_t)by * (size_t)p.mx + (size_t)bx], 1u);
        if (kMirror) atomicAdd(&counts[(size_t)(top - by) * (size_t)p.mx + (size_t)bx], 1u);
      }
    }
  }
}

// Adds the slots' statistics to the caller's three totals.
__global__ __launch_bounds__(64) void k_stats_sum(const unsigned long long* __restrict__ slots,
                                                  unsigned long long* __restrict__ stats) {
  const int q = threadIdx.x;
  if (q >= 3) return;
  unsigned long long t = 0;
  for (int k = 0; k < kStatSlots; ++k) t += slots[4 * k + q];
  if (t) atomicAdd(&stats[q], t);
}

// Normalise + convolve.  Taps are row-major over the stencil with the zero taps dropped
// on the host; neighbours clamp to the edge; acc accumulates the terms w[k] * count in
// tap order in binary32 (the first term alone, then one addition per tap) and
// A = acc * scale.  The kernels also reduce the largest count of the map (one atomic
// per workgroup).  Three forms of the same arithmetic:
//   * one tap at offset (0, 0) (a point source): elementwise, four pixels per thread
//     with 16-byte loads and stores;
//   * a stencil of half-width at most kNcHalo: a workgroup stages a 64 x 32 output tile
//     plus halo in LDS (sized to the stencil; counts converted to binary32 there, the
//     conversion every term applies), a thread sums four neighbouring pixels of two rows;
//     each wave issues all its staging loads (whole tile rows) before the first LDS store.  The tap builders cap the
//     half-width at 15 pixels;
//   * a stencil of reach at most one pixel (3 x 3) on a map whose width is a multiple
//     of 4 with 16-byte aligned buffers: no LDS.  A wavefront takes kR1Cols = 256
//     columns (four per lane, 16-byte loads and stores) and kR1Rows rows, loading the
//     rows y0 - 1 .. y0 + kR1Rows (clamped) and, by scalar loads, the column on each
//     side of its 256; a lane's outer neighbours come from the adjacent lanes by DPP
//     wavefront shifts, the wavefront's outer lanes taking the side columns.  The terms are added in raster order over the 3 x 3 neighbourhood with a
//     zero weight where the tap list has no tap: that is the tap order, and a zero term
//     (0 * count = +0) leaves a sum of non-negative terms unchanged, so the arithmetic
//     is that of the tap list.
constexpr int kNcTw = 64, kNcTh = 32, kNcHalo = 16;
constexpr int kR1Cols = 256, kR1Rows = 8;

__device__ __forceinline__ void nc_block_max(uint32_t cmax, uint32_t* maxc) {
  __shared__ uint32_t s_max[4];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) cmax = max(cmax, (uint32_t)__shfl_xor((int)cmax, o, kWave));
  if ((threadIdx.x & 63) == 0) s_max[threadIdx.x >> 6] = cmax;
  __syncthreads();
  if (threadIdx.x == 0 && maxc) atomicMax(maxc, max(max(s_max[0], s_max[1]), max(s_max[2], s_max[3])));
}

__global__ __launch_bounds__(256) void k_normalize_point(const uint32_t* __restrict__ counts,
                                                         float* __restrict__ map, int64_t npx,
                                                         bool vec4, const float* __restrict__ w,
                                                         float scale, uint32_t* __restrict__ maxc) {
  const float w0 = w[0];
  uint32_t cmax = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  if (vec4) {
    const uint4* c4 = reinterpret_cast<const uint4*>(counts);
    float4* m4 = reinterpret_cast<float4*>(map);
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < npx / 4; v += stride) {
      const uint4 c = c4[v];
      cmax = max(max(cmax, max(c.x, c.y)), max(c.z, c.w));
      m4[v] = make_float4((w0 * (float)c.x) * scale, (w0 * (float)c.y) * scale,
                          (w0 * (float)c.z) * scale, (w0 * (float)c.w) * scale);
    }
  } else {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < npx; v += stride) {
      const uint32_t c = counts[v];
      cmax = max(cmax, c);
      map[v] = (w0 * (float)c) * scale;
    }
  }
  nc_block_max(cmax, maxc);
}

// Taps of a row in groups of four columns from -rx on.
__host__ __device__ inline int nc_groups(int rx) { return (2 * rx + 4) / 4; }

// Tile staged in LDS with its halo; a thread sums 4 neighbouring pixels of two rows.  For a row
// of taps it takes them four at a time: eight values in registers serve 4 x 4 products, so
// LDS gives 16 bytes where a read a product took 64, and the products bound the time
// (2048^2 pixels, radii of 2 and 7 pixels: 95 us for both, now 75; one of 7 alone 74, now 53).  The weights are laid out densely, 0 where
// the list has no tap; a group's weights are read by all lanes at once.  Small stencils on maps
// whose rows are no multiple of 16 bytes are bound by memory: 4094^2 pixels, a radius of one, 51 us
// (60 with a store a pixel and with taps from a multiple of four columns on, which made two
// groups of three taps).  kPairs: stores of two pixels.
template <bool kPairs>
__global__ __launch_bounds__(256) void k_normalize_convolve_lds(
    const uint32_t* __restrict__ counts, float* __restrict__ map, int32_t mx, int32_t my,
    const float* __restrict__ w, const int32_t* __restrict__ off, int32_t ntaps, int32_t rx,
    int32_t ry, float scale, uint32_t* __restrict__ maxc) {
  extern __shared__ float4 nc_lds[];  // weights [2 ry + 1][groups], tile [kNcTh + 2 ry][16 + groups]
  __shared__ int s_first[2 * kNcHalo + 1], s_end[2 * kNcHalo + 1];
  const int x0 = blockIdx.x * kNcTw, y0 = blockIdx.y * kNcTh;
  const int hx = rx, groups = nc_groups(rx), rows = 2 * ry + 1;
  float4* wt4 = nc_lds;
  float4* tile4 = nc_lds + rows * groups;
  float* wt = (float*)wt4;
  float* tile = (float*)tile4;
  const int lw = kNcTw + 4 * groups, lh = kNcTh + 2 * ry;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // staging: wave w takes tile rows w, w + 4, ...; lane l the columns l and 64 + l; all
  // loads are issued before the first LDS store
  constexpr int kRowsPerWave = (kNcTh + 2 * kNcHalo + 3) / 4;
  uint32_t va[kRowsPerWave], vb[kRowsPerWave];
  const int gxa = min(max(x0 - hx + lane, 0), mx - 1), gxb = min(max(x0 - hx + 64 + lane, 0), mx - 1);
#pragma unroll
  for (int r = 0; r < kRowsPerWave; ++r) {
    const int ly = wave + 4 * r;
    va[r] = vb[r] = 0u;
    if (ly < lh) {  // uniform per wave
      const uint32_t* row = counts + (size_t)min(max(y0 - ry + ly, 0), my - 1) * mx;
      va[r] = row[gxa];
      if (lane < lw - 64) vb[r] = row[gxb];
    }
  }
  for (int k = threadIdx.x; k < rows * groups * 4; k += 256) wt[k] = 0.0f;
  if (threadIdx.x < rows) {
    s_first[threadIdx.x] = 4 * groups;
    s_end[threadIdx.x] = 0;
  }
  uint32_t cmax = 0;
  const bool own_a = lane >= hx && x0 - hx + lane < mx;  // own columns: [hx, hx + 64)
  const bool own_b = lane < hx && x0 - hx + 64 + lane < mx;  // and [64, 64 + hx)
#pragma unroll
  for (int r = 0; r < kRowsPerWave; ++r) {
    const int ly = wave + 4 * r;
    if (ly < lh) {
      tile[ly * lw + lane] = (float)va[r];
      if (lane < lw - 64) tile[ly * lw + 64 + lane] = (float)vb[r];
      if (ly >= ry && ly < ry + kNcTh && y0 - ry + ly < my) {
        if (own_a) cmax = max(cmax, va[r]);
        if (own_b) cmax = max(cmax, vb[r]);
      }
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k < ntaps; k += 256) {
    const int c = off[2 * k] + hx, row = off[2 * k + 1] + ry;
    wt[row * groups * 4 + c] = w[k];
    atomicMin(&s_first[row], c);
    atomicMax(&s_end[row], c + 1);
  }
  __syncthreads();
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float acc[2][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[0][i] = acc[1][i] = 0.0f;
  for (int row = 0; row < rows; ++row) {
    const int first = uniform(s_first[row]), end = uniform(s_end[row]);
    if (first >= end) continue;
    const float4* t = tile4 + (ty + row) * (lw / 4) + tx;
    const int step = 16 * (lw / 4);
    float4 a = t[first / 4], b = t[step + first / 4];
    for (int g = first / 4; 4 * g < end; ++g) {
      const float4 wg = wt4[row * groups + g], a1 = t[g + 1], b1 = t[step + g + 1];
      const float va[8] = {a.x, a.y, a.z, a.w, a1.x, a1.y, a1.z, a1.w};
      const float vb[8] = {b.x, b.y, b.z, b.w, b1.x, b1.y, b1.z, b1.w};
      const float u[4] = {wg.x, wg.y, wg.z, wg.w};
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (4 * g + q >= first && 4 * g + q < end) {  // uniform
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            acc[0][i] = acc[0][i] + u[q] * va[q + i];
            acc[1][i] = acc[1][i] + u[q] * vb[q + i];
          }
        }
      a = a1;
      b = b1;
    }
  }
  const int gx = x0 + 4 * tx;
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int gy = y0 + ty + 16 * r;
    if (gy >= my) continue;
    float* o = map + (size_t)gy * mx + gx;
#pragma unroll
    for (int i = 0; i < 4; i += kPairs ? 2 : 1) {
      if (gx + i >= mx) continue;
      if (kPairs)  // mx is even and the map 8-byte aligned
        *reinterpret_cast<float2*>(o + i) = make_float2(acc[r][i] * scale, acc[r][i + 1] * scale);
      else
        o[i] = acc[r][i] * scale;
    }
  }
  nc_block_max(cmax, maxc);
}

// v of lane l - 1 (lane 0 takes lo) and of lane l + 1 (lane 63 takes hi), by DPP
// wavefront shifts.
__device__ __forceinline__ float from_lane_below(float v, float lo) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(lo), __float_as_int(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float from_lane_above(float v, float hi) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(hi), __float_as_int(v), 0x130, 0xf, 0xf, false));
}

__global__ __launch_bounds__(256) void k_normalize_convolve_r1(
    const uint32_t* __restrict__ counts, float* __restrict__ map, int32_t mx, int32_t my,
    const float* __restrict__ w, const int32_t* __restrict__ off, int32_t ntaps, float scale,
    uint32_t* __restrict__ maxc) {
  const int lane = threadIdx.x & (kWave - 1);
  const int ncx = (mx + kR1Cols - 1) / kR1Cols;
  // the wave's index, read from the first lane so that everything derived from it (tile
  // origin, row offsets, the neighbouring columns' loads) stays in scalar registers;
  // 32-bit arithmetic: the launcher admits maps below 2^30 pixels
  const int item = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int x0 = item % ncx * kR1Cols;
  const int y0 = item / ncx * kR1Rows;
  uint32_t cmax = 0;
  if (y0 < my) {  // uniform per wave (the last workgroup's waves may lie past the map)
    // the 3 x 3 weights in raster order (uniform), zero where there is no tap
    float W[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) W[i] = 0.0f;
    for (int k = 0; k < ntaps; ++k) {
      const int i = (off[2 * k + 1] + 1) * 3 + off[2 * k] + 1;
      const float wk = w[k];
#pragma unroll
      for (int j = 0; j < 9; ++j) W[j] = j == i ? wk : W[j];
    }
    const int xq = x0 + 4 * lane;  // the lane's four columns xq .. xq + 3
    const bool own = xq < mx;      // mx % 4 == 0: a quad lies wholly inside or outside
    const bool has_right = xq + 4 < mx;
    const uint32_t qx = (uint32_t)min(xq, mx - 4);
    // the columns beside the wavefront's 256, clamped to the map (uniform: scalar loads)
    const uint32_t hl = (uint32_t)max(x0 - 1, 0), hr = (uint32_t)min(x0 + kR1Cols, mx - 1);
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    u4 q[kR1Rows + 2];  // all the rows' loads in flight before the first use
    uint32_t ql[kR1Rows + 2], qr[kR1Rows + 2];
#pragma unroll
    for (int r = 0; r < kR1Rows + 2; ++r) {
      const uint32_t row = (uint32_t)min(max(y0 - 1 + r, 0), my - 1) * (uint32_t)mx;
      q[r] = ldg(reinterpret_cast<const u4*>(counts), (row + qx) >> 2);
      ql[r] = counts[row + hl];
      qr[r] = counts[row + hr];
    }
    // per row: the lane's four values and their outer neighbours (the left one of column
    // 0 is column 0 itself through the clamped load; the right one of column mx - 1 is
    // column mx - 1 itself)
    float V[kR1Rows + 2][6];
#pragma unroll
    for (int r = 0; r < kR1Rows + 2; ++r) {
      V[r][1] = (float)q[r].x;
      V[r][2] = (float)q[r].y;
      V[r][3] = (float)q[r].z;
      V[r][4] = (float)q[r].w;
      V[r][0] = from_lane_below(V[r][4], (float)ql[r]);
      const float rn = from_lane_above(V[r][1], (float)qr[r]);
      V[r][5] = has_right ? rn : V[r][4];
    }
#pragma unroll
    for (int r = 0; r < kR1Rows; ++r) {
      float o[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {  // column xq + j: values V[.][j .. j + 2]
        float acc = W[0] * V[r][j];
        acc = acc + W[1] * V[r][j + 1];
        acc = acc + W[2] * V[r][j + 2];
        acc = acc + W[3] * V[r + 1][j];
        acc = acc + W[4] * V[r + 1][j + 1];
        acc = acc + W[5] * V[r + 1][j + 2];
        acc = acc + W[6] * V[r + 2][j];
        acc = acc + W[7] * V[r + 2][j + 1];
        acc = acc + W[8] * V[r + 2][j + 2];
        o[j] = acc * scale;
      }
      const int y = y0 + r;
      if (own && y < my) {
        reinterpret_cast<float4*>(map)[((uint32_t)y * (uint32_t)mx + (uint32_t)xq) >> 2] =
            make_float4(o[0], o[1], o[2], o[3]);
        const u4 c = q[r + 1];
        cmax = max(cmax, max(max(c.x, c.y), max(c.z, c.w)));
      }
    }
  }
  nc_block_max(cmax, maxc);
}

// Exclusive prefix sum of nb counters in place by one 1024-lane workgroup: each lane
// sums a contiguous chunk, a Hillis-Steele scan over the 1024 chunk sums, then each
// lane rewrites its chunk.
__global__ __launch_bounds__(1024) void k_scan_u32(uint32_t* v, int64_t nb) {
  __shared__ uint32_t part[1024];
  const int64_t per = (nb + 1023) / 1024;
  const int64_t b0 = threadIdx.x * per, b1 = min(b0 + per, nb);
  uint32_t sum = 0;
  for (int64_t b = b0; b < b1; ++b) sum += v[b];
  part[threadIdx.x] = sum;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const uint32_t x = threadIdx.x >= (unsigned)off ? part[threadIdx.x - off] : 0u;
    __syncthreads();
    part[threadIdx.x] += x;
    __syncthreads();
  }
  uint32_t run = part[threadIdx.x] - sum;
  for (int64_t b = b0; b < b1; ++b) {
    const uint32_t h = v[b];
    v[b] = run;
    run += h;
  }
}

// Adds one to h[k] for every active lane and returns the lane's place: h[k] before, plus the
// lanes below with the same k.  Lanes that share the first active lane's k, then the first of
// the others', add together: neighbours mostly do, and the atomics of one address go one
// after another (8192 keys in order over 8 bins: 26 us each alone).
__device__ __forceinline__ uint32_t bucket_add(uint32_t* h, uint32_t k, bool act) {
  const int lane = threadIdx.x & (kWave - 1);
  uint32_t place = 0;
#pragma unroll
  for (int round = 0; round < 2; ++round) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(act);
    if (m == 0) return place;
    const int first = __builtin_ctzll(m);
    const uint32_t k0 = (uint32_t)__builtin_amdgcn_readlane((int)k, first);
    const bool mine = act && k == k0;
    const uint64_t same = __builtin_amdgcn_ballot_w64(mine);
    uint32_t at = 0;
    if (lane == first) at = atomicAdd(&h[k0], (uint32_t)__popcll(same));
    at = (uint32_t)__builtin_amdgcn_readlane((int)at, first);
    if (mine) place = at + (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
    act = act && !mine;
  }
  if (act) place = atomicAdd(&h[k], 1u);
  return place;
}

__global__ void k_bucket_count(const uint32_t* __restrict__ key, int64_t n, uint32_t* hist) {
  for (int64_t i0 = blockIdx.x * (int64_t)blockDim.x; i0 < n; i0 += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = i0 + threadIdx.x;
    bucket_add(hist, i < n ? key[i] : 0u, i < n);
  }
}

__global__ void k_bucket_scatter(const uint32_t* __restrict__ key, int64_t n, uint32_t* cursor,
                                 int32_t* order) {
  for (int64_t i0 = blockIdx.x * (int64_t)blockDim.x; i0 < n; i0 += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = i0 + threadIdx.x;
    const uint32_t at = bucket_add(cursor, i < n ? key[i] : 0u, i < n);
    if (i < n) order[at] = (int32_t)i;
  }
}

}  // namespace

hipError_t launch_bucket_order(const uint32_t* key, int64_t n, int32_t nbins, uint32_t* hist,
                               int32_t* order, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (n > INT32_MAX || nbins <= 0) return hipErrorInvalidValue;
  hipError_t e = launch_fill_u32(hist, (size_t)nbins, 0u, st);
  if (e != hipSuccess) return e;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_bucket_count, dim3((unsigned)blocks), dim3(256), 0, st, key, n, hist);
  e = launch_scan_u32(hist, nbins, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_bucket_scatter, dim3((unsigned)blocks), dim3(256), 0, st, key, n, hist, order);
  return hipGetLastError();
}

hipError_t launch_scan_u32(uint32_t* v, int64_t nb, hipStream_t st) {
  if (nb <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_scan_u32, dim3(1), dim3(1024), 0, st, v, nb);
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const size_t quads = (uintptr_t)p % 16 == 0 ? n / 4 : 0;
  const size_t blocks = std::min<size_t>(65536, ((quads ? quads : n) + 255) / 256);
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, p, n, quads, v);
  return hipGetLastError();
}

hipError_t launch_fill_u64(uint64_t* p, size_t n, uint64_t v, hipStream_t st) {
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)blocks), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

namespace {

// Whether the short division holds for rows [row0, row1) (see k_rayshoot): |y| is smallest
// beside the lattice's crossing of y = 0, which the rows around it bracket, and r_k >= y^2.
bool safe_rows(const RayParams& p, int32_t row0, int32_t row1) {
  auto y = [&](int32_t j) { return std::fabs(p.cy + ((float)(j - (p.ny >> 1)) + 0.5f) * p.hy); };
  const double c = 0.5 * p.ny - 0.5 - (double)p.cy / p.hy;
  float ymin = std::min(y(row0), y(row1 - 1));
  for (int d = -3; d <= 3; ++d) {
    const double j = std::floor(c) + d;
    if (j >= row0 && j < row1) ymin = std::min(ymin, y((int32_t)j));
  }
  const float xmax = std::fabs(p.cx) + p.hx * p.nx + std::max(std::fabs(p.x1), std::fabs(p.x2));
  const float ymax = std::fabs(p.cy) + p.hy * p.ny;
  auto scale = [](float k) { return k >= 0x1p-40f && k <= 0x1p40f; };
  return ymin >= 0x1p-19f && xmax <= 0x1p19f && ymax <= 0x1p19f && std::fabs(p.sx) <= 0x1p40f &&
         std::fabs(p.sy) <= 0x1p40f && scale(p.kx) && scale(p.ky) && (p.m2 == 0.0f || p.m2 >= 0x1p-40f);
}

template <bool kMirror, bool kSafe>
hipError_t shoot_tiles(const RayParams& p, uint32_t* counts, unsigned long long* stats, uint32_t slot_mask,
                       int num_cu, hipStream_t st) {
  // 128 x 64 rays a workgroup, 32 a thread; 64 x 32 where the lattice is too small to give
  // every CU eight such tiles (3200^2 rays into 512^2: 12 against 51 us) or so coarse that
  // 128 x 64 rays cover more than 512 pixels without a lens (near one they spread over
  // several times as many, and a box beyond RS_CAP bins counts ray by ray; 7000 x 5210 rays,
  // 2.4 a pixel side: 50 against 265 us).  Where 64 x 32 rays cover more than 512 pixels the
  // coarse form (neighbouring rays on neighbouring lanes, 24 KiB of bins): 12000^2 rays over twice
  // the window's width, 0.5 / 0.75 / 1 / 1.5 rays a pixel side, 1.48 / 1.20 / 0.72 / 0.29 ms for 2.60
  // / 2.20 / 1.29 / 0.49; at 2 (288 pixels) 0.26 without it, and 32 KiB of bins slower for finer ones.
  // 32768^2 rays into 2048^2: 373 us with the large tile, 537 with the small one; 128 x 128 rays take
  // 515 (95 VGPRs, larger boxes).
  const float cover = 128.0f * 64.0f * p.hx * p.kx * p.hy * p.ky;
  const int rows = p.row1 - p.row0;
  auto tiles = [&](int tx, int ty) { return dim3((p.nx + tx - 1) / tx, (rows + ty - 1) / ty); };
  const dim3 big = tiles(128, 64), small = tiles(64, 32);
  if ((int64_t)big.x * big.y >= 8 * (int64_t)num_cu && cover <= 512.0f) {
    hipLaunchKernelGGL((k_rayshoot<kMirror, kSafe, 8, 4, false>), big, dim3(RS_THREADS), 0, st, p, counts, stats,
                       slot_mask);
  } else if (cover > 4.0f * 512.0f) {
    hipLaunchKernelGGL((k_rayshoot<kMirror, kSafe, 4, 2, true>), small, dim3(RS_THREADS), 0, st, p, counts,
                       stats, slot_mask);
  } else {
    hipLaunchKernelGGL((k_rayshoot<kMirror, kSafe, 4, 2, false>), small, dim3(RS_THREADS), 0, st, p, counts, stats,
                       slot_mask);
  }
  return hipGetLastError();
}

// Rows [row0, row1) of p, each ray shot once (kMirror false) or, for rows of the upper
// half whose mirror rows are part of the call, once for the pair (kMirror true).
template <bool kMirror>
hipError_t shoot_rows(RayParams p, int32_t row0, int32_t row1, uint32_t* counts,
                      unsigned long long* stats, uint32_t slot_mask, int num_cu, hipStream_t st) {
  if (row1 <= row0) return hipSuccess;
  p.row0 = row0;
  p.row1 = row1;
  return safe_rows(p, row0, row1) ? shoot_tiles<kMirror, true>(p, counts, stats, slot_mask, num_cu, st)
                                  : shoot_tiles<kMirror, false>(p, counts, stats, slot_mask, num_cu, st);
}

}  // namespace

hipError_t launch_rayshoot(const RayParams& p, uint32_t* counts, unsigned long long* stats,
                           unsigned long long* slots, int num_cu, hipStream_t st) {
  if (p.row1 <= p.row0) return hipSuccess;
  hipError_t e = hipSuccess;
  const bool in_slots = stats && slots;
  unsigned long long* ss = in_slots ? slots : stats;
  const uint32_t mask = in_slots ? kStatSlots - 1 : 0u;
  if (in_slots) e = launch_fill_u64((uint64_t*)ss, 4 * kStatSlots, 0ull, st);
  // Mirror pairs need a lattice and a window centred on y = 0 and an even row count;
  // the rows paired inside [row0, row1) form [a, b) with a + b = ny.
  const int32_t a = std::max(p.row0, p.ny - p.row1), b = std::min(p.row1, p.ny - p.row0);
  if (e != hipSuccess) return e;
  if (!(p.cy == 0.0f && p.sy == 0.0f && (p.ny & 1) == 0 && a < b)) {
    e = shoot_rows<false>(p, p.row0, p.row1, counts, ss, mask, num_cu, st);
  } else {
    e = shoot_rows<true>(p, p.ny / 2, b, counts, ss, mask, num_cu, st);
    if (e == hipSuccess) e = shoot_rows<false>(p, p.row0, a, counts, ss, mask, num_cu, st);
    if (e == hipSuccess) e = shoot_rows<false>(p, b, p.row1, counts, ss, mask, num_cu, st);
  }
  if (e == hipSuccess && in_slots) {
    hipLaunchKernelGGL(k_stats_sum, dim3(1), dim3(64), 0, st, ss, stats);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_normalize_convolve(const uint32_t* counts, float* map, int32_t mx, int32_t my,
                                     const float* d_w, const int32_t* d_off, int32_t ntaps,
                                     int32_t rx, int32_t ry, float scale, uint32_t* d_maxc,
                                     hipStream_t st) {
  if (mx <= 0 || my <= 0 || ntaps < 1 || rx < 0 || ry < 0) return hipErrorInvalidValue;
  if (rx == 0 && ry == 0) {
    if (ntaps != 1) return hipErrorInvalidValue;  // only the tap (0, 0) has no reach
    const int64_t npx = (int64_t)mx * my;
    const bool vec4 = npx % 4 == 0 && ((uintptr_t)counts % 16) == 0 && ((uintptr_t)map % 16) == 0;
    int64_t blocks = ((vec4 ? npx / 4 : npx) + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(k_normalize_point, dim3((unsigned)blocks), dim3(256), 0, st, counts, map, npx,
                       vec4, d_w, scale, d_maxc);
  } else if (rx <= 1 && ry <= 1 && (int64_t)mx * my < ((int64_t)1 << 30) && mx % 4 == 0 &&
             ((uintptr_t)counts % 16) == 0 && ((uintptr_t)map % 16) == 0) {
    if (ntaps > 9) return hipErrorInvalidValue;
    const int64_t waves = (int64_t)((mx + kR1Cols - 1) / kR1Cols) * ((my + kR1Rows - 1) / kR1Rows);
    hipLaunchKernelGGL(k_normalize_convolve_r1, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, st,
                       counts, map, mx, my, d_w, d_off, ntaps, scale, d_maxc);
  } else {
    if (rx > kNcHalo || ry > kNcHalo) return hipErrorInvalidValue;
    const size_t lds = 16 * (size_t)nc_groups(rx) * (2 * ry + 1) +
                       sizeof(float) * (kNcTw + 4 * nc_groups(rx)) * (kNcTh + 2 * ry);
    dim3 grid((mx + kNcTw - 1) / kNcTw, (my + kNcTh - 1) / kNcTh);
    auto* kernel = mx % 2 == 0 && ((uintptr_t)map % 8) == 0 ? k_normalize_convolve_lds<true> : k_normalize_convolve_lds<false>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), lds, st, counts, map, mx, my, d_w, d_off, ntaps, rx, ry, scale, d_maxc);
  }
  return hipGetLastError();
}

}  // namespace morse
