// grid_build.hip -- GPU build of the uniform grid (the "Preprocess" phase of
// the paper's Table 5): FP64 scene packing, bounds reduction, per-cell
// counting, exclusive prefix scan, scatter of primitive references, and an
// in-cell sort that makes the reference order deterministic.
//
// Compiled with -ffp-contract=off: the cell lists must equal, bit for bit,
// those of the grid definition (primitive boxes widened by delta, spheres
// kept only where their centre lies within r of the widened cell box).
#include <algorithm>

#include "tr_internal.h"

namespace {

using namespace trd;

constexpr int kBlock = 256;

__device__ __forceinline__ void prim_box(const trh::BuildArgs &a, int64_t k, double lo[3],
                                         double hi[3]) {
  if (k < a.n_s) {
    const double4 s = a.sph64[k];
    lo[0] = s.x - s.w; lo[1] = s.y - s.w; lo[2] = s.z - s.w;
    hi[0] = s.x + s.w; hi[1] = s.y + s.w; hi[2] = s.z + s.w;
  } else if (k >= (int64_t)a.n_s + a.n_c) {  // triangle: min/max of its vertices
    const int64_t m = k - a.n_s - a.n_c;
    const double4 A = a.triA64[m], B = a.triB64[m], C = a.triC64[m];
    const double av[3] = {A.x, A.y, A.z}, bv[3] = {B.x, B.y, B.z}, cv[3] = {C.x, C.y, C.z};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      double mn = av[q], mx = av[q];
      mn = bv[q] < mn ? bv[q] : mn;
      mx = bv[q] > mx ? bv[q] : mx;
      mn = cv[q] < mn ? cv[q] : mn;
      mx = cv[q] > mx ? cv[q] : mx;
      lo[q] = mn;
      hi[q] = mx;
    }
  } else {
    const int64_t m = k - a.n_s;
    const double4 A = a.cylA64[m], B = a.cylB64[m];
    const double av[3] = {A.x, A.y, A.z}, bv[3] = {B.x, B.y, B.z};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const double mn = av[q] < bv[q] ? av[q] : bv[q];
      const double mx = av[q] < bv[q] ? bv[q] : av[q];
      lo[q] = mn - A.w;
      hi[q] = mx + A.w;
    }
  }
}

__device__ __forceinline__ int32_t cell_coord(const trh::BuildArgs &a, int q, double x) {
  const double f = floor((x - a.lo[q]) * a.inv[q]);
  if (!(f >= 0.0)) return 0;
  if (f > (double)(a.res[q] - 1)) return a.res[q] - 1;
  return (int32_t)f;
}

__device__ __forceinline__ bool sphere_in_cell(const trh::BuildArgs &a, const double4 s,
                                               int32_t ix, int32_t iy, int32_t iz) {
  const int32_t idx[3] = {ix, iy, iz};
  const double c[3] = {s.x, s.y, s.z};
  double d2 = 0.0;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const double cl = (a.lo[q] + (double)idx[q] * a.h[q]) - a.delta;
    const double ch = (a.lo[q] + (double)(idx[q] + 1) * a.h[q]) + a.delta;
    double e = 0.0;
    if (c[q] < cl) e = cl - c[q];
    else if (c[q] > ch) e = c[q] - ch;
    d2 = d2 + e * e;
  }
  return d2 <= s.w * s.w;
}

// Visit every cell primitive k is listed in.  kLanes lanes share a primitive:
// lane g takes the cells of its box whose linear index (x fastest) is g, g +
// kLanes, ...  A protein-sized scene has only tens of thousands of primitives,
// too few for one thread each to fill the chip.
constexpr int kLanes = 16;

template <class F>
__device__ __forceinline__ void for_prim_cells(const trh::BuildArgs &a, int64_t k, int g,
                                               F &&visit) {
  double lo[3], hi[3];
  prim_box(a, k, lo, hi);
  int32_t c0[3], n[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    c0[q] = cell_coord(a, q, lo[q] - a.delta);
    n[q] = cell_coord(a, q, hi[q] + a.delta) - c0[q] + 1;
  }
  const bool sph = k < a.n_s;
  double4 s = make_double4(0, 0, 0, 0);
  if (sph) s = a.sph64[k];
  // first cell of this lane, then steps of kLanes along x with carries
  int32_t ix = g, iy = 0, iz = 0;
  while (ix >= n[0]) { ix -= n[0]; ++iy; }
  while (iy >= n[1]) { iy -= n[1]; ++iz; }
  while (iz < n[2]) {
    const int32_t x = c0[0] + ix, y = c0[1] + iy, z = c0[2] + iz;
    if (!sph || sphere_in_cell(a, s, x, y, z))
      visit((uint32_t)(((int64_t)z * a.res[1] + y) * a.res[0] + x));
    ix += kLanes;
    while (ix >= n[0]) {
      ix -= n[0];
      if (++iy == n[1]) { iy = 0; ++iz; }
    }
  }
}

__global__ void k_pack(const trh::PackArgs P) {
  const int64_t n_s = P.n_s, n_c = P.n_c;
  const double *sc = P.sc, *sr = P.sr, *ca = P.ca, *cb = P.cb, *cr = P.cr;
  const float *srgb = P.srgb, *sop = P.sop, *crgb = P.crgb, *cop = P.cop;
  double4 *sph64 = P.sph64, *cylA64 = P.cylA64, *cylW64 = P.cylW64, *cylB64 = P.cylB64;
  float4 *albedo = P.albedo;
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_s + n_c && k < n_s + n_c + P.n_t) {
    const int64_t m = k - n_s - n_c;
    P.triA64[m] = make_double4(P.tv0[3 * m], P.tv0[3 * m + 1], P.tv0[3 * m + 2], 0.0);
    P.triB64[m] = make_double4(P.tv1[3 * m], P.tv1[3 * m + 1], P.tv1[3 * m + 2], 0.0);
    P.triC64[m] = make_double4(P.tv2[3 * m], P.tv2[3 * m + 1], P.tv2[3 * m + 2], 0.0);
    albedo[k] = make_float4(P.trgb[3 * m], P.trgb[3 * m + 1], P.trgb[3 * m + 2],
                            P.top ? P.top[m] : 1.0f);
  }
  if (k < n_s) {
    sph64[k] = make_double4(sc[3 * k], sc[3 * k + 1], sc[3 * k + 2], sr[k]);
    albedo[k] = make_float4(srgb[3 * k], srgb[3 * k + 1], srgb[3 * k + 2], sop ? sop[k] : 1.0f);
  } else if (k < n_s + n_c) {
    const int64_t m = k - n_s;
    const double a[3] = {ca[3 * m], ca[3 * m + 1], ca[3 * m + 2]};
    const double b[3] = {cb[3 * m], cb[3 * m + 1], cb[3 * m + 2]};
    const double ab[3] = {b[0] - a[0], b[1] - a[1], b[2] - a[2]};
    const double L = sqrt((ab[0] * ab[0] + ab[1] * ab[1]) + ab[2] * ab[2]);
    cylA64[m] = make_double4(a[0], a[1], a[2], cr[m]);
    cylW64[m] = make_double4(ab[0] / L, ab[1] / L, ab[2] / L, L);
    cylB64[m] = make_double4(b[0], b[1], b[2], 0.0);
    albedo[k] = make_float4(crgb[3 * m], crgb[3 * m + 1], crgb[3 * m + 2], cop ? cop[m] : 1.0f);
  }
}

// FP32 copies for the wavefront walk, with positions relative to the centre of
// the grid box (the FP32 frame: the smallest magnitudes, so the least rounding,
// wherever the scene sits).  Spheres and cylinders carry their squared radius
// (squared in FP64, then rounded), which is all the FP32 tests use.
//
// The same pass takes the scene's bounding radius about that centre: the
// largest distance from it of any point of any primitive (a sphere's centre
// distance plus its radius, a cylinder's farther end plus its radius, a
// triangle's farthest vertex), in FP64, as the bit pattern of a non-negative
// double (whose order is the integer order of its bits) maxed into *rmax64
// (zero on entry): one atomic per workgroup.
__device__ __forceinline__ double dist3(double x, double y, double z) {
  return sqrt((x * x + y * y) + z * z);
}

__device__ __forceinline__ void pack32(const trh::BuildArgs &a, const trh::Pack32Args &P, int64_t k) {
  const int64_t n_s = a.n_s, n_c = a.n_c;
  const double4 *sph64 = a.sph64, *cylA64 = a.cylA64, *cylB64 = a.cylB64, *cylW64 = P.cylW64;
  float4 *sph32 = P.sph32, *cylA32 = P.cylA32, *cylW32 = P.cylW32;
  const double ox = P.origin[0], oy = P.origin[1], oz = P.origin[2];
  double ext = 0.0;  // this primitive's farthest point from the centre
  if (k >= n_s + n_c && k < n_s + n_c + a.n_t) {
    // triangle: v0 in the FP32 frame, its edges (differences taken in FP64),
    // and |e1 x e2| (the scale of the determinant) in v0's fourth word
    const int64_t m = k - n_s - n_c;
    const double4 A = a.triA64[m], B = a.triB64[m], C = a.triC64[m];
    const double e1[3] = {B.x - A.x, B.y - A.y, B.z - A.z};
    const double e2[3] = {C.x - A.x, C.y - A.y, C.z - A.z};
    const double nx = e1[1] * e2[2] - e1[2] * e2[1];
    const double ny = e1[2] * e2[0] - e1[0] * e2[2];
    const double nz = e1[0] * e2[1] - e1[1] * e2[0];
    P.tri32[3 * m] = make_float4((float)(A.x - ox), (float)(A.y - oy), (float)(A.z - oz),
                                 (float)sqrt((nx * nx + ny * ny) + nz * nz));
    ext = fmax(dist3(A.x - ox, A.y - oy, A.z - oz),
               fmax(dist3(B.x - ox, B.y - oy, B.z - oz), dist3(C.x - ox, C.y - oy, C.z - oz)));
    P.tri32[3 * m + 1] = make_float4((float)e1[0], (float)e1[1], (float)e1[2], 0.0f);
    P.tri32[3 * m + 2] = make_float4((float)e2[0], (float)e2[1], (float)e2[2], 0.0f);
  }
  if (k < n_s) {
    const double4 s = sph64[k];
    sph32[k] = make_float4((float)(s.x - ox), (float)(s.y - oy), (float)(s.z - oz), (float)(s.w * s.w));
    ext = dist3(s.x - ox, s.y - oy, s.z - oz) + s.w;
  } else if (k < n_s + n_c) {
    const int64_t m = k - n_s;
    const double4 a = cylA64[m], w = cylW64[m];
    cylA32[m] = make_float4((float)(a.x - ox), (float)(a.y - oy), (float)(a.z - oz), (float)(a.w * a.w));
    cylW32[m] = make_float4((float)w.x, (float)w.y, (float)w.z, (float)w.w);
    const double4 b = cylB64[m];
    // The bounding sphere of the (open) cylinder, after the spheres: centre
    // the axis midpoint, squared radius (L/2)^2 + rho^2, padded by 2^-9 and
    // rounded up, so the cylinder stays inside the FP32 sphere by a margin
    // far above the FP32 rounding of the test against it.
    const double hl = 0.5 * w.w;
    const float bb = (float)((hl * hl + a.w * a.w) * (1.0 + 0x1p-9));
    sph32[k] = make_float4((float)(0.5 * (a.x + b.x) - ox), (float)(0.5 * (a.y + b.y) - oy),
                           (float)(0.5 * (a.z + b.z) - oz), nextafterf(bb, INFINITY));
    ext = fmax(dist3(a.x - ox, a.y - oy, a.z - oz), dist3(b.x - ox, b.y - oy, b.z - oz)) + a.w;
  }
  // every thread gets here (no early return): the workgroup's maximum
  __shared__ double wave_ext[kBlock / 64];
  for (int off = 32; off > 0; off >>= 1) ext = fmax(ext, __shfl_xor(ext, off, 64));
  if ((threadIdx.x & 63) == 0) wave_ext[threadIdx.x >> 6] = ext;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < kBlock / 64; ++q) ext = fmax(ext, wave_ext[q]);
    if (ext > 0.0) atomicMax(P.rmax64, (unsigned long long)__double_as_longlong(ext));
  }
}

// Per-block min/max of primitive boxes -> scratch[block*6 .. +6].
__global__ __launch_bounds__(kBlock) void k_bounds_partial(const trh::BuildArgs a, double *part) {
  __shared__ double red[6][kBlock];
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  const int64_t N = (int64_t)a.n_s + a.n_c + a.n_t;
  for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < N;
       k += (int64_t)gridDim.x * kBlock) {
    double bl[3], bh[3];
    prim_box(a, k, bl, bh);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      lo[q] = bl[q] < lo[q] ? bl[q] : lo[q];
      hi[q] = bh[q] > hi[q] ? bh[q] : hi[q];
    }
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    red[q][threadIdx.x] = lo[q];
    red[3 + q][threadIdx.x] = hi[q];
  }
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const double x = red[q][threadIdx.x + s];
        if (x < red[q][threadIdx.x]) red[q][threadIdx.x] = x;
        const double y = red[3 + q][threadIdx.x + s];
        if (y > red[3 + q][threadIdx.x]) red[3 + q][threadIdx.x] = y;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < 6) part[(int64_t)blockIdx.x * 6 + threadIdx.x] = red[threadIdx.x][0];
}

__global__ __launch_bounds__(kBlock) void k_bounds_final(const double *part, int32_t n_part,
                                                         double *out6) {
  __shared__ double red[6][kBlock];
  double v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  for (int32_t b = threadIdx.x; b < n_part; b += kBlock) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const double x = part[(int64_t)b * 6 + q];
      const double y = part[(int64_t)b * 6 + 3 + q];
      v[q] = x < v[q] ? x : v[q];
      v[3 + q] = y > v[3 + q] ? y : v[3 + q];
    }
  }
#pragma unroll
  for (int q = 0; q < 6; ++q) red[q][threadIdx.x] = v[q];
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const double x = red[q][threadIdx.x + s];
        if (x < red[q][threadIdx.x]) red[q][threadIdx.x] = x;
        const double y = red[3 + q][threadIdx.x + s];
        if (y > red[3 + q][threadIdx.x]) red[3 + q][threadIdx.x] = y;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < 6) out6[threadIdx.x] = red[threadIdx.x][0];
}

__global__ void k_fill_u32(uint32_t *p, int64_t n, uint32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// Zero the per-cell counts (and the two words of total64).
__global__ void k_grid_init(uint32_t *count, int64_t n, unsigned long long *total64) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t i = t; i < n; i += (int64_t)gridDim.x * blockDim.x) count[i] = 0u;
  if (t < 2) total64[t] = 0ull;
}

// Per-cell counts (workgroups below n_count) and the FP32 copies (the rest):
// both need only the grid's parameters, so they share a launch.  The
// references are totalled by the scan: an atomic per workgroup on one word,
// 7 ns each, was half of the counting of 10^6 objects (810 us).
__global__ __launch_bounds__(kBlock) void k_count_pack(const trh::BuildArgs a, const trh::Pack32Args P,
                                                       uint32_t n_count, uint32_t *count) {
  if (blockIdx.x < n_count) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t k = t / kLanes;
    if (k < (int64_t)a.n_s + a.n_c + a.n_t)
      for_prim_cells(a, k, (int)(t % kLanes), [&](uint32_t c) { atomicAdd(&count[c], 1u); });
  } else {
    pack32(a, P, (int64_t)(blockIdx.x - n_count) * kBlock + threadIdx.x);
  }
}

// Whether the references and the walk lists fit their buffers: the kernels
// after the scan are launched before the host has read the total, and leave
// everything alone when it does not fit (the host then grows the buffers and
// launches them again).
__device__ __forceinline__ bool fits(const unsigned long long *total64, unsigned long long cap) {
  return total64[0] <= cap;
}

__global__ void k_scatter(trh::BuildArgs a, const uint32_t *cell_begin, uint32_t *cursor,
                          uint32_t *refs, const unsigned long long *total64, unsigned long long cap) {
  if (!fits(total64, cap)) return;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t k = t / kLanes;
  if (k >= (int64_t)a.n_s + a.n_c + a.n_t) return;
  for_prim_cells(a, k, (int)(t % kLanes), [&](uint32_t c) {
    const uint32_t pos = atomicAdd(&cursor[c], 1u);
    refs[cell_begin[c] + pos] = (uint32_t)k;
  });
}

// Ascending ids inside each cell (the scatter's atomics leave them in any
// order).  A block orders the lists of kBlock consecutive cells, whose
// references are one contiguous range of refs.  The range and the block's cell
// offsets are staged in LDS with coalesced loads; then every reference, one
// per thread, finds its cell by binary search over the offsets and goes to
// the slot given by its rank, the number of smaller ids in the same list (a
// primitive enters a cell once, so ranks are distinct).  Work per thread is
// the length of its own list, so the long lists of dense regions do not hold
// a wave back the way a per-cell sort does.  A block whose range exceeds the
// stage sorts in place in global memory instead (same result).
//
// The FP32 walk's view of the occupied cells is written on the way: each
// reference also goes to its place in the cell's walk list (whose offset the
// scan left in the cell's record), as its record offset, 16 x its id (the
// byte offset of its 16-byte FP32 records), with bit 0 set on a list's last
// entry; -1 ends the list, and the cell's record gets the list's first entry.
// One 8-byte load gives the walk the cell's first unit of work, and it knows
// a cell's last test when it makes it.  (The host keeps ids below 2^27 and
// the lists below 2^29 words, so both fit a signed 32-bit word.)
constexpr int kSortStage = 8192;  // refs per block staged in LDS (32 KiB)

__global__ __launch_bounds__(kBlock) void k_sort_cells(const uint32_t *cell_begin, int64_t n_cells,
                                                       uint32_t *refs, uint32_t *wrefs,
                                                       trd::CellInfo *info,
                                                       const unsigned long long *total64,
                                                       unsigned long long cap) {
  if (!fits(total64, cap)) return;
  __shared__ uint32_t stage[kSortStage];
  __shared__ uint32_t offs[kBlock + 1];
  __shared__ uint32_t woffs[kBlock];  // walk lists
  const int64_t c0 = (int64_t)blockIdx.x * kBlock;
  const int64_t c = c0 + threadIdx.x;
  const int nb = (int)min((int64_t)kBlock, n_cells - c0);  // cells in this block
  const uint32_t r0 = cell_begin[c0], r1 = cell_begin[c0 + nb];
  const uint32_t n = r1 - r0;
  if (n <= (uint32_t)kSortStage) {
    for (uint32_t i = threadIdx.x; i < n; i += kBlock) stage[i] = refs[r0 + i];
    for (int i = threadIdx.x; i <= nb; i += kBlock) offs[i] = cell_begin[c0 + i] - r0;
    if ((int)threadIdx.x < nb) woffs[threadIdx.x] = (uint32_t)info[c].a >> 2;  // (read only if occupied)
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n; i += kBlock) {
      // last k with offs[k] <= i; offs[0] = 0 <= i < n = offs[nb]
      int lo = 0, hi = nb;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (offs[mid] <= i) lo = mid; else hi = mid;
      }
      const uint32_t b = offs[lo], e = offs[lo + 1];
      const uint32_t v = stage[i];
      uint32_t rank = 0;
      for (uint32_t j = b; j < e; ++j) rank += stage[j] < v ? 1u : 0u;
      refs[r0 + b + rank] = v;
      const uint32_t entry = (v << 4) | (rank + 1 == e - b ? 1u : 0u);
      wrefs[woffs[lo] + rank] = entry;
      if (rank + 1 == e - b) wrefs[woffs[lo] + rank + 1] = 0xFFFFFFFFu;
      if (rank == 0) info[c0 + lo].c = (int32_t)entry;
    }
  } else if (c < n_cells) {
    const uint32_t b = cell_begin[c], e = cell_begin[c + 1];
    for (uint32_t i = b + 1; i < e; ++i) {
      const uint32_t v = refs[i];
      uint32_t j = i;
      while (j > b && refs[j - 1] > v) {
        refs[j] = refs[j - 1];
        --j;
      }
      refs[j] = v;
    }
    if (e > b) {
      const uint32_t w = (uint32_t)info[c].a >> 2;
      for (uint32_t i = b; i < e; ++i) wrefs[w + (i - b)] = (refs[i] << 4) | (i + 1 == e ? 1u : 0u);
      wrefs[w + (e - b)] = 0xFFFFFFFFu;
      info[c].c = (int32_t)((refs[b] << 4) | (e - b == 1 ? 1u : 0u));
    }
  }
}

// ---- empty-space distance field for the FP32 traversal
// dist(c) = Chebyshev distance, in cells, from c to the nearest occupied
// cell, capped at cap <= kDistCap (0 for occupied cells; cap 1 turns the
// jumps off: the walk is then a plain 3D-DDA).  Computed as three
// separable passes g(x) = min_r max(|r|, g(x + r e_axis)): the L-infinity
// distance is the min over occupied y of max over axes of |x_a - y_a|, and
// max distributes over min, so the axes can be taken one at a time.
// Bound by the latency of its byte loads where the nearest list is far: the
// loads of kDistStep distances to both sides go out together.
constexpr int kDistCap = 32;
constexpr int kDistStep = 4;

__global__ void k_dist_pass(const uint8_t *in, uint8_t *out, int32_t rx, int32_t ry, int32_t rz,
                            int axis, int32_t cap) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n = (int64_t)rx * ry * rz;
  if (c >= n) return;
  const int32_t row = (int32_t)c / rx;  // (a grid has at most 512^3 cells)
  const int32_t ix = (int32_t)c - row * rx, iz = row / ry, iy = row - iz * ry;
  const int32_t p = axis == 0 ? ix : (axis == 1 ? iy : iz);
  const int32_t len = axis == 0 ? rx : (axis == 1 ? ry : rz);
  const int64_t stride = axis == 0 ? 1 : (axis == 1 ? (int64_t)rx : (int64_t)rx * ry);
  int32_t best = in[c];
  for (int32_t r0 = 1; r0 < best; r0 += kDistStep) {  // a neighbour r away can only give >= r
    int32_t v[kDistStep];
#pragma unroll
    for (int32_t q = 0; q < kDistStep; ++q) {
      const int32_t r = r0 + q;
      const int32_t a = p - r >= 0 ? (int32_t)in[c - r * stride] : cap;
      const int32_t b = p + r < len ? (int32_t)in[c + r * stride] : cap;
      v[q] = max(r, min(a, b));
    }
#pragma unroll
    for (int32_t q = 0; q < kDistStep; ++q) best = min(best, v[q]);
  }
  out[c] = (uint8_t)best;
}

// Records of the empty cells: (-distance, bit 31 and the empty blocks ahead).
// dc is the cell's Chebyshev distance (the cube of half-size dc - 1 about it is
// empty); the blocks are those ahead of it, per octant of a ray's direction.
// From the cell, the block of side 2m + 1 that extends ahead in octant o (axis
// a towards -a where bit a of o is set) is the cube of half-size m about the
// cell m steps along that octant's diagonal, so it is empty when that cell's
// distance is at least m + 1.  Such blocks grow with m while the condition
// holds; the record keeps the largest m, M <= 7 (and 2M + 1 within the cap),
// in three bits per octant, and a ray in that octant jumps max(dc, 2M + 1)
// cells ahead.  (The walk is clamped to the part of the cube ahead of it, so a
// block that is empty ahead of the cell is enough.)  The scan stays inside the
// grid.  Bound by the latency of its byte loads: the eight octants' loads of a
// step go out together (one octant after the other, each step's load waited
// for the one before).
__global__ __launch_bounds__(kBlock) void k_empty_cells(const uint8_t *d, int64_t n_cells, int32_t rx,
                                                        int32_t ry, int32_t rz, int32_t cap,
                                                        trd::CellInfo *info) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n_cells) return;
  const int32_t dc = (int32_t)d[c];
  if (dc == 0) return;  // occupied
  const int32_t row = (int32_t)c / rx;  // (a grid has at most 512^3 cells)
  const int32_t ix = (int32_t)c - row * rx, iz = row / ry, iy = row - iz * ry;
  const int32_t mcap = min(7, (cap - 1) / 2);
  uint32_t ext = 0, open = 0xFFu;  // open: octants still growing
  for (int32_t m = 1; m <= mcap && open; ++m) {
    // octants whose diagonal leaves the grid
    uint32_t out = 0;
    if (ix + m >= rx) out |= 0x55u;
    if (ix - m < 0) out |= 0xAAu;
    if (iy + m >= ry) out |= 0x33u;
    if (iy - m < 0) out |= 0xCCu;
    if (iz + m >= rz) out |= 0x0Fu;
    if (iz - m < 0) out |= 0xF0u;
    open &= ~out;
    const int32_t sy = m * rx, sz = m * rx * ry;
    int32_t v[8];
#pragma unroll
    for (int o = 0; o < 8; ++o) {
      const int32_t at = (int32_t)c + ((o & 1) ? -m : m) + ((o & 2) ? -sy : sy) + ((o & 4) ? -sz : sz);
      v[o] = d[((open >> o) & 1u) ? at : (int32_t)c];
    }
#pragma unroll
    for (int o = 0; o < 8; ++o) {
      if (((open >> o) & 1u) && v[o] >= m + 1) ext += 1u << (3 * o);
      else open &= ~(1u << o);
    }
  }
  trd::CellInfo r;
  r.a = -dc;
  r.c = (int32_t)(0x80000000u | ext);
  info[c] = r;
}

// ---- the cells' scan: references and walk-list words (a cell's references
// plus one end marker, none for an empty cell) before each cell.  Two
// launches: totals of 4096 cells each, then every workgroup adds up the totals
// before its own and scans its cells.  The second also leaves what the next
// kernels want of a cell: its count zeroed (the scatter's cursor), its
// distance field started (0 or cap) and an occupied cell's list offset.
constexpr int kCellsPer = 16;                      // cells per thread, consecutive
constexpr int kCellsBlock = kBlock * kCellsPer;    // cells per workgroup
struct CellSums {
  unsigned long long refs;  // (64 bits: overlapping large primitives pass 2^32)
  unsigned long long occupied;
};

__device__ __forceinline__ CellSums block_sum(CellSums v) {
  __shared__ CellSums part[kBlock / 64];
  for (int o = 32; o > 0; o >>= 1) {
    v.refs += __shfl_xor(v.refs, o, 64);
    v.occupied += __shfl_xor(v.occupied, o, 64);
  }
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  v = part[0];
  for (int q = 1; q < kBlock / 64; ++q) {
    v.refs += part[q].refs;
    v.occupied += part[q].occupied;
  }
  __syncthreads();
  return v;
}

__global__ __launch_bounds__(kBlock) void k_cell_sums(const uint32_t *count, int64_t n_cells,
                                                      CellSums *sums) {
  const int64_t base = (int64_t)blockIdx.x * kCellsBlock;
  CellSums v{0ull, 0ull};
#pragma unroll
  for (int q = 0; q < kCellsPer; ++q) {
    const int64_t c = base + q * kBlock + threadIdx.x;
    const uint32_t n = c < n_cells ? count[c] : 0u;
    v.refs += n;
    v.occupied += n ? 1u : 0u;
  }
  v = block_sum(v);
  if (threadIdx.x == 0) sums[blockIdx.x] = v;
}

__global__ __launch_bounds__(kBlock) void k_cell_scan(uint32_t *count, int64_t n_cells,
                                                      const CellSums *sums, uint32_t cap,
                                                      uint32_t *cell_begin, uint8_t *d,
                                                      trd::CellInfo *info,
                                                      unsigned long long *total64,
                                                      unsigned long long *h_total) {
  __shared__ uint32_t stage[kCellsBlock];  // counts, then each cell's references before it
  __shared__ uint32_t wref[kBlock / 64], wocc[kBlock / 64];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t base = (int64_t)blockIdx.x * kCellsBlock;
  CellSums b{0ull, 0ull};
  for (int32_t i = t; i < (int32_t)blockIdx.x; i += kBlock) {
    b.refs += sums[i].refs;
    b.occupied += sums[i].occupied;
  }
  b = block_sum(b);
  if (blockIdx.x == gridDim.x - 1 && t == 0) {  // the totals
    const unsigned long long R = b.refs + sums[blockIdx.x].refs;
    cell_begin[n_cells] = (uint32_t)R;
    count[n_cells] = (uint32_t)(R + b.occupied + sums[blockIdx.x].occupied);  // walk-list words
    total64[0] = R;
    h_total[0] = R;
    h_total[1] = total64[1];
  }
#pragma unroll
  for (int q = 0; q < kCellsPer; ++q) {
    const int64_t c = base + q * kBlock + t;
    stage[q * kBlock + t] = c < n_cells ? count[c] : 0u;
  }
  __syncthreads();
  uint32_t n[kCellsPer], refs = 0, occ = 0;
#pragma unroll
  for (int q = 0; q < kCellsPer; ++q) {
    n[q] = stage[t * kCellsPer + q];
    refs += n[q];
    occ += n[q] ? 1u : 0u;
  }
  uint32_t ir = refs, io = occ;  // inclusive over the wave
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t vr = __shfl_up(ir, o, 64), vo = __shfl_up(io, o, 64);
    if (lane >= o) {
      ir += vr;
      io += vo;
    }
  }
  if (lane == 63) {
    wref[wv] = ir;
    wocc[wv] = io;
  }
  __syncthreads();
  uint32_t r = (uint32_t)b.refs + ir - refs, w = (uint32_t)b.occupied + io - occ;
  for (int q = 0; q < wv; ++q) {
    r += wref[q];
    w += wocc[q];
  }
  w += r;
#pragma unroll
  for (int q = 0; q < kCellsPer; ++q) {
    const int64_t c = base + t * kCellsPer + q;
    if (n[q] && c < n_cells) info[c].a = (int32_t)(w << 2);
    stage[t * kCellsPer + q] = r;
    r += n[q];
    w += n[q] ? n[q] + 1u : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kCellsPer; ++q) {  // (count and d in the order of the first loop: coalesced)
    const int64_t c = base + q * kBlock + t;
    if (c < n_cells) {
      cell_begin[c] = stage[q * kBlock + t];
      d[c] = count[c] ? 0 : (uint8_t)cap;
      count[c] = 0u;
    }
  }
}

// ---- exclusive scan: blocks of kScanItems, block sums scanned recursively
constexpr int kScanPer = 4;
constexpr int kScanItems = kBlock * kScanPer;

__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *sh, uint32_t &total) {
  // Hillis-Steele over kBlock values in shared memory
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int off = 1; off < kBlock; off <<= 1) {
    const uint32_t add = (int)threadIdx.x >= off ? sh[threadIdx.x - off] : 0u;
    __syncthreads();
    sh[threadIdx.x] += add;
    __syncthreads();
  }
  total = sh[kBlock - 1];
  const uint32_t incl = sh[threadIdx.x];
  __syncthreads();
  return incl - v;
}

__global__ __launch_bounds__(kBlock) void k_scan_block(uint32_t *data, int64_t n, uint32_t *sums) {
  __shared__ uint32_t sh[kBlock];
  const int64_t base = (int64_t)blockIdx.x * kScanItems + (int64_t)threadIdx.x * kScanPer;
  uint32_t v[kScanPer];
  uint32_t run = 0;
#pragma unroll
  for (int q = 0; q < kScanPer; ++q) {
    v[q] = base + q < n ? data[base + q] : 0u;
    run += v[q];
  }
  uint32_t total;
  uint32_t off = block_excl_scan(run, sh, total);
#pragma unroll
  for (int q = 0; q < kScanPer; ++q) {
    if (base + q < n) data[base + q] = off;
    off += v[q];
  }
  if (threadIdx.x == 0 && sums) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kBlock) void k_scan_add(uint32_t *data, int64_t n,
                                                     const uint32_t *offs) {
  const uint32_t add = offs[blockIdx.x];
  const int64_t base = (int64_t)blockIdx.x * kScanItems + (int64_t)threadIdx.x * kScanPer;
#pragma unroll
  for (int q = 0; q < kScanPer; ++q)
    if (base + q < n) data[base + q] += add;
}

inline unsigned blocks_for(int64_t n, int b = kBlock) {
  return (unsigned)((n + b - 1) / b);
}

// ---- linear BVH (Karras, "Maximizing parallelism in the construction of
// BVHs, octrees, and k-d trees", HPG 2012).  Primitives are ordered by the
// 30-bit Morton code of their box centres (10 bits per axis over the grid
// box); the N - 1 internal nodes then follow from the sorted codes alone:
// node i covers the run of leaves that share the longest common prefix with
// leaf i, split where that prefix grows.  Equal codes are told apart by
// their position in the sorted order.

__device__ __forceinline__ uint32_t morton30(uint32_t x, uint32_t y, uint32_t z) {
  uint32_t m = 0;
#pragma unroll
  for (int b = 0; b < 10; ++b)
    m |= (((x >> b) & 1u) << (3 * b + 2)) | (((y >> b) & 1u) << (3 * b + 1)) | (((z >> b) & 1u) << (3 * b));
  return m;
}

__global__ void k_bvh_morton(const trh::BuildArgs a, int64_t n, double lx, double ly, double lz,
                             double sx, double sy, double sz, uint32_t *keys, uint32_t *vals) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  double lo[3], hi[3];
  prim_box(a, k, lo, hi);
  const double c[3] = {0.5 * (lo[0] + hi[0]), 0.5 * (lo[1] + hi[1]), 0.5 * (lo[2] + hi[2])};
  const double l[3] = {lx, ly, lz}, sc[3] = {sx, sy, sz};
  uint32_t q[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    double f = floor((c[i] - l[i]) * sc[i]);
    f = f < 0.0 ? 0.0 : (f > 1023.0 ? 1023.0 : f);
    q[i] = (uint32_t)f;
  }
  keys[k] = morton30(q[0], q[1], q[2]);
  vals[k] = (uint32_t)k;
}

// Stable LSD radix sort of the codes (with their primitive ids), 8 bits a
// pass.  A block takes a tile of 1024 keys in four chunks of 256.  Pass
// structure: count each digit per tile, scan the digit-major count table (so
// a tile's slot for digit d follows every smaller digit and every earlier
// tile's d), then scatter: a key's place is its tile's slot for its digit,
// plus the keys of that digit in earlier chunks, in lower waves of its chunk
// (per-wave counts in LDS) and in lower lanes of its wave (the lanes whose
// digit matches, from 8 ballots).  Up to kBvhSmall keys the scatter's
// workgroups read the raw counts (at most 128 of each digit) and scan them
// themselves, in place of the scan's three launches.
constexpr int kRadixTile = 1024;

__global__ __launch_bounds__(256) void k_radix_count(const uint32_t *keys, int64_t n, int shift,
                                                     int64_t nb, uint32_t *cnt) {
  __shared__ uint32_t hist[256];
  const int t = threadIdx.x;
  const int64_t b = blockIdx.x;
  hist[t] = 0u;
  __syncthreads();
  for (int c = 0; c < 4; ++c) {
    const int64_t i = b * kRadixTile + c * 256 + t;
    if (i < n) atomicAdd(&hist[(keys[i] >> shift) & 255u], 1u);
  }
  __syncthreads();
  cnt[(int64_t)t * nb + b] = hist[t];
  if (b == 0 && t == 0) cnt[256 * nb] = 0u;
}

__global__ __launch_bounds__(256) void k_radix_scatter(const uint32_t *keys, const uint32_t *vals,
                                                       int64_t n, int shift, int64_t nb,
                                                       const uint32_t *off, uint32_t *keys2,
                                                       uint32_t *vals2, bool scanned) {
  __shared__ uint32_t run[256];      // next place of each digit in this tile
  __shared__ uint32_t wcnt[4][256];  // keys of each digit in each wave of the chunk
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t b = blockIdx.x;
  if (scanned) {
    run[t] = off[(int64_t)t * nb + b];
  } else {  // raw counts: this digit's keys in all tiles, and in the earlier ones
    uint32_t all = 0, before = 0;
    for (int64_t q = 0; q < nb; ++q) {
      const uint32_t v = off[(int64_t)t * nb + q];
      all += v;
      before += q < b ? v : 0u;
    }
    uint32_t total;
    run[t] = block_excl_scan(all, wcnt[0], total) + before;
  }
  for (int c = 0; c < 4; ++c) {
#pragma unroll
    for (int q = 0; q < 4; ++q) wcnt[q][t] = 0u;
    __syncthreads();
    const int64_t i = b * kRadixTile + c * 256 + t;
    const bool valid = i < n;
    const uint32_t key = valid ? keys[i] : 0u;
    const uint32_t d = (key >> shift) & 255u;
    uint64_t m = __ballot(valid);  // valid lanes with the same digit
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const uint64_t bb = __ballot((d >> bit) & 1u);
      m &= ((d >> bit) & 1u) ? bb : ~bb;
    }
    const uint64_t below = m & ((1ull << lane) - 1ull);
    if (valid && below == 0) wcnt[w][d] = (uint32_t)__popcll(m);  // the digit's lowest lane
    __syncthreads();
    if (valid) {
      uint32_t pos = run[d] + (uint32_t)__popcll(below);
      for (int q = 0; q < w; ++q) pos += wcnt[q][d];
      if ((int64_t)pos < n) {
        keys2[pos] = key;
        vals2[pos] = vals[i];
      }
    }
    __syncthreads();
    run[t] += wcnt[0][t] + wcnt[1][t] + wcnt[2][t] + wcnt[3][t];
    __syncthreads();
  }
}

// Child encoding: c >= 0 internal node c; c < 0 leaf at sorted position -c - 1.
__device__ __forceinline__ int prefix_len(const uint32_t *keys, int64_t n, int64_t i, int64_t j) {
  if (j < 0 || j >= n) return -1;
  const uint32_t a = keys[i], b = keys[j];
  if (a == b) return 32 + __clz((uint32_t)(i ^ j));
  return __clz(a ^ b);
}

__global__ void k_bvh_internal(const uint32_t *keys, int64_t n, int32_t *left, int32_t *right,
                               int32_t *parent_i, int32_t *other, uint32_t *flags) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < 2) flags[i] = 0u;  // largest depth; nodes left to k_bvh_top
  if (i >= n - 1) return;
  const int64_t d = prefix_len(keys, n, i, i + 1) - prefix_len(keys, n, i, i - 1) >= 0 ? 1 : -1;
  const int dmin = prefix_len(keys, n, i, i - d);
  int64_t lmax = 2;
  while (lmax < 2 * n && prefix_len(keys, n, i, i + lmax * d) > dmin) lmax *= 2;
  int64_t l = 0;
  for (int64_t t = lmax / 2; t >= 1; t /= 2)
    if (prefix_len(keys, n, i, i + (l + t) * d) > dmin) l += t;
  const int64_t j = i + l * d;
  const int dnode = prefix_len(keys, n, i, j);
  int64_t s = 0, t = 0, div = 2;
  do {
    t = (l + div - 1) / div;
    if (prefix_len(keys, n, i, i + (s + t) * d) > dnode) s += t;
    div *= 2;
  } while (t > 1);
  const int64_t g = i + s * d + (d < 0 ? -1 : 0);
  const int64_t lo = i < j ? i : j, hi = i < j ? j : i;
  const int32_t lc = lo == g ? (int32_t)(-g - 1) : (int32_t)g;
  const int32_t rc = hi == g + 1 ? (int32_t)(-(g + 1) - 1) : (int32_t)(g + 1);
  left[i] = lc;
  right[i] = rc;
  other[i] = (int32_t)j;  // node i covers the leaves from i to j
  if (lc >= 0) parent_i[lc] = (int32_t)i;
  if (rc >= 0) parent_i[rc] = (int32_t)i;
  if (i == 0) parent_i[0] = -1;
}

// Box of a child: a leaf's primitive box widened by margin, or the stored
// box of an internal node (written by an earlier launch).
__device__ __forceinline__ void child_box(const trh::BuildArgs &a, const uint32_t *vals,
                                          const double *ibox, int32_t c, double margin,
                                          double lo[3], double hi[3]) {
  if (c < 0) {
    prim_box(a, (int64_t)vals[-c - 1], lo, hi);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      lo[q] -= margin;
      hi[q] += margin;
    }
  } else {
    const double *b = ibox + 6 * (int64_t)c;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      lo[q] = b[q];
      hi[q] = b[3 + q];
    }
  }
}

// Depth of every internal node: the links up to the root.  A path's split
// lengths rise strictly through at most 62 values (30 code bits, then position
// bits), so depths stay below 64, which bounds the loop; links are clamped to
// the node range.  The largest goes to *out: a wave maximum, then the
// workgroup's in LDS, then one atomic per workgroup.
__global__ __launch_bounds__(kBlock) void k_bvh_depth(const int32_t *parent_i, int64_t m, int32_t *dep,
                                                      uint32_t *out) {
  __shared__ int32_t wmax[kBlock / 64];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int32_t v = 0;
  if (i < m) {
    int32_t p = (int32_t)i;
    while (p != 0 && v < 63) {
      p = parent_i[p];
      p = (uint32_t)p < (uint32_t)m ? p : 0;
      ++v;
    }
    dep[i] = v;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t b = wmax[0];
    for (int k = 1; k < kBlock / 64; ++k) b = max(b, wmax[k]);
    atomicMax(out, (uint32_t)b);
  }
}

// Box of internal node i: the union of its children's.
__device__ __forceinline__ void node_box(const trh::BuildArgs &a, const uint32_t *vals, int64_t i,
                                         const int32_t *left, const int32_t *right, double *ibox,
                                         double margin) {
  double l0[3], h0[3], l1[3], h1[3];
  child_box(a, vals, ibox, left[i], margin, l0, h0);
  child_box(a, vals, ibox, right[i], margin, l1, h1);
  double *b = ibox + 6 * i;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    b[k] = l0[k] < l1[k] ? l0[k] : l1[k];
    b[3 + k] = h0[k] > h1[k] ? h0[k] : h1[k];
  }
}

// Boxes of a tree of at most kBvhSmall leaves in two launches, in place of one
// for each of its some 25 levels.  Workgroup w takes the nodes whose leaves all
// lie in its kBvhChunk (node i covers leaves from i to other[i], so it is one
// of the chunk's indices), deepest level first, a barrier between levels, leaf
// boxes read before the first level and inner boxes kept in LDS; the nodes
// across chunks, about a dozen for each chunk's end, are listed and left to one
// workgroup (k_bvh_top).  Each level costs a barrier and a read of LDS or L2,
// not a launch.  26,318 leaves: all levels in 16 + 20 us, the whole build
// 308 -> 129 us (with the depths and the sort in fewer launches, above).
constexpr int kBvhChunk = 512;
// Up to here: a node's index fits the list's 18 bits, and the last workgroup's share
// has grown to what the levels' launches cost (a build in chunks / by levels, with
// its wait: 8,000 leaves 113 / 225 us, 26,000 127 / 232, 65,000 182 / 250, 131,072 268 / 260).
constexpr int64_t kBvhSmall = 131072;

__global__ __launch_bounds__(kBvhChunk) void k_bvh_chunks(const trh::BuildArgs a, const uint32_t *vals,
                                                          int64_t m, const int32_t *dep,
                                                          const int32_t *other, const int32_t *left,
                                                          const int32_t *right, double *ibox,
                                                          double margin, uint32_t *flags,
                                                          uint32_t *list) {
  __shared__ int32_t lo_d, hi_d;            // depths of this chunk's own nodes
  __shared__ double box[6][kBvhChunk];      // their boxes
  const int64_t base = (int64_t)blockIdx.x * kBvhChunk, i = base + threadIdx.x;
  if (threadIdx.x == 0) {
    lo_d = 64;
    hi_d = -1;
  }
  __syncthreads();
  const int64_t j = i < m ? other[i] : 0;
  const bool own = i < m && j >= base && j < base + kBvhChunk;
  const int32_t d = own ? dep[i] : -1;
  if (own) {
    atomicMin(&lo_d, d);
    atomicMax(&hi_d, d);
  } else if (i < m) {
    list[atomicAdd(&flags[1], 1u)] = (uint32_t)dep[i] << 18 | (uint32_t)i;
  }
  __syncthreads();
  const int32_t first = hi_d, last = lo_d;
  int32_t c[2] = {0, 0};
  double v[2][6];  // the two children's boxes
  if (own) {
    c[0] = left[i];
    c[1] = right[i];
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (c[k] < 0) child_box(a, vals, ibox, c[k], margin, v[k], v[k] + 3);
  }
  for (int32_t q = first; q >= last; --q) {
    if (d == q) {
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (c[k] >= 0) {
#pragma unroll
          for (int x = 0; x < 6; ++x) v[k][x] = box[x][c[k] - base];
        }
#pragma unroll
      for (int x = 0; x < 3; ++x) {
        const double l = v[0][x] < v[1][x] ? v[0][x] : v[1][x];
        const double h = v[0][3 + x] > v[1][3 + x] ? v[0][3 + x] : v[1][3 + x];
        ibox[6 * i + x] = box[x][threadIdx.x] = l;
        ibox[6 * i + 3 + x] = box[3 + x][threadIdx.x] = h;
      }
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(1024) void k_bvh_top(const trh::BuildArgs a, const uint32_t *vals,
                                                  const int32_t *left, const int32_t *right,
                                                  double *ibox, double margin,
                                                  const uint32_t *flags, const uint32_t *list,
                                                  unsigned long long *h_depth) {
  const int32_t deepest = (int32_t)flags[0];
  const uint32_t n = flags[1];
  // a thread's first node is held ready, as in k_bvh_chunks: its links, and
  // the boxes of children that are leaves
  const uint32_t v0 = threadIdx.x < n ? list[threadIdx.x] : ~0u;
  const int64_t i0 = v0 & 0x3ffffu;
  const int32_t d0 = v0 == ~0u ? -1 : (int32_t)(v0 >> 18);
  int32_t c[2] = {0, 0};
  double b[2][6];
  if (d0 >= 0) {
    c[0] = left[i0];
    c[1] = right[i0];
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (c[k] < 0) child_box(a, vals, ibox, c[k], margin, b[k], b[k] + 3);
  }
  for (int32_t q = deepest; q >= 0; --q) {
    if (d0 == q) {
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (c[k] >= 0) child_box(a, vals, ibox, c[k], margin, b[k], b[k] + 3);
#pragma unroll
      for (int x = 0; x < 3; ++x) {
        ibox[6 * i0 + x] = b[0][x] < b[1][x] ? b[0][x] : b[1][x];
        ibox[6 * i0 + 3 + x] = b[0][3 + x] > b[1][3 + x] ? b[0][3 + x] : b[1][3 + x];
      }
    }
    for (uint32_t k = threadIdx.x + 1024; k < n; k += 1024) {
      const uint32_t v = list[k];
      if ((int32_t)(v >> 18) == q) node_box(a, vals, v & 0x3ffffu, left, right, ibox, margin);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) *h_depth = (unsigned long long)deepest;
}

// Boxes of the internal nodes at depth d: the union of their children's
// boxes (a deeper level's, stored by the previous launch, or a leaf's).
__global__ void k_bvh_level(const trh::BuildArgs a, const uint32_t *vals, int64_t m,
                            const int32_t *dep, int32_t d, const int32_t *left,
                            const int32_t *right, double *ibox, double margin) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m || dep[i] != d) return;
  node_box(a, vals, i, left, right, ibox, margin);
}

// Traversal records, one per internal node (64 bytes): both children's
// boxes in the FP32 frame, rounded outwards, then the children (an internal
// node index, or -(primitive id) - 1 for a leaf).
__global__ void k_bvh_pack(const trh::BuildArgs a, const uint32_t *vals, int64_t n,
                           const int32_t *left, const int32_t *right, const double *ibox,
                           double margin, double ox, double oy, double oz, float4 *nodes) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n - 1) return;
  const double o[3] = {ox, oy, oz};
  float f[12];
  int32_t ch[2] = {left[i], right[i]};
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    double lo[3], hi[3];
    child_box(a, vals, ibox, ch[c], margin, lo, hi);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      f[6 * c + q] = __double2float_rd(lo[q] - o[q]);
      f[6 * c + 3 + q] = __double2float_ru(hi[q] - o[q]);
    }
    if (ch[c] < 0) ch[c] = -(int32_t)vals[-ch[c] - 1] - 1;
  }
  float4 *r = nodes + 4 * i;
  r[0] = make_float4(f[0], f[1], f[2], f[3]);
  r[1] = make_float4(f[4], f[5], f[6], f[7]);
  r[2] = make_float4(f[8], f[9], f[10], f[11]);
  r[3] = make_float4(__int_as_float(ch[0]), __int_as_float(ch[1]), 0.0f, 0.0f);
}

}  // namespace

namespace trh {

hipError_t launch_pack(const PackArgs &p, hipStream_t st) {
  const int64_t N = p.n_s + p.n_c + p.n_t;
  if (N == 0) return hipSuccess;
  k_pack<<<blocks_for(N), kBlock, 0, st>>>(p);
  return hipGetLastError();
}

static int32_t bounds_blocks(int64_t N) {
  int64_t b = (N + kBlock - 1) / kBlock;
  if (b < 1) b = 1;
  if (b > 1024) b = 1024;
  return (int32_t)b;
}

int64_t bounds_scratch_doubles(int64_t n_prims) { return 6 * (int64_t)bounds_blocks(n_prims); }

hipError_t launch_bounds(const BuildArgs &a, double *scratch, double *out6, hipStream_t st) {
  const int32_t nb = bounds_blocks((int64_t)a.n_s + a.n_c + a.n_t);
  k_bounds_partial<<<nb, kBlock, 0, st>>>(a, scratch);
  k_bounds_final<<<1, kBlock, 0, st>>>(scratch, nb, out6);
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t b = blocks_for(n);
  if (b > 65536) b = 65536;
  k_fill_u32<<<(unsigned)b, kBlock, 0, st>>>(p, n, v);
  return hipGetLastError();
}

hipError_t launch_count_pack(const BuildArgs &a, const Pack32Args &p, uint32_t *count, int64_t n_cells,
                             unsigned long long *total64, hipStream_t st) {
  const int64_t N = (int64_t)a.n_s + a.n_c + a.n_t;
  k_grid_init<<<(unsigned)std::min<int64_t>(blocks_for(n_cells + 1), 65536), kBlock, 0, st>>>(
      count, n_cells + 1, total64);
  if (N > 0) {
    const unsigned nc = blocks_for(N * kLanes);
    k_count_pack<<<nc + blocks_for(N), kBlock, 0, st>>>(a, p, nc, count);
  }
  return hipGetLastError();
}

int64_t cell_scan_words(int64_t n_cells) {
  return (n_cells + kCellsBlock - 1) / kCellsBlock * (int64_t)(sizeof(CellSums) / 4);
}

hipError_t launch_cell_scan(uint32_t *count, int64_t n_cells, int32_t cap, uint32_t *scratch,
                            uint32_t *cell_begin, uint8_t *d0, trd::CellInfo *info,
                            unsigned long long *total64, unsigned long long *h_total, hipStream_t st) {
  const unsigned nb = (unsigned)((n_cells + kCellsBlock - 1) / kCellsBlock);
  if (cap < 1 || cap > kDistCap) cap = kDistCap;
  k_cell_sums<<<nb, kBlock, 0, st>>>(count, n_cells, (CellSums *)scratch);
  k_cell_scan<<<nb, kBlock, 0, st>>>(count, n_cells, (const CellSums *)scratch, (uint32_t)cap, cell_begin,
                                     d0, info, total64, h_total);
  return hipGetLastError();
}

int64_t scan_scratch_u32(int64_t n) {
  int64_t total = 0;
  while (n > kScanItems) {
    n = (n + kScanItems - 1) / kScanItems;
    total += n;
  }
  return total + 1;
}

hipError_t launch_scan(uint32_t *data, int64_t n, uint32_t *scratch, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (n <= kScanItems) {
    k_scan_block<<<1, kBlock, 0, st>>>(data, n, nullptr);
    return hipGetLastError();
  }
  const int64_t nb = (n + kScanItems - 1) / kScanItems;
  uint32_t *sums = scratch;
  k_scan_block<<<(unsigned)nb, kBlock, 0, st>>>(data, n, sums);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = launch_scan(sums, nb, scratch + nb, st);
  if (e != hipSuccess) return e;
  k_scan_add<<<(unsigned)nb, kBlock, 0, st>>>(data, n, sums);
  return hipGetLastError();
}

hipError_t launch_lists(const BuildArgs &a, const uint32_t *cell_begin, int64_t n_cells, uint32_t *cursor,
                        uint32_t *refs, uint32_t *wrefs, trd::CellInfo *info,
                        const unsigned long long *total64, int64_t cap, hipStream_t st) {
  const int64_t N = (int64_t)a.n_s + a.n_c + a.n_t;
  if (N == 0) return hipSuccess;
  k_scatter<<<blocks_for(N * kLanes), kBlock, 0, st>>>(a, cell_begin, cursor, refs, total64,
                                                       (unsigned long long)cap);
  k_sort_cells<<<blocks_for(n_cells), kBlock, 0, st>>>(cell_begin, n_cells, refs, wrefs, info, total64,
                                                       (unsigned long long)cap);
  return hipGetLastError();
}

int64_t bvh_sort_counts(int64_t n) { return 256 * ((n + kRadixTile - 1) / kRadixTile) + 1; }

hipError_t launch_bvh_tree(const BuildArgs &a, const double lo[3], const double hi[3],
                           BvhScratch &w, hipStream_t st) {
  const int64_t n = (int64_t)a.n_s + a.n_c + a.n_t;
  if (n < 2) return hipSuccess;
  const unsigned nb = blocks_for(n);
  double sc[3];
  for (int q = 0; q < 3; ++q) sc[q] = hi[q] > lo[q] ? 1024.0 / (hi[q] - lo[q]) : 0.0;
  k_bvh_morton<<<nb, kBlock, 0, st>>>(a, n, lo[0], lo[1], lo[2], sc[0], sc[1], sc[2], w.keys, w.vals);
  uint32_t *k0 = w.keys, *v0 = w.vals, *k1 = w.keys2, *v1 = w.vals2;
  const int64_t tiles = (n + kRadixTile - 1) / kRadixTile;
  for (int shift = 0; shift < 30; shift += 8) {
    k_radix_count<<<(unsigned)tiles, 256, 0, st>>>(k0, n, shift, tiles, w.flags);
    const bool scanned = n > kBvhSmall;
    if (scanned) {
      const hipError_t e = launch_scan(w.flags, 256 * tiles + 1, w.scan_scratch, st);
      if (e != hipSuccess) return e;
    }
    k_radix_scatter<<<(unsigned)tiles, 256, 0, st>>>(k0, v0, n, shift, tiles, w.flags, k1, v1, scanned);
    std::swap(k0, k1);
    std::swap(v0, v1);
  }
  // 4 passes: the sorted arrays are back in keys / vals; keys2 / vals2 are free
  const int64_t m = n - 1;
  const unsigned nbm = blocks_for(m);
  k_bvh_internal<<<nbm, kBlock, 0, st>>>(w.keys, n, w.left, w.right, w.parent_i, w.other, w.flags);
  k_bvh_depth<<<nbm, kBlock, 0, st>>>(w.parent_i, m, w.height, w.flags);
  return hipGetLastError();
}

bool bvh_small(int64_t n) { return n <= kBvhSmall; }

hipError_t launch_bvh_boxes(const BuildArgs &a, const BvhScratch &w, int32_t max_depth,
                            double margin, const double origin[3], float4 *nodes,
                            unsigned long long *h_depth, hipStream_t st) {
  const int64_t n = (int64_t)a.n_s + a.n_c + a.n_t;
  if (n < 2) return hipSuccess;
  const int64_t m = n - 1;
  const unsigned nbm = blocks_for(m);
  if (bvh_small(n)) {
    k_bvh_chunks<<<blocks_for(m, kBvhChunk), kBvhChunk, 0, st>>>(a, w.vals, m, w.height, w.other, w.left,
                                                                 w.right, w.ibox, margin, w.flags, w.keys2);
    k_bvh_top<<<1, 1024, 0, st>>>(a, w.vals, w.left, w.right, w.ibox, margin, w.flags, w.keys2,
                                  h_depth);
  }
  else for (int32_t d = max_depth; d >= 0; --d)
    k_bvh_level<<<nbm, kBlock, 0, st>>>(a, w.vals, m, w.height, d, w.left, w.right, w.ibox, margin);
  k_bvh_pack<<<nbm, kBlock, 0, st>>>(a, w.vals, n, w.left, w.right, w.ibox, margin, origin[0],
                                     origin[1], origin[2], nodes);
  return hipGetLastError();
}

hipError_t launch_empty_cells(const int32_t res[3], int32_t cap, uint8_t *d0, uint8_t *d1,
                              trd::CellInfo *info, hipStream_t st) {
  const int64_t n = (int64_t)res[0] * res[1] * res[2];
  if (n <= 0) return hipSuccess;
  const unsigned nb = blocks_for(n);
  if (cap < 1 || cap > kDistCap) cap = kDistCap;
  k_dist_pass<<<nb, kBlock, 0, st>>>(d0, d1, res[0], res[1], res[2], 0, cap);
  k_dist_pass<<<nb, kBlock, 0, st>>>(d1, d0, res[0], res[1], res[2], 1, cap);
  k_dist_pass<<<nb, kBlock, 0, st>>>(d0, d1, res[0], res[1], res[2], 2, cap);
  k_empty_cells<<<nb, kBlock, 0, st>>>(d1, n, res[0], res[1], res[2], cap, info);
  return hipGetLastError();
}

}  // namespace trh
