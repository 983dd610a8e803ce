// render_plain.hip -- the plain double-precision GPU path: every step in
// FP64, with no re-solves.  This is the GPU counterpart of the paper's
// renderer as it was built ("double precision option for all calculations",
// Sec. 2) and the baseline the FP32 wavefront kernel is measured against.
//
// Two kernels give the same frames: k_render_f64, which queues the rays of a
// tile's hits, and k_render_plain_f64, one thread per pixel over a plain
// 3D-DDA, whose traversal counts are those of the method's definition (launches
// with a stats buffer, and frames with little to trace: see plain_is_faster).
//
// Compiled with -ffp-contract=off and written in the same expression order
// as the definition of the method (camera, intersections, normals,
// sampling, shading), so that primary hits reproduce bit for bit.
#include <algorithm>

#include "tr_internal.h"

namespace {

using namespace trd;

constexpr double kEps = 1e-4;  // secondary-ray t_min (world units)

struct Cnt {
  uint32_t rays, cells, st, sh, ct, ch, tt, th;
};

// Nearest hit (lexicographic min of (t, id)) or any hit with t in
// (tmin, tmax], visiting the grid cells the ray crosses in order.
//
// On axis a the ray meets the grid plane of index p (at lo + p h) at
// t = b_a + p g_a, with b_a = (lo_a - o_a) / d_a and g_a = h_a / d_a: the
// first crossing is one FMA from the entry cell's plane, and each later one
// |g_a| further.  The walk keeps, per axis, the next crossing, the cells
// left before the grid's side and the step of the cell's linear index.  Any
// walk that visits every cell the segment crosses gives the same nearest
// hit: the lists hold every primitive within the insertion margin of a cell,
// far above the FP64 rounding of the crossings.
template <bool ANY, bool TRI>
__device__ int trace_f64(const SceneDev &S, const double o[3], const double d[3], double tmin,
                         double tmax, int32_t skip, double &bt, int32_t &bk, Cnt &c) {
  c.rays++;
  bool found = false;
  bt = INFINITY;
  bk = -1;
  // the part of (tmin, tmax] inside the grid box, axis by axis
  double tin = tmin, tout = tmax;
  double b[3], g[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (d[a] == 0.0) {
      if (o[a] < S.lo[a] || o[a] > S.hi[a]) return 0;
      b[a] = g[a] = 0.0;
      continue;
    }
    b[a] = (S.lo[a] - o[a]) / d[a];
    g[a] = S.h[a] / d[a];
    const double tl = b[a], th = (S.hi[a] - o[a]) / d[a];
    tin = fmax(tin, fmin(tl, th));
    tout = fmin(tout, fmax(tl, th));
  }
  if (tin > tout) return 0;
  // entry cell (clamped into the grid); per axis the next crossing, the
  // time between crossings, the cells left to the grid's side and the step
  // of the linear index (a grid has at most 512^3 cells: 32-bit indices)
  int32_t left[3], stride[3];
  double tn[3], dt[3];
  const int32_t plane_cells[3] = {1, S.res[0], S.res[0] * S.res[1]};
  int32_t cell = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double f = floor((o[a] + tin * d[a] - S.lo[a]) * S.inv[a]);
    const int32_t i = f >= 0.0 ? (f < (double)S.res[a] ? (int32_t)f : S.res[a] - 1) : 0;
    cell += i * plane_cells[a];
    if (d[a] > 0.0) {
      tn[a] = fma((double)(i + 1), g[a], b[a]);
      dt[a] = g[a];
      left[a] = S.res[a] - 1 - i;
      stride[a] = plane_cells[a];
    } else if (d[a] < 0.0) {
      tn[a] = fma((double)i, g[a], b[a]);
      dt[a] = -g[a];
      left[a] = i;
      stride[a] = -plane_cells[a];
    } else {
      tn[a] = INFINITY;
      dt[a] = 0.0;
      left[a] = 0;
      stride[a] = 0;
    }
  }
  const double t1 = tout;
  for (;;) {
    c.cells++;
    const uint32_t e = S.cell_begin[(uint32_t)cell + 1u];
    for (uint32_t r = S.cell_begin[(uint32_t)cell]; r < e; ++r) {
      const int32_t k = (int32_t)S.refs[r];
      if (k == skip) continue;
      double t;
      int h;
      if (k < S.n_s) {
        c.st++;
        h = hit_sphere_f64(S.sph64[k], o, d, tmin, tmax, t);
        c.sh += h;
      } else if (TRI && k >= S.n_s + S.n_c) {
        const int32_t m = k - S.n_s - S.n_c;
        c.tt++;
        h = hit_triangle_f64(S.triA64[m], S.triB64[m], S.triC64[m], o, d, tmin, tmax, t);
        c.th += h;
      } else {
        c.ct++;
        h = hit_cylinder_f64(S.cylA64[k - S.n_s], S.cylW64[k - S.n_s], o, d, tmin, tmax, t);
        c.ch += h;
      }
      if (h) {
        if (ANY) {
          bt = t;
          bk = k;
          return 1;
        }
        if (!found || t < bt || (t == bt && k < bk)) {
          found = true;
          bt = t;
          bk = k;
        }
      }
    }
    // leave through the nearest plane; stop once the best hit lies in the
    // cells already seen, or at the end of the segment or the grid
    const int a = tn[0] <= tn[1] ? (tn[0] <= tn[2] ? 0 : 2) : (tn[1] <= tn[2] ? 1 : 2);
    if (!ANY && found && bt <= fmin(tn[a], t1)) return 1;
    if (!(tn[a] < t1) || left[a] == 0) return found;
    --left[a];
    cell += stride[a];
    tn[a] += dt[a];
  }
}

template <bool TRI>
__device__ __forceinline__ void normal_f64(const SceneDev &S, int32_t k, const double o[3],
                                           const double d[3], double t, double n[3]) {
  if (k < S.n_s) {
    const double4 s = S.sph64[k];
    const double P[3] = {o[0] + t * d[0], o[1] + t * d[1], o[2] + t * d[2]};
    n[0] = (P[0] - s.x) / s.w;
    n[1] = (P[1] - s.y) / s.w;
    n[2] = (P[2] - s.z) / s.w;
  } else if (TRI && k >= S.n_s + S.n_c) {
    const int32_t m = k - S.n_s - S.n_c;
    triangle_normal_f64(S.triA64[m], S.triB64[m], S.triC64[m], n);
  } else {
    const double4 a = S.cylA64[k - S.n_s], w4 = S.cylW64[k - S.n_s];
    const double w[3] = {w4.x, w4.y, w4.z};
    const double D[3] = {o[0] - a.x, o[1] - a.y, o[2] - a.z};
    const double sax = dot3d(D, w) + t * dot3d(d, w);
#pragma unroll
    for (int q = 0; q < 3; ++q) n[q] = ((D[q] + t * d[q]) - sax * w[q]) / a.w;
  }
}

// One thread per pixel.  Variants: counting, layered compositing and triangles are
// compiled in only for jobs that need them (each costs registers, and so
// occupancy, in the others).
template <bool STATS, bool LAYERED, bool TRI>
__global__ __launch_bounds__(256) void k_render_plain_f64(const JobDev J, uint64_t *stats) {
  __shared__ uint32_t red[TR_STAT_COUNT];
  if (STATS) {
    if (threadIdx.x < TR_STAT_COUNT) red[threadIdx.x] = 0;
    __syncthreads();
  }
  const int32_t i = blockIdx.x * 16 + (threadIdx.x & 15);
  const int32_t j = blockIdx.y * 16 + (threadIdx.x >> 4);
  Cnt c{0, 0, 0, 0, 0, 0, 0, 0};
  uint32_t n_hit = 0, n_ao = 0, n_sh = 0;
  if (i < J.W && j < J.H) {
    const SceneDev &S = J.sc;
    const int64_t pid = (int64_t)j * J.W + i;
    double o[3], d[3];
    primary_ray_f64(J, i, j, o, d);
    // Surfaces along the primary ray, front to back: one for opaque
    // rendering; with layers, the ray continues through a primitive of
    // opacity < 1 from the hit point (skipping it only when leaving it) and
    // the colours composite by the transmittance in front of each surface.
    double acc[3] = {0.0, 0.0, 0.0};
    double T = 1.0;
    double tmin = 0.0;
    int32_t pskip = -1;
    int hit = 0;
    int32_t k0 = -1;
    uint32_t amask = 0;
    uint32_t lmask = 0;
    const int32_t layers = LAYERED ? J.layers : 1;
    for (int32_t layer = 0; layer < layers; ++layer) {
      double t;
      int32_t k;
      if (!trace_f64<false, TRI>(S, o, d, tmin, INFINITY, pskip, t, k, c)) break;
      if (layer == 0) {
        hit = 1;
        k0 = k;
        n_hit = 1;
      }
      double N[3], P[3];
      normal_f64<TRI>(S, k, o, d, t, N);
#pragma unroll
      for (int q = 0; q < 3; ++q) P[q] = o[q] + t * d[q];
      const bool front = dot3d(N, d) < 0.0;
      if (!front) {
        N[0] = -N[0];
        N[1] = -N[1];
        N[2] = -N[2];
      }
      const int32_t skip = front ? k : -1;
      uint32_t am = 0, lm = 0;
      double D[3] = {0.0, 0.0, 0.0};
      double Hs[3] = {0.0, 0.0, 0.0};  // Phong highlight (white, after the albedo)
      for (int l = 0; l < J.n_lights; ++l) {
        const double cl = dot3d(N, J.ldir[l]);
        if (!(cl > kLightMin)) continue;
        n_sh++;
        double tt;
        int32_t kk;
        if (trace_f64<true, TRI>(S, P, J.ldir[l], kEps, INFINITY, skip, tt, kk, c)) {
          lm |= 1u << l;
        } else {
#pragma unroll
          for (int ch = 0; ch < 3; ++ch) D[ch] += J.lcol[l][ch] * cl;
          if (J.ks > 0.0) {
            // light direction mirrored about N, against the way back to the eye
            double R[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) R[q] = 2.0 * cl * N[q] - J.ldir[l][q];
            const double rv = -dot3d(R, d);
            if (rv > 0.0) {
              const double f = J.ks * pow(rv, J.shin);
#pragma unroll
              for (int ch = 0; ch < 3; ++ch) Hs[ch] += J.lcol[l][ch] * f;
            }
          }
        }
      }
      double ao = 1.0;
      if (J.S > 0) {
        int32_t aocc = 0;
        for (int s = 0; s < J.S; ++s) {
          uint32_t b1, b2;
          ao_uniform_bits((uint32_t)pid, (uint32_t)s + ((uint32_t)layer << 16), J.view_id,
                          (uint32_t)J.aa, J.key0, J.key1, b1, b2);
          double w[3];
          ao_dir_f64(N, b1, b2, w);
          n_ao++;
          double tt;
          int32_t kk;
          if (trace_f64<true, TRI>(S, P, w, kEps, J.ao_maxdist, skip, tt, kk, c)) {
            aocc++;
            if (s < 32) am |= 1u << s;
          }
        }
        ao = (double)(J.S - aocc) / (double)J.S;
      }
      if (layer == 0) {
        amask = am;
        lmask = lm;
      }
      const float4 alb = S.albedo[k];
      const double albv[3] = {(double)alb.x, (double)alb.y, (double)alb.z};
      const double alpha = LAYERED ? (double)alb.w : 1.0;
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) {
        const double v = albv[ch] * (D[ch] + J.sky * ao) + Hs[ch];
        acc[ch] += T * alpha * (v < 0.0 ? 0.0 : (v > 1.0 ? 1.0 : v));
      }
      T *= 1.0 - alpha;
      if (!(alpha < 1.0)) break;
#pragma unroll
      for (int q = 0; q < 3; ++q) o[q] = P[q];
      tmin = kEps;
      pskip = front ? -1 : k;
    }
    double col[3];
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) col[ch] = acc[ch] + T * (double)J.bg[ch];
    J.rgb[pid * 3 + 0] = (float)col[0];
    J.rgb[pid * 3 + 1] = (float)col[1];
    J.rgb[pid * 3 + 2] = (float)col[2];
    if (J.hit_id) J.hit_id[pid] = hit ? k0 : -1;
    if (J.ao_mask) J.ao_mask[pid] = amask;
    if (J.light_mask) J.light_mask[pid] = (uint8_t)lmask;
    if (STATS) {
      atomicAdd(&red[TR_STAT_PIXELS], 1u);
      atomicAdd(&red[TR_STAT_HIT_PIXELS], n_hit);
      atomicAdd(&red[TR_STAT_AO_RAYS], n_ao);
      atomicAdd(&red[TR_STAT_SHADOW_RAYS], n_sh);
      atomicAdd(&red[TR_STAT_RAYS_TRACED], c.rays);
      atomicAdd(&red[TR_STAT_CELLS], c.cells);
      atomicAdd(&red[TR_STAT_SPH_TESTS], c.st);
      atomicAdd(&red[TR_STAT_SPH_HITS], c.sh);
      atomicAdd(&red[TR_STAT_CYL_TESTS], c.ct);
      atomicAdd(&red[TR_STAT_CYL_HITS], c.ch);
      atomicAdd(&red[TR_STAT_TRI_TESTS], c.tt);
      atomicAdd(&red[TR_STAT_TRI_HITS], c.th);
    }
  }
  if (STATS) {
    __syncthreads();
    if (threadIdx.x < TR_STAT_COUNT && red[threadIdx.x])
      atomicAdd((unsigned long long *)&stats[threadIdx.x], (unsigned long long)red[threadIdx.x]);
  }
}

// ------------------------------------------------ the queued FP64 renderer
// The same frames as k_render_plain_f64, bit for bit: every decision and every
// colour comes from the same FP64 expressions on the same rays; which cells a
// ray visits does not matter as long as no occupied one is left out.  One wave
// per tile of 8 x 8 pixels or part of one (group_entry).  A wave traces its
// pixels' primary rays, one a lane, and keeps the hits in LDS; then the light
// and AO rays of all its hits are dealt to its lanes, an idle lane taking the
// next as soon as half of the lanes are idle; then it shades its pixels, one a
// lane.  (One thread per pixel ran with 19 of 64 lanes active: a wave waited
// for its longest ray eighteen times over.)  The walk jumps over empty cells
// by the cell records of the FP32 walk (the distance to the nearest occupied
// cell, or the empty block ahead in the ray's octant) and stops at the
// scene's bounding sphere.  965 x 1137, 26,318 objects, 16 AO samples:
// 4.02 -> 1.30 ms (128 x 128 of 64 spheres 215 -> 55 us).

// State of one ray's walk.
struct Walk {
  double o[3], d[3];
  double b[3], g[3];  // the walk enters cell i of axis a at t = b_a + i g_a
  double t1, bt;      // end of the walk; best t (nearest hit)
  int32_t i[3];       // cell
  int32_t oct;        // octant of d (bit a: d_a < 0)
  int32_t flat;       // axes with d_a = 0 (bits)
  int32_t rc;         // byte offset of the cursor in the cell's walk list, or -(distance)
  int32_t nk;         // entry there (16 id, bit 0 on the last), or negative (see CellInfo)
  int32_t bk;         // best primitive (nearest hit), or one that was hit; -1 none
  int32_t skip;       // primitive never reported (-1 none)
};

__device__ __forceinline__ void walk_cell(const SceneDev &S, Walk &w) {
  const int32_t c = (w.i[2] * S.res[1] + w.i[1]) * S.res[0] + w.i[0];
  const CellInfo ci = S.cellinfo[c];
  w.rc = ci.a;
  w.nk = ci.c;
}

// Clip the ray to the grid box and the bounding sphere and enter the walk;
// false when it misses either.  (The sphere is padded by 2^-10 of its radius,
// far above the FP64 rounding while the origin is within 2^10 radii of it;
// beyond that the box alone clips.)
__device__ __forceinline__ bool walk_setup(const SceneDev &S, Walk &w, double tmin, double tmax) {
  double tin = tmin, tout = tmax;
  double q[3];
  w.oct = 0;
  w.flat = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double inv = 1.0 / w.d[a];  // (infinite on a flat axis: its slab times too)
    const double tl = (S.lo[a] - w.o[a]) * inv, th = (S.hi[a] - w.o[a]) * inv;
    tin = fmax(tin, fmin(tl, th));
    tout = fmin(tout, fmax(tl, th));
    w.oct |= w.d[a] < 0.0 ? 1 << a : 0;
    w.flat |= w.d[a] == 0.0 ? 1 << a : 0;
    w.g[a] = S.h[a] * inv;
    w.b[a] = w.d[a] < 0.0 ? tl + w.g[a] : tl;
    if (w.d[a] == 0.0) {  // its planes are never crossed
      w.b[a] = INFINITY;
      w.g[a] = 0.0;
      if (w.o[a] < S.lo[a] || w.o[a] > S.hi[a]) tout = -INFINITY;
    }
    q[a] = w.o[a] - S.org[a];
  }
  const double bb = -dot3d(q, w.d);
  const double l[3] = {q[0] + bb * w.d[0], q[1] + bb * w.d[1], q[2] + bb * w.d[2]};
  const double ll = dot3d(l, l);
  if (bb * bb + ll < (double)S.rguard2_32) {
    const double disc = (double)S.rb2_32 - ll;
    const double sq = sqrt(fmax(disc, 0.0));
    tin = fmax(tin, bb - sq);
    tout = disc >= 0.0 ? fmin(tout, bb + sq) : -INFINITY;
  }
  w.t1 = tout;
  w.bt = INFINITY;
  w.bk = -1;
  if (!(tin <= tout)) return false;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double f = floor((fma(tin, w.d[a], w.o[a]) - S.lo[a]) * S.inv[a]);
    w.i[a] = f >= 0.0 ? (f < (double)S.res[a] ? (int32_t)f : S.res[a] - 1) : 0;
  }
  walk_cell(S, w);
  return true;
}

// One unit of a walk: test the entry it holds, then, with none left in the
// cell, move on.  False when the walk is over.
template <bool ANY, bool TRI>
__device__ __forceinline__ bool walk_unit(const SceneDev &S, Walk &w, double tmin, double tmax) {
  if (w.nk >= 0) {
    const int32_t k = w.nk >> 4;
    const bool last = (w.nk & 1) != 0;
    bool hit = false;
    double t = 0.0;
    if (k != w.skip) {
      if (k < S.n_s) {
        hit = hit_sphere_f64(S.sph64[k], w.o, w.d, tmin, tmax, t);
      } else if (TRI && k >= S.n_s + S.n_c) {
        const int32_t m = k - S.n_s - S.n_c;
        hit = hit_triangle_f64(S.triA64[m], S.triB64[m], S.triC64[m], w.o, w.d, tmin, tmax, t);
      } else {
        // First the cylinder's bounding sphere (about the axis midpoint): a
        // ray that passes it by a margin far above the rounding (2^-9 of its
        // squared radius, and 2^-40 of the distance's square) has no root on
        // the cylinder, and most rays do.
        const double4 A = S.cylA64[k - S.n_s], W = S.cylW64[k - S.n_s];
        const double hl = 0.5 * W.w;
        const double c[3] = {fma(hl, W.x, A.x) - w.o[0], fma(hl, W.y, A.y) - w.o[1],
                             fma(hl, W.z, A.z) - w.o[2]};
        const double cb = dot3d(c, w.d);
        const double cl[3] = {c[0] - cb * w.d[0], c[1] - cb * w.d[1], c[2] - cb * w.d[2]};
        const double ll = dot3d(cl, cl), r2 = hl * hl + A.w * A.w;
        if (ll <= fma(r2, 1.0 + 0x1p-9, 0x1p-40 * (cb * cb + ll)))
          hit = hit_cylinder_f64(A, W, w.o, w.d, tmin, tmax, t);
      }
    }
    if (hit) {
      if (ANY) {
        w.bk = k;
        return false;
      }
      if (t < w.bt || (t == w.bt && k < w.bk)) {
        w.bt = t;
        w.bk = k;
      }
    }
    if (!last) {
      w.rc += 4;
      w.nk = (int32_t)*(const uint32_t *)((const char *)S.wrefs + (uint32_t)w.rc);
      return true;
    }
    w.nk = (int32_t)0x80000000u;  // (rc >= 0 and no block ahead: a unit step)
  }
  // The block of m cells per axis ahead is empty beyond this one (m = 1: just
  // this cell): on to where the ray leaves it.
  const int32_t mo = (w.nk >> (3 * w.oct)) & 7;
  const int32_t m = max(max(-w.rc, 1), 2 * mo + 1);
  int32_t n[3];
  double t[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    n[a] = w.i[a] + (((w.flat >> a) & 1) ? 0 : (((w.oct >> a) & 1) ? -m : m));
    t[a] = fma((double)n[a], w.g[a], w.b[a]);
  }
  const double tn = fmin(t[0], fmin(t[1], t[2]));
  if (!(tn < fmin(w.t1, w.bt))) return false;  // past the end, or the best hit
  const int ax = t[0] == tn ? 0 : (t[1] == tn ? 1 : 2);
  bool in = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (a == ax) {
      w.i[a] = n[a];
    } else {  // the cell of the exit point, kept between this cell and the block's last
      const int32_t e = n[a] - (((w.flat >> a) & 1) ? 0 : (((w.oct >> a) & 1) ? -1 : 1));
      const int32_t f = (int32_t)floor((fma(tn, w.d[a], w.o[a]) - S.lo[a]) * S.inv[a]);
      w.i[a] = min(max(f, min(w.i[a], e)), max(w.i[a], e));
    }
    in = in && (uint32_t)w.i[a] < (uint32_t)S.res[a];
  }
  if (!in) return false;
  walk_cell(S, w);
  return true;
}

struct LdsF64 {
  double P[3][64], N[3][64];  // hit points and facing normals
  int32_t skip[64];           // the primitive the pixel's secondary rays skip
  uint32_t lv[64], lm[64];    // lights with N.L > 2^-40; those occluded
  uint32_t am[64], ao[64];    // occluded AO samples: bits, count
  int32_t hits[64];           // slots with a hit, in order
};

constexpr int kRefill64 = 32;  // lanes at work below which idle ones take new rays

template <bool LAYERED, bool TRI>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3)))
void k_render_f64(const JobDev J, int64_t n_tiles, uint32_t first, uint32_t whole, int32_t part_log2, int32_t chunk_log2,
                  uint32_t turn) {
  __shared__ LdsF64 L;
  const SceneDev &S = J.sc;
  const int32_t lane = threadIdx.x;
  const int64_t entry = group_entry(first + blockIdx.x, whole, part_log2, chunk_log2, turn, n_tiles);
  if (entry < 0) return;
  const uint32_t tile = (uint32_t)(entry >> 7), tiles_x = ((uint32_t)J.W + 7u) / 8u;
  int32_t tx = (int32_t)(tile % tiles_x), ty = (int32_t)(tile / tiles_x);
  if (chunk_log2) block_tile(tile, tiles_x, ((uint32_t)J.H + 7u) / 8u, chunk_log2, tx, ty);
  const int32_t part = (int32_t)(entry & 127) - 1;
  const int32_t npx = part < 0 ? 64 : 64 >> part_log2;
  const int32_t px = lane + (part < 0 ? 0 : part * npx);  // pixel of the tile
  const int32_t i = tx * 8 + (px & 7), j = ty * 8 + (px >> 3);
  const bool mine = lane < npx && i < J.W && j < J.H;
  const int64_t pid = (int64_t)j * J.W + i;

  double acc[3] = {0.0, 0.0, 0.0}, T = 1.0;  // colour in front, and what it lets through
  double d[3] = {0.0, 0.0, 0.0};
  int32_t pskip = -1, k0 = -1;
  uint32_t am0 = 0, lm0 = 0;
  bool alive = mine;  // the camera ray goes on
  const int32_t layers = LAYERED ? J.layers : 1;
  for (int32_t layer = 0; layer < layers; ++layer) {
    // ---- nearest hits of the camera rays, a pixel a lane
    Walk w;
    bool run = false;
    const double tmin = layer ? kEps : 0.0;
    if (alive) {
      if (layer == 0) {
        primary_ray_f64(J, i, j, w.o, d);
      } else {
#pragma unroll
        for (int q = 0; q < 3; ++q) w.o[q] = L.P[q][lane];
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) w.d[q] = d[q];
      w.skip = pskip;
      run = walk_setup(S, w, tmin, INFINITY);
    }
    while (__ballot(run)) {
      if (run) run = walk_unit<false, TRI>(S, w, tmin, INFINITY);
    }
    const bool hit = alive && w.bk >= 0;
    const int32_t k = w.bk;
    bool front = false;
    if (hit) {
      double N[3], P[3];
      normal_f64<TRI>(S, k, w.o, w.d, w.bt, N);
#pragma unroll
      for (int q = 0; q < 3; ++q) P[q] = w.o[q] + w.bt * w.d[q];
      front = dot3d(N, w.d) < 0.0;
      if (!front) {
        N[0] = -N[0];
        N[1] = -N[1];
        N[2] = -N[2];
      }
      uint32_t lv = 0;
      for (int l = 0; l < J.n_lights; ++l) lv |= dot3d(N, J.ldir[l]) > kLightMin ? 1u << l : 0u;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        L.P[q][lane] = P[q];
        L.N[q][lane] = N[q];
      }
      L.skip[lane] = front ? k : -1;
      L.lv[lane] = lv;
      L.lm[lane] = 0;
      L.am[lane] = 0;
      L.ao[lane] = 0;
    }
    const uint64_t hm = __ballot(hit);
    if (!hm) break;
    if (hit) L.hits[__popcll(hm & ((1ull << lane) - 1ull))] = lane;
    __syncthreads();
    // ---- their light rays, then AO rays: ray r of hit h is number h per + r
    const uint32_t per = (uint32_t)(J.n_lights + J.S);
    const uint32_t total = (uint32_t)__popcll(hm) * per;
    uint32_t next = 0;
    bool have = false;
    int32_t slot = 0;
    uint32_t r = 0;
    run = false;
    for (;;) {
      if (have && !run) {  // hand in the result
        if (w.bk >= 0) {
          if (r < (uint32_t)J.n_lights) {
            atomicOr(&L.lm[slot], 1u << r);
          } else {
            const uint32_t s = r - (uint32_t)J.n_lights;
            atomicAdd(&L.ao[slot], 1u);
            if (s < 32u) atomicOr(&L.am[slot], 1u << s);
          }
        }
        have = false;
      }
      const uint64_t idle = __ballot(!have);
      const uint32_t n = next + (uint32_t)__popcll(idle & ((1ull << lane) - 1ull));
      next = min(total, next + (uint32_t)__popcll(idle));
      if (!have && n < total) {
        const uint32_t h = n / per;
        r = n - h * per;
        slot = L.hits[h];
        const bool ao = r >= (uint32_t)J.n_lights;
        if (ao || ((L.lv[slot] >> r) & 1u)) {
          have = true;
#pragma unroll
          for (int q = 0; q < 3; ++q) w.o[q] = L.P[q][slot];
          if (ao) {
            const int32_t sp = slot + (part < 0 ? 0 : part * npx);
            const uint32_t spid = (uint32_t)((int64_t)(ty * 8 + (sp >> 3)) * J.W + tx * 8 + (sp & 7));
            const double N[3] = {L.N[0][slot], L.N[1][slot], L.N[2][slot]};
            uint32_t b1, b2;
            ao_uniform_bits(spid, (r - (uint32_t)J.n_lights) + ((uint32_t)layer << 16), J.view_id,
                            (uint32_t)J.aa, J.key0, J.key1, b1, b2);
            ao_dir_f64(N, b1, b2, w.d);
          } else {
#pragma unroll
            for (int q = 0; q < 3; ++q) w.d[q] = J.ldir[r][q];
          }
          w.skip = L.skip[slot];
          run = walk_setup(S, w, kEps, ao ? J.ao_maxdist : INFINITY);
        }
      }
      if (!__ballot(have)) {
        if (next == total) break;
        continue;
      }
      const double tmax = r >= (uint32_t)J.n_lights ? J.ao_maxdist : INFINITY;
      const int32_t least = next < total ? kRefill64 : 1;
      for (int32_t it = 0; __popcll(__ballot(run)) >= (it < 2 ? 1 : least); ++it)
        if (run) run = walk_unit<true, TRI>(S, w, kEps, tmax);
    }
    __syncthreads();
    // ---- shade the pixels
    if (hit) {
      const double N[3] = {L.N[0][lane], L.N[1][lane], L.N[2][lane]};
      const uint32_t lv = L.lv[lane], lm = L.lm[lane];
      double D[3] = {0.0, 0.0, 0.0};
      double Hs[3] = {0.0, 0.0, 0.0};  // Phong highlight (white, after the albedo)
      for (int l = 0; l < J.n_lights; ++l) {
        if (!((lv >> l) & 1u) || ((lm >> l) & 1u)) continue;
        const double cl = dot3d(N, J.ldir[l]);
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) D[ch] += J.lcol[l][ch] * cl;
        if (J.ks > 0.0) {
          // light direction mirrored about N, against the way back to the eye
          double R[3];
#pragma unroll
          for (int q = 0; q < 3; ++q) R[q] = 2.0 * cl * N[q] - J.ldir[l][q];
          const double rv = -dot3d(R, d);
          if (rv > 0.0) {
            const double f = J.ks * pow(rv, J.shin);
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) Hs[ch] += J.lcol[l][ch] * f;
          }
        }
      }
      const double ao = J.S > 0 ? (double)(J.S - (int32_t)L.ao[lane]) / (double)J.S : 1.0;
      if (layer == 0) {
        k0 = k;
        am0 = L.am[lane];
        lm0 = lm;
      }
      const float4 alb = S.albedo[k];
      const double albv[3] = {(double)alb.x, (double)alb.y, (double)alb.z};
      const double alpha = LAYERED ? (double)alb.w : 1.0;
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) {
        const double v = albv[ch] * (D[ch] + J.sky * ao) + Hs[ch];
        acc[ch] += T * alpha * (v < 0.0 ? 0.0 : (v > 1.0 ? 1.0 : v));
      }
      T *= 1.0 - alpha;
      pskip = front ? -1 : k;
      alive = alpha < 1.0;
    } else {
      alive = false;
    }
    __syncthreads();
  }
  if (mine) {
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) J.rgb[pid * 3 + ch] = (float)(acc[ch] + T * (double)J.bg[ch]);
    if (J.hit_id) J.hit_id[pid] = k0;
    if (J.ao_mask) J.ao_mask[pid] = am0;
    if (J.light_mask) J.light_mask[pid] = (uint8_t)lm0;
  }
}

}  // namespace

namespace trh {

// Whether one thread per pixel is the faster kernel.  The queued kernel costs
// 2.4 ns for each workgroup (a wave a tile, 1.2 to 8 of them; 1080p 154 us for
// a frame of background, where a thread per pixel takes 31), and its rays 2 to 9
// times less the more objects there are; a thread traces its pixel's rays one
// after the other, so a small frame takes as long as its slowest pixel.
// Modelled on 128 x 128 to 3860 x 4548, 0 to 16 AO samples, 1 to 10^6 objects,
// whole views, far ones and background; measured, us, queued / thread per pixel:
// one sphere at 1080p, 0, 4 and 16 samples 163 / 47, 210 / 98, 326 / 245, at 128 x
// 128 22 / 18, 23 / 28, 28 / 61; 64 spheres at 965 x 1137 178 / 78, 298 / 254, 559 /
// 774; 26,318 objects at 965 x 1137 408 / 400, 687 / 1359, 1355 / 4230.  Over those
// launches the choice is within a tenth of the better kernel, but for some frames of
// 64 spheres (3860 x 4548 at 4 samples 2910 / 2430, 320 x 240 at none 52 / 40).  With
// layers a pixel's rays are taken twice (64 spheres at opacity 0.5, up to 4 layers, no
// AO, 640 x 480 138 / 85, 1080p 251 / 177).
static bool plain_is_faster(const trd::JobDev &job, int64_t workgroups) {
  const double n = std::max(1.0, (double)job.sc.n_s + job.sc.n_c + job.sc.n_t);
  const double rays = (1 + job.n_lights + job.S) * (job.layers > 1 ? 2 : 1), traced = rays * covered_pixels(job);
  // ns; the slowest pixel's beyond what a queued wave waits for too
  const double slowest = traced > 0.0 ? 2500.0 * rays * std::pow(n, 0.36) : 0.0;
  const double plain = 0.015 * ((double)job.W * job.H) + 0.0147 * std::pow(n, 0.28) * traced;
  const double queued = 2.4 * (double)workgroups + 0.015 * std::pow(n, 0.19) * traced;
  return std::max(slowest, plain) < queued;
}

template <bool STATS, bool LAYERED>
static void launch_plain(const trd::JobDev &job, uint64_t *stats, hipStream_t st) {
  const dim3 grid((unsigned)(((int64_t)job.W + 15) / 16), (unsigned)(((int64_t)job.H + 15) / 16));
  if (job.sc.n_t > 0) k_render_plain_f64<STATS, LAYERED, true><<<grid, 256, 0, st>>>(job, stats);
  else k_render_plain_f64<STATS, LAYERED, false><<<grid, 256, 0, st>>>(job, stats);
}

hipError_t launch_render_plain_f64(const trd::JobDev &job, uint64_t *stats, hipStream_t st) {
  const bool lay = job.layers > 1, tri = job.sc.n_t > 0;
  const int64_t tiles = (((int64_t)job.W + 7) / 8) * (((int64_t)job.H + 7) / 8);
  const Groups g = split_groups(tiles, 1, true, (int32_t)(((int64_t)job.W + 7) / 8));
  if (stats || plain_is_faster(job, g.workgroups)) {
    if (!stats && lay) launch_plain<false, true>(job, nullptr, st);
    else if (!stats) launch_plain<false, false>(job, nullptr, st);
    else if (lay) launch_plain<true, true>(job, stats, st);
    else launch_plain<true, false>(job, stats, st);
    return hipGetLastError();
  }
  // (several launches where the workgroups are more than HIP takes in one: frames
  // of a few columns and 10^8 rows.  Each but the last a multiple of 8, for the XCDs.)
  constexpr int64_t kMost = kMaxWorkgroups / trd::kQueueXcds * trd::kQueueXcds;
  for (int64_t at = 0; at < g.workgroups; at += kMost) {
    const unsigned n = (unsigned)std::min(kMost, g.workgroups - at);
    const uint32_t first = (uint32_t)at;
    if (lay && tri) k_render_f64<true, true><<<n, 64, 0, st>>>(job, tiles, first, g.whole, g.part_log2, g.chunk_log2, g.turn);
    else if (lay) k_render_f64<true, false><<<n, 64, 0, st>>>(job, tiles, first, g.whole, g.part_log2, g.chunk_log2, g.turn);
    else if (tri) k_render_f64<false, true><<<n, 64, 0, st>>>(job, tiles, first, g.whole, g.part_log2, g.chunk_log2, g.turn);
    else k_render_f64<false, false><<<n, 64, 0, st>>>(job, tiles, first, g.whole, g.part_log2, g.chunk_log2, g.turn);
  }
  return hipGetLastError();
}

}  // namespace trh
