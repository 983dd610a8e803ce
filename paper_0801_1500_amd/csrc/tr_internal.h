// tr_internal.h -- host-side internals shared by the library's translation units.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>

#include "../../include/tr.h"
#include "tr_device.h"

namespace trh {

// Uniform-grid parameters, computed on the host from the device bounds.
struct GridParams {
  double lo[3], hi[3], h[3], inv[3];
  double delta;
  int32_t res[3];
  int64_t n_cells;
};

// Inputs of the count / scatter kernels.
struct BuildArgs {
  int32_t n_s, n_c, n_t;
  const double4 *sph64, *cylA64, *cylB64;
  const double4 *triA64, *triB64, *triC64;
  double lo[3], h[3], inv[3], delta;
  int32_t res[3];
};

// ---- grid build launchers (grid_build.hip) ----
// albedo = (r, g, b, opacity); sop / cop / top may be null (opaque)
struct PackArgs {
  int64_t n_s, n_c, n_t;
  const double *sc, *sr, *ca, *cb, *cr, *tv0, *tv1, *tv2;
  const float *srgb, *sop, *crgb, *cop, *trgb, *top;
  double4 *sph64, *cylA64, *cylW64, *cylB64, *triA64, *triB64, *triC64;
  float4 *albedo;
};
hipError_t launch_pack(const PackArgs &p, hipStream_t st);
// FP32 copies with positions relative to origin (the centre of the grid box);
// also maxes the scene's bounding radius about origin (FP64 bits) into
// *rmax64
struct Pack32Args {
  const double4 *cylW64;
  double origin[3];
  float4 *sph32, *cylA32, *cylW32, *tri32;
  unsigned long long *rmax64;
};
// bounds: out6 = (lo xyz, hi xyz); scratch >= bounds_scratch_doubles(N) doubles
int64_t bounds_scratch_doubles(int64_t n_prims);
hipError_t launch_bounds(const BuildArgs &a, double *scratch, double *out6, hipStream_t st);
hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t st);
// per-cell counts (count[n_cells + 1] and total64[2] are zeroed first) and the
// FP32 copies
hipError_t launch_count_pack(const BuildArgs &a, const Pack32Args &p, uint32_t *count, int64_t n_cells,
                             unsigned long long *total64, hipStream_t st);
// exclusive scan of the counts into cell_begin[n_cells + 1]: zeroes the counts
// (count[n_cells] = walk-list words), starts the distance field d0, leaves the
// occupied cells' list offsets in info, and the reference total in total64[0]
// and, with total64[1], in h_total (pinned).  scratch: cell_scan_words words.
int64_t cell_scan_words(int64_t n_cells);
hipError_t launch_cell_scan(uint32_t *count, int64_t n_cells, int32_t cap, uint32_t *scratch,
                            uint32_t *cell_begin, uint8_t *d0, trd::CellInfo *info,
                            unsigned long long *total64, unsigned long long *h_total, hipStream_t st);
// reference lists, sorted, and walk lists; nothing is written when the
// reference total exceeds cap
hipError_t launch_lists(const BuildArgs &a, const uint32_t *cell_begin, int64_t n_cells, uint32_t *cursor,
                        uint32_t *refs, uint32_t *wrefs, trd::CellInfo *info,
                        const unsigned long long *total64, int64_t cap, hipStream_t st);
// empty-space distances (d0: started by the scan; d1: n_cells bytes) and the
// records of the empty cells.
// cap: largest stored distance, 1..32 (1 = no jumps); anything else = 32
hipError_t launch_empty_cells(const int32_t res[3], int32_t cap, uint8_t *d0, uint8_t *d1,
                              trd::CellInfo *info, hipStream_t st);
// exclusive scan of n+1 entries in place (data[n] must be 0 on entry)
int64_t scan_scratch_u32(int64_t n);
hipError_t launch_scan(uint32_t *data, int64_t n_plus_1, uint32_t *scratch, hipStream_t st);

// Linear BVH over all primitives (n >= 2): 4 float4 per internal node (see
// k_bvh_pack); node 0 is the root.  Scratch sizes: keys, vals, keys2, vals2: n;
// flags (the sort's digit counts): bvh_sort_counts(n); left, right, parent_i,
// other, height: n - 1; ibox: 6 (n - 1) doubles; scan_scratch:
// scan_scratch_u32(bvh_sort_counts(n)).
// launch_bvh_tree sorts, builds the hierarchy and leaves each internal
// node's depth (links from the root) in height[] and the largest depth in
// flags[0]; launch_bvh_boxes then computes the boxes from the deepest nodes up
// and packs the records.  A small tree (bvh_small) needs no max_depth from the
// host, and leaves the largest depth in *h_depth (pinned).
struct BvhScratch {
  uint32_t *keys, *vals, *keys2, *vals2, *flags, *scan_scratch;
  int32_t *left, *right, *parent_i, *other, *height;
  double *ibox;
};
// Entries of the BVH walk's per-lane traversal stack.  A walk that visits a
// node at depth d holds at most d deferred siblings, so a tree of depth
// <= kBvhStack never overflows it; deeper trees are refused before launch.
constexpr int kBvhStack = 48;
int64_t bvh_sort_counts(int64_t n);
hipError_t launch_bvh_tree(const BuildArgs &a, const double lo[3], const double hi[3],
                           BvhScratch &w, hipStream_t st);
hipError_t launch_bvh_boxes(const BuildArgs &a, const BvhScratch &w, int32_t max_depth,
                            double margin, const double origin[3], float4 *nodes,
                            unsigned long long *h_depth, hipStream_t st);
bool bvh_small(int64_t n);

// ---- frame output (frame_out.hip) ----
// values -> bytes, floor(clamp(v, 0, 1) * 255 + 1/2); any alignment
hipError_t launch_quantize_rgb8(const float *in, int64_t n, uint8_t *out, hipStream_t st);
// Run-length Targa file of an 8-bit RGB image [H][W][3] (1 <= W, H <= 65535):
// sizes computes row_bytes[H], row_off[H] (absolute file offsets of the rows)
// and *total (the file size, also to pinned host memory); write then fills out[0, *total), which must
// hold *total bytes.
hipError_t launch_tga_sizes(const uint8_t *rgb, int32_t W, int32_t H, int64_t *row_bytes,
                            int64_t *row_off, int64_t *total, int64_t *h_total, hipStream_t st);
hipError_t launch_tga_write(const uint8_t *rgb, int32_t W, int32_t H, const int64_t *row_off,
                            const int64_t *total, uint8_t *out, hipStream_t st);
// rgb[i] = (rgb[i] + planes[0][i] + ... + planes[n_planes - 1][i]) / (n_planes + 1),
// summed in that order; planes are n floats apart
hipError_t launch_aa_mean(float *rgb, const float *planes, int32_t n_planes, int64_t n,
                          hipStream_t st);

// ---- render launchers ----
// Pixels of the job's frame that its scene may cover: the outline of the
// bounding sphere, as if it were centred (all of them from inside, none with
// the sphere behind the eye).
inline double covered_pixels(const trd::JobDev &J) {
  const double px = (double)J.W * J.H, r2 = J.sc.rb2_32;
  double d2 = 0.0, ahead = 0.0;
  for (int a = 0; a < 3; ++a) {
    const double v = J.sc.org[a] - J.eye[a];
    d2 += v * v;
    ahead += v * J.f[a];
  }
  if (!(d2 > r2)) return px;
  if (ahead < 0.0 && ahead * ahead > r2) return 0.0;
  const double across = std::sqrt(r2 / (d2 - r2)) / J.th * J.H;
  return std::min(across, (double)J.W) * std::min(across, (double)J.H) *
         (across < std::max(J.W, J.H) ? 0.25 * M_PI : 1.0);
}
hipError_t launch_render_plain_f64(const trd::JobDev &job, uint64_t *stats, hipStream_t st);

// Entries of a launch of one workgroup per entry over tiles of n_jobs frames
// (trd::group_entry): the first 8 whole tiles as they are, each later one in
// 2^part_log2 parts.  Whole frames (blocks) of more than 1,024 tiles are dealt
// to the XCDs in blocks of 2 x 4 tiles, so that an L2 serves rays that visit
// the same cells.  One frame of 26,318 objects, single tiles / blocks of 8: 640 x
// 480 256, 245 us; 965 x 1137 717, 697; 1930 x 2274 2200, 2177; 3860 x 4548
// 8160, 8080; 4 antialiasing passes of 965 x 1137 2520, 2407; 8 frames of 1080p
// over 10^6 objects, whose cells are four times the L2s, 31.2, 30.2 ms.  Larger
// blocks leave the XCDs unlike shares of a frame: 128 tiles (8 x 16) are 1 to 3%
// faster than 8 where the frame's width suits them and up to 14% slower where it
// does not, slower than persistent waves too (8 frames over 10^6 objects, waves /
// 8 / 128: 1152 x 864 5930, 5600, 6390 us; 1280 x 1024 8010, 7720, 8260; 1920 x
// 1080 8920, 8580, 8490).  Over 20 widths from 640 to 4096, three and eight frames of
// 1080 rows, blocks of 8 / 128 to persistent waves: 10^6 objects 0.914 / 0.933 and
// 0.970 / 0.977, 200,000 0.935 / 0.918 and 0.980 / 0.953, 26,318 0.891 / 0.910 and 0.937
// / 0.942.  Ranges of a frame's tiles run in row order: single tiles.
// A launch has fewer than 2^32 threads (HIP's limit for a dimension of the
// grid); callers compare the count, split tail and all.
constexpr int64_t kMaxWorkgroups = (int64_t)UINT32_MAX / 64;
struct Groups {
  uint32_t whole;     // in groups of 8 tiles
  int32_t part_log2;
  int32_t chunk_log2;
  uint32_t turn;
  int64_t workgroups;         // of 64 threads; may exceed kMaxWorkgroups
};
// (tiles_x: of the largest frame)
inline Groups split_groups(int64_t tiles, int32_t n_jobs, bool blocks, int32_t tiles_x) {
  const int64_t split = (int64_t)((n_jobs > 1 ? 20.0 : 60.0) * std::sqrt((double)tiles));
  Groups g;
  g.part_log2 = tiles <= 1024 ? 3 : 2;
  g.chunk_log2 = blocks && tiles > 1024 ? 3 : 0;
  const int64_t in = (int64_t)trd::kQueueXcds << g.chunk_log2;  // tiles in a group of chunks
  g.whole = tiles > 1024 && tiles > split ? (uint32_t)((tiles - split) / in) << g.chunk_log2 : 0u;
  const int64_t groups = (tiles + in - 1) / in << g.chunk_log2;
  // groups of 8 blocks in a band of 4 rows; an even number comes back to the same
  // rotations after 8 / gcd(8, number) bands
  const uint32_t band = tiles_x % 16 ? 1u : (uint32_t)tiles_x / 16u;
  g.turn = band % 2u ? UINT32_MAX : band * (band % 8u == 0u ? 1u : band % 4u == 0u ? 2u : 4u);
  g.workgroups = (g.whole + ((groups - g.whole) << g.part_log2)) * trd::kQueueXcds;
  return g;
}

struct WaveLaunch {
  const trd::JobDev *jobs;   // device array
  int32_t n_jobs;
  int64_t n_tiles;           // total tiles in the queue
  uint32_t *tile_counter;    // device, trd::kQueueWords words zeroed before the launch
  uint64_t *stats;           // device or null
  int32_t tile_w, banks, refill_below, count_ops;
  int32_t stripe;            // tiles per tile-queue stripe (a power of two)
  // One workgroup per entry (two banks asked for, no stats), or part_log2 = -1
  // for persistent waves drawing from the tile queue:
  uint32_t whole;            // groups of 8 tiles that are entries as they are
  int32_t part_log2;         // entries of each later tile, log2
  int32_t chunk_log2;        // see Groups
  uint32_t turn;
  int32_t n_waves;           // waves launched
  int32_t resolve;
  int32_t trans;             // some job composites transparent layers
  int32_t tri;               // some job's scene has triangles
  int32_t bvh;               // walk the scenes' BVHs instead of their grids
};
hipError_t launch_render_wave(const WaveLaunch &L, hipStream_t st);
// write n job table entries (device memory) from the host's jobs, passed as
// kernel arguments, kPutJobs a launch
constexpr int kPutJobs = 3;
hipError_t launch_put_jobs(const trd::JobDev *J, int32_t n, trd::JobDev *dst, hipStream_t st);

// FP32 FMA rate (TFLOP/s) of non-packed v_fma_f32 over the whole device
hipError_t measure_fma_rate(hipStream_t st, int32_t n_cus, double *tflops);

hipError_t launch_debug_philox(int64_t n, const uint32_t *ctr, const uint32_t *key, uint32_t *out,
                               hipStream_t st);
hipError_t launch_debug_ao_dirs(int64_t n, const float *nrm, const uint32_t *pix,
                                const uint32_t *smp, uint32_t view, uint32_t k0, uint32_t k1,
                                float *w, hipStream_t st);

}  // namespace trh
