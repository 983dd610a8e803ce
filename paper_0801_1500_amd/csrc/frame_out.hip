// frame_out.hip -- 8-bit output of a rendered frame (the paper's "Image I/O"
// phase, Table 5, moved onto the GPU): every float value v becomes
// floor(min(max(v, 0), 1) * 255 + 1/2), NaN becoming 0.
//
// A streaming kernel, bound by HBM: 4 bytes read and 1 byte written per
// value.  Each thread converts four float4 groups placed 256 groups apart, so
// every load and store instruction of a wave covers one contiguous span
// (1 KiB of input, 256 B of output); the data is touched once, so it is read
// and written non-temporally.  The rounding is exact: a float times 255 is
// exact in double, so the conversion runs in FP64 (two FP64 ops per value
// are far below the memory time).
//
// Also here: the mean over an antialiased frame's sample planes, another
// streaming pass (A * 4 bytes read and 4 written per value), and the
// run-length Targa file of an 8-bit image (see k_tga_rows).
#include <algorithm>

#include "tr_internal.h"

namespace {

typedef float vf4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kPerThread = 4;                     // float4 groups per thread
constexpr int kGroups = kThreads * kPerThread;    // float4 groups per block

__device__ __forceinline__ uint32_t q8(float x) {
  double v = (double)x;
  v = v > 0.0 ? v : 0.0;  // also NaN
  v = v < 1.0 ? v : 1.0;
  return (uint32_t)floor(v * 255.0 + 0.5);
}

// n4 float4 groups of a 16-byte aligned input to 4-byte words of the output.
__global__ __launch_bounds__(kThreads) void k_quantize_vec(const vf4 *__restrict__ in,
                                                           uint32_t *__restrict__ out, int64_t n4) {
  const int64_t base = (int64_t)blockIdx.x * kGroups + threadIdx.x;
  vf4 v[kPerThread];
#pragma unroll
  for (int j = 0; j < kPerThread; ++j) {
    const int64_t i = base + (int64_t)j * kThreads;
    if (i < n4) v[j] = __builtin_nontemporal_load(&in[i]);
  }
#pragma unroll
  for (int j = 0; j < kPerThread; ++j) {
    const int64_t i = base + (int64_t)j * kThreads;
    if (i < n4) {
      const uint32_t w = q8(v[j].x) | (q8(v[j].y) << 8) | (q8(v[j].z) << 16) | (q8(v[j].w) << 24);
      __builtin_nontemporal_store(w, &out[i]);
    }
  }
}

// Any alignment and the values past the last whole group: one value per thread.
__global__ __launch_bounds__(kThreads) void k_quantize_scalar(const float *__restrict__ in,
                                                              uint8_t *__restrict__ out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i < n) out[i] = (uint8_t)q8(in[i]);
}

// Mean of an antialiased pixel's samples: sample 0 is already in rgb, samples
// 1..n_planes in the planes; the sum runs in sample order, so the result
// does not depend on how the samples were scheduled.
__global__ __launch_bounds__(kThreads) void k_aa_mean(float *rgb, const float *planes,
                                                      int32_t n_planes, int64_t n, float count) {
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads) {
    float sum = rgb[i];
    const float *p = planes + i;
    for (int32_t a = 0; a < n_planes; ++a, p += n) sum += *p;
    rgb[i] = sum / count;
  }
}

// ---- Targa file, run-length true colour (the packet rule is written out
// with the host-side declaration).  One workgroup per image row; each thread
// takes kTgaPx adjacent pixels.  A pixel's role follows from its neighbours
// alone: it belongs to a run when it equals a neighbour; a segment (a maximal
// run of one colour, or a maximal stretch of pixels in no run) starts where
// the role changes or a run changes colour; packets are the 128-pixel pieces
// of segments.  A pixel's segment starts at the last start at or before it: in
// its own thread, else the last one of the lower threads (a max scan over the
// workgroup), else the segment still open from the row's previous step.  A run
// packet's 4 bytes belong to its last pixel, a raw packet's header byte to its
// first, so a pixel's byte position is the exclusive prefix sum of these sizes
// along the row.  Pass 1 sums each row, a scan turns the sums into row
// offsets, pass 2 recomputes the roles and writes.  The file is 18 header
// bytes, the rows, 26 footer bytes.
//
// Bound by HBM in principle (the image read twice, the file written once),
// in fact by latency: one wave per row, 36 byte loads a lane and single-byte
// stores took 55 and 73 us at 3860 x 4548.  The workgroup covers up to 8192
// pixels at once, so a row is one step; a thread's pixels and their neighbours
// are three loads of aligned words; their roles are bit masks, a dozen
// operations for all eight (36 and 49 us with a compare and a select each);
// and pass 2 puts the row's bytes together
// in LDS and writes them out as words: 17 and 26 us.

constexpr int kTgaHead = 18, kTgaFoot = 26;
constexpr int kTgaPx = 8;  // pixels per thread per step
__constant__ char kTgaSig[18] = "TRUEVISION-XFILE.";  // footer signature (with its zero)

__device__ __forceinline__ uint32_t px3(const uint8_t *row, int32_t x) {
  const uint8_t *p = row + 3 * (int64_t)x;
  return (uint32_t)p[0] | ((uint32_t)p[1] << 8) | ((uint32_t)p[2] << 16);
}

typedef uint32_t vw4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t vw2 __attribute__((ext_vector_type(2), aligned(4)));

// The 12 pixels from p (any alignment), R G B in the low bytes, from the ten
// aligned words they lie in.
__device__ __forceinline__ void load_px12(const uint8_t *p, uint32_t w[kTgaPx + 4]) {
  const uint32_t sh = (uint32_t)((uintptr_t)p & 3u);
  const uint32_t *a = (const uint32_t *)((uintptr_t)p & ~(uintptr_t)3);
  const vw4 u0 = *(const vw4 *)a, u1 = *(const vw4 *)(a + 4);
  const vw2 u2 = *(const vw2 *)(a + 8);
  const uint32_t u[10] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w, u2.x, u2.y};
  uint32_t v[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) v[i] = __builtin_amdgcn_alignbyte(u[i + 1], u[i], sh);
#pragma unroll
  for (int k = 0; k < kTgaPx + 4; ++k) {
    const int b = 3 * k, i = b >> 2, r = b & 3;
    const uint32_t x = r < 2 ? v[i] >> (8 * r) : __builtin_amdgcn_alignbyte(v[i + 1], v[i], r);
    w[k] = x & 0xFFFFFFu;
  }
}

// Inclusive sum over the wave's lanes by DPP: shifts within each row of 16
// lanes, then the sums of the rows before.
__device__ __forceinline__ int32_t wave_sum_scan(int32_t x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
  return x;
}

template <bool WRITE>
__global__ __launch_bounds__(1024) void k_tga_rows(const uint8_t *__restrict__ rgb, int32_t W,
                                                   int32_t H, int64_t *__restrict__ row_bytes,
                                                   const int64_t *__restrict__ row_off,
                                                   const int64_t *__restrict__ total,
                                                   uint8_t *__restrict__ out) {
  extern __shared__ uint32_t stage32[];  // WRITE: the step's bytes, 4 a pixel at most, and 4 more
  uint8_t *const stage = (uint8_t *)stage32;
  __shared__ int32_t wave_start[16], wave_bytes[16];  // per wave: last segment start, bytes
  const int32_t y = blockIdx.x;
  const int32_t t = threadIdx.x, lane = t & 63, wv = t >> 6, n_wv = (int32_t)blockDim.x >> 6;
  const uint8_t *row = rgb + (int64_t)y * W * 3;
  const uint8_t *const img_end = rgb + (int64_t)H * W * 3;
  if (WRITE && y == 0) {
    // header (no image id or colour map, type 10, width, height, 24 bits, rows
    // top first) and footer (no extension or developer area, the signature)
    if (t < kTgaHead) {
      uint8_t v = 0;
      switch (t) {
        case 2: v = 10; break;
        case 12: v = (uint8_t)(W & 255); break;
        case 13: v = (uint8_t)(W >> 8); break;
        case 14: v = (uint8_t)(H & 255); break;
        case 15: v = (uint8_t)(H >> 8); break;
        case 16: v = 24; break;
        case 17: v = 0x20; break;
        default: break;
      }
      out[t] = v;
    } else if (t < kTgaHead + kTgaFoot) {
      const int32_t k = t - kTgaHead;  // footer byte
      out[*total - kTgaFoot + k] = k < 8 ? (uint8_t)0 : (uint8_t)kTgaSig[k - 8];
    }
  }
  int64_t done = WRITE ? row_off[y] : 0;  // WRITE: where the step's bytes go; else bytes so far
  int32_t open_seg = 0;  // first pixel of the segment still open at the step's start
  for (int32_t x0 = 0; x0 < W; x0 += (int32_t)blockDim.x * kTgaPx) {
    const int32_t xb = x0 + kTgaPx * t;  // this thread's first pixel
    // the thread's pixels and two neighbours on each side
    // (bit k of the masks below: pixel xb - 2 + k)
    uint32_t w[kTgaPx + 4];
    const int32_t lo_k = max(0, 2 - xb), hi_k = min(kTgaPx + 4, W - xb + 2);
    const uint32_t has = hi_k > lo_k ? ((1u << hi_k) - 1u) & ~((1u << lo_k) - 1u) : 0u;
    const uint8_t *const p = row + 3 * (int64_t)(xb - 2);
    const uintptr_t a = (uintptr_t)p & ~(uintptr_t)3;
    if (a >= (uintptr_t)rgb && a + 40 <= (uintptr_t)img_end) {  // (within the image's bytes)
      load_px12(p, w);
    } else {
#pragma unroll
      for (int k = 0; k < kTgaPx + 4; ++k) w[k] = ((has >> k) & 1u) ? px3(row, xb - 2 + k) : 0u;
    }
    uint32_t eq = 0;  // equal to the next pixel
#pragma unroll
    for (int k = 0; k < kTgaPx + 3; ++k) eq |= w[k] == w[k + 1] ? 1u << k : 0u;
    eq &= has & (has >> 1);
    constexpr uint32_t kMine = ((1u << kTgaPx) - 1u) << 2;
    const uint32_t run = eq | (eq << 1);  // (of pixels 1 to 10)
    // a segment starts at a row's first pixel, where the role changes, and in a
    // run where the colour does; it ends where the next one starts
    const uint32_t starts = has & (~(has << 1) | (run ^ (run << 1)) | (run & ~(eq << 1)));
    const uint32_t ends = has & (~(has >> 1) | (starts >> 1));
    const uint32_t mine = has & kMine;
    const uint32_t my_starts = starts & kMine;
    const int32_t last_start = my_starts ? xb - 2 + 31 - __builtin_clz(my_starts) : -1;
    // last segment start of the threads below and of the wave
    const uint64_t sm = __ballot(my_starts != 0);
    const uint64_t lower = sm & ((1ull << lane) - 1ull);
    const int32_t src = lower ? 63 - __builtin_clzll(lower) : 0;
    int32_t below = __shfl(last_start, src);
    if (!lower) below = -1;
    const int32_t m = max(below, last_start);
    if (lane == 63) wave_start[wv] = m;
    __syncthreads();
    int32_t step_last = -1;
    for (int32_t k = 0; k < n_wv; ++k) {
      const int32_t v = wave_start[k];
      if (k < wv) below = max(below, v);
      step_last = max(step_last, v);
    }
    const int32_t seg_before = below >= 0 ? below : open_seg;
    // Packets: the open segment's may end and begin at one place here, 128
    // pixels on (a segment that starts here has no second packet here).
    const int32_t k_in = (xb - seg_before) & 127;  // position of the first pixel in its packet
    const uint32_t open = my_starts ? (my_starts & -my_starts) - 1u : ~0u;  // before the first start
    const int32_t cut = (128 - k_in) & 127;  // pixel (of mine) where a packet begins
    const uint32_t cut_bit = cut < kTgaPx ? (4u << cut) & open : 0u;
    const uint32_t cut_end = k_in + kTgaPx > 127 ? (4u << (127 - k_in)) & open : 0u;
    const uint32_t firsts = (starts | cut_bit) & mine, lasts = (ends | cut_end) & mine;
    const uint32_t raw = mine & ~run;
    const int32_t sum = 3 * __popc(raw) + __popc(raw & firsts) + 4 * __popc(mine & run & lasts);
    const int32_t incl = wave_sum_scan(sum);
    if (lane == 63) wave_bytes[wv] = incl;
    __syncthreads();
    int32_t before = 0, step_bytes = 0;
    for (int32_t k = 0; k < n_wv; ++k) {
      const int32_t v = wave_bytes[k];
      if (k < wv) before += v;
      step_bytes += v;
    }
    if (WRITE) {
      // byte `at` of the step is stage[off + at]: words of the stage and of the
      // file then have the same alignment
      const int32_t off = (int32_t)((uintptr_t)(out + done) & 3u);
      int32_t at = before + incl - sum, kk = k_in - 1;
#pragma unroll
      for (int j = 0; j < kTgaPx; ++j) {
        const uint32_t bit = 4u << j;
        kk = (firsts & bit) ? 0 : kk + 1;  // position in its packet
        const uint32_t p0 = w[j + 2];
        const uint8_t r = (uint8_t)(p0 & 255u), g = (uint8_t)((p0 >> 8) & 255u), b = (uint8_t)(p0 >> 16);
        if (raw & bit) {
          uint8_t *const q = stage + off + at + ((firsts & bit) ? 1 : 0);
          q[0] = b;
          q[1] = g;
          q[2] = r;
          // the header sits before the packet's first pixel: 1 + 3 kk bytes
          // back, in the file already when that was in the previous step
          // (whose stores the barriers since have completed)
          if (lasts & bit) {
            const int32_t ha = (firsts & bit) ? at : at - 1 - 3 * kk;
            if (ha >= 0) stage[off + ha] = (uint8_t)kk;
            else out[done + ha] = (uint8_t)kk;
          }
          at += (firsts & bit) ? 4 : 3;
        } else if (mine & lasts & bit) {
          uint8_t *const q = stage + off + at;
          q[0] = (uint8_t)(0x80 | kk);
          q[1] = b;
          q[2] = g;
          q[3] = r;
          at += 4;
        }
      }
      __syncthreads();
      // whole words of the file, then the bytes before and after them
      uint8_t *const base = out + done - off;  // (word-aligned)
      const int32_t lo = off ? 1 : 0, hi = (off + step_bytes) >> 2;
      for (int32_t i = lo + t; i < hi; i += (int32_t)blockDim.x) ((uint32_t *)base)[i] = stage32[i];
      if (hi < lo) {  // all within one word
        if (t >= off && t < off + step_bytes) base[t] = stage[t];
      } else {
        if (t >= off && t < 4 * lo) base[t] = stage[t];
        if (t < 4 && 4 * hi + t < off + step_bytes) base[4 * hi + t] = stage[4 * hi + t];
      }
    }
    done += step_bytes;
    if (step_last >= 0) open_seg = step_last;
    __syncthreads();  // (the shared arrays are free for the next step)
  }
  if (!WRITE && t == 0) row_bytes[y] = done;
}

// Row offsets (exclusive sum of row sizes, after the header) and the file
// size (also to pinned host memory), in one workgroup: each thread sums a contiguous block of rows, the
// block sums are scanned in LDS, then each thread writes its rows' offsets.
__global__ __launch_bounds__(1024) void k_tga_offsets(const int64_t *__restrict__ row_bytes,
                                                      int32_t H, int64_t *__restrict__ row_off,
                                                      int64_t *__restrict__ total,
                                                      int64_t *__restrict__ h_total) {
  __shared__ int64_t part[1024];
  const int32_t t = threadIdx.x;
  const int32_t per = (H + 1023) / 1024;
  const int32_t b = min(H, t * per), e = min(H, b + per);
  int64_t s = 0;
  for (int32_t i = b; i < e; ++i) s += row_bytes[i];
  part[t] = s;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {
    const int64_t v = t >= d ? part[t - d] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int64_t at = kTgaHead + (t ? part[t - 1] : 0);
  for (int32_t i = b; i < e; ++i) {
    row_off[i] = at;
    at += row_bytes[i];
  }
  if (t == 1023) *total = *h_total = kTgaHead + part[1023] + kTgaFoot;
}

}  // namespace

namespace trh {

hipError_t launch_aa_mean(float *rgb, const float *planes, int32_t n_planes, int64_t n,
                          hipStream_t st) {
  if (n <= 0 || n_planes <= 0) return hipSuccess;
  int64_t blocks = (n + kThreads - 1) / kThreads;
  if (blocks > 8192) blocks = 8192;  // grid-stride beyond 2M threads
  k_aa_mean<<<(unsigned)blocks, kThreads, 0, st>>>(rgb, planes, n_planes, n, (float)(n_planes + 1));
  return hipGetLastError();
}

hipError_t launch_quantize_rgb8(const float *in, int64_t n, uint8_t *out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const bool aligned = ((uintptr_t)in % 16 == 0) && ((uintptr_t)out % 4 == 0);
  int64_t done = 0;
  if (aligned) {
    const int64_t n4 = n / 4;
    if (n4 > 0) {
      const int64_t blocks = (n4 + kGroups - 1) / kGroups;
      k_quantize_vec<<<(unsigned)blocks, kThreads, 0, st>>>((const vf4 *)in, (uint32_t *)out, n4);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    done = n4 * 4;
  }
  const int64_t rest = n - done;
  if (rest > 0) {
    const int64_t blocks = (rest + kThreads - 1) / kThreads;
    k_quantize_scalar<<<(unsigned)blocks, kThreads, 0, st>>>(in + done, out + done, rest);
  }
  return hipGetLastError();
}

}  // namespace trh

namespace trh {

// Threads per row: enough for the row in one step, in whole waves.
static unsigned tga_threads(int32_t W) {
  const int n = (W + kTgaPx - 1) / kTgaPx;
  return (unsigned)std::min(1024, (n + 63) / 64 * 64);
}

hipError_t launch_tga_sizes(const uint8_t *rgb, int32_t W, int32_t H, int64_t *row_bytes,
                            int64_t *row_off, int64_t *total, int64_t *h_total, hipStream_t st) {
  k_tga_rows<false><<<(unsigned)H, tga_threads(W), 0, st>>>(rgb, W, H, row_bytes, nullptr, nullptr, nullptr);
  k_tga_offsets<<<1, 1024, 0, st>>>(row_bytes, H, row_off, total, h_total);
  return hipGetLastError();
}

hipError_t launch_tga_write(const uint8_t *rgb, int32_t W, int32_t H, const int64_t *row_off,
                            const int64_t *total, uint8_t *out, hipStream_t st) {
  const unsigned n = tga_threads(W);
  k_tga_rows<true><<<(unsigned)H, n, n * kTgaPx * 4 + 8, st>>>(rgb, W, H, nullptr, row_off, total, out);
  return hipGetLastError();
}

}  // namespace trh
