// The loss of Sec. 4.5, (1 - lambda) L1 + lambda (1 - mean SSIM), and its
// image gradient, over every view of a frame (images concatenated).
//
// SSIM per pixel and channel from local statistics under an 11 x 11
// Gaussian window (sigma 1.5, zero padding outside the view): means m_x,
// m_y and second moments s_xx, s_yy, s_xy;
//   S = (2 m_x m_y + C1)(2 (s_xy - m_x m_y) + C2)
//       / ((m_x^2 + m_y^2 + C1)((s_xx - m_x^2) + (s_yy - m_y^2) + C2)).
// The gradient of the mean of S with respect to the image is the window
// applied once more, to the per-pixel partials of S with respect to m_x,
// s_xx and s_xy:
//   dS/dx(p) = sum_q G(q - p) [dS/dm_x(q) + 2 x(p) dS/ds_xx(q) + y(p) dS/ds_xy(q)].
// Two stencil kernels over tiles of kTileW x kTileH pixels, a workgroup of
// three wavefronts (one per channel) each (frames of few tiles: two others, at
// the end of the file):
//   ssim_fwd  statistics, S, the three partials (times -lambda / n) to the
//             workspace (nine planes of all pixels: partial k of channel c
//             in plane 3 c + k), per-tile sums of S and |x - y|
//   ssim_bwd  the window over the partials, the L1 term, d_image
// and one workgroup adds the per-tile sums into the loss.
//
// A wavefront walks down its tile row by row (kTileH + 10 rows).  Each lane
// has two neighbouring columns: the row's window sums from 12 values a plane
// (six 8-byte LDS reads; the row was staged by the whole wavefront, and the
// next two are already on their way from memory), then one step of the column
// pass, in which a row's value goes into the eleven outputs it belongs to: ten
// registers a plane and column that shift by one as they are added to
// (acc[j] = g h + acc[j + 1]).  SSIM depends on the second moments of x and y
// through their sum only, so four planes are windowed, x, y, x^2 + y^2 and
// x y.  (The sum's rounding is that of a larger number than either square's: the
// gradient's error against float64 is 4.1e-6 at 1080p with noise of 0.1, with
// five planes 4.0e-6, and 1.8e-5 against 1.5e-5 on smooth images with noise of
// 0.01.)  No barriers.  kTileH: 1080p gives three wavefronts per SIMD; 24 and 32
// rows have fewer halo rows but leave the SIMDs unevenly loaded (fwd 59 and
// 66, bwd 54 and 104 us).
// Bound by instruction issue, 79 % of the cycles forward and 57 % backward
// (which reads 133 MB in its 48 us): 1080p 89 -> 51 us forward, 85 -> 48 us
// backward against 16x16 tiles with an LDS patch per channel (676 columns of
// work for 256 pixels in its row pass, a barrier after every pass).
#include <cmath>
#include <vector>

#include "ubs_internal.hpp"

namespace ubs {

constexpr int kSsimR = 5;                        // window half-width
constexpr int kTaps = 2 * kSsimR + 1;
constexpr int kTileW = 128, kTileH = 16;         // two columns per lane
constexpr int kRowW = kTileW + 2 * kSsimR;       // 138 staged pixels of a row
constexpr int kRowPad = 140;
constexpr int kSsimThreads = 192;                // one wavefront per channel
constexpr float kC1 = 0.01f * 0.01f;
constexpr float kC2 = 0.03f * 0.03f;
constexpr int kSsimViewChunk = 64;
// Which frames take the kernels for few tiles, of 16 x 16 pixels: those of up to
// kFewTiles such tiles (loss and gradient in us, these / the walk: 2040 tiles
// 59 / 67, 2268 64 / 68, 2400 67 / 68, 2772 69 / 69, 3600 80 / 70), and those of
// narrow views, whose 128 x 16 tiles are so empty that they hold at most
// kFewPerWalk tiles of 16 x 16 each (1024 views of 32x32, two each, 105 / 196;
// 33x16384, three, 70 / 89; 1000 views of 48x48, three, 201 / 255; 64x16384,
// four, 103 / 89; 1024 views of 64x64, four, 370 / 333).
constexpr uint64_t kFewTiles = 2304, kFewPerWalk = 3;
// Of those, frames of up to this many tiles take a workgroup's three channels
// side by side (64x48 15.1 us, one after the other 19.7; 320x180 18 / 22;
// 480x270, 510 tiles, 25.0 / 26.7): two such workgroups fit a CU.  More tiles
// take workgroups of one channel at a time, of which eight fit (500x290, 608
// tiles, 32.3 / 29.0; 640x480 42.5 / 35.9).
constexpr uint64_t kFewOneRound = 512;

struct SsimView {
  int32_t W, H, tiles_x;
  uint32_t tile_base, pix_base;
  uint32_t _pad[3];
};

struct SsimViewChunk {
  SsimView v[kSsimViewChunk];
  int32_t first, count;
};

// Up to kFewViews descriptors travel with the launches; more are written to
// the workspace first, a launch of its own that takes 4 us and that the
// forward waits for.
constexpr int kFewViews = 8;
struct SsimViews {
  SsimView few[kFewViews];
  const SsimView* many;   // or nullptr
  int32_t n;
};

__global__ void ssim_upload_kernel(SsimViewChunk c, SsimView* __restrict__ dst) {
  const int k = threadIdx.x;
  if (k < c.count) dst[c.first + k] = c.v[k];
}

// Normalised taps of the 11-tap Gaussian (sigma 1.5), filled by the host.
struct SsimTaps {
  float g[2 * kSsimR + 1];
};

__device__ __forceinline__ SsimView ssim_view_of_tile(const SsimViews& vs, uint32_t tile) {
  if (vs.many) {
    // the last view whose first tile is at or before this one, a wavefront's 64
    // probes at a time (two rounds of loads for 1024 views, where a binary
    // search waits for ten, one after the other: 1024 views of 32x32 137 -> 130 us)
    int lo = 0, n = vs.n;
    while (n > 1) {
      const int step = (n + 63) / 64, at = int(threadIdx.x & 63) * step;
      const bool past = at < n && vs.many[lo + at].tile_base <= tile;
      const int k = __builtin_amdgcn_readfirstlane(63 - __clzll(__ballot(past))) * step;
      lo += k;
      n = min(step, n - k);
    }
    return vs.many[lo];
  }
  SsimView v = vs.few[0];
#pragma unroll
  for (int k = 1; k < kFewViews; ++k)
    if (k < vs.n && vs.few[k].tile_base <= tile) v = vs.few[k];
  return v;
}

// S of one pixel and channel from its windowed x, y, x^2 + y^2 and x y; d: its
// partials with respect to m_x, s_xx and s_xy, times scale.
__device__ __forceinline__ float ssim_point(const float (&st)[4], float scale, float (&d)[3]) {
  const float mx = st[0], my = st[1];
  const float m2 = mx * mx + my * my;
  const float a1 = 2.0f * mx * my + kC1;
  const float a2 = 2.0f * (st[3] - mx * my) + kC2;
  const float b1 = m2 + kC1;
  const float b2 = (st[2] - m2) + kC2;
  const float ib = 1.0f / (b1 * b2);
  const float ib1 = b2 * ib, ib2 = b1 * ib;
  const float S = a1 * a2 * ib;
  const float d_m = 2.0f * my * (a2 - a1) * ib - 2.0f * mx * S * (ib1 - ib2);
  d[0] = scale * d_m;
  d[1] = scale * (-S * ib2);
  d[2] = scale * (2.0f * a1 * ib);
  return S;
}

// a b + c into a register of its own: the compiler would add into c and copy
// the sum to where it is wanted, which doubles the column pass.
__device__ __forceinline__ float fma_to(float a, float b, float c) {
  float d;
  asm("v_fma_f32 %0, %1, %2, %3" : "=v"(d) : "s"(a), "v"(b), "v"(c));
  return d;
}

// One step of the column pass of one plane and column: h, the row's window
// sum, goes into the eleven outputs it belongs to; returns the one it
// completes (the output kSsimR rows above).
__device__ __forceinline__ float column_step(float (&acc)[kTaps - 1], const SsimTaps& t, float h) {
  const float out = fma_to(t.g[kTaps - 1], h, acc[0]);
#pragma unroll
  for (int j = 0; j + 1 < kTaps - 1; ++j) acc[j] = fma_to(t.g[kTaps - 2 - j], h, acc[j + 1]);
  acc[kTaps - 2] = t.g[0] * h;
  return out;
}

// The row's window sums of a lane's two columns, of one staged plane: twelve
// values, v[5] and v[6] are the columns' own.
__device__ __forceinline__ void row_pass(const float* row, int lane, const SsimTaps& t,
                                         float (&v)[kTaps + 1], float (&h)[2]) {
  const float2* p = reinterpret_cast<const float2*>(row) + lane;
#pragma unroll
  for (int k = 0; k < (kTaps + 1) / 2; ++k) {
    const float2 x = p[k];
    v[2 * k] = x.x;
    v[2 * k + 1] = x.y;
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    h[c] = t.g[0] * v[c];
#pragma unroll
    for (int k = 1; k < kTaps; ++k) h[c] += t.g[k] * v[c + k];
  }
}

// Two neighbouring floats; a row of an odd width starts at any 4 bytes.
typedef float Pair __attribute__((ext_vector_type(2), aligned(4)));

struct SsimTileAt {
  int W, H, x0, y0, rows;   // the view's size, the tile's first pixel, its rows
  size_t pix;               // the view's first pixel
};
__device__ __forceinline__ SsimTileAt ssim_tile_at(const SsimViews& views, uint32_t tile) {
  const SsimView V = ssim_view_of_tile(views, tile);
  const int lt = int(tile - V.tile_base);
  const int ty = lt / V.tiles_x, tx = lt - ty * V.tiles_x;
  SsimTileAt t;
  t.W = V.W;
  t.H = V.H;
  t.x0 = tx * kTileW;
  t.y0 = ty * kTileH;
  t.rows = min(kTileH, V.H - t.y0);
  t.pix = V.pix_base;
  return t;
}

// LDS accesses of a wavefront's lanes before and after it stay in that order
// (the hardware executes them in order; this holds the compiler to it).
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}

constexpr int kRowLoads = (kRowW + 63) / 64;   // staged pixels per lane

// A lane's staged columns x0 - 5 + lane + 64 m: clamped into the row (what
// was loaded for a column outside is replaced by 0).
struct RowColumns {
  int at[kRowLoads];
  bool in[kRowLoads];
};
__device__ __forceinline__ RowColumns row_columns(const SsimTileAt& t, int lane) {
  RowColumns r;
#pragma unroll
  for (int m = 0; m < kRowLoads; ++m) {
    const int gx = t.x0 - kSsimR + lane + 64 * m;
    r.in[m] = gx >= 0 && gx < t.W;
    r.at[m] = min(max(gx, 0), t.W - 1);
  }
  return r;
}

__global__ void __launch_bounds__(kSsimThreads) ssim_fwd_kernel(
    SsimViews views, const float* __restrict__ image, const float* __restrict__ target,
    SsimTaps taps, float scale, float* __restrict__ dstat, uint32_t n_pixels, double* __restrict__ tile_sums) {
  __shared__ __align__(16) float s_row[3][4][kRowPad];
  __shared__ double s_red[2][3];
  const uint32_t tile = blockIdx.x;
  const int lane = threadIdx.x & 63, ch = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const SsimTileAt at = ssim_tile_at(views, tile);
  const RowColumns cols = row_columns(at, lane);
  float(*row_of)[kRowPad] = s_row[ch];
  struct Loaded {
    float x[kRowLoads], y[kRowLoads];
  };
  auto load = [&](Loaded& to, int row) {
    const size_t first = 3 * (at.pix + size_t(min(max(at.y0 - kSsimR + row, 0), at.H - 1)) * at.W) + ch;
    const float *ix = image + first, *iy = target + first;
#pragma unroll
    for (int m = 0; m < kRowLoads; ++m) {
      const uint32_t o = 3u * uint32_t(cols.at[m]);
      to.x[m] = ix[o];
      to.y[m] = iy[o];
    }
  };
  float acc[2][4][kTaps - 1];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int j = 0; j < kTaps - 1; ++j) acc[c][q][j] = 0.0f;
  double s_sum = 0.0, l1_sum = 0.0;
  const int px = at.x0 + 2 * lane;
  const bool two = px + 1 < at.W;
  const int n_rows = at.rows + 2 * kSsimR;
  auto step = [&](Loaded& in_row, int row) {
    const bool row_in = at.y0 - kSsimR + row >= 0 && at.y0 - kSsimR + row < at.H;
    wave_order();
#pragma unroll
    for (int m = 0; m < kRowLoads; ++m)
      if (lane + 64 * m < kRowW) {
        const int i = lane + 64 * m;
        const bool in = row_in && cols.in[m];
        const float x = in ? in_row.x[m] : 0.0f, y = in ? in_row.y[m] : 0.0f;
        row_of[0][i] = x;
        row_of[1][i] = y;
        row_of[2][i] = x * x + y * y;
        row_of[3][i] = x * y;
      }
    wave_order();
    if (row + 2 < n_rows) load(in_row, row + 2);
    float st[2][4], own[2][2];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float v[kTaps + 1], h[2];
      row_pass(row_of[q], lane, taps, v, h);
      if (q < 2) {
        own[0][q] = v[kSsimR];
        own[1][q] = v[kSsimR + 1];
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) st[c][q] = column_step(acc[c][q], taps, h[c]);
    }
    // |x - y| of the row's own pixels (columns outside hold 0)
    if (row >= kSsimR && row < at.rows + kSsimR)
      l1_sum += double(fabsf(own[0][0] - own[0][1])) +
                (two ? double(fabsf(own[1][0] - own[1][1])) : 0.0);
    if (row < 2 * kSsimR) return;
    float d[2][3];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const float S = ssim_point(st[c], scale, d[c]);
      if (px + c < at.W) s_sum += double(S);
    }
    float* out = dstat + size_t(3 * ch) * n_pixels + at.pix +
                 size_t(at.y0 - 2 * kSsimR + row) * at.W;
    if (two) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        *reinterpret_cast<Pair*>(out + k * size_t(n_pixels) + uint32_t(px)) = Pair{d[0][k], d[1][k]};
    } else if (px < at.W) {
#pragma unroll
      for (int k = 0; k < 3; ++k) out[k * size_t(n_pixels) + uint32_t(px)] = d[0][k];
    }
  };
  Loaded even, odd;
  load(even, 0);
  load(odd, 1);
  for (int row = 0; row < n_rows; row += 2) {
    step(even, row);
    if (row + 1 < n_rows) step(odd, row + 1);
  }
  // tile sums of S and |x - y|
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    s_sum += __shfl_xor(s_sum, o, 64);
    l1_sum += __shfl_xor(l1_sum, o, 64);
  }
  if (lane == 0) {
    s_red[0][ch] = s_sum;
    s_red[1][ch] = l1_sum;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    tile_sums[2 * size_t(tile)] = s_red[0][0] + s_red[0][1] + s_red[0][2];
    tile_sums[2 * size_t(tile) + 1] = s_red[1][0] + s_red[1][1] + s_red[1][2];
  }
}

__global__ void __launch_bounds__(kSsimThreads) ssim_bwd_kernel(
    SsimViews views, const float* __restrict__ image, const float* __restrict__ target, SsimTaps taps, float l1_weight,
    const float* __restrict__ dstat, uint32_t n_pixels, float* __restrict__ d_image) {
  __shared__ __align__(16) float s_row[3][3][kRowPad];
  const int lane = threadIdx.x & 63, ch = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const SsimTileAt at = ssim_tile_at(views, blockIdx.x);
  const RowColumns cols = row_columns(at, lane);
  float(*row_of)[kRowPad] = s_row[ch];
  struct Loaded {
    float v[3][kRowLoads];
  };
  auto load = [&](Loaded& to, int row) {
    const float* plane = dstat + size_t(3 * ch) * n_pixels + at.pix +
                         size_t(min(max(at.y0 - kSsimR + row, 0), at.H - 1)) * at.W;
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int m = 0; m < kRowLoads; ++m)
        to.v[p][m] = plane[p * size_t(n_pixels) + uint32_t(cols.at[m])];
  };
  float acc[2][3][kTaps - 1];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int j = 0; j < kTaps - 1; ++j) acc[c][q][j] = 0.0f;
  const int px = at.x0 + 2 * lane;
  uint32_t own[2];   // the lane's two columns, clamped into the row
#pragma unroll
  for (int c = 0; c < 2; ++c) own[c] = 3u * uint32_t(min(px + c, at.W - 1));
  const int n_rows = at.rows + 2 * kSsimR;
  auto step = [&](Loaded& in_row, int row) {
    const bool row_in = at.y0 - kSsimR + row >= 0 && at.y0 - kSsimR + row < at.H;
    wave_order();
#pragma unroll
    for (int m = 0; m < kRowLoads; ++m)
      if (lane + 64 * m < kRowW)
#pragma unroll
        for (int p = 0; p < 3; ++p)
          row_of[p][lane + 64 * m] = row_in && cols.in[m] ? in_row.v[p][m] : 0.0f;
    wave_order();
    // the output row's own pixels (loads return in order: asked for after the
    // next row, they would wait for it)
    const size_t first = 3 * (at.pix + size_t(at.y0 + max(row - 2 * kSsimR, 0)) * at.W) + ch;
    float ix[2], iy[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      ix[c] = image[first + own[c]];
      iy[c] = target[first + own[c]];
    }
    __builtin_amdgcn_sched_barrier(0);
    if (row + 2 < n_rows) load(in_row, row + 2);
    float w[2][3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      float v[kTaps + 1], h[2];
      row_pass(row_of[p], lane, taps, v, h);
#pragma unroll
      for (int c = 0; c < 2; ++c) w[c][p] = column_step(acc[c][p], taps, h[c]);
    }
    if (row < 2 * kSsimR) return;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const float diff = ix[c] - iy[c];
      const float sgn = diff > 0.0f ? 1.0f : (diff < 0.0f ? -1.0f : 0.0f);
      const float g = w[c][0] + 2.0f * ix[c] * w[c][1] + iy[c] * w[c][2] + l1_weight * sgn;
      if (px + c < at.W) d_image[first + own[c]] = g;
    }
  };
  Loaded even, odd;
  load(even, 0);
  load(odd, 1);
  for (int row = 0; row < n_rows; row += 2) {
    step(even, row);
    if (row + 1 < n_rows) step(odd, row + 1);
  }
}

// ---------------------------------------------------------------------------
// Frames of few tiles: a wavefront that walks 26 rows is then all that a SIMD
// has, and takes a microsecond a row.  These kernels take a tile of 16 x 16 by
// kFewThreads threads per channel, all of a patch at once, passes separated by
// barriers; the chip's idle SIMDs pay for the halo.  NCH channels side by side,
// the others one after the other.
// ---------------------------------------------------------------------------
constexpr int kSsimTile = 16;
constexpr int kSsimP = kSsimTile + 2 * kSsimR;   // 26
constexpr int kSsimTmpW = kSsimTile + 1;         // padded row of the row-pass buffer (LDS banks)
constexpr int kFewThreads = 256;

// Separable window over an LDS patch, NQ quantities at once: rows first
// (kSsimP rows x 16 columns into tmp), then columns (16 x 16, left in
// in[q][r][c] for r, c < 16, from where each thread reads its pixel).  A
// thread computes 8 consecutive outputs from 18 consecutive inputs held in
// registers (a sliding window), so each output costs about 2.3 LDS reads
// instead of 11.  in[q][kSsimP][kSsimP], tmp[q][kSsimP][kSsimTmpW].
constexpr int kSsimRun = 8;                       // outputs per thread and pass
constexpr int kSsimSpan = kSsimRun + 2 * kSsimR;  // 18 inputs per run

template <int NQ>
__device__ __forceinline__ void window_16x16(float (*in)[kSsimP][kSsimP],
                                             float (*tmp)[kSsimP][kSsimTmpW], const SsimTaps& t,
                                             float* out) {
  const int tid = threadIdx.x % kFewThreads;
  constexpr int kRuns = kSsimTile / kSsimRun;     // 2 runs per row or column
  // rows: task = (q, r, run)
  for (int task = tid; task < NQ * kSsimP * kRuns; task += kFewThreads) {
    const int q = task / (kSsimP * kRuns), rem = task % (kSsimP * kRuns);
    const int r = rem / kRuns, c0 = (rem % kRuns) * kSsimRun;
    float v[kSsimSpan];
#pragma unroll
    for (int k = 0; k < kSsimSpan; ++k) v[k] = in[q][r][c0 + k];
#pragma unroll
    for (int o = 0; o < kSsimRun; ++o) {
      float acc = 0.0f;
#pragma unroll
      for (int k = 0; k <= 2 * kSsimR; ++k) acc += t.g[k] * v[o + k];
      tmp[q][r][c0 + o] = acc;
    }
  }
  __syncthreads();
  // columns: task = (q, c, run), results into in[q][r][c]
  for (int task = tid; task < NQ * kSsimTile * kRuns; task += kFewThreads) {
    const int q = task / (kSsimTile * kRuns), rem = task % (kSsimTile * kRuns);
    const int c = rem % kSsimTile, r0 = (rem / kSsimTile) * kSsimRun;
    float v[kSsimSpan];
#pragma unroll
    for (int k = 0; k < kSsimSpan; ++k) v[k] = tmp[q][r0 + k][c];
#pragma unroll
    for (int o = 0; o < kSsimRun; ++o) {
      float acc = 0.0f;
#pragma unroll
      for (int k = 0; k <= 2 * kSsimR; ++k) acc += t.g[k] * v[o + k];
      in[q][r0 + o][c] = acc;
    }
  }
  __syncthreads();
  const int r = tid / kSsimTile, c = tid % kSsimTile;
#pragma unroll
  for (int q = 0; q < NQ; ++q) out[q] = in[q][r][c];
}

struct FewTileAt {
  int W, H, tx, ty;
  size_t pix;   // the view's first pixel
};
__device__ __forceinline__ FewTileAt few_tile_at(const SsimViews& views, uint32_t tile) {
  const SsimView V = ssim_view_of_tile(views, tile);
  const int lt = int(tile - V.tile_base);
  const int ty = lt / V.tiles_x;
  return FewTileAt{V.W, V.H, lt - ty * V.tiles_x, ty, size_t(V.pix_base)};
}

template <int NCH>
__global__ void __launch_bounds__(NCH * kFewThreads) ssim_fwd_few_kernel(
    SsimViews views, const float* __restrict__ image, const float* __restrict__ target,
    SsimTaps taps, float scale, float* __restrict__ dstat, uint32_t n_pixels,
    double* __restrict__ tile_sums) {
  __shared__ float s_all[NCH][4][kSsimP][kSsimP];   // x, y, x^2 + y^2, x y
  __shared__ float s_tmp[NCH][4][kSsimP][kSsimTmpW];
  __shared__ double s_red[2][4 * NCH];
  const uint32_t tile = blockIdx.x;
  const FewTileAt at = few_tile_at(views, tile);
  const int wg_ch = __builtin_amdgcn_readfirstlane(threadIdx.x / kFewThreads);
  const int tid = threadIdx.x % kFewThreads;
  const int x0 = at.tx * kSsimTile - kSsimR, y0 = at.ty * kSsimTile - kSsimR;
  const int r = tid / kSsimTile, c = tid % kSsimTile;
  const int px = at.tx * kSsimTile + c, py = at.ty * kSsimTile + r;
  float(*s_in)[kSsimP][kSsimP] = s_all[wg_ch];
  double s_sum = 0.0, l1_sum = 0.0;
#pragma unroll 1
  for (int ch = wg_ch; ch < 3; ch += NCH) {
    for (int e = tid; e < kSsimP * kSsimP; e += kFewThreads) {
      const int pr = e / kSsimP, pc = e % kSsimP;
      const int gx = x0 + pc, gy = y0 + pr;
      float a = 0.0f, b = 0.0f;
      if (gx >= 0 && gx < at.W && gy >= 0 && gy < at.H) {
        const size_t q = 3 * (at.pix + size_t(gy) * at.W + gx) + ch;
        a = image[q];
        b = target[q];
      }
      s_in[0][pr][pc] = a;
      s_in[1][pr][pc] = b;
      s_in[2][pr][pc] = a * a + b * b;
      s_in[3][pr][pc] = a * b;
    }
    __syncthreads();
    const float l1 = fabsf(s_in[0][r + kSsimR][c + kSsimR] - s_in[1][r + kSsimR][c + kSsimR]);
    __syncthreads();
    float st[4];
    window_16x16<4>(s_in, s_tmp[wg_ch], taps, st);
    if (px < at.W && py < at.H) {
      float d[3];
      s_sum += double(ssim_point(st, scale, d));
      l1_sum += double(l1);
      float* out = dstat + size_t(3 * ch) * n_pixels + at.pix + size_t(py) * at.W + px;
#pragma unroll
      for (int k = 0; k < 3; ++k) out[k * size_t(n_pixels)] = d[k];
    }
    if (NCH < 3) __syncthreads();
  }
  // tile sums of S and |x - y|
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    s_sum += __shfl_xor(s_sum, o, 64);
    l1_sum += __shfl_xor(l1_sum, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    s_red[0][threadIdx.x >> 6] = s_sum;
    s_red[1][threadIdx.x >> 6] = l1_sum;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < 4 * NCH; ++k) t += s_red[threadIdx.x][k];
    tile_sums[2 * size_t(tile) + threadIdx.x] = t;
  }
}

template <int NCH>
__global__ void __launch_bounds__(NCH * kFewThreads) ssim_bwd_few_kernel(
    SsimViews views, const float* __restrict__ image, const float* __restrict__ target,
    SsimTaps taps, float l1_weight, const float* __restrict__ dstat, uint32_t n_pixels,
    float* __restrict__ d_image) {
  __shared__ float s_all[NCH][3][kSsimP][kSsimP];   // d/dm, d/dsxx, d/dsxy
  __shared__ float s_tmp[NCH][3][kSsimP][kSsimTmpW];
  const FewTileAt at = few_tile_at(views, blockIdx.x);
  const int wg_ch = __builtin_amdgcn_readfirstlane(threadIdx.x / kFewThreads);
  const int tid = threadIdx.x % kFewThreads;
  const int x0 = at.tx * kSsimTile - kSsimR, y0 = at.ty * kSsimTile - kSsimR;
  const int px = at.tx * kSsimTile + tid % kSsimTile, py = at.ty * kSsimTile + tid / kSsimTile;
  const bool inside = px < at.W && py < at.H;
  float(*s_in)[kSsimP][kSsimP] = s_all[wg_ch];
#pragma unroll 1
  for (int ch = wg_ch; ch < 3; ch += NCH) {
    const size_t own = 3 * (at.pix + (inside ? size_t(py) * at.W + px : 0)) + ch;
    const float x = image[own], y = target[own];
    for (int e = tid; e < kSsimP * kSsimP; e += kFewThreads) {
      const int r = e / kSsimP, c = e % kSsimP;
      const int gx = x0 + c, gy = y0 + r;
      float v[3] = {0.0f, 0.0f, 0.0f};
      if (gx >= 0 && gx < at.W && gy >= 0 && gy < at.H) {
        const float* q = dstat + size_t(3 * ch) * n_pixels + at.pix + size_t(gy) * at.W + gx;
#pragma unroll
        for (int k = 0; k < 3; ++k) v[k] = q[k * size_t(n_pixels)];
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) s_in[k][r][c] = v[k];
    }
    __syncthreads();
    float w[3];
    window_16x16<3>(s_in, s_tmp[wg_ch], taps, w);
    if (inside) {
      const float diff = x - y;
      const float sgn = diff > 0.0f ? 1.0f : (diff < 0.0f ? -1.0f : 0.0f);
      d_image[own] = w[0] + 2.0f * x * w[1] + y * w[2] + l1_weight * sgn;
    }
    if (NCH < 3) __syncthreads();
  }
}

// loss = (1 - lambda) sum|x - y| / n + lambda (1 - sum S / n)
__global__ void __launch_bounds__(256) ssim_loss_kernel(const double* __restrict__ tile_sums,
                                                        uint32_t n_tiles, double n_entries,
                                                        double lambda, double* __restrict__ loss) {
  __shared__ double s_red[2][4];
  double s = 0.0, l = 0.0;
  for (uint32_t k = threadIdx.x; k < n_tiles; k += 256) {
    s += tile_sums[2 * size_t(k)];
    l += tile_sums[2 * size_t(k) + 1];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    s += __shfl_xor(s, o, 64);
    l += __shfl_xor(l, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    s_red[0][threadIdx.x >> 6] = s;
    s_red[1][threadIdx.x >> 6] = l;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double S = (s_red[0][0] + s_red[0][1]) + (s_red[0][2] + s_red[0][3]);
    const double L1 = (s_red[1][0] + s_red[1][1]) + (s_red[1][2] + s_red[1][3]);
    *loss = (1.0 - lambda) * L1 / n_entries + lambda * (1.0 - S / n_entries);
  }
}

}  // namespace ubs

using namespace ubs;

static uint64_t ssim_align(uint64_t x) { return (x + 255) & ~uint64_t(255); }

extern "C" ubs_status ubs_ssim_loss(int32_t n_views, const int32_t* sizes, const float* image,
                                    const float* target, float lambda_ssim, float* d_image,
                                    double* loss, void* ws, uint64_t ws_bytes,
                                    uint64_t* ws_bytes_needed, void* stream) {
  if (n_views < 0 || n_views > UBS_MAX_VIEWS || (n_views > 0 && !sizes)) return UBS_ERR_ARG;
  if (!(lambda_ssim >= 0.0f && lambda_ssim <= 1.0f)) return UBS_ERR_ARG;
  std::vector<SsimView> vs(size_t(n_views > 0 ? n_views : 0));
  uint64_t pixels = 0, n_walk = 0, n_few = 0;   // (tiles of 128 x 16 and of 16 x 16)
  for (int v = 0; v < n_views; ++v) {
    const int W = sizes[2 * v], H = sizes[2 * v + 1];
    if (W < 1 || H < 1 || W > 16384 || H > 16384) return UBS_ERR_ARG;
    SsimView s{};
    s.W = W;
    s.H = H;
    s.pix_base = uint32_t(pixels);
    n_walk += uint64_t((W + kTileW - 1) / kTileW) * uint64_t((H + kTileH - 1) / kTileH);
    n_few += uint64_t((W + kSsimTile - 1) / kSsimTile) * uint64_t((H + kSsimTile - 1) / kSsimTile);
    pixels += uint64_t(W) * uint64_t(H);
    if (pixels > 0x7fffffffull) return UBS_ERR_UNSUPPORTED;
    vs[size_t(v)] = s;
  }
  const uint64_t off_views = 0;
  const uint64_t off_sums = ssim_align(off_views + sizeof(SsimView) * uint64_t(n_views > 0 ? n_views : 1));
  auto dstat_at = [&](uint64_t tiles) { return ssim_align(off_sums + 16 * (tiles > 0 ? tiles : 1)); };
  auto bytes = [&](uint64_t tiles) { return ssim_align(dstat_at(tiles) + 36 * pixels); };
  bool few = n_few <= kFewTiles || n_few <= kFewPerWalk * n_walk;
  if (!ws) {
    if (!ws_bytes_needed) return UBS_ERR_ARG;
    *ws_bytes_needed = bytes(few ? n_few : n_walk);
    return UBS_OK;
  }
  // (a workspace that holds no more than the walk's fewer sums takes the walk)
  if (ws_bytes < bytes(n_few)) few = false;
  const uint64_t tiles = few ? n_few : n_walk;
  if (ws_bytes < bytes(tiles)) return UBS_ERR_CAPACITY;
  const int tile_w = few ? kSsimTile : kTileW, tile_h = few ? kSsimTile : kTileH;
  uint64_t first_tile = 0;
  for (SsimView& s : vs) {
    s.tiles_x = (s.W + tile_w - 1) / tile_w;
    s.tile_base = uint32_t(first_tile);
    first_tile += uint64_t(s.tiles_x) * uint64_t((s.H + tile_h - 1) / tile_h);
  }
  if (pixels > 0 && (!image || !target || !d_image)) return UBS_ERR_ARG;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* base = static_cast<char*>(ws);
  SsimView* dviews = reinterpret_cast<SsimView*>(base + off_views);
  double* sums = reinterpret_cast<double*>(base + off_sums);
  float* dstat = reinterpret_cast<float*>(base + dstat_at(tiles));
  SsimViews views{};
  views.n = n_views;
  for (int k = 0; k < n_views && k < kFewViews; ++k) views.few[k] = vs[size_t(k)];
  if (n_views > kFewViews) views.many = dviews;
  for (int first = 0; n_views > kFewViews && first < n_views; first += kSsimViewChunk) {
    SsimViewChunk c{};
    c.first = first;
    c.count = n_views - first < kSsimViewChunk ? n_views - first : kSsimViewChunk;
    for (int k = 0; k < c.count; ++k) c.v[k] = vs[size_t(first + k)];
    hipLaunchKernelGGL(ssim_upload_kernel, dim3(1), dim3(64), 0, st, c, dviews);
  }
  SsimTaps taps{};
  {
    double g[2 * kSsimR + 1], tot = 0.0;
    for (int k = 0; k <= 2 * kSsimR; ++k) {
      const double x = double(k - kSsimR);
      g[k] = std::exp(-x * x / (2.0 * 1.5 * 1.5));
      tot += g[k];
    }
    for (int k = 0; k <= 2 * kSsimR; ++k) taps.g[k] = float(g[k] / tot);
  }
  const double n_entries = 3.0 * double(pixels);
  if (tiles > 0) {
    const float scale = float(-double(lambda_ssim) / n_entries);
    const float l1_weight = float((1.0 - double(lambda_ssim)) / n_entries);
    const dim3 grid{unsigned(tiles)}, block{unsigned(few ? (n_few <= kFewOneRound ? 3 : 1) * kFewThreads : kSsimThreads)};
    const auto fwd = !few ? ssim_fwd_kernel
                          : (n_few <= kFewOneRound ? ssim_fwd_few_kernel<3> : ssim_fwd_few_kernel<1>);
    const auto bwd = !few ? ssim_bwd_kernel
                          : (n_few <= kFewOneRound ? ssim_bwd_few_kernel<3> : ssim_bwd_few_kernel<1>);
    hipLaunchKernelGGL(fwd, grid, block, 0, st, views, image, target, taps, scale, dstat,
                       uint32_t(pixels), sums);
    hipLaunchKernelGGL(bwd, grid, block, 0, st, views, image, target, taps, l1_weight, dstat,
                       uint32_t(pixels), d_image);
  }
  if (loss && tiles > 0)
    hipLaunchKernelGGL(ssim_loss_kernel, dim3(1), dim3(256), 0, st, sums, uint32_t(tiles),
                       n_entries, double(lambda_ssim), loss);
  return hipGetLastError() == hipSuccess ? UBS_OK : UBS_ERR_HIP;
}
