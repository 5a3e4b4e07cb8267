// Relocation of dead primitives (Sec. 4.5 cloning rule with the MCMC
// primitive management the paper adopts): every primitive whose opacity is
// below o_min (or whose parameters are not finite) copies a live primitive
// picked with probability proportional to opacity, and the N copies of a
// picked primitive (itself included) share o' = 1 - (1 - o)^(1/N).
//
//   weights   per primitive: w = o if live, -1 if dead; o kept
//   scan      inclusive float64 scan of w (exact: live opacities are
//             float32 values >= o_min, so every partial sum is a multiple
//             of 2^-31 below 2^22 for n < 2^22; the order of the additions
//             does not matter) and, in the same three launches, the exclusive
//             scan of the dead flags: a dead primitive's slot
//   sample    slot k: first j with cdf[j] > u_k * total (float64), one
//             atomic per slot on the copy count of j
//   plan      per primitive, the one whose rows it takes (its pick where it is
//             dead, itself where it is picked) or that nothing changes; the new
//             opacities
//   apply     row by row: a dead primitive takes its pick's row, the moments of
//             both are zeroed
#include <cmath>
#include <mutex>

#include "ubs_internal.hpp"

namespace ubs {

constexpr int kRelThreads = 256;
constexpr int kRelItems = 16;
constexpr int kRelTile = kRelThreads * kRelItems;

struct RelocState {
  unsigned long long n_dead;
  double total;   // cdf[n - 1]
};

struct RelocLayout {
  uint64_t cdf, o_keep, offs, src, targets, counts, sums_u32, sums_f64, state, bytes;
  uint32_t n_tiles;
};

constexpr uint64_t align256(uint64_t x) { return (x + 255) & ~uint64_t(255); }

constexpr RelocLayout reloc_layout(int64_t n) {
  RelocLayout L{};
  const uint64_t un = uint64_t(n);
  L.n_tiles = uint32_t((un + kRelTile - 1) / kRelTile);
  uint64_t off = 0;
  L.cdf = off;      off = align256(off + 8 * un);
  L.o_keep = off;   off = align256(off + 4 * un);
  L.offs = off;     off = align256(off + 4 * un);
  L.src = off;      off = align256(off + 4 * un);
  L.targets = off;  off = align256(off + 4 * un);
  L.counts = off;   off = align256(off + 4 * un);
  L.sums_u32 = off; off = align256(off + 4 * (uint64_t(L.n_tiles) + 1));
  L.sums_f64 = off; off = align256(off + 8 * (uint64_t(L.n_tiles) + 1));
  L.state = off;    off = align256(off + sizeof(RelocState));
  // the size that ws_bytes has always had to be (4 bytes a primitive are spare)
  L.bytes = align256(off + 4 * un);
  return L;
}

// Workspace of ubs_relocate_noalloc: a relocation of up to
// UBS_RELOCATE_NOALLOC_MAX_N primitives, one copy per GPU, kept for the
// life of the process.  Every word a call reads is first written by that
// call (weights, counts, scans), so nothing needs clearing between calls.
constexpr uint64_t kNoallocBytes = reloc_layout(UBS_RELOCATE_NOALLOC_MAX_N).bytes;
static __device__ __align__(256) unsigned char scratch[kNoallocBytes];

// Bound by the read of all parameters.  A value's exponent is looked at through
// its bits, so that the loads of a primitive's rows need not wait for each
// other: 38 us -> 33 us at 36 rows of 1M.
__global__ void __launch_bounds__(kRelThreads) reloc_weights_kernel(
    const float* __restrict__ params, int64_t n, int F, int o_row, float o_min,
    double* __restrict__ w, float* __restrict__ o_keep, uint32_t* __restrict__ counts) {
  const int64_t i = int64_t(blockIdx.x) * kRelThreads + threadIdx.x;
  if (i >= n) return;
  uint32_t top = 0u;   // largest magnitude's bits; infinities and NaN from 0x7f800000
  int r = 0;
  for (; r + 8 <= F; r += 8) {
    float x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = params[int64_t(r + k) * n + i];
#pragma unroll
    for (int k = 0; k < 8; ++k) top = max(top, __float_as_uint(x[k]) & 0x7fffffffu);
  }
  for (; r < F; ++r) top = max(top, __float_as_uint(params[int64_t(r) * n + i]) & 0x7fffffffu);
  const float o = params[int64_t(o_row) * n + i];
  const bool live = top < 0x7f800000u && o >= o_min;
  w[i] = live ? double(o) : -1.0;
  o_keep[i] = o;
  counts[i] = 0u;
}

// Scan of a value per thread over the workgroup: inclusive, and the total.
template <typename T>
__device__ __forceinline__ T wg_inclusive_scan(T v, T* lds4, T* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  T x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const T y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) lds4[wave] = x;
  __syncthreads();
  T base = T(0), tot = T(0);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (k < wave) base += lds4[k];
    tot += lds4[k];
  }
  __syncthreads();
  *total = tot;
  return base + x;
}

// Inclusive float64 scan of the weights and exclusive scan of the dead flags:
// per-tile sums, one workgroup scans them, apply.  A thread adds kRelItems
// consecutive weights, which it reads from LDS: from memory, 128 bytes apart
// from its neighbours', they took 19 us instead of 7 us to apply at 1M.
struct RelTile {
  double w[kRelTile + kRelThreads];   // a thread's weights start 17 doubles apart
};
__device__ __forceinline__ void load_tile(RelTile& s, const double* __restrict__ w, int64_t n,
                                          double (&vals)[kRelItems], double* sum, uint32_t* dead) {
  const int64_t base = int64_t(blockIdx.x) * kRelTile;
#pragma unroll
  for (int k = 0; k < kRelItems; ++k) {
    const int e = k * kRelThreads + int(threadIdx.x);
    s.w[e + e / kRelItems] = base + e < n ? w[base + e] : 0.0;
  }
  __syncthreads();
  *sum = 0.0;
  *dead = 0u;
#pragma unroll
  for (int k = 0; k < kRelItems; ++k) {
    vals[k] = s.w[threadIdx.x * (kRelItems + 1) + k];
    *sum += fmax(vals[k], 0.0);
    *dead += vals[k] < 0.0 ? 1u : 0u;
  }
}

__global__ void __launch_bounds__(kRelThreads) reloc_tile_sums_kernel(
    const double* __restrict__ w, int64_t n, double* __restrict__ sums,
    uint32_t* __restrict__ dead_sums) {
  __shared__ RelTile tile;
  __shared__ double lds4[4];
  __shared__ uint32_t ldsu[4];
  double vals[kRelItems], s, tot;
  uint32_t d, dtot;
  load_tile(tile, w, n, vals, &s, &d);
  wg_inclusive_scan(s, lds4, &tot);
  wg_inclusive_scan(d, ldsu, &dtot);
  if (threadIdx.x == 0) {
    sums[blockIdx.x] = tot;
    dead_sums[blockIdx.x] = dtot;
  }
}

__global__ void __launch_bounds__(kRelThreads) reloc_sums_kernel(
    double* __restrict__ sums, uint32_t* __restrict__ dead_sums, uint32_t n_tiles,
    RelocState* __restrict__ state, uint64_t* __restrict__ n_dead_out) {
  __shared__ double lds4[4];
  __shared__ uint32_t ldsu[4];
  double carry = 0.0;
  uint32_t dcarry = 0u;
  for (uint32_t b = 0; b < n_tiles; b += kRelThreads) {
    const uint32_t i = b + threadIdx.x;
    const double v = i < n_tiles ? sums[i] : 0.0;
    const uint32_t d = i < n_tiles ? dead_sums[i] : 0u;
    double tot;
    uint32_t dtot;
    const double incl = wg_inclusive_scan(v, lds4, &tot);
    const uint32_t dincl = wg_inclusive_scan(d, ldsu, &dtot);
    if (i < n_tiles) {   // exclusive
      sums[i] = carry + incl - v;
      dead_sums[i] = dcarry + dincl - d;
    }
    carry += tot;
    dcarry += dtot;
  }
  if (threadIdx.x == 0) {
    state->n_dead = dcarry;
    if (n_dead_out) *n_dead_out = dcarry;
  }
}

// slots[i]: the dead primitives before i, and kDead where i is one.
constexpr uint32_t kDead = 0x80000000u;

__global__ void __launch_bounds__(kRelThreads) reloc_scan_kernel(
    double* __restrict__ w, int64_t n, const double* __restrict__ sums,
    const uint32_t* __restrict__ dead_sums, uint32_t* __restrict__ slots,
    RelocState* __restrict__ state) {
  __shared__ RelTile tile;
  __shared__ double lds4[4];
  __shared__ uint32_t ldsu[4];
  __shared__ uint32_t s_slot[kRelTile + kRelThreads];
  double vals[kRelItems], s, tot;
  uint32_t d, dtot;
  load_tile(tile, w, n, vals, &s, &d);
  double run = sums[blockIdx.x] + wg_inclusive_scan(s, lds4, &tot) - s;
  uint32_t at = dead_sums[blockIdx.x] + wg_inclusive_scan(d, ldsu, &dtot) - d;
  const int64_t base = int64_t(blockIdx.x) * kRelTile;
#pragma unroll
  for (int k = 0; k < kRelItems; ++k) {
    const int e = int(threadIdx.x) * (kRelItems + 1) + k;
    const bool dead = vals[k] < 0.0;
    run += fmax(vals[k], 0.0);
    tile.w[e] = run;
    s_slot[e] = at | (dead ? kDead : 0u);
    at += dead ? 1u : 0u;
    if (base + int64_t(threadIdx.x) * kRelItems + k == n - 1) state->total = run;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kRelItems; ++k) {
    const int e = k * kRelThreads + int(threadIdx.x);
    if (base + e < n) {
      w[base + e] = tile.w[e + e / kRelItems];
      slots[base + e] = s_slot[e + e / kRelItems];
    }
  }
}

// First index j with cdf[j] > x (strict) or >= x, cdf non-decreasing; n if none.
template <bool STRICT>
__device__ __forceinline__ int64_t first_index(const double* __restrict__ cdf, int64_t n, double x) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = lo + ((hi - lo) >> 1);
    const bool past = STRICT ? cdf[mid] > x : cdf[mid] >= x;
    if (past) hi = mid; else lo = mid + 1;
  }
  return lo;
}

// Dead slot k picks the first j with cdf[j] > u_k * total; when the product
// rounds to the total itself (u within an ulp of 1) there is none, and the
// pick is the last live primitive (the first j with cdf[j] >= total).
// Bound by the latency of the probes one after the other: 31 us for 300k slots
// of 1M, and the same with the first ten of a search's twenty in LDS.
__global__ void __launch_bounds__(kRelThreads) reloc_sample_kernel(
    const double* __restrict__ cdf, int64_t n, const RelocState* __restrict__ state,
    const double* __restrict__ uniforms, uint32_t* __restrict__ targets,
    uint32_t* __restrict__ counts, uint32_t* __restrict__ targets_out) {
  const int64_t k = int64_t(blockIdx.x) * kRelThreads + threadIdx.x;
  const double total = state->total;
  if (k >= int64_t(state->n_dead) || !(total > 0.0)) return;
  int64_t j = first_index<true>(cdf, n, uniforms[k] * total);
  if (j >= n) j = first_index<false>(cdf, n, total);
  targets[k] = uint32_t(j);
  if (targets_out) targets_out[k] = uint32_t(j);
  atomicAdd(&counts[j], 1u);
}

constexpr uint32_t kUnchanged = 0xffffffffu;

// The primitive whose rows i takes, and its new opacity: o_keep holds the old
// ones, so no thread reads what another writes.
__global__ void __launch_bounds__(kRelThreads) reloc_plan_kernel(
    float* __restrict__ params, int64_t n, int o_row, const float* __restrict__ o_keep,
    const uint32_t* __restrict__ targets, const uint32_t* __restrict__ counts,
    const RelocState* __restrict__ state, const uint32_t* __restrict__ slots,
    uint32_t* __restrict__ src_of) {
  const int64_t i = int64_t(blockIdx.x) * kRelThreads + threadIdx.x;
  if (i >= n || !(state->total > 0.0)) return;
  const uint32_t slot = slots[i];
  uint32_t src = kUnchanged;
  if (slot & kDead) src = targets[slot & ~kDead];
  else if (counts[i] > 0u) src = uint32_t(i);
  src_of[i] = src;
  if (src != kUnchanged)
    params[int64_t(o_row) * n + i] =
        float(1.0 - pow(1.0 - double(o_keep[src]), 1.0 / (double(counts[src]) + 1.0)));
}

// Row by row.  Workgroup b runs on XCD b % 8, and an XCD takes a contiguous
// eighth of the (row, chunk of primitives) pairs, so that it gathers from one
// row at a time, 4 MB at 1M primitives, mostly out of its own L2.  Bound by the
// two thirds of the time that the partial lines of three arrays take to write
// (whole lines, read first where a primitive keeps its moments, take as long at
// any share from 4 % to 30 % dead) and by the gather, 64 lines an instruction:
// 361 -> 298 us at 36 rows of 1M, 30 % dead, against a thread per (row,
// primitive) pair that read four words to find out what to do.  Picks are
// never dead and their rows but the opacity's stay as they are, so no thread
// reads what another writes.
constexpr int kApplyItems = 4;
constexpr int kApplyChunk = kRelThreads * kApplyItems;
constexpr unsigned kApplyGroups = 2048;   // eight workgroups of four wavefronts per CU

__global__ void __launch_bounds__(kRelThreads) reloc_apply_kernel(
    float* __restrict__ params, float* __restrict__ m, float* __restrict__ v, int64_t n, int F,
    int o_row, const RelocState* __restrict__ state, const uint32_t* __restrict__ src) {
  if (!(state->total > 0.0)) return;
  const uint32_t chunks = uint32_t((n + kApplyChunk - 1) / kApplyChunk);   // at most 2^21
  const uint32_t units = chunks * uint32_t(F);
  const uint32_t xcd = blockIdx.x & 7u, per = gridDim.x >> 3;
  const uint32_t end = uint32_t(uint64_t(units) * (xcd + 1) / 8);
  for (uint32_t u = uint32_t(uint64_t(units) * xcd / 8) + (blockIdx.x >> 3); u < end; u += per) {
    const uint32_t r = u / chunks;
    const int64_t first = int64_t(u - r * chunks) * kApplyChunk + threadIdx.x;
    const int64_t row = int64_t(r) * n;
    uint32_t s[kApplyItems];
    float val[kApplyItems];
#pragma unroll
    for (int k = 0; k < kApplyItems; ++k) {
      const int64_t i = first + k * kRelThreads;
      s[k] = i < n ? src[i] : kUnchanged;
    }
    if (int(r) != o_row) {
#pragma unroll
      for (int k = 0; k < kApplyItems; ++k) {
        const uint32_t i = uint32_t(first + k * kRelThreads);
        if (s[k] != kUnchanged && s[k] != i) val[k] = params[row + s[k]];
      }
#pragma unroll
      for (int k = 0; k < kApplyItems; ++k) {
        const uint32_t i = uint32_t(first + k * kRelThreads);
        if (s[k] != kUnchanged && s[k] != i) params[row + i] = val[k];
      }
    }
#pragma unroll
    for (int k = 0; k < kApplyItems; ++k)
      if (s[k] != kUnchanged) {
        const int64_t i = first + k * kRelThreads;
        m[row + i] = 0.0f;
        v[row + i] = 0.0f;
      }
  }
}

// Device address of `scratch` on the current device, looked up once per
// device (each GPU holds its own copy of the array at its own address).
static ubs_status noalloc_scratch(char** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptr[kMaxDevices] = {};
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return UBS_ERR_HIP;
  if (dev < 0 || dev >= kMaxDevices) return UBS_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return UBS_ERR_HIP;
    ptr[dev] = p;
  }
  *out = static_cast<char*>(ptr[dev]);
  return UBS_OK;
}

static ubs_status relocate_args(int32_t dim, int32_t rot, int64_t n, float o_min) {
  if (dim < 3 || dim > kMaxDim || (rot != UBS_ROT_QUAT && rot != UBS_ROT_SKEW) || n < 0)
    return UBS_ERR_ARG;
  if (!dim_ok(dim)) return UBS_ERR_UNSUPPORTED;
  if (n > (int64_t(1) << 31) - 1) return UBS_ERR_UNSUPPORTED;
  if (!(o_min >= 0.0f)) return UBS_ERR_ARG;
  return UBS_OK;
}

// The relocation's launches over a workspace at `base` laid out by L.
static ubs_status relocate_run(int32_t dim, int32_t rot, int64_t n, float* params, float* m,
                               float* v, const double* uniforms, float o_min, char* base,
                               const RelocLayout& L, uint32_t* targets_out,
                               uint64_t* n_dead_out, void* stream) {
  const ParamRows pr = param_rows(dim - 3, rot);
  hipStream_t st = static_cast<hipStream_t>(stream);
  double* cdf = reinterpret_cast<double*>(base + L.cdf);
  float* o_keep = reinterpret_cast<float*>(base + L.o_keep);
  uint32_t* slots = reinterpret_cast<uint32_t*>(base + L.offs);
  uint32_t* src = reinterpret_cast<uint32_t*>(base + L.src);
  uint32_t* targets = reinterpret_cast<uint32_t*>(base + L.targets);
  uint32_t* counts = reinterpret_cast<uint32_t*>(base + L.counts);
  double* sums = reinterpret_cast<double*>(base + L.sums_f64);
  uint32_t* dead_sums = reinterpret_cast<uint32_t*>(base + L.sums_u32);
  RelocState* state = reinterpret_cast<RelocState*>(base + L.state);
  const unsigned blocks = unsigned((n + kRelThreads - 1) / kRelThreads);
  hipLaunchKernelGGL(reloc_weights_kernel, dim3(blocks), dim3(kRelThreads), 0, st, params, n,
                     pr.F, pr.o, o_min, cdf, o_keep, counts);
  hipLaunchKernelGGL(reloc_tile_sums_kernel, dim3(L.n_tiles), dim3(kRelThreads), 0, st, cdf, n, sums,
                     dead_sums);
  hipLaunchKernelGGL(reloc_sums_kernel, dim3(1), dim3(kRelThreads), 0, st, sums, dead_sums,
                     L.n_tiles, state, n_dead_out);
  hipLaunchKernelGGL(reloc_scan_kernel, dim3(L.n_tiles), dim3(kRelThreads), 0, st, cdf, n, sums,
                     dead_sums, slots, state);
  hipLaunchKernelGGL(reloc_sample_kernel, dim3(blocks), dim3(kRelThreads), 0, st, cdf, n, state,
                     uniforms, targets, counts, targets_out);
  hipLaunchKernelGGL(reloc_plan_kernel, dim3(blocks), dim3(kRelThreads), 0, st, params, n, pr.o,
                     o_keep, targets, counts, state, slots, src);
  hipLaunchKernelGGL(reloc_apply_kernel, dim3(kApplyGroups), dim3(kRelThreads), 0, st, params, m, v,
                     n, pr.F, pr.o, state, src);
  return hipGetLastError() == hipSuccess ? UBS_OK : UBS_ERR_HIP;
}

}  // namespace ubs

using namespace ubs;

extern "C" ubs_status ubs_relocate(int32_t dim, int32_t rot, int64_t n, float* params, float* m,
                                   float* v, const double* uniforms, float o_min, void* ws,
                                   uint64_t ws_bytes, uint64_t* ws_bytes_needed,
                                   uint32_t* targets_out, uint64_t* n_dead_out, void* stream) {
  const ubs_status a = relocate_args(dim, rot, n, o_min);
  if (a != UBS_OK) return a;
  const RelocLayout L = reloc_layout(n);
  if (!ws) {
    if (!ws_bytes_needed) return UBS_ERR_ARG;
    *ws_bytes_needed = L.bytes;
    return UBS_OK;
  }
  if (ws_bytes < L.bytes) return UBS_ERR_CAPACITY;
  if (n == 0) return UBS_OK;
  if (!params || !m || !v || !uniforms) return UBS_ERR_ARG;
  return relocate_run(dim, rot, n, params, m, v, uniforms, o_min, static_cast<char*>(ws), L,
                      targets_out, n_dead_out, stream);
}

extern "C" ubs_status ubs_relocate_noalloc(int32_t dim, int32_t rot, int64_t n, float* params,
                                           float* m, float* v, const double* uniforms,
                                           float o_min, uint32_t* targets_out,
                                           uint64_t* n_dead_out, void* stream) {
  const ubs_status a = relocate_args(dim, rot, n, o_min);
  if (a != UBS_OK) return a;
  if (n > UBS_RELOCATE_NOALLOC_MAX_N) return UBS_ERR_CAPACITY;
  if (n == 0) return UBS_OK;
  if (!params || !m || !v || !uniforms) return UBS_ERR_ARG;
  char* base = nullptr;
  const ubs_status sc = noalloc_scratch(&base);
  if (sc != UBS_OK) return sc;
  return relocate_run(dim, rot, n, params, m, v, uniforms, o_min, base, reloc_layout(n),
                      targets_out, n_dead_out, stream);
}
