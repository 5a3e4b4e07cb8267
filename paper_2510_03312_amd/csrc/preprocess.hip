// Per-primitive kernels: forward preprocess (parameters -> screen-space
// records for every view of the primitive's scene) and its adjoint
// (gradients of the records, summed over views -> gradients of every
// parameter).  One lane per primitive; a lane reads its parameters once
// (component-major rows, so a wavefront's loads of one row are contiguous)
// and loops over the views of its scene.  The forward pass also copies the
// parameter rows of the primitives some view kept to a compacted copy laid
// out like the adjoint's work lists, so that the adjoint reads dense rows
// instead of gathering a fifth of every line of the parameter array.
#include <type_traits>

#include "prim_math.hpp"
#include "prim_math_f32.hpp"

namespace ubs {

constexpr int kCountBins = 64;

// The forward's forms for T: those of prim_math.hpp, or the float32 option's.
template <typename T, int C, int ROT>
struct Forms {
  using G = Geo<T, C, ROT>;
  using S = ViewState<T, C>;
  __device__ __forceinline__ static void geo(const Raw<C, ROT>& r, G& g, uint32_t variant) {
    geo_forward<T, C, ROT>(r, g, variant);
  }
  __device__ __forceinline__ static void view(const Raw<C, ROT>& r, const G& g, const DevView& V, S& s) {
    view_forward<T, C, ROT, false>(r, g, V, s);
  }
};
template <int C, int ROT>
struct Forms<float, C, ROT> {
  using G = f32::Geo<C, ROT>;
  using S = f32::ViewState<C>;
  __device__ __forceinline__ static void geo(const Raw<C, ROT>& r, G& g, uint32_t variant) {
    f32::geo_forward<C, ROT>(r, g, variant);
  }
  __device__ __forceinline__ static void view(const Raw<C, ROT>& r, const G& g, const DevView& V, S& s) {
    f32::view_forward<C, ROT>(r, g, V, s);
  }
};

template <typename T, int C, int ROT>
__global__ void __launch_bounds__(256) preprocess_fwd_kernel(DevScene S,
                                                             const DevView* __restrict__ views,
                                                             float* __restrict__ records,
                                                             LiveOut kept,
                                                             uint32_t* __restrict__ partial,
                                                             uint32_t partial_stride) {
  constexpr int F = param_rows(C, ROT).F;
  // the workgroup's parameters, kept for the copy of its kept primitives
  __shared__ float s_par[F][256];
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const bool active = i < S.n;
  bool finite = true;
  Raw<C, ROT> r;
  using Form = Forms<T, C, ROT>;
  typename Form::G g;
  if (active) {
    load_raw_rows<C, ROT>(
        [&](int k) {
          const float x = __builtin_nontemporal_load(&S.params[int64_t(k) * S.n + i]);
          s_par[k][threadIdx.x] = x;
          return x;
        },
        r);
    finite = r.finite;
    Form::geo(r, g, S.variant);
  }
  uint32_t visible = 0;
  for (int q = 0; q < S.n_views; ++q) {
    const DevView& V = views[views[S.view0 + q].by_scene];
    if (!active) continue;
    typename Form::S s;
    Form::view(r, g, V, s);
    bool live = s.live && finite;
    float4 o0, o1, o2;
    if (live) {
      o0 = make_float4(float(s.mx), float(s.my), float(s.ca), float(s.cb));
      o1 = make_float4(float(s.cc), float(s.rho), float(s.oq), float(s.beta));
      o2 = make_float4(r.rgb[0], r.rgb[1], r.rgb[2], float(s.p[2]));
      if (!isfinite(o0.x) || !isfinite(o0.y) || !isfinite(o0.z) || !isfinite(o0.w) ||
          !isfinite(o1.x) || !isfinite(o1.y) || !isfinite(o1.z) || !isfinite(o1.w) ||
          !(o1.y > 0.0f)) {
        live = false;
      }
    }
    // a culled record is marked only: its fields are not written
    const size_t rec = size_t(V.rec_base) + size_t(i);
    kept.rec_live[rec] = live ? 1u : 0u;
    if (live) {
      ++visible;
      float4* rp = reinterpret_cast<float4*>(records + rec * kRecFloats);
      store_stream(&rp[0], o0);
      store_stream(&rp[1], o1);
      store_stream(&rp[2], o2);
    }
  }
  const bool keep = active && visible > 0;
  if (active) kept.flags[i] = keep ? 1u : 0u;
  // per-workgroup counts (no atomics on a shared word per wavefront: those
  // serialise across the chip); the binning's first kernel adds them into
  // the status block.  The kept primitives go to the adjoint's list: one
  // atomic per workgroup reserves their run, and their parameter rows are
  // copied (from LDS) to the run's columns of the compacted copy.  One view: in
  // ascending order, each wavefront its own.  Several views: by number of live
  // records, in any order among equals; a primitive's gradient does not depend
  // on its entry, so results are the same.
  __shared__ uint32_t s_cnt[2], s_run, s_total;
  __shared__ uint8_t s_src[256];
  __shared__ unsigned long long s_keep[4];
  __shared__ uint32_t s_bin[kCountBins];
  if (threadIdx.x == 0) { s_cnt[0] = 0; s_cnt[1] = 0; }
  if (threadIdx.x < kCountBins) s_bin[threadIdx.x] = 0u;
  __syncthreads();
  const unsigned long long nf = __ballot(active && !finite);
  const unsigned long long km = __ballot(keep);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t vis = visible;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) vis += __shfl_xor(vis, o, 64);
  if (lane == 0) {
    if (nf) atomicAdd(&s_cnt[0], uint32_t(__popcll(nf)));
    if (vis) atomicAdd(&s_cnt[1], vis);
    s_keep[wave] = km;
  }
  __syncthreads();
  const unsigned long long m0 = s_keep[0], m1 = s_keep[1], m2 = s_keep[2], m3 = s_keep[3];
  const uint32_t which = blockIdx.x % kKeptLists;
  if (threadIdx.x == 0) {
    const uint32_t n_keep = uint32_t(__popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3));
    partial[blockIdx.x] = s_cnt[1];
    partial[partial_stride + blockIdx.x] = s_cnt[0];
    s_run = n_keep ? atomicAdd(&kept.count[which], n_keep) : 0u;
    s_total = n_keep;
  }
  __syncthreads();
  // entry q of the run: the kept primitives in thread order, or, where several
  // views see the scene, by their number of live records (kCountBins bins,
  // every second workgroup of a list the other way round, so that the ends of
  // neighbouring runs have about the same; within a bin in the order of the LDS
  // atomics)
  uint32_t q = uint32_t(__popcll(km & ((1ull << lane) - 1ull)));
  if (wave > 0) q += uint32_t(__popcll(m0));
  if (wave > 1) q += uint32_t(__popcll(m1));
  if (wave > 2) q += uint32_t(__popcll(m2));
  if (S.n_views > 1) {
    uint32_t bin = min(visible, uint32_t(kCountBins - 1));
    if ((blockIdx.x / kKeptLists) & 1u) bin = uint32_t(kCountBins - 1) - bin;
    uint32_t rank = 0;
    if (keep) rank = atomicAdd(&s_bin[bin], 1u);
    __syncthreads();
    if (wave == 0) {
      const uint32_t c = s_bin[lane];
      uint32_t incl = c;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
      }
      s_bin[lane] = incl - c;
    }
    __syncthreads();
    q = s_bin[bin] + rank;
  }
  uint32_t src = threadIdx.x;   // the thread whose primitive this one lists
  if (S.n_views > 1) {
    // entries are listed by the threads in their order, so that the copies'
    // stores stay dense (each thread listing its own primitive, sorted: 4
    // scenes in 32 views 1000 us, this way 925; unsorted 915)
    if (keep) {
      kept.pos[i] = s_run + q;
      s_src[q] = uint8_t(threadIdx.x);
    }
    __syncthreads();
    if (threadIdx.x >= s_total) return;
    src = s_src[threadIdx.x];
    q = threadIdx.x;
  } else {
    if (!keep) return;
    kept.pos[i] = s_run + q;
  }
  const uint32_t p = s_run + q;
  kept.list[size_t(which) * kept.cap + p] = blockIdx.x * 256u + src;
  float* par = kept.par + size_t(which) * kept.cap + p;
  const int64_t par_stride = int64_t(kKeptLists) * kept.cap;
#pragma unroll
  for (int k = 0; k < F; ++k) par[k * par_stride] = s_par[k][src];
}

// The backward raster leaves per record the pixel sums of
//   P = sum dx s', Q = sum dy s', U = sum dx^2 s', V = sum dx dy s',
//   E = sum dy^2 s', with s' = sigma (d loss / d alpha) / (1 - r),
//   A_o = sum sigma d loss / d alpha, A_b = sum that times log2(1 - r),
// and the colour sums (dx, dy: pixel centre minus projected mean).  With
// d sigma / d r = -beta sigma / (1 - r), r = a dx^2 + 2 b dx dy + c dy^2,
// d sigma / d o = sigma / o and d sigma / d beta = sigma ln(1 - r), the
// record-field gradients are
//   d/d mx = 2 beta (a P + b Q), d/d my = 2 beta (b P + c Q),
//   d/d a = -beta U, d/d b = -2 beta V, d/d c = -beta E,
//   d/d o = A_o / o, d/d beta = ln 2 A_b
// (in place; rf: fields 2-7 of the record as the raster used it).
__device__ __forceinline__ void record_gradient_from_sums(const float* rf, float* g) {
  const float a = rf[0], b = rf[1], c = rf[2], o = rf[4], beta = rf[5];
  const float P = g[0], Q = g[1], U = g[2], V = g[3], E = g[4];
  g[0] = 2.0f * beta * (a * P + b * Q);
  g[1] = 2.0f * beta * (b * P + c * Q);
  g[2] = -beta * U;
  g[3] = -2.0f * beta * V;
  g[4] = -beta * E;
  g[5] = g[5] / o;
  g[6] = g[6] * 0.69314718f;
}

// What the adjoint reads of a record: its live flag, gradient sums and fields
// 2-7 (every row lies inside the workspace; a culled record's are not used).
struct RecordIn {
  float sums[kGradFloats];
  float fields[6];
  uint32_t live;
};
__device__ __forceinline__ void load_record(const uint8_t* __restrict__ rec_live,
                                            const float* __restrict__ records,
                                            const float* __restrict__ grad2d, size_t rec,
                                            RecordIn& x) {
  x.live = rec_live[rec];
  const float2* gp = reinterpret_cast<const float2*>(grad2d + rec * kGradFloats);
  const float2* rp = reinterpret_cast<const float2*>(records + rec * kRecFloats + 2);
#pragma unroll
  for (int k = 0; k < kGradFloats / 2; ++k) {
    const float2 v = gp[k];
    x.sums[2 * k] = v.x;
    x.sums[2 * k + 1] = v.y;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float2 v = rp[k];
    x.fields[2 * k] = v.x;
    x.fields[2 * k + 1] = v.y;
  }
}

// The adjoint of one record: its share of the primitive's gradients is added to
// the lane's column of the sums.  (Plain adds: every column is one lane's.  LDS
// float atomics took pre_bwd from 82 to 130 us.)
template <typename T, int C, int ROT, typename Sums>
__device__ __forceinline__ void record_adjoint(const Raw<C, ROT>& r, const Geo<T, C, ROT>& g,
                                               const DevView& V, RecordIn& x,
                                               float* __restrict__ grad_row,
                                               Sums& sums, int lane) {
  record_gradient_from_sums(x.fields, x.sums);
  // (rows start 8-byte aligned)
  float2* gp = reinterpret_cast<float2*>(grad_row);
#pragma unroll
  for (int k = 0; k < 3; ++k) gp[k] = make_float2(x.sums[2 * k], x.sums[2 * k + 1]);
  grad_row[6] = x.sums[6];
  ViewState<T, C> s;
  view_forward<T, C, ROT, true>(r, g, V, s);
  view_backward<T, C, ROT>(g, V, s, x.sums, [&](int k, T y) { sums.add(k, y, lane); });
}

// The last step: gradient rows to parameter rows, written to column t of the
// compacted buffer.  AGAIN: the parameters are read once more, and what only
// this step needs of them (s, M, Sigma_xq, H) is formed again; kept over the
// views they would take the registers of the second wavefront per SIMD.
template <typename T, int C, int ROT, bool AGAIN, typename Sums>
__device__ __forceinline__ void write_gradient(const Raw<C, ROT>& r, const float* __restrict__ par,
                                               int64_t stride, uint32_t t, Geo<T, C, ROT>& g,
                                               const Sums& sums, int lane,
                                               float* __restrict__ compact) {
  auto grad = [&](int k) { return sums.get(k, lane); };
  auto out = [&](int k, T x) { compact[int64_t(k) * stride + t] = float(x); };
  if constexpr (AGAIN) {
    uint32_t t2 = t;
    asm volatile("" : "+v"(t2));
    Raw<C, ROT> r2;
    load_raw<C, ROT>(par, stride, t2, r2);
    geo_frame<T, C, ROT>(r2, g);
    if constexpr (C > 0) geo_h<T, C, ROT>(g);
    geo_backward<T, C, ROT>(r2, g, grad, out);
  } else {
    geo_backward<T, C, ROT>(r, g, grad, out);
  }
}

// Adjoint of a scene that one view sees.  One lane per entry of the kept
// lists: the primitive at entry e of list l, its parameters read from column
// t = l cap + e of the compacted copy and its gradient written to column t of
// the compacted [F][kKeptLists cap] buffer (both coalesced);
// scatter_dparams_kernel moves it to the primitive's column.
//
// Bound by latency: the float64 state leaves two wavefronts per SIMD (one
// beyond 7-D), so a workgroup is one wavefront (a SIMD takes the next as soon
// as it is free, not when its workgroup's others are), the parameters, the
// list entry and the list's count are read together, the gradient sums lie in
// LDS and not in registers, and the last step reads the parameters again.
// With the triangular forms of prim_math.hpp: 1M 7-D at 1080p 49 -> 35 us, 1M
// 6-D 55 -> 41, 1M 10-D 223 -> 43 (its state no longer spills).
// The parameters stay in registers where that costs nothing: where a SIMD has
// as many wavefronts with them (3-D, four, and 6-D skew, two: 1M 6-D skew, a
// third kept, 76 -> 72 us with the scatter, all kept 159 -> 150), and in scenes of
// up to kOneRound primitives (7-D and 6-D quaternion, one wavefront a SIMD with
// them: 65,536 kept entries at once, which a fifth or a third of 2^18 primitives
// is about: a fifth of 200,000 7-D kept 30.8 -> 25.5 us, a third of 50,000 6-D
// 20.4 -> 19.5; but 100,000 to 260,000 7-D all kept 5 to 9 % slower, and 400,000,
// a fifth kept, 40.6 -> 42.6).
// 3-D has 14 sums, in registers, and workgroups of 256 (1M, half kept: 35.7 us
// with sums in LDS and the parameters read again, 31.5 so; one wavefront a
// workgroup in two views 74, four 67).
constexpr int64_t kOneRound = 1 << 18;
constexpr int bwd_threads(int C) { return C == 0 ? 256 : 64; }
constexpr bool parameters_fit(int C, int rot) { return C == 0 || (C == 3 && rot == UBS_ROT_SKEW); }

template <typename T, int C, int ROT, bool AGAIN>
__global__ void __launch_bounds__(bwd_threads(C), AGAIN && C <= 4 ? 2 : 1) preprocess_bwd_kernel(
    DevScene S, const DevView* __restrict__ views,
    const float* __restrict__ records, float* __restrict__ grad2d, LiveIn kept,
    float* __restrict__ compact) {
  // workgroup b takes entries N (b / kKeptLists) + [0, N) of kept list
  // b mod kKeptLists (cap is a multiple of N, its threads), so the workgroups
  // holding entries come first in the grid whatever the lists' counts
  constexpr uint32_t N = bwd_threads(C);
  const uint32_t lo = blockIdx.x % kKeptLists;
  const uint32_t pos = (blockIdx.x / kKeptLists) * N + threadIdx.x;
  const uint32_t t = lo * kept.cap + pos;
  const uint32_t n_entries = kept.count[lo];
  if ((blockIdx.x / kKeptLists) * N >= n_entries) return;
  // (a lane past the list's end reads an unused entry of its own list and column)
  const uint32_t i = kept.list[t];
  const int64_t stride = int64_t(kKeptLists) * kept.cap;
  Raw<C, ROT> r;
  load_raw<C, ROT>(kept.par, stride, t, r);
  if (pos >= n_entries) return;
  const DevView& V = views[views[S.view0].by_scene];
  const size_t rec = size_t(V.rec_base) + i;
  RecordIn x;
  // (registers allow the record's read ahead of the geometry here)
  if constexpr (!AGAIN) load_record(kept.rec_live, records, grad2d, rec, x);
  Geo<T, C, ROT> g;
  geo_forward<T, C, ROT>(r, g, S.variant);
  if constexpr (AGAIN) load_record(kept.rec_live, records, grad2d, rec, x);
  auto finish = [&](auto& sums, int column) {
    sums.clear(column);
    if (x.live)
      record_adjoint<T, C, ROT>(r, g, V, x, grad2d + rec * kGradFloats, sums, column);
    write_gradient<T, C, ROT, AGAIN>(r, kept.par, stride, t, g, sums, column, compact);
  };
  if constexpr (C == 0) {
    GradSums<C, 1, true> sums;
    finish(sums, 0);
  } else {
    __shared__ GradSums<C, N, true> s_grad;
    finish(s_grad, threadIdx.x);
  }
}

// Adjoint of a scene that several views see.  A primitive is live in some of
// them only (2.3 of eight on the batched workloads), and a wavefront runs as
// many steps as its busiest lane has live records.  So each lane takes its own
// live views one after the other, and the preprocess lists the kept
// primitives of a workgroup by their number of live records: a wavefront's
// lanes then have about the same.  (The columns stay dense that way: sorting
// the entries afterwards, in groups of 1024, made every wavefront read its
// parameters from all over the group: 640 us where this takes 370.)  2M 7-D in
// 8 views 726 -> 370 us, 4 scenes in 32 views 2.05 -> 1.02 ms, the forms of
// prim_math.hpp included (580 us and 1.45 ms with all lanes in step over the
// scene's views); the preprocess pays 5 us for the sorting of the 8 views.
// Two wavefronts per SIMD to 7-D, at 7-D with 14 registers spilled.
constexpr int kManyViews = 32;   // views of a live mask
constexpr int kViewWords = int(sizeof(DevView) / 4);

template <typename T, int C, int ROT>
__global__ void __launch_bounds__(bwd_threads(C), C <= 4 ? 2 : 1) preprocess_bwd_many_kernel(
    DevScene S, const DevView* __restrict__ views,
    const float* __restrict__ records, float* __restrict__ grad2d, LiveIn kept,
    float* __restrict__ compact) {
  __shared__ uint32_t s_views[kManyViews][kViewWords];
  constexpr uint32_t N = bwd_threads(C);
  const uint32_t lo = blockIdx.x % kKeptLists;
  const uint32_t pos = (blockIdx.x / kKeptLists) * N + threadIdx.x;
  const uint32_t n_entries = kept.count[lo];
  if ((blockIdx.x / kKeptLists) * N >= n_entries) return;
  const bool active = pos < n_entries;
  // (a lane past the list's end reads an unused entry of its own list and column)
  const uint32_t t = lo * kept.cap + pos;
  const uint32_t entry = kept.list[t];
  const uint32_t i = active ? entry : 0u;
  const int64_t stride = int64_t(kKeptLists) * kept.cap;
  Raw<C, ROT> r;
  load_raw<C, ROT>(kept.par, stride, t, r);
  auto view = [&](int q) -> const DevView& { return *reinterpret_cast<const DevView*>(s_views[q]); };
  // the descriptors of views [q0, q0 + nq) of the scene into LDS; the lane's
  // live records among them as a mask
  auto stage_views = [&](int q0, int nq) {
    __syncthreads();
    for (int w = threadIdx.x; w < nq * kViewWords; w += N)
      s_views[w / kViewWords][w % kViewWords] =
          reinterpret_cast<const uint32_t*>(views + views[S.view0 + q0 + w / kViewWords].by_scene)[w % kViewWords];
    __syncthreads();
    uint32_t live = 0u;
#pragma unroll 8
    for (int q = 0; q < nq; ++q)
      live |= (kept.rec_live[size_t(view(q).rec_base) + i] != 0 ? 1u : 0u) << q;
    return active ? live : 0u;
  };
  int nq = min(kManyViews, S.n_views);
  uint32_t live = stage_views(0, nq);
  Geo<T, C, ROT> g;
  geo_forward<T, C, ROT>(r, g, S.variant);
  auto finish = [&](auto& sums, int column) {
    sums.clear(column);
    for (int q0 = 0;;) {
      while (live != 0) {
        const int cur = __ffs(int(live)) - 1;
        live &= live - 1;
        const DevView& V = view(cur);
        const size_t rec = size_t(V.rec_base) + i;
        RecordIn y;
        load_record(kept.rec_live, records, grad2d, rec, y);
        // (not carried from view to view as float64 copies)
#pragma unroll
        for (int k = 0; k < 3; ++k) asm volatile("" : "+v"(r.mu[k]));
#pragma unroll
        for (int k = 0; k < C; ++k) asm volatile("" : "+v"(r.muq[k]));
        asm volatile("" : "+v"(r.o), "+v"(r.bx));
        record_adjoint<T, C, ROT>(r, g, V, y, grad2d + rec * kGradFloats, sums, column);
      }
      q0 += nq;
      if (q0 >= S.n_views) break;
      nq = min(kManyViews, S.n_views - q0);
      live = stage_views(q0, nq);
    }
    if (!active) return;
    write_gradient<T, C, ROT, C != 0>(r, kept.par, stride, t, g, sums, column, compact);
  };
  if constexpr (C == 0) {
    GradSums<C, 1, false> sums;
    finish(sums, 0);
  } else {
    __shared__ GradSums<C, N, false> s_grad;
    finish(s_grad, threadIdx.x);
  }
}

// Adjoint of the float32 option (a lane per list entry, all lanes in step over
// the scene's views).
template <int C, int ROT>
__global__ void __launch_bounds__(256) preprocess_bwd_f32_kernel(DevScene S,
                                                             const DevView* __restrict__ views,
                                                             const float* __restrict__ records,
                                                             float* __restrict__ grad2d,
                                                             LiveIn kept,
                                                             float* __restrict__ compact) {
  // workgroup b takes entries 256 (b / kKeptLists) + [0, 256) of kept list
  // b mod kKeptLists (cap is a multiple of 256), so the workgroups holding
  // entries come first in the grid whatever the lists' counts; thread t =
  // list cap + entry writes compacted column t
  const uint32_t lo = blockIdx.x % kKeptLists;
  const uint32_t pos = (blockIdx.x / kKeptLists) * 256u + threadIdx.x;
  const uint32_t t = lo * kept.cap + pos;
  if (pos >= kept.count[lo]) return;
  const int64_t i = kept.list[t];
  const int64_t stride = int64_t(kKeptLists) * kept.cap;
  Raw<C, ROT> r;
  // (dense rows of the compacted copy the preprocess wrote)
  load_raw<C, ROT>(kept.par, stride, t, r);
  f32::Geo<C, ROT> g;
  f32::geo_forward<C, ROT>(r, g, S.variant);
  f32::GeoGrad<C> G;
  f32::geograd_zero<C>(G);
  for (int q = 0; q < S.n_views; ++q) {
    const DevView& V = views[views[S.view0 + q].by_scene];
    const size_t rec = size_t(V.rec_base) + size_t(i);
    // the record's sums and fields are read together with its live flag
    // (every row lies inside the workspace; a culled record's are unused)
    const bool live = kept.rec_live[rec] != 0;
    const float* rp = records + rec * kRecFloats;
    float gr[kGradFloats], rf[6];
    float* gp = grad2d + rec * kGradFloats;
#pragma unroll
    for (int k = 0; k < kGradFloats; ++k) gr[k] = gp[k];
#pragma unroll
    for (int k = 0; k < 6; ++k) rf[k] = rp[2 + k];
    // (the loads stay ahead of the branch: one wait for all three)
#pragma unroll
    for (int k = 0; k < kGradFloats; ++k) asm volatile("" : "+v"(gr[k]));
#pragma unroll
    for (int k = 0; k < 6; ++k) asm volatile("" : "+v"(rf[k]));
    if (!live) continue;
    record_gradient_from_sums(rf, gr);
#pragma unroll
    for (int k = 0; k < 7; ++k) gp[k] = gr[k];
    f32::ViewState<C> s;
    f32::view_forward<C, ROT>(r, g, V, s);
    f32::view_backward<C, ROT>(r, g, V, s, gr, G);
  }
  constexpr int F = param_rows(C, ROT).F;
  float out[F];
  f32::geo_backward<C, ROT>(r, g, G, out);
#pragma unroll
  for (int k = 0; k < F; ++k) compact[int64_t(k) * stride + t] = out[k];
}

// dparams[k, i] = compact[k, j(i)] for kept primitives (j: the column of
// their kept-list entry), 0 otherwise.  VEC primitives per thread (4: one
// 16-byte store per row, for rows that start 16-byte aligned); the rows go
// in chunks whose loads are all issued before their stores, so a wavefront
// waits for memory once per chunk rather than once per row.
constexpr int kScatterChunk = 9;

template <int VEC>
__global__ void __launch_bounds__(256) scatter_dparams_kernel(DevScene S, LiveIn kept,
                                                              const float* __restrict__ compact) {
  const int64_t i0 = (int64_t(blockIdx.x) * 256 + threadIdx.x) * VEC;
  if (i0 >= S.n) return;
  const int64_t stride = int64_t(kKeptLists) * kept.cap;
  // (a primitive's list: that of its preprocess workgroup of 256; the VEC
  // primitives of a thread share it)
  const int64_t list_base = int64_t((i0 / 256) % kKeptLists) * kept.cap;
  bool live[VEC];
  int64_t j[VEC];
#pragma unroll
  for (int q = 0; q < VEC; ++q) {
    live[q] = i0 + q < S.n && kept.flags[i0 + q] != 0;
    j[q] = live[q] ? list_base + int64_t(kept.pos[i0 + q]) : 0;
  }
  for (int k0 = 0; k0 < S.F; k0 += kScatterChunk) {
    float v[kScatterChunk][VEC];
#pragma unroll
    for (int c = 0; c < kScatterChunk; ++c)
#pragma unroll
      for (int q = 0; q < VEC; ++q)
        v[c][q] = (live[q] && k0 + c < S.F) ? compact[int64_t(k0 + c) * stride + j[q]] : 0.0f;
#pragma unroll
    for (int c = 0; c < kScatterChunk; ++c) {
      if (k0 + c >= S.F) break;
      float* row = S.dparams + int64_t(k0 + c) * S.n;
      if constexpr (VEC == 4)
        store_stream(reinterpret_cast<float4*>(row + i0), make_float4(v[c][0], v[c][1], v[c][2], v[c][3]));
      else
        store_stream(row + i0, v[c][0]);
    }
  }
}

template <typename T, int C, int ROT>
static hipError_t pre_fwd_t(const DevScene& S, const DevView* views,
                            float* records, LiveOut live, uint32_t* partial, uint32_t stride,
                            hipStream_t st) {
  const unsigned blocks = unsigned((S.n + 255) / 256);
  hipLaunchKernelGGL((preprocess_fwd_kernel<T, C, ROT>), dim3(blocks), dim3(256), 0, st, S,
                     views, records, live, partial, stride);
  return hipGetLastError();
}

template <typename T, int C, int ROT>
static hipError_t pre_bwd_t(const DevScene& S, const DevView* views,
                            const float* records, float* grad2d, LiveIn kept, float* compact,
                            hipStream_t st) {
  // one lane per entry of the kKeptLists lists of cap entries
  const uint64_t entries = uint64_t(kKeptLists) * kept.cap;
  constexpr unsigned N = bwd_threads(C);
  if constexpr (std::is_same<T, float>::value) {
    hipLaunchKernelGGL((preprocess_bwd_f32_kernel<C, ROT>), dim3(unsigned(entries / 256)),
                       dim3(256), 0, st, S, views, records, grad2d, kept, compact);
  } else if (S.n_views == 1) {
    // (beyond 7-D the state spills with the parameters in it)
    constexpr bool kMayKeep = C <= 4, kKeep = parameters_fit(C, ROT);
    if (kKeep || (kMayKeep && S.n <= kOneRound))
      hipLaunchKernelGGL((preprocess_bwd_kernel<T, C, ROT, !kMayKeep>), dim3(unsigned(entries / N)),
                         dim3(N), 0, st, S, views, records, grad2d, kept, compact);
    else
      hipLaunchKernelGGL((preprocess_bwd_kernel<T, C, ROT, !kKeep>), dim3(unsigned(entries / N)),
                         dim3(N), 0, st, S, views, records, grad2d, kept, compact);
  } else {
    hipLaunchKernelGGL((preprocess_bwd_many_kernel<T, C, ROT>), dim3(unsigned(entries / N)),
                       dim3(N), 0, st, S, views, records, grad2d, kept, compact);
  }
  // 16-byte stores when every row of dparams starts 16-byte aligned
  if (S.n % 4 == 0 && reinterpret_cast<uintptr_t>(S.dparams) % 16 == 0)
    hipLaunchKernelGGL(scatter_dparams_kernel<4>, dim3(unsigned((S.n / 4 + 255) / 256)), dim3(256),
                       0, st, S, kept, compact);
  else
    hipLaunchKernelGGL(scatter_dparams_kernel<1>, dim3(unsigned((S.n + 255) / 256)), dim3(256), 0,
                       st, S, kept, compact);
  return hipGetLastError();
}

template <typename T>
static hipError_t pre_fwd_dispatch(const DevScene& S, const DevView* views,
                                   float* records, LiveOut live, uint32_t* partial,
                                   uint32_t stride, hipStream_t st) {
  const int C = S.dim - 3;
  if (S.rot == UBS_ROT_QUAT) {
    if (C == 0) return pre_fwd_t<T, 0, 0>(S, views, records, live, partial, stride, st);
    if (C == 3) return pre_fwd_t<T, 3, 0>(S, views, records, live, partial, stride, st);
    if (C == 4) return pre_fwd_t<T, 4, 0>(S, views, records, live, partial, stride, st);
    if (C == 5) return pre_fwd_t<T, 5, 0>(S, views, records, live, partial, stride, st);
    if (C == 6) return pre_fwd_t<T, 6, 0>(S, views, records, live, partial, stride, st);
    if (C == 7) return pre_fwd_t<T, 7, 0>(S, views, records, live, partial, stride, st);
  } else {
    if (C == 0) return pre_fwd_t<T, 0, 1>(S, views, records, live, partial, stride, st);
    if (C == 3) return pre_fwd_t<T, 3, 1>(S, views, records, live, partial, stride, st);
    if (C == 4) return pre_fwd_t<T, 4, 1>(S, views, records, live, partial, stride, st);
    if (C == 5) return pre_fwd_t<T, 5, 1>(S, views, records, live, partial, stride, st);
    if (C == 6) return pre_fwd_t<T, 6, 1>(S, views, records, live, partial, stride, st);
    if (C == 7) return pre_fwd_t<T, 7, 1>(S, views, records, live, partial, stride, st);
  }
  return hipErrorInvalidValue;
}

template <typename T>
static hipError_t pre_bwd_dispatch(const DevScene& S, const DevView* views,
                                   const float* records, float* grad2d, LiveIn kept,
                                   float* compact, hipStream_t st) {
  const int C = S.dim - 3;
  if (S.rot == UBS_ROT_QUAT) {
    if (C == 0) return pre_bwd_t<T, 0, 0>(S, views, records, grad2d, kept, compact, st);
    if (C == 3) return pre_bwd_t<T, 3, 0>(S, views, records, grad2d, kept, compact, st);
    if (C == 4) return pre_bwd_t<T, 4, 0>(S, views, records, grad2d, kept, compact, st);
    if (C == 5) return pre_bwd_t<T, 5, 0>(S, views, records, grad2d, kept, compact, st);
    if (C == 6) return pre_bwd_t<T, 6, 0>(S, views, records, grad2d, kept, compact, st);
    if (C == 7) return pre_bwd_t<T, 7, 0>(S, views, records, grad2d, kept, compact, st);
  } else {
    if (C == 0) return pre_bwd_t<T, 0, 1>(S, views, records, grad2d, kept, compact, st);
    if (C == 3) return pre_bwd_t<T, 3, 1>(S, views, records, grad2d, kept, compact, st);
    if (C == 4) return pre_bwd_t<T, 4, 1>(S, views, records, grad2d, kept, compact, st);
    if (C == 5) return pre_bwd_t<T, 5, 1>(S, views, records, grad2d, kept, compact, st);
    if (C == 6) return pre_bwd_t<T, 6, 1>(S, views, records, grad2d, kept, compact, st);
    if (C == 7) return pre_bwd_t<T, 7, 1>(S, views, records, grad2d, kept, compact, st);
  }
  return hipErrorInvalidValue;
}

// partial: this launch's slice of the per-workgroup counts (visible records
// at partial[b], non-finite primitives at partial[stride + b]).
hipError_t launch_preprocess_fwd(bool fp64, const DevScene& S, const DevView* views,
                                 float* records, LiveOut live, uint32_t* partial,
                                 uint32_t stride, hipStream_t st) {
  if (S.n == 0) return hipSuccess;
  return fp64 ? pre_fwd_dispatch<double>(S, views, records, live, partial, stride, st)
              : pre_fwd_dispatch<float>(S, views, records, live, partial, stride, st);
}

hipError_t launch_preprocess_bwd(bool fp64, const DevScene& S, const DevView* views,
                                 const float* records, float* grad2d, LiveIn kept,
                                 float* compact, hipStream_t st) {
  if (S.n == 0) return hipSuccess;
  return fp64 ? pre_bwd_dispatch<double>(S, views, records, grad2d, kept, compact, st)
              : pre_bwd_dispatch<float>(S, views, records, grad2d, kept, compact, st);
}

}  // namespace ubs
