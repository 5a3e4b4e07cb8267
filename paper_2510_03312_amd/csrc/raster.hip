// Per-tile rasterisation: front-to-back compositing and its adjoint.
//
// One wavefront (64 lanes) per tile, or per band of TH / SPLIT rows of it in
// frames of few tiles and for wide tiles.  Lane l owns the pixels of column
// l % TW in rows l / TW + k * (64 / TW) of its band (a whole 16x16 tile gives
// each lane a strip of 4 pixels).  The tile's sorted records are staged through
// LDS 64 at a time (one per lane); every lane then walks the batch.  Because a lane's
// pixels share one column, dx = px - mx is shared and the quadratic form
// costs r = A + dy (B + c dy) per pixel with A, B per record.
//
// Forward: a pixel stops before the first record that would take its
// transmittance below 1e-4; the wavefront stops when all its pixels have.
// Backward: each tile is walked back to front from the last contributor;
// the transmittance in front of a record is recovered by division.  A lane
// first sums the gradient terms of its own pixels; the wavefront then folds
// the ten per-record sums of two records onto fewer lanes with lane swaps,
// finishes them with DPP sums within 16-lane rows and banks, and twenty lanes
// add the totals to the records' accumulators in one atomic instruction (four
// bands of a tile add theirs in LDS first).
//
// Both passes are bound by vector instruction issue (the per-pixel code runs
// for the 2.6 of a tile's four 64-pixel strips that a record's ellipse
// reaches, with half the lanes inside it), so they are counted in
// instructions: a strip costs the forward 4 for the support test and 13 plus
// two transcendentals inside it, the backward 4 and 25 plus four, and a
// record 22 more in the backward for its wavefront sums.  1M 7-D primitives
// at 1080p, former and present forms in turn on one device, by HIP events:
// forward 62.7 -> 58.7 us, backward 133 -> 123 us; 1M 6-D 116 -> 106 and 246 ->
// 229 us.
//
// The order of the backward's float32 operations is kept with care.  A record
// whose 2-D covariance is nearly singular (the symmetrised conditional
// covariance need not be definite) has moment sums that cancel by factors of
// 1e5 and more in the chain to the covariance, so a sum rounded differently
// changes such a gradient in its second digit; w (g . (c - S)) in place of
// sigma (T (g . (c - S))), two instructions a strip fewer (121 us), did.
//
// Both passes take every per-pixel decision (support test, skip, stop)
// through the same inline functions, so the backward pass visits exactly
// the contributors the forward pass used.
#include <type_traits>

#include "ubs_internal.hpp"

namespace ubs {

// Hardware base-2 exponential and logarithm (v_exp_f32 / v_log_f32).
__device__ __forceinline__ float hw_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float hw_log2(float x) { return __builtin_amdgcn_logf(x); }

// Record fields as staged in LDS.
struct Staged {
  float4 g0;  // mx, my, a, 2b
  float4 g1;  // c, rho, log2(o), beta
  float4 g2;  // r, g, b, (record index as bits)
};

__device__ __forceinline__ Staged stage_record(const float* __restrict__ records, uint32_t rec) {
  const float4* rp = reinterpret_cast<const float4*>(records + size_t(rec) * kRecFloats);
  const float4 a = rp[0], b = rp[1], c = rp[2];
  Staged s;
  s.g0 = make_float4(a.x, a.y, a.z, 2.0f * a.w);
  s.g1 = make_float4(b.x, b.y, hw_log2(b.z), b.w);
  s.g2 = make_float4(c.x, c.y, c.z, __uint_as_float(rec));
  return s;
}

// Whether a record may reach the pixel centres with rows in [y0, y1]: the
// half-height sqrt(rho a / det) of {r <= rho}, widened by 1 % and a pixel (a
// determinant that cancels in float32, or is no number, keeps the record).
__device__ __forceinline__ bool may_reach_rows(const Staged& s, float y0, float y1) {
  const float a = s.g0.z, b = 0.5f * s.g0.w, c = s.g1.x, rho = s.g1.y;
  const float det = a * c - b * b;
  if (!(det > 1e-3f * (a * c))) return true;
  const float h = 1.01f * sqrtf(rho * a / det) + 1.0f;
  return !(s.g0.y + h < y0) && !(s.g0.y - h > y1);
}

// Column terms of the quadratic form for one record and one lane:
// r = a dx^2 + 2 b dx dy + c dy^2 = A + dy (B + c dy), A = dx (a dx), B = 2b dx.
struct ColTerms {
  float A, B;
};
__device__ __forceinline__ ColTerms col_terms(const float4 g0, float dx) {
  return ColTerms{dx * (g0.z * dx), g0.w * dx};
}
__device__ __forceinline__ float eval_r(const ColTerms t, float c, float dy) {
  return t.A + dy * (t.B + c * dy);
}

// sigma = o (1 - r)^beta = exp2(log2 o + beta log2(1 - r)); alpha = min(0.99, sigma).
__device__ __forceinline__ float eval_sigma(float r, float lo, float beta, float* l2) {
  const float l = hw_log2(1.0f - r);
  *l2 = l;
  return hw_exp2(lo + beta * l);
}

__device__ __forceinline__ int view_of_tile(const DevView* __restrict__ views, int n_views,
                                            uint32_t tile) {
  int lo = 0, hi = n_views - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (views[mid].tile_base <= tile) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// SPLIT wavefronts share a tile, each one a band of TH / SPLIT rows.
template <int TW, int TH, int SPLIT>
struct TileGeom {
  static constexpr int ROWS = TH / SPLIT;    // rows of a wavefront's band
  static constexpr int PPL = TW * ROWS / 64; // pixels per lane
  static constexpr int RSTEP = 64 / TW;      // rows between a lane's pixels
  static_assert(TH % SPLIT == 0 && TW * ROWS % 64 == 0 && 64 % TW == 0, "tile shape");
};

// Two forms of the update.  NAN_ROWS: a stopped pixel (or one outside the
// image) gets a NaN row coordinate, its r is NaN, and the support test fails
// for every later record without a test of its own; a record is skipped whole
// where its only pixels have stopped, and the update runs under lane masks,
// without selects.  Otherwise a stopped pixel's transmittance is kept negated,
// so that every later record fails its T (1 - alpha) >= 1e-4 test, and skipping
// and stopping are taken by selects.  The first has fewer instructions where
// the SIMDs are full, the second fewer branches in a row where they are not:
// 16x16 tiles with 64 records a batch 63.0 / 58.7 us (1080p, selects / NaN
// rows), with 128 37 / 42 (1280x720) and 64.6 / 64.6 (1080p), with 256 80 / 88,
// 32x16 tiles 75 / 89 and 102 / 123, 16x8 24.5 / 25.9 and 58 / 61, 8x8 23.4 /
// 24.4, the persistent grid 175 / 182.
template <int TW, int TH, int BATCH, int SPLIT, bool NAN_ROWS>
__device__ __forceinline__ void raster_fwd_tile(
    uint32_t tile, int band, float4* s0, float4* s1, float4* s2, const float* __restrict__ records,
    const uint32_t* __restrict__ values, const uint32_t* __restrict__ ranges,
    const DevView* __restrict__ views, int n_views, float* __restrict__ image,
    float* __restrict__ t_ws, float* __restrict__ t_user, uint32_t* __restrict__ ncontrib) {
  constexpr int PPL = TileGeom<TW, TH, SPLIT>::PPL;
  constexpr int RSTEP = TileGeom<TW, TH, SPLIT>::RSTEP;
  constexpr int PER_LANE = BATCH / 64;
  const int lane = threadIdx.x;
  const DevView& V = views[view_of_tile(views, n_views, tile)];
  const uint32_t lt = tile - V.tile_base;
  const int ty = int(lt) / V.tiles_x, tx = int(lt) - ty * V.tiles_x;
  const int px = tx * TW + lane % TW;
  const int py0 = ty * TH + band * TileGeom<TW, TH, SPLIT>::ROWS + lane / TW;
  const float fx = float(px) + 0.5f;
  float T[PPL], fy[PPL], cr[PPL], cg[PPL], cb[PPL];
  uint32_t last[PPL];
#pragma unroll
  for (int k = 0; k < PPL; ++k) {
    const bool outside = px >= V.W || py0 + k * RSTEP >= V.H;
    T[k] = !NAN_ROWS && outside ? -1.0f : 1.0f;
    fy[k] = NAN_ROWS && outside ? __builtin_nanf("") : float(py0 + k * RSTEP) + 0.5f;
    cr[k] = cg[k] = cb[k] = 0.0f; last[k] = 0;
  }
  const float band_y0 = float(ty * TH + band * TileGeom<TW, TH, SPLIT>::ROWS) + 0.5f;
  const float band_y1 = band_y0 + float(TileGeom<TW, TH, SPLIT>::ROWS - 1);
  const uint32_t start = ranges[2 * size_t(tile)], end = ranges[2 * size_t(tile) + 1];
  for (uint32_t b0 = start; b0 < end; b0 += BATCH) {
    // the tile is finished once every pixel has stopped (checked per batch)
    bool running = false;
#pragma unroll
    for (int k = 0; k < PPL; ++k) running = running || (NAN_ROWS ? fy[k] == fy[k] : T[k] >= 0.0f);
    if (__ballot(running) == 0ull) break;
    __syncthreads();
    // (wavefront-uniform: the record loop runs on scalar counters)
    int nb = __builtin_amdgcn_readfirstlane(int(min(uint32_t(BATCH), end - b0)));
    if constexpr (SPLIT == 1) {
#pragma unroll
      for (int m = 0; m < PER_LANE; ++m) {
        const uint32_t idx = b0 + uint32_t(m * 64 + lane);
        if (idx < end) {
          const Staged st = stage_record(records, values[idx]);
          s0[m * 64 + lane] = st.g0;
          s1[m * 64 + lane] = st.g1;
          s2[m * 64 + lane] = st.g2;
        }
      }
    } else {
      // only the records that may reach the band, their positions with them
      int n_kept = 0;
#pragma unroll
      for (int m = 0; m < PER_LANE; ++m) {
        const int q = m * 64 + lane;
        bool keep = q < nb;
        Staged st;
        if (keep) {
          st = stage_record(records, values[b0 + uint32_t(q)]);
          keep = may_reach_rows(st, band_y0, band_y1);
        }
        const uint64_t kept = __ballot(keep);
        if (keep) {
          const int at = n_kept + __popcll(kept & ((1ull << lane) - 1ull));
          st.g2.w = __uint_as_float(b0 - start + uint32_t(q) + 1u);
          s0[at] = st.g0;
          s1[at] = st.g1;
          s2[at] = st.g2;
        }
        n_kept += __popcll(kept);
      }
      nb = n_kept;
    }
    __syncthreads();
    const uint32_t pos1 = __builtin_amdgcn_readfirstlane(b0 - start + 1u);
    for (int j = 0; j < nb; ++j) {
      const float4 g0 = s0[j], g1 = s1[j], g2 = s2[j];
      const ColTerms ct = col_terms(g0, fx - g0.x);
#pragma unroll
      for (int k = 0; k < PPL; ++k) {
        const float dy = fy[k] - g0.y;
        const float r = eval_r(ct, g1.x, dy);
        if (!(r <= g1.y)) continue;
        float l2;
        const float sigma = eval_sigma(r, g1.z, g1.w, &l2);
        const float alpha = fminf(kAlphaMax, sigma);
        const float test = T[k] * (1.0f - alpha);
        if constexpr (NAN_ROWS) {
          const uint64_t hit = __builtin_amdgcn_ballot_w64(alpha >= kAlphaMin);
          const uint64_t pass = __builtin_amdgcn_ballot_w64(test >= kTStop);
          // a hit that fails the stop test stops the pixel (rare)
          if ((hit & ~pass) != 0ull) {
            if (__builtin_amdgcn_inverse_ballot_w64(hit & ~pass)) fy[k] = __builtin_nanf("");
          }
          if (__builtin_amdgcn_inverse_ballot_w64(hit & pass)) {
            const float w = alpha * T[k];
            cr[k] += g2.x * w;
            cg[k] += g2.y * w;
            cb[k] += g2.z * w;
            T[k] = test;
            last[k] = SPLIT == 1 ? pos1 + uint32_t(j) : __float_as_uint(g2.w);
          }
        } else {
          const bool hit = alpha >= kAlphaMin;
          const bool pass = test >= kTStop;
          const bool con = hit && pass;
          const float w = con ? alpha * T[k] : 0.0f;
          cr[k] += g2.x * w;
          cg[k] += g2.y * w;
          cb[k] += g2.z * w;
          const float tn = pass ? test : -fabsf(T[k]);
          T[k] = hit ? tn : T[k];
          last[k] = con ? b0 - start + uint32_t(j) + 1u : last[k];
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < PPL; ++k) {
    const int py = py0 + k * RSTEP;
    if (px < V.W && py < V.H) {
      const size_t pix = size_t(V.pix_base) + size_t(py) * V.W + px;
      image[3 * pix] = cr[k];
      image[3 * pix + 1] = cg[k];
      image[3 * pix + 2] = cb[k];
      // (the internal copy is negated for a pixel that stopped)
      t_ws[pix] = !NAN_ROWS || fy[k] == fy[k] ? T[k] : -T[k];
      if (t_user) t_user[pix] = fabsf(T[k]);
      ncontrib[pix] = last[k];
    }
  }
}

// Next tile for this workgroup: blockIdx.x on the first visit without a work
// queue, else the next index of the queue counter (lane 0 takes it, the
// wavefront shares it).
__device__ __forceinline__ uint32_t next_tile(uint32_t* work, bool first) {
  if (!work) return first ? blockIdx.x : 0xffffffffu;
  uint32_t t = 0;
  if (threadIdx.x == 0) t = atomicAdd(work, 1u);
  return uint32_t(__shfl(int(t), 0, 64));
}

template <int TW, int TH, int BATCH, int SPLIT, bool NAN_ROWS>
__global__ void __launch_bounds__(64) raster_fwd_kernel(
    const float* __restrict__ records, const uint32_t* __restrict__ values,
    const uint32_t* __restrict__ ranges, const DevView* __restrict__ views, int n_views,
    uint32_t n_tiles, const uint32_t* __restrict__ order, uint32_t* __restrict__ work,
    float* __restrict__ image, float* __restrict__ t_ws, float* __restrict__ t_user,
    uint32_t* __restrict__ ncontrib) {
  __shared__ float4 s0[BATCH], s1[BATCH], s2[BATCH];
  for (uint32_t q = next_tile(work, true); q / SPLIT < n_tiles; q = next_tile(work, false))
    raster_fwd_tile<TW, TH, BATCH, SPLIT, NAN_ROWS>(order[q / SPLIT], int(q % SPLIT), s0, s1, s2,
                                                    records, values, ranges, views, n_views, image,
                                                    t_ws, t_user, ncontrib);
}

// Lane exchanges of gfx950: swap_halves(a, b) returns (a with its upper 32
// lanes replaced by b's lower 32, b with its lower 32 replaced by a's upper
// 32); swap_rows(a, b) does the same between a's odd rows and b's even rows
// (rows of 16 lanes).
struct FPair {
  float a, b;
};
__device__ __forceinline__ FPair swap_halves(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return FPair{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ FPair swap_rows(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return FPair{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
// Two zeros from one 64-bit move, which the compiler cannot rematerialise.
__device__ __forceinline__ void opaque_zero2(float& a, float& b) {
  uint64_t z;
  asm volatile("v_mov_b64 %0, 0" : "=v"(z));
  a = __uint_as_float(uint32_t(z));
  b = __uint_as_float(uint32_t(z >> 32));
}
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = min(x, uint32_t(__shfl_xor(int(x), o, 64)));
  return x;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = max(x, uint32_t(__shfl_xor(int(x), o, 64)));
  return x;
}

// What a lane keeps of its pixels in the backward walk: the transmittance in
// front of the current record; D, the pixel's colour gradient dotted with the
// colour composited behind it; the colour gradient; gTf = d loss / d T_final
// times T_final (HAS_DT: a gradient of the final transmittance is given; it
// enters every record's d alpha as - gTf / (1 - alpha)); the last contributor.
template <int PPL>
struct BwdPixels {
  float T[PPL], D[PPL], gR[PPL], gG[PPL], gB[PPL], gTf[PPL];
  uint32_t last[PPL];
};
// Where a wavefront's walk starts: records before `span` may contribute.
// Records at or beyond a pixel's last contributor contribute nothing to it
// unless the pixel stopped (its own alpha test fails there otherwise), so only
// records at or beyond `stop_min`, the smallest last contributor of a stopped
// pixel, need the position test.  (Both wavefront-uniform: the batch loop runs
// on scalar counters.)
struct BwdSpan {
  uint32_t span, stop_min;
};
struct BwdGradients {
  const float *d_image, *d_tfinal, *l1_image, *l1_target;
  float l1_scale;
};

template <int PPL, int RSTEP, bool HAS_DT>
__device__ __forceinline__ BwdSpan load_pixels(BwdPixels<PPL>& P, const DevView& V, int px, int py0,
                                               const float* __restrict__ t_ws,
                                               const uint32_t* __restrict__ ncontrib,
                                               const BwdGradients& G) {
  uint32_t lane_max = 0, lane_stop = 0xffffffffu;
#pragma unroll
  for (int k = 0; k < PPL; ++k) {
    const int py = py0 + k * RSTEP;
    // (a pixel outside the image keeps T = 0: the walk takes it along where no
    // position is tested, and with T = 0 its every term is 0, where T = 1 would
    // grow by 1 / (1 - alpha) a record to infinity and leave a NaN in the sums)
    float Tf = 0.0f;
    P.gR[k] = P.gG[k] = P.gB[k] = P.gTf[k] = 0.0f; P.last[k] = 0;
    if (px < V.W && py < V.H) {
      const size_t pix = size_t(V.pix_base) + size_t(py) * V.W + px;
      Tf = t_ws[pix];
      P.last[k] = ncontrib[pix];
      if (Tf < 0.0f) {   // the pixel stopped
        Tf = -Tf;
        lane_stop = min(lane_stop, P.last[k]);
      }
      if (G.d_image) {
        P.gR[k] = G.d_image[3 * pix];
        P.gG[k] = G.d_image[3 * pix + 1];
        P.gB[k] = G.d_image[3 * pix + 2];
        if (HAS_DT) P.gTf[k] = G.d_tfinal[pix] * Tf;
      } else {
        const float e0 = G.l1_image[3 * pix] - G.l1_target[3 * pix];
        const float e1 = G.l1_image[3 * pix + 1] - G.l1_target[3 * pix + 1];
        const float e2 = G.l1_image[3 * pix + 2] - G.l1_target[3 * pix + 2];
        P.gR[k] = e0 > 0.0f ? G.l1_scale : (e0 < 0.0f ? -G.l1_scale : 0.0f);
        P.gG[k] = e1 > 0.0f ? G.l1_scale : (e1 < 0.0f ? -G.l1_scale : 0.0f);
        P.gB[k] = e2 > 0.0f ? G.l1_scale : (e2 < 0.0f ? -G.l1_scale : 0.0f);
      }
    }
    P.T[k] = Tf;
    P.D[k] = 0.0f;
    lane_max = max(lane_max, P.last[k]);
  }
  return BwdSpan{uint32_t(__builtin_amdgcn_readfirstlane(wave_max_u32(lane_max))),
                 uint32_t(__builtin_amdgcn_readfirstlane(wave_min_u32(lane_stop)))};
}

// One record: the lane's pixel sums, folded (CHECK: test each pixel's last
// contributor against the record's position).
template <bool CHECK, int PPL, int RSTEP, bool HAS_DT>
__device__ __forceinline__ void bwd_record(BwdPixels<PPL>& P, const float4 g0, const float4 g1,
                                           const float4 g2, float fx, int py0, uint32_t pos,
                                           float* h) {
  const float dx = fx - g0.x;
  const ColTerms ct = col_terms(g0, dx);
  // sums over the lane's pixels (its column): q = sigma dalpha / (1 - r),
  // dx-weighted moments come from the shared dx
  // (zeroed through an opaque value: a plain zero would be rematerialised
  // on every accumulating iteration)
  float a_o, a_be, a_r, a_g, a_b, a_dr, a_dry, a_dryy;
  opaque_zero2(a_o, a_be);
  opaque_zero2(a_r, a_g);
  opaque_zero2(a_b, a_dr);
  opaque_zero2(a_dry, a_dryy);
  // (full unroll: each pixel's state is then a fixed register; a loop
  // iterated dynamically moves it in and out of a common window)
#pragma unroll
  for (int k = 0; k < PPL; ++k) {
    const float dy = float(py0 + k * RSTEP) + 0.5f - g0.y;
    const float r = eval_r(ct, g1.x, dy);
    if (!((!CHECK || pos < P.last[k]) && r <= g1.y)) continue;
    float l2;
    const float sigma = eval_sigma(r, g1.z, g1.w, &l2);
    const float alpha = fminf(kAlphaMax, sigma);
    if (!(alpha >= kAlphaMin)) continue;   // (the support's rim)
    const float ioma = fast_rcp(1.0f - alpha);
    const float Ti = P.T[k] * ioma;
    const float w = alpha * Ti;
    a_r += P.gR[k] * w;
    a_g += P.gG[k] * w;
    a_b += P.gB[k] * w;
    // d loss / d alpha = T_k g . (c_k - S_k) (- gTf / (1 - alpha)),
    // S_k the normalised colour composited behind record k; S updates as
    // S += alpha (c - S), so D = g . S as D += alpha dot
    const float dot = (P.gR[k] * g2.x + P.gG[k] * g2.y + P.gB[k] * g2.z) - P.D[k];
    const float dalpha = HAS_DT ? Ti * dot - P.gTf[k] * ioma : Ti * dot;
    P.D[k] += alpha * dot;
    P.T[k] = Ti;
    if (!(alpha < kAlphaMax)) continue;   // (sigma follows alpha below the clamp only)
    const float sd = alpha * dalpha;
    a_o += sd;
    a_be += sd * l2;
    const float q = sd * fast_rcp(1.0f - r);
    a_dr += q;
    const float qy = q * dy;
    a_dry += qy;
    a_dryy += qy * dy;
  }
  // the record's pixel sums P, Q, U, V, E, A_o, A_b and colour (zeros for
  // a record none of whose pixels contribute, a few in a hundred
  // thousand; the per-primitive adjoint turns them into record-field
  // gradients), the wavefront's halves folded onto each other: field 2p
  // in lanes 0-31 of h[p], field 2p+1 in lanes 32-63
  const float gv0 = dx * a_dr;
  const float gv[kGradFloats] = {gv0, a_dry, dx * gv0, dx * a_dry, a_dryy,
                                 a_o, a_be,  a_r,      a_g,        a_b};
#pragma unroll
  for (int p = 0; p < 5; ++p) {
    const FPair sw = swap_halves(gv[2 * p], gv[2 * p + 1]);
    h[p] = sw.a + sw.b;
  }
}

// Two records' folded sums to their totals: the value this lane holds of field
// pair_field(lane) (none where that is -1), of record a in the even rows of 16
// lanes and of record b in the odd rows.  Every step but the last two halves the
// number of registers, as a step of two registers is one of each half, row,
// half-row or bank; a single record's ten fields leave the later steps half
// empty (about 30 vector instructions a record; two at a time take 22 each: 10
// for its halves, 23 here for both).
__device__ __forceinline__ int pair_field(int lane) {
  if ((lane & 3) == 0) return 4 * ((lane >> 2) & 1) + 2 * ((lane >> 3) & 1) + (lane >> 5);
  if ((lane & 15) == 1) return 8 + (lane >> 5);
  return -1;
}
__device__ __forceinline__ float pair_total(const float* ha, const float* hb, int lane) {
  float t[5];   // rows: field 2p of a, of b, field 2p + 1 of a, of b
#pragma unroll
  for (int p = 0; p < 5; ++p) {
    const FPair sw = swap_rows(ha[p], hb[p]);
    t[p] = sw.a + sw.b;
  }
  // u0: t0 in the lower half-rows, t1 in the upper; u1: t2, t3; u2: t4;
  // then t0: banks u0, u1, u0, u1 (fields of t0, t2, t1, t3), t4: u2; then
  // the sums within the banks of four lanes.  (Two wait states between
  // the write of a register and its DPP read: by the order and the nops.)
  float u0, u1, u2;
  asm volatile(
      "s_nop 1\n\t"
      "v_add_f32_dpp %5, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %6, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %7, %4, %4 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %5, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %6, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %4, %7, %7 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %5, %5 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %6, %6 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %4, %4, %4 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %4, %4, %4 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
      : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(t[4]), "=&v"(u0), "=&v"(u1),
        "=&v"(u2));
  return (lane & 1) ? t[4] : t[0];
}

// One wavefront per tile (SPLIT 1) or per band of a tile of two; each adds its
// records' totals itself.
template <int TW, int TH, int BATCH, int SPLIT, bool HAS_DT>
__device__ __forceinline__ void raster_bwd_tile(
    uint32_t tile, int band, float4* s0, float4* s1, float4* s2, uint32_t* s_pos,
    const float* __restrict__ records, const uint32_t* __restrict__ values,
    const uint32_t* __restrict__ ranges, const DevView* __restrict__ views, int n_views,
    const float* __restrict__ t_ws, const uint32_t* __restrict__ ncontrib, const BwdGradients& G,
    float* __restrict__ grad2d) {
  using Geom = TileGeom<TW, TH, SPLIT>;
  constexpr int PPL = Geom::PPL, RSTEP = Geom::RSTEP, PER_LANE = BATCH / 64;
  const int lane = threadIdx.x;
  const DevView& V = views[view_of_tile(views, n_views, tile)];
  const uint32_t lt = tile - V.tile_base;
  const int ty = int(lt) / V.tiles_x, tx = int(lt) - ty * V.tiles_x;
  const int px = tx * TW + lane % TW;
  const int y0 = ty * TH + band * Geom::ROWS, py0 = y0 + lane / TW;
  const float fx = float(px) + 0.5f;
  const float band_y0 = float(y0) + 0.5f, band_y1 = band_y0 + float(Geom::ROWS - 1);
  const uint32_t start = ranges[2 * size_t(tile)];
  BwdPixels<PPL> P;
  const BwdSpan W = load_pixels<PPL, RSTEP, HAS_DT>(P, V, px, py0, t_ws, ncontrib, G);
  const int out_field = pair_field(lane);
  for (uint32_t hi = W.span; hi > 0;) {
    const uint32_t lo = hi > uint32_t(BATCH) ? hi - uint32_t(BATCH) : 0u;
    uint32_t cnt = hi - lo;
    __syncthreads();
    if constexpr (SPLIT == 1) {
#pragma unroll
      for (int m = 0; m < PER_LANE; ++m) {
        const uint32_t q = uint32_t(m * 64 + lane);
        if (q < cnt) {
          const Staged st = stage_record(records, values[start + lo + q]);
          s0[q] = st.g0;
          s1[q] = st.g1;
          s2[q] = st.g2;
        }
      }
    } else {
      // only the records that may reach the band
      uint32_t n_kept = 0;
#pragma unroll
      for (int m = 0; m < PER_LANE; ++m) {
        const uint32_t q = uint32_t(m * 64 + lane);
        bool keep = q < cnt;
        Staged st;
        if (keep) {
          st = stage_record(records, values[start + lo + q]);
          keep = may_reach_rows(st, band_y0, band_y1);
        }
        const uint64_t kept = __ballot(keep);
        if (keep) {
          const uint32_t at = n_kept + uint32_t(__popcll(kept & ((1ull << lane) - 1ull)));
          s0[at] = st.g0;
          s1[at] = st.g1;
          s2[at] = st.g2;
          s_pos[at] = lo + q;
        }
        n_kept += uint32_t(__popcll(kept));
      }
      cnt = n_kept;
    }
    __syncthreads();
    auto record = [&](auto check, int j, float* h) {
      bwd_record<decltype(check)::value, PPL, RSTEP, HAS_DT>(
          P, s0[j], s1[j], s2[j], fx, py0, SPLIT == 1 ? lo + uint32_t(j) : s_pos[j], h);
    };
    // one atomic instruction for two records: lane 0 of each bank adds a field
    // of the first eight and lane 1 of each row one of the last two, odd rows
    // for record b (none for jb < 0)
    auto add_pair = [&](const float* ha, const float* hb, int ja, int jb) {
      const float total = pair_total(ha, hb, lane);
      const int j = (lane & 16) ? jb : ja;
      if (out_field >= 0 && j >= 0)
        atomicAdd(grad2d + size_t(__float_as_uint(s2[j].w)) * kGradFloats + out_field, total);
    };
    auto walk = [&](auto check) {
      int j = int(cnt) - 1;
      for (; j > 0; j -= 2) {
        float ha[5], hb[5];
        record(check, j, ha);
        record(check, j - 1, hb);
        add_pair(ha, hb, j, j - 1);
      }
      if (j == 0) {   // the odd one out: paired with zeros
        float ha[5], hb[5];
        record(check, 0, ha);
#pragma unroll
        for (int p = 0; p < 5; ++p) hb[p] = 0.0f;
        add_pair(ha, hb, 0, -1);
      }
    };
    if (hi <= W.stop_min) walk(std::false_type{}); else walk(std::true_type{});
    hi = lo;
  }
}

// grad_dirty: set, so that a later backward pass over the same binning
// clears the record gradients first.
template <int TW, int TH, int BATCH, int SPLIT>
__global__ void __launch_bounds__(64) raster_bwd_kernel(
    const float* __restrict__ records, const uint32_t* __restrict__ values,
    const uint32_t* __restrict__ ranges, const DevView* __restrict__ views, int n_views,
    uint32_t n_tiles, const uint32_t* __restrict__ order, uint32_t* __restrict__ work,
    uint32_t* __restrict__ grad_dirty, const float* __restrict__ t_ws,
    const uint32_t* __restrict__ ncontrib, BwdGradients G, float* __restrict__ grad2d) {
  __shared__ float4 s0[BATCH], s1[BATCH], s2[BATCH];
  __shared__ uint32_t s_pos[SPLIT > 1 ? BATCH : 1];   // positions of the kept records
  if (blockIdx.x == 0 && threadIdx.x == 0) *grad_dirty = 1u;
  for (uint32_t q = next_tile(work, true); q / SPLIT < n_tiles; q = next_tile(work, false)) {
    const uint32_t tile = order[q / SPLIT];
    const int band = int(q % SPLIT);
    if (G.d_tfinal)
      raster_bwd_tile<TW, TH, BATCH, SPLIT, true>(tile, band, s0, s1, s2, s_pos, records, values,
                                                  ranges, views, n_views, t_ws, ncontrib, G, grad2d);
    else
      raster_bwd_tile<TW, TH, BATCH, SPLIT, false>(tile, band, s0, s1, s2, s_pos, records, values,
                                                   ranges, views, n_views, t_ws, ncontrib, G, grad2d);
  }
}

// Four bands a tile, a wavefront of one workgroup each.  The records are staged
// once for all of them, 64 at a time; a wavefront walks those that may reach its
// band (a scalar mask) and leaves their totals in LDS, and after the batch the
// bands' totals are added in a fixed order, with one atomic add a record and
// field, as for a tile of one wavefront.  Bands that each added their own totals
// did so in any order: with more than two addends a sum depends on it in its last
// bit, and gradients that cancel by a factor of a thousand and more in the chain
// to the parameters changed in their fourth digit from run to run, in one of
// twenty frames of 20,000 7-D in eight views of 160x120.  (Two bands a tile, in
// larger frames, add their own: at most two addends a tile, as two tiles of half
// the height have.  Sums in LDS there cost 8 %: 3250 tiles 76.7 -> 83.0 us.)
// The next batch's records are on their way from memory while a batch is walked.
// 64 tiles of a 3-D frame 34.8 us (32.4 with the bands' own atomics, one
// wavefront a tile 87), 300 tiles 22.8 (21.3, 52), 1200 33.0 (32.9, 65).
constexpr int kBands = 4, kBandBatch = 64, kBandThreads = 64 * kBands;

struct BandShared {
  float4 rec[3][kBandBatch];
  float total[kBands][kBandBatch * kGradFloats];
  uint32_t mask[kBands][2];        // the records of the batch that a band walked
  uint32_t id[2][kBandBatch];      // record indices, of this batch and the next
  uint32_t span[kBands];
};

template <bool HAS_DT>
__device__ __forceinline__ void raster_bwd_bands(
    uint32_t tile, BandShared& S, const float* __restrict__ records,
    const uint32_t* __restrict__ values, const uint32_t* __restrict__ ranges,
    const DevView* __restrict__ views, int n_views, const float* __restrict__ t_ws,
    const uint32_t* __restrict__ ncontrib, const BwdGradients& G, float* __restrict__ grad2d) {
  using Geom = TileGeom<16, 16, kBands>;
  constexpr int PPL = Geom::PPL, RSTEP = Geom::RSTEP;
  const int lane = threadIdx.x & 63, band = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const DevView& V = views[view_of_tile(views, n_views, tile)];
  const uint32_t lt = tile - V.tile_base;
  const int ty = int(lt) / V.tiles_x, tx = int(lt) - ty * V.tiles_x;
  const int px = tx * 16 + lane % 16;
  const int y0 = ty * 16 + band * Geom::ROWS, py0 = y0 + lane / 16;
  const float fx = float(px) + 0.5f;
  const float band_y0 = float(y0) + 0.5f, band_y1 = band_y0 + float(Geom::ROWS - 1);
  const uint32_t start = ranges[2 * size_t(tile)];
  BwdPixels<PPL> P;
  const BwdSpan W = load_pixels<PPL, RSTEP, HAS_DT>(P, V, px, py0, t_ws, ncontrib, G);
  if (lane == 0) S.span[band] = W.span;
  __syncthreads();
  uint32_t hi = 0;
#pragma unroll
  for (int b = 0; b < kBands; ++b) hi = max(hi, S.span[b]);
  hi = __builtin_amdgcn_readfirstlane(hi);
  // wavefronts 0 to 2 stage a 16-byte part of the records each, a record a lane
  float4 next = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  uint32_t next_id = 0;
  auto load = [&](uint32_t lo, uint32_t cnt) {
    if (band < 3 && uint32_t(lane) < cnt) {
      next_id = values[start + lo + uint32_t(lane)];
      next = reinterpret_cast<const float4*>(records + size_t(next_id) * kRecFloats)[band];
    }
  };
  auto store = [&](uint32_t cnt, uint32_t parity) {
    if (band < 3 && uint32_t(lane) < cnt) {
      float4 v = next;
      if (band == 0) v.w = 2.0f * v.w;
      if (band == 1) v.z = hw_log2(v.z);
      S.rec[band][lane] = v;
      if (band == 0) S.id[parity][lane] = next_id;
    }
  };
  const int out_field = pair_field(lane);
  uint32_t cnt = min(hi, uint32_t(kBandBatch)), lo = hi - cnt, parity = 0;
  load(lo, cnt);
  store(cnt, parity);
  __syncthreads();
  while (hi > 0) {
    const uint32_t next_cnt = min(lo, uint32_t(kBandBatch)), next_lo = lo - next_cnt;
    // the batch's records that may reach the band, among those before its span
    bool keep = uint32_t(lane) < cnt && lo + uint32_t(lane) < W.span;
    if (keep) {
      Staged st;
      st.g0 = S.rec[0][lane];
      st.g1 = S.rec[1][lane];
      keep = may_reach_rows(st, band_y0, band_y1);
    }
    const uint64_t mask = __ballot(keep);
    if (lane < 2) S.mask[band][lane] = uint32_t(mask >> (32 * lane));
    load(next_lo, next_cnt);
    auto walk = [&](auto check) {
      uint64_t left = mask;
      auto take = [&]() {
        const int j = 63 - __builtin_clzll(left);
        left &= ~(1ull << j);
        return j;
      };
      while (left != 0) {
        const int ja = take(), jb = left != 0 ? take() : -1, jc = max(jb, 0);
        // (both records' reads ahead of the first's sums)
        const float4 a0 = S.rec[0][ja], a1 = S.rec[1][ja], a2 = S.rec[2][ja];
        const float4 b0 = S.rec[0][jc], b1 = S.rec[1][jc], b2 = S.rec[2][jc];
        __builtin_amdgcn_sched_barrier(0);
        constexpr bool CHECK = decltype(check)::value;
        float ha[5], hb[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        bwd_record<CHECK, PPL, RSTEP, HAS_DT>(P, a0, a1, a2, fx, py0, lo + uint32_t(ja), ha);
        if (jb >= 0)   // (the odd one out is paired with zeros)
          bwd_record<CHECK, PPL, RSTEP, HAS_DT>(P, b0, b1, b2, fx, py0, lo + uint32_t(jb), hb);
        const float total = pair_total(ha, hb, lane);
        const int j = (lane & 16) ? jb : ja;
        if (out_field >= 0 && j >= 0) S.total[band][j * kGradFloats + out_field] = total;
      }
    };
    if (min(hi, W.span) <= W.stop_min) walk(std::false_type{}); else walk(std::true_type{});
    __syncthreads();
    // the bands' totals, one record field a thread (all reads ahead of the sums)
    constexpr int ENTRIES = kBandBatch * kGradFloats, ITEMS = (ENTRIES + kBandThreads - 1) / kBandThreads;
    float part[ITEMS][kBands];
    uint32_t id[ITEMS], walked[ITEMS][kBands];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const int e = min(int(threadIdx.x) + i * kBandThreads, ENTRIES - 1), q = e / kGradFloats;
      id[i] = S.id[parity][q];
#pragma unroll
      for (int b = 0; b < kBands; ++b) {
        part[i][b] = S.total[b][e];
        walked[i][b] = S.mask[b][q >> 5] >> (q & 31);
      }
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const uint32_t e = threadIdx.x + uint32_t(i * kBandThreads), q = e / kGradFloats;
      float sum = 0.0f;
#pragma unroll
      for (int b = 0; b < kBands; ++b) sum = (walked[i][b] & 1u) ? sum + part[i][b] : sum;
      if (e < cnt * kGradFloats &&
          ((walked[i][0] | walked[i][1] | walked[i][2] | walked[i][3]) & 1u) != 0u)
        atomicAdd(grad2d + size_t(id[i]) * kGradFloats + (e - q * kGradFloats), sum);
    }
    parity ^= 1u;
    store(next_cnt, parity);
    __syncthreads();
    hi = lo;
    lo = next_lo;
    cnt = next_cnt;
  }
}

__global__ void __launch_bounds__(kBandThreads) raster_bwd_bands_kernel(
    const float* __restrict__ records, const uint32_t* __restrict__ values,
    const uint32_t* __restrict__ ranges, const DevView* __restrict__ views, int n_views,
    const uint32_t* __restrict__ order, uint32_t* __restrict__ grad_dirty,
    const float* __restrict__ t_ws, const uint32_t* __restrict__ ncontrib, BwdGradients G,
    float* __restrict__ grad2d) {
  __shared__ BandShared S;
  if (blockIdx.x == 0 && threadIdx.x == 0) *grad_dirty = 1u;
  const uint32_t tile = order[blockIdx.x];
  if (G.d_tfinal)
    raster_bwd_bands<true>(tile, S, records, values, ranges, views, n_views, t_ws, ncontrib, G,
                           grad2d);
  else
    raster_bwd_bands<false>(tile, S, records, values, ranges, views, n_views, t_ws, ncontrib, G,
                            grad2d);
}

__global__ void reset_counter_kernel(uint32_t* __restrict__ c) {
  if (threadIdx.x == 0) *c = 0u;
}

// Launch geometry: one wavefront per tile (or per band of one, `split` bands
// a tile), or a persistent grid of `persistent_blocks` wavefronts taking tiles
// from a queue; either way the q-th tile handed out is order[q] (the
// binning's order, longest tiles first).
struct RasterLaunch {
  uint32_t n_tiles;
  uint32_t* work;            // queue counter, or nullptr
  uint32_t grid;
  const uint32_t* order;
  int split;
};

// Wavefronts per tile.  A frame of few tiles leaves SIMDs idle or with one
// or two wavefronts each, and its time is the chain of its longest tile: two
// or four wavefronts a tile, each staging only the records that may reach its
// band, shorten that chain.  Beyond the limits the records staged and tested
// several times (and, backward, reduced several times) cost more than that
// saves.  Measured on 16x16 tiles, one / two / four wavefronts a tile (us, 7-D or
// 3-D where marked, and 6-D):
//   forward   64 tiles (3-D) 62 / 34 / 23, 1200 46 / 26 / 20,
//             2772 47 / 29 / 26 and 52 / 33 / 29, 3600 42 / 27 / 28 and 66 / 42 / 43,
//             4480 46 / 32 / 35 and 56 / 39 / 42, 6600 51 / 45 / 50 and 59 / 53 / 60,
//             8160 62 / 58 / 67 and 111 / 105 / 120, 10000 68 / 66 / 76 and
//             77 / 78 / 89, 14400 (6-D) 118 / 126 / 147
//   backward  64 tiles (3-D) 92 / 51 / 35, 1200 66 / 39 / 33, 1900 (3-D) 190 / 118 / 89
//             and 87 / 55 / 59, 2166 61 / 45 / 45 and 80 / 59 / 61, 2772 68 / 54 / 59
//             and 75 / 61 / 68, 3600 61 / 52 / 65 and 96 / 91 / 118, 4480 76 / 68 / 86
//             and 94 / 85 / 111, 5440 89 / 85 / 111 and 117 / 114 / 153,
//             6600 98 / 103 / 138
// Backward, two stays ahead of one to about 5500 tiles; the line is drawn before,
// as a record's sum over two bands that add their own totals has more addends in
// no fixed order (see raster_bwd_bands).
// A 32x16 tile takes two wavefronts in frames of any size, a lane then has four
// pixels as in a 16x16 tile: forward 1800 tiles 75 / 50, 4080 102 / 80, backward
// with the adjoint 160 / 114 and 266 / 230 (with 256 records a batch, whose LDS
// bounds the wavefronts, forward 75 / 51 and 106 / 109).  Other shapes and batch
// depths take one.
constexpr uint32_t kFwdBands4 = 3072, kFwdBands2 = 8192, kFwdWide256 = 3072;
constexpr uint32_t kBwdBands4 = 2048, kBwdBands2 = 4352;
struct BandLimits {
  uint32_t four, two;   // tiles up to which a tile takes so many wavefronts
};
static BandLimits band_limits(bool fwd, int tw, int th, int batch) {
  if (tw == 32) return BandLimits{0u, fwd && batch > 128 ? kFwdWide256 : 0xffffffffu};
  if (tw != 16 || th != 16 || batch > 64) return BandLimits{0u, 0u};
  return fwd ? BandLimits{kFwdBands4, kFwdBands2} : BandLimits{kBwdBands4, kBwdBands2};
}

static RasterLaunch raster_geometry(uint32_t n_tiles, uint32_t* work, uint32_t persistent_blocks,
                                    const uint32_t* order, BandLimits bands,
                                    hipStream_t st) {
  RasterLaunch g{n_tiles, nullptr, n_tiles, order, 1};
  if (work && persistent_blocks > 0 && persistent_blocks < n_tiles) {
    hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(64), 0, st, work);
    g.work = work;
    g.grid = persistent_blocks;
    return g;
  }
  g.split = n_tiles <= bands.four ? 4 : (n_tiles <= bands.two ? 2 : 1);
  g.grid = n_tiles * uint32_t(g.split);
  return g;
}

template <int TW, int TH, int BATCH, int SPLIT = 1>
static hipError_t raster_fwd_t(const RasterLaunch& g, const float* records, const uint32_t* values,
                               const uint32_t* ranges, const DevView* views, int n_views,
                               float* image, float* t_ws, float* t_user, uint32_t* ncontrib,
                               hipStream_t st) {
  auto launch = [&](auto nan_rows) {
    hipLaunchKernelGGL((raster_fwd_kernel<TW, TH, BATCH, SPLIT, decltype(nan_rows)::value>),
                       dim3(g.grid), dim3(64), 0, st, records, values, ranges, views, n_views,
                       g.n_tiles, g.order, g.work, image, t_ws, t_user, ncontrib);
  };
  // (NaN rows where they are faster: see raster_fwd_tile)
  if constexpr (SPLIT > 1) {
    launch(std::true_type());
  } else if constexpr (TW == 16 && TH == 16 && BATCH == 64) {
    if (g.work) launch(std::false_type());
    else launch(std::true_type());
  } else {
    launch(std::false_type());
  }
  return hipGetLastError();
}

template <int TW, int TH, int BATCH, int SPLIT = 1>
static hipError_t raster_bwd_t(const RasterLaunch& g, uint32_t* grad_dirty, const float* records,
                               const uint32_t* values, const uint32_t* ranges,
                               const DevView* views, int n_views,
                               const float* t_ws, const uint32_t* ncontrib, const BwdGradients& G,
                               float* grad2d, hipStream_t st) {
  if constexpr (SPLIT == kBands)
    hipLaunchKernelGGL(raster_bwd_bands_kernel, dim3(g.n_tiles), dim3(kBandThreads), 0, st, records,
                       values, ranges, views, n_views, g.order, grad_dirty, t_ws, ncontrib, G,
                       grad2d);
  else
    hipLaunchKernelGGL((raster_bwd_kernel<TW, TH, BATCH, SPLIT>), dim3(g.grid), dim3(64), 0, st,
                       records, values, ranges, views, n_views, g.n_tiles, g.order, g.work,
                       grad_dirty, t_ws, ncontrib, G, grad2d);
  return hipGetLastError();
}

#define UBS_TILE_DISPATCH(FN, ...)                                                     \
  do {                                                                                 \
    const int bd = batch <= 64 ? 64 : (batch <= 128 ? 128 : 256);                      \
    if (tw == 16 && th == 16) {                                                        \
      if (bd == 64 && g.split == 4) return FN<16, 16, 64, 4>(__VA_ARGS__);             \
      if (bd == 64 && g.split == 2) return FN<16, 16, 64, 2>(__VA_ARGS__);             \
      if (bd == 64) return FN<16, 16, 64>(__VA_ARGS__);                                \
      if (bd == 128) return FN<16, 16, 128>(__VA_ARGS__);                              \
      return FN<16, 16, 256>(__VA_ARGS__);                                             \
    }                                                                                  \
    if (tw == 16 && th == 8) {                                                         \
      if (bd == 64) return FN<16, 8, 64>(__VA_ARGS__);                                 \
      if (bd == 128) return FN<16, 8, 128>(__VA_ARGS__);                               \
      return FN<16, 8, 256>(__VA_ARGS__);                                              \
    }                                                                                  \
    if (tw == 8 && th == 8) {                                                          \
      if (bd == 64) return FN<8, 8, 64>(__VA_ARGS__);                                  \
      if (bd == 128) return FN<8, 8, 128>(__VA_ARGS__);                                \
      return FN<8, 8, 256>(__VA_ARGS__);                                               \
    }                                                                                  \
    if (tw == 32 && th == 16) {                                                        \
      if (bd == 64 && g.split == 2) return FN<32, 16, 64, 2>(__VA_ARGS__);             \
      if (bd == 128 && g.split == 2) return FN<32, 16, 128, 2>(__VA_ARGS__);           \
      if (g.split == 2) return FN<32, 16, 256, 2>(__VA_ARGS__);                        \
      if (bd == 64) return FN<32, 16, 64>(__VA_ARGS__);                                \
      if (bd == 128) return FN<32, 16, 128>(__VA_ARGS__);                              \
      return FN<32, 16, 256>(__VA_ARGS__);                                             \
    }                                                                                  \
    return hipErrorInvalidValue;                                                       \
  } while (0)

hipError_t launch_raster_fwd(int tw, int th, int batch, uint32_t persistent_blocks,
                             uint32_t* work, const float* records, const uint32_t* values,
                             const uint32_t* ranges, const uint32_t* order,
                             const DevView* views, int n_views,
                             uint32_t n_tiles, float* image, float* t_ws, float* t_user,
                             uint32_t* ncontrib, hipStream_t st) {
  if (n_tiles == 0) return hipSuccess;
  const RasterLaunch g =
      raster_geometry(n_tiles, work, persistent_blocks, order,
                      band_limits(true, tw, th, batch), st);
  UBS_TILE_DISPATCH(raster_fwd_t, g, records, values, ranges, views, n_views, image, t_ws, t_user,
                    ncontrib, st);
}

hipError_t launch_raster_bwd(int tw, int th, int batch, uint32_t persistent_blocks,
                             uint32_t* work, uint32_t* grad_dirty, const float* records,
                             const uint32_t* values,
                             const uint32_t* ranges, const uint32_t* order,
                             const DevView* views, int n_views,
                             uint32_t n_tiles, const float* t_ws, const uint32_t* ncontrib,
                             const float* d_image, const float* d_tfinal, const float* l1_image,
                             const float* l1_target, float l1_scale, float* grad2d,
                             hipStream_t st) {
  if (n_tiles == 0) return hipSuccess;
  const RasterLaunch g =
      raster_geometry(n_tiles, work, persistent_blocks, order,
                      band_limits(false, tw, th, batch), st);
  const BwdGradients G{d_image, d_tfinal, l1_image, l1_target, l1_scale};
  UBS_TILE_DISPATCH(raster_bwd_t, g, grad_dirty, records, values, ranges, views, n_views, t_ws,
                    ncontrib, G, grad2d, st);
}

}  // namespace ubs
