// Per-primitive math of Universal Beta Splatting, forward and adjoint, in
// float64 (T; prim_math_f32.hpp has the float32 option's).
//
// Forward (Section 4.2, 4.3 and the projection of Section 3):
//   Sigma = L L^T with L = [[R_x diag(s_x), 0], [L_qx, L_q]]
//     -> Sigma_x = M M^T, Sigma_xq = M L_qx^T, Sigma_q = L_qx L_qx^T + L_q L_q^T
//        (M = R_x diag(s_x))
//   q = d, [t, d] or [t, d, e] (e: the view's query values beyond 7-D),
//   d = unit(mu_x - camera centre); v = q - mu_q
//   Lhat = chol(Sigma_q); w = Lhat^-1 v;
//   o(q) = o prod_i (1 - tanh(w_i^2))^(4 exp(b_qi))
//   bt_i = min(exp(b_qi), 1); K = Sigma_xq Sigma_q^-1
//   mu_c = mu_x + K diag(bt) v; Sigma_c = Sigma_x - sym(K diag(bt) Sigma_qx)
//   p = W mu_c + t; Sigma' = J W Sigma_c W^T J^T + 0.3 I; conic = Sigma'^-1
//   rho = 1 - (255 o(q))^(-1/beta_x), beta_x = 4 exp(b_x)
// The conditioning is evaluated through the inverse factor Li = Lhat^-1
// (lower triangular), never through Sigma_q^-1 itself:
//   A = Sigma_xq Li^T, H = Sigma_xq diag(bt) Li^T, y = Li diag(bt) v;
//   mu_c = mu_x + A y, Sigma_c = Sigma_x - (A H^T + H A^T) / 2
// (K = A Li).  Sigma_c, A and H do not depend on the view; a view costs the
// triangular products w and y and the projection.
// Adjoint: reverse of the above, written by hand.  A view adds to the
// gradients of Sigma_c, A, Li, bt and the direct parameters; once per
// primitive they are chained through A, H and Li:
//   Sigma_q_bar = Li^T sym(Phi(-Li_bar Li^T)) Li, Phi = lower triangle with
//   the diagonal halved
// (the Cholesky adjoint of Murray 2016 with Lhat_bar = -Li^T Li_bar Li^T,
// where Lhat^T Lhat_bar = -Li_bar Li^T).  Symmetric matrices are kept as one
// triangle, and triangular ones are multiplied within their triangles: the
// adjoint of a 7-D primitive in one view is about 1,900 instructions this
// way, 4,000 with full matrices through Sigma_q^-1.
#pragma once

#include "ubs_internal.hpp"

namespace ubs {

// exp of a float32 parameter.  In float64: x = n ln 2 + r with |r| <= ln 2 / 2
// (ln 2 in two parts, as fdlibm's exp splits it: the first with 21 trailing zero
// bits, so that n times it is exact), exp(r) = 1 + r + r^2 Q(r) with Q the polynomial of degree 9
// through (exp(r) - 1 - r) / r^2 at ten Chebyshev nodes (relative error of
// exp(r) 1.6e-17), scaled by 2^n (to infinity or zero beyond the range).
// 20 instructions; the library's exp, whose argument may be any float64, 32.
template <typename T> __device__ __forceinline__ T m_exp(float x);
template <> __device__ __forceinline__ double m_exp<double>(float x) {
  // (a NaN becomes a number here: every caller's parameter passes the finite test too)
  const float xc = __builtin_amdgcn_fmed3f(x, -1000.0f, 1000.0f);
  const float n = __builtin_rintf(xc * 1.44269504f);
  const double dn = double(n);
  double r = __builtin_fma(dn, -0x1.62e42fee00000p-1, double(xc));
  r = __builtin_fma(dn, -0x1.a39ef35793c76p-33, r);
  double q = 0x1.af38d53857513p-26;
  q = __builtin_fma(q, r, 0x1.2891a8c1d838dp-22);
  q = __builtin_fma(q, r, 0x1.71de0d9c145d0p-19);
  q = __builtin_fma(q, r, 0x1.a019b8ef67c6cp-16);
  q = __builtin_fma(q, r, 0x1.a01a01a7c8d47p-13);
  q = __builtin_fma(q, r, 0x1.6c16c17893833p-10);
  q = __builtin_fma(q, r, 0x1.11111111109adp-7);
  q = __builtin_fma(q, r, 0x1.5555555553d4fp-5);
  q = __builtin_fma(q, r, 0x1.5555555555556p-3);
  q = __builtin_fma(q, r, 0x1.0000000000001p-1);
  const double e = 1.0 + __builtin_fma(r * r, q, r);
  return __builtin_ldexp(e, int(n));
}
// 1 / sqrt(x): where both sqrt(x) and its reciprocal are needed, sqrt(x) is
// taken as x * rsqrt(x) (one library call instead of a root and a division)
template <typename T> __device__ __forceinline__ T m_rsqrt(T x);
template <> __device__ __forceinline__ double m_rsqrt<double>(double x) { return rsqrt(x); }

// Scalar factors of the opacity (the modulation terms, o(q), beta_x, rho)
// are well conditioned in their arguments, so they are evaluated in float32
// whatever T is; the linear algebra of the conditioning stays in T.
__device__ __forceinline__ float s_exp(float x) { return expf(x); }
__device__ __forceinline__ float s_log1p(float x) { return log1pf(x); }

// The same factors in the adjoint, where no decision hangs on their last bit, in
// float64: exp(y) for y <= 0 within 2.2e-10 (exp(y) = 2^n (1 + r + r^2 Q(r)), Q of
// degree 5 through six Chebyshev nodes of |r| <= ln 2 / 2, y below -800 giving 0),
// and log(1 + t) for t in [0, 1] within 8.5e-10 relative and 4.5e-10 absolute (t P(t),
// P of degree 10 through eleven).  13 and 11 instructions; the library's float32
// expf and log1pf take about 25 and 70 and round to float32, but their bits
// decide records' opacities, so the forward keeps them.
// Near w = 0 (t = 1) log(1 - tanh(w^2)) is the difference log 2 - 2 w^2 -
// log(1 + t), which goes to -w^2 and keeps an absolute error of 4.5e-10 (of 3e-8
// with log1pf): d/d b_q of a primitive queried that close to its mean, |w| below
// about 2e-5, has no correct digits, and is at most 4.5e-10 of its d/d log o(q)
// times e.
__device__ __forceinline__ double s_exp_neg(double y) {
  const double yc = __builtin_fmax(y, -800.0);
  const double n = __builtin_rint(yc * 0x1.71547652b82fep+0);
  const double r = __builtin_fma(n, -0x1.62e42fefa39efp-1, yc);
  double q = 0x1.a125285dbcbf1p-13;
  q = __builtin_fma(q, r, 0x1.6d4362097d81ap-10);
  q = __builtin_fma(q, r, 0x1.1110e0de7be2bp-7);
  q = __builtin_fma(q, r, 0x1.5554e8d9c7d96p-5);
  q = __builtin_fma(q, r, 0x1.5555555a7c16bp-3);
  q = __builtin_fma(q, r, 0x1.0000000b9847ep-1);
  return __builtin_ldexp(1.0 + __builtin_fma(r * r, q, r), int(n));
}
__device__ __forceinline__ double s_log1p_unit(double t) {
  double q = 0x1.046679cb2b7ebp-9;
  q = __builtin_fma(q, t, -0x1.b02381e6f92c7p-7);
  q = __builtin_fma(q, t, 0x1.4fed049df857ap-5);
  q = __builtin_fma(q, t, -0x1.4f61d4fd9d9cap-4);
  q = __builtin_fma(q, t, 0x1.fb00b1a6ce14cp-4);
  q = __builtin_fma(q, t, -0x1.49797a179fca6p-3);
  q = __builtin_fma(q, t, 0x1.9742f82e42739p-3);
  q = __builtin_fma(q, t, -0x1.ffb933dac867dp-3);
  q = __builtin_fma(q, t, 0x1.55532471bce50p-2);
  q = __builtin_fma(q, t, -0x1.fffff23ca5d8fp-2);
  q = __builtin_fma(q, t, 0x1.fffffff8bf536p-1);
  return q * t;
}
// (1 + tanh x) / 2 = 1 / (1 + exp(-2 x)), t = exp(-2 x)
__device__ __forceinline__ double s_half_tanh(double t) {
  const double u = 1.0 + t, y = __builtin_amdgcn_rcp(u);
  return __builtin_fma(__builtin_fma(-u, y, 1.0), y, y);
}
// 1 - y^(-1/beta) for y >= 1, as -expm1(-log(y) / beta) (no cancellation for
// y near 1)
__device__ __forceinline__ float s_rho(float y, float beta) { return -expm1f(-logf(y) / beta); }

template <int C> struct Cdim { static constexpr int V = C > 0 ? C : 1; };

// Raw parameters of one primitive (float32, as stored).
template <int C, int ROT>
struct Raw {
  float mu[3];
  float muq[Cdim<C>::V];
  float rq[4];
  float logs[3];
  float lqx[Cdim<C>::V][3];
  float lq[Cdim<C>::V][Cdim<C>::V];  // full lower triangle, diagonal as log
  float bx;
  float bq[Cdim<C>::V];
  float o;
  float rgb[3];
  bool finite;  // every loaded parameter is finite
};

// A primitive's parameters from get(row), the value in parameter row `row`
// (finite: every value read is finite).
template <int C, int ROT, typename Get>
__device__ __forceinline__ void load_raw_rows(Get get, Raw<C, ROT>& r) {
  const ParamRows pr = param_rows(C, ROT);
  bool fin = true;
  auto ld = [&](int row) {
    const float x = get(row);
    fin = fin && isfinite(x);
    return x;
  };
#pragma unroll
  for (int k = 0; k < 3; ++k) r.mu[k] = ld(pr.mu_x + k);
#pragma unroll
  for (int k = 0; k < C; ++k) r.muq[k] = ld(pr.mu_q + k);
#pragma unroll
  for (int k = 0; k < 4; ++k) r.rq[k] = (k < (ROT == UBS_ROT_QUAT ? 4 : 3)) ? ld(pr.rot + k) : 0.0f;
#pragma unroll
  for (int k = 0; k < 3; ++k) r.logs[k] = ld(pr.log_s + k);
#pragma unroll
  for (int a = 0; a < C; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) r.lqx[a][b] = ld(pr.lqx + 3 * a + b);
  int k = 0;
#pragma unroll
  for (int a = 0; a < C; ++a)
#pragma unroll
    for (int b = 0; b <= a; ++b) { r.lq[a][b] = ld(pr.lq + k); ++k; }
  r.bx = ld(pr.b_x);
#pragma unroll
  for (int k2 = 0; k2 < C; ++k2) r.bq[k2] = ld(pr.b_q + k2);
  r.o = ld(pr.o);
#pragma unroll
  for (int k2 = 0; k2 < 3; ++k2) r.rgb[k2] = ld(pr.rgb + k2);
  r.finite = fin;
}

// Primitive i of the component-major array P (row stride n), with streaming
// loads: each parameter is read once per launch.
template <int C, int ROT>
__device__ __forceinline__ void load_raw(const float* __restrict__ P, int64_t n, int64_t i,
                                         Raw<C, ROT>& r) {
  load_raw_rows<C, ROT>(
      [&](int row) { return __builtin_nontemporal_load(&P[int64_t(row) * n + i]); }, r);
}

// Index of entry (a, b) of a symmetric 3 x 3 matrix kept as 00 01 02 11 12 22.
__device__ __forceinline__ constexpr int sym3(int a, int b) {
  return a <= b ? 3 * a - a * (a + 1) / 2 + b : 3 * b - b * (b + 1) / 2 + a;
}

// View-independent quantities of a primitive.
template <typename T, int C, int ROT>
struct Geo {
  T s[3];
  T M[3][3];                         // R diag(s)
  T Sxq[3][Cdim<C>::V];
  T Li[Cdim<C>::V][Cdim<C>::V];      // chol(Sigma_q)^-1 (lower triangle)
  T A[3][Cdim<C>::V];                // Sigma_xq Li^T
  T H[3][Cdim<C>::V];                // Sigma_xq diag(bt) Li^T
  T Sc[6];                           // Sigma_c
  T bt[Cdim<C>::V];                  // min(exp(b_q), 1); 1 without the Beta condition
  T e[Cdim<C>::V];                   // 4 exp(b_q); 1 without the Beta opacity
  bool ok;
  bool beta_cond, beta_opacity;      // the Beta modulations in use (Sec. 5.3 ablations)
};

// Ablation variants (Sec. 5.3), bits of the frame's tuning flags.
constexpr uint32_t kVarNoBetaCond = UBS_TUNE_NO_BETA_COND;
constexpr uint32_t kVarNoBetaOpacity = UBS_TUNE_NO_BETA_OPACITY;

// Activated L_q (lower triangular, diagonal exp of the stored log scale).
template <typename T, int C, int ROT>
__device__ __forceinline__ T lq_entry(const Raw<C, ROT>& r, int a, int b) {
  return b < a ? T(r.lq[a][b]) : (b == a ? m_exp<T>(r.lq[a][a]) : T(0));
}

// s, M = R diag(s) and Sigma_xq = M Lqx^T; false for a zero quaternion.
template <typename T, int C, int ROT>
__device__ __forceinline__ bool geo_frame(const Raw<C, ROT>& r, Geo<T, C, ROT>& g) {
  bool ok = true;
  T R[3][3];
  if (ROT == UBS_ROT_QUAT) {
    T w = r.rq[0], x = r.rq[1], y = r.rq[2], z = r.rq[3];
    T nn = w * w + x * x + y * y + z * z;
    T inv = m_rsqrt<T>(nn);
    if (!(nn > T(0))) ok = false;
    w *= inv; x *= inv; y *= inv; z *= inv;
    R[0][0] = T(1) - T(2) * (y * y + z * z);
    R[0][1] = T(2) * (x * y - w * z);
    R[0][2] = T(2) * (x * z + w * y);
    R[1][0] = T(2) * (x * y + w * z);
    R[1][1] = T(1) - T(2) * (x * x + z * z);
    R[1][2] = T(2) * (y * z - w * x);
    R[2][0] = T(2) * (x * z - w * y);
    R[2][1] = T(2) * (y * z + w * x);
    R[2][2] = T(1) - T(2) * (x * x + y * y);
  } else {
    T w1 = r.rq[0], w2 = r.rq[1], w3 = r.rq[2];
    R[0][0] = T(1); R[0][1] = -w3;  R[0][2] = w2;
    R[1][0] = w3;   R[1][1] = T(1); R[1][2] = -w1;
    R[2][0] = -w2;  R[2][1] = w1;   R[2][2] = T(1);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) g.s[k] = m_exp<T>(r.logs[k]);
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) g.M[a][b] = R[a][b] * g.s[b];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int k = 0; k < C; ++k)
      g.Sxq[a][k] = g.M[a][0] * T(r.lqx[k][0]) + g.M[a][1] * T(r.lqx[k][1]) + g.M[a][2] * T(r.lqx[k][2]);
  return ok;
}

// H = Sigma_xq diag(bt) Li^T.
template <typename T, int C, int ROT>
__device__ __forceinline__ void geo_h(Geo<T, C, ROT>& g) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    T SD[Cdim<C>::V];
#pragma unroll
    for (int m = 0; m < C; ++m) SD[m] = g.Sxq[a][m] * g.bt[m];
#pragma unroll
    for (int k = 0; k < C; ++k) {
      T acc = SD[0] * g.Li[k][0];
#pragma unroll
      for (int m = 1; m <= k; ++m) acc += SD[m] * g.Li[k][m];
      g.H[a][k] = acc;
    }
  }
}

template <typename T, int C, int ROT>
__device__ __forceinline__ void geo_forward(const Raw<C, ROT>& r, Geo<T, C, ROT>& g,
                                            uint32_t variant) {
  g.ok = geo_frame<T, C, ROT>(r, g) && r.finite;
  g.beta_cond = (variant & kVarNoBetaCond) == 0;
  g.beta_opacity = (variant & kVarNoBetaOpacity) == 0;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = a; b < 3; ++b)
      g.Sc[sym3(a, b)] = g.M[a][0] * g.M[b][0] + g.M[a][1] * g.M[b][1] + g.M[a][2] * g.M[b][2];
  if constexpr (C > 0) {
    // Sigma_q and its Cholesky factor, lower triangles (Lh in place of Sigma_q)
    T Lq[Cdim<C>::V][Cdim<C>::V], Lh[Cdim<C>::V][Cdim<C>::V];
#pragma unroll
    for (int a = 0; a < C; ++a)
#pragma unroll
      for (int b = 0; b <= a; ++b) Lq[a][b] = lq_entry<T, C, ROT>(r, a, b);
#pragma unroll
    for (int a = 0; a < C; ++a)
#pragma unroll
      for (int b = 0; b <= a; ++b) {
        T acc = T(r.lqx[a][0]) * T(r.lqx[b][0]) + T(r.lqx[a][1]) * T(r.lqx[b][1]) +
                T(r.lqx[a][2]) * T(r.lqx[b][2]);
#pragma unroll
        for (int k = 0; k <= b; ++k) acc += Lq[a][k] * Lq[b][k];
        Lh[a][b] = acc;
      }
#pragma unroll
    for (int j = 0; j < C; ++j) {
      T d = Lh[j][j];
#pragma unroll
      for (int k = 0; k < j; ++k) d -= Lh[j][k] * Lh[j][k];
      if (!(d > T(0))) { g.ok = false; d = T(1); }
      const T inv = m_rsqrt<T>(d);
      g.Li[j][j] = inv;
#pragma unroll
      for (int i = j + 1; i < C; ++i) {
        T acc = Lh[i][j];
#pragma unroll
        for (int k = 0; k < j; ++k) acc -= Lh[i][k] * Lh[j][k];
        Lh[i][j] = acc * inv;
      }
    }
    // inverse of the lower factor
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
      for (int i = j + 1; i < C; ++i) {
        T acc = Lh[i][j] * g.Li[j][j];
#pragma unroll
        for (int k = j + 1; k < i; ++k) acc += Lh[i][k] * g.Li[k][j];
        g.Li[i][j] = -acc * g.Li[i][i];
      }
#pragma unroll
    for (int k = 0; k < C; ++k) {
      T eb = m_exp<T>(r.bq[k]);
      g.bt[k] = (g.beta_cond && r.bq[k] < 0.0f) ? eb : T(1);
      g.e[k] = g.beta_opacity ? T(4) * eb : T(1);
    }
    // A, H and the conditional covariance
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int k = 0; k < C; ++k) {
        T acc = g.Sxq[a][0] * g.Li[k][0];
#pragma unroll
        for (int m = 1; m <= k; ++m) acc += g.Sxq[a][m] * g.Li[k][m];
        g.A[a][k] = acc;
      }
    geo_h<T, C, ROT>(g);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = a; b < 3; ++b) {
        T acc = g.A[a][0] * g.H[b][0] + g.H[a][0] * g.A[b][0];
#pragma unroll
        for (int k = 1; k < C; ++k) acc += g.A[a][k] * g.H[b][k] + g.H[a][k] * g.A[b][k];
        g.Sc[sym3(a, b)] -= T(0.5) * acc;
      }
  }
}

// Per-view forward state kept for the adjoint.
template <typename T, int C>
struct ViewState {
  T dir[3];              // unit query direction
  T idist;               // 1 / |mu_x - camera centre|
  T v[Cdim<C>::V];       // q - mu_q
  T w[Cdim<C>::V];       // Li v
  T y[Cdim<C>::V];       // Li diag(bt) v
  T ell[Cdim<C>::V];     // log(1 - tanh(w^2))
  T rt[Cdim<C>::V];      // (1 + tanh(w^2)) / 2
  T prod;                // o(q) / o
  T oq;                  // o(q)
  T p[3];                // camera-frame mean
  T iz;                  // 1 / p_z
  T Tm[2][3];            // J W
  T U[2][3];             // J W Sigma_c
  T ca, cb, cc;          // conic
  T mx, my;              // projected mean (pixels)
  T beta;
  T rho;
  bool live;
};

// ADJOINT: for the adjoint, with its scalar factors (rho and live are unused there).
template <typename T, int C, int ROT, bool ADJOINT>
__device__ __forceinline__ void view_forward(const Raw<C, ROT>& r, const Geo<T, C, ROT>& g,
                                             const DevView& V, ViewState<T, C>& s) {
  bool live = g.ok;
  T oq = T(r.o);
  T mu_c[3] = {T(r.mu[0]), T(r.mu[1]), T(r.mu[2])};
  if constexpr (C > 0) {
    T dv[3] = {T(r.mu[0]) - T(V.cam[0]), T(r.mu[1]) - T(V.cam[1]), T(r.mu[2]) - T(V.cam[2])};
    T dd = dv[0] * dv[0] + dv[1] * dv[1] + dv[2] * dv[2];
    T inv = m_rsqrt<T>(dd);
    s.idist = inv;
#pragma unroll
    for (int k = 0; k < 3; ++k) s.dir[k] = dv[k] * inv;
    T q[Cdim<C>::V];
    if constexpr (C >= 4) {   // [t, d, query values of the view beyond 7-D]
      q[0] = T(V.time); q[1] = s.dir[0]; q[2] = s.dir[1]; q[3] = s.dir[2];
#pragma unroll
      for (int k = 4; k < C; ++k) q[k] = T(V.query[k - 4]);
    } else if constexpr (C == 3) {
      q[0] = s.dir[0]; q[1] = s.dir[1]; q[2] = s.dir[2];
    } else {
#pragma unroll
      for (int k = 0; k < C; ++k) q[k] = s.dir[k];   // C < 3: leading direction components
    }
    T Dv[Cdim<C>::V];
#pragma unroll
    for (int k = 0; k < C; ++k) {
      s.v[k] = q[k] - T(r.muq[k]);
      Dv[k] = g.bt[k] * s.v[k];
    }
    // whitening and opacity: log(1 - tanh x) = log 2 - 2x - log1p(exp(-2x))
    T lsum = T(0);
#pragma unroll
    for (int i = 0; i < C; ++i) {
      T acc = g.Li[i][0] * s.v[0], acc2 = g.Li[i][0] * Dv[0];
#pragma unroll
      for (int k = 1; k <= i; ++k) {
        acc += g.Li[i][k] * s.v[k];
        acc2 += g.Li[i][k] * Dv[k];
      }
      s.w[i] = acc;
      s.y[i] = acc2;
      const T x = acc * acc;
      // Gaussian opacity (ablation): e = 1 and ell = -w^2 / 2
      if constexpr (ADJOINT) {
        const T t = s_exp_neg(T(-2) * x);
        s.rt[i] = s_half_tanh(t);
        s.ell[i] = g.beta_opacity
                       ? T(0.69314718055994530942) - T(2) * x - s_log1p_unit(t)
                       : T(-0.5) * x;
      } else {
        s.ell[i] = g.beta_opacity
                       ? T(0.69314718055994530942) - T(2) * x - T(s_log1p(s_exp(-2.0f * float(x))))
                       : T(-0.5) * x;
      }
      lsum += g.e[i] * s.ell[i];
    }
    s.prod = ADJOINT ? s_exp_neg(lsum) : T(s_exp(float(lsum)));
    oq = T(r.o) * s.prod;
    // mu_c = mu_x + A y
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int k = 0; k < C; ++k) mu_c[a] += g.A[a][k] * s.y[k];
  }
  s.oq = oq;
  // projection
  T p[3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
    p[a] = T(V.R[3 * a]) * mu_c[0] + T(V.R[3 * a + 1]) * mu_c[1] + T(V.R[3 * a + 2]) * mu_c[2] + T(V.t[a]);
#pragma unroll
  for (int a = 0; a < 3; ++a) s.p[a] = p[a];
  if (!(p[2] > T(kNear))) live = false;
  T z = p[2] > T(kNear) ? p[2] : T(1);
  T iz = T(1) / z;
  s.iz = iz;
  T fx = T(V.fx), fy = T(V.fy);
  T J00 = fx * iz, J02 = -fx * p[0] * iz * iz;
  T J11 = fy * iz, J12 = -fy * p[1] * iz * iz;
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    s.Tm[0][b] = J00 * T(V.R[b]) + J02 * T(V.R[6 + b]);
    s.Tm[1][b] = J11 * T(V.R[3 + b]) + J12 * T(V.R[6 + b]);
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b)
      s.U[a][b] = s.Tm[a][0] * g.Sc[sym3(0, b)] + s.Tm[a][1] * g.Sc[sym3(1, b)] +
                  s.Tm[a][2] * g.Sc[sym3(2, b)];
  const T Sp00 = s.U[0][0] * s.Tm[0][0] + s.U[0][1] * s.Tm[0][1] + s.U[0][2] * s.Tm[0][2] + T(kDilation);
  const T Sp01 = s.U[0][0] * s.Tm[1][0] + s.U[0][1] * s.Tm[1][1] + s.U[0][2] * s.Tm[1][2];
  const T Sp11 = s.U[1][0] * s.Tm[1][0] + s.U[1][1] * s.Tm[1][1] + s.U[1][2] * s.Tm[1][2] + T(kDilation);
  T det = Sp00 * Sp11 - Sp01 * Sp01;
  if (!(det > T(0)) || !(Sp00 > T(0)) || !(Sp11 > T(0))) live = false;
  T idet = T(1) / (det > T(0) ? det : T(1));
  s.mx = fx * p[0] * iz + T(V.cx);
  s.my = fy * p[1] * iz + T(V.cy);
  s.ca = Sp11 * idet;
  s.cb = -Sp01 * idet;
  s.cc = Sp00 * idet;
  s.beta = T(4) * T(s_exp(r.bx));
  if (!(oq >= T(kAlphaMin))) live = false;
  T oqs = oq >= T(kAlphaMin) ? oq : T(1);
  s.rho = T(s_rho(float(T(255) * oqs), float(s.beta)));
  if (!(s.rho > T(0))) live = false;
  s.live = live;
}

// The gradients w.r.t. the view-independent quantities, summed over views.
// Rows: G_Sc (6), bt, G_A (3 C), G_Li (lower triangle, row-major), mu_x, mu_q,
// b_q, b_x, o, rgb.
struct GradRows {
  int sc, bt, a, li, mu, muq, bq, bx, o, rgb, N;
};
__host__ __device__ constexpr GradRows grad_rows(int C) {
  GradRows r{};
  int k = 0;
  r.sc = k; k += 6;
  r.bt = k; k += C;
  r.a = k; k += 3 * C;
  r.li = k; k += C * (C + 1) / 2;
  r.mu = k; k += 3;
  r.muq = k; k += C;
  r.bq = k; k += C;
  r.bx = k; k += 1;
  r.o = k; k += 1;
  r.rgb = k; k += 3;
  r.N = k;
  return r;
}

// The sums of LANES primitives, in LDS: a lane's column holds its primitive's.
// A view's contribution is added in float64.  G_Sc, and with ONE_VIEW G_A and bt,
// stay float64: the last step forms parts of most parameters' gradients from
// them, whose error they would be if rounded (rotations and log scales of one 7-D
// view 3.6e-8 relative to float64, with the three in float64 2.5e-8).  The others
// are rounded as they are kept.  (G_A in float64 over several views made that
// adjoint 6 % slower by its LDS traffic, and it is no further off without than the
// forms through Sigma_q^-1 were: 7-D in eight views 5.7e-8 against 7.0e-8.)
template <int C, int LANES, bool ONE_VIEW>
struct GradSums {
  static constexpr int kWide = ONE_VIEW ? grad_rows(C).li : grad_rows(C).bt;
  static constexpr int kRows = grad_rows(C).N - kWide;
  double wide[kWide][LANES];
  float row[kRows][LANES];
  __host__ __device__ __forceinline__ void clear(int lane) {
#pragma unroll
    for (int k = 0; k < kWide; ++k) wide[k][lane] = 0.0;
#pragma unroll
    for (int k = 0; k < kRows; ++k) row[k][lane] = 0.0f;
  }
  __host__ __device__ __forceinline__ void add(int k, double x, int lane) {
    if (k < kWide) wide[k][lane] += x;
    else row[k - kWide][lane] = float(double(row[k - kWide][lane]) + x);
  }
  __host__ __device__ __forceinline__ double get(int k, int lane) const {
    return k < kWide ? wide[k][lane] : double(row[k - kWide][lane]);
  }
};

// Adjoint of view_forward for one view.  gr: d loss / d record fields
// (mx, my, a, b, c, o(q), beta, r, g, b); add(row, x) adds to a gradient row.
template <typename T, int C, int ROT, typename Add>
__device__ __forceinline__ void view_backward(const Geo<T, C, ROT>& g, const DevView& V,
                                              const ViewState<T, C>& s, const float* gr, Add add) {
  constexpr GradRows row = grad_rows(C);
  add(row.rgb, T(gr[7]));
  add(row.rgb + 1, T(gr[8]));
  add(row.rgb + 2, T(gr[9]));
  add(row.bx, T(gr[6]) * s.beta);
  // conic = Sigma'^-1:  G_Sigma' = -A G_A A with G_A = [[ga, gb/2], [gb/2, gc]]
  T a = s.ca, b = s.cb, c = s.cc;
  T ga = T(gr[2]), gb = T(0.5) * T(gr[3]), gc = T(gr[4]);
  T P00 = a * ga + b * gb, P01 = a * gb + b * gc;   // A G_A
  T P10 = b * ga + c * gb, P11 = b * gb + c * gc;
  T G00 = -(P00 * a + P01 * b);
  T G01 = -(P00 * b + P01 * c);
  T G11 = -(P10 * b + P11 * c);
  // Sigma' = Tm Sc Tm^T + 0.3 I
  T GT[2][3];   // G_Sigma' Tm
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    GT[0][j] = G00 * s.Tm[0][j] + G01 * s.Tm[1][j];
    GT[1][j] = G01 * s.Tm[0][j] + G11 * s.Tm[1][j];
  }
#pragma unroll
  for (int i = 0; i < 3; ++i)   // G_Sc = Tm^T G_Sigma' Tm
#pragma unroll
    for (int j = i; j < 3; ++j) add(row.sc + sym3(i, j), s.Tm[0][i] * GT[0][j] + s.Tm[1][i] * GT[1][j]);
  T GTm[2][3];  // 2 G_Sigma' Tm Sc
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    GTm[0][j] = T(2) * (G00 * s.U[0][j] + G01 * s.U[1][j]);
    GTm[1][j] = T(2) * (G01 * s.U[0][j] + G11 * s.U[1][j]);
  }
  // Tm = J W  ->  G_J = GTm W^T  (W row-major in V.R)
  T GJ00 = GTm[0][0] * T(V.R[0]) + GTm[0][1] * T(V.R[1]) + GTm[0][2] * T(V.R[2]);
  T GJ02 = GTm[0][0] * T(V.R[6]) + GTm[0][1] * T(V.R[7]) + GTm[0][2] * T(V.R[8]);
  T GJ11 = GTm[1][0] * T(V.R[3]) + GTm[1][1] * T(V.R[4]) + GTm[1][2] * T(V.R[5]);
  T GJ12 = GTm[1][0] * T(V.R[6]) + GTm[1][1] * T(V.R[7]) + GTm[1][2] * T(V.R[8]);
  // p -> (fx p_x / z, fy p_y / z), J00 = fx / z, J02 = -fx p_x / z^2, ...
  T iz = s.iz;
  T fxz = T(V.fx) * iz, fyz = T(V.fy) * iz;
  T xz = s.p[0] * iz, yz = s.p[1] * iz;
  T gmx = T(gr[0]), gmy = T(gr[1]);
  T gp[3];
  gp[0] = fxz * (gmx - GJ02 * iz);
  gp[1] = fyz * (gmy - GJ12 * iz);
  gp[2] = fxz * (T(2) * GJ02 * iz * xz - gmx * xz - GJ00 * iz) +
          fyz * (T(2) * GJ12 * iz * yz - gmy * yz - GJ11 * iz);
  T gmc[3];
#pragma unroll
  for (int j = 0; j < 3; ++j)
    gmc[j] = T(V.R[j]) * gp[0] + T(V.R[3 + j]) * gp[1] + T(V.R[6 + j]) * gp[2];
  T goq = T(gr[5]);
  if constexpr (C == 0) {
    add(row.o, goq);
#pragma unroll
    for (int i = 0; i < 3; ++i) add(row.mu + i, gmc[i]);
  } else {
    // mu_c = mu_x + A y, y = Li diag(bt) v
    T gy[Cdim<C>::V];
#pragma unroll
    for (int k = 0; k < C; ++k) {
      gy[k] = g.A[0][k] * gmc[0] + g.A[1][k] * gmc[1] + g.A[2][k] * gmc[2];
#pragma unroll
      for (int i = 0; i < 3; ++i) add(row.a + C * i + k, gmc[i] * s.y[k]);
    }
    // ---- opacity ----  o(q) = o exp(sum e_i ell_i),  ell = log(1 - tanh(w^2)),
    // d ell / d w = -2 w (1 + tanh(w^2))
    add(row.o, goq * s.prod);
    const T go = goq * s.oq;
    T gw[Cdim<C>::V];
#pragma unroll
    for (int i = 0; i < C; ++i) {
      if (g.beta_opacity) {
        const T ge = go * g.e[i];
        add(row.bq + i, ge * s.ell[i]);
        gw[i] = T(-4) * ge * s.rt[i] * s.w[i];
      } else {
        gw[i] = -go * s.w[i];   // d(-w^2/2)/dw; no b_q dependence
      }
    }
    // w = Li v, y = Li diag(bt) v
    T gv[Cdim<C>::V];
#pragma unroll
    for (int k = 0; k < C; ++k) {
      T ty = g.Li[k][k] * gy[k], tw = g.Li[k][k] * gw[k];
#pragma unroll
      for (int i = k + 1; i < C; ++i) {
        ty += g.Li[i][k] * gy[i];
        tw += g.Li[i][k] * gw[i];
      }
      add(row.bt + k, ty * s.v[k]);
      gv[k] = g.bt[k] * ty + tw;
    }
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
      for (int j = 0; j <= i; ++j)
        add(row.li + i * (i + 1) / 2 + j, (gy[i] * g.bt[j] + gw[i]) * s.v[j]);
    // v = q - mu_q ; q = [t, d] or d ; d = unit(mu_x - cam)
#pragma unroll
    for (int k = 0; k < C; ++k) add(row.muq + k, -gv[k]);
    T gd[3] = {T(0), T(0), T(0)};
    if constexpr (C >= 4) { gd[0] = gv[1]; gd[1] = gv[2]; gd[2] = gv[3]; }
    else if constexpr (C == 3) { gd[0] = gv[0]; gd[1] = gv[1]; gd[2] = gv[2]; }
    else {
#pragma unroll
      for (int k = 0; k < C; ++k) gd[k] = gv[k];
    }
    T dg = s.dir[0] * gd[0] + s.dir[1] * gd[1] + s.dir[2] * gd[2];
#pragma unroll
    for (int k = 0; k < 3; ++k) add(row.mu + k, gmc[k] + (gd[k] - s.dir[k] * dg) * s.idist);
  }
}

// Final chain from the view-independent gradients to the raw parameters.
// grad(row) is the sum of a gradient row; out(row, value) takes the gradient of
// one parameter row.
template <typename T, int C, int ROT, typename Grad, typename Out>
__device__ __forceinline__ void geo_backward(const Raw<C, ROT>& r, const Geo<T, C, ROT>& g,
                                             Grad grad, Out out) {
  const ParamRows pr = param_rows(C, ROT);
  constexpr GradRows row = grad_rows(C);
  T Gsc[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) Gsc[k] = grad(row.sc + k);
  T GM[3][3];
  // Sigma_c = M M^T - ... (G_Sc symmetric): G_M = 2 G_Sc M
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      GM[i][j] = T(2) * (Gsc[sym3(i, 0)] * g.M[0][j] + Gsc[sym3(i, 1)] * g.M[1][j] +
                         Gsc[sym3(i, 2)] * g.M[2][j]);
  if constexpr (C > 0) {
    // Sigma_c = Sigma_x - (A H^T + H A^T) / 2: G_A -= G_Sc H, G_H = -G_Sc A;
    // A = Sigma_xq Li^T, H = Sigma_xq diag(bt) Li^T
    T GL[Cdim<C>::V][Cdim<C>::V];   // w.r.t. Li (lower triangle)
    T GX[3][Cdim<C>::V];            // w.r.t. Sigma_xq
    T Gbt[Cdim<C>::V];
#pragma unroll
    for (int i = 0; i < C; ++i) {
#pragma unroll
      for (int j = 0; j <= i; ++j) GL[i][j] = grad(row.li + i * (i + 1) / 2 + j);
      Gbt[i] = grad(row.bt + i);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      T GA[Cdim<C>::V], GH[Cdim<C>::V];
#pragma unroll
      for (int k = 0; k < C; ++k) {
        GA[k] = grad(row.a + C * a + k);
        GH[k] = T(0);
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          GA[k] -= Gsc[sym3(a, b)] * g.H[b][k];
          GH[k] -= Gsc[sym3(a, b)] * g.A[b][k];
        }
      }
#pragma unroll
      for (int m = 0; m < C; ++m) {
        T xa = GA[m] * g.Li[m][m], xh = GH[m] * g.Li[m][m];
#pragma unroll
        for (int k = m + 1; k < C; ++k) {
          xa += GA[k] * g.Li[k][m];
          xh += GH[k] * g.Li[k][m];
        }
        GX[a][m] = xa + g.bt[m] * xh;
        Gbt[m] += g.Sxq[a][m] * xh;
#pragma unroll
        for (int k = m; k < C; ++k) GL[k][m] += (GA[k] + GH[k] * g.bt[m]) * g.Sxq[a][m];
      }
    }
    // W = sym(-GL Li^T) (lower triangle mirrored): G_Sq + G_Sq^T = Li^T W Li
    T GSs[Cdim<C>::V][Cdim<C>::V];
    {
      T W[Cdim<C>::V][Cdim<C>::V];
#pragma unroll
      for (int i = 0; i < C; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
          T acc = GL[i][0] * g.Li[j][0];
#pragma unroll
          for (int k = 1; k <= j; ++k) acc += GL[i][k] * g.Li[j][k];
          W[i][j] = W[j][i] = -acc;
        }
#pragma unroll
      for (int j = 0; j < C; ++j) {
        T WL[Cdim<C>::V];   // column j of W Li
#pragma unroll
        for (int i = 0; i < C; ++i) {
          T acc = W[i][j] * g.Li[j][j];
#pragma unroll
          for (int k = j + 1; k < C; ++k) acc += W[i][k] * g.Li[k][j];
          WL[i] = acc;
        }
#pragma unroll
        for (int i = j; i < C; ++i) {
          T acc = g.Li[i][i] * WL[i];
#pragma unroll
          for (int k = i + 1; k < C; ++k) acc += g.Li[k][i] * WL[k];
          GSs[i][j] = GSs[j][i] = acc;
        }
      }
    }
    // Sigma_q = Lqx Lqx^T + Lq Lq^T ; Sigma_xq = M Lqx^T
#pragma unroll
    for (int k = 0; k < C; ++k)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        T acc = GX[0][k] * g.M[0][j] + GX[1][k] * g.M[1][j] + GX[2][k] * g.M[2][j];
#pragma unroll
        for (int m = 0; m < C; ++m) acc += GSs[k][m] * T(r.lqx[m][j]);
        out(pr.lqx + 3 * k + j, acc);
      }
    int idx = 0;
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
      for (int j = 0; j <= i; ++j) {
        const T Ljj = lq_entry<T, C, ROT>(r, j, j);
        T acc = GSs[i][j] * Ljj;
#pragma unroll
        for (int m = j + 1; m < C; ++m) acc += GSs[i][m] * T(r.lq[m][j]);
        out(pr.lq + idx, i == j ? acc * Ljj : acc);
        ++idx;
      }
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
#pragma unroll
        for (int k = 0; k < C; ++k) GM[i][j] += GX[i][k] * T(r.lqx[k][j]);
      }
#pragma unroll
    for (int k = 0; k < C; ++k) {
      out(pr.mu_q + k, grad(row.muq + k));
      T gbq = grad(row.bq + k);
      if (g.beta_cond && r.bq[k] < 0.0f) gbq += Gbt[k] * g.bt[k];
      out(pr.b_q + k, gbq);
    }
  }
  // M = R diag(s)
  T GR[3][3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    T acc = T(0);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      GR[i][j] = GM[i][j] * g.s[j];
      acc += GM[i][j] * g.M[i][j];   // M = R diag(s): d/d log s_j = sum_i GM_ij R_ij s_j
    }
    out(pr.log_s + j, acc);
  }
  if (ROT == UBS_ROT_QUAT) {
    T iq = m_rsqrt<T>(T(r.rq[0]) * T(r.rq[0]) + T(r.rq[1]) * T(r.rq[1]) +
                      T(r.rq[2]) * T(r.rq[2]) + T(r.rq[3]) * T(r.rq[3]));
    T w = T(r.rq[0]) * iq, x = T(r.rq[1]) * iq, y = T(r.rq[2]) * iq, z = T(r.rq[3]) * iq;
    T gw = T(2) * (-z * GR[0][1] + y * GR[0][2] + z * GR[1][0] - x * GR[1][2] - y * GR[2][0] + x * GR[2][1]);
    T gx = T(2) * (y * GR[0][1] + z * GR[0][2] + y * GR[1][0] - T(2) * x * GR[1][1] - w * GR[1][2] +
                   z * GR[2][0] + w * GR[2][1] - T(2) * x * GR[2][2]);
    T gy = T(2) * (-T(2) * y * GR[0][0] + x * GR[0][1] + w * GR[0][2] + x * GR[1][0] + z * GR[1][2] -
                   w * GR[2][0] + z * GR[2][1] - T(2) * y * GR[2][2]);
    T gz = T(2) * (-T(2) * z * GR[0][0] - w * GR[0][1] + x * GR[0][2] + w * GR[1][0] - T(2) * z * GR[1][1] +
                   y * GR[1][2] + x * GR[2][0] + y * GR[2][1]);
    T dotq = w * gw + x * gx + y * gy + z * gz;
    out(pr.rot + 0, (gw - w * dotq) * iq);
    out(pr.rot + 1, (gx - x * dotq) * iq);
    out(pr.rot + 2, (gy - y * dotq) * iq);
    out(pr.rot + 3, (gz - z * dotq) * iq);
  } else {
    out(pr.rot + 0, GR[2][1] - GR[1][2]);
    out(pr.rot + 1, GR[0][2] - GR[2][0]);
    out(pr.rot + 2, GR[1][0] - GR[0][1]);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    out(pr.mu_x + k, grad(row.mu + k));
    out(pr.rgb + k, grad(row.rgb + k));
  }
  out(pr.b_x, grad(row.bx));
  out(pr.o, grad(row.o));
}

}  // namespace ubs
