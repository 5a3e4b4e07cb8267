// The per-primitive math of prim_math.hpp for the float32 option
// (UBS_TUNE_PRE_FP32), evaluated through full matrices and K = Sigma_xq
// Sigma_q^-1.  The triangular forms of prim_math.hpp are cheaper and, in
// float64, the same to the records' last bit; in float32 another order of
// operations is another record: with them a third of the records changed in
// their last bits, and the image's error against float64 grew from 6.6e-5 to
// 1.1e-4 (100,000 7-D primitives at 640x480).
#pragma once

#include "prim_math.hpp"

namespace ubs {
namespace f32 {

// View-independent quantities of a primitive.
template <int C, int ROT>
struct Geo {
  float s[3];
  float M[3][3];                         // R diag(s)
  float Sx[3][3];
  float Sxq[3][Cdim<C>::V];
  float Lh[Cdim<C>::V][Cdim<C>::V];      // chol(Sigma_q)
  float Li[Cdim<C>::V][Cdim<C>::V];      // Lh^-1 (lower)
  float bt[Cdim<C>::V];                  // min(exp(b_q), 1); 1 without the Beta condition
  float e[Cdim<C>::V];                   // 4 exp(b_q); 1 without the Beta opacity
  bool ok;
  bool beta_cond, beta_opacity;      // the Beta modulations in use (Sec. 5.3 ablations)
};

// Activated L_q (lower triangular, diagonal exp of the stored log scale).
template <int C, int ROT>
__device__ __forceinline__ float lq_entry(const Raw<C, ROT>& r, int a, int b) {
  return b < a ? r.lq[a][b] : (b == a ? expf(r.lq[a][a]) : 0.0f);
}

template <int C, int ROT>
__device__ __forceinline__ void geo_forward(const Raw<C, ROT>& r, Geo<C, ROT>& g,
                                            uint32_t variant) {
  g.ok = r.finite;
  g.beta_cond = (variant & kVarNoBetaCond) == 0;
  g.beta_opacity = (variant & kVarNoBetaOpacity) == 0;
  float R[3][3];
  if (ROT == UBS_ROT_QUAT) {
    float w = r.rq[0], x = r.rq[1], y = r.rq[2], z = r.rq[3];
    float nn = w * w + x * x + y * y + z * z;
    float inv = rsqrtf(nn);
    if (!(nn > 0.0f)) g.ok = false;
    w *= inv; x *= inv; y *= inv; z *= inv;
    R[0][0] = 1.0f - 2.0f * (y * y + z * z);
    R[0][1] = 2.0f * (x * y - w * z);
    R[0][2] = 2.0f * (x * z + w * y);
    R[1][0] = 2.0f * (x * y + w * z);
    R[1][1] = 1.0f - 2.0f * (x * x + z * z);
    R[1][2] = 2.0f * (y * z - w * x);
    R[2][0] = 2.0f * (x * z - w * y);
    R[2][1] = 2.0f * (y * z + w * x);
    R[2][2] = 1.0f - 2.0f * (x * x + y * y);
  } else {
    float w1 = r.rq[0], w2 = r.rq[1], w3 = r.rq[2];
    R[0][0] = 1.0f; R[0][1] = -w3;  R[0][2] = w2;
    R[1][0] = w3;   R[1][1] = 1.0f; R[1][2] = -w1;
    R[2][0] = -w2;  R[2][1] = w1;   R[2][2] = 1.0f;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) g.s[k] = expf(r.logs[k]);
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) g.M[a][b] = R[a][b] * g.s[b];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b <= a; ++b) {
      g.Sx[a][b] = g.M[a][0] * g.M[b][0] + g.M[a][1] * g.M[b][1] + g.M[a][2] * g.M[b][2];
      g.Sx[b][a] = g.Sx[a][b];
    }
  if constexpr (C > 0) {
    float Lq[Cdim<C>::V][Cdim<C>::V];
#pragma unroll
    for (int a = 0; a < C; ++a)
#pragma unroll
      for (int b = 0; b < C; ++b) Lq[a][b] = lq_entry<C, ROT>(r, a, b);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int k = 0; k < C; ++k)
        g.Sxq[a][k] = g.M[a][0] * r.lqx[k][0] + g.M[a][1] * r.lqx[k][1] + g.M[a][2] * r.lqx[k][2];
    float Sq[Cdim<C>::V][Cdim<C>::V];
#pragma unroll
    for (int a = 0; a < C; ++a)
#pragma unroll
      for (int b = 0; b < C; ++b) {
        float acc = r.lqx[a][0] * r.lqx[b][0] + r.lqx[a][1] * r.lqx[b][1] +
                r.lqx[a][2] * r.lqx[b][2];
#pragma unroll
        for (int k = 0; k < C; ++k) acc += Lq[a][k] * Lq[b][k];
        Sq[a][b] = acc;
      }
    // Cholesky of Sigma_q (lower, positive diagonal)
#pragma unroll
    for (int j = 0; j < C; ++j) {
      float d = Sq[j][j];
#pragma unroll
      for (int k = 0; k < j; ++k) d -= g.Lh[j][k] * g.Lh[j][k];
      if (!(d > 0.0f)) { g.ok = false; d = 1.0f; }
      float inv = rsqrtf(d);
      g.Lh[j][j] = d * inv;
      g.Li[j][j] = inv;
#pragma unroll
      for (int i = j + 1; i < C; ++i) {
        float acc = Sq[i][j];
#pragma unroll
        for (int k = 0; k < j; ++k) acc -= g.Lh[i][k] * g.Lh[j][k];
        g.Lh[i][j] = acc * inv;
      }
#pragma unroll
      for (int i = 0; i < j; ++i) g.Lh[i][j] = 0.0f;
    }
    // inverse of the lower factor
#pragma unroll
    for (int j = 0; j < C; ++j) {
#pragma unroll
      for (int i = 0; i < C; ++i) {
        if (i < j) { g.Li[i][j] = 0.0f; continue; }
        if (i == j) continue;   // 1 / Lh[i][i], set by the factorisation
        float acc = 0.0f;
#pragma unroll
        for (int k = j; k < i; ++k) acc += g.Lh[i][k] * g.Li[k][j];
        g.Li[i][j] = -acc * g.Li[i][i];
      }
    }
#pragma unroll
    for (int k = 0; k < C; ++k) {
      float eb = expf(r.bq[k]);
      g.bt[k] = (g.beta_cond && r.bq[k] < 0.0f) ? eb : 1.0f;
      g.e[k] = g.beta_opacity ? 4.0f * eb : 1.0f;
    }
  }
}

// Per-view forward state kept for the adjoint.
template <int C>
struct ViewState {
  float dir[3];              // unit query direction
  float dist;                // |mu_x - camera centre|
  float v[Cdim<C>::V];       // q - mu_q
  float w[Cdim<C>::V];       // Lh^-1 v
  float ell[Cdim<C>::V];     // log(1 - tanh(w^2))
  float oq;                  // o(q)
  float mu_c[3];
  float Sc[3][3];
  float p[3];                // camera-frame mean
  float Tm[2][3];            // J W
  float Sp00, Sp01, Sp11;
  float ca, cb, cc;          // conic
  float mx, my;              // projected mean (pixels)
  float beta;
  float rho;
  bool live;
};

template <int C, int ROT>
__device__ __forceinline__ void view_forward(const Raw<C, ROT>& r, const Geo<C, ROT>& g,
                                             const DevView& V, ViewState<C>& s) {
  bool live = g.ok;
  float oq = r.o;
  float mu_c[3] = {r.mu[0], r.mu[1], r.mu[2]};
  float Sc[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) Sc[a][b] = g.Sx[a][b];
  if constexpr (C > 0) {
    float dv[3] = {r.mu[0] - V.cam[0], r.mu[1] - V.cam[1], r.mu[2] - V.cam[2]};
    float dd = dv[0] * dv[0] + dv[1] * dv[1] + dv[2] * dv[2];
    float inv = rsqrtf(dd);
    float dist = dd * inv;
    s.dist = dist;
#pragma unroll
    for (int k = 0; k < 3; ++k) s.dir[k] = dv[k] * inv;
    float q[Cdim<C>::V];
    if constexpr (C >= 4) {   // [t, d, query values of the view beyond 7-D]
      q[0] = V.time; q[1] = s.dir[0]; q[2] = s.dir[1]; q[3] = s.dir[2];
#pragma unroll
      for (int k = 4; k < C; ++k) q[k] = V.query[k - 4];
    } else if constexpr (C == 3) {
      q[0] = s.dir[0]; q[1] = s.dir[1]; q[2] = s.dir[2];
    } else {
#pragma unroll
      for (int k = 0; k < C; ++k) q[k] = s.dir[k];   // C < 3: leading direction components
    }
#pragma unroll
    for (int k = 0; k < C; ++k) s.v[k] = q[k] - r.muq[k];
    // whitening and opacity: log(1 - tanh x) = log 2 - 2x - log1p(exp(-2x))
    float lsum = 0.0f;
#pragma unroll
    for (int i = 0; i < C; ++i) {
      float acc = 0.0f;
#pragma unroll
      for (int k = 0; k <= i; ++k) acc += g.Li[i][k] * s.v[k];
      s.w[i] = acc;
      float x = acc * acc;
      // Gaussian opacity (ablation): e = 1 and ell = -w^2 / 2
      s.ell[i] = g.beta_opacity
                     ? 0.69314718f - 2.0f * x - float(log1pf(expf(-2.0f * x)))
                     : -0.5f * x;
      lsum += g.e[i] * s.ell[i];
    }
    oq = r.o * float(s_exp(float(lsum)));
    // conditioning: K = Sigma_xq Sigma_q^-1 = (Sigma_xq Lh^-T) Lh^-1
    float K[3][Cdim<C>::V];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      float A[Cdim<C>::V];
#pragma unroll
      for (int k = 0; k < C; ++k) {
        float acc = 0.0f;
#pragma unroll
        for (int m = 0; m <= k; ++m) acc += g.Sxq[a][m] * g.Li[k][m];
        A[k] = acc;
      }
#pragma unroll
      for (int k = 0; k < C; ++k) {
        float acc = 0.0f;
#pragma unroll
        for (int m = k; m < C; ++m) acc += A[m] * g.Li[m][k];
        K[a][k] = acc;
      }
    }
    float Dv[Cdim<C>::V];
#pragma unroll
    for (int k = 0; k < C; ++k) Dv[k] = g.bt[k] * s.v[k];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      float acc = 0.0f;
#pragma unroll
      for (int k = 0; k < C; ++k) acc += K[a][k] * Dv[k];
      mu_c[a] += acc;
    }
    float X[3][3];   // K diag(bt) Sigma_qx
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k < C; ++k) acc += K[a][k] * g.bt[k] * g.Sxq[b][k];
        X[a][b] = acc;
      }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) Sc[a][b] -= 0.5f * (X[a][b] + X[b][a]);
  }
  s.oq = oq;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    s.mu_c[a] = mu_c[a];
#pragma unroll
    for (int b = 0; b < 3; ++b) s.Sc[a][b] = Sc[a][b];
  }
  // projection
  float p[3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
    p[a] = V.R[3 * a] * mu_c[0] + V.R[3 * a + 1] * mu_c[1] + V.R[3 * a + 2] * mu_c[2] + V.t[a];
#pragma unroll
  for (int a = 0; a < 3; ++a) s.p[a] = p[a];
  if (!(p[2] > float(kNear))) live = false;
  float z = p[2] > float(kNear) ? p[2] : 1.0f;
  float iz = 1.0f / z;
  float fx = V.fx, fy = V.fy;
  float J00 = fx * iz, J02 = -fx * p[0] * iz * iz;
  float J11 = fy * iz, J12 = -fy * p[1] * iz * iz;
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    s.Tm[0][b] = J00 * V.R[b] + J02 * V.R[6 + b];
    s.Tm[1][b] = J11 * V.R[3 + b] + J12 * V.R[6 + b];
  }
  float U[2][3];   // Tm Sc
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b)
      U[a][b] = s.Tm[a][0] * Sc[0][b] + s.Tm[a][1] * Sc[1][b] + s.Tm[a][2] * Sc[2][b];
  s.Sp00 = U[0][0] * s.Tm[0][0] + U[0][1] * s.Tm[0][1] + U[0][2] * s.Tm[0][2] + float(kDilation);
  s.Sp01 = U[0][0] * s.Tm[1][0] + U[0][1] * s.Tm[1][1] + U[0][2] * s.Tm[1][2];
  s.Sp11 = U[1][0] * s.Tm[1][0] + U[1][1] * s.Tm[1][1] + U[1][2] * s.Tm[1][2] + float(kDilation);
  float det = s.Sp00 * s.Sp11 - s.Sp01 * s.Sp01;
  if (!(det > 0.0f) || !(s.Sp00 > 0.0f) || !(s.Sp11 > 0.0f)) live = false;
  float idet = 1.0f / (det > 0.0f ? det : 1.0f);
  s.mx = fx * p[0] * iz + V.cx;
  s.my = fy * p[1] * iz + V.cy;
  s.ca = s.Sp11 * idet;
  s.cb = -s.Sp01 * idet;
  s.cc = s.Sp00 * idet;
  s.beta = 4.0f * float(s_exp(r.bx));
  if (!(oq >= float(kAlphaMin))) live = false;
  float oqs = oq >= float(kAlphaMin) ? oq : 1.0f;
  s.rho = float(s_rho(float((255) * oqs), float(s.beta)));
  if (!(s.rho > 0.0f)) live = false;
  s.live = live;
}

// Gradients w.r.t. the view-independent quantities, summed over views
// (accumulated in float32: each view's contribution is evaluated in T).
template <int C>
struct GeoGrad {
  float Sx[3][3];
  float Sxq[3][Cdim<C>::V];
  float Z[Cdim<C>::V][Cdim<C>::V];   // w.r.t. Sigma_q^-1 (symmetric part used)
  float Lh[Cdim<C>::V][Cdim<C>::V];  // w.r.t. chol(Sigma_q) (lower)
  float mu[3], muq[Cdim<C>::V], bq[Cdim<C>::V], bt[Cdim<C>::V];
  float bx, o, rgb[3];
};

template <int C>
__device__ __forceinline__ void geograd_zero(GeoGrad<C>& G) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
#pragma unroll
    for (int b = 0; b < 3; ++b) G.Sx[a][b] = 0.0f;
#pragma unroll
    for (int k = 0; k < C; ++k) G.Sxq[a][k] = 0.0f;
    G.mu[a] = 0.0f;
    G.rgb[a] = 0.0f;
  }
#pragma unroll
  for (int a = 0; a < C; ++a) {
#pragma unroll
    for (int b = 0; b < C; ++b) { G.Z[a][b] = 0.0f; G.Lh[a][b] = 0.0f; }
    G.muq[a] = G.bq[a] = G.bt[a] = 0.0f;
  }
  G.bx = G.o = 0.0f;
}

// Adjoint of view_forward for one view.  gr: d loss / d record fields
// (mx, my, a, b, c, o(q), beta, r, g, b).
template <int C, int ROT>
__device__ __forceinline__ void view_backward(const Raw<C, ROT>& r, const Geo<C, ROT>& g,
                                              const DevView& V, const ViewState<C>& s,
                                              const float* gr, GeoGrad<C>& G) {
  G.rgb[0] += gr[7];
  G.rgb[1] += gr[8];
  G.rgb[2] += gr[9];
  G.bx += gr[6] * s.beta;
  // conic = Sigma'^-1:  G_Sigma' = -A G_A A with G_A = [[ga, gb/2], [gb/2, gc]]
  float a = s.ca, b = s.cb, c = s.cc;
  float ga = gr[2], gb = 0.5f * gr[3], gc = gr[4];
  float P00 = a * ga + b * gb, P01 = a * gb + b * gc;   // A G_A
  float P10 = b * ga + c * gb, P11 = b * gb + c * gc;
  float G00 = -(P00 * a + P01 * b);
  float G01 = -(P00 * b + P01 * c);
  float G11 = -(P10 * b + P11 * c);
  // Sigma' = Tm Sc Tm^T + 0.3 I
  float Gs[2][2] = {{G00, G01}, {G01, G11}};
  float GT[2][3];   // Gs Tm
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) GT[i][j] = Gs[i][0] * s.Tm[0][j] + Gs[i][1] * s.Tm[1][j];
  float Gc[3][3];   // Tm^float Gs Tm
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) Gc[i][j] = s.Tm[0][i] * GT[0][j] + s.Tm[1][i] * GT[1][j];
  float GTm[2][3];  // 2 Gs Tm Sc
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      GTm[i][j] = 2.0f * (GT[i][0] * s.Sc[0][j] + GT[i][1] * s.Sc[1][j] + GT[i][2] * s.Sc[2][j]);
  // Tm = J W  ->  G_J = GTm W^T  (W row-major in V.R)
  float GJ00 = GTm[0][0] * V.R[0] + GTm[0][1] * V.R[1] + GTm[0][2] * V.R[2];
  float GJ02 = GTm[0][0] * V.R[6] + GTm[0][1] * V.R[7] + GTm[0][2] * V.R[8];
  float GJ11 = GTm[1][0] * V.R[3] + GTm[1][1] * V.R[4] + GTm[1][2] * V.R[5];
  float GJ12 = GTm[1][0] * V.R[6] + GTm[1][1] * V.R[7] + GTm[1][2] * V.R[8];
  float z = s.p[2];
  float iz = 1.0f / z, iz2 = iz * iz, iz3 = iz2 * iz;
  float fx = V.fx, fy = V.fy;
  float gmx = gr[0], gmy = gr[1];
  float gp[3];
  gp[0] = gmx * fx * iz + GJ02 * (-fx * iz2);
  gp[1] = gmy * fy * iz + GJ12 * (-fy * iz2);
  gp[2] = gmx * (-fx * s.p[0] * iz2) + gmy * (-fy * s.p[1] * iz2) + GJ00 * (-fx * iz2) +
          GJ02 * (2.0f * fx * s.p[0] * iz3) + GJ11 * (-fy * iz2) + GJ12 * (2.0f * fy * s.p[1] * iz3);
  float gmc[3];
#pragma unroll
  for (int j = 0; j < 3; ++j)
    gmc[j] = V.R[j] * gp[0] + V.R[3 + j] * gp[1] + V.R[6 + j] * gp[2];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    G.mu[i] += gmc[i];
#pragma unroll
    for (int j = 0; j < 3; ++j) G.Sx[i][j] += Gc[i][j];
  }
  float goq = gr[5];
  if constexpr (C == 0) {
    G.o += goq;
  } else {
    // ---- conditioning ----
    // Z = Sigma_q^-1 = Li^T Li
    float Z[Cdim<C>::V][Cdim<C>::V];
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
      for (int j = 0; j < C; ++j) {
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k < C; ++k) acc += g.Li[k][i] * g.Li[k][j];
        Z[i][j] = acc;
      }
    float Dv[Cdim<C>::V], ZDv[Cdim<C>::V], u[Cdim<C>::V], Zu[Cdim<C>::V];
#pragma unroll
    for (int k = 0; k < C; ++k) Dv[k] = g.bt[k] * s.v[k];
#pragma unroll
    for (int k = 0; k < C; ++k) {
      float acc = 0.0f, acc2 = 0.0f;
#pragma unroll
      for (int m = 0; m < C; ++m) acc += Z[k][m] * Dv[m];
      ZDv[k] = acc;
#pragma unroll
      for (int m = 0; m < 3; ++m) acc2 += g.Sxq[m][k] * gmc[m];
      u[k] = acc2;
    }
#pragma unroll
    for (int k = 0; k < C; ++k) {
      float acc = 0.0f;
#pragma unroll
      for (int m = 0; m < C; ++m) acc += Z[k][m] * u[m];
      Zu[k] = acc;
    }
    // Q = Sxq^float G Sxq ; GS = G Sxq
    float GS[3][Cdim<C>::V];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int k = 0; k < C; ++k)
        GS[i][k] = Gc[i][0] * g.Sxq[0][k] + Gc[i][1] * g.Sxq[1][k] + Gc[i][2] * g.Sxq[2][k];
    float Q[Cdim<C>::V][Cdim<C>::V];
#pragma unroll
    for (int k = 0; k < C; ++k)
#pragma unroll
      for (int l = 0; l < C; ++l)
        Q[k][l] = g.Sxq[0][k] * GS[0][l] + g.Sxq[1][k] * GS[1][l] + g.Sxq[2][k] * GS[2][l];
    // G_Sxq += gmc (Z Dv)^T - G Sxq (Z D + D Z)
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int l = 0; l < C; ++l) {
        float acc = gmc[i] * ZDv[l];
#pragma unroll
        for (int k = 0; k < C; ++k) acc -= GS[i][k] * (Z[k][l] * g.bt[l] + g.bt[k] * Z[k][l]);
        G.Sxq[i][l] += acc;
      }
    // G_Z += sym(u Dv^T) - (Q D + D Q)/2
#pragma unroll
    for (int k = 0; k < C; ++k)
#pragma unroll
      for (int l = 0; l < C; ++l)
        G.Z[k][l] += 0.5f * (u[k] * Dv[l] + Dv[k] * u[l]) - 0.5f * (Q[k][l] * g.bt[l] + g.bt[k] * Q[k][l]);
    // d bt_k += (Z u)_k v_k - (Z Q)_kk ;  g_v += bt (Z u)
    float gv[Cdim<C>::V];
#pragma unroll
    for (int k = 0; k < C; ++k) {
      float zq = 0.0f;
#pragma unroll
      for (int m = 0; m < C; ++m) zq += Z[k][m] * Q[m][k];
      G.bt[k] += Zu[k] * s.v[k] - zq;
      gv[k] = g.bt[k] * Zu[k];
    }
    // ---- opacity ----  o(q) = o exp(sum e_i ell_i),  ell = log(1 - tanh(w^2))
    float prod;
    {
      float lsum = 0.0f;
#pragma unroll
      for (int i = 0; i < C; ++i) lsum += g.e[i] * s.ell[i];
      prod = float(s_exp(float(lsum)));
    }
    G.o += goq * prod;
    float gw[Cdim<C>::V];
#pragma unroll
    for (int i = 0; i < C; ++i) {
      if (g.beta_opacity) {
        G.bq[i] += goq * s.oq * s.ell[i] * g.e[i];
        float x = s.w[i] * s.w[i];
        float th = float(tanhf(float(x)));
        gw[i] = goq * s.oq * g.e[i] * (-(1.0f + th)) * 2.0f * s.w[i];
      } else {
        gw[i] = -goq * s.oq * s.w[i];   // d(-w^2/2)/dw; no b_q dependence
      }
    }
    // w = Li v:  g_v += Li^T gw ; G_Lh += -tril((Li^T gw) w^T)
    float ut[Cdim<C>::V];
#pragma unroll
    for (int k = 0; k < C; ++k) {
      float acc = 0.0f;
#pragma unroll
      for (int i = k; i < C; ++i) acc += g.Li[i][k] * gw[i];
      ut[k] = acc;
      gv[k] += acc;
    }
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
      for (int j = 0; j <= i; ++j) G.Lh[i][j] -= ut[i] * s.w[j];
    // v = q - mu_q ; q = [t, d] or d ; d = unit(mu_x - cam)
#pragma unroll
    for (int k = 0; k < C; ++k) G.muq[k] -= gv[k];
    float gd[3] = {0.0f, 0.0f, 0.0f};
    if constexpr (C >= 4) { gd[0] = gv[1]; gd[1] = gv[2]; gd[2] = gv[3]; }
    else if constexpr (C == 3) { gd[0] = gv[0]; gd[1] = gv[1]; gd[2] = gv[2]; }
    else {
#pragma unroll
      for (int k = 0; k < C; ++k) gd[k] = gv[k];
    }
    float dg = s.dir[0] * gd[0] + s.dir[1] * gd[1] + s.dir[2] * gd[2];
    float idist = 1.0f / s.dist;
#pragma unroll
    for (int k = 0; k < 3; ++k) G.mu[k] += (gd[k] - s.dir[k] * dg) * idist;
  }
}

// Final chain from the view-independent gradients to the raw parameters.
// out[] is indexed by parameter row.
template <int C, int ROT>
__device__ __forceinline__ void geo_backward(const Raw<C, ROT>& r, const Geo<C, ROT>& g,
                                             const GeoGrad<C>& G, float* out) {
  const ParamRows pr = param_rows(C, ROT);
  float GM[3][3];
  // Sigma_x = M M^T (G_Sx symmetric): G_M = 2 G_Sx M
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      GM[i][j] = (G.Sx[i][0] + G.Sx[0][i]) * g.M[0][j] + (G.Sx[i][1] + G.Sx[1][i]) * g.M[1][j] +
                 (G.Sx[i][2] + G.Sx[2][i]) * g.M[2][j];
  if constexpr (C > 0) {
    float Z[Cdim<C>::V][Cdim<C>::V];
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
      for (int j = 0; j < C; ++j) {
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k < C; ++k) acc += g.Li[k][i] * g.Li[k][j];
        Z[i][j] = acc;
      }
    // G_Sq = -Z sym(G_Z) Z + sym(Li^T Phi(Lh^float G_Lh) Li)
    float GSq[Cdim<C>::V][Cdim<C>::V];
    {
      float A1[Cdim<C>::V][Cdim<C>::V];
#pragma unroll
      for (int i = 0; i < C; ++i)
#pragma unroll
        for (int j = 0; j < C; ++j) {
          float acc = 0.0f;
#pragma unroll
          for (int k = 0; k < C; ++k) acc += Z[i][k] * 0.5f * (G.Z[k][j] + G.Z[j][k]);
          A1[i][j] = acc;
        }
#pragma unroll
      for (int i = 0; i < C; ++i)
#pragma unroll
        for (int j = 0; j < C; ++j) {
          float acc = 0.0f;
#pragma unroll
          for (int k = 0; k < C; ++k) acc += A1[i][k] * Z[k][j];
          GSq[i][j] = -acc;
        }
      float Pm[Cdim<C>::V][Cdim<C>::V];   // Phi(Lh^float G_Lh)
#pragma unroll
      for (int i = 0; i < C; ++i)
#pragma unroll
        for (int j = 0; j < C; ++j) {
          if (j > i) { Pm[i][j] = 0.0f; continue; }
          float acc = 0.0f;
#pragma unroll
          for (int k = 0; k < C; ++k) acc += g.Lh[k][i] * G.Lh[k][j];
          Pm[i][j] = (i == j) ? 0.5f * acc : acc;
        }
      float B1[Cdim<C>::V][Cdim<C>::V];   // Li^T Pm
#pragma unroll
      for (int i = 0; i < C; ++i)
#pragma unroll
        for (int j = 0; j < C; ++j) {
          float acc = 0.0f;
#pragma unroll
          for (int k = 0; k < C; ++k) acc += g.Li[k][i] * Pm[k][j];
          B1[i][j] = acc;
        }
      float S1[Cdim<C>::V][Cdim<C>::V];   // B1 Li
#pragma unroll
      for (int i = 0; i < C; ++i)
#pragma unroll
        for (int j = 0; j < C; ++j) {
          float acc = 0.0f;
#pragma unroll
          for (int k = 0; k < C; ++k) acc += B1[i][k] * g.Li[k][j];
          S1[i][j] = acc;
        }
#pragma unroll
      for (int i = 0; i < C; ++i)
#pragma unroll
        for (int j = 0; j < C; ++j) GSq[i][j] += 0.5f * (S1[i][j] + S1[j][i]);
    }
    // Sigma_q = Lqx Lqx^T + Lq Lq^T ; Sigma_xq = M Lqx^T
    float GSs[Cdim<C>::V][Cdim<C>::V];   // G_Sq + G_Sq^T
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
      for (int j = 0; j < C; ++j) GSs[i][j] = GSq[i][j] + GSq[j][i];
#pragma unroll
    for (int k = 0; k < C; ++k)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        float acc = 0.0f;
#pragma unroll
        for (int m = 0; m < C; ++m) acc += GSs[k][m] * r.lqx[m][j];
#pragma unroll
        for (int m = 0; m < 3; ++m) acc += G.Sxq[m][k] * g.M[m][j];
        out[pr.lqx + 3 * k + j] = float(acc);
      }
    int idx = 0;
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
      for (int j = 0; j <= i; ++j) {
        float acc = 0.0f;
#pragma unroll
        for (int m = j; m < C; ++m) acc += GSs[i][m] * lq_entry<C, ROT>(r, m, j);
        out[pr.lq + idx] = float(i == j ? acc * lq_entry<C, ROT>(r, i, i) : acc);
        ++idx;
      }
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k < C; ++k) acc += G.Sxq[i][k] * r.lqx[k][j];
        GM[i][j] += acc;
      }
#pragma unroll
    for (int k = 0; k < C; ++k) {
      out[pr.mu_q + k] = float(G.muq[k]);
      float gbq = G.bq[k];
      if (g.beta_cond && r.bq[k] < 0.0f) gbq += G.bt[k] * g.bt[k];
      out[pr.b_q + k] = float(gbq);
    }
  }
  // M = R diag(s)
  float GR[3][3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    float acc = 0.0f;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      GR[i][j] = GM[i][j] * g.s[j];
      acc += GM[i][j] * g.M[i][j];   // M = R diag(s): d/d log s_j = sum_i GM_ij R_ij s_j
    }
    out[pr.log_s + j] = float(acc);
  }
  if (ROT == UBS_ROT_QUAT) {
    float iq = rsqrtf(r.rq[0] * r.rq[0] + r.rq[1] * r.rq[1] +
                      r.rq[2] * r.rq[2] + r.rq[3] * r.rq[3]);
    float w = r.rq[0] * iq, x = r.rq[1] * iq, y = r.rq[2] * iq, z = r.rq[3] * iq;
    float gw = 2.0f * (-z * GR[0][1] + y * GR[0][2] + z * GR[1][0] - x * GR[1][2] - y * GR[2][0] + x * GR[2][1]);
    float gx = 2.0f * (y * GR[0][1] + z * GR[0][2] + y * GR[1][0] - 2.0f * x * GR[1][1] - w * GR[1][2] +
                   z * GR[2][0] + w * GR[2][1] - 2.0f * x * GR[2][2]);
    float gy = 2.0f * (-2.0f * y * GR[0][0] + x * GR[0][1] + w * GR[0][2] + x * GR[1][0] + z * GR[1][2] -
                   w * GR[2][0] + z * GR[2][1] - 2.0f * y * GR[2][2]);
    float gz = 2.0f * (-2.0f * z * GR[0][0] - w * GR[0][1] + x * GR[0][2] + w * GR[1][0] - 2.0f * z * GR[1][1] +
                   y * GR[1][2] + x * GR[2][0] + y * GR[2][1]);
    float dotq = w * gw + x * gx + y * gy + z * gz;
    out[pr.rot + 0] = float((gw - w * dotq) * iq);
    out[pr.rot + 1] = float((gx - x * dotq) * iq);
    out[pr.rot + 2] = float((gy - y * dotq) * iq);
    out[pr.rot + 3] = float((gz - z * dotq) * iq);
  } else {
    out[pr.rot + 0] = float(GR[2][1] - GR[1][2]);
    out[pr.rot + 1] = float(GR[0][2] - GR[2][0]);
    out[pr.rot + 2] = float(GR[1][0] - GR[0][1]);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    out[pr.mu_x + k] = float(G.mu[k]);
    out[pr.rgb + k] = float(G.rgb[k]);
  }
  out[pr.b_x] = float(G.bx);
  out[pr.o] = float(G.o);
}

}  // namespace f32
}  // namespace ubs
