"""The per-primitive adjoint's mathematics (``csrc/prim_math.hpp``), compiled
for the host, against float64: the polynomials that replace library functions
stay within the bounds their comments state, and the parameter gradients are
off float64 autograd of the oracle by no more than the float32 sums they are
kept in account for.

Bars of the gradients (relative L2 error of a block).  The error of sums over
views that are rounded to float32 once per view, each exact contribution added
before the rounding, is formed here from the oracle's contributions (2.5e-8 for
one view).  mu_x, mu_q and rgb are such sums: their bar is that error (5 % for
ties).  In quadrature with it, b_x has the rounding of beta (3e-8), and o the
error of log1p's polynomial times the exponents (4.6e-10 times up to 100).  The
last step adds rounded parts to others: one rounding more is sqrt 2 times the
error, two sqrt 3.  Rotations and log scales have none from one view (G_Sc and
G_A are float64 there), one from several; L_qx, L_q and b_q one, and two."""
import os
import subprocess

import numpy as np
import pytest
import torch

from oracle import preprocess as opp
from paper_2510_03312_amd import build as hip_build
from synth.scenes import SceneSpec, look_at_view

HARNESS = r'''
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>
// the device functions as host functions, the hardware's instructions by their meaning
#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
static inline float host_med3(float x, float lo, float hi) { return fminf(fmaxf(x, lo), hi); }
static inline double host_rcp(double x) { return double(float(1.0 / x)); }   // to 2^-24
#define __builtin_amdgcn_fmed3f host_med3
#define __builtin_amdgcn_rcp host_rcp
#define isfinite(x) __builtin_isfinite(x)
__attribute__((host)) static inline double rsqrt(double x) { return 1.0 / sqrt(x); }
#include "prim_math.hpp"
using namespace ubs;

static std::vector<float> read_floats(const char* path) {
  std::vector<float> v;
  FILE* f = fopen(path, "rb");
  fseek(f, 0, SEEK_END);
  v.resize(size_t(ftell(f)) / 4);
  rewind(f);
  if (fread(v.data(), 4, v.size(), f) != v.size()) exit(2);
  fclose(f);
  return v;
}

template <int C, int ROT, bool ONE_VIEW>
static void gradients(const char* in, const char* out, size_t n, int n_views) {
  const std::vector<float> d = read_floats(in);
  constexpr int F = param_rows(C, ROT).F;
  const float* par = d.data();
  const float* vw = par + F * n;
  const float* gr = vw + 23 * n_views;   // [view][primitive][10]
  std::vector<float> res(F * n);
  std::vector<DevView> views(n_views);
  for (int v = 0; v < n_views; ++v) memcpy(&views[v], vw + 23 * v, 23 * 4);
  for (size_t i = 0; i < n; ++i) {
    Raw<C, ROT> r;
    load_raw<C, ROT>(par, int64_t(n), int64_t(i), r);
    Geo<double, C, ROT> g;
    geo_forward<double, C, ROT>(r, g, 0u);
    static GradSums<C, 1, ONE_VIEW> sums;
    sums.clear(0);
    for (int v = 0; v < n_views; ++v) {
      const float* q = gr + (size_t(v) * n + i) * 10;
      ViewState<double, C> s;
      view_forward<double, C, ROT, true>(r, g, views[v], s);
      view_backward<double, C, ROT>(g, views[v], s, q, [&](int k, double x) { sums.add(k, x, 0); });
    }
    geo_backward<double, C, ROT>(r, g, [&](int k) { return sums.get(k, 0); },
                                 [&](int k, double x) { res[size_t(k) * n + i] = float(x); });
  }
  FILE* f = fopen(out, "wb");
  fwrite(res.data(), 4, res.size(), f);
  fclose(f);
}

int main(int argc, char** argv) {
  if (!strcmp(argv[1], "poly")) {
    double e_exp = 0, e_neg = 0, r_log = 0, a_log = 0, e_tanh = 0;
    for (int k = 0; k <= 400000; ++k) {
      const float x = -87.0f + 174.0f * float(k) / 400000.0f;
      e_exp = fmax(e_exp, fabs(m_exp<double>(x) / exp(double(x)) - 1.0));
      const double y = -700.0 * k / 400000.0;
      e_neg = fmax(e_neg, fabs(s_exp_neg(y) / exp(y) - 1.0));
      const double t = (k + 0.0) / 400000.0, l = log1p(t);
      a_log = fmax(a_log, fabs(s_log1p_unit(t) - l));
      if (t > 0) r_log = fmax(r_log, fabs(s_log1p_unit(t) / l - 1.0));
      e_tanh = fmax(e_tanh, fabs(s_half_tanh(t) * (1.0 + t) - 1.0));
    }
    r_log = fmax(r_log, fabs(s_log1p_unit(1e-12) / log1p(1e-12) - 1.0));
    printf("%.17g %.17g %.17g %.17g %.17g\n", e_exp, e_neg, r_log, a_log, e_tanh);
    return 0;
  }
  const int dim = atoi(argv[1]), rot = atoi(argv[2]);
  const size_t n = size_t(atoll(argv[5]));
  const int nv = atoi(argv[6]);
#define RUN(C, ROT) (nv == 1 ? gradients<C, ROT, true> : gradients<C, ROT, false>)(argv[3], argv[4], n, nv)
  if (dim == 3 && rot == 0) RUN(0, 0);
  else if (dim == 6 && rot == 1) RUN(3, 1);
  else if (dim == 7 && rot == 0) RUN(4, 0);
  else if (dim == 10 && rot == 0) RUN(7, 0);
  else return 3;
  return 0;
}
'''

GRAD_COLS = [0, 1, 2, 3, 4, 6, 7, 8, 9, 10]   # record fields with a gradient, in its order


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    if not os.path.exists(hip_build.HIPCC):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("primmath")
    src = d / "prim.hip"
    src.write_text(HARNESS)
    exe = d / "prim"
    subprocess.run([hip_build.HIPCC, *hip_build.FLAGS, "--cuda-host-only", "-w", str(src), "-o",
                    str(exe)], check=True, capture_output=True)
    return str(exe), d


def test_polynomials_stay_within_their_bounds(harness):
    out = subprocess.run([harness[0], "poly"], check=True, capture_output=True, text=True).stdout
    e_exp, e_neg, r_log, a_log, e_tanh = (float(x) for x in out.split())
    print(out)
    assert e_exp <= 2.3e-16                     # an ulp
    assert e_neg <= 2.3e-10 and r_log <= 8.5e-10 and a_log <= 4.6e-10 and e_tanh <= 1e-14


def _case(dim, rot, n, n_views):
    """Primitives of ordinary shape and orientation in front of every view."""
    rng, sl = np.random.default_rng(5), opp.field_slices(dim, rot)
    p = 0.4 * rng.normal(size=(sl["_F"].stop, n))
    p[sl["mu_x"]] = rng.uniform(-1.0, 1.0, (3, n))
    p[sl["rot"]] = rng.normal(size=p[sl["rot"]].shape) * (0.3 if rot else 1.0)
    p[sl["log_s_x"]] = rng.normal(size=(3, n)) / 2 - 1.5
    p[sl["b_q"]] -= 0.7
    p[sl["o"]], p[sl["rgb"]] = rng.uniform(0.1, 1.0, (1, n)), rng.uniform(size=(3, n))
    sc = SceneSpec(dim, rot, p.astype(np.float32))
    views = [look_at_view((4 * np.sin(a), 0.3, -4 * np.cos(a)), 640, 480, time=k / max(1, n_views - 1))
             for k, a in enumerate(np.linspace(0.0, 1.0, n_views))]
    P = torch.tensor(sc.params.astype(np.float64), requires_grad=True)
    # each view's contribution in float64, for the records that view keeps
    gr = rng.normal(size=(n_views, n, 10)).astype(np.float32)
    parts = np.zeros((n_views,) + sc.params.shape)
    for v, view in enumerate(views):
        out = opp.preprocess(P, dim, rot, view)
        gr[v, ~out["valid"].numpy()] = 0.0
        rec = out["rec"][:, GRAD_COLS]
        g, = torch.autograd.grad(rec, P, torch.tensor(gr[v].astype(np.float64)))
        parts[v] = g.numpy()
    parts = np.nan_to_num(parts)
    return sc, views, gr, parts


def _run(harness, sc, views, gr):
    exe, d = harness
    vw = []
    for v in views:
        R, t = np.asarray(v.R, np.float32), np.asarray(v.t, np.float32)
        cam = -(R.astype(np.float64).T @ t.astype(np.float64))
        vw.append(np.concatenate([R.ravel(), t, cam, [v.fx, v.fy, v.cx, v.cy, v.time], v.query]))
    np.concatenate([sc.params.ravel(), np.concatenate(vw), gr.ravel()]).astype(np.float32).tofile(
        d / "in.bin")
    subprocess.run([exe, str(sc.dim), str(sc.rot), str(d / "in.bin"), str(d / "out.bin"), str(sc.n),
                    str(len(views))], check=True)
    return np.fromfile(d / "out.bin", dtype=np.float32).reshape(sc.params.shape).astype(np.float64)


@pytest.mark.parametrize("dim,rot,n_views", [(3, 0, 1), (6, 1, 1), (7, 0, 1), (10, 0, 1), (3, 0, 8),
                                             (6, 1, 8), (7, 0, 2), (7, 0, 8), (10, 0, 8)])
def test_gradients_against_float64(harness, dim, rot, n_views):
    sc, views, gr, parts = _case(dim, rot, 20000, n_views)
    got, ref = _run(harness, sc, views, gr), parts.sum(0)
    rounded = np.zeros(sc.params.shape, np.float32)
    for p in parts:
        rounded = (rounded.astype(np.float64) + p).astype(np.float32)
    err = lambda a, s: float(np.linalg.norm((a - ref)[s]) / np.linalg.norm(ref[s]))  # noqa: E731
    report, bad = [], []
    for name, s in opp.field_slices(dim, rot).items():
        if name == "_F" or s.stop <= s.start:
            continue
        e, sums = err(got, s), err(rounded, s)
        more = {"mu_x": 0, "mu_q": 0, "rgb": 0, "b_x": 0, "o": 0, "rot": n_views > 1,
                "log_s_x": n_views > 1, "L_qx": 1 + (n_views > 1), "L_q": 1 + (n_views > 1), "b_q": 1 + (n_views > 1)}
        apart = {"b_x": 3e-8, "o": 4.6e-8 if dim > 3 else 0.0}.get(name, 0.0)
        bar = 1.05 * np.hypot(sums * np.sqrt(1.0 + more[name]), apart)
        report.append(f"{name} {e:.2e} (sums {sums:.2e})")
        if e > bar:
            bad.append((name, e, bar))
    print(f"dim {dim} rot {rot} views {n_views}: " + ", ".join(report))
    assert not bad, bad
