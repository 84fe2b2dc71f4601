"""The FP64 node arithmetic of the device code, compiled for the host: its own
logarithm, exponential and quotient, and the collision, against 80-bit values.

The section of hlbm_device.hpp from its helpers to the row sweep holds nothing
but arithmetic.  The hardware's builtins become host functions (the reciprocal
seed is cut to 22 bits, fewer than the hardware gives) and the two lines of
assembly, a zero and a fused multiply-add, what they stand for."""
import ctypes
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2002_03644_amd", "csrc", "hlbm_device.hpp")

PRELUDE = r"""
#include <math.h>
#include <stdint.h>
#include <string.h>
#define __device__
#define __forceinline__ inline
#define __builtin_nontemporal_store(v, p) (*(p) = (v))
#define __builtin_bit_cast(T, x) bits_as<T>(x)
template <class T, class U> static inline T bits_as(U u) { T t; memcpy(&t, &u, sizeof t); return t; }
static inline double seed_rcp(double x) {
  double r = 1.0 / x;
  uint64_t b; memcpy(&b, &r, 8); b &= ~((1ull << 30) - 1); memcpy(&r, &b, 8);
  return r;
}
static inline double mant(double x) { int e; return frexp(x, &e); }
static inline int expo(double x) { int e; frexp(x, &e); return e; }
#define __builtin_amdgcn_rcp seed_rcp
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_logf log2f
#define __builtin_amdgcn_frexp_mant mant
#define __builtin_amdgcn_frexp_exp expo
#define __builtin_amdgcn_ldexp ldexp
#define __expf expf
#define __logf logf
#define HLBM_IS_F32 0
using real = double;
constexpr int kQ = 9, kPlanes = 10;
constexpr int kFlagPhiFD = 1, kFlagE1Centred = 2, kFlagE2Off = 4, kFlagPreciseTheta = 8,
              kFlagFeq3 = 16;
"""

HARNESS = r"""
typedef long double ld;
// units in the last place of the 80-bit value, rounded to double
static double ulps(double got, ld want) {
  int e; frexpl(want, &e);
  return (double)(fabsl(got - want) / ldexpl(1.0L, e - 53));
}
extern "C" void math_errors(const double *x, int n, double *out) {  // log, exp, exp - 1, quotient
  for (int k = 0; k < 4; ++k) out[k] = 0;
  for (int i = 0; i < n; ++i) {
    const double a = x[i], b = x[n + i], y = x[2 * n + i];
    out[0] = fmax(out[0], a == 1.0 ? fabs(log_near(a, 0)) : ulps(log_near(a, 0), logl(a)));
    out[1] = fmax(out[1], ulps(exp_near(y, 0.0, 0), expl(y)));
    if (fabs(y) < 0.3 && y != 0.0) out[2] = fmax(out[2], ulps(exp_near(y, 1.0, 0), expm1l(y)));
    out[3] = fmax(out[3], ulps(div_fast(a, b), (ld)a / b));
  }
}
// Post-collision populations of n nodes: `fast` as the device forms them, `want`
// in type R as the method writes them down (moments, closure, stress), in 64 bits
// through the projection of the nine coefficients that the device code holds.
template <class R>
static void plain(const DomainArgs &d, const double *o, const double *v, R (&f)[9]) {
  const R one = 1, cs2 = one / 3, r = o[0], u = o[1], w = o[2], t = o[3], pxx = o[4], pyy = o[5],
          pxy = o[6], sg = d.sigma, mu = d.mu;
  const R dxux = ((R)v[0] - v[1]) / 2, dyux = ((R)v[2] - v[3]) / 2, dxuy = ((R)v[4] - v[5]) / 2,
          dyuy = ((R)v[6] - v[7]) / 2;
  const R Ex = (u > 0 ? (R)v[9] - v[10] : (R)v[8] - v[9]), Ey = (w > 0 ? (R)v[12] - v[13] : (R)v[11] - v[12]);
  const R p = r * cs2 * t, e2 = p * (R)d.e2c * (dxux + dyuy), X = Ex + e2, Y = Ey + e2;
  const R tp = mu + p / 2, keep = one - p / tp;
  const R fxx = -tp * (dxux - dyuy), fxy = -tp * (dyux + dxuy);
  const R axx = keep * (sg * (pxx - p - r * u * u + X / 2) + (one - sg) * fxx);
  const R ayy = keep * (sg * (pyy - p - r * w * w + Y / 2) - (one - sg) * fxx);
  const R axy = keep * (sg * (pxy - r * u * w) + (one - sg) * fxy);
  const R c = cs2 * (t - one), bxxy = w * axx + 2 * u * axy, bxyy = u * ayy + 2 * w * axy;
  const R Axx = r * u * u + r * c + axx + X / 2, Ayy = r * w * w + r * c + ayy + Y / 2;
  const R Axy = r * u * w + axy, Axxy = r * u * u * w + r * c * w + bxxy;
  const R Axyy = r * u * w * w + r * c * u + bxyy;
  const R A4 = r * u * u * w * w + r * c * (u * u + w * w) + r * c * c + 2 * (u * bxyy + w * bxxy) +
               (c - u * u) * ayy + (c - w * w) * axx - 4 * u * w * axy;
  if constexpr (sizeof(R) == sizeof(double)) {
    project(r, r * u, r * w, Axx, Axy, Ayy, Axxy, Axyy, A4, f);
    return;
  }
  const int cx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1}, cy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
  for (int k = 0; k < 9; ++k) {
    const int n = abs(cx[k]) + abs(cy[k]);
    const R wt = n == 0 ? (R)4 / 9 : n == 1 ? one / 9 : one / 36;
    const R hx = cx[k] * cx[k] - cs2, hy = cy[k] * cy[k] - cs2;
    f[k] = wt * (r + 3 * (cx[k] * r * u + cy[k] * r * w) + (R)4.5 * (hx * Axx + hy * Ayy) +
                 9 * cx[k] * cy[k] * Axy + (R)13.5 * (cx[k] * hy * Axyy + cy[k] * hx * Axxy) +
                 (R)20.25 * hx * hy * A4);
  }
}
extern "C" void collisions(double mu, double sigma, int n, const double *nodes, const double *nbs,
                           double *fast, double *in64, ld *in80) {
  DomainArgs d;
  memset(&d, 0, sizeof d);
  d.mu = mu; d.sigma = sigma; d.sigma1 = 1.0 - sigma; d.half_mu = mu * 0.5;
  d.e2c = 0.6; d.e2h = 0.3; d.e2k = 0.6 * kCs2 / 4.0; d.k4 = 2.25; d.theta_ref = 1.0;
  for (int i = 0; i < n; ++i) {
    const double *o = nodes + 7 * i, *v = nbs + 14 * i;
    const NodeState s{o[0], o[1], o[2], o[3], o[4], o[5], o[6]};
    const NodeStencil t{v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10], v[11],
                        v[12], v[13]};
    double f[9], phi, pt;
    collide(d, s, t, d.sigma, d.sigma1, f, phi, pt);
    ld g[9];
    for (int k = 0; k < 9; ++k) fast[9 * i + k] = f[k];
    plain<double>(d, o, v, f);
    plain<ld>(d, o, v, g);
    for (int k = 0; k < 9; ++k) in64[9 * i + k] = f[k], in80[9 * i + k] = g[k];
  }
}
"""


@pytest.fixture(scope="module")
def node(tmp_path_factory):
    if np.finfo(np.longdouble).nmant < 63 or not shutil.which("g++"):
        pytest.skip("needs g++ and 80-bit long doubles")
    s = open(SRC).read()
    args = s[s.index("struct DomainArgs {"):s.index("// State offset")]
    a = re.search(r"// -+ helpers\n", s).end()
    body = s[a:re.search(r"// -+ the step\n", s).start()]
    body = re.sub(r'asm volatile\("s_mov_b32[^;]*;', "zero = 0;", body)
    body = re.sub(r'asm\("v_fma_f64[^;]*;', "r = __builtin_fma(a, b, near_const(c, zero));", body)
    assert "asm" not in re.sub(r"//.*", "", body)
    d = tmp_path_factory.mktemp("node")
    src, so = str(d / "node.cpp"), str(d / "node.so")
    with open(src, "w") as f:
        f.write(PRELUDE + args + body + HARNESS)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-mfma", "-ffp-contract=off", "-shared",
                           "-fPIC", "-w", src, "-o", so])
    return ctypes.CDLL(so)


def test_logarithm_exponential_and_quotient(node):
    """Units in the last place over densities e^-8 .. e^8, close to 1 and around
    the ends of the reduced range, and arguments of the exponential in -8 .. 8.
    Bounds: the roundings of the last operations, see the functions."""
    g = np.random.default_rng(0)
    n = 400000
    x = np.exp(g.uniform(-8, 8, n))
    x[:n // 4] = 1 + g.uniform(-1, 1, n // 4) * 2.0 ** g.uniform(-50, -2, n // 4)
    edge = np.sqrt(0.5) * 2.0 ** g.integers(-3, 4, n // 8)
    x[n // 4:n // 4 + n // 8] = edge * (1 + g.integers(-8, 9, n // 8) * 2.0 ** -52)
    x[-1] = 1.0
    y = g.uniform(-8, 8, n)
    y[:n // 2] = g.uniform(-0.4, 0.4, n // 2)
    arg = np.concatenate([x, g.permutation(x), y])
    out = (ctypes.c_double * 4)()
    node.math_errors(arg.ctypes.data_as(ctypes.c_void_p), n, out)
    log, exp, expm1, quotient = out[:]
    assert log < 1.2, log
    assert exp < 1.1, exp
    assert expm1 < 1.2, expm1
    assert quotient < 0.51, quotient


@pytest.mark.parametrize("sigma", [0.0, 0.3, 1.0])
@pytest.mark.parametrize("mu", [1.5e-6, 1e-3])
def test_collision_rounds_no_more_than_the_formulas(node, mu, sigma):
    """RMS rounding of the populations and of the momentum they carry, against the
    same collision in 80 bits: no larger than that of the formulas evaluated as
    they stand in 64."""
    g = np.random.default_rng(1)
    n = 100000
    rho, th = g.uniform(0.8, 1.2, n), g.uniform(0.17, 0.23, n)
    u, v = g.uniform(-0.2, 0.2, (2, n))
    near = lambda a, s: a[:, None] + s * g.normal(size=(n, 4))  # noqa: E731
    ux, uy = near(u, 1e-3), near(v, 1e-3)
    gam = rho * u * (1 - th - u * u), rho * v * (1 - th - v * v)
    gx, gy = near(gam[0], 1e-3)[:, :3], near(gam[1], 1e-3)[:, :3]
    gx[:, 1], gy[:, 1] = gam
    p = rho * th / 3
    neq = 1e-4 * g.normal(size=(3, n))
    nodes = np.ascontiguousarray(np.stack([rho, u, v, th, p + rho * u * u + neq[0],
                                           p + rho * v * v + neq[1], rho * u * v + neq[2]], 1))
    nbs = np.ascontiguousarray(np.concatenate([ux, uy, gx, gy], 1))
    fast, in64, in80 = np.empty((n, 9)), np.empty((n, 9)), np.empty((n, 9), np.longdouble)
    node.collisions(ctypes.c_double(mu), ctypes.c_double(sigma), n,
                    *(a.ctypes.data_as(ctypes.c_void_p) for a in (nodes, nbs, fast, in64, in80)))
    cx, cy = np.array([0, 1, 0, -1, 0, 1, -1, -1, 1]), np.array([0, 0, 1, 0, -1, 1, 1, -1, -1])

    def rms(a):
        e = a - in80
        # per-population rounding along the axes, diagonals and at rest; momentum of
        # independently rounded populations (they part at the next streaming)
        k = [np.sqrt((e[:, q] ** 2).mean()) for q in range(9)]
        return [np.sqrt(sum(float(k[q]) ** 2 * c[q] ** 2 for q in range(9))) for c in (cx, cy)] + [
            float(np.sqrt((e ** 2).mean()))]

    for a, b in zip(rms(fast), rms(in64)):
        assert a <= b, (a / b)
