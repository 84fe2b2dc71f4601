"""The FP64 node arithmetic of the device code, compiled for the host: its own
logarithm, exponential and quotient against 80-bit values.

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
