// Device code of the D2Q9 hybrid LBM step for gfx950 (MI355X).
//
// Included by the per-precision translation units (hlbm_kernels_f32.hip,
// hlbm_kernels_f64.hip) with HLBM_REAL defined.  The arithmetic follows the
// HLBM of arXiv 2002.03644 in moment (Hermite-coefficient) space:
//   - moments rho, rho u, Pi from the populations (Eqs. rhoalgo, ualgo);
//   - theta from the entropy closure (Eq. Entropie expression), p = rho c_s^2
//     theta (Eq. perfect gas), local tau = mu / p, taubar = tau + 1/2 (Sec. 3.1);
//   - lattice-closure correction E1 = d_a(rho u_a (1 - theta - u_a^2)) by the
//     upwind difference of Sec. 3.2 (sgn(u) = 0, i.e. centred, for |u| within
//     the rounding band sgn_eps), E2 = p (2 - gamma) div u (Eq. E2 corr term);
//   - HRR stress a1 = sigma a1PR + (1 - sigma) a1FD (Eq. a1sigalgo), with a1PR in
//     closed form (the projection of F - f^eq + psi/2 on H_ab) and a1FD from
//     centred velocity gradients (Eq. a1FD), and the recursion to xxy, yyx,
//     xxyy (Sec. 3.3);
//   - post-collision populations f* = f^eq + (1 - 1/taubar) f^1 + psi/2
//     (Eq. streamalgo) as one projection of nine Hermite coefficients;
//   - pull streaming F'_i(x) = f*_i(x - c_i);
//   - entropy update (Eq. sequaalgo): upwind MUSCL with the van Albada slope,
//     5-point Fourier term, viscous heat Phi (Eq. viscous heat discret or the
//     finite-difference form), explicit Euler.
//
// Data layout in HBM: ten planes [p][ny][nx] (x fastest), p = 0..8 the
// populations and p = 9 the entropy; two such buffers are ping-ponged.  In
// the FP32 form the planes hold deviations g_i = F_i - f^eq_i(rho_ref, 0,
// theta_ref) and ds = s - s_ref, which keeps the small fluctuations that
// drive the dynamics out of the rounding of the O(1) rest state.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#if !defined(HLBM_REAL) || !defined(HLBM_NS) || !defined(HLBM_IS_F32)
#error "define HLBM_REAL, HLBM_NS and HLBM_IS_F32 before including hlbm_device.hpp"
#endif

namespace hlbm {
namespace HLBM_NS {  // one namespace per precision: no shared symbols

using real = HLBM_REAL;

constexpr int kQ = 9;
constexpr int kPlanes = 10;

// Arguments shared by every per-domain kernel.
struct DomainArgs {
  long long plane;     // elements per plane (padded)
  int nx, ny, bcx, bcy;
  int pitch;           // elements per state row (nx rounded up to 64)
  int flags;           // bit 0: Phi by finite differences, bit 1: centred E1, bit 2: no E2,
                       // bit 3: precise theta, bit 4: third-order expansion
  real mu, sigma, lambda, inv_cv, gm1, e2c, gamma, sgn_eps;
  real rho_ref, theta_ref, log_rho_ref, s_ref;
  real fref[kQ];       // deviation reference populations (zero in the FP64 form)
  real wall_u_lo, wall_u_hi, wall_theta;  // bcy == kBcWall: wall velocities, temperature
  // constants of the step formed once on the host (see node_state and collide)
  real th_off;         // theta - lapv: theta_ref with the precise-theta flag, else 0
  real eps_u;          // sgn_eps, infinite for the centred E1
  real sigma1;         // 1 - sigma
  real half_mu;        // mu / 2
  real e2h, e2k;       // E2's factor: (2 - gamma) / 2, and times cs2 / 2; zero without E2
  real cref;           // cs2 (theta_ref - 1)
  real k4;             // 9 / 4, zero for the third-order expansion
};

// State offset (within a plane) of node i = y nx + x of the dense [ny][nx]
// order used by the field arrays.
__device__ __forceinline__ long long state_off(const DomainArgs &d, long long i) {
  if (d.pitch == d.nx) return i;
  const int y = (int)(i / d.nx);
  return (long long)y * d.pitch + (i - (long long)y * d.nx);
}

struct StepArgs {
  DomainArgs d;
  const real *src;     // plane 0 of the state read this step
  real *dst;           // plane 0 of the state written
  unsigned *status;    // bit 0 set when a node diverged
  int rows;            // output rows per strip
  int nbx, nby;        // workgroups along x and y
  int xcd_remap;       // 1: spread spatial neighbours onto the same XCD
};

constexpr int kFlagPhiFD = 1, kFlagE1Centred = 2, kFlagE2Off = 4;
constexpr int kFlagPreciseTheta = 8;  // theta - theta_ref from expm1 / log1p (see node_dtheta)
// Hermite expansion truncated at third order (the original model of Sec. 2.3):
// the xxyy coefficient of every projected population, equilibrium and
// off-equilibrium alike, is zero (the deviation reference drops it too).
constexpr int kFlagFeq3 = 16;
constexpr int kBcWall = 2;  // rows y = 0 and y = ny - 1 are walls (ghosts beyond them clamp)

// ---------------------------------------------------------------- helpers
__device__ __forceinline__ int map_index(int v, int n, int bc) {
  if (bc == 0) {
    int r = v % n;
    return r < 0 ? r + n : r;
  }
  return v < 0 ? 0 : (v >= n ? n - 1 : v);
}

// Rows of a sweep in order, as map_index maps them, without a division a row.
struct RowWalk {
  int v, r;  // virtual row, and its wrapped index (periodic axis)
  __device__ __forceinline__ RowWalk(int v0, int n, int bc) : v(v0), r(map_index(v0, n, bc)) {}
  __device__ __forceinline__ int next(int n, int bc) {  // this row's index; moves to the next row
    const int now = bc == 0 ? r : (v < 0 ? 0 : (v >= n ? n - 1 : v));
    ++v;
    r = r + 1 >= n ? 0 : r + 1;
    return now;
  }
};

__device__ __forceinline__ float fma_r(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_r(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float min_r(float a, float b) { return __builtin_fminf(a, b); }
__device__ __forceinline__ double min_r(double a, double b) { return __builtin_fmin(a, b); }
__device__ __forceinline__ float rcp_fast(float x) { return __builtin_amdgcn_rcpf(x); }
// The hardware seed has about half the bits; two Newton-Raphson steps on the
// residual 1 - x r bring it within about half a unit in the last place, in 5
// instructions against 12 of the IEEE division (which also handles zero,
// infinities and subnormals, where this gives NaN: the operands here are
// densities, pressures and limited sums of squares of a state that is flagged
// when it is not positive and finite).
__device__ __forceinline__ double rcp_fast(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
  return __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
}
// A quotient takes as many: one step on the seed and one on the quotient's own
// residual, which leaves its rounding alone (half a unit; times rcp_fast, 1.5).
__device__ __forceinline__ double div_fast(double a, double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = __builtin_fma(__builtin_fma(-b, r, 1.0), r, r);
  const double q = a * r;
  return __builtin_fma(__builtin_fma(-b, q, a), r, q);
}
__device__ __forceinline__ float div_fast(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }
__device__ __forceinline__ float exp_r(float x) { return __expf(x); }
__device__ __forceinline__ double exp_r(double x) { return exp(x); }
__device__ __forceinline__ float log_r(float x) { return __logf(x); }
__device__ __forceinline__ double log_r(double x) { return log(x); }
__device__ __forceinline__ float sqrt_r(float x) { return __builtin_sqrtf(x); }
__device__ __forceinline__ double sqrt_r(double x) { return sqrt(x); }

constexpr double kCs2 = 1.0 / 3.0;

// Global access through a uniform base pointer and a 32-bit byte offset, so
// the address is SGPR base + VGPR offset (no 64-bit address arithmetic).
__device__ __forceinline__ real load_at(const real *base, unsigned byte_off) {
  return *(const real *)((const char *)base + byte_off);
}
__device__ __forceinline__ void store_at(real *base, unsigned byte_off, real v) {
  *(real *)((char *)base + byte_off) = v;
}
// Streaming store: the new state is not read again before the whole grid is
// written, so it bypasses cache retention.
__device__ __forceinline__ void store_stream(real *base, unsigned byte_off, real v) {
  __builtin_nontemporal_store(v, (real *)((char *)base + byte_off));
}

// Projection of the nine Hermite coefficients onto the D2Q9 populations:
// f_i = w_i [A0 + c.A/cs2 + H2:A2/(2 cs2^2) + (Hxxy Axxy + Hyyx Ayyx)/(2 cs2^3)
//            + Hxxyy Axxyy/(4 cs2^4)], written out per velocity class.
__device__ __forceinline__ void project(real A0, real Ax, real Ay, real Axx, real Axy, real Ayy,
                                        real Axxy, real Axyy, real Axxyy, real f[kQ]) {
  const real b0 = A0 - real(1.5) * (Axx + Ayy) + real(2.25) * Axxyy;
  f[0] = real(4.0 / 9.0) * b0;
  const real bx = A0 + real(3) * Axx - real(1.5) * Ayy - real(4.5) * Axxyy;
  const real ox = real(3) * Ax - real(4.5) * Axyy;
  f[1] = real(1.0 / 9.0) * (bx + ox);
  f[3] = real(1.0 / 9.0) * (bx - ox);
  const real by = A0 + real(3) * Ayy - real(1.5) * Axx - real(4.5) * Axxyy;
  const real oy = real(3) * Ay - real(4.5) * Axxy;
  f[2] = real(1.0 / 9.0) * (by + oy);
  f[4] = real(1.0 / 9.0) * (by - oy);
  const real bd = A0 + real(3) * (Axx + Ayy) + real(9) * Axxyy;
  const real dxy = real(9) * Axy;
  const real dx = real(3) * Ax + real(9) * Axyy;
  const real dy = real(3) * Ay + real(9) * Axxy;
  f[5] = real(1.0 / 36.0) * ((bd + dxy) + (dx + dy));
  f[6] = real(1.0 / 36.0) * ((bd - dxy) - (dx - dy));
  f[7] = real(1.0 / 36.0) * ((bd + dxy) - (dx + dy));
  f[8] = real(1.0 / 36.0) * ((bd - dxy) + (dx - dy));
}

// Node moments from the stored planes.  dr = rho - rho_ref (rho itself in the
// FP64 form), Pi deviations likewise relative to the rest state p_ref I.
struct NodeMoments {
  real dr, rho, jx, jy, pxx, pyy, pxy;
};

__device__ __forceinline__ NodeMoments node_moments(const real F[kQ], const DomainArgs &d) {
  NodeMoments m;
  const real r = ((F[0] + F[1]) + (F[2] + F[3])) + ((F[4] + F[5]) + (F[6] + F[7])) + F[8];
  m.dr = r;
  m.rho = r + d.rho_ref;
  const real d57 = F[5] - F[7];
  m.jx = ((F[1] - F[3]) + d57) + (F[8] - F[6]);
  m.jy = ((F[2] - F[4]) + d57) + (F[6] - F[8]);
  const real diag = (F[5] + F[6]) + (F[7] + F[8]);
  m.pxx = (F[1] + F[3]) + diag;
  m.pyy = (F[2] + F[4]) + diag;
  m.pxy = (F[5] - F[6]) + (F[7] - F[8]);
  return m;
}

// Natural logarithm of a normal number from the hardware's base-two one, the
// product with ln 2 = hi + lo kept to the last bit: the three operations that the
// open AMDGPU back end of LLVM lowers log to, without what it adds for zero and
// infinity, which give NaN here (such a density flags the state either way).
__device__ __forceinline__ float log_normal(float x) {
  const float y = __builtin_amdgcn_logf(x);
  constexpr float hi = 0x1.62e42ep-1f, lo = 0x1.efa39ep-25f;
  const float r = y * hi;
  return r + fma_r(y, lo, fma_r(y, hi, -r));
}

#if !HLBM_IS_F32
// A double constant that the compiler cannot lift out of the row loop: there
// the thirty constants of the two functions below would hold sixty vector
// registers for the whole sweep.  `zero` is an opaque zero (see opaque_zero); the
// constant is formed in scalar registers beside its use.
__device__ __forceinline__ int opaque_zero() {
  int zero;
  asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
  return zero;
}
__device__ __forceinline__ double near_const(const double c, const int zero) {
  const unsigned long long bits = __builtin_bit_cast(unsigned long long, c);
  const unsigned hi = (unsigned)(bits >> 32) ^ (unsigned)zero;
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | (unsigned)bits);
}

// a b + c with c = near_const(value): written out, as the compiler would copy
// the constant to a vector register for its two-operand form first.
__device__ __forceinline__ double fma_const(double a, double b, const double c, const int zero) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(near_const(c, zero)));
  return r;
}

// Their own logarithm and exponential take the FP64 sweep's node from about 110
// to 60 instructions for theta, and without library constants held across the
// row loop and the library's second, precise-theta branch it needs 153 vector
// registers instead of 208: three waves per SIMD.  2048^2 164 -> 152 us per step,
// Couette 2 x 100 15.6 -> 13.6.  theta over rho = e^-8 .. e^8, s = -1 .. 1 is at
// most 7.5 units of 2^-53 off, 1.0 near rho = 1 and s = 0, as with the library's
// (the argument's rounding).

// ln 2 = hi + lo, hi with 21 trailing zero bits: k hi is exact for |k| < 2^11.
constexpr double kLn2Hi = 0x1.62e42feep-1, kLn2Lo = 0x1.a39ef35793c76p-33;

// ln x of a positive normal number, x = 2^k m with m in [sqrt(1/2), sqrt(2)):
// k ln 2 + 2 atanh(t), t = f / (2 + f), f = m - 1, by the series of atanh to t^21
// (|t| < 0.172: truncated below 2^-56 of t).  With 2 t = f - t f the leading term
// is f itself, which is exact, and t's own rounding only enters times f: within
// 1.2 units in the last place (0.9 measured; 2.0 with 2 t for the leading term and
// ln 2 in one part).  Anything else (zero, negative, infinite) gives no meaningful
// number; the density it is taken of flags the state.
__device__ __forceinline__ double log_near(double x, const int zero) {
  double m = __builtin_amdgcn_frexp_mant(x);  // [1/2, 1)
  int k = __builtin_amdgcn_frexp_exp(x);
  const bool low = m < 0.70710678118654752440;
  m = low ? m + m : m;
  k = low ? k - 1 : k;
  const double f = m - 1.0;
  const double t = f * rcp_fast(m + 1.0);
  const double z = t * t;
  double p = near_const(2.0 / 21.0, zero);
  p = fma_const(p, z, 2.0 / 19.0, zero);
  p = fma_const(p, z, 2.0 / 17.0, zero);
  p = fma_const(p, z, 2.0 / 15.0, zero);
  p = fma_const(p, z, 2.0 / 13.0, zero);
  p = fma_const(p, z, 2.0 / 11.0, zero);
  p = fma_const(p, z, 2.0 / 9.0, zero);
  p = fma_const(p, z, 2.0 / 7.0, zero);
  p = fma_const(p, z, 2.0 / 5.0, zero);
  p = fma_const(p, z, 2.0 / 3.0, zero);
  const double e = (double)k, hi = near_const(kLn2Hi, zero);
  const double sum = __builtin_fma(e, hi, f);
  const double lost = __builtin_fma(e, hi, -sum) + f;  // its rounding, exactly
  const double low_part = __builtin_fma(e, near_const(kLn2Lo, zero), lost);
  return sum + __builtin_fma(-t, __builtin_fma(-z, p, f), low_part);
}

// e^x - off, off 0 or 1: 2^k + 2^k (e^r - 1) - off with k = round(x / ln 2), |r|
// <= ln 2 / 2 in two parts of ln 2 and e^r - 1 by the Taylor series to r^13
// (truncated below 2^-57), so off = 1 is accurate relative to itself (expm1).
// Within 1.1 units in the last place (1.0 measured).
__device__ __forceinline__ double exp_near(double x, const double off, const int zero) {
  const double k = __builtin_rint(x * near_const(1.44269504088896340736, zero));
  double r = __builtin_fma(-k, near_const(kLn2Hi, zero), x);
  r = __builtin_fma(-k, near_const(kLn2Lo, zero), r);
  double p = near_const(1.0 / 6227020800.0, zero);
  p = fma_const(p, r, 1.0 / 479001600.0, zero);
  p = fma_const(p, r, 1.0 / 39916800.0, zero);
  p = fma_const(p, r, 1.0 / 3628800.0, zero);
  p = fma_const(p, r, 1.0 / 362880.0, zero);
  p = fma_const(p, r, 1.0 / 40320.0, zero);
  p = fma_const(p, r, 1.0 / 5040.0, zero);
  p = fma_const(p, r, 1.0 / 720.0, zero);
  p = fma_const(p, r, 1.0 / 120.0, zero);
  p = fma_const(p, r, 1.0 / 24.0, zero);
  p = fma_const(p, r, 1.0 / 6.0, zero);
  p = __builtin_fma(p, r, 0.5);
  const double q = __builtin_fma(r * r, p, r);
  const double scale = __builtin_amdgcn_ldexp(1.0, (int)k);
  return __builtin_fma(scale, q, scale - off);
}
#endif

// theta from the stored entropy (deviation form: ds = s - s_ref), as the fields and
// reductions give it: any density has the value the functions give it (zero 0,
// negative NaN, infinite infinite), in FP64 with the library's.
__device__ __forceinline__ real field_theta(real rho, real sv, const DomainArgs &d) {
  return d.theta_ref * exp_r(sv * d.inv_cv + d.gm1 * (log_r(rho) - d.log_rho_ref));
}

// theta - theta_ref with relative accuracy on the deviation itself:
// theta_ref expm1(ds / c_v + (gamma - 1) ln(rho / rho_ref)), the density ratio
// from dr = rho - rho_ref in FP32 (log1p), rho itself in the FP64 form
// (rho_ref = 0, theta_ref = 1 there).  The Fourier term's Laplacian is taken
// of these deviations: in slow, well-resolved flows the temperature
// differences between neighbours are a few 1e-6 of theta, which absolute
// FP32 values would round to a few per cent.
//
// FP64 takes exp_near with off = 1.  FP32 uses the hardware exp and log with the
// classic corrections that make them accurate relative to small results:
// Goldberg's log1p(y) = ln(u) y / (u - 1) with u = 1 + y, exact when u rounds to
// 1, and expm1 by its Taylor series for |x| < 1/4, else Kahan's (u - 1) x / ln(u)
// with u = e^x.
#if HLBM_IS_F32
__device__ __forceinline__ float log1p_fast(float y) {
  const float u = 1.0f + y;
  const float um1 = u - 1.0f;
  return um1 == 0.0f ? y : __logf(u) * div_fast(y, um1);
}
__device__ __forceinline__ float expm1_fast(float x) {
  // |x| < 1/4: the Taylor series to x^7 (truncation below 1e-9 of the result)
  if (fabsf(x) < 0.25f) {
    const float p = 1.0f / 5040.0f;
    return x * (1.0f + x * (0.5f + x * (1.0f / 6.0f + x * (1.0f / 24.0f +
                x * (1.0f / 120.0f + x * (1.0f / 720.0f + x * p))))));
  }
  const float u = __expf(x);
  const float um1 = u - 1.0f;
  if (um1 == -1.0f) return -1.0f;
  return um1 * div_fast(x, __logf(u));
}
__device__ __forceinline__ float node_dtheta(float dr, float rho, float sv, const DomainArgs &d) {
  return d.theta_ref * expm1_fast(sv * d.inv_cv + d.gm1 * log1p_fast(dr / d.rho_ref));
}
#endif

// van Albada limited slope b phi(a/b), phi(r) = (r^2 + r)/(r^2 + 1), zero for
// a b <= 0; written as a b (a + b)/(a^2 + b^2).  Differences so small that
// a^2 + b^2 leaves the normal range (below 1e-30 in FP32, where the stored
// entropy deviation can reach them) give the limit value 0 instead of 0/0.
__device__ __forceinline__ real tiny_sq() { return sizeof(real) == 4 ? real(1e-30) : real(1e-300); }
__device__ __forceinline__ real van_albada(real a, real b) {
  const real ab = a * b;
  const real den = fma_r(a, a, b * b);
  return (ab > real(0) && den > tiny_sq()) ? div_fast(ab * (a + b), den) : real(0);
}

// Upwind MUSCL derivative u ds/dx at a node from the four differences around it,
// dmm = s-1 - s-2, dm = s0 - s-1, dp = s1 - s0, dpp = s2 - s1: u > 0 takes u [dm
// + (slope(dm, dp) - slope(dmm, dm)) / 2], u < 0 the mirror image, u = 0 gives 0.
__device__ __forceinline__ real muscl(real u, real dmm, real dm, real dp, real dpp) {
  const bool pos = u > real(0);
  const real d01 = pos ? dm : dp;
  const real sl0 = van_albada(d01, pos ? dp : dm);
  const real sl1 = van_albada(pos ? dmm : dpp, d01);
  return u * fma_r(real(0.5), sl0 - sl1, d01);
}

// Fourier and viscous heat over rho theta.
__device__ __forceinline__ real heat_term(const DomainArgs &d, real lap, real phi, real pt) {
  return div_fast(fma_r(d.lambda, lap, phi), pt);
}

// Laplacian of theta (or of theta - theta_ref, the same).
__device__ __forceinline__ real laplacian(real c, real e, real w, real n, real s) {
  return fma_r(real(-4), c, (e + w) + (n + s));
}

// What a node's neighbours and its own collision need of its moments.  lapv:
// theta, or theta - theta_ref accurate relative to itself with the
// precise-theta flag (the Laplacian's constant shift cancels); theta = lapv +
// th_off either way.
struct NodeState {
  real dr, ux, uy, lapv, pxx, pyy, pxy;
};

// Running divergence check of a lane's nodes: least density and temperature,
// and a sum that is NaN once a velocity or temperature was not finite.
struct Health {
  real least = real(1), acc = real(0);
  __device__ __forceinline__ void add(real rho, real ux, real uy, real th) {
    least = min_r(min_r(least, rho), th);
    acc = fma_r((ux + uy) + th, real(0), acc);
  }
  __device__ __forceinline__ bool bad() const { return !(least > real(0)) || acc != acc; }
};

// Moments, theta and Gamma of one node from its nine populations and entropy.
__device__ __forceinline__ NodeState node_state(const DomainArgs &d, const real (&F)[kQ],
                                                const real sv, Health &health, real &gx,
                                                real &gy) {
  const NodeMoments m = node_moments(F, d);
  const real inv_rho = rcp_fast(m.rho);
  NodeState o;
  o.dr = m.dr;
  o.pxx = m.pxx;
  o.pyy = m.pyy;
  o.pxy = m.pxy;
  o.ux = m.jx * inv_rho;
  o.uy = m.jy * inv_rho;
  real th;
#if HLBM_IS_F32
  if (d.flags & kFlagPreciseTheta) {
    o.lapv = node_dtheta(m.dr, m.rho, sv, d);
    th = o.lapv + d.th_off;
  } else {
    th = o.lapv = d.theta_ref * exp_r(sv * d.inv_cv + d.gm1 * (log_normal(m.rho) - d.log_rho_ref));
  }
#else
  const int zero = opaque_zero();
  o.lapv = exp_near(sv * d.inv_cv + d.gm1 * log_near(m.rho, zero), d.th_off, zero);
  th = o.lapv + d.th_off;
#endif
  const real omt = real(1) - th;
  gx = m.rho * o.ux * fma_r(-o.ux, o.ux, omt);
  gy = m.rho * o.uy * fma_r(-o.uy, o.uy, omt);
  health.add(m.rho, o.ux, o.uy, th);
  return o;
}

// Neighbour values of a collision: velocities and Gamma of the four neighbours,
// and Gamma of the node itself.
struct NodeStencil {
  real uxe, uxw, uxn, uxs, uye, uyw, uyn, uys, gxe, gxc, gxw, gyn, gyc, gys;
};

// E1 of one axis: the difference of Gamma upwind of the node's velocity,
// centred inside the rounding band (or everywhere with the centred flag, whose
// band is infinite), as one difference of selected values.
__device__ __forceinline__ real upwind_gamma(const DomainArgs &d, real u, real gw, real gc,
                                             real ge) {
  const bool back = u > d.eps_u, fore = u < -d.eps_u;
  const real diff = (back ? gc : ge) - (fore ? gc : gw);
  return (back || fore ? real(1) : real(0.5)) * diff;
}

// Gradients, correction term, HRR stress and the nine post-collision
// populations of one node, with its viscous heat phi and rho theta (pt).  sg,
// sg1: sigma and 1 - sigma.  One result wherever it is inlined: FP32 leaves the
// fused multiply-adds to the compiler (within an expression only), FP64 writes
// them out.
//
// FP64: in absolute populations and few operations.
//   - with tp = taubar p = mu + p / 2, 1 - 1/taubar = (mu - p / 2) / tp and
//     tau / taubar = mu / tp: one reciprocal in place of three divisions;
//   - the recursion and the Hermite coefficients are linear in a1, so a1 is
//     multiplied by 1 - 1/taubar first; with X = ux^2 + c, Y = uy^2 + c,
//     b = (1 - 1/taubar) a1:
//       Axxy  = uy (rho ux^2 + rho c + bxx) + 2 ux bxy,
//       Axxyy = Y (rho ux^2 + bxx) + X byy + rho c uy^2 + 4 ux uy bxy + rho c^2;
//   - the populations along an axis are summed from the terms that cancel first
//     (rho + 3 Axx), so that no partial sum is larger than it has to be, and
//     multiplied by their weight last.  With the factor 1/9 carried from the start
//     and one sum for both axes (ten FP64 instructions a node less, 1 % of the time
//     at 1500 x 1100, 0.4 % at 8192^2) a step rounded more than the formulas as they
//     stand: after 20 to 50 steps of eight flows velocities 3 to 7 % and densities
//     1 to 3 % further from the exact ones; this way velocities level to 2 %
//     closer, densities level.
// FP32: deviations from the rest reference formed from deviations (p - p_ref,
// rho c - rho_ref c_ref, rho c^2 - rho_ref c_ref^2).  Its rounding is kept term
// by term: E1 is discontinuous in the sign of u, so where a velocity crosses
// zero another rounding anywhere flips nodes (a 256^2 flow with steep
// gradients: 1e-3 of the velocity at single nodes after 50 steps).
__device__ __forceinline__ void collide(const DomainArgs &d, const NodeState &o,
                                        const NodeStencil &n, const real sg, const real sg1,
                                        real (&f)[kQ], real &phi, real &pt) {
#if HLBM_IS_F32
  const real cs2 = real(kCs2);
  const real ux = o.ux, uy = o.uy, th = o.lapv + d.th_off, rho = o.dr + d.rho_ref;
  // doubled velocity gradients (their factors 1/2 are exact wherever they go)
  const real gxx = n.uxe - n.uxw, gxy = n.uye - n.uyw;
  const real gyx = n.uxn - n.uxs, gyy = n.uyn - n.uys;
  const real S = gxx - gyy, T = gyx + gxy;
  const real p = rho * cs2 * th;
  const real dth = th - d.theta_ref;
  const real dp = cs2 * (o.dr * th + d.rho_ref * dth);  // p - p_ref
  const real tau = d.mu * rcp_fast(p);
  const real taub = tau + real(0.5);
  const real itaub = rcp_fast(taub);
  const real e2 = d.e2h * p * (gxx + gyy);
  const real Exx = upwind_gamma(d, ux, n.gxw, n.gxc, n.gxe) + e2;
  const real Eyy = upwind_gamma(d, uy, n.gys, n.gyc, n.gyn) + e2;
  const real rux = rho * ux, ruy = rho * uy;
  const real ruxx = rux * ux, ruyy = ruy * uy, ruxy = rux * uy;
  // HRR stress
  const real htp = real(-0.5) * (taub * p);
  real a1xx = sg1 * (htp * S), a1yy = -a1xx, a1xy = sg1 * (htp * T);
  if (sg != real(0)) {
    const real prxx = (o.pxx - dp) - ruxx + real(0.5) * Exx;
    const real pryy = (o.pyy - dp) - ruyy + real(0.5) * Eyy;
    const real prxy = o.pxy - ruxy;
    a1xx = sg * prxx + a1xx;
    a1yy = sg * pryy + a1yy;
    a1xy = sg * prxy + a1xy;
  }
  const real c = cs2 * (th - real(1));
  const real ux2 = ux + ux, uy2 = uy + uy;
  const real a1xxy = uy * a1xx + ux2 * a1xy;
  const real a1xyy = ux * a1yy + uy2 * a1xy;
  const real a1xxyy = real(2) * (ux * a1xyy + uy * a1xxy) + (c - ux * ux) * a1yy +
                      (c - uy * uy) * a1xx - ux2 * uy2 * a1xy;
  const real om = real(1) - itaub;
  const real drc = dp - cs2 * o.dr;
  const real dc = cs2 * dth;
  const real drc2 = o.dr * c * c + d.rho_ref * dc * (c + d.cref);
  const real Axx = ruxx + drc + om * a1xx + real(0.5) * Exx;
  const real Ayy = ruyy + drc + om * a1yy + real(0.5) * Eyy;
  const real Axy = ruxy + om * a1xy;
  const real rc = rho * c;
  const real Axxy = ruxx * uy + rc * uy + om * a1xxy;
  const real Axyy = ruyy * ux + rc * ux + om * a1xyy;
  const real Axxyy = (d.flags & kFlagFeq3)
                         ? real(0)
                         : ruxx * uy * uy + rc * (ux * ux + uy * uy) + drc2 + om * a1xxyy;
  project(o.dr, rux, ruy, Axx, Axy, Ayy, Axxy, Axyy, Axxyy, f);
  if (d.flags & kFlagPhiFD) {
    const real aa = real(0.5) * S, bb = real(0.5) * T;
    phi = d.mu * (aa * aa + bb * bb);
  } else {
    phi = (real(-0.5) * (tau * itaub)) * (a1xx * gxx + a1xy * T + a1yy * gyy);
  }
  pt = rho * th;
#else
  constexpr real cs2 = real(kCs2);
  const real ux = o.ux, uy = o.uy;
  const real th = o.lapv + d.th_off;
  const real rho = o.dr;
  // doubled velocity gradients
  const real gxx = n.uxe - n.uxw, gxy = n.uye - n.uyw;
  const real gyx = n.uxn - n.uxs, gyy = n.uyn - n.uys;
  const real S = gxx - gyy, T = gyx + gxy;
  pt = rho * th;
  const real tp = fma_r(pt, real(0.5 * kCs2), d.mu);
  const real rtp = rcp_fast(tp);
  const real om = fma_r(pt, real(-0.5 * kCs2), d.mu) * rtp;
  const real c = cs2 * (th - real(1));
  const real rc = rho * c;
  const real dp = cs2 * pt;
  // (E1 + E2) / 2
  const real e1x = upwind_gamma(d, ux, n.gxw, n.gxc, n.gxe);
  const real e1y = upwind_gamma(d, uy, n.gys, n.gyc, n.gyn);
  const real e2 = d.e2k * (pt * (gxx + gyy));
  const real hEx = fma_r(e1x, real(0.5), e2);
  const real hEy = fma_r(e1y, real(0.5), e2);
  const real rux = rho * ux, ruy = rho * uy;
  const real uxx = ux * ux, uyy = uy * uy;
  const real ruxx = rux * ux, ruyy = ruy * uy, ruxy = rux * uy;
  // HRR stress
  const real fd = sg1 * fma_r(pt, real(-0.25 * kCs2), -d.half_mu);
  const real fS = fd * S, fT = fd * T;
  const real prxx = o.pxx - ((dp + ruxx) - hEx);
  const real pryy = o.pyy - ((dp + ruyy) - hEy);
  const real prxy = o.pxy - ruxy;
  const real axx = fma_r(sg, prxx, fS), ayy = fma_r(sg, pryy, -fS), axy = fma_r(sg, prxy, fT);
  if (d.flags & kFlagPhiFD) {
    phi = (real(0.5) * d.half_mu) * fma_r(S, S, T * T);
  } else {
    phi = -(d.half_mu * rtp) * fma_r(axx, gxx, fma_r(axy, T, ayy * gyy));
  }
  const real bxx = om * axx, byy = om * ayy, bxy = om * axy;
  const real Nx = ruxx + bxx, Ny = ruyy + byy;
  const real Axx = (ruxx + rc) + (bxx + hEx), Ayy = (ruyy + rc) + (byy + hEy), Axy = ruxy + bxy;
  const real ux2 = ux + ux, uy2 = uy + uy;
  const real P1 = ux2 * bxy, P2 = uy2 * bxy;
  const real Axxy = fma_r(uy, Nx + rc, P1), Axyy = fma_r(ux, Ny + rc, P2);
  const real X = uxx + c, Y = uyy + c;
  const real Axxyy =
      fma_r(Y, Nx, fma_r(rc, uyy, fma_r(X, byy, fma_r(uy2, P1, rc * c))));
  // projection on the nine populations
  constexpr real w0 = real(4.0 / 9.0), w1 = real(1.0 / 9.0), w2 = real(1.0 / 36.0);
  const real s = Axx + Ayy;
  const real Z = d.k4 * Axxyy;
  f[0] = w0 * (fma_r(real(-1.5), s, rho) + Z);
  const real px = fma_r(real(-1.5), Ayy, fma_r(real(-2), Z, fma_r(real(3), Axx, rho)));
  const real py = fma_r(real(-1.5), Axx, fma_r(real(-2), Z, fma_r(real(3), Ayy, rho)));
  const real ox = fma_r(real(3), rux, real(-4.5) * Axyy);
  const real oy = fma_r(real(3), ruy, real(-4.5) * Axxy);
  f[1] = w1 * (px + ox);
  f[3] = w1 * (px - ox);
  f[2] = w1 * (py + oy);
  f[4] = w1 * (py - oy);
  const real bd = fma_r(real(3), s, fma_r(real(4), Z, rho));
  const real dxy = real(9) * Axy;
  const real dx = fma_r(real(3), rux, real(9) * Axyy);
  const real dy = fma_r(real(3), ruy, real(9) * Axxy);
  const real ep = bd + dxy, em = bd - dxy, gp = dx + dy, gm = dx - dy;
  f[5] = w2 * (ep + gp);
  f[7] = w2 * (ep - gp);
  f[6] = w2 * (em - gm);
  f[8] = w2 * (em + gm);
#endif
}

// --------------------------------------------------------------- the step
//
// One workgroup owns a tile of CW output columns (x0 a multiple of CW, so
// every row segment it stores is aligned) and `rows` output rows, plus a
// radius-2 halo.  Lanes 0..CW-1 handle the tile's columns; an extra wave
// holds the four halo columns (x0-2, x0-1, x0+CW, x0+CW+1) on its first four
// lanes.  In the LDS rings a column sits at position ri = column - (x0 - 2).
// Each lane sweeps the rows of the strip through three stages:
//   A(j)  moments of row j from the ten planes: u, Gamma_x, theta and s go into
//         LDS rings, the rest stays in registers;
//   B(k)  collision of row k (radius-1 stencil: x-neighbours through the rings,
//         y-neighbours from the lane's registers), its heat and the x part of
//         its entropy's advection: the six populations with c_x != 0 into LDS
//         rings, the rest into the lane's registers;
//   C(k)  pull streaming of row k out of those and its entropy update, storing
//         both.
// Iteration i runs A(i+1) and B(i), a barrier, issues the loads of row i+2 and
// runs C(i-1), and a second barrier: B(i) needs its x-neighbours of row i (of
// the previous iteration) and its own column's rows i-1 .. i+1, so it follows
// A(i+1) without a barrier and only one row of node state is carried.
//
// The x part of the entropy's advection reads only row k's own s, so B forms
// it; C has the y part from the lane's last four differences of s, which pass
// from row to row in registers.
//
// Ring depths are the smallest the two barriers allow: u_x, u_y, Gamma_x, theta
// and s two rows (A(i+1) writes while B(i) reads), populations by the row they
// stream from: c_y = 0 -> 2, c_y = +1 (read one row later) -> 3, c_y = -1 -> 1.
// 22 rows in all: 17.8 KB at CW = 192 in FP32.
//
// Every lane runs every stage of every row, also where a stencil reaches past
// the ring or a row's inputs are not there yet: such values are read by no
// valid node, and without branches around the stages their results need no
// merging (a third of the sweep's instructions were moves).  `lo` and `hi` keep
// those reads of a ring's neighbours inside the structure.  Only loads and
// stores look at the lane, and the divergence check counts valid nodes only.
template <int W>
struct LevelRings {
  real lo[64];
  real ux[2][W], uy[2][W], gx[2][W], th[2][W], s[2][W];
  real f0[2][2][W];  // populations 1, 3   (c_y =  0)
  real fp[3][2][W];  // populations 5, 6   (c_y = +1)
  real fm[2][W];     // populations 7, 8   (c_y = -1)
  real hi[64];
};

// Per-lane registers of one time level.
struct LevelRegs {
  // A -> B: the newest row (n), B's row (c) and the row below it (m); ds: s minus
  // the row below's
  real n_dr = 0, n_pxx = 0, n_pyy = 0, n_pxy = 0, n_ux = 0, n_uy = 0, n_th = 1, n_gx = 0, n_gy = 0;
  real n_s = 0, n_ds = 0;
  real c_dr = 0, c_pxx = 0, c_pyy = 0, c_pxy = 0, c_ux = 0, c_uy = 0, c_th = 1, c_gx = 0, c_gy = 0;
  real c_s = 0, c_ds = 0;
  real m_ux = 0, m_uy = 0, m_th = 1, m_gy = 0;
  real p_s = 0, p_ds = 0, q_ds = 0;  // s and ds of the rows below
  // B -> C: last B row (b), the row below it (p), and of two rows below (q)
  real b_adv = 0, b_heat = 0, b_vy = 0, b_f0 = 0, b_f2 = 0, b_f4 = 0;
  real p_adv = 0, p_heat = 0, p_vy = 0, p_f0 = 0, p_f2 = 0, q_f2 = 0;
};

// A(j): moments of one node of row j from its nine populations and entropy;
// z = j mod 2.
template <int W>
__device__ __forceinline__ void level_a(const DomainArgs &d, LevelRegs &g, LevelRings<W> &R,
                                        const int z, const int ri, const real (&F)[kQ],
                                        const real sv, Health &health) {
  real gx, gy;
  const NodeState o = node_state(d, F, sv, health, gx, gy);
  R.ux[z][ri] = o.ux;
  R.uy[z][ri] = o.uy;
  R.gx[z][ri] = gx;
  R.th[z][ri] = o.lapv;
  R.s[z][ri] = sv;
  g.m_ux = g.c_ux;
  g.m_uy = g.c_uy;
  g.m_th = g.c_th;
  g.m_gy = g.c_gy;
  g.c_dr = g.n_dr;
  g.c_pxx = g.n_pxx;
  g.c_pyy = g.n_pyy;
  g.c_pxy = g.n_pxy;
  g.c_ux = g.n_ux;
  g.c_uy = g.n_uy;
  g.c_th = g.n_th;
  g.c_gx = g.n_gx;
  g.c_gy = g.n_gy;
  g.q_ds = g.p_ds;
  g.p_ds = g.c_ds;
  g.c_ds = g.n_ds;
  g.n_ds = sv - g.n_s;
  g.p_s = g.c_s;
  g.c_s = g.n_s;
  g.n_s = sv;
  g.n_dr = o.dr;
  g.n_pxx = o.pxx;
  g.n_pyy = o.pyy;
  g.n_pxy = o.pxy;
  g.n_ux = o.ux;
  g.n_uy = o.uy;
  g.n_th = o.lapv;
  g.n_gx = gx;
  g.n_gy = gy;
}

// B(k): collision, heat and x advection of row k (row k + 1 was the last A);
// z = k mod 2, sc = k mod 3.
template <int W>
__device__ __forceinline__ void level_b(const DomainArgs &d, LevelRegs &g, LevelRings<W> &R,
                                        const int z, const int sc, const int ri, const real sg,
                                        const real sg1) {
  NodeStencil n;
  n.uxe = R.ux[z][ri + 1];
  n.uxw = R.ux[z][ri - 1];
  n.uye = R.uy[z][ri + 1];
  n.uyw = R.uy[z][ri - 1];
  n.gxe = R.gx[z][ri + 1];
  n.gxw = R.gx[z][ri - 1];
  n.uxn = g.n_ux;
  n.uxs = g.m_ux;
  n.uyn = g.n_uy;
  n.uys = g.m_uy;
  n.gyn = g.n_gy;
  n.gxc = g.c_gx;
  n.gyc = g.c_gy;
  n.gys = g.m_gy;
  const real the = R.th[z][ri + 1], thw = R.th[z][ri - 1];
  const real se = R.s[z][ri + 1], sw = R.s[z][ri - 1];
  const real see = R.s[z][ri + 2], sww = R.s[z][ri - 2];
  const NodeState o{g.c_dr, g.c_ux, g.c_uy, g.c_th, g.c_pxx, g.c_pyy, g.c_pxy};
  real f[kQ], phi, pt;
  collide(d, o, n, sg, sg1, f, phi, pt);
  R.f0[z][0][ri] = f[1];
  R.f0[z][1][ri] = f[3];
  R.fp[sc][0][ri] = f[5];
  R.fp[sc][1][ri] = f[6];
  R.fm[0][ri] = f[7];
  R.fm[1][ri] = f[8];
  g.q_f2 = g.p_f2;
  g.p_adv = g.b_adv;
  g.p_heat = g.b_heat;
  g.p_vy = g.b_vy;
  g.p_f0 = g.b_f0;
  g.p_f2 = g.b_f2;
  g.b_f0 = f[0];
  g.b_f2 = f[2];
  g.b_f4 = f[4];
  g.b_vy = o.uy;
  g.b_heat = heat_term(d, laplacian(g.c_th, the, thw, g.n_th, g.m_th), phi, pt);
  g.b_adv = muscl(o.ux, sw - sww, g.c_s - sw, se - g.c_s, see - se);
}

// C(k): pull streaming of row k and its entropy update (row k + 1 was the
// last B); z = k mod 2, pm = (k - 1) mod 3 (the slots of row k in f0 and of row
// k - 1 in fp).
template <int W>
__device__ __forceinline__ void level_c(const LevelRegs &g, const LevelRings<W> &R, const int z,
                                        const int pm, const int ri, real (&Fo)[kQ], real &snew) {
  Fo[0] = g.p_f0;                  // row k, this column
  Fo[1] = R.f0[z][0][ri - 1];
  Fo[3] = R.f0[z][1][ri + 1];
  Fo[2] = g.q_f2;                  // row k - 1, this column
  Fo[5] = R.fp[pm][0][ri - 1];
  Fo[6] = R.fp[pm][1][ri + 1];
  Fo[4] = g.b_f4;                  // row k + 1, this column
  Fo[7] = R.fm[0][ri + 1];
  Fo[8] = R.fm[1][ri - 1];
  // row k's s and the differences around it; the newest A was row k + 2
  snew = g.p_s - (g.p_adv + muscl(g.p_vy, g.q_ds, g.p_ds, g.c_ds, g.n_ds)) + g.p_heat;
}

template <bool kValue>
struct Flag {
  static constexpr bool value = kValue;
};
// Batched items: the skip of a frozen domain is decided once per item for
// the whole workgroup (another workgroup can set the flag at any moment, and
// waves that read it at different times would disagree and pair up barriers
// across items).  Every thread reads the flag word before the item's first
// loads are issued (one request per wave, no branch, so no wait for it is
// placed before those loads); the sweep's first barrier, an OR over the
// threads, then decides for all of them, so the flag's latency overlaps the
// loads.
__device__ __forceinline__ unsigned domain_frozen(const unsigned *status) {
  return __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <bool kBatch>
__device__ __forceinline__ bool barrier_skip(unsigned frozen) {
  if constexpr (kBatch) return __syncthreads_or(frozen != 0u) != 0;
  __syncthreads();
  return false;
}

// One tile (bx, by) of one domain: src / dst point at plane 0 of the two
// state buffers, planes are `d.plane` elements apart.  Ends with a barrier,
// so the rings can be reused by the next tile.  kBatch: returns after the
// prologue when any thread's `frozen` is nonzero (see domain_frozen).
template <int CW, bool kBatch = false>
__device__ __forceinline__ void sweep_tile(const DomainArgs &d, const real *src0, real *dst0,
                                           unsigned *status, const int rows, const int bx,
                                           const int by, const unsigned frozen,
                                           LevelRings<CW + 4> &R) {
  const int t = threadIdx.x;
  const real *src[kPlanes];
  real *dst[kPlanes];
#pragma unroll
  for (int q = 0; q < kPlanes; ++q) {
    src[q] = src0 + (long long)q * d.plane;
    dst[q] = dst0 + (long long)q * d.plane;
  }
  const int x0 = bx * CW, y0 = by * rows;
  // lane -> ring position: tile lanes at 2..CW+1, halo lanes at 0, 1, CW+2, CW+3
  const int h = t - CW;
  const int ri = t < CW ? t + 2 : (h < 2 ? h : (h < 4 ? CW + h : 0));
  const int vx = x0 - 2 + ri;
  const int cx = map_index(vx, d.nx, d.bcx);
  const int nrow = min(rows, d.ny - y0);
  const bool own_col = t < CW && vx < d.nx;
  constexpr unsigned kEl = sizeof(real);
  Health health;
  LevelRegs g;

  real ld[kPlanes];
  auto load_row = [&](const int j) {  // virtual row j, at a 32-bit byte offset
    const unsigned off = (unsigned)(map_index(y0 - 2 + j, d.ny, d.bcy) * d.pitch + cx) * kEl;
#pragma unroll
    for (int q = 0; q < kPlanes; ++q) ld[q] = load_at(src[q], off);
  };
  auto stage_a = [&](const int z) {
    real F[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) F[q] = ld[q];
    level_a(d, g, R, z, ri, F, ld[9], health);
  };

  // A(i + 1), B(i), a barrier, the loads of row i + 2 and (kOut) C(i - 1).  The
  // loads come before C's stores: a wait for them never waits for this row's
  // stores as well.  m = i mod 3, mp = (i + 1) mod 3.
  int m = 0, mp = 1;
  auto row = [&](const int i, auto kOut) {
    const int z = i & 1;
    stage_a(1 - z);
    // wall rows take the projected stress alone: their rebuilt populations
    // carry the wall's finite-difference stress
    const int yk = y0 - 2 + i;
    const bool wall_row = d.bcy == kBcWall && (yk == 0 || yk == d.ny - 1);
    level_b(d, g, R, z, m, ri, wall_row ? real(1) : d.sigma, wall_row ? real(0) : d.sigma1);
    __syncthreads();
    if (i + 2 <= nrow + 3) load_row(i + 2);
    if constexpr (kOut.value) {
      real Fo[kQ], snew;
      level_c(g, R, 1 - z, mp, ri, Fo, snew);
      if (own_col) {
        const unsigned off = (unsigned)((y0 + i - 3) * d.pitch + vx) * kEl;
#pragma unroll
        for (int q = 0; q < kQ; ++q) store_stream(dst[q], off, Fo[q]);
        store_stream(dst[9], off, snew);
      }
    }
    m = mp;
    mp = mp == 2 ? 0 : mp + 1;
    __syncthreads();
  };

  load_row(0);
  stage_a(0);
  load_row(1);
  if (barrier_skip<kBatch>(frozen)) return;
  for (int i = 0; i < 3; ++i) row(i, Flag<false>());
  for (int i = 3; i <= nrow + 2; ++i) row(i, Flag<true>());
  if (health.bad()) atomicOr(status, 1u);
}

// Whole-domain step: one workgroup per tile.
template <int CW>
__global__ __launch_bounds__(CW + 64) __attribute__((amdgpu_waves_per_eu(HLBM_IS_F32 ? 6 : 3)))
void k_step(StepArgs a) {
  __shared__ LevelRings<CW + 4> R;
  int bid = blockIdx.x;
  const int nblk = a.nbx * a.nby;
  if (a.xcd_remap) {
    // Workgroups are dealt round-robin to the 8 XCDs; give each XCD a
    // contiguous range of tiles so halo re-reads stay in its L2.
    const int per = (nblk + 7) >> 3;
    const int xcd = bid & 7, k = bid >> 3;
    const int full = nblk - (per - 1) * 8;  // XCDs that get `per` tiles
    bid = xcd < full ? xcd * per + k : full * per + (xcd - full) * (per - 1) + k;
  }
  sweep_tile<CW>(a.d, a.src, a.dst, a.status, a.rows, bid % a.nbx, bid / a.nbx, 0, R);
}

// Batched step: a persistent grid walks a list of (domain, tile) items in a
// static order (tile_walk; no atomics: the launch can be captured and
// replayed).  Items of a domain whose divergence flag is set are skipped, so
// a diverged domain freezes while the others go on (see domain_frozen).
struct BatchArgs {
  const DomainArgs *doms;
  const long long *offs;  // element offset of each domain's state in a buffer
  const int4 *items;      // (domain, bx, by, strip rows; the kernels read the first three)
  int nitems;
  const real *src_buf;
  real *dst_buf;
  unsigned *status;       // one word per domain
  int rows;
  // tile kernels: when set, the moments (rho, u_x, u_y, theta) of the new
  // state go to mom[c * mom_sc + foffs[domain] + y nx + x], c = 0..3, as
  // k_batch_moments computes them
  real *mom;
  const long long *foffs;
  long long mom_sc;
  // tile kernels: when set, a pending learned correction (moments cx,
  // increments cdl, channel stride mom_sc, per-domain partial sums cparts;
  // see k_corr_apply) is applied to the state as it is loaded, as
  // k_corr_apply would have stored it
  const float *cx, *cdl;
  const double *cparts;
  int cconserve;
};

// This workgroup's share of the persistent walk over n items: items first,
// first + step, ... below end.  Workgroups are dealt round-robin to the
// eight XCDs (workgroup b to XCD b mod 8); with at least eight workgroups XCD x
// gets a contiguous eighth of the items, taken in order by its workgroups, so
// tiles and strips that share halo rows and columns, and the cache lines their rows
// share, go through one L2: 8 x 256^2 two-step tiles 14.3 -> 13.2 us per step, 8 x
// 128^2 7.6 -> 5.8; also batches larger than the last-level cache (two-step FP32
// strips: 16 x 1024^2 203 -> 192).  The first n mod 8 XCDs, which have a workgroup
// more where each workgroup takes one item, get the item more: shares rounded
// otherwise leave one workgroup two items in a row (2 x 1024^2 FP64 on 192 x 28
// strips, 444 items: 142 us per step).
struct TileWalk {
  int first, step, end;
};
__device__ __forceinline__ TileWalk tile_walk(const int n) {
  const int g = (int)gridDim.x, b = (int)blockIdx.x;
  if (g < 8) return TileWalk{b, g, n};
  const int x = b & 7, per = n >> 3, more = n & 7;
  const int lo = x * per + min(x, more);
  return TileWalk{lo + (b >> 3), (g - x + 7) >> 3, lo + per + (x < more ? 1 : 0)};
}

// FP64 takes 186 registers here, so two waves per SIMD: held to three it spills 14
// of them in every row (us per step, three -> two waves: 12 x 200^2 on 192 x 16
// strips 70 -> 57, 4 x 1024^2 on 64 x 64 304 -> 218, on 128 x 32 215 -> 198).
template <int CW>
__global__ __launch_bounds__(CW + 64) __attribute__((amdgpu_waves_per_eu(HLBM_IS_F32 ? 4 : 2)))
void k_step_batch(BatchArgs a) {
  __shared__ LevelRings<CW + 4> R;
  const TileWalk walk = tile_walk(a.nitems);
  for (int it = walk.first; it < walk.end; it += walk.step) {
    const int4 w = a.items[it];
    const int dm = __builtin_amdgcn_readfirstlane(w.x);
    const DomainArgs d = a.doms[dm];
    const long long off = a.offs[dm];
    // after the loads it must not wait for (memory counters drain in order)
    const unsigned frozen = domain_frozen(a.status + dm);
    sweep_tile<CW, true>(d, a.src_buf + off, a.dst_buf + off, a.status + dm, a.rows,
                         __builtin_amdgcn_readfirstlane(w.y), __builtin_amdgcn_readfirstlane(w.z),
                         frozen, R);
  }
}

}  // namespace HLBM_NS
}  // namespace hlbm

#include "hlbm_step2.hpp"
#include "closure_device.hpp"  // the per-node correction the tile kernels can apply
#include "hlbm_tile.hpp"

namespace hlbm {
namespace HLBM_NS {

// ------------------------------------------------------ initialisation
//
// F0 = f^eq + f^1[a1FD] - psi/2 (algorithm of Sec. 3.5, steps 2-4), one
// thread per node, stencils read straight from the input fields.
struct InitArgs {
  DomainArgs d;
  const real *rho, *ux, *uy, *s;
  real *dst;  // ten planes
};

__device__ __forceinline__ void load_node(const InitArgs &a, int x, int y, real &r, real &u,
                                          real &v, real &th) {
  const int cx = map_index(x, a.d.nx, a.d.bcx), cy = map_index(y, a.d.ny, a.d.bcy);
  const long long i = (long long)cy * a.d.nx + cx;
  r = a.rho[i];
  u = a.ux[i];
  v = a.uy[i];
  // absolute entropy in: theta = rho^(gamma-1) exp(s / c_v)
  th = exp_r(a.s[i] * a.d.inv_cv + a.d.gm1 * log_r(r));
}

__global__ void k_init(InitArgs a) {
  const DomainArgs &d = a.d;
  const long long n = (long long)d.nx * d.ny;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const int x = (int)(i % d.nx), y = (int)(i / d.nx);
    real rho, ux, uy, th, re, ue, ve, te, rw, uw, vw, tw, rn, un, vn, tn, rs, us, vs, ts;
    load_node(a, x, y, rho, ux, uy, th);
    load_node(a, x + 1, y, re, ue, ve, te);
    load_node(a, x - 1, y, rw, uw, vw, tw);
    load_node(a, x, y + 1, rn, un, vn, tn);
    load_node(a, x, y - 1, rs, us, vs, ts);
    const real cs2 = real(kCs2);
    const real dxux = real(0.5) * (ue - uw), dxuy = real(0.5) * (ve - vw);
    const real dyux = real(0.5) * (un - us), dyuy = real(0.5) * (vn - vs);
    const real div = dxux + dyuy;
    const real p = rho * cs2 * th;
    const real tau = d.mu / p, taub = tau + real(0.5);
    auto gam = [](real r, real u, real t) { return r * u * ((real(1) - t) - u * u); };
    const real gc = gam(rho, ux, th), gxe = gam(re, ue, te), gxw = gam(rw, uw, tw);
    const real gcy = gam(rho, uy, th), gyn = gam(rn, vn, tn), gys = gam(rs, vs, ts);
    real e1x, e1y;
    if (d.flags & kFlagE1Centred) {
      e1x = real(0.5) * (gxe - gxw);
      e1y = real(0.5) * (gyn - gys);
    } else {
      const real ep = d.sgn_eps;
      e1x = ux > ep ? gc - gxw : (ux < -ep ? gxe - gc : real(0.5) * (gxe - gxw));
      e1y = uy > ep ? gcy - gys : (uy < -ep ? gyn - gcy : real(0.5) * (gyn - gys));
    }
    const real e2 = (d.flags & kFlagE2Off) ? real(0) : d.e2c * p * div;
    const real Exx = e1x + e2, Eyy = e1y + e2;
    const real tp = taub * p;
    const real a1xx = -tp * (dxux - dyuy), a1yy = -a1xx, a1xy = -tp * (dyux + dxuy);
    const real c = cs2 * (th - real(1));
    const real a1xxy = uy * a1xx + real(2) * ux * a1xy;
    const real a1xyy = ux * a1yy + real(2) * uy * a1xy;
    const real a1xxyy = real(2) * (ux * a1xyy + uy * a1xxy) + (c - ux * ux) * a1yy +
                        (c - uy * uy) * a1xx - real(4) * ux * uy * a1xy;
    const real rc = rho * c;
    const real cref = cs2 * (d.theta_ref - real(1));
    const real A0 = rho - d.rho_ref;
    const real Axx = rho * ux * ux + (rc - d.rho_ref * cref) + a1xx - real(0.5) * Exx;
    const real Ayy = rho * uy * uy + (rc - d.rho_ref * cref) + a1yy - real(0.5) * Eyy;
    const real Axy = rho * ux * uy + a1xy;
    const real Axxy = rho * ux * ux * uy + rc * uy + a1xxy;
    const real Axyy = rho * ux * uy * uy + rc * ux + a1xyy;
    const real Axxyy = (d.flags & kFlagFeq3) ? real(0)
                                             : rho * ux * ux * uy * uy + rc * (ux * ux + uy * uy) +
                                                   (rc * c - d.rho_ref * cref * cref) + a1xxyy;
    real f[kQ];
    project(A0, rho * ux, rho * uy, Axx, Axy, Ayy, Axxy, Axyy, Axxyy, f);
    const long long P = d.plane;
    const long long o = (long long)y * d.pitch + x;
#pragma unroll
    for (int q = 0; q < kQ; ++q) a.dst[q * P + o] = f[q];
    a.dst[9 * P + o] = a.s[i] - d.s_ref;
  }
}

// ------------------------------------------------------------ walls
//
// Isothermal moving walls on the rows y = 0 and y = ny - 1 (bcy == kBcWall),
// a regularised wet-node wall: our reading of the wall condition that the
// thermal Couette case of Sec. 4.4 takes from an earlier paper without
// stating it.  After every step (and after initialisation) each wall node is
// rebuilt as f^eq(rho_w, U, 0, theta_w) + f^1[a1FD], psi taken as zero, with
//   rho_w = its c_y = 0 populations plus twice those that arrived from the
//           interior (no mass flux through the wall);
//   a1FD  from the velocity gradient at the wall: zero along it, one-sided
//         second order across it, (-3 u_w + 4 u_1 - u_2) / 2 over the new
//         velocities of the next two rows;
//   s_w   = c_v ln(theta_w / rho_w^(gamma - 1)).
// One thread per wall node, in place: a thread reads its node and two rows
// of the interior, which no thread writes (ny >= 4).
struct WallArgs {
  DomainArgs d;
  real *state;  // plane 0 of the current state
};

// One wall node from its streamed populations F[0..8] and the new velocities of the
// next two rows inside; its populations and entropy in place.  side: 0 the wall
// y = 0, 1 the other.
__device__ __forceinline__ void wall_rebuild(const DomainArgs &d, const int side, real (&F)[kPlanes],
                                             const real u1x, const real u1y, const real u2x,
                                             const real u2y) {
  const int dir = side ? -1 : 1;
  const real U = side ? d.wall_u_hi : d.wall_u_lo;
  // arrived from the interior: c_y = -1 (4, 7, 8) at y = 0, c_y = +1 (2, 5, 6) at the top;
  // the rest state's share of the sum is exactly rho_ref, so this is rho_w - rho_ref
  const real in = side ? (F[2] + F[5]) + F[6] : (F[4] + F[7]) + F[8];
  const real dr = ((F[0] + F[1]) + F[3]) + real(2) * in;
  const real rho = dr + d.rho_ref;
  const real half = real(0.5) * real(dir);
  const real dyux = half * ((real(4) * u1x - u2x) - real(3) * U);
  const real dyuy = half * (real(4) * u1y - u2y);
  const real cs2 = real(kCs2);
  const real th = d.wall_theta;
  const real p = rho * cs2 * th;
  const real tp = (d.mu / p + real(0.5)) * p;  // taubar p
  // a1FD = -taubar p (grad u + grad u^T - div I) with d/dx = 0 and div = dyuy
  const real a1xx = tp * dyuy, a1yy = -a1xx, a1xy = -tp * dyux;
  const real c = cs2 * (th - real(1));
  const real a1xxy = real(2) * U * a1xy;
  const real a1xyy = U * a1yy;
  const real a1xxyy = real(2) * U * a1xyy + (c - U * U) * a1yy + c * a1xx;
  // deviations from the rest reference formed from deviations (theta_w is
  // exact, so nothing cancels): rho c - rho_ref c_ref = (p - p_ref) - cs2
  // (rho - rho_ref), rho c^2 - rho_ref c_ref^2 = dr c^2 + rho_ref dc (c + c_ref)
  const real rc = rho * c;
  const real cref = cs2 * (d.theta_ref - real(1));
  const real dth = th - d.theta_ref;
  const real dp = cs2 * (dr * th + d.rho_ref * dth);
  const real drc = dp - cs2 * dr;
  const real drc2 = dr * c * c + d.rho_ref * (cs2 * dth) * (c + cref);
  const real Axx = rho * U * U + drc + a1xx;
  const real Ayy = drc + a1yy;
  const real Axy = a1xy;
  const real Axxy = a1xxy;
  const real Axyy = rc * U + a1xyy;
  const real Axxyy = (d.flags & kFlagFeq3) ? real(0) : rc * U * U + drc2 + a1xxyy;
  real f[kQ];
  project(dr, rho * U, real(0), Axx, Axy, Ayy, Axxy, Axyy, Axxyy, f);
#pragma unroll
  for (int q = 0; q < kQ; ++q) F[q] = f[q];
  // s_w - s_ref = c_v (ln(theta_w / theta_ref) - (gamma - 1) ln(rho_w / rho_ref))
  F[9] = (log_r(th) - log_r(d.theta_ref) - d.gm1 * (log_r(rho) - d.log_rho_ref)) / d.inv_cv;
}

__device__ __forceinline__ void wall_node(const WallArgs &a, const int t) {
  const DomainArgs &d = a.d;
  const int side = t >= d.nx ? 1 : 0;
  const int x = t - side * d.nx;
  const int yw = side ? d.ny - 1 : 0, dir = side ? -1 : 1;
  const long long P = d.plane;
  real *node = a.state + (long long)yw * d.pitch + x;
  real F[kPlanes];
#pragma unroll
  for (int q = 0; q < kQ; ++q) F[q] = node[q * P];
  auto velocity = [&](int y, real &ux, real &uy) {
    const real *p = a.state + (long long)y * d.pitch + x;
    real G[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) G[q] = p[q * P];
    const NodeMoments m = node_moments(G, d);
    ux = m.jx / m.rho;
    uy = m.jy / m.rho;
  };
  real u1x, u1y, u2x, u2y;
  velocity(yw + dir, u1x, u1y);
  velocity(yw + 2 * dir, u2x, u2y);
  wall_rebuild(d, side, F, u1x, u1y, u2x, u2y);
#pragma unroll
  for (int q = 0; q < kPlanes; ++q) node[q * P] = F[q];
}

__global__ void k_wall(WallArgs a) {
  const int n = 2 * a.d.nx;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x)
    wall_node(a, t);
}

}  // namespace HLBM_NS
}  // namespace hlbm

#include "hlbm_resident.hpp"

namespace hlbm {
namespace HLBM_NS {

// ------------------------------------------------------------ moments
struct FieldArgs {
  DomainArgs d;
  const real *state;
  real *rho, *ux, *uy, *s, *theta;
};

__global__ void k_moments(FieldArgs a) {
  const DomainArgs &d = a.d;
  const long long n = (long long)d.nx * d.ny, P = d.plane;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const long long o = state_off(d, i);
    real F[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) F[q] = a.state[q * P + o];
    const real sv = a.state[9 * P + o];
    const NodeMoments m = node_moments(F, d);
    if (a.rho) a.rho[i] = m.rho;
    if (a.ux) a.ux[i] = m.jx / m.rho;
    if (a.uy) a.uy[i] = m.jy / m.rho;
    if (a.s) a.s[i] = sv + d.s_ref;
    if (a.theta) a.theta[i] = field_theta(m.rho, sv, d);
  }
}

// Absolute populations out / in.
struct PopArgs {
  DomainArgs d;
  real *state;
  real *F9;
  real *s;
  int to_state;
};

__global__ void k_populations(PopArgs a) {
  const DomainArgs &d = a.d;
  const long long n = (long long)d.nx * d.ny, P = d.plane;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const long long o = state_off(d, i);
    if (a.to_state) {
#pragma unroll
      for (int q = 0; q < kQ; ++q) a.state[q * P + o] = a.F9[q * n + i] - d.fref[q];
      a.state[9 * P + o] = a.s[i] - d.s_ref;
    } else {
#pragma unroll
      for (int q = 0; q < kQ; ++q) a.F9[q * n + i] = a.state[q * P + o] + d.fref[q];
    }
  }
}

// ------------------------------------------------------- reductions
// Per-workgroup FP64 partials of {mass, mom x, mom y, energy, bad, max CFL}.
constexpr int kRedThreads = 256;
constexpr int kRedVals = 6;

struct ReduceArgs {
  DomainArgs d;
  const real *state;
  double *partials;  // [gridDim.x][kRedVals]
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

__global__ __launch_bounds__(kRedThreads) void k_reduce(ReduceArgs a) {
  const DomainArgs &d = a.d;
  const long long n = (long long)d.nx * d.ny, P = d.plane;
  const double cv = kCs2 / (double)d.gm1;
  double acc[kRedVals] = {0, 0, 0, 0, 0, 0};
  // Fixed per-thread assignment and fixed combine order: deterministic.
  for (long long i = blockIdx.x * (long long)kRedThreads + threadIdx.x; i < n;
       i += (long long)gridDim.x * kRedThreads) {
    const long long o = state_off(d, i);
    real F[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) F[q] = a.state[q * P + o];
    const real sv = a.state[9 * P + o];
    const NodeMoments m = node_moments(F, d);
    const double rho = (double)m.rho;
    const double ux = (double)m.jx / rho, uy = (double)m.jy / rho;
    const double th = (double)field_theta(m.rho, sv, d);
    acc[0] += rho;
    acc[1] += (double)m.jx;
    acc[2] += (double)m.jy;
    acc[3] += rho * cv * th + 0.5 * rho * (ux * ux + uy * uy);
    const bool ok = rho > 0.0 && th > 0.0 && __builtin_isfinite(ux + uy + th + (double)sv);
    acc[4] += ok ? 0.0 : 1.0;
    const double cfl = ok ? sqrt(ux * ux + uy * uy) + sqrt((double)d.gamma * kCs2 * th) : 0.0;
    acc[5] = fmax(acc[5], cfl);
  }
  __shared__ double sm[kRedThreads / 64][kRedVals];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < kRedVals; ++k) {
    const double v = k == 5 ? wave_max(acc[k]) : wave_sum(acc[k]);
    if (lane == 0) sm[w][k] = v;
  }
  __syncthreads();
  if (threadIdx.x < kRedVals) {
    const int k = threadIdx.x;
    double v = sm[0][k];
    for (int ww = 1; ww < kRedThreads / 64; ++ww) v = k == 5 ? fmax(v, sm[ww][k]) : v + sm[ww][k];
    a.partials[(long long)blockIdx.x * kRedVals + k] = v;
  }
}

// Second pass: one workgroup combines the partials in a fixed order.
__global__ __launch_bounds__(kRedThreads) void k_reduce_final(const double *partials, int nparts,
                                                              double *out) {
  double acc[kRedVals] = {0, 0, 0, 0, 0, 0};
  for (int b = threadIdx.x; b < nparts; b += kRedThreads) {
#pragma unroll
    for (int k = 0; k < kRedVals; ++k) {
      const double v = partials[(long long)b * kRedVals + k];
      acc[k] = k == 5 ? fmax(acc[k], v) : acc[k] + v;
    }
  }
  __shared__ double sm[kRedThreads / 64][kRedVals];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < kRedVals; ++k) {
    const double v = k == 5 ? wave_max(acc[k]) : wave_sum(acc[k]);
    if (lane == 0) sm[w][k] = v;
  }
  __syncthreads();
  if (threadIdx.x < kRedVals) {
    const int k = threadIdx.x;
    double v = sm[0][k];
    for (int ww = 1; ww < kRedThreads / 64; ++ww) v = k == 5 ? fmax(v, sm[ww][k]) : v + sm[ww][k];
    out[k] = v;
  }
}

// s = c_v ln(theta / rho^(gamma-1)).
__global__ void k_entropy(const real *rho, const real *theta, real *s, long long n, real inv_cv,
                          real gm1) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    s[i] = (log_r(theta[i]) - gm1 * log_r(rho[i])) / inv_cv;
  }
}

}  // namespace HLBM_NS
}  // namespace hlbm
