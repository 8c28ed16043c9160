// What the two eigensolver files share: wave helpers, complex arithmetic, the reflector of a bulge
// step, and the hand-over of a sweep's reflectors from wave 0 to the waves that apply them to Z.
#pragma once

#include "vbrdf_internal.hpp"

namespace vbrdf {

constexpr double kUlp = 2.220446049250313e-16;
constexpr double kSafeMin = 2.2250738585072014e-308;

__device__ inline double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1)
    if (o < (int)blockDim.x) v += __shfl_xor(v, o);
  return v;
}
__device__ inline int wave_max(int v) {
  for (int o = 32; o > 0; o >>= 1)
    if (o < (int)blockDim.x) v = max(v, __shfl_xor(v, o));
  return v;
}
__device__ inline double block_sum(double v, double* sred) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) sred[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0.0;
  const int nw = (blockDim.x + 63) >> 6;
  for (int w = 0; w < nw; ++w) r += sred[w];
  __syncthreads();
  return r;
}

// Eigenvalues closer than this cannot be told apart in a matrix of Frobenius norm hnorm: copies of one multiple
// eigenvalue, whose couplings are rounding noise.
__device__ inline double same_eigenvalue(double hnorm) { return 8.0 * kUlp * hnorm; }

// Whether a 2 x 2 block with off-diagonal entries b, c and a complex pair of imaginary part im is two such copies
// whose noise couples them in one direction only (c = 1e-140 beside b = 1e-13 in orders with next to no
// scattering). Taken as a pair, its eigenvector would have real and imaginary parts parallel to im / |b| (1e-60: a
// singular eigenvector matrix, and a response of 1e10 for one of 1e-15); real eigenvalues with the
// coupling dropped are as close to the matrix. Other blocks of copies have im / |b| above 1e-3, but for one in
// 1e5 orders or so.
__device__ inline bool uncoupled_copies(double b, double c, double im, double hnorm) {
  const double most = fmax(fabs(b), fabs(c));
  return most <= same_eigenvalue(hnorm) && im <= 1e-6 * most;
}

struct Cx {
  double re, im;
};
__device__ inline Cx cmul(Cx a, Cx b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ inline Cx csub(Cx a, Cx b) { return {a.re - b.re, a.im - b.im}; }
__device__ inline double cabs1(Cx a) { return fabs(a.re) + fabs(a.im); }
__device__ inline Cx cdiv(Cx a, Cx b) {
  // Smith's algorithm
  if (fabs(b.re) >= fabs(b.im)) {
    double r = b.im / b.re, d = b.re + b.im * r;
    return {(a.re + a.im * r) / d, (a.im - a.re * r) / d};
  }
  double r = b.re / b.im, d = b.im + b.re * r;
  return {(a.re * r + a.im) / d, (a.im * r - a.re) / d};
}
__device__ inline Cx cguard(Cx d, double smin) {
  if (cabs1(d) < smin) return {smin, 0.0};
  return d;
}

// Solve the 2x2 complex system [[a, b], [c, d]] x = r by Gaussian elimination with pivoting;
// tiny pivots are replaced by smin (perturbation in the style of LAPACK's eigenvector solver).
__device__ inline void csolve2(Cx a, Cx b, Cx c, Cx d, Cx r0, Cx r1, double smin, Cx& x0, Cx& x1) {
  if (cabs1(a) >= cabs1(c)) {
    a = cguard(a, smin);
    Cx f = cdiv(c, a);
    Cx d2 = cguard(csub(d, cmul(f, b)), smin);
    Cx s1 = csub(r1, cmul(f, r0));
    x1 = cdiv(s1, d2);
    x0 = cdiv(csub(r0, cmul(b, x1)), a);
  } else {
    Cx f = cdiv(a, c);
    Cx b2 = cguard(csub(b, cmul(f, d)), smin);
    Cx s0 = csub(r0, cmul(f, r1));
    x1 = cdiv(s0, b2);
    x0 = cdiv(csub(r1, cmul(d, x1)), c);
  }
}

// Orders LDS (and global) accesses of different lanes of one wave: a wave's memory operations
// execute in order, so a compiler scheduling barrier is all the hand-off needs.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Action codes of the QR driver (sctl[4]).
enum : int { kActDeflated = 0, kActSweep = 1, kActRotate = 2, kActStop = 3, kActMulti = 4 };

// Z-update descriptor of one QR iteration, produced by wave 0 and applied by the other waves
// during the next iteration (double-buffered): kind 0 none, 1 sweep (reflectors of steps lo..hh-1
// as (tau, u1, u2) triples in the slot's reflector buffer), 2 rotation of columns hh-1, hh by
// (cs, sn) stored at the start of the reflector buffer. `stop` ends the QR loop after this
// iteration; it lives in the double-buffered slot so that wave 0 cannot overwrite it (in the
// next iteration) before every wave has read it.
struct ZOp {
  int kind, lo, hh, stop, nb;  // nb > 0: multi-bulge pass over lo..hh with nb bulges (no Z op)
};

// Applies the reflectors of a sweep over lo..hh (rf[3 k .. 3 k + 2] = (tau, u1, u2) of step k; the
// last one has two elements) to the line e(k) = L[k st], k = lo..hh: a row of Z or of H from the
// right, or a column of H from the left (the reflectors are symmetric, so both read the same).
__device__ __forceinline__ void sweep_line(const double* rf, double* __restrict__ L, int64_t st, int lo, int hh) {
  double z0 = L[(int64_t)lo * st], z1 = L[(int64_t)(lo + 1) * st];
  for (int k0 = lo; k0 <= hh - 1; k0 += 8) {
    double zb[8];  // entries of the next 8 steps, loaded ahead (not yet written)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int c = k0 + 2 + j;
      zb[j] = (c <= hh) ? L[(int64_t)c * st] : 0.0;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = k0 + j;
      if (k <= hh - 1) {
        const bool three = k < hh - 1;
        double z2 = three ? zb[j] : 0.0;
        const double tau = rf[3 * k];
        if (tau != 0.0) {
          const double u1 = rf[3 * k + 1], u2 = rf[3 * k + 2];
          const double w = tau * (z0 + u1 * z1 + (three ? u2 * z2 : 0.0));
          z0 -= w;
          z1 -= w * u1;
          if (three) z2 -= w * u2;
        }
        L[(int64_t)k * st] = z0;
        z0 = z1;
        z1 = z2;
      }
    }
  }
  L[(int64_t)hh * st] = z0;
}

// Reflector (I - tau u u^T), u = (1, u1, u2), taking (x, y, z) to (beta, 0, 0),
// beta = -sign(x) ||(x, y, z)||; the identity (tau = 0, beta = x) when y = z = 0.
__device__ __forceinline__ void householder3(double x, double y, double z, double& tau, double& u1, double& u2,
                                             double& beta) {
  tau = 0.0;
  u1 = 0.0;
  u2 = 0.0;
  beta = x;
  if (y == 0.0 && z == 0.0) return;
  double xs = x, ys = y, zs = z, unscale = 1.0;
  double s2 = xs * xs + ys * ys + zs * zs;
  if (s2 < 0x1p-900) {  // keep the squares clear of the subnormal range
    xs *= 0x1p600;
    ys *= 0x1p600;
    zs *= 0x1p600;
    unscale = 0x1p-600;
    s2 = xs * xs + ys * ys + zs * zs;
  }
  double r = __builtin_amdgcn_rsq(s2);
  const double h2 = 0.5 * s2;
  r = r * fma(-h2 * r, r, 1.5);
  r = r * fma(-h2 * r, r, 1.5);
  const double nrm = s2 * r;
  const double ax = fabs(xs);
  tau = fma(ax, r, 1.0);
  const double dd = ax + nrm;
  double q = __builtin_amdgcn_rcp(dd);
  q = fma(q, fma(-dd, q, 1.0), q);
  q = fma(q, fma(-dd, q, 1.0), q);
  const double sc = copysign(q, xs);
  u1 = ys * sc;
  u2 = zs * sc;
  beta = -copysign(nrm, xs) * unscale;
}

}  // namespace vbrdf
