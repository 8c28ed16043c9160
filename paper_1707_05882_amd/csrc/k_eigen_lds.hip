// Eigensolver of the systems of at most kLdsMaxn rows (Sec. 3.A, eq. 43-45), the whole Hessenberg
// matrix in LDS: Householder reduction in registers, multi-bulge and single double-shift QR, eigenvectors
// of the quasi-triangular factor. Same steps, deflation tests, shifts and output conventions as the
// form for larger systems (k_eigen.hip); one workgroup of 8 waves per system.
//
// The solver is a chain of short dependent steps, and with one problem per compute unit their
// latency is its time. Cycles of one system of n = 128 (n = 32) by phase, before -> now:
//   reduction                       1.52 M -> 0.89 M   (0.20 M -> 0.12 M)
//   decisions and single sweeps     1.7 M  -> 0.91 M   (0.8 M  -> 0.22 M)
//   multi-bulge passes              4.1 M  -> 3.1 M    (0.15 M -> 0.33 M, now for 20 rows and more)
//   eigenvectors                    0.70 M -> 0.41 M   (0.11 M -> 0.05 M)
//   in all                          8.1 M  -> 5.6 M    (1.25 M -> 0.78 M; n = 64: 2.65 M -> 1.82 M)
// Before: reduction in LDS, barriers around every deflation, a multi-bulge step that waited for its columns
// of Z and read its reflector's input and wrote its zeros through LDS, eight bulges or none.
#include <type_traits>

#include "eigen_common.hpp"

namespace vbrdf {

constexpr int kLd = kLdsMaxn + 1;           // row stride of H in LDS
constexpr int kTail = kLdsMaxn * kLd;       // three private doubles per lane lie behind the matrix
constexpr int kBulgeGap = 4;                // rows between the bulges of a pass
constexpr int kBulges = kEigenThreads / 64;  // one bulge per wave
// Multi-bulge passes run while the active block has at least kPassMin rows and fewer than kPassIts
// iterations have gone by without a deflation. A pass costs nearly the same per bulge for 4 bulges as for
// 8, and fewer of them fit a small block: 8 from 48 rows on, 6 from 32, 4 below (n = 32: 1.07 -> 0.93 M
// cycles against single sweeps below 32 rows; 12 against 6 iterations: n = 128 6.24 -> 6.08 M).
constexpr int kPassMin = 20, kPassIts = 12;

struct EigenLds {
  double H[kTail + 3 * 64];
  double refl[2 * 3 * kLdsMaxn];  // reflectors or shifts of the current and of the last iteration
  double lre[kLdsMaxn], lim[kLdsMaxn];
  double red[16];
  int blk[kLdsMaxn];  // block sizes of the quasi-triangular factor (2 at a pair's first row, 0 at its second)
  ZOp zops[2];
  int fail;
};

// Sum over the 16 lanes of a DPP row, in every lane.
__device__ inline double dpp_row_sum(double x) {
  auto ror = [](double v, auto n) {
    constexpr int ctrl = 0x120 + decltype(n)::value;  // row_ror:n
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, ctrl, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), ctrl, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
  };
  x += ror(x, std::integral_constant<int, 8>{});
  x += ror(x, std::integral_constant<int, 4>{});
  x += ror(x, std::integral_constant<int, 2>{});
  x += ror(x, std::integral_constant<int, 1>{});
  return x;
}

// x of lane l (uniform), in every lane.
__device__ __forceinline__ double lane_value(double x, int l) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Householder reduction to Hessenberg form of a system of at most 16 kR = 32 kC rows, with the matrix in
// registers. Held in LDS, a step's two-sided update reads the matrix four times and writes it twice
// and is bound by the LDS rate (12000 cycles a step at n = 128, a fifth of the eigensolver). Here a
// thread keeps rows tr + 16 i, columns tc + 32 j (tr < 16, tc < 32) in kR kC doubles, both products
// w = A^T v and y = A v come from one pass over them, and the update
//     H A H = A - v p^T - q v^T,  p = tau w - (tau^2 s / 2) v,  q = tau y - (tau^2 s / 2) v,  s = v^T A v
// is one more. A wave holds all rows of 4 kC columns, so w is summed over rows of 16 lanes, and y over
// 4 lanes and then over the 8 waves through LDS. No block is left out where v is zero: the branches
// cost more than the operations (n = 128: 0.89 M cycles, 1.10 M with the branches, 1.52 M in LDS).
// G: the matrix; H: LDS, receives the Hessenberg matrix (and holds the vectors before); QV: v_k and tau_k
// as the other reductions; sq[wave]: the wave's part of ||G||_F^2.
template <int kR, int kC>
__device__ __forceinline__ void reg_hessenberg(const double* __restrict__ G, int n, double* __restrict__ QV, double* H,
                                               double* sq) {
  static_assert(kEigenThreads == 512, "16 x 32 threads");
  constexpr int kN = 16 * kR;
  static_assert(kN == 32 * kC && kN % 64 == 0, "whole waves per vector");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tr = lane & 15, tcl = lane >> 4, tc = 4 * wave + tcl;
  double* sv = H;             // [2][kN]: v of the current and of the next step
  double* sw = H + 2 * kN;    // [kN]: w
  double* yq = H + 3 * kN;    // [kN]: y
  double* sy = H + 4 * kN;    // [8][kN]: the waves' parts of y
  double* ss = H + 12 * kN;   // [8]: the waves' parts of s
  double* st = H + 12 * kN + 8;  // [2]: tau
  double a[kR][kC];
#pragma unroll
  for (int i = 0; i < kR; ++i)
#pragma unroll
    for (int j = 0; j < kC; ++j) a[i][j] = G[(int64_t)min(tr + 16 * i, n - 1) * n + min(tc + 32 * j, n - 1)];
  double part = 0.0;
#pragma unroll
  for (int i = 0; i < kR; ++i)
#pragma unroll
    for (int j = 0; j < kC; ++j) {
      if (tr + 16 * i >= n || tc + 32 * j >= n) a[i][j] = 0.0;
      part += a[i][j] * a[i][j];
    }
  part = wave_sum(part);
  if (lane == 0) sq[wave] = part;
  // v and tau of step k from column k, by the wave that holds it; the column takes its final form
  auto produce = [&](int k) __attribute__((always_inline)) {
    if (wave != ((k & 31) >> 2)) return;  // uniform
    double* v = sv + (k & 1) * kN;
    double x[kR], on[kC];  // the column by weights 0 and 1: selected by index, the matrix would leave the registers
#pragma unroll
    for (int j = 0; j < kC; ++j) on[j] = (k >> 5) == j ? 1.0 : 0.0;
#pragma unroll
    for (int i = 0; i < kR; ++i) {
      x[i] = a[i][0] * on[0];
#pragma unroll
      for (int j = 1; j < kC; ++j) x[i] += a[i][j] * on[j];
    }
    double sig = 0.0, x0 = 0.0;
#pragma unroll
    for (int i = 0; i < kR; ++i) {
      const int r = tr + 16 * i;
      sig += r > k + 1 ? x[i] * x[i] : 0.0;
      x0 += r == k + 1 ? x[i] : 0.0;
    }
    sig = dpp_row_sum(sig);
    x0 = dpp_row_sum(x0);
    // beta = -sign(x0) ||.||, tau = 1 + |x0| / ||.||, 1 / (x0 - beta) = sign(x0) / (|x0| + ||.||)
    const bool none = sig == 0.0;  // already reduced
    const double s2 = none ? 1.0 : x0 * x0 + sig;
    double r = __builtin_amdgcn_rsq(s2);
    const double h2 = 0.5 * s2;
    r = r * fma(-h2 * r, r, 1.5);
    r = r * fma(-h2 * r, r, 1.5);
    const double nrm = s2 * r, ax = fabs(x0), dd = ax + nrm;
    double q = __builtin_amdgcn_rcp(dd);
    q = fma(q, fma(-dd, q, 1.0), q);
    q = fma(q, fma(-dd, q, 1.0), q);
    const double tau = none ? 0.0 : fma(ax, r, 1.0), scal = none ? 0.0 : copysign(q, x0);
    const double beta = none ? x0 : -copysign(nrm, x0);
    if (tcl != (k & 3)) return;
    if (tr == 0) {
      st[k & 1] = tau;
      QV[(int64_t)(n - 1) * n + k] = tau;
    }
#pragma unroll
    for (int i = 0; i < kR; ++i) {
      const int rr = tr + 16 * i;
      const double vr = rr <= k ? 0.0 : (rr == k + 1 ? 1.0 : x[i] * scal);
      v[rr] = vr;
      if (rr > k && rr < n) QV[(int64_t)k * n + rr - k - 1] = vr;
      const double e = rr <= k ? x[i] : (rr == k + 1 ? beta : 0.0);
#pragma unroll
      for (int j = 0; j < kC; ++j) a[i][j] = on[j] != 0.0 ? e : a[i][j];
    }
  };
  if (n > 2) produce(0);
  __syncthreads();
  for (int k = 0; k + 2 < n; ++k) {
    const double tau = st[k & 1];
    const double* v = sv + (k & 1) * kN;
    double vr[kR], vc[kC], w[kC], y[kR];
#pragma unroll
    for (int i = 0; i < kR; ++i) vr[i] = v[tr + 16 * i];
#pragma unroll
    for (int j = 0; j < kC; ++j) vc[j] = v[tc + 32 * j];
#pragma unroll
    for (int i = 0; i < kR; ++i) {
      y[i] = a[i][0] * vc[0];
#pragma unroll
      for (int j = 1; j < kC; ++j) y[i] += a[i][j] * vc[j];
    }
    // the lanes exchange halves, then quarters, of their sums; at the end a lane holds kR / 4 rows
    double h[kR / 2], q[kR / 4], sp = 0.0;
#pragma unroll
    for (int i = 0; i < kR / 2; ++i) {
      const bool up = tcl >> 1;
      const double keep = up ? y[i + kR / 2] : y[i], send = up ? y[i] : y[i + kR / 2];
      h[i] = keep + __shfl_xor(send, 32);
    }
#pragma unroll
    for (int j = 0; j < kC; ++j) w[j] = vr[0] * a[0][j];
#pragma unroll
    for (int i = 1; i < kR; ++i)
#pragma unroll
      for (int j = 0; j < kC; ++j) w[j] += vr[i] * a[i][j];
#pragma unroll
    for (int i = 0; i < kR; ++i) sp += vr[i] * y[i];
#pragma unroll
    for (int i = 0; i < kR / 4; ++i) {
      const bool up = tcl & 1;
      const double keep = up ? h[i + kR / 4] : h[i], send = up ? h[i] : h[i + kR / 4];
      q[i] = keep + __shfl_xor(send, 16);
    }
#pragma unroll
    for (int j = 0; j < kC; ++j) {
      w[j] = dpp_row_sum(w[j]);
      if (tr == j) sw[tc + 32 * j] = w[j];
    }
    sp = dpp_row_sum(sp);
    sp += __shfl_xor(sp, 16);
    sp += __shfl_xor(sp, 32);
    if (lane == 0) ss[wave] = sp;
    const int ib = (tcl >> 1) * (kR / 2) + (tcl & 1) * (kR / 4);
#pragma unroll
    for (int i = 0; i < kR / 4; ++i) sy[wave * kN + tr + 16 * (ib + i)] = q[i];
    __syncthreads();
    if (tid < kN) {
      double t[8];
#pragma unroll
      for (int x = 0; x < 8; ++x) t[x] = sy[x * kN + tid];
      yq[tid] = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
    }
    const double s = lane_value(dpp_row_sum(lane < 8 ? ss[lane] : 0.0), 0);
    const double half = 0.5 * tau * tau * s;
    double p[kC];  // columns up to k have their final form
#pragma unroll
    for (int j = 0; j < kC; ++j) p[j] = tc + 32 * j > k ? tau * sw[tc + 32 * j] - half * vc[j] : 0.0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kR; ++i) {
      const double qi = tau * yq[tr + 16 * i] - half * vr[i];
#pragma unroll
      for (int j = 0; j < kC; ++j) a[i][j] -= qi * vc[j] + vr[i] * p[j];
    }
    if (k + 3 < n) produce(k + 1);
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < kR; ++i)
#pragma unroll
    for (int j = 0; j < kC; ++j) {
      const int r = tr + 16 * i, c = tc + 32 * j;
      if (r < n && c < n) H[r * kLd + c] = a[i][j];
    }
  __syncthreads();
}

// The three-element steps of a double-shift sweep over rows/columns lo..hh of an n x n matrix in LDS, run
// by one wave: x, y, z carry the reflector's input from step to step, rf[3 k .. 3 k + 2] receives (tau, u1,
// u2) of step k. A step touches rows k..k+2 (columns >= k) and columns k..k+2 (rows <= k+3); every lane
// loads the 4 x 3 corner these share and updates it itself, and so holds the next input. The rest is n - 3
// uniform jobs of three elements: job j < n - k - 3 is column k + 3 + j (rows k..k+2, from the left), the
// others are rows 0..k-1 (columns k..k+2, from the right). A lane takes job lane and, for n > 67 (kTwo),
// lane + 64; idle ones work on the private slot dum.
template <bool kTwo>
__device__ __forceinline__ void lds_sweep(double* __restrict__ H, int n, int lo, int hh, double& x, double& y, double& z,
                                          double* rf, int lane, int dum) {
  const int ja = lane, jb = lane + 64;
  for (int k = lo; k < hh - 1; ++k) {
    const int kb = k * (kLd + 1);
    double b[4][3];  // rows k..k+3, columns k..k+2 (row k+3 is unused when k+3 > hh)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) b[i][j] = H[kb + i * kLd + j];
    const bool cola = k < n - 3 - ja;
    const int ia = ja >= n - 3 ? dum : (cola ? kb + 3 + ja : kb + (ja - n + 3) * kLd);
    const int sa = ja < n - 3 && cola ? kLd : 1;
    double va[3], vb[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) va[i] = H[ia + i * sa];
    const bool colb = k < n - 3 - jb;
    const int ib = jb >= n - 3 ? dum : (colb ? kb + 3 + jb : kb + (jb - n + 3) * kLd);
    const int sb = jb < n - 3 && colb ? kLd : 1;
    if (kTwo)
#pragma unroll
      for (int i = 0; i < 3; ++i) vb[i] = H[ib + i * sb];
    wave_sync();  // all loads of the step precede its stores
    double tau, u1, u2, beta;
    householder3(x, y, z, tau, u1, u2, beta);
    {
      const double w = tau * (va[0] + u1 * va[1] + u2 * va[2]);
      H[ia] = va[0] - w;
      H[ia + sa] = va[1] - w * u1;
      H[ia + 2 * sa] = va[2] - w * u2;
    }
    if (kTwo) {
      const double w = tau * (vb[0] + u1 * vb[1] + u2 * vb[2]);
      H[ib] = vb[0] - w;
      H[ib + sb] = vb[1] - w * u1;
      H[ib + 2 * sb] = vb[2] - w * u2;
    }
    // corner: rows k..k+2 from the left, then rows k..k+3 from the right
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const double w = tau * (b[0][j] + u1 * b[1][j] + u2 * b[2][j]);
      b[0][j] -= w;
      b[1][j] -= w * u1;
      b[2][j] -= w * u2;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double w = tau * (b[i][0] + u1 * b[i][1] + u2 * b[i][2]);
      b[i][0] -= w;
      b[i][1] -= w * u1;
      b[i][2] -= w * u2;
    }
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) H[kb + i * kLd + j] = b[i][j];
      if (k + 3 <= hh) {
#pragma unroll
        for (int j = 0; j < 3; ++j) H[kb + 3 * kLd + j] = b[3][j];
      }
      if (k > lo) {
        H[kb - 1] = beta;
        H[kb - 1 + kLd] = 0.0;
        H[kb - 1 + 2 * kLd] = 0.0;
      }
      rf[3 * k] = tau;
      rf[3 * k + 1] = u1;
      rf[3 * k + 2] = u2;
    }
    wave_sync();
    x = b[1][0];
    y = b[2][0];
    z = b[3][0];
  }
}

// Multi-bulge pass over rows/columns lo..hh of an n x n matrix held in LDS (n <= 128), with Z (Z(r, c) at
// ZT[c n + r]) in global memory: wave b chases bulge b (shift pair sh[4 b .. 4 b + 3]) kBulgeGap rows behind bulge b - 1. A chain step moves every bulge one row: each
// wave forms its reflector (from column k - 1, or from the shift polynomial when it enters at row lo),
// applies it from the left to rows k..k+2, then after a barrier from the right to columns k..k+2 of H
// and Z. Rows of different bulges in a left phase and columns in a right phase are disjoint, and a
// bulge's reflector input is not touched by the neighbours within a step (gap >= 4). The step is
// bound by the rate of the LDS (about 8 cycles for each 64-lane access of 8 bytes, eight waves at a
// time): a lane takes up to two lines per phase, with idle lanes on a private slot dum, the
// reflector's input comes from the lane that has column k - 1, and that lane also stores beta and the zeros.
// The wave's three columns of Z (rows lane and lane + 64) stay in registers from step to step: after a
// step column k is final for this bulge and is stored, and column k + 3, loaded at the start of the
// step, joins the other two (the bulge ahead, on k + 4..k + 6, stored it one step before).
// Measured at n = 128: 1.7 k cycles a step with eight bulges, 12.8 passes of 130 to 150 steps.
__device__ __forceinline__ void lds_multibulge(double* __restrict__ H, int n, double* __restrict__ ZT, int lo, int hh,
                                               int nb, const double* sh, int dum) {
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nsteps = (hh - lo) + kBulgeGap * (nb - 1);
  // lanes beyond the matrix carry its last row along, so that no load or store of Z needs a predicate
  const int zr0 = min(lane, n - 1), zr1 = min(lane + 64, n - 1);
  struct Z2 {
    double a, b;
  };
  auto zload = [&](int c) __attribute__((always_inline)) {
    return Z2{ZT[(int64_t)c * n + zr0], ZT[(int64_t)c * n + zr1]};
  };
  auto zstore = [&](int c, double a, double b) __attribute__((always_inline)) {
    ZT[(int64_t)c * n + zr0] = a;
    ZT[(int64_t)c * n + zr1] = b;
  };
  // za, zb, zc: columns k..k + 2 of Z; zd receives column k + 3. The caller rotates the four by name: a
  // copy from one to the next would wait for the load.
  auto step = [&](int t, Z2& za, Z2& zb, Z2& zc, Z2& zd) __attribute__((always_inline)) {
    const int k = lo + t - kBulgeGap * wv;
    const bool on = wv < nb && k >= lo && k <= hh - 1;  // uniform
    const bool three = k < hh - 1;
    double tau = 0.0, u1 = 0.0, u2 = 0.0, beta = 0.0;
    if (wv < nb && k == lo - 1) {  // the bulge enters at the next step (columns lo.. are with the bulge ahead no more)
      zb = zload(lo);
      zc = zload(lo + 1);
      zd = zload(lo + 2);
    }
    if (on) {
      if (t == 0) {  // the first bulge
        za = zload(lo);
        zb = zload(lo + 1);
        zc = zload(lo + 2);
      }
      zd = zload(min(k + 3, hh));
      // columns c0 + lane and 64 further, c0 = k - 1: that column holds the reflector's input and takes
      // (beta, 0, 0). At k = 0 there is none, and the lanes have just the 128 columns to cover.
      const int c0 = max(k - 1, 0), ca = c0 + lane, cb = ca + 64;
      const bool one = c0 + 64 < n;  // some lane has a second column
      const int ia = ca < n ? k * kLd + ca : dum, sa = ca < n ? kLd : 1;
      const int ib = cb < n ? k * kLd + cb : dum, sb = cb < n ? kLd : 1;
      double va[3], vb[3];
      va[0] = H[ia];
      va[1] = H[ia + sa];
      va[2] = three ? H[ia + 2 * sa] : 0.0;
      if (one) {
        vb[0] = H[ib];
        vb[1] = H[ib + sb];
        vb[2] = three ? H[ib + 2 * sb] : 0.0;
      }
      double x, y, z;
      if (k == lo) {
        const double s1r = sh[4 * wv], s1i = sh[4 * wv + 1], s2r = sh[4 * wv + 2], s2i = sh[4 * wv + 3];
        const double a0 = H[lo * kLd + lo], a1 = H[(lo + 1) * kLd + lo];
        const double rs = __builtin_amdgcn_rcp(fabs(a0 - s2r) + fabs(s2i) + fabs(a1));  // any scale will do
        const double a1s = a1 * rs;
        x = a1s * H[lo * kLd + lo + 1] + (a0 - s1r) * ((a0 - s2r) * rs) - s1i * (s2i * rs);
        y = a1s * (a0 + H[(lo + 1) * kLd + lo + 1] - s1r - s2r);
        z = a1s * H[(lo + 2) * kLd + lo + 1];
      } else {
        x = lane_value(va[0], 0);
        y = lane_value(va[1], 0);
        z = lane_value(va[2], 0);
      }
      wave_sync();  // all reads of the phase precede its stores
      householder3(x, y, z, tau, u1, u2, beta);
      const bool in = lane == 0 && k > lo && tau != 0.0;
      {
        const double w = tau * (va[0] + u1 * va[1] + u2 * va[2]);
        H[ia] = in ? beta : va[0] - w;
        H[ia + sa] = in ? 0.0 : va[1] - w * u1;
        if (three) H[ia + 2 * sa] = in ? 0.0 : va[2] - w * u2;
      }
      if (one) {
        const double w = tau * (vb[0] + u1 * vb[1] + u2 * vb[2]);
        H[ib] = vb[0] - w;
        H[ib + sb] = vb[1] - w * u1;
        if (three) H[ib + 2 * sb] = vb[2] - w * u2;
      }
    }
    __syncthreads();
    if (on) {
      const int rmax = min(k + 3, hh);
      const int ia = lane <= rmax ? lane * kLd + k : dum, ib = lane + 64 <= rmax ? (lane + 64) * kLd + k : dum;
      double va[3], vb[3];
      va[0] = H[ia];
      va[1] = H[ia + 1];
      va[2] = three ? H[ia + 2] : 0.0;
      if (rmax >= 64) {
        vb[0] = H[ib];
        vb[1] = H[ib + 1];
        vb[2] = three ? H[ib + 2] : 0.0;
      }
      wave_sync();
      {
        const double w = tau * (va[0] + u1 * va[1] + u2 * va[2]);
        H[ia] = va[0] - w;
        H[ia + 1] = va[1] - w * u1;
        if (three) H[ia + 2] = va[2] - w * u2;
      }
      if (rmax >= 64) {
        const double w = tau * (vb[0] + u1 * vb[1] + u2 * vb[2]);
        H[ib] = vb[0] - w;
        H[ib + 1] = vb[1] - w * u1;
        if (three) H[ib + 2] = vb[2] - w * u2;
      }
      const double zc0 = three ? zc.a : 0.0, zc1 = three ? zc.b : 0.0;
      const double w0 = tau * (za.a + u1 * zb.a + u2 * zc0), w1 = tau * (za.b + u1 * zb.b + u2 * zc1);
      zb.a -= w0 * u1;
      zb.b -= w1 * u1;
      zstore(k, za.a - w0, za.b - w1);
      if (three) {
        zc.a -= w0 * u2;
        zc.b -= w1 * u2;
      } else {
        zstore(k + 1, zb.a, zb.b);
      }
    }
    __syncthreads();
  };
  Z2 z0{0.0, 0.0}, z1 = z0, z2 = z0, z3 = z0;
  for (int t = 0; t < nsteps; t += 4) {
    step(t, z0, z1, z2, z3);
    if (t + 1 < nsteps) step(t + 1, z1, z2, z3, z0);
    if (t + 2 < nsteps) step(t + 2, z2, z3, z0, z1);
    if (t + 3 < nsteps) step(t + 3, z3, z0, z1, z2);
  }
}

// Iteration of wave 0: deflations until something is to be done, then that: a rotation that splits a real
// 2 x 2 block, a single sweep, the shifts of a multi-bulge pass, or the end. Every lane decides for itself from
// the same values; hh, its and tot are the state. op receives what the other waves have to do next.
struct QrState {
  int hh, its, tot;  // bottom of the active block, iterations since the last deflation and in all
};

__device__ __forceinline__ void qr_decide(EigenLds& s, int n, QrState& q, double hnorm, int sweep_cap, double* rf,
                                          ZOp* op, int lane) {
  double* H = s.H;
#define HH(r, c) H[(r) * kLd + (c)]
  for (;;) {
    const int hh = q.hh;
    if (hh < 0) {
      if (lane == 0) *op = ZOp{0, 0, 0, 1, 0};
      return;
    }
    // the lowest negligible subdiagonal entry, scanned from the bottom 64 rows at a time
    int l = 0;
    double t11 = 0.0, t12 = 0.0, t21 = 0.0, t22 = 0.0;  // the trailing 2 x 2 block
    for (int top = hh; top >= 0; top -= 64) {
      const int k = top - lane, kk = max(k, 1);
      const double hks = HH(kk, kk - 1), hus = HH(kk - 1, kk), d0 = HH(kk, kk), d1 = HH(kk - 1, kk - 1);
      if (top == hh) {
        t11 = lane_value(d1, 0);
        t12 = lane_value(hus, 0);
        t21 = lane_value(hks, 0);
        t22 = lane_value(d0, 0);
      }
      const double hk = fabs(hks);
      bool small = hk <= kSafeMin || (q.its >= 40 && hk <= kUlp * hnorm);
      double tst = fabs(d1) + fabs(d0);
      if (tst == 0.0) {
        if (kk >= 2) tst += fabs(HH(kk - 1, kk - 2));
        if (kk + 1 <= hh) tst += fabs(HH(kk + 1, kk));
      }
      if (!small && hk <= kUlp * tst) {
        const double hu = fabs(hus);
        const double ab = fmax(hk, hu), ba = fmin(hk, hu);
        const double dd = fabs(d1 - d0);
        const double aa = fmax(fabs(d0), dd), bb = fmin(fabs(d0), dd);
        const double sum = aa + ab;
        small = ba * (ab / sum) <= fmax(kSafeMin, kUlp * (bb * (aa / sum)));
      }
      const unsigned long long hit = __ballot(k >= 1 && small);  // the lowest lane holds the lowest entry
      if (hit) {
        l = top - __builtin_ctzll(hit);
        break;
      }
    }
    if (l > 0 && lane == 0) HH(l, l - 1) = 0.0;
    if (l == hh) {  // 1x1 block
      if (lane == 0) {
        s.lre[hh] = hh > 0 ? t22 : t11;
        s.lim[hh] = 0.0;
        s.blk[hh] = 1;
      }
      q.hh = hh - 1;
      q.its = 0;
      wave_sync();
      continue;
    }
    const double p = 0.5 * (t11 - t22), bc = t12 * t21, disc = p * p + bc;
    const double root = sqrt(fabs(disc));
    if (l == hh - 1) {
      const int h1 = hh - 1;
      if (disc < 0.0) {
        const bool copies = uncoupled_copies(t12, t21, root, hnorm);
        if (lane == 0) {
          if (copies) HH(hh, h1) = 0.0;
          s.lre[h1] = copies ? t11 : 0.5 * (t11 + t22);
          s.lre[hh] = copies ? t22 : 0.5 * (t11 + t22);
          s.lim[h1] = copies ? 0.0 : root;
          s.lim[hh] = copies ? 0.0 : -root;
          s.blk[h1] = copies ? 1 : 2;
          s.blk[hh] = copies ? 1 : 0;
        }
        q.hh = hh - 2;
        q.its = 0;
        wave_sync();
        continue;
      }
      // real pair: rotate the block to upper triangular form (first column = eigenvector of the first
      // eigenvalue) so that both become 1x1 blocks
      const double zz = p + copysign(root, p), l1 = t22 + zz;
      double v0 = t12, v1 = l1 - t11;
      if (fabs(l1 - t22) + fabs(t21) > fabs(v0) + fabs(v1)) {
        v0 = l1 - t22;
        v1 = t21;
      }
      const double big = fmax(fabs(v0), fabs(v1));
      double cs = 1.0, sn = 0.0;
      if (big > 0.0) {
        const double rb = 1.0 / big;
        v0 *= rb;
        v1 *= rb;
        const double rn = 1.0 / sqrt(v0 * v0 + v1 * v1);
        cs = v0 * rn;
        sn = v1 * rn;
      }
      wave_sync();
      for (int c = h1 + lane; c < n; c += 64) {
        const double x = HH(h1, c), y = HH(hh, c);
        HH(h1, c) = cs * x + sn * y;
        HH(hh, c) = -sn * x + cs * y;
      }
      wave_sync();
      for (int r = lane; r <= hh; r += 64) {
        const double x = HH(r, h1), y = HH(r, hh);
        HH(r, h1) = cs * x + sn * y;
        HH(r, hh) = -sn * x + cs * y;
      }
      wave_sync();
      if (lane == 0) {
        HH(hh, h1) = 0.0;
        s.lre[h1] = HH(h1, h1);
        s.lre[hh] = HH(hh, hh);
        s.lim[h1] = s.lim[hh] = 0.0;
        s.blk[h1] = s.blk[hh] = 1;
        rf[0] = cs;
        rf[1] = sn;
        *op = ZOp{2, 0, hh, 0, 0};
      }
      q.hh = hh - 2;
      q.its = 0;
      wave_sync();
      return;
    }
    const int its = ++q.its, tot = ++q.tot;
    if (its > 100 || tot > 60 * n || (sweep_cap > 0 && tot > sweep_cap)) {
      if (lane == 0) {
        s.fail = 1;
        *op = ZOp{0, 0, 0, 1, 0};
      }
      return;
    }
    const int rows = hh - l + 1;
    if (its < kPassIts && rows >= kPassMin) {
      // one shift pair per bulge: the eigenvalues of the 2x2 diagonal blocks ending at rows hh, hh - 2, ...
      // (both roots of a real pair)
      const int nb = rows >= 48 ? kBulges : (rows >= 32 ? 6 : 4);
      if (lane < nb) {
        const int j = hh - 2 * lane;
        const double a = HH(j - 1, j - 1), b = HH(j - 1, j), c = HH(j, j - 1), d = HH(j, j);
        const double pj = 0.5 * (a - d), bcj = b * c, dj = pj * pj + bcj, rj = sqrt(fabs(dj));
        double s1r, s2r, s1i = 0.0;
        if (dj >= 0.0) {
          const double zz = pj + copysign(rj, pj);
          s1r = d + zz;
          s2r = zz != 0.0 ? d - bcj / zz : d;
        } else {
          s1r = s2r = d + pj;
          s1i = rj;
        }
        rf[4 * lane] = s1r;
        rf[4 * lane + 1] = s1i;
        rf[4 * lane + 2] = s2r;
        rf[4 * lane + 3] = -s1i;
      }
      if (lane == 0) *op = ZOp{0, l, hh, 0, nb};
      return;
    }
    // single sweep. Shifts = eigenvalues of the trailing 2 x 2 block; a real pair is replaced by the root
    // closer to its last entry used twice (keeps the iteration from stagnating on real clusters).
    double h22 = t22, hp = p, hbc = bc, hdisc = disc, hroot = root;
    if (its % 10 == 0) {  // exceptional, from the top or the bottom of the block in turn
      const double e = its % 20 == 10 ? fabs(HH(l + 1, l)) + fabs(HH(l + 2, l + 1))
                                      : fabs(HH(hh, hh - 1)) + fabs(HH(hh - 1, hh - 2));
      h22 = 0.75 * e + (its % 20 == 10 ? HH(l, l) : HH(hh, hh));
      hp = 0.0;
      hbc = -0.4375 * e * e;
      hdisc = hbc;
      hroot = sqrt(fabs(hdisc));
    }
    double s1r, s1i = 0.0, s2r;
    if (hdisc >= 0.0) {
      const double zz = hp + copysign(hroot, hp);
      const double d1 = zz, d2 = zz != 0.0 ? -hbc / zz : 0.0;  // root - h22
      s1r = s2r = h22 + (fabs(d1) <= fabs(d2) ? d1 : d2);
    } else {
      s1r = s2r = h22 + hp;
      s1i = hroot;
    }
    wave_sync();
    // first column of (H - s1)(H - s2) at row l, in product form (no cancellation), at some scale
    const double a0 = HH(l, l), a1 = HH(l + 1, l);
    const double rs = __builtin_amdgcn_rcp(fabs(a0 - s2r) + fabs(s1i) + fabs(a1));
    const double a1s = a1 * rs;
    double x = a1s * HH(l, l + 1) + (a0 - s1r) * ((a0 - s2r) * rs) + s1i * (s1i * rs);
    double y = a1s * (a0 + HH(l + 1, l + 1) - s1r - s2r);
    double z = a1s * HH(l + 2, l + 1);
    if (n > 67)
      lds_sweep<true>(H, n, l, hh, x, y, z, rf, lane, kTail + 3 * lane);
    else
      lds_sweep<false>(H, n, l, hh, x, y, z, rf, lane, kTail + 3 * lane);
    // final two-element step on rows/columns hh - 1, hh
    const int k = hh - 1;
    double tau, u1, u2, beta;
    householder3(x, y, 0.0, tau, u1, u2, beta);
    if (tau != 0.0 && lane == 0) {
      HH(k, k - 1) = beta;
      HH(k + 1, k - 1) = 0.0;
    }
    for (int c = k + lane; c < n; c += 64) {
      const double h0 = HH(k, c), h1 = HH(k + 1, c), w = tau * (h0 + u1 * h1);
      HH(k, c) = h0 - w;
      HH(k + 1, c) = h1 - w * u1;
    }
    wave_sync();
    for (int r = lane; r <= hh; r += 64) {
      const double h0 = HH(r, k), h1 = HH(r, k + 1), w = tau * (h0 + u1 * h1);
      HH(r, k) = h0 - w;
      HH(r, k + 1) = h1 - w * u1;
    }
    if (lane == 0) {
      rf[3 * k] = tau;
      rf[3 * k + 1] = u1;
      rf[3 * k + 2] = 0.0;
      *op = ZOp{1, l, hh, 0, 0};
    }
    wave_sync();
    return;
  }
#undef HH
}

// Rows t0, t0 + nt, ... of Z (Z(r, c) at ZT[c n + r]) take the op of the iteration before.
__device__ __forceinline__ void apply_to_z(const ZOp& op, const double* rf, double* __restrict__ ZT, int n, int t0, int nt) {
  if (op.kind == 0) return;
  for (int r = t0; r < n; r += nt) {
    if (op.kind == 1) {
      sweep_line(rf, ZT + r, n, op.lo, op.hh);
    } else {
      const double cs = rf[0], sn = rf[1];
      double *a = ZT + (int64_t)(op.hh - 1) * n + r, *b = ZT + (int64_t)op.hh * n + r;
      const double x = *a, y = *b;
      *a = cs * x + sn * y;
      *b = -sn * x + cs * y;
    }
  }
}

// Component block [sb, i] (one row, or the two of a complex pair) of the eigenvector of lam = wr + i wi, from
// the row sums r0 (row sb) and r1 (row i); ts, ti: rows sb and i of T. Eigenvalues closer than `same` (a few
// ulp ||G||) cannot be told apart: a diagonal entry (or pair) that close to lam is another copy of the same
// multiple eigenvalue of a diagonalisable matrix (e.g. the unscattered Stokes components at one node,
// 1/mu^2), and its Schur coupling is rounding noise. Its component is zero instead of that noise divided
// by a guarded pivot, which would make the copies' eigenvectors parallel.
__device__ __forceinline__ void back_substitute(const EigenLds& s, int sb, int i, double tss, double tsi, double tis,
                                                double tii, double wr, double wi, Cx r0, Cx r1, double same, Cx& x0,
                                                Cx& x1) {
  const Cx lam{wr, wi};
  x0 = x1 = Cx{0.0, 0.0};
  const double smin = fmax(kUlp * (fabs(wr) + fabs(wi)), kSafeMin);
  if (sb == i) {
    const Cx d0{tii - wr, -wi};
    if (cabs1(d0) <= same) return;
    if (wi == 0.0)
      x1.re = r1.re / (fabs(d0.re) < smin ? smin : d0.re);
    else
      x1 = cdiv(r1, cguard(d0, smin));
  } else if (cabs1(csub(Cx{s.lre[sb], s.lim[sb]}, lam)) > same && cabs1(csub(Cx{s.lre[i], s.lim[i]}, lam)) > same) {
    csolve2(csub(Cx{tss, 0.0}, lam), Cx{tsi, 0.0}, Cx{tis, 0.0}, csub(Cx{tii, 0.0}, lam), r0, r1, smin, x0, x1);
  }
}

// The eigenvector's components in its own block: 1, or the eigenvector of the pair's 2 x 2 block.
__device__ __forceinline__ void own_block(double a, double b, double c, double d, double wr, double wi, bool first,
                                          Cx& x0, Cx& x1) {
  const Cx lam{wr, wi};
  const Cx v0a{b, 0.0}, v1a = csub(lam, Cx{a, 0.0});  // (b, lambda - a)
  const Cx v0b = csub(lam, Cx{d, 0.0}), v1b{c, 0.0};  // (lambda - d, c)
  const bool up = cabs1(v0a) + cabs1(v1a) >= cabs1(v0b) + cabs1(v1b);
  x0 = up ? v0a : v0b;
  x1 = up ? v1a : v1b;
  if (cabs1(x0) + cabs1(x1) == 0.0) {
    if (first)
      x0.re = 1.0;
    else
      x1.re = 1.0;
  }
}

// Eigenvectors of the quasi-triangular T, n <= 64: T stays in LDS and X (row stride 65) lies behind it; a group
// of 8 lanes takes one eigenvector (a complex pair's with its first column) from its own block up, with no
// barrier: the other groups of the wave run in step, the other waves on their own.
__device__ __forceinline__ void eigenvectors_small(EigenLds& s, int n, double same, double* __restrict__ XT) {
  constexpr int kLdx = 65, kLanes = 8;
  static_assert(64 * kLd + 64 * kLdx <= kTail, "T and X fit");
  const int tid = threadIdx.x;
  const double* T = s.H;
  double* X = s.H + 64 * kLd;
  for (int t = tid; t < 64 * kLdx; t += kEigenThreads) X[t] = 0.0;
  __syncthreads();
  const int j = tid / kLanes, part = tid % kLanes;
  const double wr = j < n ? s.lre[j] : 0.0, wi = j < n ? s.lim[j] : 0.0;
  const bool mine = j < n && wi >= 0.0;
  const bool cplx = mine && wi > 0.0;
  const int bend = cplx ? j + 1 : j;
  if (mine && part == 0) {
    if (cplx) {
      Cx x0, x1;
      own_block(T[j * kLd + j], T[j * kLd + j + 1], T[(j + 1) * kLd + j], T[(j + 1) * kLd + j + 1], wr, wi, true, x0, x1);
      X[j * kLdx + j] = x0.re;
      X[j * kLdx + j + 1] = x0.im;
      X[(j + 1) * kLdx + j] = x1.re;
      X[(j + 1) * kLdx + j + 1] = x1.im;
    } else {
      X[j * kLdx + j] = 1.0;
    }
  }
  wave_sync();
  const bool any = __any(cplx);
  const int jl = cplx ? j + 1 : j;  // column of the imaginary part
  for (int i = min(n, (tid / 64 + 1) * 8) - 1; i >= 0;) {
    const int sb = s.blk[i] == 0 ? i - 1 : i;
    const bool act = mine && i < j;
    double p0r = 0.0, p1r = 0.0, p0i = 0.0, p1i = 0.0;
    if (act)
      for (int c = i + 1 + part; c <= bend; c += kLanes) {
        const double ts = T[sb * kLd + c], ti = T[i * kLd + c], xr = X[c * kLdx + j], xi = X[c * kLdx + jl];
        p0r -= ts * xr;
        p1r -= ti * xr;
        p0i -= ts * xi;
        p1i -= ti * xi;
      }
#pragma unroll
    for (int o = 1; o < kLanes; o <<= 1) {
      p1r += __shfl_xor(p1r, o);
      if (sb < i) p0r += __shfl_xor(p0r, o);  // uniform, as the next
      if (any) {
        p0i += __shfl_xor(p0i, o);
        p1i += __shfl_xor(p1i, o);
      }
    }
    if (act && part == 0) {
      Cx x0, x1;
      back_substitute(s, sb, i, T[sb * kLd + sb], T[sb * kLd + i], T[i * kLd + sb], T[i * kLd + i], wr, wi,
                      Cx{p0r, cplx ? p0i : 0.0}, Cx{p1r, cplx ? p1i : 0.0}, same, x0, x1);
      X[i * kLdx + j] = x1.re;
      if (cplx) X[i * kLdx + j + 1] = x1.im;
      if (sb < i) {
        X[sb * kLdx + j] = x0.re;
        if (cplx) X[sb * kLdx + j + 1] = x0.im;
      }
    }
    wave_sync();
    i = sb - 1;
  }
  // normalise: the largest modulus becomes 1
  double mx = 0.0;
  if (mine)
    for (int q = part; q < n; q += kLanes) mx = fmax(mx, fabs(X[q * kLdx + j]) + (cplx ? fabs(X[q * kLdx + j + 1]) : 0.0));
  for (int o = 1; o < kLanes; o <<= 1) mx = fmax(mx, __shfl_xor(mx, o));
  const double sc = mx > 0.0 ? 1.0 / mx : 1.0;
  if (mine)
    for (int q = part; q < n; q += kLanes) {
      X[q * kLdx + j] *= sc;
      if (cplx) X[q * kLdx + j + 1] *= sc;
    }
  __syncthreads();
  for (int t = tid; t < n * n; t += kEigenThreads) XT[t] = X[(t / n) * kLdx + t % n];
}

// The same for n > 64: X takes T's place in LDS (T goes to the workspace first), all eigenvectors advance
// together over T's blocks from the bottom, the block's two rows of T staged in LDS and the next one's
// loaded ahead; four lanes per eigenvector.
__device__ __forceinline__ void eigenvectors_large(EigenLds& s, int n, double same, double* __restrict__ TG,
                                                   double* __restrict__ XT) {
  const int tid = threadIdx.x;
  constexpr int NT = kEigenThreads;
  double* X = s.H;  // X(i, j) at X[i kLd + j]
  for (int t = tid; t < n * n; t += NT) TG[t] = X[(t / n) * kLd + t % n];
  __syncthreads();
  double* trow = s.refl;  // rows sb and i of the current block: [2][n]
  for (int t = tid; t < n * kLd; t += NT) X[t] = 0.0;
  __syncthreads();
  const int j = tid / 4, part = tid % 4;  // 4 lanes each for up to 128 eigenvectors
  const double wr = j < n ? s.lre[j] : 0.0, wi = j < n ? s.lim[j] : 0.0;
  const bool mine = j < n && wi >= 0.0;
  const bool cplx = mine && wi > 0.0;
  const int bend = cplx ? j + 1 : j, jl = bend;
  if (mine && part == 0) {
    if (cplx) {
      Cx x0, x1;
      const double* t = TG + (int64_t)j * n + j;
      own_block(t[0], t[1], t[n], t[n + 1], wr, wi, true, x0, x1);
      X[j * kLd + j] = x0.re;
      X[j * kLd + j + 1] = x0.im;
      X[(j + 1) * kLd + j] = x1.re;
      X[(j + 1) * kLd + j + 1] = x1.im;
    } else {
      X[j * kLd + j] = 1.0;
    }
  }
  const bool any = __any(cplx);
  double ps = 0.0, pi = 0.0;  // rows of the next block, entry tid
  auto fetch = [&](int last) {
    const int first = s.blk[last] == 0 ? last - 1 : last;
    ps = TG[(int64_t)first * n + min(tid, n - 1)];
    pi = TG[(int64_t)last * n + min(tid, n - 1)];
  };
  fetch(n - 1);
  for (int i = n - 1; i >= 0;) {
    const int sb = s.blk[i] == 0 ? i - 1 : i;  // block rows [sb, i]
    __syncthreads();  // the previous block's rows are no longer read
    if (tid < n) {
      trow[tid] = ps;
      trow[n + tid] = pi;
    }
    if (sb > 0) fetch(sb - 1);
    __syncthreads();
    const double *ts = trow, *ti = trow + n;
    const bool act = mine && i < j;
    double p0r = 0.0, p1r = 0.0, p0i = 0.0, p1i = 0.0;
    if (act) {
      if (any) {
        for (int c = i + 1 + part; c <= bend; c += 4) {
          const double xr = X[c * kLd + j], xi = X[c * kLd + jl];
          p0r -= ts[c] * xr;
          p1r -= ti[c] * xr;
          p0i -= ts[c] * xi;
          p1i -= ti[c] * xi;
        }
      } else {
#pragma unroll 4
        for (int c = i + 1 + part; c <= bend; c += 4) {
          const double xr = X[c * kLd + j];
          p0r -= ts[c] * xr;
          p1r -= ti[c] * xr;
        }
      }
    }
#pragma unroll
    for (int o = 1; o < 4; o <<= 1) {
      p1r += __shfl_xor(p1r, o);
      if (sb < i) p0r += __shfl_xor(p0r, o);  // uniform, as the next
      if (any) {
        p0i += __shfl_xor(p0i, o);
        p1i += __shfl_xor(p1i, o);
      }
    }
    if (act && part == 0) {
      Cx x0, x1;
      back_substitute(s, sb, i, ts[sb], ts[i], ti[sb], ti[i], wr, wi, Cx{p0r, cplx ? p0i : 0.0},
                      Cx{p1r, cplx ? p1i : 0.0}, same, x0, x1);
      X[i * kLd + j] = x1.re;
      if (cplx) X[i * kLd + j + 1] = x1.im;
      if (sb < i) {
        X[sb * kLd + j] = x0.re;
        if (cplx) X[sb * kLd + j + 1] = x0.im;
      }
    }
    wave_sync();
    i = sb - 1;
  }
  double mx = 0.0;
  if (mine)
    for (int q = part; q < n; q += 4) mx = fmax(mx, fabs(X[q * kLd + j]) + (cplx ? fabs(X[q * kLd + j + 1]) : 0.0));
  for (int o = 1; o < 4; o <<= 1) mx = fmax(mx, __shfl_xor(mx, o));
  const double sc = mx > 0.0 ? 1.0 / mx : 1.0;
  if (mine)
    for (int q = part; q < n; q += 4) {
      X[q * kLd + j] *= sc;
      if (cplx) X[q * kLd + j + 1] *= sc;
    }
  __syncthreads();
  for (int t = tid; t < n * n; t += NT) XT[t] = X[(t / n) * kLd + t % n];
}

__device__ __forceinline__ void lds_eigen(const Item& it, double* base, int32_t* status, EigenLds& s, int sweep_cap) {
  const int n = it.n, tid = threadIdx.x, lane = tid & 63;
  const bool wave0 = tid < 64;
  const double* G = base + (int64_t)kBufG * n * n;
  double* ZT = base + (int64_t)kBufZ * n * n;  // Z(r, c) = ZT[c n + r]
  double* XT = base + (int64_t)kBufX * n * n;  // eigenvector j, component i at XT[i n + j]
  double* QV = base + (int64_t)kBufYS * n * n;  // v_k at QV[k n + i], tau_k at QV[(n-1) n + k]
  double* ex = base + extras_off(n);
  for (int t = tid; t < n * n; t += kEigenThreads) ZT[t] = (t / n) == (t % n) ? 1.0 : 0.0;
  if (n <= 64)
    reg_hessenberg<4, 2>(G, n, QV, s.H, s.red);
  else
    reg_hessenberg<8, 4>(G, n, QV, s.H, s.red);
  // Frobenius norm (invariant under the similarities that follow): backstop scale for deflation in clusters
  // of nearly equal eigenvalues where the local test cannot be met
  double nrm2 = 0.0;
  for (int w = 0; w < kEigenThreads / 64; ++w) nrm2 += s.red[w];
  const double hnorm = sqrt(nrm2);
  if (tid == 0) {
    s.zops[0] = s.zops[1] = ZOp{0, 0, 0, 0, 0};
    s.fail = 0;
  }
  __syncthreads();
  // Wave 0 decides and chases single sweeps on its own; the other waves apply its last reflectors to Z
  // meanwhile. A multi-bulge pass takes all waves.
  QrState q{n - 1, 0, 0};
  for (int iter = 0;; ++iter) {
    const int slot = iter & 1;
    double* rf = s.refl + slot * 3 * kLdsMaxn;
    if (wave0)
      qr_decide(s, n, q, hnorm, sweep_cap, rf, &s.zops[slot], lane);
    else if (iter > 0)
      apply_to_z(s.zops[slot ^ 1], s.refl + (slot ^ 1) * 3 * kLdsMaxn, ZT, n, tid - 64, kEigenThreads - 64);
    __syncthreads();
    const ZOp op = s.zops[slot];  // not rewritten before the barrier of the next iteration
    if (op.nb > 0) lds_multibulge(s.H, n, ZT, op.lo, op.hh, op.nb, rf, kTail + 3 * lane);
    if (op.stop) break;
  }
  if (s.fail) {
    if (tid == 0) status[it.layer] = -5;
    return;
  }
  for (int t = tid; t < n; t += kEigenThreads) {
    ex[t] = s.lre[t];
    ex[n + t] = s.lim[t];
  }
  const double same = same_eigenvalue(hnorm);
  if (n <= 64)
    eigenvectors_small(s, n, same, XT);
  else
    eigenvectors_large(s, n, same, base + (int64_t)kBufYT * n * n, XT);
}

// One workgroup per problem of at most kLdsMaxn rows: workgroup b solves items[order[b]] (order null:
// items[b]); larger problems are left to k_eigen_big.
__global__ __launch_bounds__(kEigenThreads) void k_eigen_lds(const Item* items, double* ws, int32_t* status, int sweep_cap,
                                                              const int32_t* order, int weak) {
  const Item it = items[order ? order[blockIdx.x] : blockIdx.x];
  if (it.n > kLdsMaxn || layer_failed(status, it.layer) || weak_done(weak, ws, it)) return;
  __shared__ EigenLds s;
  lds_eigen(it, ws + it.ws, status, s, sweep_cap);
}

// Persistent form: every workgroup takes the next position of `order` from the counter `queue` (reset to 0
// before the launch) and solves that problem, until n_items are taken; every wave reaches the exit
// once the counter passes n_items.
__global__ __launch_bounds__(kEigenThreads) void k_eigen_lds_persistent(const Item* items, double* ws, int32_t* status,
                                                                         int sweep_cap, const int32_t* order,
                                                                         int32_t* queue, int n_items, int weak) {
  __shared__ EigenLds s;
  __shared__ int snext;
  for (;;) {
    __syncthreads();  // the previous problem is done with the LDS
    if (threadIdx.x == 0) snext = atomicAdd(queue, 1);
    __syncthreads();
    const int pos = snext;
    if (pos >= n_items) return;
    const Item it = items[order[pos]];
    if (it.n > kLdsMaxn || layer_failed(status, it.layer) || weak_done(weak, ws, it)) continue;
    lds_eigen(it, ws + it.ws, status, s, sweep_cap);
  }
}

}  // namespace vbrdf
