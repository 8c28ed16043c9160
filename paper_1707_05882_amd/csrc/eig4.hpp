// Eigen-decomposition of one real 4 x 4 matrix by one thread: the Stokes block of a node in the
// iteration for weakly coupled orders (k_weak.hip). Plain C++ on caller-provided arrays, so the same
// code runs on the host for its test.
#pragma once

#include <math.h>

#if defined(__HIPCC__)
#define VBRDF_HD __host__ __device__
#else
#define VBRDF_HD
#endif

namespace vbrdf {

// Columns of eigenvectors whose determinant falls below this are taken as dependent.
constexpr double kEig4MinDet = 1e-6;

// Rotation of rows p, q of H (from the left) and of columns p, q of H and Z (from the right).
VBRDF_HD inline void eig4_rotate(double* H, double* Z, int p, int q, double c, double s) {
  for (int j = 0; j < 4; ++j) {
    const double a = H[4 * p + j], b = H[4 * q + j];
    H[4 * p + j] = c * a + s * b;
    H[4 * q + j] = c * b - s * a;
  }
  for (int i = 0; i < 4; ++i) {
    const double a = H[4 * i + p], b = H[4 * i + q];
    H[4 * i + p] = c * a + s * b;
    H[4 * i + q] = c * b - s * a;
    const double x = Z[4 * i + p], y = Z[4 * i + q];
    Z[4 * i + p] = c * x + s * y;
    Z[4 * i + q] = c * y - s * x;
  }
}

// Householder similarity with the vector (x, y, z) on rows and columns k, k + 1, k + 2 (m = 3) or
// k, k + 1 (m = 2, z = 0).
VBRDF_HD inline void eig4_reflect(double* H, double* Z, int k, int m, double x, double y, double z) {
  const double nrm = sqrt(x * x + y * y + z * z);
  if (!(nrm > 0.0)) return;
  const double v0 = x + (x >= 0.0 ? nrm : -nrm);
  const double beta = 2.0 / (v0 * v0 + y * y + z * z);
  const double v[3] = {v0, y, z};
  for (int j = 0; j < 4; ++j) {
    double w = 0.0;
    for (int r = 0; r < m; ++r) w += v[r] * H[4 * (k + r) + j];
    w *= beta;
    for (int r = 0; r < m; ++r) H[4 * (k + r) + j] -= w * v[r];
  }
  for (int i = 0; i < 4; ++i) {
    double w = 0.0, u = 0.0;
    for (int r = 0; r < m; ++r) {
      w += v[r] * H[4 * i + k + r];
      u += v[r] * Z[4 * i + k + r];
    }
    w *= beta;
    u *= beta;
    for (int r = 0; r < m; ++r) {
      H[4 * i + k + r] -= w * v[r];
      Z[4 * i + k + r] -= u * v[r];
    }
  }
}

// Eigenvalues (wr, wi) and normalised eigenvectors of the row-major 4 x 4 matrix H, in the storage
// of the eigensolver: a complex pair occupies columns j, j + 1 with wi[j] > 0, which hold the real
// and the imaginary part of the eigenvector of wr[j] + i wi[j]. noise: absolute size below which
// differences within H carry no information (rounding of the matrix it was taken from). H is
// overwritten; Q (4 x 4 row-major) receives the columns; X is scratch of 32 doubles. Returns false
// when the iteration does not converge or the columns are nearly dependent.
// Method: Givens reduction to Hessenberg form, double-shift QR on the whole matrix (with 4 rows
// restricting the updates to the active window gains nothing), 2 x 2 blocks with real eigenvalues
// split by a rotation, back-substitution in complex arithmetic.
VBRDF_HD inline bool eig4(double* H, double* Q, double* X, double* wr, double* wi, double noise) {
  double off = 0.0, nrm = 0.0;
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j) {
      const double a = fabs(H[4 * i + j]);
      if (!(a <= 1e300)) return false;
      nrm = fmax(nrm, a);
      if (i != j) off = fmax(off, a);
      Q[4 * i + j] = i == j ? 1.0 : 0.0;
    }
  if (off <= noise) {  // the Stokes components are uncoupled to rounding
    for (int i = 0; i < 4; ++i) {
      wr[i] = H[5 * i];
      wi[i] = 0.0;
    }
    return true;
  }
  // unit scale, so that no square below leaves the range
  const double inv = 1.0 / nrm;
  if (!(inv <= 1e300)) return false;
  for (int i = 0; i < 16; ++i) H[i] *= inv;
  noise *= inv;
  double* Z = Q;
  for (int k = 0; k < 2; ++k)
    for (int i = 3; i > k + 1; --i) {
      const double a = H[4 * (i - 1) + k], b = H[4 * i + k];
      const double r = sqrt(a * a + b * b);
      if (b == 0.0 || !(r > 0.0)) continue;
      eig4_rotate(H, Z, i - 1, i, a / r, b / r);
      H[4 * i + k] = 0.0;
    }
  const double eps = 2.220446049250313e-16;
  int hi = 3, its = 0;
  int first = 0, second = 0;  // bit masks: rows that start and end a complex pair
  while (hi >= 0) {
    int lo = hi;
    for (; lo > 0; --lo) {
      const double sub = fabs(H[4 * lo + lo - 1]);
      double ref = fabs(H[5 * lo]) + fabs(H[5 * (lo - 1)]);
      if (ref == 0.0) ref = 1.0;
      if (sub <= eps * ref) {
        H[4 * lo + lo - 1] = 0.0;
        break;
      }
    }
    if (lo == hi) {
      --hi;
      its = 0;
      continue;
    }
    const double a = H[5 * (hi - 1)], b = H[4 * (hi - 1) + hi], c = H[4 * hi + hi - 1], d = H[5 * hi];
    if (lo == hi - 1) {
      const double p = 0.5 * (a - d), disc = p * p + b * c;
      if (disc >= 0.0) {  // eigenvector (z, c) of the eigenvalue d + z further from d
        const double z = p + (p >= 0.0 ? sqrt(disc) : -sqrt(disc));
        const double r = sqrt(z * z + c * c);
        eig4_rotate(H, Z, hi - 1, hi, z / r, c / r);  // c != 0 here
        H[4 * hi + hi - 1] = 0.0;
      } else {
        first |= 1 << (hi - 1);
        second |= 1 << hi;
      }
      hi -= 2;
      its = 0;
      continue;
    }
    if (++its > 60) return false;
    double s = a + d, t = a * d - b * c;
    if (its % 10 == 0) {  // exceptional shift
      const double w = fabs(c) + fabs(H[4 * (hi - 1) + hi - 2]);
      s = 1.5 * w;
      t = w * w;
    }
    const double h00 = H[5 * lo], h10 = H[4 * (lo + 1) + lo];
    double x = h00 * h00 + H[4 * lo + lo + 1] * h10 - s * h00 + t;
    double y = h10 * (h00 + H[5 * (lo + 1)] - s);
    double z = h10 * H[4 * (lo + 2) + lo + 1];
    for (int k = lo; k < hi; ++k) {
      const bool three = k + 2 <= hi;
      // scaled so that squares neither overflow nor vanish
      const double sc = fabs(x) + fabs(y) + (three ? fabs(z) : 0.0);
      if (sc > 0.0) eig4_reflect(H, Z, k, three ? 3 : 2, x / sc, y / sc, three ? z / sc : 0.0);
      if (k > lo) {
        H[4 * (k + 1) + k - 1] = 0.0;
        if (three) H[4 * (k + 2) + k - 1] = 0.0;
      }
      x = H[4 * (k + 1) + k];
      y = k + 2 <= hi ? H[4 * (k + 2) + k] : 0.0;
      z = k + 3 <= hi ? H[4 * (k + 3) + k] : 0.0;
    }
  }
  // eigenvectors of the quasi-triangular H, X[8 j + 2 i], X[8 j + 2 i + 1]: component i of column j
  for (int j = 0; j < 4; ++j) {
    double* x = X + 8 * j;
    for (int i = 0; i < 8; ++i) x[i] = 0.0;
    if (second >> j & 1) {  // the conjugate: its column takes the imaginary part below
      wr[j] = wr[j - 1];
      wi[j] = -wi[j - 1];
      continue;
    }
    double lr = H[5 * j], li = 0.0;
    x[2 * j] = 1.0;
    if (first >> j & 1) {
      const double a = H[5 * j], b = H[4 * j + j + 1], c = H[4 * (j + 1) + j], d = H[5 * (j + 1)];
      lr = 0.5 * (a + d);
      li = sqrt(fmax(0.0, -(0.25 * (a - d) * (a - d) + b * c)));
      if (fabs(b) >= fabs(c)) {  // (b, lambda - a) / b
        x[2 * j + 2] = (lr - a) / b;
        x[2 * j + 3] = li / b;
      } else {  // (lambda - d, c) / c
        x[2 * j] = (lr - d) / c;
        x[2 * j + 1] = li / c;
        x[2 * j + 2] = 1.0;
      }
    }
    wr[j] = lr;
    wi[j] = li;
    for (int i = j - 1; i >= 0; --i) {
      double rr = 0.0, ri = 0.0;
      for (int k = i + 1; k < 4; ++k) {
        rr -= H[4 * i + k] * x[2 * k];
        ri -= H[4 * i + k] * x[2 * k + 1];
      }
      if (!(second >> i & 1)) {
        const double pr = H[5 * i] - lr, pi = -li;
        const double den = pr * pr + pi * pi;
        // components of one cluster whose eigenvalues agree to rounding stay unmixed
        if (sqrt(den) <= noise && fabs(rr) + fabs(ri) <= 8.0 * noise) continue;
        if (!(den > 0.0)) return false;
        x[2 * i] = (rr * pr + ri * pi) / den;
        x[2 * i + 1] = (ri * pr - rr * pi) / den;
        continue;
      }
      // rows i - 1, i of a complex pair: Cramer's rule on (H - lambda) x = r
      const int g = i - 1;
      double sr = 0.0, si = 0.0;
      for (int k = i + 1; k < 4; ++k) {
        sr -= H[4 * g + k] * x[2 * k];
        si -= H[4 * g + k] * x[2 * k + 1];
      }
      const double a = H[5 * g] - lr, b = H[4 * g + i], c = H[4 * i + g], d = H[5 * i] - lr;
      const double dr = a * d - li * li - b * c, di = -li * (a + d);
      const double den = dr * dr + di * di;
      if (!(den > 0.0)) return false;
      // numerators: s (d - i li) - b r and (a - i li) r - c s
      const double n0r = sr * d + si * li - b * rr, n0i = si * d - sr * li - b * ri;
      const double n1r = a * rr + li * ri - c * sr, n1i = a * ri - li * rr - c * si;
      x[2 * g] = (n0r * dr + n0i * di) / den;
      x[2 * g + 1] = (n0i * dr - n0r * di) / den;
      x[2 * i] = (n1r * dr + n1i * di) / den;
      x[2 * i + 1] = (n1i * dr - n1r * di) / den;
      --i;
    }
  }
  for (int j = 0; j < 4; ++j) {
    wr[j] *= nrm;
    wi[j] *= nrm;
  }
  for (int j = 0; j < 4; ++j)  // real columns: the pair's second column is the imaginary part
    for (int i = 0; i < 4; ++i) H[4 * i + j] = (second >> j & 1) ? X[8 * (j - 1) + 2 * i + 1] : X[8 * j + 2 * i];
  for (int i = 0; i < 4; ++i) {  // Q = Z H, row by row
    const double z0 = Z[4 * i], z1 = Z[4 * i + 1], z2 = Z[4 * i + 2], z3 = Z[4 * i + 3];
    for (int j = 0; j < 4; ++j) Q[4 * i + j] = z0 * H[j] + z1 * H[4 + j] + z2 * H[8 + j] + z3 * H[12 + j];
  }
  for (int j = 0; j < 4; ++j) {
    if (second >> j & 1) continue;
    const int e = j + (first >> j & 1);
    double q = 0.0;
    for (int i = 0; i < 4; ++i)
      for (int k = j; k <= e; ++k) q += Q[4 * i + k] * Q[4 * i + k];
    q = 1.0 / sqrt(q);
    if (!(q <= 1e300)) return false;
    for (int i = 0; i < 4; ++i)
      for (int k = j; k <= e; ++k) Q[4 * i + k] *= q;
  }
  // nearly dependent columns (a defective block): 4 x 4 determinant by 2 x 2 minors
  auto mn = [&](int r0, int r1, int c0, int c1) { return Q[4 * r0 + c0] * Q[4 * r1 + c1] - Q[4 * r0 + c1] * Q[4 * r1 + c0]; };
  const double det = mn(0, 1, 0, 1) * mn(2, 3, 2, 3) - mn(0, 1, 0, 2) * mn(2, 3, 1, 3) + mn(0, 1, 0, 3) * mn(2, 3, 1, 2) +
                     mn(0, 1, 1, 2) * mn(2, 3, 0, 3) - mn(0, 1, 1, 3) * mn(2, 3, 0, 2) + mn(0, 1, 2, 3) * mn(2, 3, 0, 1);
  return fabs(det) >= kEig4MinDet;
}

}  // namespace vbrdf
