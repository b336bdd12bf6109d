// Small dense symmetric solves on the host: the Gram system of the
// projection guess (up to 17 unknowns) and the normal equations of the input
// estimation (up to 384).  Header-only, so that a CPU test can build them
// without the device code.
#pragma once

#include <algorithm>
#include <cmath>
#include <vector>

namespace sw {

// Eigen-decomposition of a symmetric n x n matrix (row-major, destroyed) by
// cyclic Jacobi rotations: A = V diag(w) V^T, V row-major with eigenvectors
// in its columns.
inline void sym_eig(int n, std::vector<double>& A, std::vector<double>& V, std::vector<double>& w) {
  V.assign((size_t)n * n, 0.0);
  for (int i = 0; i < n; ++i) V[(size_t)i * n + i] = 1.0;
  auto a = [&](int i, int j) -> double& { return A[(size_t)i * n + j]; };
  auto v = [&](int i, int j) -> double& { return V[(size_t)i * n + j]; };
  for (int sweep = 0; sweep < 100; ++sweep) {
    double off = 0.0, diag = 0.0;
    for (int i = 0; i < n; ++i) {
      diag += a(i, i) * a(i, i);
      for (int j = i + 1; j < n; ++j) off += a(i, j) * a(i, j);
    }
    if (off <= 1e-32 * diag || off == 0.0) break;
    for (int p = 0; p < n; ++p)
      for (int q = p + 1; q < n; ++q) {
        const double apq = a(p, q);
        if (apq == 0.0) continue;
        // rotation in the (p, q) plane that zeroes a(p, q)
        const double th = (a(q, q) - a(p, p)) / (2.0 * apq);
        const double t = (th >= 0.0 ? 1.0 : -1.0) / (std::fabs(th) + std::sqrt(th * th + 1.0));
        const double cs = 1.0 / std::sqrt(t * t + 1.0), sn = t * cs;
        a(p, p) -= t * apq;
        a(q, q) += t * apq;
        a(p, q) = a(q, p) = 0.0;
        for (int r = 0; r < n; ++r) {
          if (r != p && r != q) {
            const double arp = a(r, p), arq = a(r, q);
            a(r, p) = a(p, r) = cs * arp - sn * arq;
            a(r, q) = a(q, r) = sn * arp + cs * arq;
          }
          const double vrp = v(r, p), vrq = v(r, q);
          v(r, p) = cs * vrp - sn * vrq;
          v(r, q) = sn * vrp + cs * vrq;
        }
      }
  }
  w.resize(n);
  for (int i = 0; i < n; ++i) w[i] = a(i, i);
}

// theta = V W^+ V^T h for A = V diag(w) V^T, eigenvalues at or below
// rel_cut times the largest dropped; returns how many were kept.
inline int truncated_solve(int n, const std::vector<double>& V, const std::vector<double>& w, const double* h,
                    double* theta, double rel_cut) {
  double wmax = 0.0;
  for (int i = 0; i < n; ++i) wmax = std::max(wmax, w[i]);
  std::vector<double> y(n, 0.0);
  int kept = 0;
  for (int k = 0; k < n; ++k) {
    if (!(wmax > 0.0 && w[k] > rel_cut * wmax)) continue;
    double acc = 0.0;
    for (int i = 0; i < n; ++i) acc += V[(size_t)i * n + k] * h[i];
    y[k] = acc / w[k];
    ++kept;
  }
  for (int i = 0; i < n; ++i) {
    double acc = 0.0;
    for (int k = 0; k < n; ++k) acc += V[(size_t)i * n + k] * y[k];
    theta[i] = acc;
  }
  return kept;
}

// theta = A^+ h for a symmetric n x n A (row-major, destroyed), eigenvalues at
// or below rel_cut times the largest dropped; returns how many were kept: what
// sym_eig and truncated_solve give, without the eigenvectors (150 unknowns:
// 14 ms with them, 1.5 without).  Householder reflections to a tridiagonal
// matrix T = Q^T A Q, then implicit QL steps with Wilkinson's shift to its
// eigenvalues (Bowdler, Martin, Reinsch and Wilkinson 1968), each plane
// rotation applied to the one vector g = Q^T h as it is made; the truncated
// quotients go back through the rotations and the reflections in reverse.  The
// reflections take the rows by falling diagonal entry and QL the small end of T
// first, so that rounding in the large rows does not reach the small ones'
// results before their turn.
// Its errors are those of the largest eigenvalue, Jacobi's of a positive
// matrix those of the scaled one (Demmel and Veselic 1992): on rows of unequal
// size (records of unequal amplitude, late shifts) QL loses their ratio.  Error
// of the solution against 40 digits, QL over Jacobi, geometric means over
// records of marches (9 to 48 unknowns) by the ratio of the largest diagonal
// entry to the smallest: 0.5 below n / 4, 0.6 to n / 2, 0.9 to n, 1.2 to 2 n (in
// the given order and from the large end: 0.7, 1.1, 1.4, 1.7); 150 unknowns and
// a ratio of 2e5: 70 (330).  So QL up to a ratio of n / 2 (rows of zeros apart,
// which no reflection touches).  Matrices past it or with a negative diagonal
// entry, values that are not finite, cuts below 1e-12, and matrices QL does not
// finish take the Jacobi way.
inline int sym_pinv_solve(int n, std::vector<double>& A, const double* h, double* theta, double rel_cut) {
  auto jacobi = [&](std::vector<double>& M) {
    std::vector<double> V, w;
    sym_eig(n, M, V, w);
    return truncated_solve(n, V, w, h, theta, rel_cut);
  };
  bool finite = true;
  for (int i = 0; i < n; ++i) finite = finite && std::isfinite(h[i]);
  for (const double v : A) finite = finite && std::isfinite(v);
  double dmax = 0.0, dmin = INFINITY;
  bool even = true;
  for (int i = 0; i < n; ++i) {
    const double v = A[(size_t)i * n + i];
    even = even && v >= 0.0;
    dmax = std::max(dmax, v);
    if (v > 0.0) dmin = std::min(dmin, v);
  }
  even = even && (dmax == 0.0 || dmax <= 0.5 * n * dmin);
  if (!finite || !even || n < 3 || rel_cut < 1e-12) return jacobi(A);
  const std::vector<double> A0(A);
  std::vector<int> order(n);
  for (int i = 0; i < n; ++i) order[i] = i;
  std::stable_sort(order.begin(), order.end(),
                   [&](int i, int j) { return A0[(size_t)i * n + i] > A0[(size_t)j * n + j]; });
  std::vector<double> d(n), e(n, 0.0), g(n), refl((size_t)n * n), beta(n, 0.0), p(n);
  for (int i = 0; i < n; ++i) {
    g[i] = h[order[i]];
    for (int j = 0; j < n; ++j) A[(size_t)i * n + j] = A0[(size_t)order[i] * n + order[j]];
  }
  // reflection k zeroes column k below the subdiagonal: H = I - beta v v^T, v
  // kept in row k of refl (entries k + 1 .. n - 1)
  for (int k = 0; k + 2 < n; ++k) {
    double* v = &refl[(size_t)k * n];
    double big = 0.0;
    for (int i = k + 1; i < n; ++i) big = std::max(big, std::fabs(A[(size_t)i * n + k]));
    d[k] = A[(size_t)k * n + k];
    if (big == 0.0) continue;  // nothing below the diagonal: beta 0, e 0
    double nrm2 = 0.0;
    for (int i = k + 1; i < n; ++i) {
      v[i] = A[(size_t)i * n + k] / big;
      nrm2 += v[i] * v[i];
    }
    const double alpha = v[k + 1] >= 0.0 ? -std::sqrt(nrm2) : std::sqrt(nrm2);
    e[k] = alpha * big;
    const double vv = nrm2 - 2.0 * alpha * v[k + 1] + alpha * alpha;  // |v|^2 after the next line
    v[k + 1] -= alpha;
    beta[k] = 2.0 / vv;
    // p = beta A v (rows of the symmetric A as its columns), then
    // A <- A - v q^T - q v^T with q = p - (beta / 2) (v.p) v
    std::fill(p.begin() + k + 1, p.end(), 0.0);
    for (int i = k + 1; i < n; ++i) {
      const double s = beta[k] * v[i];
      const double* row = &A[(size_t)i * n];
      for (int j = k + 1; j < n; ++j) p[j] += s * row[j];
    }
    double vp = 0.0, vg = 0.0;
    for (int i = k + 1; i < n; ++i) {
      vp += v[i] * p[i];
      vg += v[i] * g[i];
    }
    for (int i = k + 1; i < n; ++i) {
      p[i] -= 0.5 * beta[k] * vp * v[i];
      g[i] -= beta[k] * vg * v[i];
    }
    for (int i = k + 1; i < n; ++i) {
      const double vi = v[i], qi = p[i];
      double* row = &A[(size_t)i * n];
      for (int j = k + 1; j < n; ++j) row[j] -= vi * p[j] + qi * v[j];
    }
  }
  d[n - 2] = A[(size_t)(n - 2) * n + n - 2];
  d[n - 1] = A[(size_t)(n - 1) * n + n - 1];
  e[n - 2] = A[(size_t)(n - 1) * n + n - 2];
  // QL, the small end of T first: e[i] couples i and i + 1
  std::reverse(d.begin(), d.end());
  std::reverse(e.begin(), e.begin() + (n - 1));
  std::reverse(g.begin(), g.end());
  struct Rot {
    int i;
    double c, s;
  };
  std::vector<Rot> rots;
  rots.reserve(2 * (size_t)n * n);
  const double eps = 2.220446049250313e-16;
  for (int l = 0; l < n; ++l) {
    for (int turn = 0;; ++turn) {
      int m = l;
      while (m + 1 < n && std::fabs(e[m]) > eps * (std::fabs(d[m]) + std::fabs(d[m + 1]))) ++m;
      if (m == l) break;
      if (turn == 60) {
        A = A0;
        return jacobi(A);
      }
      // shift: the eigenvalue of the leading 2 x 2 block nearest d[l]
      const double t = (d[l + 1] - d[l]) / (2.0 * e[l]);
      double x = d[m] - d[l] + e[l] / (t + std::copysign(std::hypot(t, 1.0), t));
      double c = 1.0, s = 1.0, shift = 0.0;
      int i = m - 1;
      for (; i >= l; --i) {
        const double f = s * e[i], b = c * e[i], r = std::hypot(f, x);
        e[i + 1] = r;
        if (r == 0.0) {  // the matrix splits here
          d[i + 1] -= shift;
          e[m] = 0.0;
          break;
        }
        s = f / r;
        c = x / r;
        const double y = d[i + 1] - shift, z = (d[i] - y) * s + 2.0 * c * b;
        shift = s * z;
        d[i + 1] = y + shift;
        x = c * z - b;
        const double gi = g[i], gj = g[i + 1];
        g[i] = c * gi - s * gj;
        g[i + 1] = s * gi + c * gj;
        rots.push_back({i, c, s});
      }
      if (i >= l) continue;
      d[l] -= shift;
      e[l] = x;
      e[m] = 0.0;
    }
  }
  double wmax = 0.0;
  for (int i = 0; i < n; ++i) wmax = std::max(wmax, d[i]);
  int kept = 0;
  for (int i = 0; i < n; ++i) {
    const bool keep = wmax > 0.0 && d[i] > rel_cut * wmax;
    g[i] = keep ? g[i] / d[i] : 0.0;
    kept += keep;
  }
  for (size_t k = rots.size(); k-- > 0;) {
    const Rot& R = rots[k];
    const double gi = g[R.i], gj = g[R.i + 1];
    g[R.i] = R.c * gi + R.s * gj;
    g[R.i + 1] = R.c * gj - R.s * gi;
  }
  std::reverse(g.begin(), g.end());
  for (int k = n - 3; k >= 0; --k) {
    if (beta[k] == 0.0) continue;
    const double* v = &refl[(size_t)k * n];
    double vg = 0.0;
    for (int i = k + 1; i < n; ++i) vg += v[i] * g[i];
    for (int i = k + 1; i < n; ++i) g[i] -= beta[k] * vg * v[i];
  }
  for (int i = 0; i < n; ++i) theta[order[i]] = g[i];
  return kept;
}

// Solves G theta = h for a symmetric positive semidefinite G (leading
// dimension ldg) in the least-squares sense, on the unit-diagonal scaling
// D G D (D = diag(G)^-1/2) truncated at rel_cut: theta = D (D G D)^+ D h.
inline void psd_solve(int m, const double* G, int ldg, const double* h, double* theta, double rel_cut) {
  std::vector<double> d(m), A((size_t)m * m), V, w, hs(m), ts(m);
  for (int i = 0; i < m; ++i) {
    const double gi = G[i * ldg + i];
    d[i] = gi > 0.0 ? 1.0 / std::sqrt(gi) : 0.0;
  }
  for (int i = 0; i < m; ++i)
    for (int j = 0; j < m; ++j) A[(size_t)i * m + j] = d[i] * 0.5 * (G[i * ldg + j] + G[j * ldg + i]) * d[j];
  sym_eig(m, A, V, w);
  for (int i = 0; i < m; ++i) hs[i] = d[i] * h[i];
  truncated_solve(m, V, w, hs.data(), ts.data(), rel_cut);
  for (int i = 0; i < m; ++i) theta[i] = d[i] * ts[i];
}

}  // namespace sw
