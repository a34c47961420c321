// Symmetric eigendecomposition on the host (fp64): Householder reduction to
// tridiagonal form followed by implicit symmetric QR steps with a Wilkinson
// shift (the textbook method; e.g. Golub & Van Loan, Sec. 8.3), accumulating
// every transformation into the eigenvector matrix. Used by the fit, which is
// off the per-token path; 128 x 128 takes about a millisecond. The eigenvector matrix is
// held transposed (row k = eigenvector column k), so that every reflection and rotation
// updates whole contiguous rows. A QR sweep's rotations are recorded and applied to the
// eigenvector rows together, a block of columns at a time: a row is read and written once
// per sweep instead of once per rotation. The row loops are compiled for AVX-512 and AVX2
// too (chosen when the library is loaded), without fused multiply-adds, so every element
// takes the same operations in the same order on any host: results do not depend on it.
#include <algorithm>
#include <cmath>
#include <numeric>
#include <vector>

#include "host_common.hpp"

namespace spectra {

namespace {

// Rotations k = 0 .. cnt - 1 of rows (lo + k, lo + k + 1) of Qt (n columns), in order.
SPECTRA_ROW_CLONES void apply_rotations(double* Qt, int n, int lo, int cnt, const double* c, const double* s) {
  constexpr int RB = 32;  // columns per block: the carried row stays in registers
  int r0 = 0;
  for (; r0 + RB <= n; r0 += RB) {
    double carry[RB];
    double* row = Qt + (size_t)lo * n + r0;
    for (int r = 0; r < RB; ++r) carry[r] = row[r];
    for (int k = 0; k < cnt; ++k) {
      double* next = row + n;
      const double ck = c[k], sk = s[k];
      for (int r = 0; r < RB; ++r) {
        const double q1 = carry[r], q2 = next[r];
        row[r] = ck * q1 + sk * q2;
        carry[r] = -sk * q1 + ck * q2;
      }
      row = next;
    }
    for (int r = 0; r < RB; ++r) row[r] = carry[r];
  }
  for (int k = 0; k < cnt; ++k) {
    double* r1 = Qt + (size_t)(lo + k) * n;
    double* r2 = r1 + n;
    for (int r = r0; r < n; ++r) {
      const double q1 = r1[r], q2 = r2[r];
      r1[r] = c[k] * q1 + s[k] * q2;
      r2[r] = -s[k] * q1 + c[k] * q2;
    }
  }
}

// Reduce symmetric A (n x n, row-major, overwritten) to tridiagonal T = Q^T A Q; Qt holds
// Q transposed; work: 4 n values.
SPECTRA_ROW_CLONES void householder_tridiagonal(double* A, double* Qt, int n, double* work) {
#define a(i, j) A[(size_t)(i) * n + (j)]
  double *v = work, *pv = work + n, *qv = work + 2 * n, *sr = work + 3 * n;
  for (int k = 0; k + 2 < n; ++k) {
    const int m = n - k - 1;  // length of the column below the diagonal
    double norm2 = 0.0;
    for (int i = 0; i < m; ++i) norm2 += a(k + 1 + i, k) * a(k + 1 + i, k);
    if (norm2 == 0.0) continue;
    const double x0 = a(k + 1, k);
    const double root = __builtin_sqrt(norm2), alpha = x0 >= 0 ? -root : root;
    for (int i = 0; i < m; ++i) v[i] = a(k + 1 + i, k);
    v[0] -= alpha;
    double vtv = 0.0;
    for (int i = 0; i < m; ++i) vtv += v[i] * v[i];
    if (vtv == 0.0) continue;
    const double beta = 2.0 / vtv;  // H = I - beta v v^T on indices k+1..n-1
    // p = beta * A_sub v ; K = beta/2 * v^T p ; w = p - K v ; A_sub -= v w^T + w v^T
    // (A_sub symmetric: row j of A_sub is its column j, so the sums run as row updates;
    // each pv[i] still adds its terms in ascending j)
    for (int i = 0; i < m; ++i) pv[i] = 0.0;
    for (int j = 0; j < m; ++j) {
      const double vj = v[j];
      const double* row = &a(k + 1 + j, k + 1);
      for (int i = 0; i < m; ++i) pv[i] += row[i] * vj;
    }
    for (int i = 0; i < m; ++i) pv[i] *= beta;
    double vp = 0.0;
    for (int i = 0; i < m; ++i) vp += v[i] * pv[i];
    const double K = 0.5 * beta * vp;
    for (int i = 0; i < m; ++i) qv[i] = pv[i] - K * v[i];
    for (int i = 0; i < m; ++i)
      for (int j = 0; j < m; ++j) a(k + 1 + i, k + 1 + j) -= v[i] * qv[j] + qv[i] * v[j];
    a(k + 1, k) = alpha;
    a(k, k + 1) = alpha;
    for (int i = 1; i < m; ++i) {
      a(k + 1 + i, k) = 0.0;
      a(k, k + 1 + i) = 0.0;
    }
    // Q <- Q H, i.e. rows k+1.. of Qt: s_r = sum_j v_j Qt[k+1+j][r] (ascending j), then
    // Qt[k+1+j][r] -= (beta s_r) v_j
    for (int r = 0; r < n; ++r) sr[r] = 0.0;
    for (int j = 0; j < m; ++j) {
      const double vj = v[j];
      const double* row = &Qt[(size_t)(k + 1 + j) * n];
      for (int r = 0; r < n; ++r) sr[r] += row[r] * vj;
    }
    for (int r = 0; r < n; ++r) sr[r] *= beta;
    for (int j = 0; j < m; ++j) {
      const double vj = v[j];
      double* row = &Qt[(size_t)(k + 1 + j) * n];
      for (int r = 0; r < n; ++r) row[r] -= sr[r] * vj;
    }
  }
#undef a
}

}  // namespace

spectra_status eigh_sym(const double* a_in, int n, double* w, double* v_out) {
  if (n <= 0 || n > 1024) return fail(SPECTRA_EINVAL, "eigh: n=%d out of range", n);
  std::vector<double> T((size_t)n * n), Qt((size_t)n * n, 0.0);
  double fro = 0.0;
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) {
      const double x = 0.5 * (a_in[(size_t)i * n + j] + a_in[(size_t)j * n + i]);
      if (!std::isfinite(x)) return fail(SPECTRA_ENUMERIC, "eigh: non-finite input");
      T[(size_t)i * n + j] = x;
      fro += x * x;
    }
  for (int i = 0; i < n; ++i) Qt[(size_t)i * n + i] = 1.0;
  std::vector<double> work((size_t)4 * n);
  householder_tridiagonal(T.data(), Qt.data(), n, work.data());
  auto t = [&](int i, int j) -> double& { return T[(size_t)i * n + j]; };
  const double eps = 2.220446049250313e-16;
  const double tiny = 1e-300 + eps * std::sqrt(fro) * 1e-3;

  // Apply P = [[c, s], [-s, c]] on rows/cols (k, k+1): T <- P T P^T (Q <- Q P^T, rows k and
  // k+1 of Qt, at the end of the sweep).
  // Entries outside columns / rows k - 1 .. k + 2 of the two rows / columns are zero.
  auto rotate = [&](int k, double c, double s, int lo, int hi) {
    const int j0 = std::max(lo, k - 1), j1 = std::min(hi, k + 2);
    auto window = [&](int m) {  // j0 .. j0 + m - 1
      double* r1 = &t(k, j0);
      double* r2 = &t(k + 1, j0);
      for (int j = 0; j < m; ++j) {
        const double x1 = r1[j], x2 = r2[j];
        r1[j] = c * x1 + s * x2;
        r2[j] = -s * x1 + c * x2;
      }
      double* col = &t(j0, k);
      for (int i = 0; i < m; ++i) {
        const double c1 = col[(size_t)i * n], c2 = col[(size_t)i * n + 1];
        col[(size_t)i * n] = c * c1 + s * c2;
        col[(size_t)i * n + 1] = -s * c1 + c * c2;
      }
    };
    if (j1 - j0 == 3)
      window(4);  // unrolled: every rotation but a sweep's first and last
    else
      window(j1 - j0 + 1);
  };
  std::vector<double> rot_c(n), rot_s(n);

  int hi = n - 1;
  long iters = 0;
  const long max_iters = 60L * n;
  while (hi > 0) {
    for (int i = 0; i < hi; ++i) {
      if (std::fabs(t(i + 1, i)) <= eps * (std::fabs(t(i, i)) + std::fabs(t(i + 1, i + 1))) ||
          std::fabs(t(i + 1, i)) < tiny) {
        t(i + 1, i) = 0.0;
        t(i, i + 1) = 0.0;
      }
    }
    while (hi > 0 && t(hi, hi - 1) == 0.0) --hi;
    if (hi == 0) break;
    int lo = hi - 1;
    while (lo > 0 && t(lo, lo - 1) != 0.0) --lo;
    if (++iters > max_iters) return fail(SPECTRA_ENUMERIC, "eigh: QR iteration did not converge");
    // Wilkinson shift from the trailing 2x2 of the unreduced block [lo, hi]
    const double an = t(hi, hi), bn = t(hi, hi - 1);
    const double delta = 0.5 * (t(hi - 1, hi - 1) - an);
    const double sgn = delta >= 0 ? 1.0 : -1.0;
    const double mu = an - bn * bn / (delta + sgn * std::hypot(delta, bn));
    double x = t(lo, lo) - mu, z = t(lo + 1, lo);
    for (int k = lo; k < hi; ++k) {
      const double r = std::hypot(x, z);
      const double c = r == 0.0 ? 1.0 : x / r, s = r == 0.0 ? 0.0 : z / r;
      rotate(k, c, s, lo, hi);
      rot_c[k - lo] = c;
      rot_s[k - lo] = s;
      if (k + 1 < hi) {
        x = t(k + 1, k);
        z = t(k + 2, k);
      }
    }
    apply_rotations(Qt.data(), n, lo, hi - lo, rot_c.data(), rot_s.data());
  }
  // Sort descending (stable by position), sign-normalise, write out.
  std::vector<int> order(n);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int i, int j) { return t(i, i) > t(j, j); });
  for (int jo = 0; jo < n; ++jo) {
    const int j = order[jo];
    w[jo] = t(j, j);
    int imax = 0;
    double vmax = -1.0;
    const double* qj = &Qt[(size_t)j * n];
    for (int i = 0; i < n; ++i) {
      const double x = std::fabs(qj[i]);
      if (x > vmax) {
        vmax = x;
        imax = i;
      }
    }
    const double sg = qj[imax] < 0 ? -1.0 : 1.0;
    for (int i = 0; i < n; ++i) v_out[(size_t)i * n + jo] = sg * qj[i];
  }
  return SPECTRA_OK;
}

}  // namespace spectra
