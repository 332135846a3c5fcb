// Closed-form orthonormal eigenbases of the 1D operators L_n(alpha,beta,gamma)
// of eq. (3.1), from the spectral lemmas of Sec. 3.2 (Lemmas 3.1-3.4),
// normalised as eq. (4.5) requires (L = V Lambda V^T with V^T V = I).
//
// Host code only.  Accuracy measures (not in the paper, whose footnote to
// eq. (4.5) reports that entrywise assembly was less accurate than `eig`):
//  * every angle is k*pi*a/b with integers a, b; the numerator is reduced
//    exactly in integer arithmetic to the first octant before one
//    floating-point multiply, so no angle carries a large-argument error;
//  * eigenvalues are evaluated as 4 sin^2(theta/2), which equals the lemmas'
//    2 - 2 cos(theta) but keeps full relative accuracy for small theta.
#include <cmath>
#include <cstdint>
#include <cstring>
#include <utility>
#include <vector>

namespace kp {

// sin(pi * m / d) for integers m and d > 0, with exact argument reduction.
static double sinpi_frac(int64_t m, int64_t d) {
  int64_t a = m % (2 * d);
  if (a < 0) a += 2 * d;                 // a in [0, 2d)
  double sign = 1.0;
  if (a >= d) { a -= d; sign = -1.0; }   // sin(x + pi) = -sin(x)
  if (2 * a > d) a = d - a;              // sin(pi - x) = sin(x); a/d in [0, 1/2]
  if (4 * a > d) {                       // sin(x) = cos(pi/2 - x), argument <= pi/4
    return sign * std::cos((M_PI * (double)(d - 2 * a)) / (double)(2 * d));
  }
  return sign * std::sin((M_PI * (double)a) / (double)d);
}

// cos(pi * m / d) = sin(pi * (d - 2m) / (2d)).
static double cospi_frac(int64_t m, int64_t d) { return sinpi_frac(d - 2 * m, 2 * d); }

// sin or cos of pi * m / d for every residue m of the period 2d, evaluated
// once: a basis needs about n^2 values of them.
struct PiTable {
  std::vector<double> v;
  int64_t period;
  PiTable(bool cosine, int64_t d) : v((size_t)(2 * d)), period(2 * d) {
    for (int64_t m = 0; m < 2 * d; ++m) v[m] = cosine ? cospi_frac(m, d) : sinpi_frac(m, d);
  }
  double operator()(int64_t m) const {
    const int64_t a = m % period;
    return v[a < 0 ? a + period : a];
  }
};

// Fills Q (n x n, row-major, Q[j*n + c] = entry j of eigenvector c) and the
// eigenvalues lam[c] in ascending order.  Returns 0, or -1 for bad input.
int basis_1d(int n, int bc, double* Q, double* lam) {
  if (n < 3 || !Q || !lam) return -1;
  const int64_t N = n;
  switch (bc) {
    case 0: {  // periodic, Lemma 3.1: constant, cos/sin pairs, alternating (n even)
      const double c0 = 1.0 / std::sqrt((double)n), c1 = std::sqrt(2.0 / (double)n);
      int col = 0;
      for (int64_t j = 0; j < N; ++j) Q[j * n + col] = c0;
      lam[col++] = 0.0;
      const PiTable cosine(true, N), sine(false, N);
      for (int64_t k = 1; 2 * k < N; ++k) {
        const double s = sinpi_frac(k, N);     // theta_k / 2 = pi k / n
        for (int64_t j = 1; j <= N; ++j) {
          Q[(j - 1) * n + col] = c1 * cosine(2 * j * k);       // angle 2 pi j k / n
          Q[(j - 1) * n + col + 1] = c1 * sine(2 * j * k);
        }
        lam[col] = lam[col + 1] = 4.0 * s * s;
        col += 2;
      }
      if (N % 2 == 0) {
        for (int64_t j = 1; j <= N; ++j) Q[(j - 1) * n + col] = (j % 2 ? -c0 : c0);
        lam[col++] = 4.0;
      }
      return col == n ? 0 : -1;
    }
    case 1: {  // Dirichlet, Lemma 3.2: sin(j k pi / (n+1)), norm^2 = (n+1)/2
      const double c = std::sqrt(2.0 / (double)(N + 1));
      const PiTable sine(false, N + 1);
      for (int64_t k = 1; k <= N; ++k) {
        const double s = sinpi_frac(k, 2 * (N + 1));
        lam[k - 1] = 4.0 * s * s;
        for (int64_t j = 1; j <= N; ++j)
          Q[(j - 1) * n + (k - 1)] = c * sine(j * k);
      }
      return 0;
    }
    case 2: {  // Neumann, Lemma 3.3: cos((j - 1/2)(k - 1) pi / n)
      const PiTable cosine(true, 2 * N);
      for (int64_t k = 1; k <= N; ++k) {
        const double c = (k == 1) ? 1.0 / std::sqrt((double)N) : std::sqrt(2.0 / (double)N);
        const double s = sinpi_frac(k - 1, 2 * N);
        lam[k - 1] = 4.0 * s * s;
        for (int64_t j = 1; j <= N; ++j)
          Q[(j - 1) * n + (k - 1)] = c * cosine((2 * j - 1) * (k - 1));
      }
      return 0;
    }
    case 3:    // Dirichlet-Neumann, Lemma 3.4: sin(j (2k-1) pi / (2n+1))
    case 4: {  // Neumann-Dirichlet: cos((j - 1/2)(2k-1) pi / (2n+1))
      const int64_t D = 2 * N + 1;
      const double c = 2.0 / std::sqrt((double)D);   // norm^2 = (2n+1)/4
      const PiTable wave = bc == 3 ? PiTable(false, D) : PiTable(true, 2 * D);
      for (int64_t k = 1; k <= N; ++k) {
        const double s = sinpi_frac(2 * k - 1, 2 * D);
        lam[k - 1] = 4.0 * s * s;
        for (int64_t j = 1; j <= N; ++j)
          Q[(j - 1) * n + (k - 1)] = c * wave((bc == 3 ? j : 2 * j - 1) * (2 * k - 1));
      }
      return 0;
    }
    default:
      return -1;
  }
}

// Folding.  A reflection j -> n-1-j maps every eigenvector of a Dirichlet,
// Neumann or periodic operator (suitably phased) to plus or minus itself, so
// a product with the basis splits into one half-size product with the
// symmetric vectors, on x_j + x_{n-1-j}, and one with the antisymmetric ones,
// on x_j - x_{n-1-j}.  On a periodic axis with 4 | n each half is again
// (anti)symmetric about the middle of [0, n/2), which gives four quarters.
// The mixed operators (DN, ND) have no such symmetry.
//
// Groups G in {1, 2, 4}; m = ceil(n/G) positions; group sizes m each, except
// n - m for the antisymmetric group of an odd axis.  The groups' order:
//   G = 2: symmetric, antisymmetric
//   G = 4: x_j + x_{n-1-j} paired by + then - with its mirror h-1-j
//          (h = n/2), then x_j - x_{n-1-j} paired by + then -.
// Chosen to make the padded work (groups x ceil16(m)^2) least, the fewer
// groups on a tie.
int fold_groups(int n, int bc) {
  if (bc == 3 || bc == 4) return 1;
  auto cost = [&](int G) {
    const int64_t p = ((n + G - 1) / G + 15) / 16 * 16;
    return G * p * p;
  };
  int best = 1;
  if (cost(2) < cost(best)) best = 2;
  if (bc == 0 && n % 4 == 0 && cost(4) < cost(best)) best = 4;
  return best;
}

// The eigenbasis in group order: Qh (m x n, row-major) holds the entries of
// the vectors at positions j < m, lam the eigenvalues and perm the index each
// vector has in basis_1d's order (on a periodic axis the vectors are other
// orthonormal pairs of the same eigenspaces, centred on (n-1)/2).
// Q and l are basis_1d's.
int fold_basis(int n, int bc, int G, const double* Q, const double* l, double* Qh, double* lam,
               int* perm) {
  if (n < 3 || !Q || !l || !Qh || !lam || !perm) return -1;
  const int m = (n + G - 1) / G;
  if (G == 1) {
    std::memcpy(Qh, Q, sizeof(double) * (size_t)n * n);
    for (int c = 0; c < n; ++c) perm[c] = c;
  } else if (bc != 0) {
    if (G != 2 || (bc != 1 && bc != 2)) return -1;
    // both lemmas' vectors alternate: columns 0, 2, ... are symmetric
    for (int c = 0; c < n; ++c) {
      const int nat = c < m ? 2 * c : 2 * (c - m) + 1;
      perm[c] = nat;
      for (int j = 0; j < m; ++j)
        Qh[(size_t)j * n + c] = (c >= m && 2 * j == n - 1) ? 0.0 : Q[(size_t)j * n + nat];
    }
  } else {
    // cos and sin of theta = pi k (2j - n + 1) / n
    const int64_t N = n;
    const double c0 = 1.0 / std::sqrt((double)n), c1 = std::sqrt(2.0 / (double)n);
    const int ncos = (n + 1) / 2;               // k = 0 .. ncos - 1
    std::vector<std::pair<int, bool>> order;    // (k, is a cosine)
    if (G == 2) {
      for (int k = 0; k < ncos; ++k) order.push_back({k, true});
      for (int k = 1; k <= n / 2; ++k) order.push_back({k, false});
    } else {
      if (n % 4 != 0) return -1;
      for (int k = 0; k < ncos; k += 2) order.push_back({k, true});
      for (int k = 1; k < ncos; k += 2) order.push_back({k, true});
      for (int k = 1; k <= n / 2; k += 2) order.push_back({k, false});
      for (int k = 2; k <= n / 2; k += 2) order.push_back({k, false});
    }
    if ((int)order.size() != n) return -1;
    const PiTable cosv(true, N), sinv(false, N);
    for (int c = 0; c < n; ++c) {
      const int64_t k = order[c].first;
      const bool cosine = order[c].second;
      const double amp = (k == 0 || 2 * k == N) ? c0 : c1;
      perm[c] = k == 0 ? 0 : (2 * k == N ? n - 1 : (int)(cosine ? 2 * k - 1 : 2 * k));
      for (int64_t j = 0; j < m; ++j) {
        const int64_t a = k * (2 * j - N + 1);
        double v = amp * (cosine ? cosv(a) : sinv(a));
        if (!cosine && 2 * j == N - 1) v = 0.0;
        Qh[(size_t)j * n + c] = v;
      }
    }
  }
  for (int c = 0; c < n; ++c) lam[c] = l[perm[c]];
  return 0;
}

}  // namespace kp
