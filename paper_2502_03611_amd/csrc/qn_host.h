// Host-side eigen-data shared by the single-problem and batched contexts.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <iterator>
#include <vector>

namespace qn {

// Closed-form eigenpairs of h^-2 tridiag(-1, 2, -1) of order n (Section 3.2
// eq. Sy; Section 4.2 with M = I): S[j][k] = sqrt(2/(n+1)) sin((j+1)(k+1) pi/(n+1)),
// lam_k = 4 (n+1)^2 sin^2((k+1) pi / (2(n+1))) (0-based).  The sine argument
// is reduced as an integer first, so S is exactly symmetric.
inline void sine_eigen(int n, std::vector<double>& S, std::vector<double>& lam) {
  const long long m = n + 1;
  const double pi = 3.14159265358979323846;
  S.assign((size_t)n * n, 0.0);
  lam.assign((size_t)n, 0.0);
  const double nrm = std::sqrt(2.0 / (double)m);
  for (int j = 1; j <= n; ++j)
    for (int k = 1; k <= n; ++k) {
      const long long red = ((long long)j * k) % (2 * m);
      S[(size_t)(j - 1) * n + (k - 1)] = nrm * std::sin(pi * (double)red / (double)m);
    }
  for (int k = 1; k <= n; ++k) {
    const double s = std::sin(pi * k / (2.0 * m));
    lam[k - 1] = 4.0 * (double)(m * m) * s * s;
  }
}

inline int fold_block(int n) { return (((n + 1) / 2 + 31) / 32) * 32; }

// Dense padded form: S (p x p, zero outside n x n) and lam (p, padded with lam_max).
inline void dense_eigen(int n, int p, std::vector<double>& Sp, std::vector<double>& lp) {
  std::vector<double> S, lam;
  sine_eigen(n, S, lam);
  Sp.assign((size_t)p * p, 0.0);
  lp.assign((size_t)p, lam[n - 1]);
  for (int j = 0; j < n; ++j) {
    for (int k = 0; k < n; ++k) Sp[(size_t)j * p + k] = S[(size_t)j * n + k];
    lp[j] = lam[j];
  }
}

// Folded forward products of the 3D split-bf16 path: along an axis of n
// points the input is folded about the centre (rows j < hp the mirror sums
// U[j] + U[n-1-j], rows hp + j the differences; the middle row of odd n once),
// hp = ceil(n / 2) rounded up to 32; usable when 2 hp equals the padded
// extent.  Forward operand Sf (2 hp x hp): row t < hp holds even mode 2 t,
// row hp + t odd mode 2 t + 1, each at j < ceil(n / 2) (zero rows for modes
// from n on), from the dense padded S (p x p, S[j][k] = entry j of mode k).
inline int fold_half(int n) { return (((n + 1) / 2 + 31) / 32) * 32; }
inline void fold_forward(int n, int p, const std::vector<double>& Sp, std::vector<double>& Sf) {
  const int hp = fold_half(n), h = (n + 1) / 2;
  Sf.assign((size_t)2 * hp * hp, 0.0);
  for (int pos = 0; pos < 2 * hp; ++pos) {
    const int m = pos < hp ? 2 * pos : 2 * (pos - hp) + 1;
    if (m >= n) continue;
    for (int j = 0; j < h; ++j) Sf[(size_t)pos * hp + j] = Sp[(size_t)j * p + m];
  }
}

// Folded form (block bk): FeT, FoT, Fe, Fo (bk x bk each, concatenated in that
// order) and lam in split order (2 bk, padded with lam_max).
inline void fold_eigen(int n, int bk, std::vector<double>& F4, std::vector<double>& ls) {
  std::vector<double> S, lam;
  sine_eigen(n, S, lam);
  const int h = n / 2, ne = h + (n & 1), no = h;
  const size_t bb = (size_t)bk * bk;
  F4.assign(4 * bb, 0.0);
  double* FeT = F4.data();
  double* FoT = FeT + bb;
  double* Fe = FoT + bb;
  double* Fo = Fe + bb;
  for (int k = 0; k < ne; ++k)
    for (int i = 0; i < ne; ++i) {
      const double v = S[(size_t)k * n + 2 * i];
      FeT[(size_t)k * bk + i] = v;
      Fe[(size_t)i * bk + k] = v;
    }
  for (int k = 0; k < h; ++k)
    for (int i = 0; i < no; ++i) {
      const double v = S[(size_t)k * n + 2 * i + 1];
      FoT[(size_t)k * bk + i] = v;
      Fo[(size_t)i * bk + k] = v;
    }
  ls.assign((size_t)2 * bk, lam[n - 1]);
  for (int i = 0; i < ne; ++i) ls[i] = lam[2 * i];
  for (int i = 0; i < no; ++i) ls[bk + i] = lam[2 * i + 1];
}

// Homogeneous Neumann data (ghost nodes, Section 3.2): the 1D stiffness
// matrix S = h^-2 [2 -2; -1 2 -1; ...; -2 2] of order n is W^-1 K with K
// symmetric and W = diag(1/2, 1, .., 1, 1/2) (Section 4.2 with a diagonal
// mass); its eigenvectors T[j][k] = cos(j k pi / (n - 1)) (integer-reduced
// argument), eigenvalues lam_k = 4 h^-2 sin^2(k pi / (2 (n - 1))) (ih2 = h^-2), and
// T^-1 = diag(1 / c_k) T^T W with c_k = (n - 1) / 2, or n - 1 for k = 0 and
// k = n - 1.  Folded like fold_eigen, with the forward blocks taken from T^-1
// (FeT[j][i] = T^-1[2i][j]) and the inverse blocks from T (Fe[i][j] =
// T[j][2i]): both have the reflection parity of the sine case, because W is
// symmetric about the centre.
inline void fold_cosine(int n, double ih2, int bk, std::vector<double>& F4,
                        std::vector<double>& ls) {
  const long long m = n - 1;
  const double pi = 3.14159265358979323846;
  auto T = [&](int j, int k) {
    const long long red = ((long long)j * k) % (2 * m);
    return std::cos(pi * (double)red / (double)m);
  };
  auto w = [&](int j) { return (j == 0 || j == n - 1) ? 0.5 : 1.0; };
  auto c = [&](int k) { return (k == 0 || k == n - 1) ? (double)m : 0.5 * (double)m; };
  auto Tinv = [&](int k, int j) { return T(j, k) * w(j) / c(k); };
  const int h = n / 2, ne = h + (n & 1), no = h;
  const size_t bb = (size_t)bk * bk;
  F4.assign(4 * bb, 0.0);
  double* FeT = F4.data();
  double* FoT = FeT + bb;
  double* Fe = FoT + bb;
  double* Fo = Fe + bb;
  for (int j = 0; j < ne; ++j)
    for (int i = 0; i < ne; ++i) {
      FeT[(size_t)j * bk + i] = Tinv(2 * i, j);
      Fe[(size_t)i * bk + j] = T(j, 2 * i);
    }
  for (int j = 0; j < h; ++j)
    for (int i = 0; i < no; ++i) {
      FoT[(size_t)j * bk + i] = Tinv(2 * i + 1, j);
      Fo[(size_t)i * bk + j] = T(j, 2 * i + 1);
    }
  std::vector<double> lam((size_t)n);
  for (int k = 0; k < n; ++k) {
    const double s = std::sin(pi * (double)k / (2.0 * (double)m));
    lam[k] = 4.0 * ih2 * s * s;
  }
  ls.assign((size_t)2 * bk, lam[n - 1]);
  for (int i = 0; i < ne; ++i) ls[i] = lam[2 * i];
  for (int i = 0; i < no; ++i) ls[bk + i] = lam[2 * i + 1];
}

// ---------------------------------------------------------------- spectral elements
// Q^k spectral elements with Gauss-Lobatto nodes (Section 3.1 and the remark on
// Gauss-Lobatto integration; Section 4.2 for the diagonalisation).

// Gauss-Lobatto nodes (ascending) and weights of order k >= 1 on [-1, 1]: the
// two ends and the k - 1 roots of P_k', found by Newton's method on P_k' (P_k''
// from Legendre's equation) from the Chebyshev-Lobatto points; weights
// 2 / (k (k + 1) P_k(x)^2).
inline void gl_nodes(int k, std::vector<double>& x, std::vector<double>& w) {
  const double pi = 3.14159265358979323846;
  auto legendre = [k](double t, double& pk, double& dpk) {
    double p0 = 1.0, p1 = t;
    if (k == 0) { pk = 1.0; dpk = 0.0; return; }
    for (int j = 1; j < k; ++j) {
      const double p2 = ((2.0 * j + 1.0) * t * p1 - j * p0) / (j + 1.0);
      p0 = p1;
      p1 = p2;
    }
    pk = p1;
    dpk = k * (t * p1 - p0) / (t * t - 1.0);  // interior points only
  };
  x.assign((size_t)k + 1, 0.0);
  w.assign((size_t)k + 1, 0.0);
  x[0] = -1.0;
  x[k] = 1.0;
  for (int j = 1; j < k; ++j) {
    double t = -std::cos(pi * j / k);
    for (int it = 0; it < 100; ++it) {
      double pk, dpk;
      legendre(t, pk, dpk);
      const double d2 = (2.0 * t * dpk - k * (k + 1.0) * pk) / (1.0 - t * t);
      const double step = dpk / d2;
      t -= step;
      if (std::fabs(step) < 1e-16) break;
    }
    x[j] = t;
  }
  for (int j = 0; j <= k; ++j) {
    double p0 = 1.0, p1 = x[j];
    for (int i = 1; i < k; ++i) {
      const double p2 = ((2.0 * i + 1.0) * x[j] * p1 - i * p0) / (i + 1.0);
      p0 = p1;
      p1 = p2;
    }
    const double pk = k == 0 ? 1.0 : p1;
    w[j] = 2.0 / (k * (k + 1.0) * pk * pk);
  }
}

// One axis: E elements of order k on [0, L]; lumped mass m and dense
// stiffness S of the unknown nodes (Dirichlet: the E k - 1 interior nodes;
// Neumann: all E k + 1).
inline void sem_axis(int elements, int k, double length, bool neumann, std::vector<double>& m,
                     std::vector<double>& S, std::vector<double>* nodes = nullptr) {
  std::vector<double> xi, w;
  gl_nodes(k, xi, w);
  const int nq = k + 1;
  std::vector<double> D((size_t)nq * nq);  // D[q][p] = psi_p'(xi_q)
  for (int q = 0; q < nq; ++q)
    for (int p = 0; p < nq; ++p) {
      if (p == q) {
        double v = 0.0;
        for (int r = 0; r < nq; ++r)
          if (r != p) v += 1.0 / (xi[p] - xi[r]);
        D[(size_t)q * nq + p] = v;
      } else {
        double num = 1.0, den = 1.0;
        for (int r = 0; r < nq; ++r) {
          if (r != p && r != q) num *= xi[q] - xi[r];
          if (r != p) den *= xi[p] - xi[r];
        }
        D[(size_t)q * nq + p] = num / den;
      }
    }
  const double jac = 0.5 * length / elements;
  const int ntot = elements * k + 1;
  std::vector<double> mt((size_t)ntot, 0.0), st((size_t)ntot * ntot, 0.0);
  for (int e = 0; e < elements; ++e)
    for (int p = 0; p < nq; ++p) {
      const int gp = e * k + p;
      mt[gp] += w[p] * jac;
      for (int r = 0; r < nq; ++r) {
        double v = 0.0;
        for (int q = 0; q < nq; ++q) v += w[q] * D[(size_t)q * nq + p] * D[(size_t)q * nq + r];
        st[(size_t)gp * ntot + e * k + r] += v / jac;
      }
    }
  const int lo = neumann ? 0 : 1, n = neumann ? ntot : ntot - 2;
  if (nodes) {
    nodes->assign((size_t)n, 0.0);
    for (int i = 0; i < n; ++i) {
      const int g = lo + i, e = std::min(g / k, elements - 1), q = g - e * k;
      (*nodes)[i] = (2.0 * e + 1.0 + xi[q]) * jac;
    }
  }
  m.assign((size_t)n, 0.0);
  S.assign((size_t)n * n, 0.0);
  for (int i = 0; i < n; ++i) {
    m[i] = mt[lo + i];
    for (int j = 0; j < n; ++j) S[(size_t)i * n + j] = st[(size_t)(lo + i) * ntot + lo + j];
  }
}

// Symmetric eigen-decomposition A = Q diag(d) Q^T by cyclic Jacobi rotations
// (A: n x n row-major, destroyed); columns of Q are the eigenvectors, sorted
// by ascending eigenvalue.
inline void jacobi_eigen(int n, std::vector<double>& A, std::vector<double>& Q,
                         std::vector<double>& d) {
  Q.assign((size_t)n * n, 0.0);
  for (int i = 0; i < n; ++i) Q[(size_t)i * n + i] = 1.0;
  auto a = [&](int i, int j) -> double& { return A[(size_t)i * n + j]; };
  double scale = 0.0;
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) scale += a(i, j) * a(i, j);
  scale = std::sqrt(scale);
  for (int sweep = 0; sweep < 60; ++sweep) {
    double off = 0.0;
    for (int i = 0; i < n; ++i)
      for (int j = i + 1; j < n; ++j) off += a(i, j) * a(i, j);
    if (std::sqrt(off) <= 1e-17 * scale) break;
    for (int p = 0; p < n; ++p)
      for (int q = p + 1; q < n; ++q) {
        const double apq = a(p, q);
        if (std::fabs(apq) <= 1e-300 * scale) continue;
        // rotation angle that zeroes a(p, q): tan from the smaller root
        const double theta = (a(q, q) - a(p, p)) / (2.0 * apq);
        const double t = (theta >= 0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
        const double c = 1.0 / std::sqrt(t * t + 1.0), sn = t * c;
        for (int r = 0; r < n; ++r) {  // columns p, q
          const double arp = a(r, p), arq = a(r, q);
          a(r, p) = c * arp - sn * arq;
          a(r, q) = sn * arp + c * arq;
        }
        for (int r = 0; r < n; ++r) {  // rows p, q
          const double apr = a(p, r), aqr = a(q, r);
          a(p, r) = c * apr - sn * aqr;
          a(q, r) = sn * apr + c * aqr;
        }
        a(p, q) = a(q, p) = 0.0;
        for (int r = 0; r < n; ++r) {
          const double vp = Q[(size_t)r * n + p], vq = Q[(size_t)r * n + q];
          Q[(size_t)r * n + p] = c * vp - sn * vq;
          Q[(size_t)r * n + q] = sn * vp + c * vq;
        }
      }
  }
  std::vector<int> order((size_t)n);
  for (int i = 0; i < n; ++i) order[i] = i;
  std::sort(order.begin(), order.end(), [&](int x, int y) { return a(x, x) < a(y, y); });
  std::vector<double> Qs((size_t)n * n);
  d.assign((size_t)n, 0.0);
  for (int c = 0; c < n; ++c) {
    d[c] = a(order[c], order[c]);
    for (int r = 0; r < n; ++r) Qs[(size_t)r * n + c] = Q[(size_t)r * n + order[c]];
  }
  Q.swap(Qs);
}

// Folded eigen-data of H = M^-1 S for a reflection-symmetric axis (uniform
// elements): B = M^-1/2 S M^-1/2 is split into its even block (basis
// (e_j + e_{n-1-j}) / sqrt 2, j < n/2, and the centre e_{n/2} for odd n) and its
// odd block ((e_j - e_{n-1-j}) / sqrt 2), each diagonalised by Jacobi; with
// T = M^-1/2 T~ and T^-1 = T~^T M^1/2 (Section 4.2) the blocks are laid out as
// the folded kernels read them: FeT[j][i] = T^-1[i][j], Fe[i][j] = T[j][i] for
// even modes i and folded nodes j (FoT, Fo likewise for odd modes); lam in
// split spectral order, padded with lam_max.  Returns lam_min.
inline double fold_sem(int n, const std::vector<double>& m, const std::vector<double>& S, int bk,
                       std::vector<double>& F4, std::vector<double>& ls) {
  const int h = n / 2, ne = h + (n & 1), no = h;
  const double r2 = std::sqrt(0.5);
  auto B = [&](int i, int j) { return S[(size_t)i * n + j] / std::sqrt(m[i] * m[j]); };
  std::vector<double> Be((size_t)ne * ne), Bo((size_t)no * no);
  for (int a = 0; a < ne; ++a)
    for (int b = 0; b < ne; ++b) {
      double v;
      if (a < h && b < h)
        v = 0.5 * (B(a, b) + B(a, n - 1 - b) + B(n - 1 - a, b) + B(n - 1 - a, n - 1 - b));
      else if (a < h)  // b is the centre
        v = r2 * (B(a, b) + B(n - 1 - a, b));
      else if (b < h)
        v = r2 * (B(a, b) + B(a, n - 1 - b));
      else
        v = B(a, b);
      Be[(size_t)a * ne + b] = v;
    }
  for (int a = 0; a < no; ++a)
    for (int b = 0; b < no; ++b)
      Bo[(size_t)a * no + b] =
          0.5 * (B(a, b) - B(a, n - 1 - b) - B(n - 1 - a, b) + B(n - 1 - a, n - 1 - b));
  std::vector<double> Qe, de, Qo, dd;
  jacobi_eigen(ne, Be, Qe, de);
  jacobi_eigen(no, Bo, Qo, dd);
  const size_t bb = (size_t)bk * bk;
  F4.assign(4 * bb, 0.0);
  double* FeT = F4.data();
  double* FoT = FeT + bb;
  double* Fe = FoT + bb;
  double* Fo = Fe + bb;
  for (int i = 0; i < ne; ++i)
    for (int j = 0; j < ne; ++j) {
      const double t = (j < h ? r2 : 1.0) * Qe[(size_t)j * ne + i];  // T~ entry at node j
      FeT[(size_t)j * bk + i] = t * std::sqrt(m[j]);
      Fe[(size_t)i * bk + j] = t / std::sqrt(m[j]);
    }
  for (int i = 0; i < no; ++i)
    for (int j = 0; j < no; ++j) {
      const double t = r2 * Qo[(size_t)j * no + i];
      FoT[(size_t)j * bk + i] = t * std::sqrt(m[j]);
      Fo[(size_t)i * bk + j] = t / std::sqrt(m[j]);
    }
  double lmax = de.empty() ? 0.0 : de.back(), lmin = de.empty() ? 0.0 : de.front();
  if (!dd.empty()) {
    lmax = std::max(lmax, dd.back());
    lmin = std::min(lmin, dd.front());
  }
  ls.assign((size_t)2 * bk, lmax);
  for (int i = 0; i < ne; ++i) ls[i] = de[i];
  for (int i = 0; i < no; ++i) ls[bk + i] = dd[i];
  return lmin;
}

// Banded H = M^-1 S of one axis: Hb[j][d + k] = H[j][j + d], |d| <= k (0 off the grid).
inline void sem_band(int n, int k, const std::vector<double>& m, const std::vector<double>& S,
                     std::vector<double>& Hb) {
  const int w = 2 * k + 1;
  Hb.assign((size_t)n * w, 0.0);
  for (int j = 0; j < n; ++j)
    for (int d = -k; d <= k; ++d)
      if (j + d >= 0 && j + d < n) Hb[(size_t)j * w + d + k] = S[(size_t)j * n + j + d] / m[j];
}

inline uint16_t bf16_rne(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

inline float bf16_value(uint16_t h) {
  uint32_t u = (uint32_t)h << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}

// Multiply-adds of an unrolled stage of the factored transforms (qn_fast.h):
// even lengths halve, odd ones are contracted.
inline double fast_work(int q) {
  double w = 0.0;
  for (; q > 2 && q % 2 == 0; q /= 2) w += q * q / 8.0 + 1.5 * q;
  return w + (q > 2 ? q * q / 2.0 + q : q);
}

// Stage lengths of the factored transform of an axis of N intervals
// (qn_fast.hip): 2N = Q R, both instantiated, with the fewest multiply-adds
// per point; false when 2N has no such factorisation.
inline bool fast_stages(int N, int* Qo, int* Ro) {
  static const int big[] = {20, 24, 28, 30, 32, 36, 40, 44, 48, 50, 52, 56, 60, 64};
  auto is_big = [](int q) { return std::find(std::begin(big), std::end(big), q) != std::end(big); };
  double best = 1e300;
  for (int q = 4; q <= 64; ++q) {
    if ((2 * N) % q != 0) continue;
    const int r = 2 * N / q;
    const bool small = q <= 32 && r >= 4 && r <= 32;
    if (!small && !(is_big(q) && is_big(r))) continue;
    // two even lengths, then any to 32, then the longer ones: fewer registers
    // per thread, so more waves in flight
    const double w = fast_work(q) / q + fast_work(r) / r + (!small ? 1e6 : ((q | r) & 1) ? 1e3 : 0.0);
    if (w < best) {
      best = w;
      *Qo = q;
      *Ro = r;
    }
  }
  return best < 1e300;
}

// Device tables of a factored axis: twiddle pairs (see FastAxis) and the
// eigenvalues 4 h^-2 sin^2(pi k / 2N) of the modes k = 0 .. 2N - 1, continued
// evenly (k = 0 and N do not exist for Dirichlet data and get the largest).
inline void fast_tables(int N, int Q, int R, bool neumann, double ih2, std::vector<double>& tw,
                        std::vector<double>& lam) {
  const double pi = 3.14159265358979323846, nrm = std::sqrt(2.0 / N);
  const int nt = (Q / 2) * (R / 2) + 1;
  tw.resize(2 * (size_t)nt);
  for (int i = 0; i < nt; ++i) {  // i <= N / 2
    const double c = nrm * (2 * i == N ? 0.0 : std::cos(pi * i / N)), s = nrm * std::sin(pi * i / N);
    tw[2 * i] = neumann ? -s : c;
    tw[2 * i + 1] = neumann ? c : s;
  }
  lam.resize(2 * (size_t)N);
  for (int k = 0; k <= N; ++k) {
    const double s = std::sin(pi * k / (2.0 * N));
    lam[k] = 4.0 * ih2 * s * s;
  }
  if (!neumann) lam[0] = lam[N] = lam[N - 1];
  for (int k = N + 1; k < 2 * N; ++k) lam[k] = lam[2 * N - k];
}

// Whether the factored axes of a small grid stay factored (else every axis takes
// its dense product).  A thread walks the two stages of its class alone, a chain
// of work(Q) + work(R) multiply-adds; where a dense product is a single launch of
// few tiles, that chain is the longer one for prime-like stages (4 x 23, 4 x 29,
// 4 x 31, 5 x 26).  chain: its length per factored axis, 0 for dense ones.  The
// lines lie where an iteration bound by the GPU takes as long either way (us,
// dense and factored; where the host bounds the launches a factored solve saves
// one more of them, 45^2 33 and 33):
//   2D, at most two tiles per axis, both factored: 57 x 63 (chains of 576 in all)
//   29.2 and 29.3, 45^2 (596) 29.2 and 30.0, 61^2 (1044) 29.4 and 33.4; 92^2 (1064)
//   34.0 and 34.1.  Only y, which saves a launch: 57 x 72 (460) 33.1 and 33.0, 61 x 58
//   (522) 29.4 and 30.5.  Only x, which saves none: 100 x 127 (172) 33.9 and 32.0, 100 x
//   123 (542) 34.0 and 34.4, a solve 20.4 and 22.6.
//   3D, one tile per axis: 51^3 (693) 43.4 and 43.7, 64^3 (714) 43.5 and 44.6, 61 x 63 x
//   63 (754) 43.7 and 45.1, 57^3 (1380) 43.5 and 49.0; 61 x 58 x 58 with z alone 47.9 and
//   45.2, two factored axes have two thirds of the limit (61 x 61 x 58, 1044: 43.5 and
//   45.8; 63 x 63 x 58, 232: 47.6 and 45.9); two fields, where the dense launches carry twice the padding: 45^3 (894)
//   46.6 and 46.4, 64^3 51.0 and 52.0.  One axis of two tiles: 127 x 61 x 31 (754) 52.6
//   and 48.4, 127 x 61 x 61 (1216) 53.4 and 54.7.
inline bool fast_pays(int dim, const int* n, const int* p, const double* chain, int fields) {
  double sum = 0.0, values = 1.0, padded = 1.0;
  int count = 0, tiles = 0, most = 0, sides = 0;
  for (int a = 0; a < dim; ++a) {
    sum += chain[a];
    count += chain[a] > 0.0;
    values *= n[a];
    padded *= p[a];
    tiles += p[a] / 64;
    most = std::max(most, p[a]);
    if (chain[a] > 0.0) sides += p[a];
  }
  if (count == 0 || most > 128 || tiles > 4) return true;
  if (dim == 2) return sum <= (count == 2 ? 4.55 : chain[1] > 0.0 ? 7.3 : 3.0) * sides;
  if (count == 1) return true;
  if (fields > 1) sum *= values / padded;
  return sum <= (tiles == 3 ? 700.0 : 1024.0) * count / 3.0;
}

// The same for the classes of a batch, `planes` fields of n^2 points in all.  While
// a line pass is one round of workgroups with room to spare (two per CU, 16 lines
// each) it is a launch that its chain is part of: 61^2 (chain of 522) x 80 instances
// 50 us an iteration both ways, 64^2 (238) x 100 52 and 49.  Beyond, the factored
// passes' arithmetic counts, over n^2 points of the 64^2 that a dense tile pads to:
// 61^2 x 128 51 dense and 54 factored, x 1127 196 and 243, 64^2 x 180 57 and 64; 56^2
// (220) x 1024 155 and 162, 62^2 (148) x 1091 193 and 193.
inline bool fast_pays_batched(int n, double chain, double planes) {
  return n > 64 || planes * ((n + 15) / 16) <= 448.0 || chain * n * n <= 165.0 * 4096.0;
}

// Whether the dense products of a solve take the strip form (qn_gemm_strip.h):
// when the padded tiles do enough more matrix-core operations than the strips,
// whose rate is 0.8-0.9 of the tiles' (255^3 0.73 against 0.67 ms at a ratio of
// 1.0; 400^3 3.9 and 6.6 ms at 1.35, 200^3 0.40 and 0.52 ms at 1.9).  On smaller
// grids a strip launch leaves the chip to too few waves and the ratio has to be
// larger.  3D from 2^18 to 2^20 values: 2.1 in FP64 (60 x 70 x 64, 1.8: 60 and 54
// us an iteration; 66 x 31 x 200, 4.7: 72 and 126; 66^3, 5.1: 67 and 114); in FP32,
// whose tiles are faster, only from 2^27 operations of the tiles on (60 x 35 x 66
// of two fields, 0.87 of that, 2.7: 63 and 60; 164 x 31 x 63, 0.84, 2.3: 66 and
// 57.5; 66 x 36 x 127, 1.1, 3.2: 64 and 66), at a ratio of 2.4 up to 2^28 (217 x 63 x
// 31, 2.25: 70 and 65; 274 x 63 x 31, 2.26: 82 and 74; 96 x 66 x 31 of two fields,
// 4.7: 66 and 84) and 2.1 beyond (66 x 109 x 63 of two fields, 2.1: 78 and 85).
// From 2^20 to 2^22 values in FP32 1.75 in 3D where x pads to the tile's 128 (63 x
// 214 x 72 of two fields, 1.64: 128 and 123; 127 x 198 x 89, 1.69: 131 and 126; 66 x
// 127 x 127, 1.84: 88 and 92), else 1.5 (275 x 44 x 175, 1.67: 0.83 of the tiles'
// time; batches of 95^2 x 132, 1.68: 79 and 87, 194^2 x 31, 1.57: 89 and 93, x 92: 147
// and 143 but 100 and 105 a solve).  From there to 2^24 1.4 and 1.27 (254 x 254 x 66,
// 1.38: 239 and 214; 254 x 130 x 127 of two fields, 1.44: 271 and 288; 127 x 313 x 130,
// 1.26: 242 and 234; 280 x 63 x 277, 1.27: 210 and 226), 1.33 in 2D (batches of 222^2 x
// 121, 1.29: 185 and 170, 210^2 x 136, 1.4: 194 and 210).
// Below 2^18 values, in 2D below 2^20, never (52^3 35 against 29 us a solve, 200^2 46
// and 36, 390^2 58 and 51).
// Row strides stay below 2^26 elements (32-bit lane offsets of three rows).  n,
// p, dense: extents, padded extents and which axes have a dense product.
inline bool use_strips(int dim, const int* n, const int* p, const bool* dense, int fields,
                       bool fp32) {
  double values = fields, tiles = 0.0, strips = 0.0;
  for (int a = 0; a < dim; ++a) values *= n[a];
  if (values < (dim == 3 ? 262144.0 : 1048576.0) || (dim == 3 && (double)p[0] * p[1] >= 67108864.0)) return false;
  auto up16 = [](int v) { return (v + 15) / 16 * 16; };
  for (int a = 0; a < dim; ++a) {
    if (!dense[a]) continue;
    const int ne = (n[a] + 1) / 2;
    double t = (double)fields * p[a] * up16(ne), s = 2.0 * fields * up16(ne) * (ne + 3);
    for (int b = 0; b < dim; ++b)
      if (b != a) {
        t *= p[b];
        s *= b == 0 ? 2.0 * up16((n[0] + 1) / 2) : (double)n[b];
      }
    tiles += t;
    strips += s;
  }
  double least = 1.25;
  if (values < 1048576.0) {
    if (fp32 && tiles < 134217728.0) return false;
    least = fp32 && tiles < 268435456.0 ? 2.4 : 2.1;
  } else if (values < 16777216.0 && fp32) {
    const bool full = dim == 3 && p[0] % 128 == 0;
    least = values < 4194304.0 ? (full ? 1.75 : 1.5) : full ? 1.4 : dim == 3 ? 1.27 : 1.33;
  }
  return tiles > least * strips;
}

}  // namespace qn
