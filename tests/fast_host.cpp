// Host build of the factored transform's stages (csrc/qn_fast.h) for every
// interval count the host rule accepts, against the defining sums, with every
// element access checked against its line.  Usage: fast_host <lo> <hi>;
// prints "<N> <sym> <Q> <R> <max error / bound>" and exits non-zero on a fault.
#define __device__
#define __forceinline__ inline
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "qn_fast.h"
#include "qn_host.h"

using namespace qn;

template <typename T>
struct Checked {  // stands in for the kernels' element pointers
  std::vector<T>* v;
  long long at;
  Checked operator+(long long d) const { return {v, at + d}; }
  T& at_byte(unsigned b) const {
    const long long k = at + (long long)(b / sizeof(T));
    if (k < 0 || k >= (long long)v->size()) {
      std::printf("out of range: %lld of %zu\n", k, v->size());
      std::exit(2);
    }
    return (*v)[(size_t)k];
  }
};

template <typename T>
T ld(Checked<T> s, unsigned off) { return s.at_byte(off); }

template <int Q, typename T>
void one_stage1(Checked<T> base, int N, int R, int off, T sg, long long es, int line,
                const Pair<T>* tw, Pair<T>* lds) {
  const int rh = R / 2;
  for (int b = 0; b <= rh; ++b) {
    T x[Q];
    load_class<Q, T>(base, (unsigned)sizeof(T) * (unsigned)(line + b * es),
                     (unsigned)sizeof(T) * (unsigned)(line + (rh - b) * es), N, R, b, off, sg, es, x);
    stage1_emit<Q, T>(x, tw, b, [&](int k, T p, T q) { lds[k * (rh + 1) + b] = {p, q}; });
  }
}

template <int R, typename T>
void one_stage2(const Pair<T>* lds, int Q, int N, int off, T sg, std::vector<T>& out,
                std::vector<int>& hits) {
  for (int k1 = 0; k1 <= Q / 2; ++k1) {
    T v[R];
    T p[33], q[33];
    for (int b = 0; b <= R / 2; ++b) {
      p[b] = lds[(R / 2 + 1) * k1 + b].p;
      q[b] = lds[(R / 2 + 1) * k1 + b].q;
    }
    stage2<R, T>(p, q, v);
    for_modes<R>(Q, N, k1, off, [&](int k2, int u, bool mir) {
      const int pos = u + (mir ? Q / 2 - k1 : k1);
      if (pos < 0 || pos >= (int)out.size()) {
        std::printf("mode out of range: %d of %zu\n", pos, out.size());
        std::exit(2);
      }
      out[pos] = mir ? sg * v[k2] : v[k2];
      ++hits[pos];
    });
  }
}

template <typename T>
double check(int N, int Q, int R, bool neumann) {
  const int off = neumann ? 0 : 1, n = neumann ? N + 1 : N - 1;
  const T sg = neumann ? T(1) : T(-1);
  std::vector<double> twd, lam;
  fast_tables(N, Q, R, neumann, 1.0, twd, lam);
  std::vector<Pair<T>> tw(twd.size() / 2), lds((size_t)(Q / 2 + 1) * (R / 2 + 1));
  for (size_t i = 0; i < tw.size(); ++i) tw[i] = {(T)twd[2 * i], (T)twd[2 * i + 1]};
  const long long es = 3;  // three interleaved lines, the middle one transformed
  std::vector<T> x((size_t)n * 3, T(NAN)), out(n, T(NAN));
  std::vector<int> hits(n, 0);
  for (int j = 0; j < n; ++j) x[3 * j + 1] = (T)std::sin(1.7 * j * j + 0.3 * N);
  Checked<T> base{&x, 0};
  switch (Q) {
#define X(L) case L: one_stage1<L, T>(base, N, R, off, sg, es, 1, tw.data(), lds.data()); break;
    X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17) X(18) X(19) X(20)
    X(21) X(22) X(23) X(24) X(25) X(26) X(27) X(28) X(29) X(30) X(31) X(32) X(36) X(40) X(44) X(48)
    X(50) X(52) X(56) X(60) X(64)
#undef X
    default: std::exit(3);
  }
  switch (R) {
#define X(L) case L: one_stage2<L, T>(lds.data(), Q, N, off, sg, out, hits); break;
    X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17) X(18) X(19) X(20)
    X(21) X(22) X(23) X(24) X(25) X(26) X(27) X(28) X(29) X(30) X(31) X(32) X(36) X(40) X(44) X(48)
    X(50) X(52) X(56) X(60) X(64)
#undef X
    default: std::exit(3);
  }
  // every mode once; S x = sqrt(2/N) sum'' x_j sin / cos(pi j k / N), the ends of Neumann data halved
  double err = 0.0;
  const double nx = std::sqrt((double)n);  // ||x||_2 <= sqrt(n), so |S x| <= nx too
  const int stride = n > 300 ? 7 : 1;
  for (int p = 0; p < n; ++p) {
    if (hits[p] != 1) {
      std::printf("mode %d written %d times (N %d)\n", p, hits[p], N);
      std::exit(2);
    }
    if (p % stride != 0 && p != n - 1) continue;
    long double s = 0.0L;
    for (int j = 0; j < n; ++j) {
      const long long red = ((long long)(j + off) * (p + off)) % (2 * N);
      const long double t = 3.14159265358979323846264338327950288L * red / N;
      const long double w = neumann && (j == 0 || j == n - 1) ? 0.5L : 1.0L;
      s += w * (long double)x[3 * j + 1] * (neumann ? cosl(t) : sinl(t));
    }
    s *= sqrtl(2.0L / N);
    err = std::max(err, (double)fabsl((long double)out[p] - s));
  }
  // two stages of at most 64-term sums: (64 + 64 + 8) roundings of terms bounded by ||x||
  return err / (136.0 * std::ldexp(1.0, -53) * nx);
}

int main(int argc, char** argv) {
  const int lo = std::atoi(argv[1]), hi = std::atoi(argv[2]);
  for (int N = lo; N <= hi; ++N) {
    int Q = 0, R = 0;
    if (!fast_stages(N, &Q, &R)) continue;
    for (int sym = 0; sym < 2; ++sym)
      std::printf("%d %d %d %d %.4f\n", N, sym, Q, R, check<double>(N, Q, R, sym == 1));
  }
  return 0;
}
