// Stages of the factored mode products (qn_fast.hip): fully unrolled real
// DFTs of short fixed length with compile-time coefficients, and the classes
// of a line that one thread loads and stores.  Also compiled for the host by
// its test (tests/fast_host.cpp).
#pragma once

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#endif

// Instantiated stage lengths, one kernel per list (a pair (Q, R) needs both in
// the same list): even lengths to 32, which need at most 128 registers, all
// lengths to 32, and longer stages.
#define QN_FAST_EVEN(X) X(4) X(6) X(8) X(10) X(12) X(14) X(16) X(18) X(20) X(22) X(24) X(26) X(28) X(30) X(32)
#define QN_FAST_ODD(X) X(5) X(7) X(9) X(11) X(13) X(15) X(17) X(19) X(21) X(23) X(25) X(27) X(29) X(31)
#define QN_FAST_BIG(X) X(20) X(24) X(28) X(30) X(32) X(36) X(40) X(44) X(48) X(50) X(52) X(56) X(60) X(64)

namespace qn {

// cos and sin of 2 pi k / q by octant reduction in integers and a Taylor sum
// on [0, pi/4] (truncation below 2^-60), evaluated at compile time.
constexpr double fx_sin_small(double x) {
  double s = 1.0;
  for (int i = 19; i >= 3; i -= 2) s = 1.0 - x * x / (double)(i * (i - 1)) * s;
  return x * s;
}
constexpr double fx_cos_small(double x) {
  double s = 1.0;
  for (int i = 20; i >= 2; i -= 2) s = 1.0 - x * x / (double)(i * (i - 1)) * s;
  return s;
}
constexpr double kFxTwoPi = 6.283185307179586476925286766559;
// angle = 2 pi num / den with den = 8 q, num = 8 k reduced to [0, den / 8]
constexpr double fx_sin(int k, int q);
constexpr double fx_cos(int k, int q) {
  const int den = 8 * q;
  int num = 8 * (((k % q) + q) % q);
  if (2 * num > den) num = den - num;  // cos(2 pi - t) = cos t
  bool neg = false;
  if (4 * num > den) {  // cos(pi - t) = -cos t
    num = den / 2 - num;
    neg = true;
  }
  const double v = 8 * num > den ? fx_sin_small(kFxTwoPi * (den / 4 - num) / den)
                                 : fx_cos_small(kFxTwoPi * num / den);
  return neg ? -v : v;
}
constexpr double fx_sin(int k, int q) { return fx_cos(4 * k - q, 4 * q); }  // cos(t - pi/2)

template <int Q>
struct FxTab {
  double c[Q], s[Q];
  constexpr FxTab() : c(), s() {
    for (int k = 0; k < Q; ++k) {
      c[k] = fx_cos(k, Q);
      s[k] = fx_sin(k, Q);
    }
  }
};

// Real DFT of x[0 .. Q-1]: emit(k * STEP, C_k, S_k) for k = 0 .. Q/2 with
// C_k = sum x_a cos(2 pi a k / Q), S_k = sum x_a sin(2 pi a k / Q).  Even
// lengths split off the odd k (contracted about Q/4: Q^2/8 multiply-adds) and
// recurse on x_a + x_{a + Q/2} for the even k; odd lengths are contracted
// about their centre (Q^2/2).
template <int Q, int STEP, typename T, typename E>
__device__ __forceinline__ void rdft(const T (&x)[Q], E&& emit) {
  static constexpr FxTab<Q> tab{};
  if constexpr (Q == 1) {
    emit(0, x[0], T(0));
  } else if constexpr (Q == 2) {
    emit(0, x[0] + x[1], T(0));
    emit(STEP, x[0] - x[1], T(0));
  } else if constexpr (Q % 2 == 0) {
    constexpr int H = Q / 2, A = (H - 1) / 2;  // pairs a, H - a with 1 <= a <= A
    const T z0 = x[0] - x[H];
    T u[A + 1], v[A + 1];
    u[0] = v[0] = T(0);
#pragma unroll
    for (int a = 1; a <= A; ++a) {
      const T za = x[a] - x[a + H], zb = x[H - a] - x[Q - a];
      u[a] = za - zb;
      v[a] = za + zb;
    }
    T zm = T(0);
    if constexpr (H % 2 == 0) zm = x[H / 2] - x[H / 2 + H];
#pragma unroll
    for (int k = 1; k <= H; k += 2) {
      T C = z0, S = T(0);
      if constexpr (H % 2 == 0) S = (k & 2) ? -zm : zm;
#pragma unroll
      for (int a = 1; a <= A; ++a) {
        C += u[a] * T(tab.c[(a * k) % Q]);
        if (k != H) S += v[a] * T(tab.s[(a * k) % Q]);
      }
      emit(k * STEP, C, S);
    }
    T y[H];
#pragma unroll
    for (int a = 0; a < H; ++a) y[a] = x[a] + x[a + H];
    rdft<H, 2 * STEP>(y, emit);
  } else {
    constexpr int A = (Q - 1) / 2;
    T u[A + 1], v[A + 1], c0 = x[0];
    u[0] = v[0] = T(0);
#pragma unroll
    for (int a = 1; a <= A; ++a) {
      u[a] = x[a] + x[Q - a];
      v[a] = x[a] - x[Q - a];
      c0 += u[a];
    }
    emit(0, c0, T(0));
#pragma unroll
    for (int k = 1; k <= A; ++k) {
      T C = x[0], S = T(0);
#pragma unroll
      for (int a = 1; a <= A; ++a) {
        C += u[a] * T(tab.c[(a * k) % Q]);
        S += v[a] * T(tab.s[(a * k) % Q]);
      }
      emit(k * STEP, C, S);
    }
  }
}

// out[k] = p[0] + (R even) (-1)^k p[STEP R/2] + sum_{0 < b < R/2}
// (p[b STEP] cos(2 pi b k / R) + q[b STEP] sin(2 pi b k / R)), k = 0 .. R-1:
// the transpose of rdft, split by the parity of b.
template <int R, int STEP, typename T, int PB>
__device__ __forceinline__ void irdft(const T (&p)[PB], const T (&q)[PB], T (&out)[R]) {
  static constexpr FxTab<R> tab{};
  if constexpr (R == 1) {
    out[0] = p[0];
  } else if constexpr (R == 2) {
    out[0] = p[0] + p[STEP];
    out[1] = p[0] - p[STEP];
  } else if constexpr (R % 2 == 0) {
    constexpr int H = R / 2;
    T F[H];
#pragma unroll
    for (int k = 0; k <= H / 2; ++k) {
      T c = T(0), s = T(0);
      if constexpr (H % 2 == 1) c = (k & 1) ? -p[H * STEP] : p[H * STEP];
#pragma unroll
      for (int b = 1; b < H; b += 2) {
        if (4 * k != R) c += p[b * STEP] * T(tab.c[(b * k) % R]);
        if (k != 0) s += q[b * STEP] * T(tab.s[(b * k) % R]);
      }
      if (k == 0)
        F[0] = c;
      else if (4 * k == R)
        F[k] = s;
      else {
        F[k] = s + c;
        F[H - k] = s - c;
      }
    }
    T g[H];
    irdft<H, 2 * STEP>(p, q, g);
#pragma unroll
    for (int k = 0; k < H; ++k) {
      out[k] = g[k] + F[k];
      out[k + H] = g[k] - F[k];
    }
  } else {
    constexpr int A = (R - 1) / 2;
    T c0 = p[0];
#pragma unroll
    for (int b = 1; b <= A; ++b) c0 += p[b * STEP];
    out[0] = c0;
#pragma unroll
    for (int k = 1; k <= A; ++k) {
      T c = p[0], s = T(0);
#pragma unroll
      for (int b = 1; b <= A; ++b) {
        c += p[b * STEP] * T(tab.c[(b * k) % R]);
        s += q[b * STEP] * T(tab.s[(b * k) % R]);
      }
      out[k] = c + s;
      out[R - k] = c - s;
    }
  }
}

template <typename T>
struct alignas(2 * sizeof(T)) Pair {  // twiddle
  T p, q;
};

// Element at byte offset `off` from a workgroup-uniform address: kept apart
// so that the address stays in scalar registers.
template <typename T>
__device__ __forceinline__ T ld(const T* s, unsigned off) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(s) + off);
}
template <typename T>
__device__ __forceinline__ void st(T* s, unsigned off, T v) {
  *reinterpret_cast<T*>(reinterpret_cast<char*>(s) + off) = v;
}

// Loads the class b of one line for a stage of length Q over stride R:
// x[a] = continued x at j = R a + b.  base: position 0 of the workgroup's
// first line (uniform); voff, moff: byte offsets of the line plus b (R/2 - b)
// axis strides es.
template <int Q, typename T, typename P>
__device__ __forceinline__ void load_class(P base, unsigned voff, unsigned moff, int N, int R,
                                           int b, int off, T sg, long long es, T (&x)[Q]) {
  const int rh = R >> 1;
#pragma unroll
  for (int a = 0; a < Q; ++a) {
    const bool direct = (Q & 1) ? a <= (Q - 1) / 2 : a < Q / 2;
    if (direct) {
      const P s = base + (long long)(a * R - off) * es;
      // j = 0 (b = 0) and, for odd Q, j = N (b = R/2) vanish for Dirichlet data
      const bool edge = (a == 0 && b == 0) || ((Q & 1) && a == (Q - 1) / 2 && 2 * b == R);
      const bool dead = ((a == 0) || ((Q & 1) && a == (Q - 1) / 2)) && edge && off;
      x[a] = dead ? T(0) : ld(s, voff);
    } else {
      // j = R a + b > N continues to 2N - j = (2N - R a - R/2) + (R/2 - b)
      const P s = base + (long long)(2 * N - a * R - rh - off) * es;
      const bool dead = 2 * a == Q && b == 0 && off;
      x[a] = dead ? T(0) : sg * ld(s, moff);
    }
  }
}

// Visits the modes of class k1 held as v[k2], k = k1 + Q k2, that are not
// duplicates: f(k2, u, mirrored), stored at position u + k1 or, mirrored
// (2N - k), u + (Q/2 - k1).
template <int R, typename F>
__device__ __forceinline__ void for_modes(int Q, int N, int k1, int off, F&& f) {
  const bool self = k1 == 0 || 2 * k1 == Q;  // k and 2N - k lie in the same class
#pragma unroll
  for (int k2 = 0; k2 < R; ++k2) {
    const bool direct = (R & 1) ? k2 <= (R - 1) / 2 : k2 < R / 2;
    if (direct) {
      bool live = true;
      if (k2 == 0) live = !(k1 == 0 && off);
      if ((R & 1) && k2 == (R - 1) / 2) live = !(2 * k1 == Q && off);
      if (live) f(k2, Q * k2 - off, false);
    } else {
      const bool live = !self || (2 * k2 == R && k1 == 0 && !off);
      if (live) f(k2, 2 * N - Q * k2 - (Q >> 1) - off, true);
    }
  }
}

// Stage 1 of class b: DFT over a and twiddle; emit(k, p, q) for k = 0 .. Q/2.
template <int Q, typename T, typename E>
__device__ __forceinline__ void stage1_emit(const T (&x)[Q], const Pair<T>* __restrict__ tw, int b,
                                            E&& emit) {
  rdft<Q, 1>(x, [&](int k, T C, T S) {
    const Pair<T> w = ld(tw, (unsigned)(b * k) * (unsigned)sizeof(Pair<T>));
    // w = scale (cos, sin)(2 pi b k / 2N), rotated for Neumann data
    emit(k, C * w.q + S * w.p, C * w.p - S * w.q);
  });
}

// Stage 2 of class k1: DFT over b of the pairs of b = 0 .. R/2.
template <int R, typename T, int M>
__device__ __forceinline__ void stage2(T (&p)[M], const T (&q)[M], T (&out)[R]) {
  p[0] *= T(0.5);
  if constexpr (R % 2 == 0) p[R / 2] *= T(0.5);
  irdft<R, 1>(p, q, out);
}

}  // namespace qn
