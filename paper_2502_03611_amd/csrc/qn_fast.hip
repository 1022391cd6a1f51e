// Factored mode products: the eigen-transform of an axis in two register
// stages instead of one dense product with S.
//
// With N = n + 1 (Dirichlet) or n - 1 (Neumann) intervals the 1D eigenvectors
// of the finite-difference stiffness matrix (Section 3.2 eq. Sy, Section 4.2)
// are sin(pi j k / N) or cos(pi j k / N): S x is the length-2N DFT of x
// continued oddly (evenly) about both ends.  For 2N = Q R the DFT splits
// (Cooley-Tukey): with j = R a + b, k = k1 + Q k2,
//   Y_b[k1] = sum_a x[R a + b] w_Q^{a k1},   T_b[k1] = w_2N^{b k1} Y_b[k1],
//   X[k1 + Q k2] = sum_b w_R^{b k2} T_b[k1].
// The continuation makes T_{R-b} = -+ conj(T_b) and X purely imaginary
// (real), so only b = 0 .. R/2 and k1 = 0 .. Q/2 are formed, every x is loaded
// once, and both stages are real: one thread owns a class j = +-b (mod R) of
// one line in stage 1 and a class k = +-k1 (mod Q) in stage 2, and the classes
// are exchanged once through LDS.  A transform of 512 intervals (32 x 32)
// takes about 20 multiply-adds per point where the reflection-folded dense
// product takes 256, so the kernels are bound by HBM: 16 bytes per point and
// pass.  Sums have at most 16 terms per stage, so rounding
// is below the dense product's.
//
// Along the axis a thread reads and writes in strides of R (Q) elements, so
// no staging is needed for coalescing: y and z passes put 16 neighbouring
// lines, 128 bytes, in consecutive lanes; x passes put
// the R/2 + 1 classes of one row in consecutive lanes, whose loads are
// consecutive elements.  The last forward axis keeps its modes in registers,
// divides them by the shifted eigenvalue sums (Section 4.1 eq. fin_inverse)
// and runs the inverse transform at once: one pass over HBM for the forward
// transform, the divide and the inverse one.  The transforms are their own
// inverses (scale sqrt(2/N) in the twiddles).
//
// Stage lengths are compile-time (qn_fast.h); a workgroup-uniform switch
// selects them, so one kernel serves every N whose 2N factors.

#include <algorithm>
#include <atomic>

#include "qn_fast.h"
#include "qn_internal.h"

namespace qn {
namespace {

// Kernel families: stage lengths all even and at most 32, any to 32, longer.
enum Family { EVEN = 0, ANY = 1, BIG = 2 };
#define QN_FAST_SWITCH(len)                                \
  if constexpr (FAM == BIG) {                              \
    switch (len) { QN_FAST_BIG(X) }                        \
  } else if constexpr (FAM == ANY) {                       \
    switch (len) { QN_FAST_EVEN(X) QN_FAST_ODD(X) }        \
  } else {                                                 \
    switch (len) { QN_FAST_EVEN(X) }                       \
  }

typedef double T;
constexpr int FAST_THREADS = 320;  // at most 17 (33) classes of 16 (8) lines


// x / d for d > 0: the hardware reciprocal (relative error e0), one Newton
// step (e0^2) and one residual correction of the quotient (e0^4 and an FP64
// rounding; e0 is about 2^-23).
__device__ __forceinline__ double quotient(double x, double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
  const double q = x * r;
  return __builtin_fma(__builtin_fma(-d, q, x), r, q);
}

// Stage 1 of class b into LDS, pair k at k * ks; stage 2 from LDS, pair b at b * bs.
template <int Q, typename T>
__device__ __forceinline__ void stage1_lds(const T (&x)[Q], const Pair<T>* __restrict__ tw, int b,
                                       Pair<T>* lds, int ks) {
  stage1_emit<Q, T>(x, tw, b, [&](int k, T p, T q) { lds[k * ks] = Pair<T>{p, q}; });
}
template <int R, typename T>
__device__ __forceinline__ void stage2_lds(const Pair<T>* lds, int bs, T (&out)[R]) {
  T p[R / 2 + 1], q[R / 2 + 1];
#pragma unroll
  for (int b = 0; b <= R / 2; ++b) {
    const Pair<T> v = lds[b * bs];
    p[b] = v.p;
    q[b] = v.q;
  }
  stage2<R, T>(p, q, out);
}

// ------------------------------------------------------------- y and z passes

// One transform (DIV = 0) or forward transform, divide and inverse transform
// (DIV = 1) of the lines of C consecutive x positions, in place.
template <int FAM, int DIV>
__global__ __launch_bounds__(FAST_THREADS, FAM == EVEN ? 4 : 2) void k_fast_lines(LineArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  Pair<T>* lds = reinterpret_cast<Pair<T>*>(smem);
  const int C = 1 << a.lc;
  const int xt = blockIdx.x % a.xtiles, o = blockIdx.x / a.xtiles;
  const int plane = o / a.oy;
  const int inst = plane % a.inst_mod;
  if (a.skip && a.skip[inst]) return;
  const int N = a.N, Q = a.Q, R = a.R, off = a.off;
  const T sg = off ? T(-1) : T(1);
  const int t = threadIdx.x, line = t & (C - 1), c = t >> a.lc;
  const bool lower = xt < a.xsplit;  // even and odd modes of a dense x axis, or all of a natural one
  const int x0 = lower ? xt * C : a.cbk + (xt - a.xsplit) * C, lim = lower ? a.ce : a.cbk + a.co;
  const int xl = x0 + line < lim ? line : lim - 1 - x0;  // lanes past the end repeat the last line
  const bool live_x = x0 + line < lim;
  const int oi = o % a.om, opos = oi < a.oe ? oi : a.obk + oi - a.oe;
  T* base = a.out + (long long)(o / a.om) * a.s1 + (long long)opos * a.s0 + x0;
  const unsigned eb = (unsigned)a.es * 8, lb = line * 8, xb = xl * 8;  // bytes: axis stride, line
  const Pair<T>* tw = (const Pair<T>*)a.tw;
  const int rh = R >> 1, qh = Q >> 1;
  const bool in1 = c <= rh, in2 = c <= qh;

#define X(L)                                                                                       \
  case L: {                                                                                        \
    if (in1) {                                                                                     \
      T x[L];                                                                                      \
      load_class<L, T>((const T*)base, xb + c * eb, xb + (rh - c) * eb, N, R, c, off, sg, a.es, x); \
      stage1_lds<L, T>(x, tw, c, lds + (c << a.lc) + line, (rh + 1) << a.lc);                          \
    }                                                                                              \
    break;                                                                                         \
  }
  QN_FAST_SWITCH(Q)
#undef X
  __syncthreads();
  if constexpr (DIV == 0) {
#define X(L)                                                                                       \
  case L: {                                                                                        \
    if (in2) {                                                                                     \
      T v[L];                                                                                      \
      stage2_lds<L, T>(lds + (((rh + 1) * c) << a.lc) + line, C, v);                                   \
      if (live_x)                                                                                  \
        for_modes<L>(Q, N, c, off, [&](int k2, int u, bool mir) {                                  \
          st(base + (long long)u * a.es, lb + (mir ? qh - c : c) * eb, mir ? sg * v[k2] : v[k2]);  \
        });                                                                                        \
    }                                                                                              \
    break;                                                                                         \
  }
    QN_FAST_SWITCH(R)
#undef X
  } else {
    double scale, beta;
    a.coef.get((long long)inst * a.coef_stride, scale, beta);
    if (a.cscale) scale *= a.cscale[plane / a.comp_div];
    const double den0 = scale * (a.lamX[x0 + xl] + (a.lamY ? a.lamY[opos] : 0.0)) + beta;
#define X(L)                                                                                       \
  case L: {                                                                                        \
    T v[L];                                                                                        \
    if (in2) {                                                                                     \
      stage2_lds<L, T>(lds + (((rh + 1) * c) << a.lc) + line, C, v);                                   \
      const unsigned cb = c * 8; /* lam[k], k = 0 .. 2N - 1: continued evenly */                   \
      _Pragma("unroll") for (int k2 = 0; k2 < L; ++k2) {                                           \
        v[k2] = quotient(v[k2], __builtin_fma(scale, ld(a.lam + Q * k2, cb), den0));            \
      }                                                                                            \
      if (off) { /* the modes k = 0 and k = N do not exist */                                      \
        if (c == 0) {                                                                              \
          v[0] = T(0);                                                                             \
          if (L % 2 == 0) v[L / 2] = T(0);                                                         \
        }                                                                                          \
        if (L % 2 == 1 && 2 * c == Q) v[(L - 1) / 2] = T(0);                                       \
      }                                                                                            \
    }                                                                                              \
    __syncthreads(); /* stage 2 reads done; the same LDS takes the inverse's pairs */              \
    if (in2) stage1_lds<L, T>(v, tw, c, lds + (c << a.lc) + line, (qh + 1) << a.lc);                   \
    break;                                                                                         \
  }
    QN_FAST_SWITCH(R)
#undef X
    __syncthreads();
#define X(L)                                                                                       \
  case L: {                                                                                        \
    if (in1) {                                                                                     \
      T v[L];                                                                                      \
      stage2_lds<L, T>(lds + (((qh + 1) * c) << a.lc) + line, C, v);                                   \
      if (live_x)                                                                                  \
        for_modes<L>(R, N, c, off, [&](int k2, int u, bool mir) {                                  \
          st(base + (long long)u * a.es, lb + (mir ? rh - c : c) * eb, mir ? sg * v[k2] : v[k2]);  \
        });                                                                                        \
    }                                                                                              \
    break;                                                                                         \
  }
    QN_FAST_SWITCH(Q)
#undef X
  }
}

// ------------------------------------------------------------------- x passes

// Transform of rows (the contiguous axis): a.rows rows of the tensor, a.lines
// per workgroup.  EPI 0: into a.out (padded layout); EPI 1: into the caller's
// array a.dense (interior layout), stored or subtracted.
template <int FAM, int EPI>
__global__ __launch_bounds__(FAST_THREADS, FAM == EVEN && EPI == 0 ? 4 : 2) void k_fast_rows(RowArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  Pair<T>* lds = reinterpret_cast<Pair<T>*>(smem);
  const int N = a.N, Q = a.Q, R = a.R, off = a.off;
  const T sg = off ? T(-1) : T(1);
  const int rh = R >> 1, qh = Q >> 1;
  const int t = threadIdx.x;
  const int r0 = blockIdx.x * a.lines;
  const int rlast = min(r0 + a.lines, a.rows) - 1;
  const int pl0 = r0 / a.oy, pl1 = rlast / a.oy;
  if (a.skip) {  // every instance of the workgroup's rows has stopped
    bool any = false;
    for (int pl = pl0; pl <= pl1; ++pl) any = any || !a.skip[pl % a.inst_mod];
    if (!any) return;
  }
  const Pair<T>* tw = (const Pair<T>*)a.tw;
  // offset of row r from the array's start
  auto row_off = [&](int r, long long s1, long long s0, long long ys) {
    const int pl = r / a.oy;
    return (long long)(pl / a.om) * s1 + (long long)(pl % a.om) * s0 + (long long)(r - pl * a.oy) * ys;
  };
  const int line1 = t / (rh + 1), c1 = t - line1 * (rh + 1);
  const int line2 = t / (qh + 1), c2 = t - line2 * (qh + 1);
  const bool in1 = line1 < a.lines;
  const int row2 = r0 + line2;
  const bool in2 = line2 < a.lines && row2 <= rlast;
  const int rp = (rh + 1) | 1;  // odd class stride: stage 2 reads hit distinct banks

  const long long b0 = row_off(r0, a.is1, a.is0, a.iys);
  const T* base = a.in + b0;
  const unsigned lo = 8 * (unsigned)(row_off(min(r0 + line1, rlast), a.is1, a.is0, a.iys) - b0);
#define X(L)                                                                                       \
  case L: {                                                                                        \
    if (in1) {                                                                                     \
      T x[L];                                                                                      \
      load_class<L, T>(base, lo + 8 * c1, lo + 8 * (rh - c1), N, R, c1, off, sg, 1, x);            \
      stage1_lds<L, T>(x, tw, c1, lds + line1 * (qh + 1) * rp + c1, rp);                               \
    }                                                                                              \
    break;                                                                                         \
  }
  QN_FAST_SWITCH(Q)
#undef X
  __syncthreads();
  if (!in2) return;
  if (a.skip && a.skip[(row2 / a.oy) % a.inst_mod]) return;
  const long long o0 = row_off(r0, a.s1, a.s0, a.ys);
  T* o = a.out + o0;
  const unsigned ro = 8 * (unsigned)(row_off(row2, a.s1, a.s0, a.ys) - o0);
  const unsigned vo = ro + 8 * c2, mo = ro + 8 * (qh - c2);
  const bool sub = EPI == 1 && a.sub != 0;  // a stored solve reads no old values
  const double us = sub && a.uscale ? *a.uscale : 1.0, sp = a.step;
#define X(L)                                                                                       \
  case L: {                                                                                        \
    T v[L], old[L];                                                                                \
    /* old values in flight during stage 2, for lengths whose registers allow it */                \
    if (L <= 32 && sub)                                                                            \
      for_modes<L>(Q, N, c2, off,                                                                  \
                   [&](int k2, int u, bool mir) { old[k2] = ld(o + u, mir ? mo : vo); });          \
    stage2_lds<L, T>(lds + (line2 * (qh + 1) + c2) * rp, 1, v);                                        \
    if (sub)                                                                                       \
      for_modes<L>(Q, N, c2, off, [&](int k2, int u, bool mir) {                                   \
        const double prev = L <= 32 ? old[k2] : ld(o + u, mir ? mo : vo);                          \
        st(o + u, mir ? mo : vo, us * prev - sp * (mir ? sg * v[k2] : v[k2]));                     \
      });                                                                                          \
    else                                                                                           \
      for_modes<L>(Q, N, c2, off, [&](int k2, int u, bool mir) {                                   \
        st(o + u, mir ? mo : vo, mir ? sg * v[k2] : v[k2]);                                        \
      });                                                                                          \
    break;                                                                                         \
  }
  QN_FAST_SWITCH(R)
#undef X
}

// A kernel's limit of 64 KB of LDS is raised the first time it needs more, once
// per kernel and device (the kernels share one type, so Kern is a value).
template <auto Kern>
hipError_t allow_lds(size_t bytes) {
  static std::atomic<unsigned long long> done{0};  // one bit per device
  if (bytes <= 64 * 1024) return hipSuccess;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const unsigned long long bit = 1ull << (dev & 63);
  if (done.load(std::memory_order_relaxed) & bit) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(Kern),
                          hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_relaxed);
  return e;
}

constexpr size_t kLdsTarget = 80 * 1024;  // two workgroups per CU

int round64(int v) { return (v + 63) & ~63; }

template <int FAM, int DIV>
hipError_t lines_launch(const FastArgs& f, int nouter, hipStream_t st) {
  constexpr auto kern = k_fast_lines<FAM, DIV>;
  LineArgs a{};
  a.tw = f.ax.tw;
  a.lam = f.ax.lam;
  a.out = f.out;
  a.s1 = f.s1;
  a.s0 = f.s0;
  a.es = f.es;
  a.lamX = f.lamX;
  a.lamY = f.lamY;
  a.coef = f.coef;
  a.cscale = f.cscale;
  a.skip = f.skip;
  a.ce = f.ce;
  a.cbk = f.cbk;
  a.co = f.co;
  a.oy = f.oy;
  a.om = f.om;
  a.oe = f.oe;
  a.obk = f.obk;
  a.inst_mod = f.inst_mod;
  a.comp_div = f.comp_div;
  a.coef_stride = f.coef_stride;
  a.N = (short)f.ax.N;
  a.Q = (short)f.ax.Q;
  a.R = (short)f.ax.R;
  a.off = (short)f.ax.off;
  int lc = FAM == BIG ? 3 : 4;
  const int qh = a.Q / 2 + 1, rh = a.R / 2 + 1;
  auto bytes = [&](int l) { return (size_t)qh * rh * sizeof(Pair<T>) << l; };
  while (lc > 2 && bytes(lc) > kLdsTarget) --lc;
  // small grids: fewer lines per workgroup (shorter runs of a cache line) until
  // half the CUs have one; per iteration, to 512 workgroups and to 128: 63^3 53
  // and 48 us, 127 x 127 x 31 73 and 60, 1023^2 82 and 77
  auto tiles = [&](int cols, int l) { return (cols + (1 << l) - 1) >> l; };
  while (lc > 2 && (long long)(tiles(a.ce, lc) + tiles(a.co, lc)) * nouter < 128) --lc;
  a.lc = (short)lc;
  a.xsplit = tiles(a.ce, lc);
  a.xtiles = a.xsplit + tiles(a.co, lc);
  const int nt = round64(std::max(qh, rh) << lc);
  hipError_t e = allow_lds<kern>(bytes(lc));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)a.xtiles * nouter), dim3(nt), bytes(lc), st, a);
  return hipGetLastError();
}

template <int FAM, int EPI>
hipError_t rows_launch(const FastArgs& f, hipStream_t st) {
  RowArgs a{};
  a.tw = f.ax.tw;
  a.in = f.in;
  a.out = EPI ? f.dense : f.out;
  a.is1 = f.is1;
  a.is0 = f.is0;
  a.s1 = EPI ? f.om * f.ds0 : f.s1;
  a.s0 = EPI ? f.ds0 : f.s0;
  a.uscale = f.uscale;
  a.step = f.step;
  a.skip = f.skip;
  a.iys = f.iys;
  a.ys = EPI ? f.dys : f.ys;
  a.rows = f.rows;
  a.oy = f.oy;
  a.om = f.om;
  a.inst_mod = f.inst_mod;
  a.N = (short)f.ax.N;
  a.Q = (short)f.ax.Q;
  a.R = (short)f.ax.R;
  a.off = (short)f.ax.off;
  a.sub = f.sub != 0;
  const int qh = a.Q / 2 + 1, rh = a.R / 2 + 1, nb = std::max(qh, rh);
  const size_t per = (size_t)qh * (rh | 1) * sizeof(Pair<T>);
  int lines = 256 / nb;
  lines = std::min<int>(lines, std::max<size_t>(1, kLdsTarget / per));
  // small grids: fewer rows per workgroup (but a whole wave) until every CU has one
  lines = std::min(lines, std::max(std::max(1, 64 / nb), a.rows / 256));
  a.lines = (short)lines;
  constexpr auto kern = k_fast_rows<FAM, EPI>;
  hipError_t e = allow_lds<kern>(per * lines);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((a.rows + lines - 1) / lines), dim3(round64(lines * nb)),
                     per * lines, st, a);
  return hipGetLastError();
}

}  // namespace

namespace {
int family(const FastAxis& ax) {
  return std::max(ax.Q, ax.R) > 32 ? BIG : ((ax.Q | ax.R) & 1) ? ANY : EVEN;
}
}  // namespace

hipError_t launch_fast_lines(const FastArgs& a, int nouter, bool divide, hipStream_t st) {
  switch (family(a.ax)) {
    case EVEN: return divide ? lines_launch<EVEN, 1>(a, nouter, st) : lines_launch<EVEN, 0>(a, nouter, st);
    case ANY: return divide ? lines_launch<ANY, 1>(a, nouter, st) : lines_launch<ANY, 0>(a, nouter, st);
    default: return divide ? lines_launch<BIG, 1>(a, nouter, st) : lines_launch<BIG, 0>(a, nouter, st);
  }
}

hipError_t launch_fast_rows(const FastArgs& a, bool dense, hipStream_t st) {
  switch (family(a.ax)) {
    case EVEN: return dense ? rows_launch<EVEN, 1>(a, st) : rows_launch<EVEN, 0>(a, st);
    case ANY: return dense ? rows_launch<ANY, 1>(a, st) : rows_launch<ANY, 0>(a, st);
    default: return dense ? rows_launch<BIG, 1>(a, st) : rows_launch<BIG, 0>(a, st);
  }
}

}  // namespace qn
