// Strip form of the reflection-folded mode products (see qn_gemm_fold.hip for
// the fold): the same products with the work laid out over 16-column (row)
// strips of interior data, whatever the extents.
//
// The tile form works on extents padded to multiples of 64: at 200 points per
// axis (bk = 128 for 100 modes of each parity) a product does 1.9 times the
// arithmetic of the strips.  Here a wave owns one strip (16 or 32 columns of
// the slab, or 16 rows) and MB 16-row blocks of both mode parities, so only
// the last block, the last contraction step and the last strip carry padding.
// The data go from HBM straight into the registers of the MFMA operand (each
// load is four 128-byte runs, one chunk of 16 contraction rows ahead); the
// eigenvector blocks, shared by the four waves of a workgroup, are staged in
// LDS, double-buffered, 2 MB matrix-core instructions per fragment pair.
// Bound by the matrix cores and, at short contractions, by the loads and stores
// around them; per instruction the tiles are the faster form (511^3, no
// padding: 1.39 against 1.24 ms a product), so the strips are taken where the
// padding outweighs that (use_strips in qn_host.h).  200^3 FP64 solve 0.57 ->
// 0.40 ms, 400^3 6.9 -> 3.9 ms, 150 x 203 x 176 FP32 0.23 -> 0.17 ms.  (With
// vector address arithmetic and tail selects in every chunk, nine other vector
// instructions per matrix one, 0.41 and 4.1 ms.)  The
// contraction runs in the same order as in the tile form (steps of four rows
// from row 0), so the results are the same bits.
//
// Instantiated per element type by qn_gemm_strip64.hip and qn_gemm_strip32.hip.
#pragma once

#include <algorithm>

#include "qn_internal.h"
#include "qn_mfma.h"

namespace qn {
namespace strip {

constexpr int KC = 16;  // contraction rows per LDS stage

template <typename T>
__device__ __forceinline__ T divide_by(T x, double scale, double lam, double beta) {
  if constexpr (sizeof(T) == 4)
    return quotf(x, __builtin_fmaf((float)scale, (float)lam, (float)beta));
  else
    return quot(x, scale * lam + beta);
}

// LDS stage of the eigenvector blocks: KC rows of 16 MB entries of each parity
// (FP32: rows an odd number of 64-byte groups apart, so that the two rows one
// read touches in a cycle fall on distinct banks).
template <typename T, int MB>
struct Stage {
  static constexpr int LD = 16 * MB + ((sizeof(T) == 4 && MB % 2 == 0) ? 16 : 0);
  static constexpr int VE = 16 / sizeof(T);
  static constexpr int NV = 2 * KC * 16 * MB / VE;   // 16-byte vectors
  static constexpr int NA = (NV + 255) / 256;
  typedef T V __attribute__((ext_vector_type(VE)));
  T s[2][2][KC][LD];
  V r[NA];
};

// The stage's global loads, advanced by `step` elements per chunk.  Rows past bk
// repeat others: they feed accumulators that are not stored.  With whole rows
// per 256 vectors of one parity the addresses are scalar but for one offset.
template <typename T, int MB>
struct Loader {
  using S = Stage<T, MB>;
  typedef typename S::V V;
  static constexpr int ROW = 16 * MB / S::VE;  // vectors of a row
  static constexpr bool SCALAR = MB == 4;
  static constexpr int NP = SCALAR ? 2 : S::NA;
  const T* p[NP];
  int off = 0, bk;
  __device__ __forceinline__ Loader(const StripArgs& a, int tid, int m0) : bk(a.bk) {
    if constexpr (SCALAR) {
      p[0] = (const T*)a.Fe;
      p[1] = (const T*)a.Fo;
      off = (tid / ROW) * bk + min(m0 + (tid % ROW) * S::VE, bk - S::VE);
    } else {
#pragma unroll
      for (int q = 0; q < S::NA; ++q) {
        const int v = min(tid + 256 * q, S::NV - 1);
        p[q] = (const T*)(v / ROW / KC ? a.Fo : a.Fe) + (v / ROW % KC) * bk +
               min(m0 + (v % ROW) * S::VE, bk - S::VE);
      }
    }
  }
  __device__ __forceinline__ void next(V (&r)[S::NA], int step) {
    if constexpr (SCALAR) {
#pragma unroll
      for (int q = 0; q < S::NA; ++q)
        r[q] = *reinterpret_cast<const V*>(p[q / (S::NA / 2)] + q % (S::NA / 2) * (256 / ROW) * bk + off);
      p[0] += step;
      p[1] += step;
    } else {
#pragma unroll
      for (int q = 0; q < S::NA; ++q) {
        r[q] = *reinterpret_cast<const V*>(p[q]);
        p[q] += step;
      }
    }
  }
};

// Column group g of a split or natural axis: first position and valid width.
__device__ __forceinline__ void group_of(const StripArgs& a, int g, int width, int& pos, int& lim) {
  if (g < a.ge) {
    pos = g * width;
    lim = a.ce;
  } else {
    pos = a.cbk + (g - a.ge) * width;
    lim = a.cbk + a.co;
  }
}

// Form L (y and z axes).  INV = 0: forward (spatial rows k and n-1-k folded),
// INV = 1: inverse.  NCB: 16-column blocks per wave.
template <typename T, int MB, int NCB, int INV, int DIV>
__global__ __launch_bounds__(256, MB * NCB <= 6 && MB <= 4 ? 3 : 2) void k_strip_left(StripArgs a) {
  using MF = Mfma<T>;
  using S = Stage<T, MB>;
  typedef typename S::V V;
  __shared__ __attribute__((aligned(16))) T As[2][2][KC][S::LD];
  const int mtiles = a.mtiles;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int mt = t % mtiles, wg = t / mtiles;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int n = a.n, h = a.h, odd = a.odd, bk = a.bk, ne = h + odd;
  const int m0 = mt * 16 * MB;
  const int live_blocks = (ne - m0 + 15) / 16;  // the last block tile may have fewer than MB
  const int strip = min(wg * 4 + wave, a.strips - 1);  // spare waves repeat the last strip
  const int o = strip / a.groups, g = strip - o * a.groups;
  const int plane = o / a.oy;
  const int inst = plane % a.inst_mod;
  bool live = wg * 4 + wave < a.strips;
  if (a.skip) {
    const int s0 = wg * 4, s1 = min(wg * 4 + 3, a.strips - 1);
    bool any = false;
    for (int p = s0 / a.groups / a.oy; p <= s1 / a.groups / a.oy; ++p) any = any || !a.skip[p % a.inst_mod];
    if (!any) return;
    live = live && !a.skip[inst];
  }
  int oi = o % a.om;
  const int opos = oi < a.oe ? oi : a.obk + oi - a.oe;  // y position of a z product
  int pos, lim;
  group_of(a, g, 16 * NCB, pos, lim);
  const long long base = (long long)(o / a.om) * a.s1 + (long long)opos * a.s0;
  const T* in = (const T*)a.in + base;
  T* out = (T*)a.out + base;
  int col[NCB];
  bool ok[NCB];
#pragma unroll
  for (int j = 0; j < NCB; ++j) {
    const int c = pos + 16 * j + lr;
    ok[j] = live && c < lim;
    col[j] = min(c, lim - 1);
  }

  typename MF::v4 acce[MB][NCB], acco[MB][NCB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NCB; ++j) acce[i][j] = acco[i][j] = typename MF::v4{0, 0, 0, 0};

  V ra[S::NA];
  Loader<T, MB> ld(a, tid, m0);
  auto aload = [&]() { ld.next(ra, KC * bk); };
  auto astore = [&](int buf) {
#pragma unroll
    for (int q = 0; q < S::NA; ++q) {
      const int v = tid + 256 * q;
      const int mm = (v % (16 * MB / S::VE)) * S::VE, kk = (v / (16 * MB / S::VE)) % KC,
                par = v / (16 * MB / S::VE) / KC;
      if (v < S::NV) *reinterpret_cast<V*>(&As[buf][par][kk][mm]) = ra[q];
    }
  };
  T lo[2][KC / 4][NCB], hi[2][KC / 4][NCB];
  // Chunks inside the folded rows: scalar row addresses, one offset per lane
  // (the upper rows of a forward product run backwards).
  const unsigned off0 = (unsigned)(lk * a.es) * (unsigned)sizeof(T);
  const unsigned off1 = INV ? off0 : (unsigned)((3 - lk) * a.es) * (unsigned)sizeof(T);
  auto at = [&](long long row, unsigned off, int j) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(in + row * a.es) +
                                       (off + (unsigned)col[j] * (unsigned)sizeof(T)));
  };
  auto bload = [&](int k0, T (&l)[KC / 4][NCB], T (&u)[KC / 4][NCB]) {
    if (k0 + KC <= h) {
#pragma unroll
      for (int s = 0; s < KC / 4; ++s)
#pragma unroll
        for (int j = 0; j < NCB; ++j) {
          l[s][j] = at(k0 + 4 * s, off0, j);
          u[s][j] = at(INV ? bk + k0 + 4 * s : n - 4 - k0 - 4 * s, off1, j);
        }
      return;
    }
#pragma unroll
    for (int s = 0; s < KC / 4; ++s) {
      const int k = k0 + 4 * s + lk;
      const int r0 = INV ? min(k, ne - 1) : min(k, h);
      const int r1 = INV ? (h > 0 ? bk + min(k, h - 1) : 0) : (k < h ? n - 1 - k : min(h, n - 1));
      const T* p0 = in + (long long)min(r0, n - 1) * a.es;
      const T* p1 = in + (long long)r1 * a.es;
#pragma unroll
      for (int j = 0; j < NCB; ++j) {
        l[s][j] = p0[col[j]];
        u[s][j] = p1[col[j]];
      }
    }
  };
  const int nk = (ne + KC - 1) / KC;
  auto compute = [&](int kc, const T (&l)[KC / 4][NCB], const T (&u)[KC / 4][NCB]) {
    const int buf = kc & 1;
    T e[KC / 4][NCB], d[KC / 4][NCB];
    const bool full = kc * KC + KC <= h;
#pragma unroll
    for (int s = 0; s < KC / 4; ++s)
#pragma unroll
      for (int j = 0; j < NCB; ++j) {
        e[s][j] = INV ? l[s][j] : l[s][j] + u[s][j];
        d[s][j] = INV ? u[s][j] : l[s][j] - u[s][j];
      }
    if (!full) {
#pragma unroll
      for (int s = 0; s < KC / 4; ++s) {
        const int k = kc * KC + 4 * s + lk;
#pragma unroll
        for (int j = 0; j < NCB; ++j) {
          if (INV)
            e[s][j] = k < ne ? e[s][j] : T(0);
          else
            e[s][j] = k < h ? e[s][j] : (k == h && odd) ? l[s][j] : T(0);
          d[s][j] = k < h ? d[s][j] : T(0);
        }
      }
    }
#pragma unroll
    for (int s = 0; s < KC / 4; ++s) {
      if (kc * KC + 4 * s >= ne) break;
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        if (i >= live_blocks) break;
        const T fe = As[buf][0][4 * s + lk][16 * i + lr], fo = As[buf][1][4 * s + lk][16 * i + lr];
#pragma unroll
        for (int j = 0; j < NCB; ++j) {
          acce[i][j] = MF::op(fe, e[s][j], acce[i][j]);
          acco[i][j] = MF::op(fo, d[s][j], acco[i][j]);
        }
      }
    }
  };
  aload();
  bload(0, lo[0], hi[0]);
  astore(0);
  __syncthreads();
  for (int kc = 0; kc < nk; kc += 2) {
    // two chunks per trip, so that the register buffers keep static names
    if (kc + 1 < nk) {
      aload();
      bload((kc + 1) * KC, lo[1], hi[1]);
    }
    compute(kc, lo[0], hi[0]);
    if (kc + 1 >= nk) break;
    astore(1);
    __syncthreads();
    if (kc + 2 < nk) {
      aload();
      bload((kc + 2) * KC, lo[0], hi[0]);
    }
    compute(kc + 1, lo[1], hi[1]);
    if (kc + 2 < nk) {
      astore(0);
      __syncthreads();
    }
  }

  double scale = 1.0, beta = 0.0, cn[NCB];
  if constexpr (DIV) {
    a.coef.get((long long)inst * a.coef_stride, scale, beta);
    if (a.cscale) scale *= a.cscale[plane / a.comp_div];
#pragma unroll
    for (int j = 0; j < NCB; ++j) cn[j] = a.lamX[col[j]] + (a.lamY ? a.lamY[opos] : 0.0);
  }
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int m = m0 + 16 * i + MF::row(lane, q);
#pragma unroll
      for (int j = 0; j < NCB; ++j) {
        if (!ok[j]) continue;
        const T p = acce[i][j][q], d = acco[i][j][q];
        if constexpr (INV) {
          if (m < h) {
            out[(long long)m * a.es + col[j]] = p + d;
            out[(long long)(n - 1 - m) * a.es + col[j]] = p - d;
          } else if (m == h && odd) {
            out[(long long)m * a.es + col[j]] = p;
          }
        } else if constexpr (DIV) {
          if (m < ne)
            out[(long long)m * a.es + col[j]] = divide_by<T>(p, scale, a.lamM[m] + cn[j], beta);
          if (m < h)
            out[(long long)(bk + m) * a.es + col[j]] = divide_by<T>(d, scale, a.lamM[bk + m] + cn[j], beta);
        } else {
          if (m < ne) out[(long long)m * a.es + col[j]] = p;
          if (m < h) out[(long long)(bk + m) * a.es + col[j]] = d;
        }
      }
    }
}

// Form R (x axis): a wave owns 16 rows.  The rows are loaded in 128-byte runs
// and folded into a wave's own LDS tile (row stride 17: conflict-free column
// reads).  INV = 0: forward, from TIN rows (the transform tensor or a caller's
// FP64 right-hand side) into the tensor; INV = 1: inverse into the caller's
// FP64 array, stored or subtracted.
template <typename T, typename TIN, int MB, int INV>
__global__ __launch_bounds__(256, MB <= 4 ? 3 : 2) void k_strip_right(StripArgs a) {
  using MF = Mfma<T>;
  using S = Stage<T, MB>;
  typedef typename S::V V;
  __shared__ __attribute__((aligned(16))) T Bs[2][2][KC][S::LD];
  __shared__ T Ds[4][2][16][17];
  const int mtiles = a.mtiles;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int mt = t % mtiles, wg = t / mtiles;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int n = a.n, h = a.h, odd = a.odd, bk = a.bk, ne = h + odd;
  const int m0 = mt * 16 * MB;
  const int live_blocks = (ne - m0 + 15) / 16;  // the last block tile may have fewer than MB
  const int r0 = wg * 64 + 16 * wave;
  if (a.skip) {
    const int p0 = wg * 64 / a.oy, p1 = min(wg * 64 + 63, a.rows - 1) / a.oy;
    bool any = false;
    for (int p = p0; p <= p1; ++p) any = any || !a.skip[p % a.inst_mod];
    if (!any) return;
  }
  auto row_off = [&](int r, long long s1, long long s0, long long ys) {
    const int p = r / a.oy;
    return (long long)(p / a.om) * s1 + (long long)(p % a.om) * s0 + (long long)(r - p * a.oy) * ys;
  };
  const TIN* src[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    src[i] = (const TIN*)a.in + row_off(min(r0 + 4 * i + lk, a.rows - 1), a.is1, a.is0, a.iys);

  typename MF::v4 acce[MB], acco[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) acce[i] = acco[i] = typename MF::v4{0, 0, 0, 0};

  V ra[S::NA];
  Loader<T, MB> ld(a, tid, m0);
  auto aload = [&]() { ld.next(ra, KC * bk); };
  auto astore = [&](int buf) {
#pragma unroll
    for (int q = 0; q < S::NA; ++q) {
      const int v = tid + 256 * q;
      const int mm = (v % (16 * MB / S::VE)) * S::VE, kk = (v / (16 * MB / S::VE)) % KC,
                par = v / (16 * MB / S::VE) / KC;
      if (v < S::NV) *reinterpret_cast<V*>(&Bs[buf][par][kk][mm]) = ra[q];
    }
  };
  T lo[4], hi[4];
  auto dload = [&](int k0) {
    const int k = k0 + lr;
    if (k0 + KC <= h) {
      const int c1 = INV ? bk + k : n - 1 - k;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        lo[i] = (T)src[i][k];
        hi[i] = (T)src[i][c1];
      }
      return;
    }
    const int c0 = INV ? min(k, ne - 1) : min(k, h);
    const int c1 = INV ? (h > 0 ? bk + min(k, h - 1) : 0) : (k < h ? n - 1 - k : 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lo[i] = (T)src[i][min(c0, n - 1)];
      hi[i] = (T)src[i][c1];
    }
  };
  auto dstore = [&](int k0) {
    const int k = k0 + lr;
    const bool full = k0 + KC <= h;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      T e, d;
      if (full) {
        e = INV ? lo[i] : lo[i] + hi[i];
        d = INV ? hi[i] : lo[i] - hi[i];
      } else if (INV) {
        e = k < ne ? lo[i] : T(0);
        d = k < h ? hi[i] : T(0);
      } else {
        e = k < h ? lo[i] + hi[i] : (k == h && odd) ? lo[i] : T(0);
        d = k < h ? lo[i] - hi[i] : T(0);
      }
      Ds[wave][0][4 * i + lk][lr] = e;
      Ds[wave][1][4 * i + lk][lr] = d;
    }
  };
  const int nk = (ne + KC - 1) / KC;
  aload();
  dload(0);
  astore(0);
  dstore(0);
  __syncthreads();
  for (int kc = 0; kc < nk; ++kc) {
    const int buf = kc & 1;
    if (kc + 1 < nk) {
      aload();
      dload((kc + 1) * KC);
    }
    T e[KC / 4], d[KC / 4];
#pragma unroll
    for (int s = 0; s < KC / 4; ++s) {
      e[s] = Ds[wave][0][lr][4 * s + lk];
      d[s] = Ds[wave][1][lr][4 * s + lk];
    }
#pragma unroll
    for (int s = 0; s < KC / 4; ++s) {
      if (kc * KC + 4 * s >= ne) break;
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        if (i >= live_blocks) break;
        acce[i] = MF::op(e[s], Bs[buf][0][4 * s + lk][16 * i + lr], acce[i]);
        acco[i] = MF::op(d[s], Bs[buf][1][4 * s + lk][16 * i + lr], acco[i]);
      }
    }
    if (kc + 1 < nk) {
      astore(buf ^ 1);
      dstore((kc + 1) * KC);  // the wave's own reads of this tile are done
      __syncthreads();
    }
  }

  const double us = INV && a.sub && a.uscale ? *a.uscale : 1.0, st = a.step;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = r0 + MF::row(lane, q);
    if (r >= a.rows) continue;
    if (a.skip && a.skip[(r / a.oy) % a.inst_mod]) continue;
    if constexpr (INV == 0) {
      T* out = (T*)a.out + row_off(r, a.s1, a.s0, a.ys);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        const int m = m0 + 16 * i + lr;
        if (m < ne) out[m] = acce[i][q];
        if (m < h) out[bk + m] = acco[i][q];
      }
    } else {
      double* out = a.dense + row_off(r, a.om * a.ds0, a.ds0, a.dys);
      double old1[MB], old2[MB];
      if (a.sub) {
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          const int m = m0 + 16 * i + lr;
          old1[i] = m < ne ? out[m] : 0.0;
          old2[i] = m < h ? out[n - 1 - m] : 0.0;
        }
      }
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        const int m = m0 + 16 * i + lr;
        const T p = acce[i][q], d = acco[i][q];
        const T v1 = m < h ? p + d : p, v2 = p - d;
        if (m < ne) out[m] = a.sub ? us * old1[i] - st * (double)v1 : (double)v1;
        if (m < h) out[n - 1 - m] = a.sub ? us * old2[i] - st * (double)v2 : (double)v2;
      }
    }
  }
}

constexpr int CAP = 7;  // (8 blocks spill)

// 16-row blocks per wave: the count whose rounds of workgroups (three per CU up
// to `three` blocks, else two) take the least time, a block counting
// as its matrix instructions and the wave's own loads, folds and stores as half
// a block (FP64 at 200^3: 7 blocks 0.425 ms a solve, 4 0.411, 2 0.449, 1 0.47; at
// 400^3: 7 4.06 ms, 5 4.46, 4 4.40).
inline int blocks_per_wave(int ne, int three, long long workgroups, int* mtiles) {
  const int nb = (ne + 15) / 16;
  int best = 1;
  long long best_cost = -1;
  for (int mb = std::min(CAP, nb); mb >= 1; --mb) {
    const long long wgs = workgroups * ((nb + mb - 1) / mb);
    const int occ = mb <= three ? 3 : 2;
    const long long cost = (wgs + 256 * occ - 1) / (256 * occ) * occ * (2 * mb + 1);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = mb;
    }
  }
  *mtiles = (nb + best - 1) / best;
  return best;
}

template <typename T>
hipError_t left(StripArgs a, int kind, hipStream_t st) {
  constexpr int NCB = sizeof(T) == 8 ? 1 : 2;
  a.ge = (a.ce + 16 * NCB - 1) / (16 * NCB);
  a.groups = a.ge + (a.co + 16 * NCB - 1) / (16 * NCB);
  a.strips = a.groups * a.nouter;
  const long long wgs = (a.strips + 3) / 4;
  const int mb = blocks_per_wave(a.h + a.odd, NCB == 1 ? 4 : 3, wgs, &a.mtiles);
  const dim3 grid((unsigned)(wgs * a.mtiles)), block(256);
#define QN_STRIP(M)                                                                      \
  case M:                                                                                \
    if (kind == STRIP_INV) hipLaunchKernelGGL((k_strip_left<T, M, NCB, 1, 0>), grid, block, 0, st, a);        \
    else if (kind == STRIP_DIV) hipLaunchKernelGGL((k_strip_left<T, M, NCB, 0, 1>), grid, block, 0, st, a);   \
    else hipLaunchKernelGGL((k_strip_left<T, M, NCB, 0, 0>), grid, block, 0, st, a);                          \
    break;
  switch (mb) {
    QN_STRIP(1) QN_STRIP(2) QN_STRIP(3) QN_STRIP(4) QN_STRIP(5) QN_STRIP(6) QN_STRIP(7)
    default: return hipErrorInvalidValue;
  }
#undef QN_STRIP
  return hipGetLastError();
}

template <typename T>
hipError_t right(StripArgs a, int kind, bool in64, hipStream_t st) {
  const long long wgs = (a.rows + 63) / 64;
  const int mb = blocks_per_wave(a.h + a.odd, 4, wgs, &a.mtiles);
  const dim3 grid((unsigned)(wgs * a.mtiles)), block(256);
#define QN_STRIP(M)                                                                      \
  case M:                                                                                \
    if (kind == STRIP_INV) hipLaunchKernelGGL((k_strip_right<T, T, M, 1>), grid, block, 0, st, a);            \
    else if (in64) hipLaunchKernelGGL((k_strip_right<T, double, M, 0>), grid, block, 0, st, a);               \
    else hipLaunchKernelGGL((k_strip_right<T, T, M, 0>), grid, block, 0, st, a);                              \
    break;
  switch (mb) {
    QN_STRIP(1) QN_STRIP(2) QN_STRIP(3) QN_STRIP(4) QN_STRIP(5) QN_STRIP(6) QN_STRIP(7)
    default: return hipErrorInvalidValue;
  }
#undef QN_STRIP
  return hipGetLastError();
}

}  // namespace strip
}  // namespace qn
