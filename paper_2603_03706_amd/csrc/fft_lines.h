// Line transforms in registers and LDS shared by the y-z kernels: DFTs of a
// lane's own points, the two-pass rows and columns whose lanes exchange
// through LDS inside one wavefront, and the row and column layouts.
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>
#include "kernels_common.h"
#include "fft_lds.h"

namespace mmk {

// 3x3 kernel multiply at (ky, kz) with the kernel slice of one kx staged in LDS as [6][PZ/2+1][PY/2+1]
template <int PY, int PZ>
__device__ __forceinline__ void kernel_mul_lds(const float* Ks, int ky, int kz, float2& mx, float2& my, float2& mz) {
  constexpr int HY = PY / 2, HZ = PZ / 2, PL = (HZ + 1) * (HY + 1);
  int ky2 = ky, kz2 = kz;
  float sy = 1.f, sz = 1.f;
  if (ky > HY) { ky2 = PY - ky; sy = -1.f; }
  if (kz > HZ) { kz2 = PZ - kz; sz = -1.f; }
  const float* K = Ks + kz2 * (HY + 1) + ky2;
  const float nxx = K[0], nyy = K[PL], nzz = K[2 * PL];
  const float nxy = sy * K[3 * PL], nxz = sz * K[4 * PL], nyz = sy * sz * K[5 * PL];
  const float2 a = mx, b = my, c = mz;
  mx = make_float2(nxx * a.x + nxy * b.x + nxz * c.x, nxx * a.y + nxy * b.y + nxz * c.y);
  my = make_float2(nxy * a.x + nyy * b.x + nyz * c.x, nxy * a.y + nyy * b.y + nyz * c.y);
  mz = make_float2(nxz * a.x + nyz * b.x + nzz * c.x, nxz * a.y + nyz * b.y + nzz * c.y);
}

__host__ __device__ constexpr int brevc(int p, int lg) {
  int r = 0;
  for (int b = 0; b < lg; ++b) r |= ((p >> b) & 1) << (lg - 1 - b);
  return r;
}
__host__ __device__ constexpr int ilog2c(int m) { return m <= 1 ? 0 : 1 + ilog2c(m >> 1); }

// cos(2 pi j / 16)
__device__ __forceinline__ constexpr float cos16(int j) {
  j &= 15;
  switch (j) {
    case 0: return 1.0f;
    case 1: case 15: return 0.92387953251128674f;
    case 2: case 14: return 0.70710678118654752f;
    case 3: case 13: return 0.38268343236508977f;
    case 4: case 12: return 0.0f;
    case 5: case 11: return -0.38268343236508977f;
    case 6: case 10: return -0.70710678118654752f;
    case 7: case 9: return -0.92387953251128674f;
    default: return -1.0f;
  }
}

// d * W_M^{k} (forward, W_M = e^{-2 pi i / M}) or d * W_M^{-k} (inverse), 0 <= k < M/2, M <= 16
template <int M, bool INV>
__device__ __forceinline__ float2 twc(float2 d, int k) {
  if (k == 0) return d;
  const int j = k * (16 / M);
  if (j == 4) return rot<INV>(d);
  const float c = cos16(j), sn = INV ? cos16(j - 4) : -cos16(j - 4);
  return make_float2(d.x * c - d.y * sn, d.x * sn + d.y * c);
}
// points per lane Q and lanes per line L of a padded length P (Q >= L):
// y rows take up to sixteen points per lane, z columns eight
template <int P, int QMAX>
struct LinePass {
  static constexpr int Q = P / 2 < QMAX ? P / 2 : QMAX, L = P / Q;
  static constexpr int lgQ = ilog2c(Q), lgL = ilog2c(L);
  static_assert(Q >= L && L >= 2, "unsupported padded length");
};

// radix-2 DIF stages h = H0 .. 1 of an in-register M-point DFT (M <= 16):
// natural order in, bit-reversed out when H0 = M/2
template <int M, bool INV, int H0>
__device__ __forceinline__ void dif_stages(float2 (&v)[M]) {
#pragma unroll
  for (int h = H0; h >= 1; h >>= 1) {
#pragma unroll
    for (int g = 0; g < M; g += 2 * h) {
#pragma unroll
      for (int i = 0; i < h; ++i) {
        const float2 a = v[g + i], b = v[g + i + h];
        v[g + i] = cadd(a, b);
        v[g + i + h] = twc<M, INV>(csub(a, b), i * (M / (2 * h)));
      }
    }
  }
}
// the same DFT of a sequence whose entries M/2 .. M-1 are zero (not read):
// the first stage has nothing to add and only scales
template <int M, bool INV>
__device__ __forceinline__ void dif_half(float2 (&v)[M]) {
#pragma unroll
  for (int i = 0; i < M / 2; ++i) v[i + M / 2] = twc<M, INV>(v[i], i);
  if constexpr (M >= 4) dif_stages<M, INV, M / 4>(v);
}

// exchange slot of value k1 from / for lane a: groups of L slots, rotated by
// k1 so that a write of fixed k1 and a read of fixed a both spread over L
// groups (and so over LDS banks)
template <int L>
__device__ __forceinline__ int xslot(int k1, int a) {
  return k1 * L + ((a + k1) & (L - 1));
}

__device__ __forceinline__ float2 conjf2(float2 a) { return make_float2(a.x, -a.y); }

// The y transforms of one row held in LDS by N lanes (lane lam).  Forward:
// inputs at slots [0, P/2), afterwards slot k holds X[k].  Inverse: slot k
// holds X[k], afterwards slots [0, P/2) hold the inverse transform (no 1/P).
// wf[k1] = W_P^{lam k1}; wv[j][n1] = W_P^{-n1 (lam + N j)}.
template <int P>
struct YRow {
  using LP = LinePass<P, 16>;
  static constexpr int Q = LP::Q, N = LP::L;
  struct Tw {
    float2 wf[Q], wv[Q / N][N];
  };
  __device__ static void twiddles(Tw& w, const float2* tw, int lam) {
#pragma unroll
    for (int k1 = 0; k1 < Q; ++k1) w.wf[k1] = tw[lam * k1];
#pragma unroll
    for (int j = 0; j < Q / N; ++j)
#pragma unroll
      for (int n1 = 0; n1 < N; ++n1) w.wv[j][n1] = conjf2(j == 0 ? w.wf[n1] : tw[n1 * (lam + N * j)]);
  }
  __device__ static void forward(float2* line, int lam, const Tw& w) {
    float2 v[Q];
#pragma unroll
    for (int n1 = 0; n1 < Q / 2; ++n1) v[n1] = line[N * n1 + lam];
    dif_half<Q, false>(v);
    wave_lds_order();
#pragma unroll
    for (int p = 0; p < Q; ++p) {
      const int k1 = brevc(p, LP::lgQ);
      line[xslot<N>(k1, lam)] = k1 ? cmul(v[p], w.wf[k1]) : v[p];
    }
    wave_lds_order();
    float2 u[Q / N][N];
#pragma unroll
    for (int j = 0; j < Q / N; ++j) {
#pragma unroll
      for (int a = 0; a < N; ++a) u[j][a] = line[xslot<N>(lam + N * j, a)];
      dif_stages<N, false, N / 2>(u[j]);
    }
    wave_lds_order();
#pragma unroll
    for (int j = 0; j < Q / N; ++j)
#pragma unroll
      for (int p = 0; p < N; ++p) line[lam + N * j + Q * brevc(p, LP::lgL)] = u[j][p];
  }
  // Two real rows A, B transformed as one row A + iB: afterwards slot
  // SM::of(0, k) holds A[k] = (X[k] + conj X[P-k]) / 2 and SM::of(1, k) holds
  // B[k] = (X[k] - conj X[P-k]) / 2i for k < P/2, except that the real values
  // at k = 0 and P/2 share the slots of k = 0: (A[0], A[P/2]) and (B[0], B[P/2]).
  template <class SM>
  __device__ static void split_pair(float2* line, int lam) {
    constexpr int H = P / 2, NI = H / N;
    float2 r[NI], q[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int k = lam + N * i;
      r[i] = line[k];
      q[i] = line[k == 0 ? H : P - k];
    }
    wave_lds_order();
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int k = lam + N * i;
      const bool z = k == 0;
      line[SM::of(0, k)] = z ? make_float2(r[i].x, q[i].x) : make_float2(0.5f * (r[i].x + q[i].x), 0.5f * (r[i].y - q[i].y));
      line[SM::of(1, k)] = z ? make_float2(r[i].y, q[i].y) : make_float2(0.5f * (r[i].y + q[i].y), 0.5f * (q[i].x - r[i].x));
    }
  }
  // The inverse's input at k = k1 + Q k2 from two half spectra laid out as
  // split_pair leaves them (both of real rows, so X[P-k] = conj X[k]):
  // A[k] + i B[k], whose inverse has A's row as real and B's as imaginary part.
  template <class SM>
  __device__ static float2 pair_value(const float2* line, int k1, int k2) {
    constexpr int H = P / 2;
    if (k2 < N / 2) {                            // k < P/2
      const int k = k1 + Q * k2;
      const float2 a = line[SM::of(0, k)], b = line[SM::of(1, k)];
      return k == 0 ? make_float2(a.x, b.x) : make_float2(a.x - b.y, a.y + b.x);
    }
    const int m = P - (k1 + Q * k2);             // 1 .. P/2
    const int i = m == H ? 0 : m;
    const float2 a = line[SM::of(0, i)], b = line[SM::of(1, i)];
    return m == H ? make_float2(a.y, b.y) : make_float2(a.x + b.y, b.x - a.y);
  }
  // SM = void: a plain row; else two half spectra (split_pair's layout)
  template <class SM = void>
  __device__ static void inverse(float2* line, int lam, const Tw& w) {
    float2 g[Q / N][N];
#pragma unroll
    for (int j = 0; j < Q / N; ++j) {
#pragma unroll
      for (int k2 = 0; k2 < N; ++k2) {
        if constexpr (std::is_void_v<SM>) g[j][k2] = line[lam + N * j + Q * k2];
        else g[j][k2] = pair_value<SM>(line, lam + N * j, k2);
      }
      dif_stages<N, true, N / 2>(g[j]);
    }
    wave_lds_order();
#pragma unroll
    for (int j = 0; j < Q / N; ++j)
#pragma unroll
      for (int n1 = 0; n1 < N; ++n1) {
        const float2 zv = g[j][brevc(n1, LP::lgL)];
        line[xslot<N>(lam + N * j, n1)] = n1 == 0 ? zv : cmul(zv, w.wv[j][n1]);
      }
    wave_lds_order();
    float2 v[Q];
#pragma unroll
    for (int k1 = 0; k1 < Q; ++k1) v[k1] = line[xslot<N>(k1, lam)];
    dif_stages<Q, true, Q / 2>(v);
    wave_lds_order();
#pragma unroll
    for (int n2 = 0; n2 < Q / 2; ++n2) line[lam + N * n2] = v[brevc(n2, LP::lgQ)];
  }
};

// The z convolution of one column held in LDS by N lanes (lane lam): the
// three components at rows c ZR + z (stride RS, ZR = P/2; rows nz .. ZR-1
// zero), forward z, the kernel multiply kmul(kz, x, y, z) at every kz, the
// inverse z; rows z < nz receive the result.  The column's 3 ZR slots serve
// as the exchange area once its inputs are in registers.
template <int P>
struct ZCol {
  using LP = LinePass<P, 8>;
  static constexpr int Q = LP::Q, N = LP::L, ZR = P / 2;
  struct Tw {
    float2 wf[Q], wv[Q / N][N];
  };
  __device__ static void twiddles(Tw& w, const float2* tw, int lam) {
#pragma unroll
    for (int k1 = 0; k1 < Q; ++k1) w.wf[k1] = tw[lam * k1];
#pragma unroll
    for (int j = 0; j < Q / N; ++j)
#pragma unroll
      for (int n1 = 0; n1 < N; ++n1) w.wv[j][n1] = conjf2(j == 0 ? w.wf[n1] : tw[n1 * (lam + N * j)]);
  }
  using Spec = float2[3][Q / N][N];
  // frequency of sp[c][j][p] after forward(): k1 + Q brev(p), k1 = lam + N j
  __device__ static int kz_of(int lam, int j, int p) { return lam + N * j + Q * brevc(p, LP::lgL); }
  __device__ static void forward(float2* col, int RS, int lam, const Tw& w, Spec& sp) {
    float2 xin[3][Q / 2];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int n1 = 0; n1 < Q / 2; ++n1) xin[c][n1] = col[(c * ZR + N * n1 + lam) * RS];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      float2 v[Q];
#pragma unroll
      for (int n1 = 0; n1 < Q / 2; ++n1) v[n1] = xin[c][n1];
      dif_half<Q, false>(v);
      wave_lds_order();
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        const int k1 = brevc(p, LP::lgQ);
        col[xslot<N>(k1, lam) * RS] = k1 ? cmul(v[p], w.wf[k1]) : v[p];
      }
      wave_lds_order();
#pragma unroll
      for (int j = 0; j < Q / N; ++j) {
#pragma unroll
        for (int a = 0; a < N; ++a) sp[c][j][a] = col[xslot<N>(lam + N * j, a) * RS];
        dif_stages<N, false, N / 2>(sp[c][j]);
      }
      wave_lds_order();
    }
  }
  // inverse z of sp (the column's slots are the exchange area); rows z < nz
  // receive the result
  __device__ static void inverse(float2* col, int RS, int nz, int lam, const Tw& w, Spec& sp) {
    float2 res[3][Q / 2];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
#pragma unroll
      for (int j = 0; j < Q / N; ++j) {
        float2 g[N];
#pragma unroll
        for (int k2 = 0; k2 < N; ++k2) g[k2] = sp[c][j][brevc(k2, LP::lgL)];
        dif_stages<N, true, N / 2>(g);
        // g[p] = sum_k2 X[k1 + Q k2] W_N^{-n1 k2} at n1 = brev(p)
#pragma unroll
        for (int n1 = 0; n1 < N; ++n1) {
          const float2 zv = g[brevc(n1, LP::lgL)];
          col[xslot<N>(lam + N * j, n1) * RS] = n1 == 0 ? zv : cmul(zv, w.wv[j][n1]);
        }
      }
      wave_lds_order();
      float2 v[Q];
#pragma unroll
      for (int k1 = 0; k1 < Q; ++k1) v[k1] = col[xslot<N>(k1, lam) * RS];
      dif_stages<Q, true, Q / 2>(v);
#pragma unroll
      for (int n2 = 0; n2 < Q / 2; ++n2) res[c][n2] = v[brevc(n2, LP::lgQ)];
      wave_lds_order();
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int n2 = 0; n2 < Q / 2; ++n2) {
        const int z = lam + N * n2;
        if (z < nz) col[(c * ZR + z) * RS] = res[c][n2];
      }
  }
  template <class KMul>
  __device__ static void convolve(float2* col, int RS, int nz, int lam, const Tw& w, KMul&& kmul) {
    Spec sp;
    forward(col, RS, lam, w, sp);
#pragma unroll
    for (int j = 0; j < Q / N; ++j)
#pragma unroll
      for (int p = 0; p < N; ++p) kmul(kz_of(lam, j, p), sp[0][j][p], sp[1][j][p], sp[2][j][p]);
    inverse(col, RS, nz, lam, w, sp);
  }
};

// LDS bank layout shared by the kernels below (64 banks of four bytes; an
// eight-byte access is served 32 lanes per cycle).  Rows are an odd number of
// slots apart.  A y row has N lanes, lane = lam * RPW + r in its wavefront
// (RPW = 64 / N rows), and the wavefront's rows are SY = N / 2 apart, so the
// 32 lanes of a half-wavefront (N / 2 values of lam, RPW rows) fall on
// distinct bank pairs; the rows of SY wavefronts interleave to fill blocks of
// 32 rows.  A z column has N consecutive lanes and the wavefront's columns
// are SZ apart (SZ = N where the tile is wide enough), for the same reason.
// Row of y-lane yrl in block g0 of wavefront `wave`:
template <int N>
__device__ __forceinline__ int yrow_of(int g0, int wave, int yrl) {
  constexpr int SY = N / 2;
  return 32 * g0 + wave % SY + SY * yrl;
}
// Column of thread t in a tile of NCOL columns, N lanes per column:
template <int N, int NCOL>
__device__ __forceinline__ int zcol_of(int t) {
  constexpr int CPW = 64 / N, SZ = NCOL <= CPW ? 1 : N < NCOL / CPW ? N : NCOL / CPW;
  const int wz = t >> 6;
  return wz % SZ + SZ * ((t & 63) / N) + SZ * CPW * (wz / SZ);
}

// M-point transforms of one row of M slots by N lanes (lane lam), in place;
// twm: W_M in LDS.
template <int M>
struct YFull {
  static constexpr int Q = M / 2 < 16 ? M / 2 : 16, N = M / Q, lgQ = ilog2c(Q), lgN = ilog2c(N);
  static_assert(N >= 2 && N <= Q, "row length");
  __device__ static void forward(float2* line, int lam, const float2* twm) {
    float2 v[Q];
#pragma unroll
    for (int n1 = 0; n1 < Q; ++n1) v[n1] = line[N * n1 + lam];
    dif_stages<Q, false, Q / 2>(v);
    wave_lds_order();
#pragma unroll
    for (int p = 0; p < Q; ++p) {
      const int k1 = brevc(p, lgQ);
      line[xslot<N>(k1, lam)] = k1 ? cmul(v[p], twm[lam * k1]) : v[p];
    }
    wave_lds_order();
    float2 u[Q / N][N];
#pragma unroll
    for (int j = 0; j < Q / N; ++j) {
#pragma unroll
      for (int a = 0; a < N; ++a) u[j][a] = line[xslot<N>(lam + N * j, a)];
      dif_stages<N, false, N / 2>(u[j]);
    }
    wave_lds_order();
#pragma unroll
    for (int j = 0; j < Q / N; ++j)
#pragma unroll
      for (int p = 0; p < N; ++p) line[lam + N * j + Q * brevc(p, lgN)] = u[j][p];
  }
  // Row of A + iB (A, B real rows before the twist by W_2M^{rj}) to their
  // spectra: A[k] = (X[k] + conj X[k']) / 2, B[k] = (X[k] - conj X[k']) / 2i
  // with k' = M - k (r = 0) or M - 1 - k (r = 1), k < M/2, at slots
  // SM::of(0, k) and SM::of(1, k); for r = 0 the real values at k = 0 and M/2
  // share the slots of k = 0.
  template <class SM>
  __device__ static void split_pair(float2* line, int lam, int r) {
    constexpr int H = M / 2, NI = H / N;
    float2 x[NI], q[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int k = lam + N * i;
      x[i] = line[k];
      q[i] = line[r ? M - 1 - k : k == 0 ? H : M - k];
    }
    wave_lds_order();
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int k = lam + N * i;
      const bool z = !r && k == 0;
      line[SM::of(0, k)] = z ? make_float2(x[i].x, q[i].x) : make_float2(0.5f * (x[i].x + q[i].x), 0.5f * (x[i].y - q[i].y));
      line[SM::of(1, k)] = z ? make_float2(x[i].y, q[i].y) : make_float2(0.5f * (x[i].y + q[i].y), 0.5f * (q[i].x - x[i].x));
    }
  }
  // spectrum of A + iB at k from the two half spectra
  template <class SM>
  __device__ static float2 pair_value(const float2* line, int k, int r) {
    constexpr int H = M / 2;
    const bool lo = k < H;
    const int m = lo ? k : r ? M - 1 - k : M - k;
    const int i = m == H ? 0 : m;                 // (r = 0, k = M/2: the shared slot)
    const float2 a = line[SM::of(0, i)], b = line[SM::of(1, i)];
    if (!r && k == 0) return make_float2(a.x, b.x);
    if (m == H) return make_float2(a.y, b.y);
    return lo ? make_float2(a.x - b.y, a.y + b.x) : make_float2(a.x + b.y, b.x - a.y);
  }
  template <class SM = void>
  __device__ static void inverse(float2* line, int lam, const float2* twm, int r) {
    float2 g[Q / N][N];
#pragma unroll
    for (int j = 0; j < Q / N; ++j) {
#pragma unroll
      for (int k2 = 0; k2 < N; ++k2) {
        if constexpr (std::is_void_v<SM>) g[j][k2] = line[lam + N * j + Q * k2];
        else g[j][k2] = pair_value<SM>(line, lam + N * j + Q * k2, r);
      }
      dif_stages<N, true, N / 2>(g[j]);
    }
    wave_lds_order();
#pragma unroll
    for (int j = 0; j < Q / N; ++j)
#pragma unroll
      for (int n1 = 0; n1 < N; ++n1) {
        const float2 zv = g[j][brevc(n1, lgN)];
        line[xslot<N>(lam + N * j, n1)] = n1 == 0 ? zv : cmul(zv, conjf2(twm[n1 * (lam + N * j)]));
      }
    wave_lds_order();
    float2 v[Q];
#pragma unroll
    for (int k1 = 0; k1 < Q; ++k1) v[k1] = line[xslot<N>(k1, lam)];
    dif_stages<Q, true, Q / 2>(v);
    wave_lds_order();
#pragma unroll
    for (int n2 = 0; n2 < Q; ++n2) line[lam + N * n2] = v[brevc(n2, lgQ)];
  }
};

}  // namespace mmk
