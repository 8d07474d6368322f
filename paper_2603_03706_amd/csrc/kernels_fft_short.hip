// y-z convolution of grids with few z planes: padded z of 1 (thin films), 4, 8
// or 16.  One kx plane of such a grid is a few dozen short lines; a workgroup
// here has just the lanes that its z columns (or, without z, its lines) need,
// one or two wavefronts for most sizes, so that a plane is loaded, transformed,
// multiplied and stored with next to no barriers and every plane of every
// instance is resident at once.  The lines are the two-pass ones of the
// exchange kernel.
//
// What bounds them: the latency of the phases (loads, line passes, store);
// the launch is one round of small workgroups.  A DP45 step of the 200x200x1
// film takes 127 us with it against 251 us with the LDS-resident passes of
// k_fft_yz (512 threads and a dozen barriers for three rows), one of the
// 16x12x4 film 116 against 140 us; both with the finalisations of stages 2
// to 6, 4.5 us each as launches of their own, riding along.  Of many modes one
// or two wavefronts gather the sums in turn, which sixteen profiled ones show,
// but less than the launches: 200x200x1 250 against 441 us, 64x64x1 232 against
// 275, eight of them 227 against 277.
#include "mm_internal.h"
#include "mm_host.h"
#include "kernels_common.h"
#include "launch.h"
#include "fft_lds.h"
#include "fft_lines.h"
#include "stage_final.h"

namespace mmk {

template <int PY, int PZ>
struct YzShort {
  static constexpr int T = 2 * PY < 64 ? 64 : 2 * PY, ZR = PZ / 2, RS = PY + 1;
  static constexpr int HY1 = PY / 2 + 1, KPL = (PZ / 2 + 1) * HY1;
  static constexpr size_t lds = sizeof(float2) * (3 * ZR * RS + PY + PZ) + sizeof(float) * 6 * KPL;
};

// work item = kx of one instance; workgroups nyz .. run finalisations (see k_fft_yzx)
template <int PY, int PZ>
__global__ __launch_bounds__((YzShort<PY, PZ>::T)) void k_fft_yzs(const InstDesc* __restrict__ descs,
                                                                  const WorkItem* __restrict__ work,
                                                                  const float2* __restrict__ tw, int nyz, int fmethod,
                                                                  int fstage) {
  using H = YzShort<PY, PZ>;
  using YR_ = YRow<PY>;
  using ZC = ZCol<PZ>;
  constexpr int T = H::T, NY = YR_::N, NZ = ZC::N, ZR = H::ZR, RS = H::RS, YR = PY / 2, KPL = H::KPL;
  constexpr int RPW = 64 / NY, SY = NY / 2, NW = T / 64, RPI = T / PY, RPO = T / YR;
  static_assert(NW % SY == 0 && T >= NZ * PY, "layout");
  extern __shared__ float2 lds[];
  if ((int)blockIdx.x >= nyz) {
    final_any(fmethod, fstage, descs, (int)blockIdx.x - nyz, reinterpret_cast<double*>(lds));
    return;
  }
  const WorkItem wi = work[blockIdx.x];
  const InstDesc& D = descs[wi.inst];
  if (transform_idle(D)) return;
  float2* B = lds;                              // rows [3][ZR][PY + 1]
  float2* twy = B + 3 * ZR * RS;
  float2* twz = twy + PY;
  float* Ks = reinterpret_cast<float*>(twz + PZ);
  const int ny = D.ny, nz = D.nz, kx = wi.item;
  MMG float2* X = gbl(D.fx) + (size_t)kx * 3 * nz * ny;
  {
    constexpr int NK = (6 * KPL + T - 1) / T, NX = (3 * ZR + RPI - 1) / RPI;
    const MMG float* K = gbl(D.kern) + (size_t)kx * 6 * KPL;
    float kv[NK];
    float2 xv[NX];
    const int y = threadIdx.x & (PY - 1), r0 = threadIdx.x / PY;
#pragma unroll
    for (int it = 0; it < NX; ++it) {
      const int row = it * RPI + r0, c = row / ZR, z = row % ZR;
      const bool in = row < 3 * ZR && z < nz && y < ny;
      const float2 v = gld2(X + (in ? (c * nz + z) * ny + y : 0));
      xv[it] = make_float2(in ? v.x : 0.f, in ? v.y : 0.f);
    }
#pragma unroll
    for (int it = 0; it < NK; ++it) kv[it] = K[min(it * T + (int)threadIdx.x, 6 * KPL - 1)];
    load_twiddles(twy, PY, tw, T);
    load_twiddles(twz, PZ, tw, T);
#pragma unroll
    for (int it = 0; it < NX; ++it) {
      const int row = it * RPI + r0;
      if (row < 3 * ZR) B[row * RS + y] = xv[it];
    }
#pragma unroll
    for (int it = 0; it < NK; ++it) {
      const int e = it * T + threadIdx.x;
      if (e < 6 * KPL) Ks[e] = kv[it];
    }
  }
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int ylam = lane / RPW, yrl = lane % RPW;
  typename YR_::Tw wy;
  YR_::twiddles(wy, twy, ylam);
#pragma unroll 1
  for (int g0 = wave / SY; 32 * g0 < 3 * ZR; g0 += NW / SY) {
    const int rho = yrow_of<NY>(g0, wave, yrl);
    if (rho < 3 * ZR && (rho & (ZR - 1)) < nz) YR_::forward(B + rho * RS, ylam, wy);
  }
  __syncthreads();
  if ((int)threadIdx.x < NZ * PY) {
    const int lam = threadIdx.x & (NZ - 1);
    typename ZC::Tw wz;
    ZC::twiddles(wz, twz, lam);
    const int ky = zcol_of<NZ, PY>(threadIdx.x);
    ZC::convolve(B + ky, RS, nz, lam, wz, [&](int kz, float2& a, float2& b, float2& c) {
      kernel_mul_lds<PY, PZ>(Ks, ky, kz, a, b, c);
    });
  }
  __syncthreads();
#pragma unroll 1
  for (int g0 = wave / SY; 32 * g0 < 3 * ZR; g0 += NW / SY) {
    const int rho = yrow_of<NY>(g0, wave, yrl);
    if (rho < 3 * ZR && (rho & (ZR - 1)) < nz) YR_::inverse(B + rho * RS, ylam, wy);
  }
  __syncthreads();
  constexpr int NO = (3 * ZR + RPO - 1) / RPO;
  const int y = threadIdx.x & (YR - 1), r0 = threadIdx.x / YR;
#pragma unroll
  for (int it = 0; it < NO; ++it) {
    const int row = it * RPO + r0, c = row / ZR, z = row % ZR;
    if (row < 3 * ZR && z < nz && y < ny) gst2(X + (c * nz + z) * ny + y, B[row * RS + y]);
  }
}

// One z plane: a kx plane is three rows.  Each row is split by the parity of
// its frequency index (see k_fft_yzh) into two M-point lines, M = Py/2, six
// lines of N lanes; the product takes its kernel values from memory, loaded
// before the first line pass.
template <int M>
struct YThin {
  static constexpr int N = YFull<M>::N, T = (6 * N + 63) / 64 * 64, RS = M + 1;
  static constexpr size_t lds = sizeof(float2) * (6 * RS + M);
};

template <int M>
__global__ __launch_bounds__(YThin<M>::T) void k_fft_y1(const InstDesc* __restrict__ descs,
                                                        const WorkItem* __restrict__ work,
                                                        const float2* __restrict__ tw, int nyz, int fmethod,
                                                        int fstage) {
  using H = YThin<M>;
  using YF = YFull<M>;
  constexpr int T = H::T, N = H::N, RS = H::RS, NP = (2 * M + T - 1) / T, NX = (M + T - 1) / T;
  extern __shared__ float2 lds[];
  if ((int)blockIdx.x >= nyz) {
    final_any(fmethod, fstage, descs, (int)blockIdx.x - nyz, reinterpret_cast<double*>(lds));
    return;
  }
  const WorkItem wi = work[blockIdx.x];
  const InstDesc& D = descs[wi.inst];
  if (transform_idle(D)) return;
  float2* B = lds;                              // lines [2 component + parity][M + 1]
  float2* twm = B + 6 * RS;
  const int ny = D.ny, kx = wi.item;
  MMG float2* X = gbl(D.fx) + (size_t)kx * 3 * ny;
  const MMG float* K = gbl(D.kern) + (size_t)kx * 6 * (M + 1);
  float2 xv[NX][3], wt[NX];
  float kv[NP][6];
#pragma unroll
  for (int it = 0; it < NX; ++it) {
    const int y = it * T + threadIdx.x;
    const bool in = y < ny;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float2 v = gld2(X + (in ? c * ny + y : 0));
      xv[it][c] = make_float2(in ? v.x : 0.f, in ? v.y : 0.f);
    }
    wt[it] = tw[min(y, M - 1) * (MMI_TW_LEN / (2 * M))];
  }
#pragma unroll
  for (int it = 0; it < NP; ++it) {
    const int ky = min(it * T + (int)threadIdx.x, 2 * M - 1), ky2 = ky > M ? 2 * M - ky : ky;
#pragma unroll
    for (int q = 0; q < 6; ++q) kv[it][q] = K[q * (M + 1) + ky2];
  }
  load_twiddles(twm, M, tw, T);
#pragma unroll
  for (int it = 0; it < NX; ++it) {
    const int y = it * T + threadIdx.x;
    if (y < M)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        B[2 * c * RS + y] = xv[it][c];
        B[(2 * c + 1) * RS + y] = cmul(xv[it][c], wt[it]);
      }
  }
  __syncthreads();
  const int line = threadIdx.x / N, lam = threadIdx.x % N;
  if (line < 6) YF::forward(B + line * RS, lam, twm);
  __syncthreads();
#pragma unroll
  for (int it = 0; it < NP; ++it) {
    const int ky = it * T + threadIdx.x;
    if (ky < 2 * M) {
      float2* p = B + (ky & 1) * RS + (ky >> 1);
      const float sy = ky > M ? -1.f : 1.f;
      const float nxx = kv[it][0], nyy = kv[it][1], nzz = kv[it][2];
      const float nxy = sy * kv[it][3], nxz = kv[it][4], nyz_ = sy * kv[it][5];
      const float2 a = p[0], b = p[2 * RS], c = p[4 * RS];
      p[0] = make_float2(nxx * a.x + nxy * b.x + nxz * c.x, nxx * a.y + nxy * b.y + nxz * c.y);
      p[2 * RS] = make_float2(nxy * a.x + nyy * b.x + nyz_ * c.x, nxy * a.y + nyy * b.y + nyz_ * c.y);
      p[4 * RS] = make_float2(nxz * a.x + nyz_ * b.x + nzz * c.x, nxz * a.y + nyz_ * b.y + nzz * c.y);
    }
  }
  __syncthreads();
  if (line < 6) YF::inverse(B + line * RS, lam, twm, 0);
  __syncthreads();
#pragma unroll
  for (int it = 0; it < NX; ++it) {
    const int y = it * T + threadIdx.x;
    if (y < ny)
#pragma unroll
      for (int c = 0; c < 3; ++c)
        gst2(X + c * ny + y, cadd(B[2 * c * RS + y], cmul(B[(2 * c + 1) * RS + y], conjf2(wt[it]))));
  }
}

}  // namespace mmk

#define MM_YZS_EACH(F)                                                                      \
  F(8, 4) F(16, 4) F(32, 4) F(64, 4) F(128, 4) F(256, 4) F(8, 8) F(16, 8) F(32, 8) F(64, 8) \
  F(128, 8) F(256, 8) F(8, 16) F(16, 16) F(32, 16) F(64, 16) F(128, 16) F(256, 16)
#define MM_Y1_EACH(F) F(4) F(8) F(16) F(32) F(64) F(128) F(256)

size_t mmk_yzs_lds(int py, int pz) {
  size_t n = 0;
#define MM_YZS_LDS(A, B) \
  if (py == A && pz == B) n = mmk::YzShort<A, B>::lds;
#define MM_Y1_LDS(A) \
  if (pz == 1 && py == 2 * A) n = mmk::YThin<A>::lds;
  MM_YZS_EACH(MM_YZS_LDS)
  MM_Y1_EACH(MM_Y1_LDS)
  // (room for a finalisation's sums)
  return n == 0 || n >= MMI_PSTRIDE * sizeof(double) ? n : MMI_PSTRIDE * sizeof(double);
}

hipError_t mmk_launch_fft_yzs(int py, int pz, int nblocks, size_t lds, const InstDesc* d, const WorkItem* w,
                              const float2* tw, hipStream_t s, int nfinal, int fmethod, int fstage) {
  if (nfinal < 0 || lds < mmk_yzs_lds(py, pz)) return hipErrorInvalidValue;
#define MM_YZS_CASE(A, B)                                                                                  \
  if (py == A && pz == B) {                                                                                \
    constexpr int T = mmk::YzShort<A, B>::T;                                                               \
    MM_LAUNCH((mmk::k_fft_yzs<A, B>), dim3(nblocks + nfinal), dim3(T), lds, s, d, w, tw, nblocks, fmethod, \
              fstage);                                                                                     \
    return hipGetLastError();                                                                              \
  }
#define MM_Y1_CASE(A)                                                                                      \
  if (pz == 1 && py == 2 * A) {                                                                            \
    constexpr int T = mmk::YThin<A>::T;                                                                    \
    MM_LAUNCH(mmk::k_fft_y1<A>, dim3(nblocks + nfinal), dim3(T), lds, s, d, w, tw, nblocks, fmethod,       \
              fstage);                                                                                     \
    return hipGetLastError();                                                                              \
  }
  MM_YZS_EACH(MM_YZS_CASE)
  MM_Y1_EACH(MM_Y1_CASE)
  return hipErrorInvalidValue;
}

hipError_t mmk_set_short_lds_limits() {
  hipError_t e = hipSuccess;
#define MM_YZS_ATTR(A, B)                                                                                  \
  if (e == hipSuccess && mmk::YzShort<A, B>::lds > 64 * 1024)                                              \
    e = hipFuncSetAttribute((const void*)mmk::k_fft_yzs<A, B>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  MM_YZS_EACH(MM_YZS_ATTR)
  return e;
}
