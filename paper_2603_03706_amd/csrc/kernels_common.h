// Small device helpers shared by the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>
#include "mm_internal.h"

namespace mmk {

// Every buffer reached through the descriptor table lives in global memory.
// Stating the address space lets the compiler emit global loads and stores
// (scalar base + 32-bit offset, vector-memory counter only) instead of flat
// ones, which carry 64-bit addresses and also wait on the LDS counter.
#define MMG __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ MMG T* gbl(T* p) {
  return (MMG T*)p;
}

// float2 through global pointers (the vector type's operators do not take
// address-space qualified operands)
__device__ __forceinline__ float2 gld2(const MMG float2* p) {
  const MMG float* q = (const MMG float*)p;
  return make_float2(q[0], q[1]);
}
__device__ __forceinline__ void gst2(MMG float2* p, float2 v) {
  MMG float* q = (MMG float*)p;
  q[0] = v.x;
  q[1] = v.y;
}

// Element i of a global array through a scalar base and an unsigned 32-bit
// byte offset (i >= 0 and i * sizeof(T) < 2^32; the host bounds instance
// sizes accordingly): with a signed index every lane would form a 64-bit
// address (sign extension and a 64-bit add per access).
template <class T>
__device__ __forceinline__ const MMG T& gat(const MMG T* p, int i) {
  return *(const MMG T*)((const MMG char*)p + (uint32_t)i * (uint32_t)sizeof(T));
}
template <class T>
__device__ __forceinline__ MMG T& gat(MMG T* p, int i) {
  return *(MMG T*)((MMG char*)p + (uint32_t)i * (uint32_t)sizeof(T));
}

// Stage input m = p0 + c1 * p1 (p1 optional), component-major per instance.
struct Src {
  const MMG float* p0;
  const MMG float* p1;
  float c1;
  __device__ __forceinline__ float ld(int idx) const {
    float v = gat(p0, idx);
    if (p1) v = fmaf(c1, gat(p1, idx), v);
    return v;
  }
};

// The same with the presence of p1 fixed at compile time, so that every
// load of a stencil (both fields when TWO) is issued without a test.
template <bool TWO>
struct SrcFixed {
  const MMG float* p0;
  const MMG float* p1;
  float c1;
  __device__ __forceinline__ explicit SrcFixed(const Src& s) : p0(s.p0), p1(s.p1), c1(s.c1) {}
  __device__ __forceinline__ float ld(int idx) const {
    float v = gat(p0, idx);
    if (TWO) v = fmaf(c1, gat(p1, idx), v);
    return v;
  }
};

// Where the input of stage `stage` lives.  RK4: 0/1 state, 2 and 4 buffer
// A, 3 buffer B.  DP45: 1 state, 2 state + h a21 k1 (not stored), 3 and 5
// buffer A, 4 and 6 buffer B, 7 the normalised candidate.
template <class CtlPtr>
__device__ __forceinline__ Src stage_src(const InstDesc& D, CtlPtr C, int method, int stage) {
  Src s;
  s.p1 = nullptr;
  s.c1 = 0.f;
  const int cur = C->cur;
  if (method == MMI_ADJ) {
    // adjoint: stage 1..nstg -> recorded stage input of the current step, 0 -> lambda_B
    const size_t vec = (size_t)3 * D.S * D.ncell;
    s.p0 = gbl((stage == 0) ? D.lam_B : D.rec_m + ((size_t)C->rec_index * D.rec_nstg + (stage - 1)) * vec);
    return s;
  }
  if (method == MMI_RK4) {
    s.p0 = gbl((stage <= 1) ? D.y[cur] : (stage == 3 ? D.st[1] : D.st[0]));
  } else {
    switch (stage) {
      case 1: s.p0 = gbl(D.y[cur]); break;
      case 2:
        s.p0 = gbl(D.y[cur]);
        s.p1 = gbl(D.k[C->slot[0]]);
        s.c1 = (float)(C->h * DPCoef::a21);
        break;
      case 3: case 5: s.p0 = gbl(D.st[0]); break;
      case 4: case 6: s.p0 = gbl(D.st[1]); break;
      default: s.p0 = gbl(D.y[1 - cur]); break;
    }
  }
  return s;
}

// Indices of the six neighbours of cell i at (x, y, z): a missing or
// non-magnetic neighbour is replaced by the cell itself, whose difference
// m_j - m_i is then exactly zero, so every load of a stencil is unconditional
// and all of them are in flight together.
__device__ __forceinline__ void neighbours(const InstDesc& D, int i, int x, int y, int z, int (&jn)[6]) {
  const int nx = D.nx, ny = D.ny, nz = D.nz;
  const int off[6] = {-1, 1, -nx, nx, -nx * ny, nx * ny};
  const bool has[6] = {x > 0, x < nx - 1, y > 0, y < ny - 1, z > 0, z < nz - 1};
#pragma unroll
  for (int q = 0; q < 6; ++q) jn[q] = has[q] ? i + off[q] : i;
  if (D.has_geom) {
    const MMG uint8_t* G = gbl(D.geom);
    uint8_t g[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) g[q] = gat(G, jn[q]);
#pragma unroll
    for (int q = 0; q < 6; ++q) jn[q] = g[q] ? jn[q] : i;
  }
}

// bdv: this cell's demag field already at hand (used when use_bdv; pass a
// pointer fixed at compile time, never one chosen at run time, so that the
// array stays in registers).
// Effective field [T] on sublattice s at cell i with its neighbours' values nb:
// Zeeman + exchange over magnetic neighbour pairs + uniaxial anisotropy +
// demag (local diagonal, or the FFT result in D.bd) + feedback c_s fb along
// x + intersublattice -B_E m_{s'}.  m holds the cell's own stage input.
// DESC: InstDesc, or a copy of the members used here held in registers.
template <class DESC>
__device__ __forceinline__ void field_nb(const DESC& D, int i, const float (&nb)[6][3],
                                         const float (&m)[2][3], int s, float fb,
                                         bool has_bd, float (&B)[3], const float* bdv = nullptr,
                                         bool use_bdv = true) {
  const float m0 = m[s][0], m1 = m[s][1], m2 = m[s][2];
  float bx = D.B0x, by = D.B0y, bz = D.B0z;
  const float cq[6] = {D.cex_x, D.cex_x, D.cex_y, D.cex_y, D.cex_z, D.cex_z};
  float sx = 0.f, sy = 0.f, sz = 0.f;
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    sx = fmaf(cq[q], nb[q][0] - m0, sx);
    sy = fmaf(cq[q], nb[q][1] - m1, sy);
    sz = fmaf(cq[q], nb[q][2] - m2, sz);
  }
  bx += sx;
  by += sy;
  bz += sz;
  const float md = m0 * D.ex + m1 * D.ey + m2 * D.ez;
  const float ck = D.cK * md;
  bx = fmaf(ck, D.ex, bx);
  by = fmaf(ck, D.ey, by);
  bz = fmaf(ck, D.ez, bz);
  if (D.demag == 1) {
    float tx = m[0][0], ty = m[0][1], tz = m[0][2];
    if (D.S == 2) { tx += m[1][0]; ty += m[1][1]; tz += m[1][2]; }
    bx = fmaf(D.nlx, tx, bx);
    by = fmaf(D.nly, ty, by);
    bz = fmaf(D.nlz, tz, bz);
  } else if (bdv && use_bdv) {
    bx += bdv[0];
    by += bdv[1];
    bz += bdv[2];
  } else if (has_bd) {
    const MMG float* bd = gbl(D.bd);
    const int nc = D.ncell;
    bx += gat(bd, i);
    by += gat(bd, nc + i);
    bz += gat(bd, 2 * nc + i);
  }
  bx = fmaf(D.csign[s], fb, bx);
  if (D.S == 2) {
    const int o = 1 - s;
    bx = fmaf(-D.BE, m[o][0], bx);
    by = fmaf(-D.BE, m[o][1], by);
    bz = fmaf(-D.BE, m[o][2], bz);
  }
  B[0] = bx;
  B[1] = by;
  B[2] = bz;
}

template <class SRC>
__device__ __forceinline__ void field_at(const InstDesc& D, const SRC& src, int i, int x, int y,
                                         int z, const float (&m)[2][3], int s, float fb,
                                         bool has_bd, float (&B)[3], const float* bdv = nullptr,
                                         bool use_bdv = true) {
  int jn[6];
  neighbours(D, i, x, y, z, jn);
  const int nc = D.ncell, base = s * 3 * nc;
  float nb[6][3];
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    nb[q][0] = src.ld(base + jn[q]);
    nb[q][1] = src.ld(base + nc + jn[q]);
    nb[q][2] = src.ld(base + 2 * nc + jn[q]);
  }
  field_nb(D, i, nb, m, s, fb, has_bd, B, bdv, use_bdv);
}

// weight of a mode's profile in the feedback field: h0 Re[e^{-i Phi} a]
__device__ __forceinline__ float feedback_weight(double h0, double cphi, double sphi, double ar, double ai) {
  return (float)(h0 * fma(cphi, ar, sphi * ai));
}

// LL torque -gamma' [m x B + alpha m x (m x B)] in the field B
template <class DESC>
__device__ __forceinline__ void ll_torque(const DESC& D, const float (&m)[3], const float (&B)[3], float (&k)[3]) {
  const float cx = m[1] * B[2] - m[2] * B[1];
  const float cy = m[2] * B[0] - m[0] * B[2];
  const float cz = m[0] * B[1] - m[1] * B[0];
  const float dx = m[1] * cz - m[2] * cy;
  const float dy = m[2] * cx - m[0] * cz;
  const float dz = m[0] * cy - m[1] * cx;
  const float a = D.alpha, gl = -D.gl;
  k[0] = gl * fmaf(a, dx, cx);
  k[1] = gl * fmaf(a, dy, cy);
  k[2] = gl * fmaf(a, dz, cz);
}

// Convolved x-transformed rows: in place in D.fx, or (D.yzh) as two terms in
// D.fy, one after the other, to be added.  e: element of [kx][c][z][y].
__device__ __forceinline__ const MMG float2* conv_rows(const InstDesc& D) { return gbl(D.yzh ? D.fy : D.fx); }
__device__ __forceinline__ float2 conv_row(const InstDesc& D, const MMG float2* X, int e) {
  float2 v = gld2(&gat(X, e));
  if (D.yzh) {
    const float2 w = gld2(&gat(X, e + D.yzh));
    v.x += w.x;
    v.y += w.y;
  }
  return v;
}

// The workgroups of one dispatch are placed on the eight XCDs round-robin
// (block b on XCD b mod 8) and every XCD has its own L2.  This maps the
// hardware block index to a logical one (a bijection on [0, gridDim.x)) so
// that each XCD works through one contiguous range of logical blocks: cells
// that are neighbours in z, two 512-cell workgroups apart, are then read
// through the same L2 instead of being fetched again by another XCD.
// With nb given, it is the bijection on [0, nb) for launches that carry other
// work in the blocks beyond, or in `lead` blocks (a multiple of eight) before.
__device__ __forceinline__ int xcd_block(int nb, int lead = 0) {
  const int b = (int)blockIdx.x - lead;
  const int q = nb >> 3, r = nb & 7, x = b & 7;
  return x * q + min(x, r) + (b >> 3);
}
__device__ __forceinline__ int xcd_block() { return xcd_block((int)gridDim.x); }

// Workgroup (of D.cpw cells) that the lw-th workgroup of an instance takes.
// Where a z-plane is a whole number P >= 64 of full workgroups, consecutive
// workgroups walk z first (lw = b nz + z takes block b of plane z), so that
// the planes a stencil reads above and below are fetched by workgroups that
// run close together on the same XCD (otherwise P workgroups apart, about
// the span an XCD has resident).  Smaller planes keep the plain order, in
// which z-neighbours are already close.  A bijection on the instance's
// workgroups; the workgroup's cells, x-rows and partial record follow it.
__device__ __forceinline__ int zmajor_wg(const InstDesc& D, int lw) {
  const int plane = D.nx * D.ny;
  if (D.cpw != MMI_WG || (plane & (MMI_WG - 1)) || plane < 64 * MMI_WG) return lw;
  const int P = plane >> MMI_LG_WG, b = lw / D.nz;
  return (lw - b * D.nz) * P + b;
}

// Cell of this thread in workgroup lw of the instance, or ncell (no cell):
// every thread of a workgroup has one, except where the workgroup holds whole
// x-rows that leave some threads over (D.cpw < MMI_WG).
__device__ __forceinline__ int wg_cell(const InstDesc& D, int lw) {
  return (int)threadIdx.x < D.cpw ? lw * D.cpw + (int)threadIdx.x : D.ncell;
}

// Coordinates of cell i = (z ny + y) nx + x: shifts and masks when nx and ny
// are powers of two, integer divisions otherwise.
__device__ __forceinline__ void cell_xyz(const InstDesc& D, int i, int& x, int& y, int& z) {
  if (D.lgnx >= 0 && D.lgny >= 0) {
    x = i & (D.nx - 1);
    const int yz = i >> D.lgnx;
    y = yz & (D.ny - 1);
    z = yz >> D.lgny;
  } else {
    const int yz = i / D.nx;
    x = i - yz * D.nx;
    z = yz / D.ny;
    y = yz - z * D.ny;
  }
}

// max that propagates NaN (a NaN anywhere makes the result NaN)
__device__ __forceinline__ double nan_max(double a, double b) {
  return (a != a || b != b) ? (a + b) : fmax(a, b);
}

// The value of lane l ^ O, exchanged by VALU permutations instead of LDS-unit
// shuffles: DPP within a row of 16 lanes, gfx950's row-swap instructions for
// 16 and 32 (swapping two copies of v leaves each lane's own half or row in
// one copy and its partner's in the other, so the pair is returned and the
// caller combines it in either order).  O = 4 reads the lane four to the
// side in the row of 16, which holds the value of lane l ^ 4 only where
// lanes l and l ^ 8 hold the same one: the butterflies below go from 32
// down, which makes them equal.
template <int O>
__device__ __forceinline__ void lane_pair(double v, double& a, double& b) {
  const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
  if constexpr (O == 32 || O == 16) {
    const auto l = O == 32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                           : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = O == 32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                           : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    a = __hiloint2double((int)h[0], (int)l[0]);
    b = __hiloint2double((int)h[1], (int)l[1]);
  } else {
    static_assert(O == 8 || O == 4 || O == 2 || O == 1, "lane distance");
    constexpr int ctrl = O == 8 ? 0x128 : O == 4 ? 0x124 : O == 2 ? 0x4E : 0xB1;
    a = v;
    b = __hiloint2double(__builtin_amdgcn_mov_dpp((int)hi, ctrl, 0xF, 0xF, false),
                         __builtin_amdgcn_mov_dpp((int)lo, ctrl, 0xF, 0xF, false));
  }
}

// wave64 butterfly sum (all lanes active); every lane ends with the same
// value, the order of additions is fixed, so the result is deterministic.
// Twelve dependent ds_bpermute round trips per double were what these sums
// waited on; with the permutations above and bit-equal results: 41 fields of
// 64 cells 36.5 vs 38.9 us per RK4 step, the 768-cell four-mode film 139 vs
// 147 us per DP45 step, 64 spheres 137 vs 139 ms for 162 steps.
template <int O = 32>
__device__ __forceinline__ double wave_sum(double v) {
  double a, b;
  lane_pair<O>(v, a, b);
  v = a + b;
  if constexpr (O > 1) return wave_sum<O / 2>(v);
  else return v;
}

// The wave sums of two values: a's in lanes 0-31, b's in lanes 32-63, each
// with the additions of wave_sum in its order.  After the exchange over 32
// lanes the halves hold the same values, so one chain of steps serves both.
__device__ __forceinline__ double wave_sum2(double u, double v) {
  double a, b, c, d;
  lane_pair<32>(u, a, b);
  lane_pair<32>(v, c, d);
  const double su = a + b, sv = c + d;
  return wave_sum<16>((threadIdx.x & 32) ? sv : su);
}

template <int O = 32>
__device__ __forceinline__ double wave_max(double v) {
  double a, b;
  lane_pair<O>(v, a, b);
  v = nan_max(a, b);
  if constexpr (O > 1) return wave_max<O / 2>(v);
  else return v;
}

// order the wavefront's LDS accesses across lanes (no instruction: a
// wavefront's LDS operations already complete in issue order)
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void cross3(const float* a, const float* b, float* o) {
  o[0] = a[1] * b[2] - a[2] * b[1];
  o[1] = a[2] * b[0] - a[0] * b[2];
  o[2] = a[0] * b[1] - a[1] * b[0];
}

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

}  // namespace mmk
