// What the whole-step kernels of small instances share (kernels_small.hip,
// kernels_small_adj.hip).
#pragma once
#include "mm_internal.h"
#include "kernels_common.h"

namespace mmk {

// The members of InstDesc that the field and the torque of a cell use.
template <int NS>
struct CellDesc {
  static constexpr int S = NS;
  int ncell, demag;
  float cex_x, cex_y, cex_z, cK, ex, ey, ez, B0x, B0y, B0z, nlx, nly, nlz, BE, gl, alpha;
  float csign[2];
  float* bd;
  __device__ __forceinline__ explicit CellDesc(const InstDesc& D)
      : ncell(D.ncell), demag(D.demag), cex_x(D.cex_x), cex_y(D.cex_y), cex_z(D.cex_z), cK(D.cK), ex(D.ex),
        ey(D.ey), ez(D.ez), B0x(D.B0x), B0y(D.B0y), B0z(D.B0z), nlx(D.nlx), nly(D.nly), nlz(D.nlz), BE(D.BE), gl(D.gl),
        alpha(D.alpha), csign{D.csign[0], D.csign[1]}, bd(nullptr) {}
};

}  // namespace mmk
