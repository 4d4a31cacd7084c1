// Tiles [first, end) of one grid of a batch through the matrix-product
// transforms, S chosen at run time (S <= 8, 256 threads); shared by the staged
// batch kernels and the persistent one.
#pragma once

#include "ibp_mdft.hpp"

namespace ibp {
namespace mdft {

#define IBP_MD_SWITCH(S_, CALL)                    \
  switch (S_) {                                    \
    case 1: { constexpr int S = 1; CALL; } break;  \
    case 2: { constexpr int S = 2; CALL; } break;  \
    case 3: { constexpr int S = 3; CALL; } break;  \
    case 4: { constexpr int S = 4; CALL; } break;  \
    case 5: { constexpr int S = 5; CALL; } break;  \
    case 6: { constexpr int S = 6; CALL; } break;  \
    case 7: { constexpr int S = 7; CALL; } break;  \
    case 8: { constexpr int S = 8; CALL; } break;  \
    default: break;                                \
  }

__device__ __forceinline__ void batch_r2c(const BatchGrid<double>& G, const double* f, unsigned first, unsigned end,
                                          Cx<double>* lds) {
  XArgs<double> a = G.x;
  a.f = f;
  const XExtra e = G.md.f;
  IBP_MD_SWITCH(e.M.S, (xr2c_tiles<XM_PLAIN, S>(a, e, e.M, first, 1u, end, kThreads, lds)))
}

__device__ __forceinline__ void batch_c2r(const BatchGrid<double>& G, double* phi, unsigned first, unsigned end,
                                          Cx<double>* lds) {
  XArgs<double> a = G.x;
  a.out = phi;
  const XExtra e = G.md.i;
  // the tiles count down from the last: tile t of the grid is t of itiles, so
  // [first, end) keeps that order
  IBP_MD_SWITCH(e.M.S, (xc2r_tiles<CM_SET, S>(a, e, e.M, first, 1u, 0u, G.md.itiles, end, kThreads, lds)))
}

template <bool INV>
__device__ __forceinline__ void batch_z(const BatchGrid<double>& G, unsigned first, unsigned end, Cx<double>* lds) {
  const ZArgs a = G.md.z;
  const ZTiles Z{(unsigned)G.y.ny, G.md.zgroups, 1u};
  if (a.lc == 4)
    IBP_MD_SWITCH(a.M.S, (z_tiles<INV, S, 4>(a, a.M, Z, first, 1u, end, kThreads, lds)))
  else
    IBP_MD_SWITCH(a.M.S, (z_tiles<INV, S, 3>(a, a.M, Z, first, 1u, end, kThreads, lds)))
}

}  // namespace mdft
}  // namespace ibp
