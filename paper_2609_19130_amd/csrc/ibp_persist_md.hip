// Persistent schedule of FP64 batches with matrix-product lines
// (ibp_persist.hpp).  Kernels of their own: the products' call costs every
// other stage registers (8 grids of 256..384-point lines, none of them on
// products: 10990 us with it, 8160 without).
#include "ibp_persist.hpp"

namespace ibp {

hipError_t persist_blocks_per_cu_md(bool wide, int P, int K, int* per_cu) {
  return persist_occupancy<double, true>(wide, P, K, per_cu);
}

hipError_t launch_persist_md(bool wide, int P, int K, const PersistArgs& a, const BatchPtrs& p, int blocks,
                             hipStream_t s) {
  return persist_launch<double, true>(wide, P, K, a, p, blocks, s);
}

}  // namespace ibp
