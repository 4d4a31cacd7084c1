// Persistent schedule of batches (ibp_persist.hpp) without matrix products: the
// mixed forms, and FP64 batches none of whose lines take them.
#include "ibp_persist.hpp"

namespace ibp {

// (lanes, rows per lane) shapes the persistent kernel is built for: the
// line-solve shapes of batches whose tallest grid has at most 512 rows
bool persist_shape_supported(int P, int K) {
  return (P == 32 && (K == 4 || K == 8 || K == 12)) || (P == 64 && K == 8);
}

hipError_t persist_blocks_per_cu_md(bool wide, int P, int K, int* per_cu);
hipError_t launch_persist_md(bool wide, int P, int K, const PersistArgs& a, const BatchPtrs& p, int blocks,
                             hipStream_t s);

template <typename T>
hipError_t persist_blocks_per_cu(bool wide, bool products, int P, int K, int* per_cu) {
  if constexpr (sizeof(T) == 8)
    if (products) return persist_blocks_per_cu_md(wide, P, K, per_cu);
  return persist_occupancy<T, false>(wide, P, K, per_cu);
}

template <typename T>
hipError_t launch_persist(bool wide, bool products, int P, int K, const PersistArgs& a, const BatchPtrs& p, int blocks,
                          hipStream_t s) {
  if constexpr (sizeof(T) == 8)
    if (products) return launch_persist_md(wide, P, K, a, p, blocks, s);
  return persist_launch<T, false>(wide, P, K, a, p, blocks, s);
}

template hipError_t persist_blocks_per_cu<double>(bool, bool, int, int, int*);
template hipError_t persist_blocks_per_cu<float>(bool, bool, int, int, int*);
template hipError_t launch_persist<double>(bool, bool, int, int, const PersistArgs&, const BatchPtrs&, int,
                                           hipStream_t);
template hipError_t launch_persist<float>(bool, bool, int, int, const PersistArgs&, const BatchPtrs&, int,
                                          hipStream_t);

}  // namespace ibp
