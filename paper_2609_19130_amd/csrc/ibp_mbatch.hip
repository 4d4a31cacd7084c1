// Matrix-product transforms (ibp_mdft.hpp) of batches: one launch per stage
// covers every grid whose lengths take them.  A block runs kBatchTiles
// consecutive tiles of one grid, the next tile's loads in flight under the
// current one's products.
#include "ibp_mbatch.hpp"
#include "ibp_xz_kernels.hpp"

namespace ibp {
namespace mdft {

#define IBP_MBATCH __global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3)))

// A block's tiles of its grid g: [first, end)
__device__ __forceinline__ int batch_tiles(const long* start, int count, unsigned tiles_of(const BatchPlan&),
                                           const BatchGrid<double>* D, unsigned* first, unsigned* end) {
  const int g = batch_grid_of(start, count, blockIdx.x);
  const unsigned total = tiles_of(D[g].md);
  *first = (unsigned)((long)blockIdx.x - start[g]) * kBatchTiles;
  *end = *first + kBatchTiles < total ? *first + kBatchTiles : total;
  return g;
}

IBP_MBATCH void kb_mxr2c(const BatchGrid<double>* __restrict__ D, const long* __restrict__ start, BatchPtrs P,
                         int count) {
  extern __shared__ double lds_raw[];
  unsigned first, end;
  const int g = batch_tiles(start, count, [](const BatchPlan& b) { return b.ftiles; }, D, &first, &end);
  batch_r2c(D[g], P.f[g], first, end, reinterpret_cast<Cx<double>*>(lds_raw));
}

IBP_MBATCH void kb_mxc2r(const BatchGrid<double>* __restrict__ D, const long* __restrict__ start, BatchPtrs P,
                         int count) {
  extern __shared__ double lds_raw[];
  unsigned first, end;
  const int g = batch_tiles(start, count, [](const BatchPlan& b) { return b.itiles; }, D, &first, &end);
  batch_c2r(D[g], P.phi[g], first, end, reinterpret_cast<Cx<double>*>(lds_raw));
}

template <bool INV>
IBP_MBATCH void kb_mz(const BatchGrid<double>* __restrict__ D, const long* __restrict__ start, int count) {
  extern __shared__ double lds_raw[];
  unsigned first, end;
  const int g = batch_tiles(start, count, [](const BatchPlan& b) { return b.ztiles; }, D, &first, &end);
  batch_z<INV>(D[g], first, end, reinterpret_cast<Cx<double>*>(lds_raw));
}

hipError_t launch_batch_xr2c(const BatchGrid<double>* d, const long* start, long nblocks, size_t lds,
                             const BatchPtrs& p, int count, hipStream_t s) {
  if (nblocks <= 0) return hipSuccess;
  if (lds > kBatchLds) return hipErrorInvalidValue;
  hipLaunchKernelGGL(kb_mxr2c, dim3((unsigned)nblocks), dim3(kThreads), lds, s, d, start, p, count);
  return hipGetLastError();
}

hipError_t launch_batch_xc2r(const BatchGrid<double>* d, const long* start, long nblocks, size_t lds,
                             const BatchPtrs& p, int count, hipStream_t s) {
  if (nblocks <= 0) return hipSuccess;
  if (lds > kBatchLds) return hipErrorInvalidValue;
  hipLaunchKernelGGL(kb_mxc2r, dim3((unsigned)nblocks), dim3(kThreads), lds, s, d, start, p, count);
  return hipGetLastError();
}

hipError_t launch_batch_z(bool inverse, const BatchGrid<double>* d, const long* start, long nblocks, size_t lds,
                          int count, hipStream_t s) {
  if (nblocks <= 0) return hipSuccess;
  if (lds > kBatchLds) return hipErrorInvalidValue;
  if (inverse)
    hipLaunchKernelGGL(kb_mz<true>, dim3((unsigned)nblocks), dim3(kThreads), lds, s, d, start, count);
  else
    hipLaunchKernelGGL(kb_mz<false>, dim3((unsigned)nblocks), dim3(kThreads), lds, s, d, start, count);
  return hipGetLastError();
}

}  // namespace mdft
}  // namespace ibp
