// Kernels and launchers of the matrix-product transforms (ibp_mdft.hpp) for
// single grids: FP64 z lines, x R2C (right-hand side given or assembled) and
// x C2R (set or add).
#include <algorithm>
#include <type_traits>

#include "ibp_mdft.hpp"

namespace ibp {
namespace mdft {

template <bool INV, int S, int LC>
__global__ __launch_bounds__(max_threads(S)) void k_mz(ZArgs A, ZTiles Z) {
  extern __shared__ double lds_raw[];
  if (A.check_done && A.ctl->done) return;
  z_tiles<INV, S, LC>(A, A.M, Z, blockIdx.x, gridDim.x, Z.total(), blockDim.x,
                      reinterpret_cast<Cx<double>*>(lds_raw));
}

template <int MODE, int S>
__global__ __launch_bounds__(max_threads(S)) void k_mxr2c(XArgs<double> A, XExtra E, unsigned base, unsigned end) {
  extern __shared__ double lds_raw[];
  xr2c_tiles<MODE, S>(A, E, E.M, base + blockIdx.x, gridDim.x, end, blockDim.x,
                      reinterpret_cast<Cx<double>*>(lds_raw));
}

template <int MODE, int S>
__global__ __launch_bounds__(max_threads(S)) void k_mxc2r(XArgs<double> A, XExtra E, unsigned base, unsigned total) {
  extern __shared__ double lds_raw[];
  if (MODE == CM_ADD && A.ctl->done) return;
  xc2r_tiles<MODE, S>(A, E, E.M, blockIdx.x, gridDim.x, base, total, total, blockDim.x,
                      reinterpret_cast<Cx<double>*>(lds_raw));
}

template <typename F>
hipError_t dispatch(int S, F&& f) {
  switch (S) {
#define IBP_CASE(s) \
  case s: return f(std::integral_constant<int, s>{});
    IBP_CASE(1) IBP_CASE(2) IBP_CASE(3) IBP_CASE(4) IBP_CASE(5) IBP_CASE(6) IBP_CASE(7) IBP_CASE(8)
    IBP_CASE(9) IBP_CASE(10) IBP_CASE(11) IBP_CASE(12) IBP_CASE(13) IBP_CASE(14) IBP_CASE(15) IBP_CASE(16)
#undef IBP_CASE
    default: return hipErrorInvalidValue;
  }
}

size_t lds_z(const Plan& M, int RS) { return ((size_t)(M.P + 1) * RS + M.P) * sizeof(Cx<double>); }
size_t lds_r2c(const Plan& M, int RS) { return lds_z(M, RS); }
size_t lds_c2r(const Plan& M, int RS, int RP) {
  return ((size_t)(M.P / 2 + 2) * RS + M.P + (RP + 1) / 2) * sizeof(Cx<double>);
}

// Threads for `tasks` tasks and `items` 16-column products of a tile of `lds`
// bytes: enough for the tasks, one a thread up to half the threads a block may
// have, and at least the block's share of the waves that a compute unit holds
// at the kernel's registers (the products spread over all of a block's waves).
// The share is among the blocks that LDS admits (`cu` threads in all); where a
// compute unit gets fewer tiles it is larger, up to a wave per product (us:
// R2C of 256 rows of 640 points 13.8 -> 9.6, of 1536 points 21.1 -> 15.3, 1024
// rows of 1000 points 23.3 -> 17.5).  Whole rounds of the four SIMDs (or 1 or
// 2 waves): blocks of 3 or 6 waves leave wave slots that the next block's
// waves do not fill (501 x 300 x 501, C2R: 2 x 6 waves 2.1 TB/s, 1 x 12 waves
// 2.8).
int block_threads(int S, int tasks, int items, size_t lds, long tiles_per_cu, int cu) {
  const int per = tasks_per_thread(S), most = max_threads(S);
  const int least = (tasks + per - 1) / per, blocks = (int)(kMaxLds / lds);
  int nt = tasks < most / 2 ? tasks : least > most / 2 ? least : most / 2;
  int share = blocks > 0 ? cu / blocks / kWave * kWave : 0;
  if (tiles_per_cu < blocks) {
    const int all = cu / (int)std::max(tiles_per_cu, 1L) / kWave * kWave;
    share = std::max(share, std::min(all, items * kWave));
  }
  share = std::min(share, most);
  if (nt < share) nt = share;
  if (nt <= kWave) return kWave;
  return nt <= 2 * kWave ? 2 * kWave : (nt + 4 * kWave - 1) / (4 * kWave) * (4 * kWave);
}
// Blocks of that shape that a compute unit holds.
int blocks_per_cu(int threads, size_t lds, int cu) {
  const int by_lds = (int)(kMaxLds / lds), by_waves = cu / threads;
  return by_lds < by_waves ? by_lds : by_waves;
}

static long tiles_per_cu(unsigned tiles, int cus) { return ((long)tiles + cus - 1) / cus; }
static int products_of(const Plan& M, int columns) { return M.MT * ((columns + 15) / 16); }

// The shape holds: every task has a thread, within the block's limits.
static bool shape_ok(int S, int tasks, int threads, size_t lds) {
  return threads <= max_threads(S) && tasks <= threads * tasks_per_thread(S) && lds <= kMaxLds;
}

// Blocks of a launch over `total` tiles: as many as the compute units hold, a
// multiple of 64 so that a block's tiles stay on the XCD that their order
// assumes.
static unsigned blocks_for(unsigned total, int threads, size_t lds, int cu, int cus) {
  const unsigned want = (unsigned)(cus * blocks_per_cu(threads, lds, cu)) / 64 * 64;
  return want == 0 || total < want ? total : want;
}

hipError_t launch_z(bool inverse, const ZArgs& a, int nplanes, hipStream_t s) {
  const size_t lds = lds_z(a.M, a.RS);
  const int C = 1 << a.lc;
  const unsigned sib = C >= 8 ? 1 : 8 / C;
  const unsigned groups = ((a.hp + C - 1) / C + sib - 1) / sib * sib;
  const ZTiles Z{(unsigned)nplanes, groups, sib};
  const int nt = block_threads(a.M.S, a.M.P << a.lc, products_of(a.M, a.M.S << a.lc), lds,
                               tiles_per_cu(Z.planes * Z.groups, a.cus), max_threads(a.M.S));
  if (a.M.S * a.M.P != a.nz || a.RS < C * a.M.S || a.lc < 2 || a.lc > 4 ||
      !shape_ok(a.M.S, a.M.P << a.lc, nt, lds))
    return hipErrorInvalidValue;
  const dim3 grid(blocks_for(Z.planes * Z.groups, nt, lds, max_threads(a.M.S), a.cus));
  return dispatch(a.M.S, [&](auto s_) {
    constexpr int S = decltype(s_)::value;
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, grid, dim3(nt), lds, s, a, Z);
      return hipGetLastError();
    };
    if constexpr (S % 2 == 1)
      if (a.lc == 4) return inverse ? go(k_mz<true, S, 4>) : go(k_mz<false, S, 4>);
    if (a.lc == 3) return inverse ? go(k_mz<true, S, 3>) : go(k_mz<false, S, 3>);
    if (a.lc == 2) return inverse ? go(k_mz<true, S, 2>) : go(k_mz<false, S, 2>);
    return hipErrorInvalidValue;
  });
}

hipError_t launch_xr2c(int mode, const XArgs<double>& a, const XExtra& e, hipStream_t s) {
  const size_t lds = lds_r2c(e.M, e.RS);
  const int cu = cu_threads(e.M.S, mode == XM_DIV);
  const unsigned base = (unsigned)(a.row_begin / (2 * e.RP)), end = (unsigned)((a.nrows + 2 * e.RP - 1) / (2 * e.RP));
  const int nt = block_threads(e.M.S, e.RP * e.M.P, products_of(e.M, e.RP * (1 + 2 * (e.M.S / 2))), lds,
                               tiles_per_cu(end - base, e.cus), cu);
  if (e.M.S * e.M.P != a.nx || e.RS < e.RP * (1 + 2 * (e.M.S / 2)) ||
      !shape_ok(e.M.S, e.RP * e.M.P, nt, lds))
    return hipErrorInvalidValue;
  const dim3 grid(blocks_for(end - base, nt, lds, cu, e.cus));
  return dispatch(e.M.S, [&](auto s_) {
    constexpr int S = decltype(s_)::value;
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, grid, dim3(nt), lds, s, a, e, base, end);
      return hipGetLastError();
    };
    if (mode == XM_DIV) return go(k_mxr2c<XM_DIV, S>);
    if (mode == XM_PLAIN) return go(k_mxr2c<XM_PLAIN, S>);
    return hipErrorInvalidValue;
  });
}

hipError_t launch_xc2r(int mode, const XArgs<double>& a, const XExtra& e, hipStream_t s) {
  const size_t lds = lds_c2r(e.M, e.RS, e.RP);
  const unsigned base = (unsigned)(a.row_begin / e.RP), total = (unsigned)((a.nrows + e.RP - 1) / e.RP) - base;
  const int nt = block_threads(e.M.S, e.RP * (e.M.P / 2 + 1), products_of(e.M, e.RP * e.M.S), lds,
                               tiles_per_cu(total, e.cus), max_threads(e.M.S));
  if (e.M.S * e.M.P != a.nx || e.RS < e.RP * e.M.S ||
      !shape_ok(e.M.S, e.RP * (e.M.P / 2 + 1), nt, lds))
    return hipErrorInvalidValue;
  const dim3 grid(blocks_for(total, nt, lds, max_threads(e.M.S), e.cus));
  return dispatch(e.M.S, [&](auto s_) {
    constexpr int S = decltype(s_)::value;
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, grid, dim3(nt), lds, s, a, e, base, total);
      return hipGetLastError();
    };
    return mode == CM_ADD ? go(k_mxc2r<CM_ADD, S>) : go(k_mxc2r<CM_SET, S>);
  });
}

}  // namespace mdft
}  // namespace ibp
