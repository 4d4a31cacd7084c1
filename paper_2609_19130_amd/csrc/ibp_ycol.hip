// FP64 wall-normal line solves with the columns held in registers (the
// method and its three recurrences: ibp_ytri_body.hpp).
//
// The staged kernel keeps a block's M columns in LDS: 98 KB at 513..768 and
// 1025..1536 rows, so one block per compute unit, whose loads, recurrences and
// stores come one after another (3.9 and 2.6 TB/s).  Here a wave holds M
// neighbouring columns (lane % M) in 64 / M partitions of K rows (lane / M): a
// lane loads and stores its own rows straight from and to memory, 16 M bytes
// of a plane at a time, nothing of the field passes through LDS, and two or
// three blocks of four waves share a compute unit.  The four waves are stacked
// along y; each recurrence is composed in a wave with shuffles and across the
// waves through a few values a column in LDS.  The first recurrence needs
// only the coefficients and runs while the field's loads are in flight.
// Bound by memory.  Measured, staged -> here, us: 384 x 600 x 400 460 -> 382,
// 1024 x 768 x 1024 3345 -> 2760 (4.7 TB/s), 632 x 1263 x 632 3074 -> 2081
// (with 32-bit indices since 1945, 4.2 TB/s), 500 x 1500 x 400 1553 -> 1167.  Where the staged kernel has two or
// more blocks per compute unit it stays: 61 against 71 us at 256^3, 367
// against 381 at 512 x 384 x 512, 922 against 989 at 501 x 1001 x 501.
#include "ibp_internal.hpp"
#include "ibp_ytri_body.hpp"

namespace ibp {

// Four waves: fewer hold less than a column, more leave waves of the compute
// unit without a block (1024 x 768 x 1024: 6 waves of 16 rows a lane 3633 us,
// 4 waves of 24 rows 2760).  Six registers a row (the value and the pivot's
// reciprocal) and about 50: three waves per SIMD up to 20 rows, two from 24
// (20 rows at two: 2121 us against 2081 at 632 x 1263 x 632).
constexpr int kYcolWaves = 4;
constexpr int ycol_occupancy(int K) { return K > 20 ? 2 : 3; }

template <int M, int K>
__global__ __launch_bounds__(kYcolWaves * kWave) __attribute__((amdgpu_waves_per_eu(ycol_occupancy(K))))
void k_ycol(YArgs<double, double> A, ZeroArgs Z) {
  constexpr int PW = kWave / M, NTAB = (K + M - 1) / M;   // partitions of a wave; table rows per thread
  constexpr int nw = kYcolWaves, nthreads = nw * kWave;
  // the coefficients: (a, c) of row p K + i at p (K + 1) + i (or the (0,0)
  // mode's three values a row)
  constexpr int kRows = nw * PW * K;
  __shared__ Cx<double> tab[nw * PW * (K + 1) > 3 * kRows / 2 ? nw * PW * (K + 1) : 3 * kRows / 2];
  // the waves' composites: [wave][value][column]
  __shared__ double ex1[nw * 4 * M], ex2[nw * 3 * M], ex3[nw * 3 * M];
  const int nzb = zero_blocks(A);
  unsigned lb = blockIdx.x;
  if (lb < (unsigned)nzb) {   // the first blocks: FP64 (0,0) mode
    if (A.zcol)
      zero_mode_column<nthreads>(Z, A.spec, A.ps, reinterpret_cast<double*>(tab));
    else
      zero_mode_part<nthreads>(Z, (int)lb, nzb);
    return;
  }
  lb -= (unsigned)nzb;
  const int ny = A.ny;
  const unsigned nkz = (unsigned)A.Q / (unsigned)A.rs;   // a plane has fewer than 2^31 columns
  // kx group by kx group, all kz of one before the next (the inverse z pass
  // starts on the groups written last); the two halves of a 128-byte line go
  // to blocks lb and lb + 8, which share an XCD
  unsigned grp = lb;
  int h = 0;
  if constexpr (M == 4) {
    const unsigned nlb = (unsigned)A.Q / M, full = nlb / 16 * 16;
    if (lb < full) {
      grp = (lb / 16) * 8 + (lb % 8);
      h = (int)(lb % 16) / 8;
    } else {
      grp = full / 2 + (lb - full) / 2;
      h = (int)((lb - full) % 2);
    }
  }
  const int kz = (int)(grp % nkz), kx0 = (int)(grp / nkz) * 8 + h * M;
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int m = lane % M, pw = lane / M, part = wave * PW + pw, s = part * K, kx = kx0 + m;

  // Loads return in order: the coefficients before the field.
  Cx<double> tl[NTAB];
#pragma unroll
  for (int i = 0; i < NTAB; ++i) {
    // rows past ny: a = 0, c = 1 and a zero right-hand side, whose solution
    // is zero and positive pivots for every shift L >= 0
    const int j = tid + i * nthreads, jc = j < ny ? j : ny - 1;
    tl[i] = Cx<double>{gbl(A.ya)[jc], gbl(A.yc)[jc]};
    if (j >= ny) tl[i] = Cx<double>{0.0, 1.0};
  }
  const bool valid = kx < A.hp;   // row padding is not solved
  const bool zero = A.singular && kx == 0 && kz == 0;
  double L = -(gbl(A.lamx)[valid ? kx : 0] + gbl(A.lamz)[kz]);
  if (!valid || zero) L = 1.0;   // singular (0,0): solved by the (0,0)-mode blocks, zeroed here
  Cx<double> d[K];
  const size_t col = (size_t)kz * A.rs + kx;
  {
    const Cx<double>* p = A.spec + (size_t)(s < ny ? s : ny - 1) * A.ps + col;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      d[i] = gld(gbl(p));
      if (s + i + 1 < ny) p += A.ps;
    }
  }
#pragma unroll
  for (int i = 0; i < NTAB; ++i) {
    const int j = tid + i * nthreads, pp = j / K;
    if (K % M == 0 || pp < nw * PW) tab[pp * (K + 1) + j - pp * K] = tl[i];
  }
  __syncthreads();
  const Cx<double>* const my = tab + part * (K + 1);

  // ---- scan 1: the partition's Moebius map of eps
  double mA = 1.0, mB = 0.0, mC = 0.0, mD = 1.0;
  auto rescale = [&](double n00, double n01, double n10, double n11) {
    const int ex = -exp2_of(n10 + n11);
    mA = scale2(n00, ex);
    mB = scale2(n01, ex);
    mC = scale2(n10, ex);
    mD = scale2(n11, ex);
  };
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const double a = my[i].x, c = my[i].y;
    rescale(a * mA + L * mC, a * mB + L * mD, a * mA + (c + L) * mC, a * mB + (c + L) * mD);
  }
#pragma unroll
  for (int off = 1; off < PW; off <<= 1) {
    const double pA = __shfl_up(mA, off * M), pB = __shfl_up(mB, off * M);
    const double pC = __shfl_up(mC, off * M), pD = __shfl_up(mD, off * M);
    if (pw >= off) rescale(mA * pA + mB * pC, mA * pB + mB * pD, mC * pA + mD * pC, mC * pB + mD * pD);
  }
  if (pw == PW - 1) {
    double* o = ex1 + wave * 4 * M + m;
    o[0] = mA;
    o[M] = mB;
    o[2 * M] = mC;
    o[3 * M] = mD;
  }
  const double eA = __shfl_up(mA, M), eB = __shfl_up(mB, M), eC = __shfl_up(mC, M), eD = __shfl_up(mD, M);
  __syncthreads();
  double e;
  {
    // eps = n / q entering the wave: the earlier waves' maps applied to 1
    // (the value beyond the lower wall does not depend on X_0)
    double n = 1.0, q = 1.0;
    for (int w = 0; w < wave; ++w) {
      const double* o = ex1 + w * 4 * M + m;
      const double n1 = o[0] * n + o[M] * q, q1 = o[2 * M] * n + o[3 * M] * q;
      const int ex = -exp2_of(q1);
      n = scale2(n1, ex);
      q = scale2(q1, ex);
    }
    e = pw == 0 ? n / q : (eA * n + eB * q) / (eC * n + eD * q);
  }
  // ---- pivots, and scan 2's map d'_out = mu d'_in + nu of the partition
  double r[K];
  double mu = 1.0;
  Cx<double> nu{0.0, 0.0};
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const double a = my[i].x, c = my[i].y;
    const double n = L + a * e;
    r[i] = rcp_nr(c + n);
    e = n * r[i];
    const double mi = a * r[i];
    if (s + i >= ny) d[i] = Cx<double>{0.0, 0.0};
    d[i] = cscale(d[i], r[i]);
    mu = mi * mu;
    nu = csub(cscale(nu, mi), d[i]);
  }
#pragma unroll
  for (int off = 1; off < PW; off <<= 1) {
    const double pm = __shfl_up(mu, off * M), px = __shfl_up(nu.x, off * M), py = __shfl_up(nu.y, off * M);
    if (pw >= off) {
      nu = Cx<double>{mu * px + nu.x, mu * py + nu.y};
      mu = mu * pm;
    }
  }
  if (pw == PW - 1) {
    double* o = ex2 + wave * 3 * M + m;
    o[0] = mu;
    o[M] = nu.x;
    o[2 * M] = nu.y;
  }
  const double em = __shfl_up(mu, M), ex = __shfl_up(nu.x, M), ey = __shfl_up(nu.y, M);
  __syncthreads();
  Cx<double> prev{0.0, 0.0};
  for (int w = 0; w < wave; ++w) {
    const double* o = ex2 + w * 3 * M + m;
    prev = Cx<double>{o[0] * prev.x + o[M], o[0] * prev.y + o[2 * M]};
  }
  if (pw > 0) prev = Cx<double>{em * prev.x + ex, em * prev.y + ey};
  // ---- d', and scan 3's map X_first = T X_below + S of the partition
  double T = 1.0;
  Cx<double> S{0.0, 0.0};
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const double a = my[i].x, c = my[i].y;
    d[i] = csub(cscale(prev, a * r[i]), d[i]);
    prev = d[i];
    S = cadd(S, cscale(d[i], T));
    r[i] = c * r[i];
    T = T * r[i];
  }
#pragma unroll
  for (int off = 1; off < PW; off <<= 1) {
    const double nT = __shfl_down(T, off * M), sx = __shfl_down(S.x, off * M), sy = __shfl_down(S.y, off * M);
    if (pw + off < PW) {
      S = Cx<double>{T * sx + S.x, T * sy + S.y};
      T = T * nT;
    }
  }
  if (pw == 0) {
    double* o = ex3 + wave * 3 * M + m;
    o[0] = T;
    o[M] = S.x;
    o[2 * M] = S.y;
  }
  const double xT = __shfl_down(T, M), xx = __shfl_down(S.x, M), xy = __shfl_down(S.y, M);
  __syncthreads();
  Cx<double> nxt{0.0, 0.0};
  for (int w = nw - 1; w > wave; --w) {
    const double* o = ex3 + w * 3 * M + m;
    nxt = Cx<double>{o[0] * nxt.x + o[M], o[0] * nxt.y + o[2 * M]};
  }
  if (pw < PW - 1) nxt = Cx<double>{xT * nxt.x + xx, xT * nxt.y + xy};
  if (zero) {
    nxt = Cx<double>{0.0, 0.0};
#pragma unroll
    for (int i = 0; i < K; ++i) d[i] = Cx<double>{0.0, 0.0};
  }
#pragma unroll
  for (int i = K - 1; i >= 0; --i) {
    d[i] = cadd(d[i], cscale(nxt, r[i]));
    nxt = d[i];
  }
  if (!valid || (zero && A.zcol)) return;
  Cx<double>* p = A.spec + (size_t)s * A.ps + col;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    if (s + i < ny) gst(gbl(p), d[i]);
    p += A.ps;
  }
}

template <int M, int K>
static hipError_t launch_ycol_mk(const YArgs<double, double>& a, const ZeroArgs& z, hipStream_t s) {
  if (kYcolWaves * (kWave / M) * K < a.ny || a.rs % 8 != 0 || a.Q % a.rs != 0) return hipErrorInvalidValue;
  const long nb = a.Q / M + zero_blocks(a);   // + the (0,0)-mode blocks
  hipLaunchKernelGGL((k_ycol<M, K>), dim3((unsigned)nb), dim3(kYcolWaves * kWave), 0, s, a, z);
  return hipGetLastError();
}

// Rows for which the staged kernel has one block per compute unit.
bool ycol_rows(int ny) { return (ny > 512 && ny <= 768) || (ny > 1024 && ny <= 1536); }

// Whole 128-byte lines while four waves hold the rows, half lines above.
hipError_t launch_ycol(const YArgs<double, double>& a, const ZeroArgs& z, hipStream_t s) {
  if (a.ny <= 640) return launch_ycol_mk<8, 20>(a, z, s);
  if (a.ny <= 768) return launch_ycol_mk<8, 24>(a, z, s);
  if (a.ny <= 1280) return launch_ycol_mk<4, 20>(a, z, s);
  return launch_ycol_mk<4, 24>(a, z, s);
}

}  // namespace ibp
