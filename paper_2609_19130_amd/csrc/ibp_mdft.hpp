// Transforms of any line length n = S P as two steps with one LDS exchange:
// an S-point DFT held in a thread's registers (S <= 16) and P-point DFTs as
// matrix products on the FP64 matrix cores (v_mfma_f64_16x16x4).
//
// Complex lines (z): with index i = j + P r in and k + S q out (j, q < P;
// r, k < S), a thread loads x[j + P r] for all r straight from memory, takes
// the S-point DFT over r, multiplies output k by W_n^{j k} and stores it to
// LDS; the P-point DFT over j of each k then yields X[k + S q], stored to
// memory from the accumulators.  The P-point matrix is used through its
// symmetry: with s_r = x_r + x_{P-r} and d_r = x_r - x_{P-r} (0 < r < P/2; x_0
// and, for even P, x_{P/2} stand alone),
//   A_q = sum_r s_r cos(2 pi q r / P),  B_q = sum_r d_r sin(2 pi q r / P),
//   y_q = A_q - i B_q,  y_{P-q} = A_q + i B_q,   q <= P/2,
// so a real product of (P/2 + 1)^2 entries serves cosine and sine each: padded to
// the steps below, n = 320 = 16 x 20 takes 102 flops a value in the products,
// 632 = 8 x 79 takes 194 and 501 = 3 x 167 takes 405, against 480 in the time
// that a large copy needs for the value's 32 bytes.  The matrix is never stored: a lane steps through
// W_P^{q r} in a table of its P roots (LDS).
//
// Real rows: R2C takes two rows a, b as one complex value through the S-point
// DFT, separates their spectra in registers and keeps k <= S/2 of each (the
// rest are conjugates); the k = 0 values are real again and share one
// complex column.  C2R starts from j <= P/2 only: the P-point DFTs over j
// are Hermitian, x[m + S q] = sum_j 2 (Re b_j cos - Im b_j sin), the terms of
// j = 0 and P/2 halved.
//
// Data columns (line, k) fill the 16-column side of the products, q the
// 16-row side, r the depth in steps of 4.
#pragma once

#include "ibp_internal.hpp"

namespace ibp {
namespace mdft {

// ---------------------------------------------------------------- S-point DFTs
// cos and sin of 2 pi k / N (quarter turns exact)
template <int N>
struct Root;
#define IBP_LIST(...) {__VA_ARGS__}
#define IBP_ROOTS(N, C, S)                              \
  template <>                                           \
  struct Root<N> {                                      \
    __device__ static constexpr double c(int k) {       \
      constexpr double t[N] = C;                        \
      return t[k];                                      \
    }                                                   \
    __device__ static constexpr double s(int k) {       \
      constexpr double t[N] = S;                        \
      return t[k];                                      \
    }                                                   \
  };
IBP_ROOTS(6, IBP_LIST(1.0, 0.5, -0.5, -1.0, -0.5, 0.5),
          IBP_LIST(0.0, 0.8660254037844386, 0.8660254037844386, 0.0, -0.8660254037844386, -0.8660254037844386))
IBP_ROOTS(9, IBP_LIST(1.0, 0.766044443118978, 0.17364817766693036, -0.5, -0.9396926207859084, -0.9396926207859084,
          -0.5, 0.17364817766693036, 0.766044443118978),
          IBP_LIST(0.0, 0.6427876096865394, 0.984807753012208, 0.8660254037844386, 0.3420201433256687,
          -0.3420201433256687, -0.8660254037844386, -0.984807753012208, -0.6427876096865394))
IBP_ROOTS(10, IBP_LIST(1.0, 0.8090169943749475, 0.30901699437494745, -0.30901699437494745, -0.8090169943749475,
          -1.0, -0.8090169943749475, -0.30901699437494745, 0.30901699437494745, 0.8090169943749475),
          IBP_LIST(0.0, 0.5877852522924731, 0.9510565162951535, 0.9510565162951535, 0.5877852522924731, 0.0,
          -0.5877852522924731, -0.9510565162951535, -0.9510565162951535, -0.5877852522924731))
IBP_ROOTS(12, IBP_LIST(1.0, 0.8660254037844386, 0.5, 0.0, -0.5, -0.8660254037844386, -1.0, -0.8660254037844386,
          -0.5, 0.0, 0.5, 0.8660254037844386),
          IBP_LIST(0.0, 0.5, 0.8660254037844386, 1.0, 0.8660254037844386, 0.5, 0.0, -0.5, -0.8660254037844386, -1.0,
          -0.8660254037844386, -0.5))
IBP_ROOTS(14, IBP_LIST(1.0, 0.9009688679024191, 0.6234898018587335, 0.2225209339563144, -0.2225209339563144,
          -0.6234898018587335, -0.9009688679024191, -1.0, -0.9009688679024191, -0.6234898018587335,
          -0.2225209339563144, 0.2225209339563144, 0.6234898018587335, 0.9009688679024191),
          IBP_LIST(0.0, 0.4338837391175581, 0.7818314824680298, 0.9749279121818236, 0.9749279121818236,
          0.7818314824680298, 0.4338837391175581, 0.0, -0.4338837391175581, -0.7818314824680298,
          -0.9749279121818236, -0.9749279121818236, -0.7818314824680298, -0.4338837391175581))
IBP_ROOTS(15, IBP_LIST(1.0, 0.9135454576426009, 0.6691306063588582, 0.30901699437494745, -0.10452846326765347, -0.5,
          -0.8090169943749475, -0.9781476007338057, -0.9781476007338057, -0.8090169943749475, -0.5,
          -0.10452846326765347, 0.30901699437494745, 0.6691306063588582, 0.9135454576426009),
          IBP_LIST(0.0, 0.4067366430758002, 0.7431448254773942, 0.9510565162951535, 0.9945218953682733,
          0.8660254037844386, 0.5877852522924731, 0.20791169081775934, -0.20791169081775934, -0.5877852522924731,
          -0.8660254037844386, -0.9945218953682733, -0.9510565162951535, -0.7431448254773942, -0.4067366430758002))
IBP_ROOTS(16, IBP_LIST(1.0, 0.9238795325112867, 0.7071067811865476, 0.3826834323650898, 0.0, -0.3826834323650898,
          -0.7071067811865476, -0.9238795325112867, -1.0, -0.9238795325112867, -0.7071067811865476,
          -0.3826834323650898, 0.0, 0.3826834323650898, 0.7071067811865476, 0.9238795325112867),
          IBP_LIST(0.0, 0.3826834323650898, 0.7071067811865476, 0.9238795325112867, 1.0, 0.9238795325112867,
          0.7071067811865476, 0.3826834323650898, 0.0, -0.3826834323650898, -0.7071067811865476,
          -0.9238795325112867, -1.0, -0.9238795325112867, -0.7071067811865476, -0.3826834323650898))
#undef IBP_ROOTS
#undef IBP_LIST

// v <- DFT of v (natural order in and out), unnormalised
template <int S, bool INV, typename T>
struct Dft {
  __device__ __forceinline__ static void run(Cx<T>* v) { Bfly<S, INV, T>::run(v); }
};
template <bool INV, typename T>
struct Dft<1, INV, T> {
  __device__ __forceinline__ static void run(Cx<T>*) {}
};
// S = A B: A-point DFTs over the stride-B subsequences, twiddles W_S^{n2 k1},
// then B-point DFTs
template <int A, int B, bool INV, typename T>
struct DftAB {
  __device__ __forceinline__ static void run(Cx<T>* v) {
    constexpr int S = A * B;
    Cx<T> u[B][A];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
#pragma unroll
      for (int n1 = 0; n1 < A; ++n1) u[n2][n1] = v[B * n1 + n2];
      Bfly<A, INV, T>::run(u[n2]);
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
      Cx<T> w[B];
#pragma unroll
      for (int n2 = 0; n2 < B; ++n2) {
        const int e = (n2 * k1) % S;
        if (e == 0)
          w[n2] = u[n2][k1];
        else if (4 * e == S)
          w[n2] = mul_mi<INV>(u[n2][k1]);
        else
          w[n2] = cmul(u[n2][k1], Cx<T>{T(Root<S>::c(e)), INV ? T(Root<S>::s(e)) : T(-Root<S>::s(e))});
      }
      Bfly<B, INV, T>::run(w);
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) v[k1 + A * k2] = w[k2];
    }
  }
};
template <bool INV, typename T> struct Dft<6, INV, T> : DftAB<2, 3, INV, T> {};
template <bool INV, typename T> struct Dft<9, INV, T> : DftAB<3, 3, INV, T> {};
template <bool INV, typename T> struct Dft<10, INV, T> : DftAB<2, 5, INV, T> {};
template <bool INV, typename T> struct Dft<12, INV, T> : DftAB<4, 3, INV, T> {};
template <bool INV, typename T> struct Dft<14, INV, T> : DftAB<2, 7, INV, T> {};
template <bool INV, typename T> struct Dft<15, INV, T> : DftAB<3, 5, INV, T> {};
template <bool INV, typename T> struct Dft<16, INV, T> : DftAB<4, 4, INV, T> {};

// Twiddle factors W^{j k}, k = 1 .. S-1, of one task, kept in registers over
// its tiles: up to 4 are all read from the table; longer sets hold W^{b j}
// (b < 4) and W^{4 a j} and form the rest as one rounded product each, which
// adds 2 to 4 % to a transform's error at S > 4 (emulated in double).
template <int S, bool INV>
struct Twiddle {
  static constexpr int NL = S < 4 ? S : 4, NH = S <= 4 ? 1 : (S + 3) / 4;
  Cx<double> lo[NL], hi[NH];
  __device__ __forceinline__ void load(int j, const Cx<double>* __restrict__ tw) {
    auto get = [&](int e) {
      Cx<double> w = tw[e];
      if (INV) w.y = -w.y;
      return w;
    };
#pragma unroll
    for (int b = 1; b < NL; ++b) lo[b] = get(j * b);
#pragma unroll
    for (int a = 1; a < NH; ++a) hi[a] = get(j * 4 * a);
  }
  __device__ __forceinline__ Cx<double> get(int k) const {
    if (k < 4) return lo[k];
    return k % 4 ? cmul(hi[k / 4], lo[k % 4]) : hi[k / 4];
  }
  __device__ __forceinline__ void apply(Cx<double> (&v)[S]) const {
#pragma unroll
    for (int k = 1; k < S; ++k) v[k] = cmul(v[k], get(k));
  }
};

// Accesses at a block-uniform base and a 32-bit byte offset of the lane: one
// address register for all the accesses of a task.
__device__ __forceinline__ Cx<double> at(const char* base, unsigned off) {
  return *reinterpret_cast<const Cx<double>*>(base + off);
}
__device__ __forceinline__ double at_d(const char* base, unsigned off) {
  return *reinterpret_cast<const double*>(base + off);
}
__device__ __forceinline__ void put(char* base, unsigned off, Cx<double> v) {
  *reinterpret_cast<Cx<double>*>(base + off) = v;
}

// ---------------------------------------------------------------- matrix products
typedef double acc4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ acc4 mma(double a, double b, acc4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// Keeps the loads before it ahead of the products after it (the compiler
// otherwise moves them next to their use, a full LDS latency per step).
__device__ __forceinline__ void keep_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// A operand: row lane % 16, depth lane / 16; B: column lane % 16, depth
// lane / 16; result v: row 4 v + lane / 16, column lane % 16.
__device__ __forceinline__ int acc_row(int lane, int v) { return 4 * v + lane / 16; }

// The P roots (cos, -sin)(2 pi e / P) into LDS: W_n^{S e} of the line's table.
__device__ __forceinline__ void load_roots(const Plan& M, const Cx<double>* __restrict__ tw, Cx<double>* roots,
                                           int nthreads) {
  for (int e = threadIdx.x; e < M.P; e += nthreads) roots[e] = tw[M.S * e];
}

// A lane's walk through W_P^{q r}, r = lk, lk + 4, ... (q = its matrix row,
// rows past P/2 repeat the last: their results are dropped).
struct Walk {
  unsigned e, step, P;
  const Cx<double>* roots;
  __device__ __forceinline__ Walk(const Plan& M, const Cx<double>* t, int q, int lk) : P(M.P), roots(t) {
    const unsigned qq = q <= M.P / 2 ? q : M.P / 2;
    e = 0;
    for (int i = 0; i < 3; ++i)
      if (i < lk) e = wrap(e + qq);
    step = wrap(wrap(2 * qq) * 2);
  }
  // values below 2 P, modulo P
  __device__ __forceinline__ unsigned wrap(unsigned v) const { return v < v - P ? v : v - P; }
  __device__ __forceinline__ Cx<double> next() {
    const Cx<double> w = roots[e];
    e = wrap(e + step);
    return w;
  }
};

// Products of the 16-row step mt and the column tile nt: A_q and -B_q of the
// real and imaginary parts.  LDS row r of NC columns sits at r RS; row P is
// zero.  Two operand sets in turn: the next step's are read during a step's
// products (KT is even).
struct Acc {
  acc4 cr, ci, sr, si;
};
__device__ __forceinline__ Acc products(const Plan& M, const Cx<double>* roots, const Cx<double>* lds, int RS, int NC,
                                        int mt, int nt, int lane) {
  Acc acc;
  acc.cr = acc.ci = acc.sr = acc.si = acc4{0.0, 0.0, 0.0, 0.0};
  const int lk = lane / 16, c = nt * 16 + lane % 16, P = M.P;
  const Cx<double>* const base = lds + (c < NC ? c : NC - 1);
  Walk w(M, roots, mt * 16 + lane % 16, lk);
  auto rows = [&](int kt, Cx<double>* x, Cx<double>* y) {
    const int r = 4 * kt + lk;
    *x = base[__mul24(2 * r <= P ? r : P, RS)];
    *y = base[__mul24(r > 0 && 2 * r < P ? P - r : P, RS)];
  };
  auto step = [&](Cx<double> a, Cx<double> x, Cx<double> y) {
    acc.cr = mma(a.x, x.x + y.x, acc.cr);
    acc.ci = mma(a.x, x.y + y.y, acc.ci);
    acc.sr = mma(a.y, x.x - y.x, acc.sr);
    acc.si = mma(a.y, x.y - y.y, acc.si);
  };
  Cx<double> a0 = w.next(), x0, y0;
  rows(0, &x0, &y0);
  for (int kt = 0; kt < M.KT; kt += 2) {
    const Cx<double> a1 = w.next();
    Cx<double> x1, y1;
    rows(kt + 1, &x1, &y1);
    keep_order();
    step(a0, x0, y0);
    a0 = w.next();
    rows(kt + 2, &x0, &y0);
    keep_order();
    step(a1, x1, y1);
  }
  return acc;
}

// A block of each transform takes tiles first, first + stride, ... below
// total.  Thread t owns the S-point tasks t, t + nthreads, ... of a tile (at
// most tasks_per_thread(S) of them), and the next tile's loads are in flight
// while the products of the current one run and its results are stored (but
// for the assembled right-hand side).  Nothing else is loaded from memory
// inside the loop (loads return in order, so waiting for a later one would
// wait for the next tile's).

// ---------------------------------------------------------------- z lines
// Column group and plane of a z tile.  Groups narrower than a 128-byte line
// come in sets of `sib` that share the line; a set's members are 8 tiles
// apart, which the round-robin dispatch places on one XCD at about the same
// time, so the line enters that XCD's L2 once (as in the register Bluestein z
// passes).  Plane by plane, forward in descending order.
struct ZTiles {
  unsigned planes, groups, sib;
  __device__ __forceinline__ unsigned total() const { return planes * groups; }
  template <bool INV>
  __device__ __forceinline__ void get(unsigned b, int* pl, int* grp) const {
    unsigned set = b, h = 0;
    if (sib > 1) {
      const unsigned full = total() / (8 * sib) * (8 * sib);
      if (b < full) {
        set = (b / (8 * sib)) * 8 + b % 8;
        h = (b % (8 * sib)) / 8;
      } else {
        set = full / sib + (b - full) / sib;
        h = (b - full) % sib;
      }
    }
    const unsigned gs = groups / sib, q = set / gs;
    *pl = (int)(INV ? q : planes - 1 - q);
    *grp = (int)((set - q * gs) * sib + h);
  }
};

// lds: (P + 1) RS values, then the P roots.  Tiles of 2^LC kx columns.
template <bool INV, int S, int LC>
__device__ __forceinline__ void z_tiles(const ZArgs& A, const Plan& M, const ZTiles& Z, unsigned first,
                                        unsigned stride, unsigned total, int nthreads, Cx<double>* lds) {
  constexpr int C = 1 << LC, NC = S << LC, ntile = (NC + 15) / 16, NT = tasks_per_thread(S);
  const int tid = threadIdx.x, P = M.P, RS = A.RS, H = P / 2;
  const unsigned rsb = (unsigned)A.rs * sizeof(Cx<double>);   // a plane's offsets stay below 2^32
  const int c = tid & (C - 1);   // nthreads is a multiple of C: every task of a thread has this column
  const int j0 = tid >> LC, js = nthreads >> LC;
  Cx<double>* const roots = lds + (size_t)(P + 1) * RS;
  load_roots(M, A.tw, roots, nthreads);
  for (int i = tid; i < NC; i += nthreads) lds[__mul24(P, RS) + i] = Cx<double>{0.0, 0.0};
  Twiddle<S, INV> w[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
    if (j0 + i * js < P) w[i].load(j0 + i * js, A.tw);
  const int lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), nw = nthreads / kWave;
  const int items = M.MT * ntile;
  Cx<double> v[NT][S];
  // every task loads: one without a row of its own reads row P - 1's, and
  // columns past hp read the row's padding or the next row (a plane ends with
  // as much padding as the widest group overhangs); neither is stored
  auto load = [&](const char* plane) {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int j = j0 + i * js < P ? j0 + i * js : P - 1;
      const unsigned off = (unsigned)j * rsb + (unsigned)c * sizeof(Cx<double>);
#pragma unroll
      for (int r = 0; r < S; ++r) v[i][r] = at(plane + (size_t)(P * r) * rsb, off);
    }
  };
  auto place = [&](unsigned b, int* col0) {
    int pl, grp;
    Z.get<INV>(b, &pl, &grp);
    pl = __builtin_amdgcn_readfirstlane(pl);
    *col0 = __builtin_amdgcn_readfirstlane(grp) << LC;
    return reinterpret_cast<char*>(A.spec + (size_t)(A.plane0 + pl) * A.ps + *col0);
  };
  unsigned b = first;
  int col0 = 0, rot = 0;
  char* plane = nullptr;
  if (b < total) {
    plane = place(b, &col0);
    load(plane);
  }
  for (; b < total; b += stride) {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      if (j0 + i * js < P) {
        Dft<S, INV, double>::run(v[i]);
        w[i].apply(v[i]);
        Cx<double>* o = lds + __mul24(j0 + i * js, RS) + c;
#pragma unroll
        for (int k = 0; k < S; ++k) o[k * C] = v[i][k];
      }
    }
    __syncthreads();
    char* const out = plane;
    const int oc0 = col0;
    if (b + stride < total) {
      plane = place(b + stride, &col0);
      load(plane);
    }
    // the first wave moves on with every tile: items left over past whole
    // rounds of the waves go to other waves each time
    int it = wave + rot < nw ? wave + rot : wave + rot - nw;
    rot = rot + 1 < nw ? rot + 1 : 0;
    for (; it < items; it += nw) {
      const int mt = it / ntile, nt = it - mt * ntile;
      const Acc a = products(M, roots, lds, RS, NC, mt, nt, lane);
      const int col = nt * 16 + lane % 16, k = col >> LC, cc = col & (C - 1), lk = lane / 16;
      if (col >= NC || oc0 + cc >= A.hp) continue;
      // row q = 16 mt + 4 i + lk goes to k + S q and k + S (P - q)
      const unsigned up = (unsigned)(k + S * lk) * rsb + (unsigned)cc * sizeof(Cx<double>);
      const unsigned down = (unsigned)(k + S * (3 - lk)) * rsb + (unsigned)cc * sizeof(Cx<double>);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int q0 = mt * 16 + 4 * i, q = q0 + lk;
        if (q > H) continue;
        const Cx<double> y1{a.cr[i] - a.si[i], a.ci[i] + a.sr[i]};
        const Cx<double> y2{a.cr[i] + a.si[i], a.ci[i] - a.sr[i]};
        put(out + (long)(S * q0) * (long)rsb, up, INV ? y2 : y1);
        if (q == 0 || 2 * q == P) continue;
        put(out + (long)(S * (P - 3 - q0)) * (long)rsb, down, INV ? y1 : y2);
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- x rows
// R2C of row pairs (2 p, 2 p + 1); tile b holds pairs [b RP, b RP + RP).  Rows
// outside [row_begin, nrows) are read as their neighbours' partners but not
// stored.  LDS columns of pair p: p (k = 0 of both rows), then per row KH
// columns.  lds: (P + 1) RS values, then the P roots.
template <int MODE, int S>
__device__ __forceinline__ void xr2c_tiles(const XArgs<double>& A, const XExtra& E, const Plan& M, unsigned first,
                                           unsigned stride, unsigned total, int nthreads, Cx<double>* lds) {
  constexpr int KH = S / 2, KF = (S - 1) / 2;   // k = 1 .. KF of both rows are separated; S even: k = S/2 is real
  constexpr int NT = tasks_per_thread(S);
  // An assembled right-hand side is loaded where it is used: its values are
  // computed on arrival, so a tile in flight hides nothing and costs registers
  // (S = 2..6 spilled 28..160 bytes a lane, S = 16 took 239; R2C, us: 4096 rows
  // of 100 points 19.7 -> 12.2, 65536 rows 70 -> 52).
  constexpr bool kLate = MODE == XM_DIV;
  const int tid = threadIdx.x;
  const int P = M.P, RS = E.RS, RP = E.RP, NC = RP * (1 + 2 * KH), n = A.nx, nz = A.nz, H = P / 2;
  const int rows = A.ny * nz;
  const QDiv qp = qdiv(P), qnz = qdiv(nz);
  Cx<double>* const roots = lds + (size_t)(P + 1) * RS;
  load_roots(M, A.twx, roots, nthreads);
  for (int i = tid; i < NC; i += nthreads) lds[__mul24(P, RS) + i] = Cx<double>{0.0, 0.0};
  int tp[NT], tj[NT];   // the tasks' row pair and j
  Twiddle<KH + 1, false> w[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    tp[i] = qquo(tid + i * nthreads, qp);
    tj[i] = tid + i * nthreads - __mul24(tp[i], P);
    if (tp[i] < RP) w[i].load(tj[i], A.twx);
  }
  const int lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), nw = nthreads / kWave;
  const int ntile = (NC + 15) / 16, items = M.MT * ntile;
  const long pgap = A.ps - (long)nz * A.rs;
  Cx<double> v[NT][S];
  // a task's rows of tile b; rows past the end read the last row (a last row
  // without a partner is its own)
  auto load_task = [&](int i, unsigned b) {
    const int row0 = (int)b * 2 * RP;
    const char* f = reinterpret_cast<const char*>(A.f + (size_t)row0 * n);
    const int p = tp[i], j = tj[i], last = rows - 1 - row0;
    const int la = 2 * p < last ? 2 * p : last, lb = 2 * p + 1 < last ? 2 * p + 1 : last;
    if constexpr (MODE == XM_DIV) {
      const int j0 = row0 / nz, k0 = row0 - j0 * nz;
      const int ja = qquo(k0 + la, qnz), jb = qquo(k0 + lb, qnz);
#pragma unroll
      for (int r = 0; r < S; ++r) {
        v[i][r].x = assemble_one(A, row0 + la, j0 + ja, k0 + la - __mul24(ja, nz), j + P * r);
        v[i][r].y = assemble_one(A, row0 + lb, j0 + jb, k0 + lb - __mul24(jb, nz), j + P * r);
      }
    } else {
      const unsigned oa = (unsigned)(la * n + j) * sizeof(double), ob = (unsigned)(lb * n + j) * sizeof(double);
#pragma unroll
      for (int r = 0; r < S; ++r) {
        v[i][r].x = at_d(f + (size_t)(P * r) * sizeof(double), oa);
        v[i][r].y = at_d(f + (size_t)(P * r) * sizeof(double), ob);
      }
    }
  };
  auto load = [&](unsigned b) {
#pragma unroll
    for (int i = 0; i < NT; ++i) load_task(i, b);
  };
  unsigned b = first;
  int rot = 0;
  if (!kLate && b < total) load(b);
  for (; b < total; b += stride) {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int p = tp[i];
      if (p >= RP) continue;
      if (kLate) load_task(i, b);
      Cx<double>* const z = v[i];
      Dft<S, false, double>::run(z);
      // per row: a[k] = A_k W^{j k}, b[k] = B_k W^{j k}
      Cx<double>* o = lds + __mul24(tj[i], RS);
      const int ca = RP + 2 * p * KH, cb = ca + KH;
      o[p] = z[0];
#pragma unroll
      for (int k = 1; k <= KH; ++k) {
        const Cx<double> t = w[i].get(k);
        if (k <= KF) {
          const Cx<double> zk = z[k], m = z[S - k];
          o[ca + k - 1] = cmul(Cx<double>{0.5 * (zk.x + m.x), 0.5 * (zk.y - m.y)}, t);
          o[cb + k - 1] = cmul(Cx<double>{0.5 * (zk.y + m.y), 0.5 * (m.x - zk.x)}, t);
        } else {
          o[ca + k - 1] = cscale(t, z[k].x);
          o[cb + k - 1] = cscale(t, z[k].y);
        }
      }
    }
    __syncthreads();
    if (!kLate && b + stride < total) load(b + stride);
    const int row0 = (int)b * 2 * RP;
    const int j0 = row0 / nz, k0 = row0 - j0 * nz;
    // byte offsets from the tile's first row (a tile's few thousand values and
    // the plane gaps between them: far below 2^32)
    char* const out = reinterpret_cast<char*>(A.spec + (size_t)row0 * A.rs + (size_t)j0 * pgap);
    auto row_off = [&](int lr) {
      return ((unsigned)lr * (unsigned)A.rs + (unsigned)qquo(k0 + lr, qnz) * (unsigned)pgap) * (unsigned)sizeof(Cx<double>);
    };
    auto stored = [&](int lr) { return row0 + lr >= A.row_begin && row0 + lr < A.nrows; };
    int it = wave + rot < nw ? wave + rot : wave + rot - nw;
    rot = rot + 1 < nw ? rot + 1 : 0;
    for (; it < items; it += nw) {
      const int mt = it / ntile, nt = it - mt * ntile;
      const Acc acc = products(M, roots, lds, RS, NC, mt, nt, lane);
      const int col = nt * 16 + lane % 16;
      if (col >= NC) continue;
      if (col < RP) {   // k = 0 of both rows: real sequences
        const bool sa = stored(2 * col), sb = stored(2 * col + 1);
        const unsigned oa = row_off(2 * col), ob = row_off(2 * col + 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int q = mt * 16 + acc_row(lane, i);
          if (q > H) continue;
          const unsigned o = (unsigned)(S * q) * sizeof(Cx<double>);
          if (sa) put(out, oa + o, Cx<double>{acc.cr[i], acc.sr[i]});
          if (sb) put(out, ob + o, Cx<double>{acc.ci[i], acc.si[i]});
          if (q == 0 && A.rowsum != nullptr) {   // the row sums
            if (sa) A.rowsum[row0 + 2 * col] = acc.cr[i];
            if (sb) A.rowsum[row0 + 2 * col + 1] = acc.ci[i];
          }
        }
      } else if constexpr (KH > 0) {
        const int lr = (col - RP) / KH, k = col - RP - lr * KH + 1;
        if (!stored(lr)) continue;
        const unsigned ro = row_off(lr);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int q = mt * 16 + acc_row(lane, i);
          if (q > H) continue;
          const Cx<double> y1{acc.cr[i] - acc.si[i], acc.ci[i] + acc.sr[i]};
          const Cx<double> y2{acc.cr[i] + acc.si[i], acc.ci[i] - acc.sr[i]};
          const int i1 = k + S * q, i2 = k + S * (P - q);
          // coefficients past n/2 are the conjugates of those at n - i; k = S/2
          // of an even S meets each one twice, and the lower one stays
          const bool lo1 = 2 * i1 <= n, lo2 = 2 * i2 <= n;
          if (lo1 || 2 * k != S)
            put(out, ro + (unsigned)(lo1 ? i1 : n - i1) * (unsigned)sizeof(Cx<double>), lo1 ? y1 : cconj(y1));
          if (q == 0 || 2 * q == P) continue;
          if (lo2 || 2 * k != S)
            put(out, ro + (unsigned)(lo2 ? i2 : n - i2) * (unsigned)sizeof(Cx<double>), lo2 ? y2 : cconj(y2));
        }
      }
    }
    __syncthreads();
  }
}

// C2R of tiles t below end; tile t of `total` (counted down from the last: the inverse z pass wrote the last
// planes last) holds rows [b RP, b RP + RP), b = base + total - 1 - t.  lds:
// (P/2 + 2) RS values (the last row zero), the P roots, then RP plane
// constants.
template <int MODE, int S>
__device__ __forceinline__ void xc2r_tiles(const XArgs<double>& A, const XExtra& E, const Plan& M, unsigned first,
                                           unsigned stride, unsigned base, unsigned total, unsigned end, int nthreads,
                                           Cx<double>* lds) {
  constexpr int NT = tasks_per_thread(S);
  const int tid = threadIdx.x;
  const int P = M.P, RS = E.RS, RP = E.RP, NC = RP * S, n = A.nx, nz = A.nz;
  const int H = P / 2, NJ = H + 1;
  const QDiv qj = qdiv(NJ), qnz = qdiv(nz);
  const long pgap = A.ps - (long)nz * A.rs;
  Cx<double>* const roots = lds + (size_t)(NJ + 1) * RS;
  double* const c00s = reinterpret_cast<double*>(roots + P);
  load_roots(M, A.twx, roots, nthreads);
  for (int i = tid; i < NC; i += nthreads) lds[__mul24(NJ, RS) + i] = Cx<double>{0.0, 0.0};
  int tr[NT], tj[NT];   // the tasks' row and j
  Twiddle<S, true> w[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    tr[i] = qquo(tid + i * nthreads, qj);
    tj[i] = tid + i * nthreads - __mul24(tr[i], NJ);
    if (tr[i] < RP) w[i].load(tj[i], A.twx);
  }
  const int lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), nw = nthreads / kWave;
  const int ntile = (NC + 15) / 16, items = M.MT * ntile;
  double cs = 2.0 * A.inv_nxnz;
  if (MODE == CM_ADD) cs = cs / A.ctl->scale[A.iter & 1];
  const double sub = MODE == CM_ADD ? A.ctl->phimean : 0.0;
  const int lk = lane / 16, lj = lane % 16;
  Cx<double> v[NT][S];
  double c00[NT];
  auto load = [&](unsigned b) {
    const int row0 = (int)b * RP, j0 = row0 / nz, k0 = row0 - j0 * nz;
    const char* sp = reinterpret_cast<const char*>(A.spec + (size_t)row0 * A.rs + (size_t)j0 * pgap);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      // every task loads: rows past the end read the last row
      const int last = (int)A.nrows - 1 - row0, lr = tr[i] < last ? tr[i] : last, jr = qquo(k0 + lr, qnz);
      const unsigned ro =
          ((unsigned)lr * (unsigned)A.rs + (unsigned)jr * (unsigned)pgap) * (unsigned)sizeof(Cx<double>);
      c00[i] = A.phi00[j0 + jr];
#pragma unroll
      for (int r = 0; r < S; ++r) {
        const int x = tj[i] + P * r;
        v[i][r] = at(sp, ro + (unsigned)(2 * x <= n ? x : n - x) * (unsigned)sizeof(Cx<double>));
      }
    }
  };
  unsigned t = first;
  int rot = 0;
  if (t < end) load(base + total - 1 - t);
  for (; t < end; t += stride) {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      if (tr[i] >= RP) continue;
      const int j = tj[i];
      // j = 0 and P/2 stand alone in the Hermitian sums; X[0] and X[n/2] of a
      // real sequence are real
      const double wt = j == 0 || 2 * j == P ? 0.5 : 1.0;
#pragma unroll
      for (int r = 0; r < S; ++r) {
        const int x = j + P * r;
        if (2 * x > n) v[i][r].y = -v[i][r].y;
        if (x == 0 || 2 * x == n) v[i][r].y = 0.0;
        v[i][r] = cscale(v[i][r], wt);
      }
      Dft<S, true, double>::run(v[i]);
      w[i].apply(v[i]);
      Cx<double>* o = lds + __mul24(j, RS) + __mul24(tr[i], S);
#pragma unroll
      for (int m = 0; m < S; ++m) o[m] = v[i][m];
      if (j == 0) c00s[tr[i]] = c00[i] * A.inv_nxnz - sub;
    }
    __syncthreads();
    if (t + stride < end) load(base + total - 1 - (t + stride));
    const int row0 = (int)(base + total - 1 - t) * RP;
    char* const out = reinterpret_cast<char*>(A.out + (size_t)row0 * n);
    int it = wave + rot < nw ? wave + rot : wave + rot - nw;
    rot = rot + 1 < nw ? rot + 1 : 0;
    for (; it < items; it += nw) {
      const int mt = it / ntile, nt = it - mt * ntile;
      acc4 ca{0.0, 0.0, 0.0, 0.0}, sa{0.0, 0.0, 0.0, 0.0};
      const int cc = nt * 16 + lj, col = cc < NC ? cc : NC - 1;
      Walk w1(M, roots, mt * 16 + lj, lk);
      auto rowv = [&](int kt) {
        const int r = 4 * kt + lk;
        return lds[__mul24(r < NJ ? r : NJ, RS) + col];
      };
      Cx<double> a0 = w1.next(), x0 = rowv(0);
      for (int kt = 0; kt < M.KT; kt += 2) {
        const Cx<double> a1 = w1.next(), x1 = rowv(kt + 1);
        keep_order();
        ca = mma(a0.x, x0.x, ca);
        sa = mma(a0.y, x0.y, sa);
        a0 = w1.next();
        x0 = rowv(kt + 2);
        keep_order();
        ca = mma(a1.x, x1.x, ca);
        sa = mma(a1.y, x1.y, sa);
      }
      if (cc >= NC) continue;
      const int lr = col / S, m = col - lr * S;
      const long row = row0 + lr;
      if (row < A.row_begin || row >= A.nrows) continue;
      const double k00 = c00s[lr];
      // row q = 16 mt + 4 i + lk goes to m + S q and m + S (P - q); sa holds
      // the sum with -sin
      const unsigned up = (unsigned)(lr * n + m + S * lk) * (unsigned)sizeof(double);
      const unsigned down = (unsigned)(lr * n + m + S * (3 - lk)) * (unsigned)sizeof(double);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int q0 = mt * 16 + 4 * i, q = q0 + lk;
        if (q > H) continue;
        double* o1 = reinterpret_cast<double*>(out + (long)(S * q0) * (long)sizeof(double) + up);
        double x1 = (ca[i] + sa[i]) * cs + k00, x2 = (ca[i] - sa[i]) * cs + k00;
        if (MODE == CM_ADD) x1 += *o1;
        *o1 = x1;
        if (q == 0 || 2 * q == P) continue;
        double* o2 = reinterpret_cast<double*>(out + (long)(S * (P - 3 - q0)) * (long)sizeof(double) + down);
        if (MODE == CM_ADD) x2 += *o2;
        *o2 = x2;
      }
    }
    __syncthreads();
  }
}

}  // namespace mdft
}  // namespace ibp
