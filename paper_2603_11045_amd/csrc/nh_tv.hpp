// nh_tv.hpp -- the discrete total-variation regulariser of the inverse
// problem (eq. tv_discrete, App. D.1) and its gradient, fused in one pass.
//
//   R(a) = dx dy dz sum_p t_p,   t_p = sqrt((d_x a / dx)^2 + (d_y a / dy)^2 + (d_z a / dz)^2 + eps^2)
//
// with forward differences along the array axes, x and y wrapping around and
// d_z a = 0 on the last plane. t_p depends on a_p and its +x, +y, +z
// neighbours, so dR/da_p collects p's own term and the terms of its -x, -y,
// -z neighbours (a 13-point stencil of a).
//
// A term is some 40 instructions (a square root and a division, both
// correctly rounded), and with the four terms of every cell computed by its
// own thread the instructions of a large grid take longer than the memory
// traffic. So there each term is computed once wherever a wave can hand it on: a
// lane walks a few rows of one column up a few planes, keeps the row's y
// weight for the next row and the plane's z weights for the next plane, and
// takes the x weight from the lane beside it. What a wave computes besides
// its cells is the row before its first, the plane below its first and the
// column before its first, the last for all its rows and planes in one go, a
// lane each. No LDS, no barrier: the waves are independent. (Small and thin
// grids keep a thread per cell, see tv_plan.)
//
// On 256 x 256 x 64 (FP32, added to a gradient: 84 MB, which stay in the
// last-level cache from call to call) the entry point took 51 us and now takes
// 31, some 15 of them two launches and a synchronisation; on 512 x 512 x 64
// (336 MB) 144 and now 85 us. What is left of the kernel is memory traffic.
//
// The workgroup's partial sum of t goes to its own slot; tv_finish_kernel sums
// the slots in a fixed order, so the value is deterministic.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "nh_kernels.hpp"

namespace nh {

constexpr int kTvBlock = 256;
constexpr int kTvMaxBlocks = 4096;
constexpr int kTvFinish = 512;
constexpr int kTvRows = 4;                  // rows of one column per lane, on grids large enough
constexpr int kTvThin = 100;                // a thread per cell up to this many columns,
constexpr int kTvCellWaves = 5;             //   and up to this many waves per SIMD of such threads
constexpr int kTvWaves = 4;                 // waves per SIMD that a plan aims at

// How waves cover the grid: lanes of 1 << lx columns, 64 >> lx groups of
// `rows` rows each, planes 0 .. pz - 1 of a unit; units x fastest.
struct TvPlan {
  int lx, rows, pz;
  int ux, uy, uz;                           // units along each axis
  int units, blocks;
};

// Small grids are bound by the launches and a wave's latency, not by instructions:
// there a thread per cell with its four terms has the shortest chain. On grids
// of few columns a wave would fill few of its lanes. The call, FP32 / FP64, a
// thread per cell against a wave per unit:
//   70 x 70 x 30          17.4 / 18.5 us, 19.0 / 20.1
//   96 x 96 x 32          18.5 / 20.3 us, 19.4 / 20.6
//   128 x 128 x 20        18.7 / 20.0 us, 18.8 / 20.4  (five waves per SIMD)
//   128 x 128 x 44        22.1 / 24.3 us, 20.7 / 22.6
//   256 x 256 x 40        34.7 / 43.4 us, 26.1 / 32.1
//   5 x 20 x 30000        37.7 / 46.8 us, 43.5 / 56.6  (100 columns)
//   12 x 10 x 30000       41.9 / 52.7 us, 39.5 / 52.1
//   1 x 1 x 100000        16.6 / 17.1 us, 56.1 / 77.4
// Otherwise narrow grids fold rows into the lanes (1 x 2000 x 300: 21.0 / 23.5 us
// with one column per wave row, 39.5 / 54.6 with 16). A unit of one row and one
// plane computes 4 terms for a cell, of 4 rows and one plane 2.5, of 4 rows and 16
// planes 1.4, but a wave's chain of terms is 4, 10 and 90 long: the larger
// units are for grids that still fill every SIMD with several waves (256 x
// 256 x 64: 4 rows, 4 planes), have rows for them (20000 x 1 x 64: 23.0 us with
// one row, 28.3 with four; 20000 x 3 x 64: 31.4 with four) and whose lanes can hold
// the column halos: 64 / (row groups * rows) planes per unit.
inline TvPlan tv_plan(int nx, int ny, int nz, int cus) {
  TvPlan P{};
  if ((long long)nx * ny <= kTvThin || (long long)nx * ny * nz <= (long long)cus * 4 * 64 * kTvCellWaves) {
    P.blocks = (int)std::min<long long>(((long long)nx * ny * nz + kTvBlock - 1) / kTvBlock, kTvMaxBlocks);
    return P;
  }
  while (P.lx < 6 && nx > 1 << P.lx) ++P.lx;
  const int groups = 64 >> P.lx;
  const long long want = (long long)cus * 4 * kTvWaves;
  P.ux = (int)(((long long)nx + (1 << P.lx) - 1) >> P.lx);
  P.rows = kTvRows;
  P.uy = (int)(((long long)ny + groups * P.rows - 1) / (groups * P.rows));
  if (P.lx < 2 || ny <= 2 * groups || (long long)P.ux * P.uy * nz < want) {
    P.rows = 1;
    P.uy = (int)(((long long)ny + groups - 1) / groups);
  }
  const long long cols = (long long)P.ux * P.uy;
  P.pz = 64 / (groups * P.rows);
  while (P.pz > 1 && cols * (((long long)nz + P.pz - 1) / P.pz) < want) P.pz >>= 1;
  P.uz = (int)(((long long)nz + P.pz - 1) / P.pz);
  P.units = (int)(cols * P.uz);
  P.blocks = (int)std::min<long long>((P.units + kTvBlock / 64 - 1) / (kTvBlock / 64), kTvMaxBlocks);
  return P;
}

template <typename R>
struct TvArgs {
  const R* alpha;
  int nx, ny, nz;
  long long nxy;
  TvPlan P;
  R ix2, iy2, iz2;                          // 1 / h_d^2
  R eps2;
  double scale;                             // weight * dx dy dz
  double* grad;                             // [nz][ny][nx] FP64
  int accumulate;                           // 1: grad += scale dR/da; 0: grad = scale dR/da
  double* partial;                          // [gridDim.x] per-workgroup sums of t
};

// The forward differences of a cell, each over h_d^2, and 1 / t, from its value
// and its +x, +y, +z neighbours' (dz = 0 on the last plane); returns t. The
// term's weight on a neighbour is c_d / t, and it is handed on as the two
// factors: a cell's gradient is a chain of fused multiply-adds over them.
template <typename R>
struct TvTerm {
  R cx, cy, cz, rt;
};
template <typename R>
__device__ __forceinline__ R tv_term(const TvArgs<R>& A, R ap, R ax, R ay, R dz, TvTerm<R>& o) {
  const R dx = ax - ap;
  const R dy = ay - ap;
  o.cx = dx * A.ix2;
  o.cy = dy * A.iy2;
  o.cz = dz * A.iz2;
  const R t = sqrt(add_rn(fma_r(mul_rn(dz, dz), A.iz2, fma_r(mul_rn(dx, dx), A.ix2, mul_rn(mul_rn(dy, dy), A.iy2))),
                          A.eps2));
  o.rt = R(1) / t;
  return t;
}

// Row j of the wrapping y axis (unsigned: -1 is the row before the first; past
// the row after the last: any row). Offsets are 64-bit, an x-y plane may hold
// 2^31 cells and more; indices that run past an axis' end are unsigned.
__device__ __forceinline__ unsigned tv_row(unsigned j, unsigned ny) {
  j = j == ~0u ? ny - 1 : j;
  j = j >= ny ? j - ny : j;
  return j >= ny ? 0 : j;
}

// The workgroup's sum of t in a fixed order: wave butterfly, then the waves in order.
template <typename R>
__device__ __forceinline__ void tv_partial(const TvArgs<R>& A, double tsum) {
  __shared__ double red[kTvBlock / 64];
  tsum = wave_sum(tsum);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = tsum;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kTvBlock / 64; ++w) s += red[w];
    A.partial[blockIdx.x] = s;
  }
}

template <typename R, int K>
__global__ void __launch_bounds__(kTvBlock) tv_kernel(TvArgs<R> A) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lx = A.P.lx, groups = 64 >> lx;
  const int tx = lane & ((1 << lx) - 1), grp = lane >> lx;
  double tsum = 0.0;
  for (int u = (int)blockIdx.x * (kTvBlock / 64) + wave; u < A.P.units; u += (int)gridDim.x * (kTvBlock / 64)) {
    const int uxy = A.P.ux * A.P.uy;
    const int uz = u / uxy, uc = u - uz * uxy, uy = uc / A.P.ux, ux = uc - uy * A.P.ux;
    const unsigned nx = A.nx, ny = A.ny, nz = A.nz;
    const unsigned x0 = (unsigned)ux << lx, k0 = (unsigned)uz * A.P.pz, k1 = min(nz, k0 + A.P.pz);
    const unsigned j0 = ((unsigned)uy * groups + grp) * K;
    const bool xin = x0 + tx < nx;
    const unsigned i = xin ? x0 + tx : 0, ip = i + 1 < nx ? i + 1 : 0;
    long long row[K + 2];                   // offsets of rows j0 - 1 .. j0 + K
#pragma unroll
    for (int s = 0; s < K + 2; ++s) row[s] = (long long)nx * tv_row(j0 - 1 + s, ny);

    // the column before the wave's first, all its rows and planes: lane
    // (plane * groups + group) * K + row computes that cell's x weight
    TvTerm<R> hx{R(0), R(0), R(0), R(0)};
    {
      const unsigned r = lane % K, hg = lane / K % groups, hk = k0 + lane / (K * groups);
      const unsigned hj = ((unsigned)uy * groups + hg) * K + r;
      if (hk < k1 && hj < ny) {
        const R* pk = A.alpha + (long long)hk * A.nxy;
        const long long ho = (long long)nx * hj;
        const unsigned hi = x0 > 0 ? x0 - 1 : nx - 1;
        const R ap = pk[ho + hi];
        const R dz = hk + 1 < nz ? pk[A.nxy + ho + hi] - ap : R(0);
        tv_term(A, ap, pk[ho + x0], pk[(long long)nx * tv_row(hj + 1, ny) + hi], dz, hx);
      }
    }

    R czb[K], rtb[K];                       // z factors of the plane below
    R av[K + 2], ax[K + 1];                 // the plane's values at i and, rows j0 - 1 .., at i + 1
    const R* pk = A.alpha + (long long)k0 * A.nxy;
#pragma unroll
    for (int s = 0; s < K + 2; ++s) av[s] = pk[row[s] + i];
#pragma unroll
    for (int s = 0; s < K + 1; ++s) ax[s] = pk[row[s] + ip];
#pragma unroll
    for (int r = 0; r < K; ++r) czb[r] = rtb[r] = R(0);
    if (k0 > 0) {
      const R* pm = pk - A.nxy;
      R bv[K + 1], bx[K];
#pragma unroll
      for (int s = 0; s < K + 1; ++s) bv[s] = pm[row[s + 1] + i];
#pragma unroll
      for (int s = 0; s < K; ++s) bx[s] = pm[row[s + 1] + ip];
#pragma unroll
      for (int r = 0; r < K; ++r) {
        TvTerm<R> o;
        tv_term(A, bv[r], bx[r], bv[r + 1], av[r + 1] - bv[r], o);
        czb[r] = o.cz;
        rtb[r] = o.rt;
      }
    }
    for (unsigned k = k0; k < k1; ++k) {
      const bool last = k + 1 == nz;
      const R* pn = A.alpha + (long long)(last ? k : k + 1) * A.nxy;
      double* gk = A.grad + (long long)k * A.nxy;
      R an[K + 2], anx[K + 1];
      double g0[K];
#pragma unroll
      for (int s = 0; s < K + 2; ++s) an[s] = pn[row[s] + i];
      if (A.accumulate) {
#pragma unroll
        for (int r = 0; r < K; ++r) g0[r] = xin && j0 + r < ny ? gk[row[r + 1] + i] : 0.0;
      }
#pragma unroll
      for (int s = 0; s < K + 1; ++s) anx[s] = pn[row[s] + ip];
      R cyb = R(0), rty = R(0);             // y factors of the row before
#pragma unroll
      for (int s = 0; s < K + 1; ++s) {
        TvTerm<R> o;
        const R t = tv_term(A, av[s], ax[s], av[s + 1], last ? R(0) : an[s] - av[s], o);
        if (s > 0) {
          const int r = s - 1, hl = ((int)(k - k0) * groups + grp) * K + r;
          // the cell is the +x neighbour of the one before it
          const R cxl = __shfl_up(o.cx, 1, 64), rtl = __shfl_up(o.rt, 1, 64);
          const R cxh = __shfl(hx.cx, hl, 64), rth = __shfl(hx.rt, hl, 64);
          R g = -fma_r(o.cz, o.rt, fma_r(o.cx, o.rt, mul_rn(o.cy, o.rt)));
          g = fma_r(tx > 0 ? cxl : cxh, tx > 0 ? rtl : rth, g);
          g = fma_r(cyb, rty, g);
          if (k > 0) g = fma_r(czb[r], rtb[r], g);
          if (xin && j0 + r < ny) {
            const double v = mul_rn(A.scale, (double)g);   // (not fused: the same gradient, added or not)
            gk[row[s] + i] = A.accumulate ? add_rn(g0[r], v) : v;
            tsum += (double)t;
          }
          czb[r] = o.cz;
          rtb[r] = o.rt;
        }
        cyb = o.cy;
        rty = o.rt;
      }
#pragma unroll
      for (int s = 0; s < K + 2; ++s) av[s] = an[s];
#pragma unroll
      for (int s = 0; s < K + 1; ++s) ax[s] = anx[s];
    }
  }
  tv_partial(A, tsum);
}

// A thread per cell with its four terms (P.rows == 0), the same factors and chain.
template <typename R>
__global__ void __launch_bounds__(kTvBlock) tv_cell_kernel(TvArgs<R> A) {
  double tsum = 0.0;
  const unsigned nx = A.nx, ny = A.ny, nz = A.nz, nxy = (unsigned)A.nxy;   // (small)
  const long long ng = A.nxy * nz;
  for (long long p = (long long)blockIdx.x * kTvBlock + threadIdx.x; p < ng; p += (long long)gridDim.x * kTvBlock) {
    const unsigned k = (unsigned)(p / nxy), c = (unsigned)(p - (long long)k * nxy), j = c / nx, i = c - j * nx;
    auto term = [&](unsigned ti, unsigned tj, unsigned tk, TvTerm<R>& o) -> R {
      const R* q = A.alpha + (long long)tk * nxy;
      const R ap = q[ti + nx * tj];
      return tv_term(A, ap, q[(ti + 1 < nx ? ti + 1 : 0) + nx * tj], q[ti + nx * (tj + 1 < ny ? tj + 1 : 0)],
                     tk + 1 < nz ? q[nxy + ti + nx * tj] - ap : R(0), o);
    };
    TvTerm<R> o, l;
    const R t = term(i, j, k, o);
    R g = -fma_r(o.cz, o.rt, fma_r(o.cx, o.rt, mul_rn(o.cy, o.rt)));
    term(i > 0 ? i - 1 : nx - 1, j, k, l);
    g = fma_r(l.cx, l.rt, g);
    term(i, j > 0 ? j - 1 : ny - 1, k, l);
    g = fma_r(l.cy, l.rt, g);
    if (k > 0) {
      term(i, j, k - 1, l);
      g = fma_r(l.cz, l.rt, g);
    }
    const double v = mul_rn(A.scale, (double)g);
    A.grad[p] = A.accumulate ? add_rn(A.grad[p], v) : v;
    tsum += (double)t;
  }
  tv_partial(A, tsum);
}

// value = scale * sum of the partials: each thread its own in order, then the
// threads by butterfly and the waves in order (one workgroup).
__global__ void __launch_bounds__(kTvFinish) tv_finish_kernel(const double* partial, int n, double scale,
                                                                double* value) {
  __shared__ double red[kTvFinish / 64];
  double s = 0.0;
#pragma unroll
  for (int b = 0; b < kTvMaxBlocks / kTvFinish; ++b) {
    const int e = b * kTvFinish + (int)threadIdx.x;
    s += e < n ? partial[e] : 0.0;
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double tot = 0.0;
    for (int w = 0; w < kTvFinish / 64; ++w) tot += red[w];
    *value = scale * tot;
  }
}

}  // namespace nh
