// The per-order kernels of libsem (N fixed at compile time, as the jit clause
// of the paper's "ax" kernel fixes it, Sec. VIII-B): the metric setup, the
// element operator (vector-ALU and matrix-core tiles), the gather-scatter
// forms, the CG start and the CG update.  The library builds them for orders
// 1..12 (sem_ax.hip, sem_vec.hip); for orders 13..15 the same text is
// compiled at run time (sem_rtc.hip), so both paths run the same kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "sem_ax_mfma.h"
#include "sem_ax_tile.h"
#include "sem_cg_dev.h"
#include "sem_device.h"
#include "sem_types.h"

namespace semk {

template <int N1>
struct AxCfg {
  // elements per work-group of the per-order kernels: about 128 threads of
  // one (i, j) column each
  static constexpr int EPB = (N1 * N1 >= 128) ? 1 : (128 / (N1 * N1));
  static constexpr int THREADS = N1 * N1 * EPB;
};

// The operator kernels: the same elements per work-group, AxTile<N1>::TPE
// threads per element.
#ifndef SEM_OP_MIN_WAVES_SPLIT
#define SEM_OP_MIN_WAVES_SPLIT 1
#endif
#ifndef SEM_OP_MIN_WAVES_COL
#define SEM_OP_MIN_WAVES_COL 1
#endif
template <int N1>
struct OpCfg {
  static constexpr int EPB = AxCfg<N1>::EPB;
  static constexpr int THREADS = AxTile<N1>::TPE * EPB;
  static constexpr int MIN_WAVES = AxTile<N1>::kSplit ? SEM_OP_MIN_WAVES_SPLIT : SEM_OP_MIN_WAVES_COL;
};

template <int N1, class P, bool CG, class SC>
__device__ __forceinline__ void ax_body(int64_t E, const typename P::TC *__restrict__ Dg,
                                        const typename P::TG *__restrict__ G, typename P::TV *u,
                                        typename P::TV *__restrict__ w,
                                        const typename P::TV *__restrict__ z,
                                        typename P::TV *__restrict__ x, const SC &scalars,
                                        double *__restrict__ part) {
  using C = OpCfg<N1>;
  using TC = typename P::TC;
  __shared__ TC sD[N1 * N1];
  __shared__ TC s1[C::EPB * AxTile<N1>::TILE];
  __shared__ TC s2[C::EPB * AxTile<N1>::TILE];
  __shared__ TC s3[AxTile<N1>::kTiles == 3 ? C::EPB * AxTile<N1>::TILE : 1];
  __shared__ double sred[CG ? C::THREADS : 1];
  ax_tile<N1, C::EPB, P, CG, false, SC>(E, (int64_t)blockIdx.x * C::EPB, Dg, G, u, w, z, x, scalars,
                                        part, sD, s1, s2, s3, sred);
}

template <int N1, class P, bool CG>
__global__ void __launch_bounds__(OpCfg<N1>::THREADS, OpCfg<N1>::MIN_WAVES)
    ax_kernel(int64_t E, const typename P::TC *__restrict__ Dg, const typename P::TG *__restrict__ G,
              typename P::TV *u, typename P::TV *__restrict__ w, const typename P::TV *__restrict__ z,
              typename P::TV *__restrict__ x,
              CgState *__restrict__ st, double *__restrict__ part) {
  GivenScalars sc{0.0, 0.0};
  if (CG) {
    if (st->done) return;  // uniform: converged solves skip all work
    sc = GivenScalars{st->alpha, st->beta};
  }
  ax_body<N1, P, CG>(E, Dg, G, u, w, z, x, sc, part);
}

// The CG operator of a folded iteration (cg_folded): the beta step of the
// last update, whose n_upd partials are part_rr and part_rz, inside.
template <int N1, class P>
__global__ void __launch_bounds__(OpCfg<N1>::THREADS, OpCfg<N1>::MIN_WAVES)
    ax_fold_kernel(int64_t E, const typename P::TC *__restrict__ Dg, const typename P::TG *__restrict__ G,
                   typename P::TV *u, typename P::TV *__restrict__ w, const typename P::TV *__restrict__ z,
                   typename P::TV *__restrict__ x,
                   CgState *__restrict__ st, double *__restrict__ part,
                   const double *__restrict__ part_rr, const double *__restrict__ part_rz, int n_upd) {
  __shared__ double sfold[2 * kFinGroup / 64];
  const FoldBeta<OpCfg<N1>::THREADS / 64> sc(st, part_rr, part_rz, n_upd, sfold);
  ax_body<N1, P, true>(E, Dg, G, u, w, z, x, sc, part);
}

// The operator with the D contractions on the matrix cores (sem_ax_mfma.h):
// ceil((N+1)^2 / 16) waves per element.
template <int N1, class P, bool CG, bool SW, class SC>
__device__ __forceinline__ void ax_mfma_body(int64_t E, const typename P::TC *__restrict__ Dg,
                                             const typename P::TG *__restrict__ G,
                                             typename P::TV *u, typename P::TV *__restrict__ w,
                                             const typename P::TV *__restrict__ z,
                                             typename P::TV *__restrict__ x, const SC &scalars,
                                             double *__restrict__ part) {
  using C = MfmaCfg<N1>;
  using TC = typename P::TC;
  __shared__ TC sD[mfma_d_size<N1, P>()];
  __shared__ TC s1[C::EPB * AxTile<N1>::TILE];
  __shared__ TC s2[C::EPB * AxTile<N1>::TILE];
  __shared__ TC s3[C::EPB * AxTile<N1>::TILE];
  __shared__ double sred[C::THREADS / 64];
  ax_tile_mfma<N1, C::EPB, P, CG, false, SW, SC>(E, (int64_t)blockIdx.x * C::EPB, Dg, G, u, w, z, x,
                                                 scalars, part, sD, s1, s2, s3, sred);
}

template <int N1, class P, bool CG>
__global__ void __launch_bounds__(MfmaCfg<N1>::THREADS, (mfma_waves_per_simd<N1, P, CG>()))
    ax_mfma_kernel(int64_t E, const typename P::TC *__restrict__ Dg,
                   const typename P::TG *__restrict__ G, typename P::TV *u,
                   typename P::TV *__restrict__ w, const typename P::TV *__restrict__ z,
                   typename P::TV *__restrict__ x,
                   CgState *__restrict__ st, double *__restrict__ part) {
  GivenScalars sc{0.0, 0.0};
  if (CG) {
    if (st->done) return;  // uniform: converged solves skip all work
    sc = GivenScalars{st->alpha, st->beta};
  }
  ax_mfma_body<N1, P, CG, false>(E, Dg, G, u, w, z, x, sc, part);
}

// As ax_fold_kernel.
template <int N1, class P>
__global__ void __launch_bounds__(MfmaCfg<N1>::THREADS, (mfma_waves_per_simd<N1, P, true>()))
    ax_mfma_fold_kernel(int64_t E, const typename P::TC *__restrict__ Dg,
                        const typename P::TG *__restrict__ G, typename P::TV *u,
                        typename P::TV *__restrict__ w, const typename P::TV *__restrict__ z,
                        typename P::TV *__restrict__ x,
                        CgState *__restrict__ st, double *__restrict__ part,
                        const double *__restrict__ part_rr, const double *__restrict__ part_rz, int n_upd) {
  __shared__ double sfold[2 * kFinGroup / 64];
  const FoldBeta<MfmaCfg<N1>::THREADS / 64> sc(st, part_rr, part_rz, n_upd, sfold);
  ax_mfma_body<N1, P, true, false>(E, Dg, G, u, w, z, x, sc, part);
}

// The element-local sem_ax, whose result goes to the caller as it is (no
// gather reads it next): the same kernel with w written by non-temporal
// stores.
template <int N1, class P>
__global__ void __launch_bounds__(MfmaCfg<N1>::THREADS, (mfma_waves_per_simd<N1, P, false>()))
    ax_mfma_local_kernel(int64_t E, const typename P::TC *__restrict__ Dg,
                         const typename P::TG *__restrict__ G, typename P::TV *u,
                         typename P::TV *__restrict__ w) {
  ax_mfma_body<N1, P, false, true>(E, Dg, G, u, w, nullptr, nullptr, GivenScalars{0.0, 0.0}, nullptr);
}

// Metric setup: coordinates of the (deformed) box mesh, isoparametric
// Jacobian by D along r, s, t, G = w_i w_j w_k det(J) J^-1 J^-T, then the
// diagonal of the element operator.  With a low-precision copy (G32 or G16,
// else null) G is rounded into it as it is formed.
//
// One thread per (i, j) column: its three coordinates along t in registers, the
// planes the r and s contractions read in LDS.  Nine contractions, the
// cofactors and the diagonal come to about 250 FP64 operations a point at
// N = 11 against the 56 bytes written, so the kernel is bound by the vector
// units and LDS; every array index is a constant (unrolled), so that the
// columns stay in registers.  A plane of coordinates is read by its own plane's
// contractions only, so plane k of the three diagonal factors replaces it once
// every thread is past it (no further LDS tile).
//
// From N = 13 on, the orders compiled at run time, the loops over the planes
// stay rolled, or run two planes at a time where their number is even (the
// diagonal's mixed part then waits in its place in memory): unrolled they made
// the first set-up of such an order wait for the compiler, N = 13 / 14 / 15 1.10
// / 1.23 / 1.15 s against 0.57 / 0.56 / 0.53 s, and gained nothing (17^3 boxes
// 605 / 692 / 791 us unrolled, 488 / 690 / 739 so; N = 15 one plane at a time
// 815).
template <int N1>
__global__ void __launch_bounds__(AxCfg<N1>::THREADS)
    setup_geom_kernel(Box b, double amp, const double *__restrict__ Dg,
                      const double *__restrict__ nodes, double *__restrict__ G,
                      double *__restrict__ diag, float *__restrict__ G32, uint16_t *__restrict__ G16) {
  using C = AxCfg<N1>;
  using T = AxTile<N1>;
  constexpr int NP = T::NP;
  constexpr int PL = N1 * N1;
  __shared__ double sD[N1 * N1];
  __shared__ double sx[3][C::EPB * T::TILE];
  __shared__ double sz[2][C::EPB * N1];  // Z0 and sin(2 pi Z0) of the element's planes

  const int tid = threadIdx.x;
  const int el = tid / PL;
  const int ij = tid - el * PL;
  const int i = ij % N1;
  const int j = ij / N1;
  const int64_t e = (int64_t)blockIdx.x * C::EPB + el;
  const bool active = e < b.E();
  for (int t = tid; t < N1 * N1; t += C::THREADS) sD[t] = Dg[t];

  const int64_t ee = active ? e : 0;
  const uint32_t eyz = b.fdx.div((uint32_t)ee);
  const uint32_t ez = b.fdy.div(eyz);
  const int ex = (int)((uint32_t)ee - eyz * (uint32_t)b.nx);
  const int ey = (int)(eyz - ez * (uint32_t)b.ny);
  const double xi_i = nodes[i], xi_j = nodes[j];
  const double X0 = (ex + 0.5 * (xi_i + 1.0)) / b.nx;
  const double Y0 = (ey + 0.5 * (xi_j + 1.0)) / b.ny;
  double *SX = sx[0] + el * T::TILE;
  double *SY = sx[1] + el * T::TILE;
  double *SZ = sx[2] + el * T::TILE;
  const double twopi = 2.0 * M_PI;
  if (ij < N1) {
    const double Z0 = ((int)ez + 0.5 * (nodes[ij] + 1.0)) / b.nz;
    sz[0][el * N1 + ij] = Z0;
    sz[1][el * N1 + ij] = amp != 0.0 ? sin(twopi * Z0) : 0.0;
  }
  __syncthreads();
  double cx[N1], cy[N1], cz[N1];
  const double bxy = amp != 0.0 ? amp * sin(twopi * X0) * sin(twopi * Y0) : 0.0;
#pragma unroll
  for (int k = 0; k < N1; ++k) {
    const double bump = bxy * sz[1][el * N1 + k];
    const int o = k * T::PLANE + j * T::P + i;
    SX[o] = cx[k] = X0 + bump;
    SY[o] = cy[k] = Y0 + bump;
    SZ[o] = cz[k] = sz[0][el * N1 + k] + bump;
  }
  double Da[N1], Db[N1];
#pragma unroll
  for (int l = 0; l < N1; ++l) {
    Da[l] = sD[i * N1 + l];
    Db[l] = sD[j * N1 + l];
  }
  const double Dii = sD[i * N1 + i], Djj = sD[j * N1 + j];
  __syncthreads();

  const double wij = nodes[N1 + i] * nodes[N1 + j];
  const int64_t base = e * NP + ij;
  constexpr bool ROLLED = N1 > 13;
  constexpr int UNROLL = !ROLLED ? N1 : (N1 % 2 == 0 ? 2 : 1);  // of the loops over the planes
  double cross[ROLLED ? 1 : N1];           // the diagonal's part from the mixed factors
  // the diagonal factors: up to N = 5 in registers until every plane is done
  // (one barrier in all), else to LDS plane by plane
  constexpr bool HELD = N1 <= 6;
  double gd[3][HELD ? N1 : 1];
#pragma unroll UNROLL
  for (int k = 0; k < N1; ++k) {
    double J[3][3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double *S = d == 0 ? SX : (d == 1 ? SY : SZ);
      double a = 0.0, bb = 0.0, c = 0.0;
#pragma unroll
      for (int l = 0; l < N1; ++l) {
        a += Da[l] * S[k * T::PLANE + j * T::P + l];
        bb += Db[l] * S[k * T::PLANE + l * T::P + i];
        c += Dg[k * N1 + l] * (d == 0 ? cx[l] : (d == 1 ? cy[l] : cz[l]));
      }
      J[d][0] = a;
      J[d][1] = bb;
      J[d][2] = c;
    }
    // cofactors; inv[m][d] = cof[d][m] / det
    const double c00 = J[1][1] * J[2][2] - J[1][2] * J[2][1];
    const double c01 = J[1][2] * J[2][0] - J[1][0] * J[2][2];
    const double c02 = J[1][0] * J[2][1] - J[1][1] * J[2][0];
    const double c10 = J[0][2] * J[2][1] - J[0][1] * J[2][2];
    const double c11 = J[0][0] * J[2][2] - J[0][2] * J[2][0];
    const double c12 = J[0][1] * J[2][0] - J[0][0] * J[2][1];
    const double c20 = J[0][1] * J[1][2] - J[0][2] * J[1][1];
    const double c21 = J[0][2] * J[1][0] - J[0][0] * J[1][2];
    const double c22 = J[0][0] * J[1][1] - J[0][1] * J[1][0];
    const double det = J[0][0] * c00 + J[0][1] * c01 + J[0][2] * c02;
    // rows of J^-1: R_m[d] = cof[d][m] / det
    const double inv = 1.0 / det;
    const double R0[3] = {c00 * inv, c10 * inv, c20 * inv};
    const double R1[3] = {c01 * inv, c11 * inv, c21 * inv};
    const double R2[3] = {c02 * inv, c12 * inv, c22 * inv};
    const double sc = wij * nodes[N1 + k] * det;
    const double g[6] = {sc * (R0[0] * R0[0] + R0[1] * R0[1] + R0[2] * R0[2]),
                         sc * (R0[0] * R1[0] + R0[1] * R1[1] + R0[2] * R1[2]),
                         sc * (R0[0] * R2[0] + R0[1] * R2[1] + R0[2] * R2[2]),
                         sc * (R1[0] * R1[0] + R1[1] * R1[1] + R1[2] * R1[2]),
                         sc * (R1[0] * R2[0] + R1[1] * R2[1] + R1[2] * R2[2]),
                         sc * (R2[0] * R2[0] + R2[1] * R2[1] + R2[2] * R2[2])};
    if (active) {
      const int64_t at = e * 6 * NP + ij + k * PL;
#pragma unroll
      for (int q = 0; q < 6; ++q) G[at + q * NP] = g[q];
      if (G32) {
#pragma unroll
        for (int q = 0; q < 6; ++q) G32[at + q * NP] = (float)g[q];
      } else if (G16) {
#pragma unroll
        for (int q = 0; q < 6; ++q) G16[at + q * NP] = bf16_bits((float)g[q]);
      }
    }
    const double Dkk = Dg[k * N1 + k];
    const double mixed = 2.0 * Dii * Djj * g[1] + 2.0 * Dii * Dkk * g[2] + 2.0 * Djj * Dkk * g[4];
    if constexpr (!ROLLED)
      cross[k] = mixed;
    else if (active)
      diag[base + k * PL] = mixed;
    gd[0][HELD ? k : 0] = g[0];
    gd[1][HELD ? k : 0] = g[3];
    gd[2][HELD ? k : 0] = g[5];
    if constexpr (!HELD) {
      __syncthreads();  // every thread is past plane k
      const int o = k * T::PLANE + j * T::P + i;
      SX[o] = g[0];
      SY[o] = g[3];
      SZ[o] = g[5];
    }
  }
  __syncthreads();
  if constexpr (HELD) {
#pragma unroll
    for (int k = 0; k < N1; ++k) {
      const int o = k * T::PLANE + j * T::P + i;
      SX[o] = gd[0][k];
      SY[o] = gd[1][k];
      SZ[o] = gd[2][k];
    }
    __syncthreads();
  }
#pragma unroll
  for (int l = 0; l < N1; ++l) {
    const double a = sD[l * N1 + i], bb = sD[l * N1 + j];
    Da[l] = a * a;
    Db[l] = bb * bb;
  }
#pragma unroll UNROLL
  for (int k = 0; k < N1; ++k) {
    double d = 0.0;
#pragma unroll
    for (int l = 0; l < N1; ++l) {
      const double c = Dg[l * N1 + k];
      d += Da[l] * SX[k * T::PLANE + j * T::P + l];
      d += Db[l] * SY[k * T::PLANE + l * T::P + i];
      d += c * c * SZ[l * T::PLANE + j * T::P + i];
    }
    if constexpr (ROLLED) {
      if (active) diag[base + k * PL] += d;
    } else {
      d += cross[k];
      if (active) diag[base + k * PL] = d;
    }
  }
}

// ------------------------------------------------------------ gather-scatter
// out32 (the Jacobi inverse only, may be null): the result rounded to FP32 too.
// Linear tiles, with the index decode of the linear update tile (LinItems):
// kLinGroup items at a time, every load of a group before its first sum
// (masked FP64 gather at N = 9, 5083 elements: 23.6 -> 20.4 us against a
// node-by-node decode).
template <int N1, int MODE, typename T>
__global__ void __launch_bounds__(kVecThreads)
    gather_kernel(Box b, int64_t L, int64_t ntiles, const T *__restrict__ wl, T *__restrict__ out,
                  float *__restrict__ out32, int chunked) {
  const int64_t tile = chunk_tile(ntiles, chunked != 0);
  if (tile >= ntiles) return;
  const LinItems<N1> P(b, tile, (int)threadIdx.x);
  T res[kVecItems];
  bool live[kVecItems];
#pragma unroll
  for (int g = 0; g < kVecItems; g += kLinGroup) {
    T v[kLinGroup][8];
    bool upd[kLinGroup];
#pragma unroll
    for (int u = 0; u < kLinGroup; ++u) {
      const typename LinItems<N1>::Item t = P.item(g + u);
      live[g + u] = t.live;
      upd[u] = t.upd;
#pragma unroll
      for (int q = 0; q < 8; ++q) v[u][q] = LinItems<N1>::has_copy(t.sh, q) ? wl[t.lo + P.off(q)] : (T)0;
    }
#pragma unroll
    for (int u = 0; u < kLinGroup; ++u) {
      // the copies in ascending element-local order (a missing one adds +0)
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < 8; ++q) s += (double)v[u][q];
      if (MODE == kGatherInverse) s = 1.0 / s;
      res[g + u] = (MODE != kGatherAssembled && !upd[u]) ? (T)0 : (T)s;
    }
    // as in the update: the next group's loads stay behind this group's sums
#pragma unroll
    for (int u = 0; u < kLinGroup; ++u) asm volatile("" : "+v"(res[g + u]) : : "memory");
  }
#pragma unroll
  for (int u = 0; u < kVecItems; ++u)
    if (live[u]) out[P.raw0 + (uint32_t)(u * kVecThreads)] = res[u];
  if (MODE == kGatherInverse && out32 != nullptr) {
#pragma unroll
    for (int u = 0; u < kVecItems; ++u)
      if (live[u]) out32[P.raw0 + (uint32_t)(u * kVecThreads)] = (float)res[u];
  }
}

// The same gather on element-column tiles (copies paired across faces, as
// in the CG update).  V: the tile shape (upd_shape).
template <int N1, int MODE, typename T, int V>
__global__ void __launch_bounds__((UpdTile<N1, T, V>::BLOCK))
    gather_col_kernel(Box b, int64_t ntiles, const T *__restrict__ wl, T *__restrict__ out,
                      float *__restrict__ out32, int chunked) {
  using U = UpdTile<N1, T, V>;
  __shared__ double sA[U::LDS];
  const int64_t tile = chunk_tile(ntiles, chunked != 0);
  if (tile >= ntiles) return;
  const ColumnPos<N1, T, V> p(b, tile, (int)threadIdx.x);
  double S[U::KN];
  column_copy_sums<N1, T, V>(p, wl, sA, S);
#pragma unroll
  for (int kk = 0; kk < U::KN; ++kk) {
    const int k = p.kb + kk;
    if (p.live && k < p.kend) {
      double v = S[kk];
      if (MODE != kGatherAssembled && p.boundary(b, k))
        v = 0.0;
      else if (MODE == kGatherInverse)
        v = 1.0 / v;
      out[p.col0 + (int64_t)k * U::COLS] = (T)v;
      if (MODE == kGatherInverse && out32 != nullptr) out32[p.col0 + (int64_t)k * U::COLS] = (float)v;
    }
  }
}

// ------------------------------------------------------------ CG kernels
template <int N1>
__global__ void __launch_bounds__(kVecThreads)
    cg_init_kernel(Box b, int64_t L, int64_t ntiles, const double *__restrict__ bvec,
                   double *__restrict__ x, double *__restrict__ z, double *__restrict__ p,
                   const double *__restrict__ minv, double *__restrict__ part_rz,
                   double *__restrict__ part_bb) {
  __shared__ double sred[2 * (kVecThreads / 64)];
  const int64_t tile = xcd_tile(ntiles);
  TileSums t{0.0, 0.0};
  if (tile < ntiles) t = cg_init_tile<N1>(b, L, tile, bvec, x, z, p, minv, sred);
  if (threadIdx.x == 0) {
    part_rz[tile] = t.a;
    part_bb[tile] = t.b;
  }
}

// V: the update tile shape (upd_shape), one kernel per candidate.
template <int N1, typename TV, int V = 0>
__global__ void __launch_bounds__((UpdTile<N1, TV, V>::BLOCK))
    cg_update_kernel(Box b, int64_t ntiles, TV *__restrict__ z, const TV *__restrict__ w,
                     const TV *__restrict__ minv, CgState *__restrict__ st,
                     double *__restrict__ part_rr, double *__restrict__ part_rz) {
  __shared__ double sred[2 * (UpdTile<N1, TV, V>::BLOCK / 64)];
  __shared__ double sA[UpdTile<N1, TV, V>::LDS];
  if (st->done) return;
  const GivenScalars sc{st->alpha, 0.0};
  const int64_t tile = chunk_tile(ntiles, tiles_chunked(ntiles));
  TileSums t{0.0, 0.0};
  if (tile < ntiles)
    t = cg_update_tile<N1, TV, V>(b, tile, z, w, minv, sc, sA, sred, (int)threadIdx.x);
  if (threadIdx.x == 0) {
    part_rr[tile] = t.a;
    part_rz[tile] = t.b;
  }
}

// The update on the default tile with z written by non-temporal stores
// (upd_streams_z), for vectors larger than the last-level cache.
template <int N1, typename TV>
__global__ void __launch_bounds__((UpdTile<N1, TV>::BLOCK))
    cg_update_stream_kernel(Box b, int64_t ntiles, TV *__restrict__ z, const TV *__restrict__ w,
                            const TV *__restrict__ minv, CgState *__restrict__ st,
                            double *__restrict__ part_rr, double *__restrict__ part_rz) {
  __shared__ double sred[2 * (UpdTile<N1, TV>::BLOCK / 64)];
  __shared__ double sA[UpdTile<N1, TV>::LDS];
  if (st->done) return;
  const GivenScalars sc{st->alpha, 0.0};
  const int64_t tile = chunk_tile(ntiles, tiles_chunked(ntiles));
  if (tile >= ntiles) return;
  const TileSums t = cg_update_tile<N1, TV, 0, true>(b, tile, z, w, minv, sc, sA, sred, (int)threadIdx.x);
  if (threadIdx.x == 0) {
    part_rr[tile] = t.a;
    part_rz[tile] = t.b;
  }
}

// The CG update of a folded iteration (cg_folded), on the default tile: the
// alpha step from the operator's n_op partials part_pap inside.
template <int N1, typename TV>
__global__ void __launch_bounds__((UpdTile<N1, TV>::BLOCK))
    cg_update_fold_kernel(Box b, int64_t ntiles, TV *__restrict__ z, const TV *__restrict__ w,
                          const TV *__restrict__ minv, CgState *__restrict__ st,
                          double *__restrict__ part_rr, double *__restrict__ part_rz,
                          const double *__restrict__ part_pap, int n_op) {
  constexpr int W = UpdTile<N1, TV>::BLOCK / 64;
  __shared__ double sred[2 * W];
  __shared__ double sfold[kFinGroup / 64];  // not sred: no barrier follows its last read
  __shared__ double sA[UpdTile<N1, TV>::LDS];
  const int64_t tile = chunk_tile(ntiles, tiles_chunked(ntiles));
  if (tile >= ntiles) return;
  const FoldAlpha<W> sc(st, part_pap, n_op, sfold);
  const TileSums t = cg_update_tile<N1, TV>(b, tile, z, w, minv, sc, sA, sred, (int)threadIdx.x);
  if (threadIdx.x == 0) {
    part_rr[tile] = t.a;
    part_rz[tile] = t.b;
  }
}

// ------------------------------------------------------------ setup helpers
template <int N1>
__global__ void __launch_bounds__(kVecThreads)
    fill_c_kernel(Box b, int64_t L, double *__restrict__ c) {
  const int64_t base = (int64_t)blockIdx.x * kVecTile + threadIdx.x;
#pragma unroll
  for (int u = 0; u < kVecItems; ++u) {
    const int64_t idx = base + (int64_t)u * kVecThreads;
    if (idx < L) c[idx] = node_at<N1>(b, idx).inv_mult();
  }
}

}  // namespace semk
