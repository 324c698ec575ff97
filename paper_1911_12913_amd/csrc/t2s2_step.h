// Device helpers shared by the step kernels (t2s2_kernels.hip, t2s2_pair.hip):
// row weights, stencil taps, the pointwise maps and the wall pass.  Internal
// linkage (anonymous namespace) in every translation unit that includes it.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "t2s2_device.h"
#include "t2s2_internal.h"

namespace t2s2 {
namespace {

// The row weights are the same for the whole wave: read them through the
// constant address space at a wave-uniform index so they become scalar loads
// (counted by lgkmcnt).  A vector load here would be waited for with the
// in-order vmcnt counter and so drain the row prefetches in flight.
template <typename Real>
__device__ inline void row_weights(const Real* table, int row, Real out[kWeightsPerNode]) {
  using CPtr = const __attribute__((address_space(4))) Real*;
  const int r = __builtin_amdgcn_readfirstlane(row);
  CPtr w = (CPtr)(table) + r * kWeightsPerNode;
#pragma unroll
  for (int k = 0; k < kWeightsPerNode; ++k) out[k] = w[k];
}


// Element at a 32-bit byte offset from a plane base: the row offset is
// formed once per row in 32 bits and shared by the nine planes.  Every
// population plane is under 4 GiB (checked when the context is created).
template <typename T>
__device__ inline const T* at_byte(const T* base, unsigned boff) {
  return reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + boff);
}
template <typename T>
__device__ inline T* at_byte(T* base, unsigned boff) {
  return reinterpret_cast<T*>(reinterpret_cast<char*>(base) + boff);
}

// The nine new values of one interior node at byte offset boff of each
// plane: rounded to nearest even, or, for the stochastic forms, by
// round_node_sr with the node's offset as its position.  FP64 rows (448
// bytes per wave) go out as non-temporal (streaming) stores: the state is
// not read again in this launch, and they reach HBM faster than write-back
// stores.  The narrower FP32 and 16-bit rows (224 and 112 bytes, not
// line-aligned) merge better in L2 and use ordinary stores (measured: FP32
// 5% faster so).
template <typename Store>
__device__ inline void store_node(Store* dst, long long plane, unsigned boff,
                                  const typename Cvt<Store>::R (&out)[kQ]) {
  constexpr bool kNt = std::is_same<Store, double>::value;
  Store r[kQ];
  if constexpr (kStochastic<Store>) {
    round_node_sr(out, boff, r);
  } else {
#pragma unroll
    for (int q = 0; q < kQ; ++q) r[q] = Cvt<Store>::st(out[q]);
  }
  store_planes<kNt>(dst, plane * sizeof(Store), boff, r);
}

// LDS rows that serve y taps hold the populations with xi_y != 0 only:
// population q is their slot y_slot(q).
constexpr int kYMoving = 6;
__device__ constexpr int y_slot(int q) {
  int n = 0;
  for (int k = 0; k < q; ++k) n += ey_of(k) != 0 ? 1 : 0;
  return n;
}

// Row index brought into [0, n) by whole periods; the rows a piece touches
// lie within a few rows of the grid, so this loops at most a few times.
__device__ inline int wrap_near(int i, int n) {
  while (i < 0) i += n;
  while (i >= n) i -= n;
  return i;
}

// acc + sum_k w[k] v(lane + offset_k) for the 4 taps of the mixed difference
// along x: offsets (-2,-1,0,+1) for a positive velocity component (sx = 0),
// (-1,0,+1,+2) for a negative one (sx = 1); the neighbours come from the
// centre values of the other lanes.
template <int sx, bool kExact = true, typename Real>
__device__ inline Real x_taps(const Real* w, Real centre, Real acc) {
  const Real m1 = from_below(centre), p1 = from_above(centre);
  if (sx == 0) {
    const Real m2 = from_below(m1);
    acc = fma_of<kExact>(w[0], m2, acc);
    acc = fma_of<kExact>(w[1], m1, acc);
    acc = fma_of<kExact>(w[2], centre, acc);
    acc = fma_of<kExact>(w[3], p1, acc);
  } else {
    const Real p2 = from_above(p1);
    acc = fma_of<kExact>(w[4], m1, acc);
    acc = fma_of<kExact>(w[5], centre, acc);
    acc = fma_of<kExact>(w[6], p1, acc);
    acc = fma_of<kExact>(w[7], p2, acc);
  }
  return acc;
}

// A row in LDS, typed as such: a choice between two LDS arrays otherwise
// reaches the instruction selector as a generic pointer and is read with
// flat loads.
template <typename Real>
using LdsPtr = const __attribute__((address_space(3))) Real*;

// Base of the full step plus the stencil of R at direction q,
// the y taps being the rows o-2 .. o+1 (positive y velocity) or o-1 .. o+2
// (negative) in row[k], k = 0..3.  FP64 sums in the order in which the
// two-step kernel, which adds each R row to the outputs around it, meets the
// terms: the rows above, the row itself (the x taps first), the rows below.
// FP32 takes the x taps first.
// x(acc): acc plus the x taps.
template <bool kExact = true, typename Real, typename Row, typename X>
__device__ __forceinline__ Real full_taps_of(int q, const Real* wy, Real acc,
                                             Row row, X x) {
  const int sy = ey_of(q) > 0 ? 0 : 1;
  if constexpr (sizeof(Real) == 4) {
    acc = x(acc);
    if (ey_of(q) != 0) {
#pragma unroll
      for (int k = 0; k < kTaps; ++k) acc = fma_of<kExact>(wy[sy * kTaps + k], row(k), acc);
    }
    return acc;
  }
  // Rows above the centre row: two for a positive y velocity, one otherwise.
  const int above = sy == 0 ? 2 : 1;
  if (ey_of(q) != 0) {
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (k < above) acc = fma_of(wy[sy * kTaps + k], row(k), acc);
  }
  acc = x(acc);
  if (ey_of(q) != 0) {
#pragma unroll
    for (int k = 1; k < kTaps; ++k)
      if (k >= above) acc = fma_of(wy[sy * kTaps + k], row(k), acc);
  }
  return acc;
}
template <bool kExact = true, typename Real, typename Row>
__device__ __forceinline__ Real full_taps(int q, const Real* wx, const Real* wy, Real centre,
                                          Real acc, Row row) {
  return full_taps_of<kExact>(q, wy, acc, row, [&](Real a) {
    if (ex_of(q) > 0) a = x_taps<0, kExact>(wx, centre, a);
    if (ex_of(q) < 0) a = x_taps<1, kExact>(wx, centre, a);
    return a;
  });
}

// Guo force term (eq 3.12) of direction q from E = (f^eq_q - w_q) / w_q:
// F_q = 3 (F . (xi_q - u)) f^eq_q with f^eq_q = w_q (1 + E).
template <bool kExact = true, typename Real>
__device__ inline Real force_term(int q, const StepParams& p, Real ux, Real uy, Real E) {
  const Real fu = fma_of<kExact>(static_cast<Real>(p.Fx), Real(ex_of(q)) - ux,
                         static_cast<Real>(p.Fy) * (Real(ey_of(q)) - uy));
  return Real(3.0 * w_of(q)) * fu * (Real(1) + E);
}

// Wall nodes of the new state (eq 3.10),
//   f~_b = f~_f + f^eq(rho_f, u_b) - f^eq(rho_f, u_f),
// from the moments of the stored new state at the nearest interior node f
// (diagonal at the corners), u_f with the force shift of eq 3.3.  Run by a
// strip's threads after its piece [y0, y1) has been marched and the block
// has passed a barrier: the sources are the nodes next to a wall among the
// piece's outputs (columns [x0, x1)), which this block has just stored, so
// the loads see them (the coherence point is L2; the buffer was not read
// earlier in the launch).  Each wall node has exactly one source node, and
// each source node is output by exactly one piece.  wall_u(c, r, side, u, v):
// the velocity of the wall's node (c, r).  kLoadsFirst keeps the conversions of
// the 16-bit forms behind all nine loads, where step_kernel otherwise takes
// them one by one and each load waits out a round trip (BF16 T2S2-FDLBM2 cavity
// 23 x 215, 20.5 us per step, 19.1 so).
template <bool kExact, bool kLoadsFirst, typename Store, typename WallU>
__device__ inline void piece_walls(const StepParams& p, Store* dst, int x0, int x1, int y0,
                                   int y1, int tid, int nthreads, WallU wall_u) {
  using Real = typename Cvt<Store>::R;
  const int nx = p.nx, ny = p.ny;
  // Interior output columns and rows of this strip-piece.
  const int cx0 = p.per_x ? x0 : max(x0, 1), cx1 = p.per_x ? x1 : min(x1, nx - 1);
  const int ry0 = p.per_y ? y0 : max(y0, 1), ry1 = p.per_y ? y1 : min(y1, ny - 1);
  if (cx0 >= cx1 || ry0 >= ry1) return;
  // Sources: (a) the rows next to the bottom and top walls, every column;
  // (b) the columns next to the left and right walls, the other rows.
  const bool rb = !p.per_y && ry0 <= 1 && 1 < ry1;
  const bool rt = !p.per_y && ry0 <= ny - 2 && ny - 2 < ry1;
  const bool cl = !p.per_x && cx0 <= 1 && 1 < cx1;
  const bool cr = !p.per_x && cx0 <= nx - 2 && nx - 2 < cx1;
  const int ncol = cx1 - cx0;
  const int nrow_a = (rb ? 1 : 0) + (rt ? 1 : 0);
  const int nrows_b = (ry1 - ry0) - nrow_a;  // rows not already in (a)
  const int nsrc = nrow_a * ncol + ((cl ? 1 : 0) + (cr ? 1 : 0)) * nrows_b;
#pragma unroll 1
  for (int k = tid; k < nsrc; k += nthreads) {
    int i, j;
    if (k < nrow_a * ncol) {
      j = (k < ncol && rb) ? 1 : ny - 2;
      i = cx0 + k % ncol;
    } else {
      const int kb = k - nrow_a * ncol;
      i = (kb < nrows_b && cl) ? 1 : nx - 2;
      // The (kb mod nrows_b)-th row of [ry0, ry1) other than rows 1 and
      // ny - 2 when those are in (a): row 1 is then ry0, row ny - 2 is ry1 - 1.
      j = ry0 + (rb ? 1 : 0) + kb % nrows_b;
    }
    const long long fb = static_cast<long long>(j) * p.pitch + i;
    Real v[kQ];
    if constexpr (kLoadsFirst) {
      Store raw[kQ];
#pragma unroll
      for (int q = 0; q < kQ; ++q) raw[q] = dst[q * p.plane + fb];
      __builtin_amdgcn_sched_barrier(0x4);
#pragma unroll
      for (int q = 0; q < kQ; ++q) v[q] = Cvt<Store>::ld(raw[q]);
    } else {
#pragma unroll
      for (int q = 0; q < kQ; ++q) v[q] = Cvt<Store>::ld(dst[q * p.plane + fb]);
    }
    double s, jx, jy;
    moment_sums(v, s, jx, jy);
    const double rho = 1.0 + s;
    const double ir = recip(rho);
    const double ux = fma_of<kExact>(jx, ir, p.half_dt * p.Fx);
    const double uy = fma_of<kExact>(jy, ir, p.half_dt * p.Fy);
    const bool wl = !p.per_x && i == 1, wr = !p.per_x && i == nx - 2;
    const bool wb = !p.per_y && j == 1, wt = !p.per_y && j == ny - 2;
#pragma unroll 1
    for (int dy = -1; dy <= 1; ++dy) {
      if ((dy == -1 && !wb) || (dy == 1 && !wt)) continue;
#pragma unroll 1
      for (int dx = -1; dx <= 1; ++dx) {
        if ((dx == -1 && !wl) || (dx == 1 && !wr)) continue;
        if (dx == 0 && dy == 0) continue;
        double ub, vb;
        wall_u(i + dx, j + dy, wall_side_of(dx, dy), ub, vb);
        Real sh[kQ];
        nee_shift<kExact>(rho, ux, uy, ub, vb, sh);
        const long long wo = static_cast<long long>(j + dy) * p.pitch + (i + dx);
#pragma unroll
        for (int q = 0; q < kQ; ++q) dst[q * p.plane + wo] = Cvt<Store>::st(v[q] + sh[q]);
      }
    }
  }
}

}  // namespace
}  // namespace t2s2
