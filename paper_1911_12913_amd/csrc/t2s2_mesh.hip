// Steps of the T2S2-FDLBM1 family (A > 0) on meshes of at most kMeshNodes
// nodes: one block holds the whole mesh, one node per thread, and takes all
// the steps of a launch without leaving the CU.  P and R live in LDS, the
// state in registers; memory is read once at the start and written once at
// the end.  A launch per step costs such a mesh 6 to 9 us, nearly all of it
// the launch, the first loads and the last stores; a step here costs its
// arithmetic and two barriers (three with walls).  Each node takes the
// expressions of step_kernel, in its order; the state between two steps is
// rounded to the storage type as if it had been stored.
#include <hip/hip_runtime.h>

#include "t2s2_device.h"
#include "t2s2_internal.h"
#include "t2s2_step.h"

namespace t2s2 {
namespace {

// acc + the x taps of x_taps, the neighbours read from LDS: v(o) is the
// value at offset o along x.
template <bool kExact, typename Real, typename V>
__device__ __forceinline__ Real x_taps_at(int ex, const Real* w, Real centre, Real acc, V v) {
  if (ex > 0) {
    acc = fma_of<kExact>(w[0], v(-2), acc);
    acc = fma_of<kExact>(w[1], v(-1), acc);
    acc = fma_of<kExact>(w[2], centre, acc);
    acc = fma_of<kExact>(w[3], v(1), acc);
  } else if (ex < 0) {
    acc = fma_of<kExact>(w[4], v(-1), acc);
    acc = fma_of<kExact>(w[5], centre, acc);
    acc = fma_of<kExact>(w[6], v(1), acc);
    acc = fma_of<kExact>(w[7], v(2), acc);
  }
  return acc;
}

// kNodes: the largest mesh of the instantiation (and its threads per block):
// half the nodes leave each thread twice the registers, and FP64 then holds
// everything without spilling.
template <typename Store, bool kForce, bool kWalls, int kNodes>
__global__ __launch_bounds__(kNodes) void mesh_steps_kernel(StepParams p, int nsteps) {
  using Real = typename Cvt<Store>::R;
  constexpr bool kExact = kExactOf<Real, kForce>;
  __shared__ Real tP[kQ * kNodes];  // [q][node]
  __shared__ Real tR[kQ * kNodes];
  const int nx = p.nx, ny = p.ny;
  const int node = threadIdx.x;
  const bool on = node < nx * ny;  // the last wave's other threads idle along
  const int c = on ? node % nx : 0, r = on ? node / nx : 0;
  const bool interior =
      on && (p.per_x || (c >= 1 && c <= nx - 2)) && (p.per_y || (r >= 1 && r <= ny - 2));
  const bool per_x = !kWalls || p.per_x, per_y = !kWalls || p.per_y;
  // Nodes at the offsets -2 .. 2 along each axis (past a wall: clamped; the
  // weight is zero there).
  int ix[5], iy[5];
#pragma unroll
  for (int o = -2; o <= 2; ++o) {
    ix[o + 2] = r * nx + (per_x ? wrap(c + o, nx) : clampi(c + o, 0, nx - 1));
    iy[o + 2] = (per_y ? wrap(r + o, ny) : clampi(r + o, 0, ny - 1)) * nx + c;
  }
  Real wx[kWeightsPerNode], wy[kWeightsPerNode];
#pragma unroll
  for (int k = 0; k < kWeightsPerNode; ++k) {
    wx[k] = weights_x<Real>(p)[c * kWeightsPerNode + k];
    wy[k] = weights_y<Real>(p)[r * kWeightsPerNode + k];
  }
  const unsigned boff = (static_cast<unsigned>(r) * static_cast<unsigned>(p.pitch) +
                         static_cast<unsigned>(c)) *
                        static_cast<unsigned>(sizeof(Store));
  Store gs[kQ];
  if (on) load_planes(static_cast<const Store*>(p.src), p.plane * sizeof(Store), boff, gs);
  Real g[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) g[q] = on ? Cvt<Store>::ld(gs[q]) : Real(0);

  const auto& k = coef<Real>(p);
  const bool src_xl = kWalls && interior && !p.per_x && c == 1;
  const bool src_xr = kWalls && interior && !p.per_x && c == nx - 2;
  const bool src_yb = kWalls && interior && !p.per_y && r == 1;
  const bool src_yt = kWalls && interior && !p.per_y && r == ny - 2;
  // Calls f(dx, dy, node) for each wall node whose nearest interior node is
  // this one.
  auto each_wall_node = [&](auto f) {
    if (!(src_xl || src_xr || src_yb || src_yt)) return;
    for (int dy = -1; dy <= 1; ++dy) {
      if ((dy == -1 && !src_yb) || (dy == 1 && !src_yt)) continue;
      for (int dx = -1; dx <= 1; ++dx) {
        if ((dx == -1 && !src_xl) || (dx == 1 && !src_xr)) continue;
        if (dx == 0 && dy == 0) continue;
        f(dx, dy, node + dy * nx + dx);
      }
    }
  };

  for (int step = 0; step < nsteps; ++step) {
    // ---- P (to LDS) and Q of every node.
    Real Q[kQ];
    Real Pown[kQ];
    {
      double s, jx, jy;
      moment_sums(g, s, jx, jy);
      Real rho, ux, uy;
      if constexpr (kForce)
        forced_velocity<kExact>(s, jx, jy, p.half_dt, p.Fx, p.Fy, rho, ux, uy);
      else
        velocity<kExact>(s, jx, jy, rho, ux, uy);
      const Real d = static_cast<Real>(s);
      Real X[kQ];
      eq_brackets<kExact>(ux, uy, X);
#pragma unroll
      for (int q = 0; q < kQ; ++q) {
        const Real E = fma_of<kExact>(rho, X[q], d);
        Real Pq = fma_of<kExact>(k.cPg, g[q], k.kP[wclass(q)] * E);
        Real Qq = fma_of<kExact>(k.cQg, g[q], k.kQ[wclass(q)] * E);
        if (kForce) {
          const Real Fq = force_term<kExact>(q, p, ux, uy, E);
          Pq = fma_of<kExact>(static_cast<Real>(p.cPF), Fq, Pq);
          Qq = fma_of<kExact>(static_cast<Real>(p.cQF), Fq, Qq);
        }
        Pown[q] = Pq;
        Q[q] = Qq;
        tP[q * kNodes + node] = Pq;
      }
    }
    __syncthreads();

    // ---- S and R of the interior nodes, R to LDS, also of the wall nodes
    // next to them (eq 3.10).
    Real R[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) R[q] = Real(0);
    if (interior) {
      Real S[kQ];
#pragma unroll
      for (int q = 0; q < kQ; ++q) {
        const Real* t = tP + q * kNodes;
        const Real centre = Pown[q];
        Real acc = x_taps_at<kExact>(ex_of(q), wx, centre, Real(0), [&](int o) { return t[ix[o + 2]]; });
        if (ey_of(q) != 0) {
          const int sy = ey_of(q) > 0 ? 0 : 1;
#pragma unroll
          for (int k2 = 0; k2 < kTaps; ++k2) {
            const int o = k2 + sy;
            acc = fma_of<kExact>(wy[sy * kTaps + k2], o == 2 ? centre : t[iy[o]], acc);
          }
        }
        S[q] = q == 0 ? centre : fma_of<kExact>(k.A, acc, centre);
      }
      double s, jx, jy;
      moment_sums(S, s, jx, jy);
      Real rho, ux, uy;
      if constexpr (kForce)
        forced_velocity<kExact>(s, jx, jy, p.half_h, p.Fx, p.Fy, rho, ux, uy);
      else
        velocity<kExact>(s, jx, jy, rho, ux, uy);
      const Real d = static_cast<Real>(s);
      Real X[kQ];
      eq_brackets<kExact>(ux, uy, X);
#pragma unroll
      for (int q = 1; q < kQ; ++q) {
        const Real E = fma_of<kExact>(rho, X[q], d);
        Real Rq = fma_of<kExact>(k.cRs, S[q], k.kR[wclass(q)] * E);
        if (kForce) Rq = fma_of<kExact>(static_cast<Real>(p.cRF), force_term<kExact>(q, p, ux, uy, E), Rq);
        R[q] = Rq;
        tR[q * kNodes + node] = Rq;
      }
      if (kWalls) {
        const Real r1 = Real(w_of(1)) * rho, r2 = Real(w_of(5)) * rho;
        each_wall_node([&](int dx, int dy, int wall) {
          const Real* Xb = wall_brackets<Real>(p, wall_side_of(dx, dy));
#pragma unroll
          for (int q = 1; q < kQ; ++q)
            tR[q * kNodes + wall] = nee_r<kExact>(wclass(q) == 1 ? r1 : r2, X[q], Xb[q], R[q]);
        });
      }
    }
    __syncthreads();

    // ---- The new state of the interior nodes, as stored; then, through LDS
    // (P is no longer read), the wall nodes'.
    if (interior) {
      Real out[kQ];
      out[0] = Q[0];
#pragma unroll
      for (int q = 1; q < kQ; ++q) {
        const Real* t = tR + q * kNodes;
        const int sy = ey_of(q) > 0 ? 0 : 1;
        Real x[5], rows[kTaps] = {};
        x[2] = R[q];
        if (ex_of(q) != 0) {
          x[1] = t[ix[1]];
          x[3] = t[ix[3]];
          if (ex_of(q) > 0) x[0] = t[ix[0]];
          if (ex_of(q) < 0) x[4] = t[ix[4]];
        }
        if (ey_of(q) != 0) {
#pragma unroll
          for (int k2 = 0; k2 < kTaps; ++k2) rows[k2] = k2 + sy == 2 ? R[q] : t[iy[k2 + sy]];
        }
        out[q] = full_taps_of<kExact>(
            q, wy, Q[q], [&](int k2) { return rows[k2]; },
            [&](Real acc) {
              return x_taps_at<kExact>(ex_of(q), wx, R[q], acc, [&](int o) { return x[o + 2]; });
            });
      }
      if constexpr (kStochastic<Store>) {
        round_node_sr(out, boff, gs);
      } else {
#pragma unroll
        for (int q = 0; q < kQ; ++q) gs[q] = Cvt<Store>::st(out[q]);
      }
#pragma unroll
      for (int q = 0; q < kQ; ++q) g[q] = Cvt<Store>::ld(gs[q]);
    }
    if (kWalls) {
      each_wall_node([&](int dx, int dy, int wall) {
        double s, jx, jy;
        moment_sums(g, s, jx, jy);
        const double rho = 1.0 + s;
        const double ir = recip(rho);
        const double ux = fma_of<kExact>(jx, ir, p.half_dt * p.Fx);
        const double uy = fma_of<kExact>(jy, ir, p.half_dt * p.Fy);
        double ub, vb;
        wall_velocity(p, c + dx, r + dy, ub, vb);
        Real sh[kQ];
        nee_shift<kExact>(rho, ux, uy, ub, vb, sh);
#pragma unroll
        for (int q = 0; q < kQ; ++q)
          tP[q * kNodes + wall] = Cvt<Store>::ld(Cvt<Store>::st(g[q] + sh[q]));
      });
      __syncthreads();
      if (on && !interior) {
#pragma unroll
        for (int q = 0; q < kQ; ++q) g[q] = tP[q * kNodes + node];
      }
    }
  }
  if (on) {
    // Exact: g holds stored values.
#pragma unroll
    for (int q = 0; q < kQ; ++q) gs[q] = Cvt<Store>::st(g[q]);
    store_planes<false>(static_cast<Store*>(p.dst), p.plane * sizeof(Store), boff, gs);
  }
}

template <typename Store, int kNodes>
hipError_t launch_mesh_n(const StepParams& p, int nsteps, hipStream_t s) {
  const dim3 b((p.nx * p.ny + kLanes - 1) / kLanes * kLanes);
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(1), b, 0, s, p, nsteps); };
  // The forms that a plan selects (plan_mesh): FP64 with a force on the smaller
  // blocks only, the reduced forms with walls only.
  constexpr bool kFp64 = std::is_same<Store, double>::value;
  const bool walls = !p.per_x || !p.per_y;
  if (p.has_force) {
    if constexpr (kFp64 && kNodes > kMeshNodes / 2) return hipErrorInvalidValue;
    else if (walls) go(mesh_steps_kernel<Store, true, true, kNodes>);
    else if constexpr (kFp64) go(mesh_steps_kernel<Store, true, false, kNodes>);
    else return hipErrorInvalidValue;
  } else {
    if (walls) go(mesh_steps_kernel<Store, false, true, kNodes>);
    else if constexpr (kFp64) go(mesh_steps_kernel<Store, false, false, kNodes>);
    else return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
template <typename Store>
hipError_t launch_mesh_t(const StepParams& p, int nsteps, hipStream_t s) {
  return p.nx * p.ny <= kMeshNodes / 2 ? launch_mesh_n<Store, kMeshNodes / 2>(p, nsteps, s)
                                       : launch_mesh_n<Store, kMeshNodes>(p, nsteps, s);
}

}  // namespace

hipError_t launch_mesh_steps(int storage, const StepParams& p, int nsteps, hipStream_t s) {
  switch (storage) {
    case kF64: return launch_mesh_t<double>(p, nsteps, s);
    case kF32: return launch_mesh_t<float>(p, nsteps, s);
    case kBF16: return launch_mesh_t<Bf16>(p, nsteps, s);
    case kF16: return launch_mesh_t<_Float16>(p, nsteps, s);
    case kBF16Sr: return launch_mesh_t<Bf16Sr>(p, nsteps, s);
    case kF16Sr: return launch_mesh_t<F16Sr>(p, nsteps, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace t2s2
