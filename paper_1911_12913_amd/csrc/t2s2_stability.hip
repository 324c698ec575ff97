// Von Neumann stability maps of the T2S2-FDLBM (Sec. 2C, eqs 4.1-4.8).
//
// For each (omega, r) point of a map, the largest spectral radius over a
// grid of modes k of the growth matrix G(k) (9 x 9, complex) of a
// perturbation f' e^{i k.x} about the uniform equilibrium f^eq(1, u):
//   model 0 (eq 4.7): G = lhs^{-1} rhs for the (B~2, B-2) family, with
//     lhs = (1 + w B-2) I + w (1/2 - 2 B-2) Gamma + rS (B~2 I + (1/2 - B~2) Gamma)
//     rhs = (1 - w (1 - B-2)) I + w (3/2 - 2 B-2) Gamma
//           - rS ((1 - B~2) I - (1/2 - B~2) Gamma);
//   model 1: the exact linearisation of the implemented eq 2.23 step (h = A
//     dt):  G = J_Q - rS J_R (I - A rS) J_P;
//   model 2: the exact linearisation of the eq 5.23 step:
//     G = J_Q - (rS/2) (J_f + J_R1 (I - rS) J_Q);
//   model 3: the exact linearisation of the eq 2.13 family step:
//     G = J_Q - rS (b0 J_f + b1 J_R (I - A rS) J_P + b2 J_R1 (I - rS) J_Q);
//     with collision weights (B-0, B-1, B-2) other than (1/2, 0, 1/2)
//     (dt Omega(f) = w (Gamma - I) f, unforced):
//     Y = J_f + w (Gamma - I) (B-0 J_f + B-1 J_R (I - A rS) J_P)
//         - rS (b0 J_f + b1 J_R (I - A rS) J_P + b2 J_R1 (I - rS) J_Q),
//     G = (aY I + aE Gamma) Y with aY = (1 + w/2) / (1 + B-2 w) and
//     aE = w (B-2 - 1/2) / (1 + B-2 w): the implicit weight solved (Gamma
//     is a projection, Gamma^2 = Gamma: f^eq keeps the moments it is built
//     from) and the state taken as f~ = f - (dt/2) Omega(f) (eq 2.19);
// with Gamma = d f^eq / d f, J_X = c_Xg I + c_Xe Gamma, and S the symbol of
// dx xi_q . D of the mixed difference (eq 4.8, imaginary unit restored in
// the exponentials).  The advection symbol multiplies from the left (it
// acts on the population it advects).
//
// The spectral radius is lim ||G^m||^(1/m), taken at m = 2^J by J squarings
// in FP64, the matrix scaled by powers of two (exact) as it goes.
//
// A block is one wave that takes every nchunks-th mode of one map point, 21
// modes at a time: three lanes per mode, three rows of its matrix in the
// registers of each, and a copy of the matrix in LDS whose elements the three
// lanes read together, so each 16-byte LDS read feeds 12 multiply-adds per
// lane and the squaring is bound by the FP64 units.  A mode stops as soon as
// it cannot be the largest: rho(G) <= ||G^n||_F^(1/n) for every n, so once
// that bound at n = 2^s lies below a radius already found at this point
// (|k| = 0 goes first, and other blocks' results are read), the rest of its
// squarings cannot change the maximum.  Measured, 30 squarings x 561
// modes, one wave per point and every squaring before -> now: the step's
// models 23.3 -> 0.80 ms (256 points), 24.5 -> 1.85 ms (1024); eq 4.7, whose
// elimination takes the whole wave per mode, 27.0 -> 2.4 and 28.4 -> 6.9 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "t2s2_device.h"
#include "t2s2_internal.h"

namespace t2s2 {
namespace {

struct cplx {
  double re, im;
};
__device__ inline cplx cadd(cplx a, cplx b) { return {a.re + b.re, a.im + b.im}; }
__device__ inline cplx csub(cplx a, cplx b) { return {a.re - b.re, a.im - b.im}; }
__device__ inline cplx cmul(cplx a, cplx b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ inline cplx cscale(cplx a, double s) { return {a.re * s, a.im * s}; }
__device__ inline double cabs2(cplx a) { return a.re * a.re + a.im * a.im; }
__device__ inline cplx cdiv(cplx a, cplx b) {
  const double d = cabs2(b);
  return {(a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d};
}

constexpr int kN = 9, kN2 = 81;
constexpr int kWantedBlocks = 2560;

// Gamma_ij = d f^eq_i / d f_j at rho = 1, velocity u (eq 3.2, c_s^2 = 1/3):
// f^eq depends on f through rho = sum f and m = sum xi f.
__device__ inline double gamma_ij(int i, int j, double ux, double uy) {
  const double exi = ex_of(i), eyi = ey_of(i), wi = w_of(i);
  const double eu = exi * ux + eyi * uy, uu = ux * ux + uy * uy;
  const double d_rho = wi * (1.0 - 4.5 * eu * eu + 1.5 * uu);
  const double d_mx = wi * (3.0 * exi + 9.0 * eu * exi - 3.0 * ux);
  const double d_my = wi * (3.0 * eyi + 9.0 * eu * eyi - 3.0 * uy);
  return d_rho + d_mx * ex_of(j) + d_my * ey_of(j);
}

constexpr int kLanesPerMode = 3, kModes = kLanes / kLanesPerMode;  // 21 modes per wave
constexpr int kRowsPerLane = kN / kLanesPerMode;

// One pass over the (up to two) matrix elements e = lane, lane + 64 of a
// 9 x 9 matrix.
template <typename F>
__device__ inline void for_elems(int lane, F f) {
  f(lane / kN, lane % kN);
  if (lane + 64 < kN2) f((lane + 64) / kN, (lane + 64) % kN);
}

// dx * symbol of xi_q . D, mixed difference with upwind weight eta, from the
// sines and cosines of the mode's angles.
__device__ inline cplx symbol_q(int q, const double (&sn)[2], const double (&cs)[2], double eta) {
  cplx s{0.0, 0.0};
  const int e[2] = {ex_of(q), ey_of(q)};
  for (int a = 0; a < 2; ++a) {
    const double si = e[a] * sn[a], co = e[a] == 0 ? 1.0 : cs[a];
    const double s2 = 2.0 * si * co, c2 = 1.0 - 2.0 * si * si;
    s.im += (1.0 - eta) * si;
    s.re += 0.5 * eta * (3.0 - 4.0 * co + c2);
    s.im += 0.5 * eta * (4.0 * si - s2);
  }
  return s;
}

// Eq 4.7: G = lhs^{-1} rhs by Gauss-Jordan elimination with partial
// pivoting, the whole wave on one mode; G is left in T.
__device__ inline void solve_paper(const StabArgs& a, int lane, const double* gam,
                                   const cplx* sym, double w, double r, cplx* X, cplx* T) {
  const double b2 = a.b2bar, bt = a.b2tilde;
  for_elems(lane, [&](int i, int j) {
    const double d = i == j ? 1.0 : 0.0, g = gam[i * kN + j];
    const cplx rs = cscale(sym[i], r);
    X[i * kN + j] = cadd({(1 + w * b2) * d + w * (0.5 - 2 * b2) * g, 0.0},
                         cscale(rs, bt * d + (0.5 - bt) * g));
    T[i * kN + j] = csub({(1 - w * (1 - b2)) * d + w * (1.5 - 2 * b2) * g, 0.0},
                         cscale(rs, (1 - bt) * d - (0.5 - bt) * g));
  });
  __syncthreads();
  for (int c = 0; c < kN; ++c) {
    int piv = c;
    double pmax = cabs2(X[c * kN + c]);
    for (int i = c + 1; i < kN; ++i) {
      const double v = cabs2(X[i * kN + c]);
      if (v > pmax) {
        pmax = v;
        piv = i;
      }
    }
    __syncthreads();
    if (lane < kN && piv != c) {
      const cplx x0 = X[c * kN + lane], t0 = T[c * kN + lane];
      X[c * kN + lane] = X[piv * kN + lane];
      T[c * kN + lane] = T[piv * kN + lane];
      X[piv * kN + lane] = x0;
      T[piv * kN + lane] = t0;
    }
    __syncthreads();
    const cplx p = X[c * kN + c];
    __syncthreads();
    if (lane < kN) {
      X[c * kN + lane] = cdiv(X[c * kN + lane], p);
      T[c * kN + lane] = cdiv(T[c * kN + lane], p);
    }
    __syncthreads();
    cplx fac[2], xr[2], tr[2];
    int n = 0;
    for_elems(lane, [&](int i, int j) {
      fac[n] = X[i * kN + c];
      xr[n] = X[c * kN + j];
      tr[n] = T[c * kN + j];
      ++n;
    });
    __syncthreads();
    n = 0;
    for_elems(lane, [&](int i, int j) {
      if (i != c) {
        X[i * kN + j] = csub(X[i * kN + j], cmul(fac[n], xr[n]));
        T[i * kN + j] = csub(T[i * kN + j], cmul(fac[n], tr[n]));
      }
      ++n;
    });
    __syncthreads();
  }
}

using Rows = cplx[kRowsPerLane][kN];

// The lane's rows of a matrix to its mode's LDS copy, for the other lanes.
// (The fences keep the compiler from moving other lanes' reads across; the
// block is one wave, so they cost nothing else.)
__device__ __forceinline__ void publish(cplx* m, int row0, const Rows& x) {
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRowsPerLane; ++r) {
#pragma unroll
    for (int j = 0; j < kN; ++j) m[(row0 + r) * kN + j] = x[r][j];
  }
  __syncthreads();
}

// The lane's rows of Gamma M, M in LDS.
__device__ __forceinline__ void gamma_times(const double* gam, const cplx* m, int row0, Rows& out) {
#pragma unroll
  for (int r = 0; r < kRowsPerLane; ++r) {
#pragma unroll
    for (int j = 0; j < kN; ++j) out[r][j] = {0.0, 0.0};
  }
#pragma unroll 1
  for (int k = 0; k < kN; ++k) {
    double g[kRowsPerLane];
#pragma unroll
    for (int r = 0; r < kRowsPerLane; ++r) g[r] = gam[(row0 + r) * kN + k];
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      const cplx b = m[k * kN + j];
#pragma unroll
      for (int r = 0; r < kRowsPerLane; ++r) {
        out[r][j].re = fma(g[r], b.re, out[r][j].re);
        out[r][j].im = fma(g[r], b.im, out[r][j].im);
      }
    }
  }
}

// The lane's rows of X M, X the lane's rows of M and M in LDS.
__device__ __forceinline__ void square(const cplx* m, const Rows& x, Rows& out) {
#pragma unroll
  for (int r = 0; r < kRowsPerLane; ++r) {
#pragma unroll
    for (int j = 0; j < kN; ++j) out[r][j] = {0.0, 0.0};
  }
#pragma unroll
  for (int k = 0; k < kN; ++k) {
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      const cplx b = m[k * kN + j];
#pragma unroll
      for (int r = 0; r < kRowsPerLane; ++r) {
        out[r][j].re = fma(x[r][k].re, b.re, out[r][j].re);
        out[r][j].im = fma(x[r][k].re, b.im, out[r][j].im);
        out[r][j].re = fma(-x[r][k].im, b.im, out[r][j].re);
        out[r][j].im = fma(x[r][k].im, b.re, out[r][j].im);
      }
    }
  }
}

__device__ __forceinline__ double max3(double v, int base) {
  return fmax(fmax(__shfl(v, base), __shfl(v, base + 1)), __shfl(v, base + 2));
}

__global__ void stability_clear(double* radius, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) radius[i] = 0.0;
}

template <bool kPaper>
__global__ __launch_bounds__(64) void stability_kernel(StabArgs a, const double* omega_p,
                                                        const double* r_p, double* radius,
                                                        int nchunks) {
  __shared__ double gam[kN2];
  __shared__ cplx mats[kModes * kN2];
  __shared__ cplx solve[kPaper ? 2 * kN2 + kN : 1];
  const int lane = threadIdx.x;
  const int point = blockIdx.x / nchunks, chunk = blockIdx.x % nchunks;
  // Lane 63 repeats lane 60's work.
  const int grp = min(lane / kLanesPerMode, kModes - 1), base = grp * kLanesPerMode;
  const int row0 = (lane - base) % kLanesPerMode * kRowsPerLane;
  cplx* const mat = mats + grp * kN2;
  for (int e = lane; e < kN2; e += 64) gam[e] = gamma_ij(e / kN, e % kN, a.ux, a.uy);
  const double w = omega_p[point], r = r_p[point];
  // collision-map coefficients
  const double A = a.A;
  const double cPg = (2 - A * w) / (2 + w), cPe = (1 + A) * w / (2 + w);
  const double cQg = (2 - w) / (2 + w), cQe = 2 * w / (2 + w);
  const double cRs = a.model == 2 ? 2 / (2 + w) : 2 / (2 + A * w);
  const double cRe = a.model == 2 ? w / (2 + w) : A * w / (2 + A * w);
  const double cFg = 2 / (2 + w), cFe = w / (2 + w);  // f from f~ (A = 0); R at h = dt
  __syncthreads();

  const int nk = a.nkx * a.nky;
  const int k0 = a.nkx > a.nky ? (a.nky - 1) * a.nky : 0;  // the mode at |k| = 0
  const int mine = chunk < nk ? (nk - 1 - chunk) / nchunks + 1 : 0;  // modes of this chunk
  const int stride = mine % 7919 == 0 ? 7907 : 7919;  // prime to mine (< 2^17.1)
  double best = 0.0;  // over this block's modes
  // Item 0 is |k| = 0, then come the chunk's modes; without item 0 where one
  // batch holds them all and nothing is left to compare with it.
  for (int first = mine < kModes ? 1 : 0; first <= mine; first += kModes) {
    const int item = first + grp;
    const bool active = item <= mine;
    // The chunk's modes in a scattered order, so that the first of them
    // already sample the whole grid for a large radius to compare with.
    const int kk = item == 0 || !active ? k0 : chunk + (item - 1) * stride % mine * nchunks;
    const double th[2] = {a.thx0 + (kk / a.nky) * a.dthx, (kk % a.nky) * a.dthy};
    double sn[2], cs[2];
    for (int k = 0; k < 2; ++k) sincos(th[k], &sn[k], &cs[k]);
    cplx rs[kRowsPerLane];  // r * symbol of the lane's rows
#pragma unroll
    for (int i = 0; i < kRowsPerLane; ++i) rs[i] = cscale(symbol_q(row0 + i, sn, cs, a.eta), r);
    auto delta = [&](int i, int j) { return row0 + i == j ? 1.0 : 0.0; };
    auto gm = [&](int i, int j) { return gam[(row0 + i) * kN + j]; };

    Rows X, Y;
    if constexpr (kPaper) {
      // One mode after the other, each by the whole wave (only the groups that
      // have one: with six modes, one squaring and 4000 points, 312 us where a wave
      // takes every mode in turn, 801 with all 21 groups, 260 so).
      cplx* const sym = solve + 2 * kN2;
      const int ngroups = min(kModes, mine + 1 - first);  // those with a mode
      for (int g = 0; g < ngroups; ++g) {
        __syncthreads();
        if (grp == g && lane < 63) {
#pragma unroll
          for (int i = 0; i < kRowsPerLane; ++i) sym[row0 + i] = symbol_q(row0 + i, sn, cs, a.eta);
        }
        __syncthreads();
        solve_paper(a, lane, gam, sym, w, r, solve, solve + kN2);
        for_elems(lane,
                  [&](int i, int j) { mats[g * kN2 + i * kN + j] = solve[kN2 + i * kN + j]; });
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < kRowsPerLane; ++i) {
#pragma unroll
        for (int j = 0; j < kN; ++j)
          X[i][j] = active ? mat[(row0 + i) * kN + j] : cplx{0.0, 0.0};
      }
    } else {
      // (I - c rS) J to LDS, then J_R times it: cRs T + cRe Gamma T.
      auto predicted = [&](double c, double jg, double je, double ss, double se, Rows& out) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kRowsPerLane; ++i) {
          const cplx f = csub({1.0, 0.0}, cscale(rs[i], c));
#pragma unroll
          for (int j = 0; j < kN; ++j)
            mat[(row0 + i) * kN + j] = cscale(f, jg * delta(i, j) + je * gm(i, j));
        }
        __syncthreads();
        gamma_times(gam, mat, row0, out);
#pragma unroll
        for (int i = 0; i < kRowsPerLane; ++i) {
#pragma unroll
          for (int j = 0; j < kN; ++j)
            out[i][j] = cadd(cscale(mat[(row0 + i) * kN + j], ss), cscale(out[i][j], se));
        }
      };
      if (a.model == 2)
        predicted(1.0, cQg, cQe, cRs, cRe, Y);
      else
        predicted(A, cPg, cPe, cRs, cRe, Y);
      if (a.model == 3) {
        // X = base - rS (b0 J_f + b1 J_R (I - A rS) J_P + b2 J_R1 (I - rS) J_Q).
        if (a.gen_bb) {
          // The explicit collision terms, w (Gamma - I) (B-0 J_f + B-1 Y).
          __syncthreads();
#pragma unroll
          for (int i = 0; i < kRowsPerLane; ++i) {
#pragma unroll
            for (int j = 0; j < kN; ++j)
              mat[(row0 + i) * kN + j] =
                  cadd({a.bb[0] * (cFg * delta(i, j) + cFe * gm(i, j)), 0.0},
                       cscale(Y[i][j], a.bb[1]));
          }
          __syncthreads();
          gamma_times(gam, mat, row0, X);
#pragma unroll
          for (int i = 0; i < kRowsPerLane; ++i) {
#pragma unroll
            for (int j = 0; j < kN; ++j)
              X[i][j] = cscale(csub(X[i][j], mat[(row0 + i) * kN + j]), w);
          }
        } else {
#pragma unroll
          for (int i = 0; i < kRowsPerLane; ++i) {
#pragma unroll
            for (int j = 0; j < kN; ++j) X[i][j] = {0.0, 0.0};
          }
        }
#pragma unroll
        for (int i = 0; i < kRowsPerLane; ++i) {
#pragma unroll
          for (int j = 0; j < kN; ++j) {
            const double f = cFg * delta(i, j) + cFe * gm(i, j);
            const double qm = a.gen_bb ? f : cQg * delta(i, j) + cQe * gm(i, j);
            const cplx m = cadd(cscale(Y[i][j], a.bt[1]), {a.bt[0] * f, 0.0});
            X[i][j] = cadd(X[i][j], csub({qm, 0.0}, cmul(rs[i], m)));
          }
        }
        predicted(1.0, cQg, cQe, cFg, cFe, Y);
#pragma unroll
        for (int i = 0; i < kRowsPerLane; ++i) {
#pragma unroll
          for (int j = 0; j < kN; ++j)
            X[i][j] = csub(X[i][j], cmul(rs[i], cscale(Y[i][j], a.bt[2])));
        }
        if (a.gen_bb) {
          // G = (aY I + aE Gamma) X
          const double aY = (1 + 0.5 * w) / (1 + a.bb[2] * w);
          const double aE = w * (a.bb[2] - 0.5) / (1 + a.bb[2] * w);
          publish(mat, row0, X);
          gamma_times(gam, mat, row0, Y);
#pragma unroll
          for (int i = 0; i < kRowsPerLane; ++i) {
#pragma unroll
            for (int j = 0; j < kN; ++j)
              X[i][j] = cadd(cscale(X[i][j], aY), cscale(Y[i][j], aE));
          }
        }
      } else {
        // X = J_Q - c2 rS (J_f (model 2) + J_R T)
        const double c2 = a.model == 2 ? 0.5 : 1.0;
#pragma unroll
        for (int i = 0; i < kRowsPerLane; ++i) {
#pragma unroll
          for (int j = 0; j < kN; ++j) {
            cplx m = Y[i][j];
            if (a.model == 2) m.re += cFg * delta(i, j) + cFe * gm(i, j);
            X[i][j] = csub({cQg * delta(i, j) + cQe * gm(i, j), 0.0},
                           cmul(cscale(rs[i], c2), m));
          }
        }
      }
    }

    // Spectral radius by squaring: G^(2^s) = 2^e X.  dead: the radius counts
    // as 0 (X is zero or not finite), or it cannot be the largest.
    double known = best;
    if (nchunks > 1)
      known = fmax(known, __hip_atomic_load(radius + point, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT));
    const double log_known = log(known);
    double e = 0.0;
    bool dead = !active;
    double biggest = 0.0;  // max |x| of the scaled matrix
    auto scale = [&](int s) {
      double m2 = 0.0, f2 = 0.0;
#pragma unroll
      for (int i = 0; i < kRowsPerLane; ++i) {
#pragma unroll
        for (int j = 0; j < kN; ++j) {
          const double v = cabs2(X[i][j]);
          m2 = fmax(m2, v);
          f2 += v;
        }
      }
      m2 = max3(m2, base);
      f2 = __shfl(f2, base) + __shfl(f2, base + 1) + __shfl(f2, base + 2);
      if (!(m2 > 0.0) || !isfinite(m2)) {
        dead = true;
        return;
      }
      const int x = ilogb(m2) / 2;  // max |x| within a factor of 2 of 2^x
      const double down = ldexp(1.0, -x);
#pragma unroll
      for (int i = 0; i < kRowsPerLane; ++i) {
#pragma unroll
        for (int j = 0; j < kN; ++j) X[i][j] = cscale(X[i][j], down);
      }
      e += x;
      biggest = sqrt(m2) * down;
      // ln rho <= ln ||G^(2^s)||_F / 2^s, f2 rounded up to a power of two
      // (f2 is that of the matrix before the scaling by 2^x); no bound where
      // the sum of squares is not finite.
      if (!(known > 0.0) || !isfinite(f2)) return;
      const double bound = (e - x + 0.5 * (ilogb(f2) + 1)) * 0.6931471805599453;
      if (bound < ldexp(log_known - 1e-11, s)) dead = true;
    };
    scale(0);
    for (int s = 1; s <= a.squarings; ++s) {
      if (__all(dead)) break;
      publish(mat, row0, X);
      square(mat, X, Y);
#pragma unroll
      for (int i = 0; i < kRowsPerLane; ++i) {
#pragma unroll
        for (int j = 0; j < kN; ++j) X[i][j] = Y[i][j];
      }
      e *= 2.0;
      if (!(s & 1) || s == a.squarings) scale(s);
    }
    double rho = 0.0;
    if (!dead) rho = exp(ldexp(e * 0.6931471805599453 + log(biggest), -a.squarings));
    best = fmax(best, wave_max(rho));
    if (lane == 0 && nchunks > 1)
      // A non-negative double orders like its bits.
      atomicMax(reinterpret_cast<unsigned long long*>(radius + point),
                __double_as_longlong(best));
  }
  if (lane == 0 && nchunks == 1) radius[point] = best;
}

}  // namespace

hipError_t launch_stability(const StabArgs& a, const double* omega, const double* r, int npoints,
                            double* radius, hipStream_t s) {
  // Blocks for the whole chip (27 KB of LDS: five waves per CU), two batches
  // of modes each or more.  Several blocks to a point keep their maximum in
  // the output, which is cleared first; an output that overlaps an input
  // takes one block per point, which reads its point before it writes.
  const int nk = a.nkx * a.nky;
  const int most = std::max(1, nk / (2 * kModes));
  auto overlaps = [&](const double* in) { return radius < in + npoints && in < radius + npoints; };
  const int nchunks = overlaps(omega) || overlaps(r)
                          ? 1
                          : std::min(most, std::max(1, kWantedBlocks / npoints));
  if (nchunks > 1)
    hipLaunchKernelGGL(stability_clear, dim3((npoints + 255) / 256), dim3(256), 0, s, radius,
                       npoints);
  const dim3 g(static_cast<unsigned>(npoints) * nchunks);
  if (a.model == 0)
    hipLaunchKernelGGL(stability_kernel<true>, g, dim3(64), 0, s, a, omega, r, radius, nchunks);
  else
    hipLaunchKernelGGL(stability_kernel<false>, g, dim3(64), 0, s, a, omega, r, radius, nchunks);
  return hipGetLastError();
}

}  // namespace t2s2
