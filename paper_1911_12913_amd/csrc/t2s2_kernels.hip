// HIP kernels of the D2Q9 T2S2-FDLBM step for gfx950 (wave64).
//
// The fused step kernel computes one full time step f~^n -> f~^{n+1} of the
// paper's Sec. 2D sequence in a single pass over HBM:
//   P = fbar^{+,h}(f~)                 pointwise (eqs 2.34, 2.51)
//   Q = f~^{+}(f~)                     pointwise (eq 2.20)
//   S = P - h xi . grad_m P            half-step characteristic (eqs 2.33, 2.35)
//   R = f(t*) from S                   pointwise with new moments (eqs 2.32, 2.52)
//   f~^{n+1} = Q - dt xi . grad_m R    (eq 2.23)
// with non-equilibrium extrapolation (eq 3.10) on wall nodes, for R (the
// stencil reads it) and for the new state, both written by the lane of the
// wall node's nearest interior node.  All populations are carried as
// deviations g = f~ - w.
//
// Work decomposition: a block owns a strip of 64 columns (56 outputs plus a
// 4-column halo each side, the reach of the two chained radius-2 stencils)
// and a segment of rows, and marches down the segment.  Each of its four
// waves handles one row per iteration.  P and R rows live in LDS ring
// buffers of 8 rows; Q stays in registers for one iteration.  Every value is
// read from HBM once per strip and written once.
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>

#include <type_traits>

#include "t2s2_device.h"
#include "t2s2_internal.h"
#include "t2s2_step.h"

namespace t2s2 {
namespace {

// ---------------------------------------------------------------------------
// Fused step.
// ---------------------------------------------------------------------------
// Resident waves per SIMD the register allocation must allow: the FP64 rings
// (68 KB per block) admit two blocks per CU; the FP32 rings admit four, which
// the FP32 / FP16 variants without a force reach without spilling (the force
// variants, the walled FP16 ones, and BF16 with its conversions, settle for
// three).
// T2S2-FDLBM2's first ring (106 KB in FP64, 53 KB in FP32) admits one and
// three blocks per CU; in FP64 on periodic meshes it holds Q alone, as
// FDLBM1's holds P, and admits two blocks.
// The family's ring (140 KB in FP64, 70 KB in FP32) admits one and two.
template <typename Store, bool kForce, bool kWalls, int kScheme>
constexpr int kMinWaves =
    sizeof(typename Cvt<Store>::R) == 8
        ? ((kScheme == 1 || (kScheme == 2 && !kWalls)) ? 2 : 1)
        : (kScheme >= 3 ? 2
                        : (((kScheme == 2 && (kWalls || std::is_same<Store, float>::value)) ||
                            kForce || kBf16Bits<Store> ||
                            kStochastic<Store> || (kWalls && !std::is_same<Store, float>::value))
                               ? 3
                               : 4));

// T2S2-FDLBM2 on a periodic mesh keeps each row's f^n in the registers of
// the wave that loaded the row, instead of in the first LDS ring: the
// waves take the phase-2 rows in the order that makes each one's phase-2
// row a row it loaded (in this iteration for waves 0 and 1, in the previous
// one for waves 2 and 3), and the ring holds Q alone.  At 4096^2: FP64
// 643 -> 503 us per step (two blocks per CU, where forming f^n again from
// a reload of the row fetched the rows twice from HBM), BF16 261 -> 232
// us; FP32 storage keeps the ring (365 against 374 us).  Walled meshes keep
// f^n in the ring: eq 3.10 reads it at wall nodes that another wave loaded.
template <typename Store, bool kWalls, int kScheme>
constexpr bool kFnRegsOf = kScheme == 2 && !kWalls && !std::is_same<Store, float>::value;

// Planes of the first LDS ring: P for T2S2-FDLBM1 (and T1S2); for
// T2S2-FDLBM2, Q = f~^+ (the field the prediction advects) and, for the
// eight moving directions, the physical f^n (not with kFnRegsOf); for the
// family, P, Q and the eight moving directions of f^n.
template <int kScheme, bool kFnRegs>
constexpr int kPPlanes =
    kScheme == 1 ? kQ : (kScheme == 2 ? (kFnRegs ? kQ : 2 * kQ - 1) : 3 * kQ - 1);

// The fused step, templated on the storage type, the presence of a body
// force, of walls, on the scheme, and on kSaveS (the discrete adjoint's
// recompute: also store S = fbar(t*) at the interior nodes, into
// p.save_s in the arithmetic type, [9][ny][pitch]):
//   kScheme 1: T2S2-FDLBM1 family (eq 2.23; A = 0 is T1S2);
//   kScheme 2: T2S2-FDLBM2 (eq 5.23): f~^{n+1} = Q + dt/2 (L(f^n) + L(f^{n+1}))
//     with f^{n+1} predicted by S = Q + dt L(Q) and unshifted with h = dt;
//     L is linear, so the two gradients are taken as one, of T = f^n + R;
//   kScheme 3: the eq 2.13 family, f~^{n+1} = Q + dt L(T) with
//     T = b0 f^n + b1 f* + b2 f^{n+1}, f* predicted as in scheme 1 and
//     f^{n+1} as in scheme 2;
//   kScheme 4: the family with collision weights other than (1/2, 0, 1/2)
//     (p.gen_bbar; host scheme 3): the base is Q2 = f^n + B-0 dt Omega(f^n)
//     and V = B-1 dt Omega(f*) is added, and the new state is formed from
//     Y = Q2 + V + dt L(T) by solving the implicit weight B-2 through Y's
//     moments.  V of a node is formed in phase 2 from that node's f* and
//     used by phase 3 of the same wave, in registers: the waves take the
//     phase-2 rows in the order that makes each one's phase-2 row the row it
//     outputs (in the same iteration for waves 2 and 3, in the next for
//     waves 0 and 1).
template <typename Store, bool kForce, bool kWalls, int kScheme, bool kSaveS = false>
__global__ __launch_bounds__(step_threads(kStorageOf<Store>, kScheme), (kMinWaves<Store, kForce, kWalls, kScheme>)) void step_kernel(
    StepParams p) {
  using Real = typename Cvt<Store>::R;
  // Scheme 1 is taken by other kernels too, which round alike (see kExactOf), and
  // the FP64 family with gradient weights (0, 1, 0) equals it.  What no other
  // kernel takes leaves its sums to the compiler.  The FP64 forms also read the
  // rings in another way (kFp64Rows): with both, the others run 1 to 3% slower
  // (walled family 16 x 10, BF16, 22.7 us per step, 23.1 so; T1S2 in FP16 with
  // stochastic rounding 31 x 33, 16.3 and 16.6; channel 1500 x 1400 FP32 61.6,
  // 64.2).
  constexpr bool kFp64Rows = sizeof(Real) == 8 && (kScheme == 1 || kScheme == 3);
  constexpr bool kExact = kFp64Rows || (kScheme == 1 && kExactOf<Real, kForce>);
  using Row = std::conditional_t<kFp64Rows, LdsPtr<Real>, const Real*>;
  // T2S2-FDLBM2, FP64, periodic: f^n of the phase-2 row from a reload.
  constexpr bool kFnRegs = kFnRegsOf<Store, kWalls, kScheme>;
  constexpr int kNP = kPPlanes<kScheme, kFnRegs>;
  constexpr int kSB = strips_per_block(kStorageOf<Store>, kScheme);
  constexpr int kThreads = step_threads(kStorageOf<Store>, kScheme);
  constexpr int kSizeP = kRing * kNP * kLanes, kSizeR = kRing * (kQ - 1) * kLanes;
  constexpr int kSizeT = kWalls ? (kQ - 1) * kLanes : 1;
  __shared__ Real ringP_all[kSB * kSizeP];  // per strip: [slot][plane][lane]
  __shared__ Real ringR_all[kSB * kSizeR];  // per strip: [slot][q-1][lane]
  // R of the top wall row ny-1, kept out of the ring: it is written (eq 3.10)
  // by the wave that computes row ny-2, in the same phase in which the ring
  // slot of row ny-1 still holds row ny-9 for the output row ny-7.
  __shared__ Real topR_all[kSB * kSizeT];

  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int half = kSB == 1 ? 0 : wave / kRowsPerIter;  // which of the block's strips
  const int t = kSB == 1 ? wave : wave % kRowsPerIter;  // which row of an iteration
  Real* const ringP = ringP_all + half * kSizeP;
  Real* const ringR = ringR_all + half * kSizeR;
  Real* const topR = topR_all + half * kSizeT;
  const int nx = p.nx, ny = p.ny;
  const Store* __restrict__ src = static_cast<const Store*>(p.src);
  Store* __restrict__ dst = static_cast<Store*>(p.dst);
  const long long plane = p.plane;

  for (int i = threadIdx.x; i < kSB * kSizeP; i += kThreads) ringP_all[i] = Real(0);
  for (int i = threadIdx.x; i < kSB * kSizeR; i += kThreads) ringR_all[i] = Real(0);
  if (kWalls)
    for (int i = threadIdx.x; i < kSB * kSizeT; i += kThreads) topR_all[i] = Real(0);

  // Work: a unit is kSB neighbouring strips, marched side by side by the
  // block's kSB groups of four waves (a strip past the last column computes
  // in its own rings and stores nothing).  The rows are cut into bands of
  // p.band rows; the unit-rows are ordered band by band, unit by unit within
  // a band, row by row within a unit, and this order is cut into nblocks
  // equal ranges (one per block, so every block does the same work).  With
  // the band height equal to one block's share, a block owns one unit of one
  // band, and the blocks of neighbouring units start on the same row and
  // march in step: the cache lines that two strips share (the halo columns)
  // are fetched from HBM once and found in L1 or L2 by the other strip.  A
  // range may run over a unit or band boundary; each piece is marched
  // separately.  XCD-aware order: the grid is a multiple of 8 and blocks are
  // dealt round-robin to the 8 XCDs, so block b runs on XCD b % 8; each XCD
  // gets a contiguous run of ranges, i.e. neighbouring units of a band share
  // one L2.
  const int G = gridDim.x;
  const int L = (blockIdx.x % 8) * (G / 8) + blockIdx.x / 8;
  if (L >= p.nblocks) return;  // padding block: whole block, before any barrier
  const long long total = static_cast<long long>(p.nunits) * ny;
  const long long band_pieces = static_cast<long long>(p.nunits) * p.band;
  long long beg = total * L / p.nblocks;
  const long long end = total * (L + 1) / p.nblocks;

  while (beg < end) {  // uniform per block
    const int b = static_cast<int>(beg / band_pieces);
    const long long rem = beg - b * band_pieces;
    const int r0 = b * p.band;
    const int hb = min(p.band, ny - r0);  // the last band may be shorter
    const int strip = static_cast<int>(rem / hb) * kSB + half;
    const int y0 = r0 + static_cast<int>(rem % hb);
    const int y1 = static_cast<int>(min(static_cast<long long>(r0 + hb), y0 + (end - beg)));
    beg += y1 - y0;

    const int x0 = strip * kStripOut;
    const int x1 = min(x0 + kStripOut, nx);
    // This lane's column; loads and weights use the wrapped (periodic) or
    // clamped (walled) column so every ring entry holds finite data.
    const int c = x0 - kHalo + lane;
    const int cm = p.per_x ? wrap(c, nx) : clampi(c, 0, nx - 1);
    Real wxr[kWeightsPerNode];
    {
      const Real* wx = weights_x<Real>(p);
#pragma unroll
      for (int k = 0; k < kWeightsPerNode; ++k) wxr[k] = wx[cm * kWeightsPerNode + k];
    }
    const bool col_interior = p.per_x || (c >= 1 && c <= nx - 2);
    const bool lane_r = lane >= 2 && lane < kLanes - 2;
    const bool lane_o = lane >= kHalo && lane < kLanes - kHalo && c < x1;
    const bool src_xl = !p.per_x && c == 1;
    const bool src_xr = !p.per_x && c == nx - 2;

    // Q of the rows of the previous and of this iteration, alternating
    // between two register arrays over the iteration pair.
    Real qA[kQ], qB[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) qA[q] = qB[q] = Real(0);
    // A value each wave forms for its own phase-2 rows, of this and of the
    // previous iteration: the family's V = B-1 dt Omega(f*) (kScheme 4,
    // formed in phase 2 for phase 3), or f^n (kFnRegs, formed in phase 1
    // for phase 2).
    Real vA[kQ], vB[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) vA[q] = vB[q] = Real(0);
    constexpr bool kFamily = kScheme >= 3;
    constexpr bool gen_bbar = kScheme == 4;

    // Iterations come in pairs (one per prefetch buffer); a trailing extra
    // iteration only reloads clamped rows and stores nothing (its rows fail
    // the row checks below).
    const int niter = ((y1 - y0 + kRowsPerIter - 1) / kRowsPerIter + 3) & ~1;

    // Row loads run two iterations ahead in two register buffers, so two
    // iterations of loads are in flight while the stencil phases compute.
    Store gA[kQ], gB[kQ];
    const int pitch = static_cast<int>(p.pitch);
    // Rows y0-4 .. y1+3 are needed; prefetches past the last one repeat it
    // (found in cache instead of fetched from HBM).
    auto load_row = [&](int pr, Store (&gb)[kQ]) {
      const int pc = min(pr, y1 + kHalo - 1);
      const int prm = p.per_y ? wrap_near(pc, ny) : clampi(pc, 0, ny - 1);
      const unsigned boff =
          (static_cast<unsigned>(prm) * static_cast<unsigned>(pitch) + static_cast<unsigned>(cm)) *
          static_cast<unsigned>(sizeof(Store));
      load_planes(src, plane * sizeof(Store), boff, gb);
    };
    load_row(y0 - kHalo + t, gA);
    load_row(y0 - kHalo + kRowsPerIter + t, gB);
    __syncthreads();  // ring zero-fill / previous piece complete

    auto iteration = [&](const int it, Store (&gb)[kQ], Real (&qnew)[kQ], const Real (&qold)[kQ],
                         Real (&vnew)[kQ], const Real (&vold)[kQ]) {
      const int p0 = y0 - kHalo + kRowsPerIter * it;

      // ---- phase 1: P (to LDS) and Q (registers) of row p0 + t; for
      // T2S2-FDLBM2 Q and f^n to LDS (P's coefficients then give f^n), or
      // f^n to registers (kFnRegs).
      {
        const int pr = p0 + t;
        Real g[kQ];
#pragma unroll
        for (int q = 0; q < kQ; ++q) g[q] = Cvt<Store>::ld(gb[q]);
        // Unconditional (rows are clamped or wrapped into the grid): the
        // buffers then stay in fixed registers with their loads in flight.
        load_row(pr + 2 * kRowsPerIter, gb);
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
        const auto& k = coef<Real>(p);
        Real* slotP = ringP + (pr & (kRing - 1)) * kNP * kLanes;
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
          // E = (f^eq_q - w_q) / w_q; P and Q take their f^eq coefficient
          // times w_q per weight class.
          const Real E = fma_of<kExact>(rho, X[q], d);
          Real Pq = fma_of<kExact>(k.cPg, g[q], k.kP[wclass(q)] * E);
          Real Qq = fma_of<kExact>(k.cQg, g[q], k.kQ[wclass(q)] * E);
          Real Fq = Real(0);
          if (kForce) {
            Fq = force_term<kExact>(q, p, ux, uy, E);
            Pq = fma_of<kExact>(static_cast<Real>(p.cPF), Fq, Pq);
            Qq = fma_of<kExact>(static_cast<Real>(p.cQF), Fq, Qq);
          }
          slotP[q * kLanes + lane] = kScheme == 2 ? Qq : Pq;
          if (kScheme == 2 && !kFnRegs && q > 0) slotP[(kQ + q - 1) * kLanes + lane] = Pq;
          if constexpr (kFnRegs) vnew[q] = Pq;
          if (kFamily) {
            slotP[(kQ + q) * kLanes + lane] = Qq;
            if (q > 0) {
              Real Uq = fma_of<kExact>(k.cU, g[q], k.kU[wclass(q)] * E);  // f^n
              if (kForce) Uq = fma_of<kExact>(static_cast<Real>(p.cUF), Fq, Uq);
              slotP[(2 * kQ + q - 1) * kLanes + lane] = Uq;
            }
          }
          qnew[q] = Qq;
          if constexpr (gen_bbar) {  // Q2 = f^n + B-0 dt Omega(f^n)
            Real Q2 = fma_of<kExact>(k.cQ2g, g[q], k.kQ2[wclass(q)] * E);
            if (kForce) Q2 = fma_of<kExact>(static_cast<Real>(p.cQ2F), Fq, Q2);
            qnew[q] = Q2;
          }
        }
      }
      __syncthreads();

      // ---- phase 2: S and R of row p0 - 2 + t (interior nodes), R (or the
      // scheme's combination T) to LDS.  The whole wave computes (the x taps
      // take neighbouring lanes' centre values); only interior lanes 2..61
      // store.
      {
        const int r = p0 - 2 + (gen_bbar || kFnRegs ? (t + 2) % kRowsPerIter : t);
        const bool row_ok =
            r >= y0 - 2 && r < y1 + 2 && (p.per_y || (r >= 1 && r <= ny - 2));
        if (row_ok) {
          const int rm = p.per_y ? wrap_near(r, ny) : r;
          Real wyr[kWeightsPerNode];
          row_weights(weights_y<Real>(p), rm, wyr);
          // One base pointer per ring row r-2 .. r+2 at this lane.
          Row rb[5];
#pragma unroll
          for (int o = 0; o < 5; ++o)
            rb[o] = (Row)(ringP + ((r + o - 2) & (kRing - 1)) * kNP * kLanes + lane);
          const auto& k = coef<Real>(p);
          // A prediction along the characteristics from ring planes
          // [base, base + 9): S = centre + fac L(centre); then f at the
          // predicted time, R = cs S + ke E (+ cf F), from S's moments with
          // force shift hf.  With want_v, also V = B-1 dt Omega(R) (all
          // nine directions; R[0] stays 0, the rest direction has no
          // gradient).
          auto predict = [&](int base, Real fac, Real cs, const Real* ke, double cf, double hf,
                             Real (&S)[kQ], Real (&R)[kQ], Real& rho, Real& ux, Real& uy,
                             Real (&X)[kQ], bool want_v, Real (&V)[kQ]) {
#pragma unroll
            for (int q = 0; q < kQ; ++q) {
              const int pq = (base + q) * kLanes;
              const Real centre = rb[2][pq];
              Real acc = Real(0);
              if (ex_of(q) > 0) acc = x_taps<0, kExact>(wxr, centre, acc);
              if (ex_of(q) < 0) acc = x_taps<1, kExact>(wxr, centre, acc);
              if (ey_of(q) != 0) {
                const int sy = ey_of(q) > 0 ? 0 : 1;
#pragma unroll
                for (int k2 = 0; k2 < kTaps; ++k2)
                  acc = fma_of<kExact>(wyr[sy * kTaps + k2], rb[k2 + sy][pq], acc);
              }
              S[q] = q == 0 ? centre : fma_of<kExact>(fac, acc, centre);
            }
            double s, jx, jy;
            moment_sums(S, s, jx, jy);
            if constexpr (kForce)
              forced_velocity<kExact>(s, jx, jy, hf, p.Fx, p.Fy, rho, ux, uy);
            else
              velocity<kExact>(s, jx, jy, rho, ux, uy);
            const Real d = static_cast<Real>(s);
            eq_brackets<kExact>(ux, uy, X);
            R[0] = Real(0);
#pragma unroll
            for (int q = 1; q < kQ; ++q) {
              const Real E = fma_of<kExact>(rho, X[q], d);
              Real Rq = fma_of<kExact>(cs, S[q], ke[wclass(q)] * E);
              if (kForce)
                Rq = fma_of<kExact>(static_cast<Real>(cf), force_term<kExact>(q, p, ux, uy, E), Rq);
              R[q] = Rq;
            }
            if (want_v) {
              // Omega(f*) dt = w (f^eq* - f*) + dt F*, in deviations from w.
#pragma unroll
              for (int q = 0; q < kQ; ++q) {
                const Real E = fma_of<kExact>(rho, X[q], d);
                Real Fq = Real(0);
                if (kForce) Fq = force_term<kExact>(q, p, ux, uy, E);
                Real Rq = fma_of<kExact>(cs, S[q], ke[wclass(q)] * E);
                if (kForce) Rq = fma_of<kExact>(static_cast<Real>(cf), Fq, Rq);
                Real Vq = k.kV[wclass(q)] * E - k.cV * Rq;
                if (kForce) Vq = fma_of<kExact>(static_cast<Real>(p.cVF), Fq, Vq);
                V[q] = Vq;
              }
            }
          };
          Real S[kQ], R[kQ], X[kQ], rho, ux, uy;
          predict(0, k.A, k.cRs, k.kR, p.cRF, p.half_h, S, R, rho, ux, uy, X, gen_bbar, vnew);
          if (kSaveS && lane_o && col_interior && r >= y0 && r < y1) {
            Real* sv = static_cast<Real*>(p.save_s);
            const unsigned boff =
                (static_cast<unsigned>(r) * static_cast<unsigned>(pitch) + static_cast<unsigned>(c)) *
                static_cast<unsigned>(sizeof(Real));
#pragma unroll
            for (int q = 0; q < kQ; ++q) *at_byte(sv + q * plane, boff) = S[q];
          }
          // The family's second prediction: f^{n+1} from Q with h = dt.
          Real R2[kQ], X2[kQ], rho2 = Real(1), ux2 = Real(0), uy2 = Real(0);
#pragma unroll
          for (int q = 0; q < kQ; ++q) R2[q] = X2[q] = Real(0);
          if constexpr (kFamily) {
            Real S2[kQ];
            predict(kQ, Real(1), k.cU, k.kU, p.cUF, p.half_dt, S2, R2, rho2, ux2, uy2, X2, false,
                    S2);
          }
          // f^n of this node (kFnRegs): formed in phase 1 of this iteration
          // by waves 0 and 1, of the previous one by waves 2 and 3.
          Real fn[kQ];
#pragma unroll
          for (int q = 0; q < kQ; ++q) fn[q] = Real(0);
          if constexpr (kFnRegs) {
#pragma unroll
            for (int q = 1; q < kQ; ++q) fn[q] = t < 2 ? vnew[q] : vold[q];
          }
          // T, the field whose gradient the full step takes: R (scheme 1),
          // f^n + R (scheme 2, halved in phase 3), b0 f^n + b1 R + b2 R2
          // (scheme 3); f^n of (row, ln) from the ring (from fn with
          // kFnRegs, where (row, ln) is always this node).
          auto t_of = [&](int q, int row, int ln, Real r1, Real r2) {
            const Real* slot = ringP + (row & (kRing - 1)) * kNP * kLanes + ln;
            if (kScheme == 2) return r1 + (kFnRegs ? fn[q] : slot[(kQ + q - 1) * kLanes]);
            if (kFamily)
              return k.b[0] * slot[(2 * kQ + q - 1) * kLanes] + k.b[1] * r1 + k.b[2] * r2;
            return r1;
          };
          if (lane_r && col_interior) {
            Real* slotR = ringR + (r & (kRing - 1)) * (kQ - 1) * kLanes;
#pragma unroll
            for (int q = 1; q < kQ; ++q) slotR[(q - 1) * kLanes + lane] = t_of(q, r, lane, R[q], R2[q]);
            // Wall nodes whose nearest interior node is this one (eq 3.10
            // on f(t*) and f(t_{n+1}); corners take the diagonal
            // neighbour).  Physical f carries no force shift:
            // u_f = sum xi R / rho = u*.
            const bool src_yb = !p.per_y && r == 1;
            const bool src_yt = !p.per_y && r == ny - 2;
            if (kWalls && (src_xl || src_xr || src_yb || src_yt)) {
              for (int dy = -1; dy <= 1; ++dy) {
                if ((dy == -1 && !src_yb) || (dy == 1 && !src_yt)) continue;
                for (int dx = -1; dx <= 1; ++dx) {
                  if ((dx == -1 && !src_xl) || (dx == 1 && !src_xr)) continue;
                  if (dx == 0 && dy == 0) continue;
                  // The shift from the brackets of u_f, formed above, and
                  // of the wall's velocity.
                  const Real* Xb = wall_brackets<Real>(p, wall_side_of(dx, dy));
                  Real* slotW = dy == 1 ? topR : ringR + ((r + dy) & (kRing - 1)) * (kQ - 1) * kLanes;
                  if constexpr (kFp64Rows) {
                    const Real r1 = Real(w_of(1)) * rho, r2 = Real(w_of(5)) * rho;
                    const Real r1b = Real(w_of(1)) * rho2, r2b = Real(w_of(5)) * rho2;
#pragma unroll
                    for (int q = 1; q < kQ; ++q) {
                      const Real wall1 = nee_r(wclass(q) == 1 ? r1 : r2, X[q], Xb[q], R[q]);
                      const Real wall2 =
                          kFamily ? nee_r(wclass(q) == 1 ? r1b : r2b, X2[q], Xb[q], R2[q]) : R2[q];
                      slotW[(q - 1) * kLanes + lane + dx] =
                          t_of(q, r + dy, lane + dx, wall1, wall2);
                    }
                  } else {
                    Real sh[kQ], sh2[kQ];
                    nee_shift_x(rho, X, Xb, sh);
#pragma unroll
                    for (int q = 0; q < kQ; ++q) sh2[q] = Real(0);
                    if constexpr (kFamily) nee_shift_x(rho2, X2, Xb, sh2);
#pragma unroll
                    for (int q = 1; q < kQ; ++q)
                      slotW[(q - 1) * kLanes + lane + dx] =
                          t_of(q, r + dy, lane + dx, R[q] + sh[q], R2[q] + sh2[q]);
                  }
                }
              }
            }
          }
        }
      }
      __syncthreads();

      // ---- phase 3: f~^{n+1} of row p0 - 4 + t (whole wave computes,
      // interior output lanes store).
      {
        const int o = p0 - 4 + t;
        const bool row_ok = o >= y0 && o < y1 && (p.per_y || (o >= 1 && o <= ny - 2));
        if (row_ok) {
          Real wyr[kWeightsPerNode];
          row_weights(weights_y<Real>(p), o, wyr);
          Row rb[5];
#pragma unroll
          for (int k = 0; k < 5; ++k) {
            rb[k] = (Row)(ringR + ((o + k - 2) & (kRing - 1)) * (kQ - 1) * kLanes + lane);
            if (kWalls && !p.per_y && o + k - 2 == ny - 1) rb[k] = (Row)(topR + lane);
          }
          Real out[kQ];
          // V of this row: formed in this iteration's phase 2 by waves 2
          // and 3, in the previous one's by waves 0 and 1.
          const bool v_now = t >= 2;
          out[0] = qold[0];
          if constexpr (gen_bbar) out[0] += v_now ? vnew[0] : vold[0];
#pragma unroll
          for (int q = 1; q < kQ; ++q) {
            const int pq = (q - 1) * kLanes;
            const Real centre = rb[2][pq];
            Real acc = kScheme == 2 ? Real(0) : qold[q];
            if constexpr (gen_bbar) acc += v_now ? vnew[q] : vold[q];
            const int sy = ey_of(q) > 0 ? 0 : 1;
            if constexpr (kFp64Rows) {
              // Each row where it is added, or ahead of the sum for the family
              // without a force (cavity 16 x 10 27.7 us per step, each where it is
              // added 28.7; scheme 1, channel 1100^2 without a force 54.9, ahead
              // 55.8, channel 1500 x 1400 88.0, ahead 89.6).
              if constexpr (kForce || kScheme == 1) {
                acc = full_taps(q, wxr, wyr, centre, acc, [&](int k) { return rb[k + sy][pq]; });
              } else {
                Real rows[kTaps] = {};
                if (ey_of(q) != 0) {
#pragma unroll
                  for (int k = 0; k < kTaps; ++k) rows[k] = rb[k + sy][pq];
                }
                acc = full_taps(q, wxr, wyr, centre, acc, [&](int k) { return rows[k]; });
              }
            } else {
              if (ex_of(q) > 0) acc = x_taps<0, kExact>(wxr, centre, acc);
              if (ex_of(q) < 0) acc = x_taps<1, kExact>(wxr, centre, acc);
              if (ey_of(q) != 0) {
#pragma unroll
                for (int k = 0; k < kTaps; ++k)
                  acc = fma_of<kExact>(wyr[sy * kTaps + k], rb[k + sy][pq], acc);
              }
            }
            out[q] = kScheme == 2 ? qold[q] + Real(0.5) * acc : acc;
          }
          if constexpr (gen_bbar) {
            // The implicit weight: f^{n+1} has Y's density and Y's momentum
            // plus B-2 dt rho F; the state is f~ = aY Y + aE (f^eq - w) + aF F
            // at that (rho, u).
            const auto& k = coef<Real>(p);
            double s, jx, jy;
            moment_sums(out, s, jx, jy);
            Real rho, ux, uy;
            if constexpr (kForce)
              forced_velocity<kExact>(s, jx, jy, p.b2dt, p.Fx, p.Fy, rho, ux, uy);
            else
              velocity<kExact>(s, jx, jy, rho, ux, uy);
            const Real d = static_cast<Real>(s);
            Real X[kQ];
            eq_brackets<kExact>(ux, uy, X);
#pragma unroll
            for (int q = 0; q < kQ; ++q) {
              const Real E = fma_of<kExact>(rho, X[q], d);
              Real o = k.aY * out[q] + k.kA[wclass(q)] * E;
              if (kForce)
                o = fma_of<kExact>(static_cast<Real>(p.aF), force_term<kExact>(q, p, ux, uy, E), o);
              out[q] = o;
            }
          }
          if (lane_o && col_interior) {
            const unsigned boff =
                (static_cast<unsigned>(o) * static_cast<unsigned>(pitch) + static_cast<unsigned>(c)) *
                static_cast<unsigned>(sizeof(Store));
            store_node(dst, plane, boff, out);
          }
        }
      }
    };

    for (int it = 0; it < niter; it += 2) {
      iteration(it, gA, qA, qB, vA, vB);
      iteration(it + 1, gB, qB, qA, vB, vA);
    }
    __syncthreads();  // the next piece reuses the rings; the piece's stores are visible
    if (kWalls)
      piece_walls<kExact, sizeof(Store) == 2>(
          p, dst, x0, x1, y0, y1, threadIdx.x % kBlockThreads, kBlockThreads,
          [&](int c2, int r2, int side, double& u, double& v) {
            // (By address, the unforced FP64 forms are 2% faster, the others slower.)
            if (kFp64Rows && !kForce) {
              u = p.uw[side][0];
              v = p.uw[side][1];
            } else {
              wall_velocity(p, c2, r2, u, v);
            }
          });
  }
}

// ---------------------------------------------------------------------------
// Tile step for small meshes (T2S2-FDLBM1 family).  A block takes one strip
// (56 output columns) and a whole tile of rows instead of marching down a
// range of rows: it loads the tile's rows with their halo of four at once,
// forms P of all of them and Q of its output rows, then S and R of all but the
// outer two rows, then the new state: three phases and two barriers, where a
// march over a few rows runs pipelined iterations of three phases each.  Each
// node takes the expressions of step_kernel.  Wave w holds rows w and (kH =
// 2) w + kWaves of the tile in every phase, so the x taps and the populations
// that do not move in y stay in its registers; the y-moving ones of P and R go
// through LDS.  kSaveS also stores S at the interior nodes, as in step_kernel.
//
// A chain of latencies bounds it on the smallest meshes: of the 9.7 us of a
// 257^2 FP64 cavity step an empty launch is 3.5, P 0.5, S and R 1.8, the new
// state and its way to memory 2.7, the wall nodes 1.2.  Sixteen waves, one per
// row, cover each other's latencies better than eight that take two rows of P
// and of S in turn (257^2 cavity FP64 9.86 -> 9.70 us, FP32 8.65 -> 7.70).  On
// larger ones the halo rows of the eight output rows count (16 of P and 12 of
// S for 8): two rows per wave give 16 output rows in FP64 and 24 in the
// narrower forms.  FP64 cavity, one row -> two rows per wave: 385^2
// 16.1 -> 12.9 us, 641^2 29.7 -> 25.7, 769^2 41.4 -> 33.0; see plan_tile.
// ---------------------------------------------------------------------------
// Tile shapes: kH rows per wave; FP64 with two has fewer waves (its LDS and
// registers hold 24 rows).
template <typename Store, int kH>
constexpr int tile_waves() {
  return kH == 2 && sizeof(typename Cvt<Store>::R) == 8 ? 12 : 16;
}
template <typename Store, int kH>
constexpr int tile_rows() {
  return kH * tile_waves<Store, kH>() - 2 * kHalo;
}

// Moments and brackets of a node, unforced FP32: velocity and eq_brackets
// with their products fused as the compiler fuses them in step_kernel, where
// the sums ux + uy and uy - ux take one of the two velocities as a product
// (uy's where kFuseY, else ux's).  Left to the compiler here, another choice
// would differ in the last bit, which stochastic rounding turns into whole
// units of the 16-bit forms.
template <bool kFuseY>
__device__ inline void moments_f32(double s, double jx, double jy, float& r, float X[kQ]) {
#pragma clang fp contract(off)
  r = 1.0f + static_cast<float>(s);
  const float r0 = __builtin_amdgcn_rcpf(r);
  const float ir = __builtin_fmaf(__builtin_fmaf(-r, r0, 1.0f), r0, r0);
  const float fx = static_cast<float>(jx), fy = static_cast<float>(jy);
  const float x = fx * ir, y = fy * ir;
  const float uu = 1.5f * __builtin_fmaf(x, x, y * y);
  X[0] = -uu;
  auto pair = [&](float e, int qp, int qm) {
    const float T = __builtin_fmaf(e, 4.5f * e, -uu);
    X[qp] = __builtin_fmaf(3.0f, e, T);
    X[qm] = __builtin_fmaf(-3.0f, e, T);
  };
  pair(x, 1, 3);
  pair(y, 2, 4);
  pair(kFuseY ? __builtin_fmaf(ir, fy, x) : __builtin_fmaf(ir, fx, y), 5, 7);
  pair(kFuseY ? __builtin_fmaf(ir, fy, -x) : __builtin_fmaf(-ir, fx, y), 6, 8);
}

template <typename Store, bool kForce, bool kWalls, bool kSaveS, int kH>
__global__ __launch_bounds__((tile_waves<Store, kH>() * kLanes)) void tile_step_kernel(
    StepParams p) {
  using Real = typename Cvt<Store>::R;
  constexpr bool kExact = kExactOf<Real, kForce>;
  constexpr int kWaves = tile_waves<Store, kH>();
  constexpr int kIn = kWaves * kH;   // rows of P
  constexpr int kMid = kIn - 4;      // rows of R
  constexpr int kOut = tile_rows<Store, kH>();
  __shared__ Real tP[kIn * kYMoving * kLanes];   // [row][slot][lane]
  __shared__ Real tR[kMid * kYMoving * kLanes];  // [row][slot][lane]
  // The walls' brackets and velocities, fetched while phase 1 waits for the
  // state: indexed by side where they are used, each would be a round trip to
  // the argument segment on the kernel's critical path (65^2 cavity 9.55 ->
  // 9.35 us).
  __shared__ Real tX[4 * kQ];
  __shared__ double tU[4][2];
  const int lane = threadIdx.x & (kLanes - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int nx = p.nx, ny = p.ny;
  const Store* __restrict__ src = static_cast<const Store*>(p.src);
  Store* __restrict__ dst = static_cast<Store*>(p.dst);
  const long long plane = p.plane;
  const int pitch = static_cast<int>(p.pitch);
  const int ntiles = (ny + kOut - 1) / kOut;
  const int strip = blockIdx.x / ntiles;
  const int y0 = (blockIdx.x % ntiles) * kOut;
  const int y1 = min(y0 + kOut, ny);
  if (strip >= p.nstrips) return;  // whole block, before any barrier

  Real xbv = Real(0);
  double uwv = 0;
  if (kWalls && threadIdx.x < 4 * kQ) {
    xbv = wall_brackets<Real>(p, 0)[threadIdx.x];
    uwv = p.uw[(threadIdx.x >> 1) & 3][threadIdx.x & 1];
  }

  const int x0 = strip * kStripOut;
  const int x1 = min(x0 + kStripOut, nx);
  const int c = x0 - kHalo + lane;
  const int cm = p.per_x ? wrap(c, nx) : clampi(c, 0, nx - 1);
  Real wxr[kWeightsPerNode];
  {
    const Real* wx = weights_x<Real>(p);
#pragma unroll
    for (int k = 0; k < kWeightsPerNode; ++k) wxr[k] = wx[cm * kWeightsPerNode + k];
  }
  const bool col_interior = p.per_x || (c >= 1 && c <= nx - 2);
  const bool lane_o = lane >= kHalo && lane < kLanes - kHalo && c < x1;
  // Strips with a wall column or columns past it (uniform per block).
  const bool side = kWalls && !p.per_x && (strip == 0 || x0 + kLanes - kHalo >= nx);
  const auto& k = coef<Real>(p);

  auto y_of = [&](int h) { return y0 - kHalo + w + kWaves * h; };
  auto interior_row = [&](int h) { return p.per_y || (y_of(h) >= 1 && y_of(h) <= ny - 2); };
  auto out_row = [&](int h) {  // uniform per wave, as all row tests
    const int j = w + kWaves * h;
    return j >= kHalo && j < kIn - kHalo && y_of(h) < y1;
  };

  // ---- phase 1: P of the wave's rows, Q of those that are output rows.
  Real pr[kH][kQ], qout[kH][kQ];
  {
    Store gr[kH][kQ];
#pragma unroll
    for (int h = 0; h < kH; ++h) {
      const int prm = p.per_y ? wrap_near(y_of(h), ny) : clampi(y_of(h), 0, ny - 1);
      const unsigned boff =
          (static_cast<unsigned>(prm) * static_cast<unsigned>(pitch) + static_cast<unsigned>(cm)) *
          static_cast<unsigned>(sizeof(Store));
      load_planes(src, plane * sizeof(Store), boff, gr[h]);
    }
#pragma unroll
    for (int h = 0; h < kH; ++h) {
      const int j = w + kWaves * h;
      Real g[kQ];
#pragma unroll
      for (int q = 0; q < kQ; ++q) g[q] = Cvt<Store>::ld(gr[h][q]);
      double s, jx, jy;
      moment_sums(g, s, jx, jy);
      Real rho, ux = Real(0), uy = Real(0), X[kQ];
      if constexpr (sizeof(Real) == 4 && !kForce) {
        moments_f32<true>(s, jx, jy, rho, X);
      } else {
        if constexpr (kForce)
          forced_velocity<kExact>(s, jx, jy, p.half_dt, p.Fx, p.Fy, rho, ux, uy);
        else
          velocity<kExact>(s, jx, jy, rho, ux, uy);
        eq_brackets<kExact>(ux, uy, X);
      }
      const Real d = static_cast<Real>(s);
      Real E[kQ], Fq[kQ];
#pragma unroll
      for (int q = 0; q < kQ; ++q) {
        E[q] = fma_of<kExact>(rho, X[q], d);
        Real Pq = fma_of<kExact>(k.cPg, g[q], k.kP[wclass(q)] * E[q]);
        if (kForce) {
          Fq[q] = force_term<kExact>(q, p, ux, uy, E[q]);
          Pq = fma_of<kExact>(static_cast<Real>(p.cPF), Fq[q], Pq);
        }
        // Formed here: moved to the later phases, the FP32 products would be
        // fused another way than in step_kernel.
        if constexpr (!kExact) asm volatile("" : "+v"(Pq));
        pr[h][q] = Pq;
        if (ey_of(q) != 0) tP[(j * kYMoving + y_slot(q)) * kLanes + lane] = Pq;
      }
      if (j >= kHalo && j < kIn - kHalo) {
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
          qout[h][q] = fma_of<kExact>(k.cQg, g[q], k.kQ[wclass(q)] * E[q]);
          if (kForce) qout[h][q] = fma_of<kExact>(static_cast<Real>(p.cQF), Fq[q], qout[h][q]);
          if constexpr (!kExact) asm volatile("" : "+v"(qout[h][q]));
        }
      }
    }
  }
  if (kWalls && threadIdx.x < 4 * kQ) {
    tX[threadIdx.x] = xbv;
    if (threadIdx.x < 8) tU[threadIdx.x >> 1][threadIdx.x & 1] = uwv;
  }
  __syncthreads();

  // ---- phase 2: S and R of all but the outer two rows.
  Real R[kH][kQ];
#pragma unroll
  for (int h = 0; h < kH; ++h) {
    const int j = w + kWaves * h;
    if (j < 2 || j >= kIn - 2) continue;
    Real* slot = tR + (j - 2) * kYMoving * kLanes + lane;
    const int r = y_of(h);
    if (!interior_row(h)) {
      // Wall rows are written from the interior rows next to them; rows past
      // them are zero.
      if (r < 0 || r >= ny) {
#pragma unroll
        for (int q = 0; q < kYMoving; ++q) slot[q * kLanes] = Real(0);
      }
      continue;
    }
    const int rm = p.per_y ? wrap_near(r, ny) : r;
    Real wyr[kWeightsPerNode];
    row_weights(weights_y<Real>(p), rm, wyr);
    const Real* rb[5];
#pragma unroll
    for (int o = 0; o < 5; ++o) rb[o] = tP + (j - 2 + o) * kYMoving * kLanes + lane;
    Real S[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const int pq = y_slot(q) * kLanes;
      const Real centre = ey_of(q) != 0 ? rb[2][pq] : pr[h][q];
      Real acc = Real(0);
      if (ex_of(q) > 0) acc = x_taps<0, kExact>(wxr, centre, acc);
      if (ex_of(q) < 0) acc = x_taps<1, kExact>(wxr, centre, acc);
      if (ey_of(q) != 0) {
        const int sy = ey_of(q) > 0 ? 0 : 1;
#pragma unroll
        for (int k2 = 0; k2 < kTaps; ++k2) acc = fma_of<kExact>(wyr[sy * kTaps + k2], rb[k2 + sy][pq], acc);
      }
      S[q] = q == 0 ? centre : fma_of<kExact>(k.A, acc, centre);
    }
    if (kSaveS && lane_o && col_interior && out_row(h)) {
      Real* sv = static_cast<Real*>(p.save_s);
      const unsigned boff =
          (static_cast<unsigned>(r) * static_cast<unsigned>(pitch) + static_cast<unsigned>(c)) *
          static_cast<unsigned>(sizeof(Real));
#pragma unroll
      for (int q = 0; q < kQ; ++q) *at_byte(sv + q * plane, boff) = S[q];
    }
    double s, jx, jy;
    moment_sums(S, s, jx, jy);
    Real rho, ux = Real(0), uy = Real(0), X[kQ];
    if constexpr (sizeof(Real) == 4 && !kForce) {
      moments_f32<kWalls>(s, jx, jy, rho, X);
    } else {
      if constexpr (kForce)
        forced_velocity<kExact>(s, jx, jy, p.half_h, p.Fx, p.Fy, rho, ux, uy);
      else
        velocity<kExact>(s, jx, jy, rho, ux, uy);
      eq_brackets<kExact>(ux, uy, X);
    }
    const Real d = static_cast<Real>(s);
#pragma unroll
    for (int q = 1; q < kQ; ++q) {
      const Real E = fma_of<kExact>(rho, X[q], d);
      Real Rq = fma_of<kExact>(k.cRs, S[q], k.kR[wclass(q)] * E);
      if (kForce) Rq = fma_of<kExact>(static_cast<Real>(p.cRF), force_term<kExact>(q, p, ux, uy, E), Rq);
      R[h][q] = Rq;
    }
    if (kWalls) {
      // Wall nodes whose nearest interior node is this one (eq 3.10 on
      // f(t*)).  A wall row's y-moving populations go to its row of tR (no
      // output reads the others, nor the corners); a wall column's values
      // are taken over by its own lane, and lanes past a wall column hold
      // zero.
      const Real r1 = Real(w_of(1)) * rho, r2 = Real(w_of(5)) * rho;
      const bool bottom = !p.per_y && r == 1, top = !p.per_y && r == ny - 2;
      const int jw = bottom ? j - 3 : j - 1;  // the wall row's row of tR
      if ((bottom || top) && jw >= 0 && jw < kMid) {
        const Real* Xb = tX + (bottom ? 2 : 3) * kQ;
        Real* wall = tR + jw * kYMoving * kLanes + lane;
#pragma unroll
        for (int q = 1; q < kQ; ++q)
          if (ey_of(q) != 0)
            wall[y_slot(q) * kLanes] = nee_r<kExact>(wclass(q) == 1 ? r1 : r2, X[q], Xb[q], R[h][q]);
      }
      if (side) {
#pragma unroll
        for (int q = 1; q < kQ; ++q) {
          const Real wr = wclass(q) == 1 ? r1 : r2;
          const Real lo = from_above(nee_r<kExact>(wr, X[q], tX[q], R[h][q]));
          const Real hi = from_below(nee_r<kExact>(wr, X[q], tX[kQ + q], R[h][q]));
          R[h][q] = col_interior ? R[h][q] : (c == 0 ? lo : (c == nx - 1 ? hi : Real(0)));
        }
      }
    }
#pragma unroll
    for (int q = 1; q < kQ; ++q)
      if (ey_of(q) != 0) slot[y_slot(q) * kLanes] = R[h][q];
  }
  __syncthreads();

  // ---- phase 3: the new state of the output rows.
#pragma unroll
  for (int h = 0; h < kH; ++h) {
    if (!out_row(h) || !interior_row(h)) continue;
    const int j = w + kWaves * h, o = y_of(h);
    Real wyr[kWeightsPerNode];
    row_weights(weights_y<Real>(p), o, wyr);
    const Real* rb[5];
#pragma unroll
    for (int k2 = 0; k2 < 5; ++k2) rb[k2] = tR + (j - kHalo + k2) * kYMoving * kLanes + lane;
    Real out[kQ];
    out[0] = qout[h][0];
#pragma unroll
    for (int q = 1; q < kQ; ++q) {
      const int pq = y_slot(q) * kLanes;
      const Real centre = ey_of(q) != 0 ? rb[2][pq] : R[h][q];
      Real acc = qout[h][q];
      const int sy = ey_of(q) > 0 ? 0 : 1;
      Real rows[kTaps] = {};
      if (ey_of(q) != 0) {
#pragma unroll
        for (int k2 = 0; k2 < kTaps; ++k2) rows[k2] = rb[k2 + sy][pq];
      }
      out[q] = full_taps<kExact>(q, wxr, wyr, centre, acc, [&](int k) { return rows[k]; });
    }
    if (lane_o && col_interior) {
      const unsigned boff =
          (static_cast<unsigned>(o) * static_cast<unsigned>(pitch) + static_cast<unsigned>(c)) *
          static_cast<unsigned>(sizeof(Store));
      store_node(dst, plane, boff, out);
    }
  }
  if (kWalls) {
    __syncthreads();  // the tile's stores are visible to the block
    piece_walls<kExact, false>(p, dst, x0, x1, y0, y1, threadIdx.x, kWaves * kLanes,
                             [&](int, int, int side, double& u, double& v) {
                               u = tU[side][0];
                               v = tU[side][1];
                             });
  }
}

// ---------------------------------------------------------------------------
// Single-stencil step: the scheme at A = 0, Guo's T1S2-FDLBM (Remark I).
// With h = 0 the half-step prediction is the identity (S = P) and the mid-step
// map returns its input (R = S), so the step is
//   f~^{n+1} = Q - dt xi . grad_m R,  R = P = [2 f~ + w f^eq + dt F] / (2 + w),
// R being the physical f^n (eqs 2.18-2.20).  R is pointwise, so one pass
// forms R and Q of a row, puts R in an LDS ring, and takes the stencil of the
// row four above.  Strips are those of step_kernel (56 outputs; the stencil
// uses 2 of the 4 halo columns each side), marched from 2 rows above the
// piece instead of 4.  Wall nodes of R take eq 3.10 from their
// nearest interior node, written by that node's lane; the new state's wall
// nodes are set after each piece (piece_walls), as in step_kernel.  Each
// output takes
// the same expressions in the same order as step_kernel at A = 0 (where
// S = P + 0 L(P) and R = 1 S + 0 E reproduce P).
//
// Ring hazards, with rows p0..p0+3 loaded in an iteration and one barrier per
// iteration between its two phases: phase 1 writes rows p0..p0+3 and, for
// eq 3.10, wall rows p0-1 and p0+4; phase 2 reads rows p0-6..p0+1.  Over 16
// slots the rows written in phase 1 of the next iteration (p0+3..p0+8) share
// no slot with the rows still being read in phase 2 of this one.
// ---------------------------------------------------------------------------
template <typename Store, bool kForce, bool kWalls>
__global__ __launch_bounds__(step_threads(kStorageOf<Store>, 0), (kMinWaves<Store, kForce, kWalls, 1>)) void single_step_kernel(
    StepParams p) {
  using Real = typename Cvt<Store>::R;
  constexpr bool kExact = false;  // no other kernel takes this step; see step_kernel
  constexpr int kSB = strips_per_block(kStorageOf<Store>, 0);
  constexpr int kThreads = step_threads(kStorageOf<Store>, 0);
  constexpr int kSizeR = kRing1 * (kQ - 1) * kLanes;
  __shared__ Real ringR_all[kSB * kSizeR];  // per strip: [slot][q-1][lane]

  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int half = kSB == 1 ? 0 : wave / kRowsPerIter;
  const int t = kSB == 1 ? wave : wave % kRowsPerIter;
  Real* const ringR = ringR_all + half * kSizeR;
  const int nx = p.nx, ny = p.ny;
  const Store* __restrict__ src = static_cast<const Store*>(p.src);
  Store* __restrict__ dst = static_cast<Store*>(p.dst);
  const long long plane = p.plane;

  for (int i = threadIdx.x; i < kSB * kSizeR; i += kThreads) ringR_all[i] = Real(0);

  // Work order and XCD-aware block map as in step_kernel.
  const int G = gridDim.x;
  const int L = (blockIdx.x % 8) * (G / 8) + blockIdx.x / 8;
  if (L >= p.nblocks) return;  // padding block: whole block, before any barrier
  const long long total = static_cast<long long>(p.nunits) * ny;
  const long long band_pieces = static_cast<long long>(p.nunits) * p.band;
  long long beg = total * L / p.nblocks;
  const long long end = total * (L + 1) / p.nblocks;

  while (beg < end) {  // uniform per block
    const int b = static_cast<int>(beg / band_pieces);
    const long long rem = beg - b * band_pieces;
    const int r0 = b * p.band;
    const int hb = min(p.band, ny - r0);
    const int strip = static_cast<int>(rem / hb) * kSB + half;
    const int y0 = r0 + static_cast<int>(rem % hb);
    const int y1 = static_cast<int>(min(static_cast<long long>(r0 + hb), y0 + (end - beg)));
    beg += y1 - y0;

    const int x0 = strip * kStripOut;
    const int x1 = min(x0 + kStripOut, nx);
    const int c = x0 - kHalo + lane;
    const int cm = p.per_x ? wrap(c, nx) : clampi(c, 0, nx - 1);
    Real wxr[kWeightsPerNode];
    {
      const Real* wx = weights_x<Real>(p);
#pragma unroll
      for (int k = 0; k < kWeightsPerNode; ++k) wxr[k] = wx[cm * kWeightsPerNode + k];
    }
    const bool col_interior = p.per_x || (c >= 1 && c <= nx - 2);
    const bool lane_o = lane >= kHalo && lane < kLanes - kHalo && c < x1;
    const bool src_xl = !p.per_x && c == 1;
    const bool src_xr = !p.per_x && c == nx - 2;

    Real qA[kQ], qB[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) qA[q] = qB[q] = Real(0);

    // Rows y0-2 .. y1+1 are needed, four per iteration from ybase = y0 - 2;
    // iteration it outputs the rows loaded in iteration it - 1 (so Q stays
    // in the registers of the wave that formed it).  Prefetches past the
    // last needed row repeat that row, which the cache still holds.
    const int ybase = y0 - kHalo1;
    const int ylast = y1 + kHalo1 - 1;
    const int niter = ((y1 - y0 + 1) / kRowsPerIter + 3) & ~1;

    Store gA[kQ], gB[kQ];
    const int pitch = static_cast<int>(p.pitch);
    auto load_row = [&](int pr, Store (&gb)[kQ]) {
      const int pc = min(pr, ylast);
      const int prm = p.per_y ? wrap_near(pc, ny) : clampi(pc, 0, ny - 1);
      const unsigned boff =
          (static_cast<unsigned>(prm) * static_cast<unsigned>(pitch) + static_cast<unsigned>(cm)) *
          static_cast<unsigned>(sizeof(Store));
      load_planes(src, plane * sizeof(Store), boff, gb);
    };
    load_row(ybase + t, gA);
    load_row(ybase + kRowsPerIter + t, gB);
    __syncthreads();  // ring zero-fill / previous piece complete

    auto iteration = [&](const int it, Store (&gb)[kQ], Real (&qnew)[kQ], const Real (&qold)[kQ]) {
      const int p0 = ybase + kRowsPerIter * it;

      // ---- phase 1: R (to LDS) and Q (registers) of row p0 + t.
      {
        const int pr = p0 + t;
        Real g[kQ];
#pragma unroll
        for (int q = 0; q < kQ; ++q) g[q] = Cvt<Store>::ld(gb[q]);
        load_row(pr + 2 * kRowsPerIter, gb);
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
        const auto& k = coef<Real>(p);
        Real R[kQ];
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
          const Real E = fma_of<kExact>(rho, X[q], d);
          Real Rq = fma_of<kExact>(k.cPg, g[q], k.kP[wclass(q)] * E);
          Real Qq = fma_of<kExact>(k.cQg, g[q], k.kQ[wclass(q)] * E);
          if (kForce) {
            const Real Fq = force_term<kExact>(q, p, ux, uy, E);
            Rq = fma_of<kExact>(static_cast<Real>(p.cPF), Fq, Rq);
            Qq = fma_of<kExact>(static_cast<Real>(p.cQF), Fq, Qq);
          }
          R[q] = Rq;
          qnew[q] = Qq;
        }
        const bool row_int = p.per_y || (pr >= 1 && pr <= ny - 2);
        if (row_int && col_interior) {
          Real* slot = ringR + (pr & (kRing1 - 1)) * (kQ - 1) * kLanes;
#pragma unroll
          for (int q = 1; q < kQ; ++q) slot[(q - 1) * kLanes + lane] = R[q];
          // Wall nodes whose nearest interior node is this one (eq 3.10;
          // corners take the diagonal neighbour), from the moments of R.
          const bool src_yb = !p.per_y && pr == 1;
          const bool src_yt = !p.per_y && pr == ny - 2;
          if (kWalls && (src_xl || src_xr || src_yb || src_yt)) {
            double s2, jx2, jy2;
            moment_sums(R, s2, jx2, jy2);
            Real rho2, ux2, uy2;
            velocity<kExact>(s2, jx2, jy2, rho2, ux2, uy2);
            Real X2[kQ];
            eq_brackets<kExact>(ux2, uy2, X2);
            for (int dy = -1; dy <= 1; ++dy) {
              if ((dy == -1 && !src_yb) || (dy == 1 && !src_yt)) continue;
              for (int dx = -1; dx <= 1; ++dx) {
                if ((dx == -1 && !src_xl) || (dx == 1 && !src_xr)) continue;
                if (dx == 0 && dy == 0) continue;
                // A source in the strip's edge lane has its wall node outside
                // the strip; no output of this strip reads it.
                if (lane + dx < 0 || lane + dx >= kLanes) continue;
                Real sh[kQ];
                nee_shift_x(rho2, X2, wall_brackets<Real>(p, wall_side_of(dx, dy)), sh);
                Real* slotW = ringR + ((pr + dy) & (kRing1 - 1)) * (kQ - 1) * kLanes;
#pragma unroll
                for (int q = 1; q < kQ; ++q) slotW[(q - 1) * kLanes + lane + dx] = R[q] + sh[q];
              }
            }
          }
        }
      }
      __syncthreads();

      // ---- phase 2: f~^{n+1} of row p0 - 4 + t (whole wave computes,
      // interior output lanes store).
      {
        const int o = p0 - kRowsPerIter + t;
        const bool row_ok = o >= y0 && o < y1 && (p.per_y || (o >= 1 && o <= ny - 2));
        if (row_ok) {
          Real wyr[kWeightsPerNode];
          row_weights(weights_y<Real>(p), o, wyr);
          const Real* rb[5];
#pragma unroll
          for (int k = 0; k < 5; ++k)
            rb[k] = ringR + ((o + k - 2) & (kRing1 - 1)) * (kQ - 1) * kLanes + lane;
          Real out[kQ];
          out[0] = qold[0];
#pragma unroll
          for (int q = 1; q < kQ; ++q) {
            const int pq = (q - 1) * kLanes;
            const Real centre = rb[2][pq];
            Real acc = qold[q];
            if (ex_of(q) > 0) acc = x_taps<0, kExact>(wxr, centre, acc);
            if (ex_of(q) < 0) acc = x_taps<1, kExact>(wxr, centre, acc);
            if (ey_of(q) != 0) {
              const int sy = ey_of(q) > 0 ? 0 : 1;
#pragma unroll
              for (int k = 0; k < kTaps; ++k) acc += wyr[sy * kTaps + k] * rb[k + sy][pq];
            }
            out[q] = acc;
          }
          if (lane_o && col_interior) {
            const unsigned boff =
                (static_cast<unsigned>(o) * static_cast<unsigned>(pitch) + static_cast<unsigned>(c)) *
                static_cast<unsigned>(sizeof(Store));
            store_node(dst, plane, boff, out);
          }
        }
      }
    };

    for (int it = 0; it < niter; it += 2) {
      iteration(it, gA, qA, qB);
      iteration(it + 1, gB, qB, qA);
    }
    __syncthreads();  // the next piece reuses the ring; the piece's stores are visible
    if (kWalls)
      piece_walls<kExact, false>(
          p, dst, x0, x1, y0, y1, threadIdx.x % kBlockThreads, kBlockThreads,
          [&](int c2, int r2, int, double& u, double& v) { wall_velocity(p, c2, r2, u, v); });
  }
}

// ---------------------------------------------------------------------------
// Auxiliary kernels: node-parallel, grid-stride.
// ---------------------------------------------------------------------------
template <typename Store>
__global__ __launch_bounds__(256) void init_macro_kernel(AuxParams a, Store* state,
                                                         const double* rho, const double* ux,
                                                         const double* uy, const double* grad) {
  const long long n = static_cast<long long>(a.nx) * a.ny;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n; i += 256LL * gridDim.x) {
    const int x = static_cast<int>(i % a.nx), y = static_cast<int>(i / a.nx);
    const double r = rho[i];
    double feq[kQ];
    feq_dev<double>(r - 1.0, r, ux[i], uy[i], feq);
    if (grad) {
      // eq 3.5 with rho0 = 1: rho0 w (2 tau + dt)/(2 c_s^2) xi_a xi_b d_a u_b
      const double dudx = grad[i], dudy = grad[n + i], dvdx = grad[2 * n + i],
                   dvdy = grad[3 * n + i];
      const double k = (2.0 * a.tau + a.dt) * 1.5;
#pragma unroll
      for (int q = 0; q < kQ; ++q) {
        const double cx = ex_of(q), cy = ey_of(q);
        const double contr = cx * cx * dudx + cx * cy * (dudy + dvdx) + cy * cy * dvdy;
        feq[q] -= w_of(q) * k * contr;
      }
    }
    const long long base = static_cast<long long>(y) * a.pitch + x;
#pragma unroll
    for (int q = 0; q < kQ; ++q) state[q * a.plane + base] = Cvt<Store>::st(feq[q]);
  }
}

template <typename Store>
__global__ __launch_bounds__(256) void load_dist_kernel(AuxParams a, Store* state,
                                                        const double* g) {
  const long long n = static_cast<long long>(a.nx) * a.ny;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n * kQ; i += 256LL * gridDim.x) {
    const long long q = i / n, j = i % n;
    const int x = static_cast<int>(j % a.nx), y = static_cast<int>(j / a.nx);
    state[q * a.plane + static_cast<long long>(y) * a.pitch + x] =
        Cvt<Store>::st(static_cast<typename Cvt<Store>::R>(g[i]));
  }
}

template <typename Store>
__global__ __launch_bounds__(256) void read_dist_kernel(AuxParams a, const Store* state,
                                                        double* g) {
  const long long n = static_cast<long long>(a.nx) * a.ny;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n * kQ; i += 256LL * gridDim.x) {
    const long long q = i / n, j = i % n;
    const int x = static_cast<int>(j % a.nx), y = static_cast<int>(j / a.nx);
    g[i] = static_cast<double>(
        Cvt<Store>::ld(state[q * a.plane + static_cast<long long>(y) * a.pitch + x]));
  }
}

template <typename Store>
__device__ inline void node_moments(const AuxParams& a, const Store* state, int x, int y,
                                    double& s, double& ux, double& uy, bool& finite) {
  const long long base = static_cast<long long>(y) * a.pitch + x;
  double v[kQ];
  finite = true;
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    v[q] = static_cast<double>(Cvt<Store>::ld(state[q * a.plane + base]));
    finite = finite && isfinite(v[q]);
  }
  double jx, jy;
  moment_sums(v, s, jx, jy);
  const double rho = 1.0 + s;
  ux = jx / rho + a.half_dt * a.Fx;
  uy = jy / rho + a.half_dt * a.Fy;
}

template <typename Store>
__global__ __launch_bounds__(256) void moments_kernel(AuxParams a, const Store* state,
                                                      double* drho, double* ux, double* uy) {
  const long long n = static_cast<long long>(a.nx) * a.ny;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n; i += 256LL * gridDim.x) {
    const int x = static_cast<int>(i % a.nx), y = static_cast<int>(i / a.nx);
    double s, u, v;
    bool fin;
    node_moments(a, state, x, y, s, u, v, fin);
    if (drho) drho[i] = s;
    if (ux) ux[i] = u;
    if (uy) uy[i] = v;
  }
}

// Deterministic two-pass reduction: fixed grid of kDiagBlocks blocks, each
// thread accumulates a fixed grid-stride subset, each wave reduces its lanes
// with wave_sum / wave_max, the block adds its four wave results in wave
// order, and one final block reduces the partials in a fixed order.
template <typename Store>
__global__ __launch_bounds__(256) void diag_partial_kernel(AuxParams a, const Store* state,
                                                           double* partials) {
  __shared__ double red[kDiagSlots][256 / kLanes];
  double acc[kDiagSlots] = {0, 0, 0, 0, 0, 0, 0, 0};
  const long long n = static_cast<long long>(a.nx) * a.ny;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n; i += 256LL * gridDim.x) {
    const int x = static_cast<int>(i % a.nx), y = static_cast<int>(i / a.nx);
    double s, u, v;
    bool fin;
    node_moments(a, state, x, y, s, u, v, fin);
    const double J = a.jx[x] * a.jy[y];
    const double rho = 1.0 + s;
    if (fin) {
      acc[0] += J * s;
      acc[1] += J * rho * 0.5 * (u * u + v * v);
      acc[2] = fmax(acc[2], sqrt(u * u + v * v));
      acc[4] += J * rho * u;
      acc[5] += J * rho * v;
    } else {
      acc[3] += 1.0;
    }
  }
  const int lane = threadIdx.x & (kLanes - 1), wave = threadIdx.x / kLanes;
#pragma unroll
  for (int k = 0; k < kDiagSlots; ++k) {
    const double v = k == 2 ? wave_max(acc[k]) : wave_sum(acc[k]);
    if (lane == 0) red[k][wave] = v;
  }
  __syncthreads();
  if (threadIdx.x < kDiagSlots) {
    const int k = threadIdx.x;
    double v = red[k][0];
    for (int w = 1; w < 256 / kLanes; ++w) v = k == 2 ? fmax(v, red[k][w]) : v + red[k][w];
    partials[blockIdx.x * kDiagSlots + k] = v;
  }
}

// Final pass: wave w reduces slots w, w + 4; lane l takes the partials of
// blocks l, l + 64, ... in that order, then the butterfly combines the
// lanes.  The loads of a lane are independent, so they are in flight
// together (a walk over the blocks one at a time waited out a cache round
// trip per block).
// The first nout slots go to result.
__global__ __launch_bounds__(256) void diag_final_kernel(const double* partials, int nblocks,
                                                         double* result, int nout) {
  const int lane = threadIdx.x & (kLanes - 1), wave = threadIdx.x / kLanes;
  for (int k = wave; k < kDiagSlots; k += 256 / kLanes) {  // uniform per wave
    double acc = 0.0;
    for (int b = lane; b < nblocks; b += kLanes) {
      const double v = partials[b * kDiagSlots + k];
      acc = (k == 2) ? fmax(acc, v) : acc + v;
    }
    acc = k == 2 ? wave_max(acc) : wave_sum(acc);
    if (lane == 0 && k < nout) result[k] = acc;
  }
}

// Sums for the global relative error of the velocity against a reference
// field (eq 3.6, and the residual form of Sec. 3C): slot 0 sum |u - u'|^2,
// slot 1 sum |u'|^2, slot 3 sum |u|^2, over all nodes, the other slots
// zero (slot 2 is a max in the final pass).  Same fixed partition and order
// as the diagnostics.
template <typename Store>
__global__ __launch_bounds__(256) void gre_partial_kernel(AuxParams a, const Store* state,
                                                          const double* uref,
                                                          const double* vref,
                                                          double* partials) {
  __shared__ double red[3][256 / kLanes];
  double acc[3] = {0.0, 0.0, 0.0};
  const long long n = static_cast<long long>(a.nx) * a.ny;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n; i += 256LL * gridDim.x) {
    const int x = static_cast<int>(i % a.nx), y = static_cast<int>(i / a.nx);
    double s, u, v;
    bool fin;
    node_moments(a, state, x, y, s, u, v, fin);
    const double ur = uref[i], vr = vref[i];
    const double du = u - ur, dv = v - vr;
    acc[0] += du * du + dv * dv;
    acc[1] += ur * ur + vr * vr;
    acc[2] += u * u + v * v;
  }
  const int lane = threadIdx.x & (kLanes - 1), wave = threadIdx.x / kLanes;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double v = wave_sum(acc[k]);
    if (lane == 0) red[k][wave] = v;
  }
  __syncthreads();
  if (threadIdx.x < kDiagSlots) {
    const int k = threadIdx.x;
    double v[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      v[j] = red[j][0];
      for (int w = 1; w < 256 / kLanes; ++w) v[j] += red[j][w];
    }
    partials[blockIdx.x * kDiagSlots + k] =
        k == 0 ? v[0] : (k == 1 ? v[1] : (k == 3 ? v[2] : 0.0));
  }
}

template <typename Store, int kScheme>
void launch_fused(const StepParams& p, dim3 g, dim3 b, hipStream_t s, bool walls) {
  if (p.has_force) {
    if (walls)
      hipLaunchKernelGGL((step_kernel<Store, true, true, kScheme>), g, b, 0, s, p);
    else
      hipLaunchKernelGGL((step_kernel<Store, true, false, kScheme>), g, b, 0, s, p);
  } else {
    if (walls)
      hipLaunchKernelGGL((step_kernel<Store, false, true, kScheme>), g, b, 0, s, p);
    else
      hipLaunchKernelGGL((step_kernel<Store, false, false, kScheme>), g, b, 0, s, p);
  }
}

template <typename Store>
void launch_single(const StepParams& p, dim3 g, dim3 b, hipStream_t s, bool walls) {
  if (p.has_force) {
    if (walls)
      hipLaunchKernelGGL((single_step_kernel<Store, true, true>), g, b, 0, s, p);
    else
      hipLaunchKernelGGL((single_step_kernel<Store, true, false>), g, b, 0, s, p);
  } else {
    if (walls)
      hipLaunchKernelGGL((single_step_kernel<Store, false, true>), g, b, 0, s, p);
    else
      hipLaunchKernelGGL((single_step_kernel<Store, false, false>), g, b, 0, s, p);
  }
}

template <typename Store, bool kSaveS, int kH>
void launch_tile_h(const StepParams& p, hipStream_t s) {
  constexpr int kRows = tile_rows<Store, kH>();
  const dim3 g(p.nstrips * ((p.ny + kRows - 1) / kRows)), b(tile_waves<Store, kH>() * kLanes);
  const bool walls = !p.per_x || !p.per_y;
  if constexpr (!kSaveS) {
    if (p.has_force) {
      if (walls)
        hipLaunchKernelGGL((tile_step_kernel<Store, true, true, false, kH>), g, b, 0, s, p);
      else
        hipLaunchKernelGGL((tile_step_kernel<Store, true, false, false, kH>), g, b, 0, s, p);
      return;
    }
  }
  if (walls)
    hipLaunchKernelGGL((tile_step_kernel<Store, false, true, kSaveS, kH>), g, b, 0, s, p);
  else
    hipLaunchKernelGGL((tile_step_kernel<Store, false, false, kSaveS, kH>), g, b, 0, s, p);
}

template <typename Store, bool kSaveS>
void launch_tile(const StepParams& p, hipStream_t s) {
  if (p.tile == 2)
    launch_tile_h<Store, kSaveS, 2>(p, s);
  else
    launch_tile_h<Store, kSaveS, 1>(p, s);
}

template <typename Store>
hipError_t launch_step_t(const StepParams& p, int grid, hipStream_t s) {
  const dim3 g(grid), b(step_threads(kStorageOf<Store>, p.single ? 0 : p.scheme));
  const bool walls = !p.per_x || !p.per_y;
  if (p.tile)
    launch_tile<Store, false>(p, s);
  else if (p.single)
    launch_single<Store>(p, g, b, s, walls);
  else if (p.scheme == 1)
    launch_fused<Store, 1>(p, g, b, s, walls);
  else if constexpr (kStochastic<Store>)
    return hipErrorInvalidValue;  // the stochastic forms run scheme 1 only
  else if (p.scheme == 2)
    launch_fused<Store, 2>(p, g, b, s, walls);
  else if (p.gen_bbar)
    launch_fused<Store, 4>(p, g, b, s, walls);
  else
    launch_fused<Store, 3>(p, g, b, s, walls);
  return hipGetLastError();
}

int aux_grid(long long n) {
  long long g = (n + 255) / 256;
  if (g > 4096) g = 4096;
  if (g < 1) g = 1;
  return static_cast<int>(g);
}

}  // namespace

size_t storage_bytes(int storage) {
  switch (storage) {
    case kF64: return 8;
    case kF32: return 4;
    case kBF16: return 2;
    case kF16: return 2;
    case kBF16Sr: return 2;
    case kF16Sr: return 2;
    default: return 0;
  }
}

#define T2S2_DISPATCH(storage, CALL)                                  \
  switch (storage) {                                                  \
    case kF64: { using Store = double; CALL; } break;                 \
    case kF32: { using Store = float; CALL; } break;                  \
    case kBF16: { using Store = Bf16; CALL; } break;                  \
    case kF16: { using Store = _Float16; CALL; } break;               \
    case kBF16Sr: { using Store = Bf16Sr; CALL; } break;              \
    case kF16Sr: { using Store = F16Sr; CALL; } break;                \
    default: return hipErrorInvalidValue;                             \
  }

template <typename Store, int kScheme>
int occupancy_s(bool force, bool walls) {
  int n = 0;
  hipError_t e;
  if (force)
    e = walls ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
                    &n, step_kernel<Store, true, true, kScheme>, step_threads(kStorageOf<Store>, kScheme), 0)
              : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                    &n, step_kernel<Store, true, false, kScheme>, step_threads(kStorageOf<Store>, kScheme), 0);
  else
    e = walls ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
                    &n, step_kernel<Store, false, true, kScheme>, step_threads(kStorageOf<Store>, kScheme), 0)
              : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                    &n, step_kernel<Store, false, false, kScheme>, step_threads(kStorageOf<Store>, kScheme), 0);
  return e == hipSuccess ? n : -1;
}

template <typename Store>
int occupancy_single(bool force, bool walls) {
  int n = 0;
  const int threads = step_threads(kStorageOf<Store>, 0);
  hipError_t e;
  if (force)
    e = walls ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, single_step_kernel<Store, true, true>, threads, 0)
              : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, single_step_kernel<Store, true, false>, threads, 0);
  else
    e = walls ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, single_step_kernel<Store, false, true>, threads, 0)
              : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, single_step_kernel<Store, false, false>, threads, 0);
  return e == hipSuccess ? n : -1;
}

template <typename Store>
int occupancy_t(bool force, bool walls, int scheme) {
  if (scheme == 0) return occupancy_single<Store>(force, walls);
  if (scheme == 1) return occupancy_s<Store, 1>(force, walls);
  if constexpr (kStochastic<Store>) {
    return -1;  // scheme 1 only
  } else {
    if (scheme == 2) return occupancy_s<Store, 2>(force, walls);
    if (scheme == 4) return occupancy_s<Store, 4>(force, walls);
    return occupancy_s<Store, 3>(force, walls);
  }
}

int step_blocks_per_cu(int storage, bool force, bool walls, int scheme) {
  switch (storage) {
    case kF64: return occupancy_t<double>(force, walls, scheme);
    case kF32: return occupancy_t<float>(force, walls, scheme);
    case kBF16: return occupancy_t<Bf16>(force, walls, scheme);
    case kF16: return occupancy_t<_Float16>(force, walls, scheme);
    case kBF16Sr: return occupancy_t<Bf16Sr>(force, walls, scheme);
    case kF16Sr: return occupancy_t<F16Sr>(force, walls, scheme);
    default: return -1;
  }
}

int step_tile_rows(int storage, int tile) {
  if (tile == 1) return tile_rows<float, 1>();
  return storage == kF64 ? tile_rows<double, 2>() : tile_rows<float, 2>();
}

hipError_t launch_step(int storage, const StepParams& p, int grid, hipStream_t s) {
  T2S2_DISPATCH(storage, return launch_step_t<Store>(p, grid, s));
  return hipSuccess;
}

// The adjoint's recompute: the unforced T2S2-FDLBM1-family step from p.src
// into p.dst, storing S into p.save_s as well.  The new state's wall nodes
// are not set (the adjoint reads it at interior nodes only).
template <typename Store>
hipError_t launch_step_save_s_t(const StepParams& p, int grid, hipStream_t s) {
  const dim3 g(grid), b(step_threads(kStorageOf<Store>, 1));
  if (p.tile) {
    launch_tile<Store, true>(p, s);
    return hipGetLastError();
  }
  if (!p.per_x || !p.per_y)
    hipLaunchKernelGGL((step_kernel<Store, false, true, 1, true>), g, b, 0, s, p);
  else
    hipLaunchKernelGGL((step_kernel<Store, false, false, 1, true>), g, b, 0, s, p);
  return hipGetLastError();
}

hipError_t launch_step_save_s(int storage, const StepParams& p, int grid, hipStream_t s) {
  if (p.has_force || p.scheme != 1 || p.single || !p.save_s) return hipErrorInvalidValue;
  // The adjoint covers the storage forms rounded to nearest.
  switch (storage) {
    case kF64: return launch_step_save_s_t<double>(p, grid, s);
    case kF32: return launch_step_save_s_t<float>(p, grid, s);
    case kBF16: return launch_step_save_s_t<Bf16>(p, grid, s);
    case kF16: return launch_step_save_s_t<_Float16>(p, grid, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_init_macro(int storage, const AuxParams& a, void* state, const double* rho,
                             const double* ux, const double* uy, const double* grad,
                             hipStream_t s) {
  const int grid = aux_grid(static_cast<long long>(a.nx) * a.ny);
  T2S2_DISPATCH(storage,
                hipLaunchKernelGGL(init_macro_kernel<Store>, dim3(grid), dim3(256), 0, s, a,
                                   static_cast<Store*>(state), rho, ux, uy, grad));
  return hipGetLastError();
}

hipError_t launch_load_dist(int storage, const AuxParams& a, void* state, const double* g,
                            hipStream_t s) {
  const int grid = aux_grid(static_cast<long long>(a.nx) * a.ny * kQ);
  T2S2_DISPATCH(storage, hipLaunchKernelGGL(load_dist_kernel<Store>, dim3(grid), dim3(256), 0,
                                            s, a, static_cast<Store*>(state), g));
  return hipGetLastError();
}

hipError_t launch_read_dist(int storage, const AuxParams& a, const void* state, double* g,
                            hipStream_t s) {
  const int grid = aux_grid(static_cast<long long>(a.nx) * a.ny * kQ);
  T2S2_DISPATCH(storage, hipLaunchKernelGGL(read_dist_kernel<Store>, dim3(grid), dim3(256), 0,
                                            s, a, static_cast<const Store*>(state), g));
  return hipGetLastError();
}

hipError_t launch_moments(int storage, const AuxParams& a, const void* state, double* drho,
                          double* ux, double* uy, hipStream_t s) {
  const int grid = aux_grid(static_cast<long long>(a.nx) * a.ny);
  T2S2_DISPATCH(storage, hipLaunchKernelGGL(moments_kernel<Store>, dim3(grid), dim3(256), 0, s,
                                            a, static_cast<const Store*>(state), drho, ux, uy));
  return hipGetLastError();
}

hipError_t launch_diagnostics(int storage, const AuxParams& a, const void* state,
                              double* partials, double* result, int nout, hipStream_t s) {
  T2S2_DISPATCH(storage,
                hipLaunchKernelGGL(diag_partial_kernel<Store>, dim3(kDiagBlocks), dim3(256), 0,
                                   s, a, static_cast<const Store*>(state), partials));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(diag_final_kernel, dim3(1), dim3(256), 0, s, partials, kDiagBlocks, result,
                     nout);
  return hipGetLastError();
}

hipError_t launch_velocity_error(int storage, const AuxParams& a, const void* state,
                                 const double* uref, const double* vref, double* partials,
                                 double* result, hipStream_t s) {
  T2S2_DISPATCH(storage,
                hipLaunchKernelGGL(gre_partial_kernel<Store>, dim3(kDiagBlocks), dim3(256), 0,
                                   s, a, static_cast<const Store*>(state), uref, vref, partials));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(diag_final_kernel, dim3(1), dim3(256), 0, s, partials, kDiagBlocks, result,
                     kDiagSlots);
  return hipGetLastError();
}

}  // namespace t2s2
