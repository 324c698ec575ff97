// Two time steps of the T2S2-FDLBM1 family in one pass over HBM (FP64
// storage, A > 0).
//
// Measured (us per step, single steps -> this kernel): Taylor-Green 4096^2
// 489 -> 348, 2048^2 137 -> 103, cavity 4097^2 532 -> 369, 2049^2 151 -> 117.
// At 4096^2 it reads 1.16 and writes 1.00 times the state per two steps (3.8
// TB/s), with the vector units 72% busy (75% of the instructions FP64); the
// 2049^2 cavity reads 1.53 and writes 1.00, 62% busy: bound by neither alone.
//
// A step reads and writes the state once, and at large meshes it runs at the
// memory's rate; taking two steps per pass halves that traffic.  A block is
// two waves that march the same 64-column strip down a range of rows: the
// first takes the state from memory through one step, the second takes the
// rows it produces through the next step and stores them, one row per wave
// and iteration, the second wave a few rows behind.  The two chained steps
// reach 8 columns and rows each side, so a strip has 48 output columns.
//
// Each wave keeps what its two stencils need of earlier rows in registers,
// not in LDS: P of the last four rows, and the output rows under way.  The
// output rows take their terms row by row (a row of R, once formed, is added
// to the three or four output rows whose stencil reads it), so R needs no
// history, and Q none beyond the accumulators it starts.  Populations with
// no, positive and negative y velocity are complete 2, 3 and 4 rows after
// their row was read (the rest population at once), and go out then; the
// first wave's go to an LDS ring of eight rows that the second wave reads.
// Every value takes the expressions of step_kernel, in its order, so the
// state is bitwise that of single steps.
#include <hip/hip_runtime.h>

#include <climits>

#include "t2s2_device.h"
#include "t2s2_internal.h"
#include "t2s2_step.h"

namespace t2s2 {
namespace {

constexpr int kPairHalo = 2 * kHalo;
constexpr int kPairWaves = 2;
constexpr int kHandRows = 8;  // rows of the ring between the two waves

typedef unsigned U32x2 __attribute__((ext_vector_type(2)));
constexpr int kNonTemporal = 2;  // buffer instruction cache policy: nt
// What a wave carries from row to row: P of the rows p-1 .. p-4 and the
// output rows p-1 .. p-4 under way, by row number modulo 4.
template <typename Real>
struct Stage {
  Real P[kQ][4];
  Real acc[kQ][4];
};

// Where a strip and a lane stand to the walls of a walled x axis.
struct WallLanes {
  bool has_l, has_r;  // the strip holds column 0, column nx - 1 (uniform)
  int c, last;        // this lane's column, nx - 1
};

// The kernel's parameters, read again from the kernarg segment at each call:
// the wall paths need more scalars than there are registers, and a scalar
// load costs less there than a spill to a vector register's lanes.
template <bool kAgain>
__device__ __forceinline__ const StepParams& params(const StepParams& p) {
  if (!kAgain) return p;
  auto k = (const __attribute__((address_space(4))) StepParams*)
      __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(k));
  return *(const StepParams*)k;
}

// On a periodic axis a node's weights for the two signs of the velocity are
// the same four in mirrored order, bit for bit (the wall-adjacent nodes of a
// walled axis, where one sign takes the central difference, break this), so
// the periodic kernels hold four.
template <bool kWalls, typename Real>
__device__ __forceinline__ void mirror_weights(Real* w) {
  if (kWalls) return;
#pragma unroll
  for (int k = 0; k < kTaps; ++k) w[kTaps + k] = w[kTaps - 1 - k];
}

// The y weights around R row r: [0..7] of its own stencil, [8..15] those
// with which its values enter the outputs around it (PairPlan::wy16),
// scalar loads at a wave-uniform row.
template <bool kWalls>
__device__ __forceinline__ void row_weights16(const double* table, int row, double (&w)[16]) {
  using CPtr = const __attribute__((address_space(4))) double*;
  CPtr t = (CPtr)(table) + row * 16;
  asm volatile("" : "+s"(t));
#pragma unroll
  for (int k = 0; k < 16; ++k)
    if (kWalls || k < 4 || (k >= 8 && k != 10 && k != 13)) w[k] = t[k];
  if (!kWalls) {
    mirror_weights<kWalls>(w);
    w[10] = w[13] = w[2];
  }
}

// One row of one step: g is row p of the step's input.  With do_mid, also
// S and R of row r = p - 2 and R's contributions to the outputs.  emit(q, d,
// v): the new value of population q of row p - d is v.  I = p modulo 4 (up
// to a constant offset), rm = r brought into the grid, bottom / top: r is
// next to a wall of the y axis; used() is called once g is no longer read.
template <int I, bool kForce, bool kWalls, typename Real, typename Used, typename Emit>
__device__ __forceinline__ void stage_row(const StepParams& p0, const double* wy16, Stage<Real>& st,
                                          const Real (&g)[kQ], const Real (&wx)[kWeightsPerNode],
                                          bool do_mid, int rm, bool bottom, bool top,
                                          const WallLanes& wl, Used used, Emit emit) {
  constexpr int i0 = I & 3, i1 = (I - 1) & 3, i2 = (I - 2) & 3, i3 = (I - 3) & 3;
  const StepParams& p = params<kWalls>(p0);
  const auto& k = coef<Real>(p);
  // The row's weights, asked for here and used after phase 1: the scalar
  // loads' latency would otherwise be waited out once per row.
  double w[16];
  row_weights16<kWalls>(wy16, rm, w);
  Real Pn[kQ], Qn[kQ];
  {
    double s, jx, jy;
    moment_sums(g, s, jx, jy);
    Real rho, ux, uy;
    velocity(s, jx, jy, rho, ux, uy);
    if (kForce) {
      ux = add_scaled(p.half_dt, p.Fx, ux);
      uy = add_scaled(p.half_dt, p.Fy, uy);
    }
    const Real d = static_cast<Real>(s);
    Real X[kQ];
    eq_brackets(ux, uy, X);
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const Real E = fma_of(rho, X[q], d);
      Pn[q] = fma_of(k.cPg, g[q], k.kP[wclass(q)] * E);
      Qn[q] = fma_of(k.cQg, g[q], k.kQ[wclass(q)] * E);
      if (kForce) {
        const Real Fq = force_term(q, p, ux, uy, E);
        Pn[q] = fma_of(static_cast<Real>(p.cPF), Fq, Pn[q]);
        Qn[q] = fma_of(static_cast<Real>(p.cQF), Fq, Qn[q]);
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);  // not above: g's registers are free only here
  used();
  emit(0, 0, Qn[0]);
#pragma unroll
  for (int q = 1; q < kQ; ++q)
    if (ey_of(q) >= 0) st.acc[q][i0] = Qn[q];

  if (!kWalls || do_mid) {
    Real S[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const Real centre = st.P[q][i2];
      Real acc = Real(0);
      if (ex_of(q) > 0) acc = x_taps<0>(wx, centre, acc);
      if (ex_of(q) < 0) acc = x_taps<1>(wx, centre, acc);
      if (ey_of(q) > 0) {
        acc = fma_of(w[0], st.P[q][i0], acc);  // row p - 4, not yet replaced
        acc = fma_of(w[1], st.P[q][i3], acc);
        acc = fma_of(w[2], centre, acc);
        acc = fma_of(w[3], st.P[q][i1], acc);
      } else if (ey_of(q) < 0) {
        acc = fma_of(w[4], st.P[q][i3], acc);
        acc = fma_of(w[5], centre, acc);
        acc = fma_of(w[6], st.P[q][i1], acc);
        acc = fma_of(w[7], Pn[q], acc);
      }
      S[q] = q == 0 ? centre : fma_of(k.A, acc, centre);
    }
    double s, jx, jy;
    moment_sums(S, s, jx, jy);
    Real rho, ux, uy;
    velocity(s, jx, jy, rho, ux, uy);
    if (kForce) {
      ux = add_scaled(p.half_h, p.Fx, ux);
      uy = add_scaled(p.half_h, p.Fy, uy);
    }
    const Real d = static_cast<Real>(s);
    Real X[kQ];
    eq_brackets(ux, uy, X);
    // Population by population, R and its contributions.  Wall nodes (eq
    // 3.10): this row's take R from the lane beside them; a wall row takes it
    // from this row, just before or after it (corners take the x wall's value
    // of this row, which is their diagonal neighbour's).
    double wb[16];  // weights of the wall row beside this one
    const bool wall_row = kWalls && __builtin_expect(bottom || top, 0);
    if (wall_row) row_weights16<kWalls>(wy16, bottom ? 0 : p.ny - 1, wb);
    const Real* xw = kWalls ? wall_brackets<Real>(p, bottom ? 2 : 3) : nullptr;
#pragma unroll
    for (int q = 1; q < kQ; ++q) {
      const Real E = fma_of(rho, X[q], d);
      Real R = fma_of(k.cRs, S[q], k.kR[wclass(q)] * E);
      if (kForce) R = fma_of(static_cast<Real>(p.cRF), force_term(q, p, ux, uy, E), R);
      const Real wr = Real(w_of(q)) * rho;
      if (kWalls && __builtin_expect(wl.has_l, 0)) {
        const Real v = from_above(nee_r(wr, X[q], wall_brackets<Real>(p, 0)[q], R));
        R = wl.c == 0 ? v : R;
      }
      if (kWalls && __builtin_expect(wl.has_r, 0)) {
        const Real v = from_below(nee_r(wr, X[q], wall_brackets<Real>(p, 1)[q], R));
        R = wl.c == wl.last ? v : R;
      }
      if (wall_row && bottom) {
        const bool corner = (wl.c == 0 && wl.has_l) || (wl.c == wl.last && wl.has_r);
        const Real Rw = corner ? R : nee_r(wr, X[q], xw[q], R);
        if (ey_of(q) > 0) {
          st.acc[q][i1] = fma_of(wb[8], Rw, st.acc[q][i1]);
          st.acc[q][i2] = fma_of(wb[9], Rw, st.acc[q][i2]);
        } else if (ey_of(q) < 0) {
          st.acc[q][i2] = fma_of(wb[12], Rw, st.acc[q][i2]);
        }
      }
      Real mid = st.acc[q][i2];
      if (ex_of(q) > 0) mid = x_taps<0>(wx, R, mid);
      if (ex_of(q) < 0) mid = x_taps<1>(wx, R, mid);
      if (ey_of(q) > 0) {
        st.acc[q][i0] = fma_of(w[8], R, st.acc[q][i0]);
        st.acc[q][i1] = fma_of(w[9], R, st.acc[q][i1]);
        mid = fma_of(w[10], R, mid);
        st.acc[q][i3] = fma_of(w[11], R, st.acc[q][i3]);
      } else if (ey_of(q) < 0) {
        st.acc[q][i1] = fma_of(w[12], R, st.acc[q][i1]);
        mid = fma_of(w[13], R, mid);
        st.acc[q][i3] = fma_of(w[14], R, st.acc[q][i3]);
        st.acc[q][i0] = fma_of(w[15], R, st.acc[q][i0]);  // row p - 4
      }
      st.acc[q][i2] = mid;
      if (wall_row && !bottom) {
        const bool corner = (wl.c == 0 && wl.has_l) || (wl.c == wl.last && wl.has_r);
        const Real Rw = corner ? R : nee_r(wr, X[q], xw[q], R);
        if (ey_of(q) > 0) {
          st.acc[q][i2] = fma_of(wb[11], Rw, st.acc[q][i2]);
        } else if (ey_of(q) < 0) {
          st.acc[q][i2] = fma_of(wb[14], Rw, st.acc[q][i2]);
          st.acc[q][i3] = fma_of(wb[15], Rw, st.acc[q][i3]);
        }
      }
    }
  }
#pragma unroll
  for (int q = 1; q < kQ; ++q)
    if (ey_of(q) == 0) emit(q, 2, st.acc[q][i2]);
#pragma unroll
  for (int q = 1; q < kQ; ++q)
    if (ey_of(q) > 0) emit(q, 3, st.acc[q][i3]);
#pragma unroll
  for (int q = 1; q < kQ; ++q)
    if (ey_of(q) < 0) emit(q, 4, st.acc[q][i0]);
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    if (ey_of(q) < 0) st.acc[q][i0] = Qn[q];
    st.P[q][i0] = Pn[q];
  }
}

// One piece: columns [x0, x1) (at most kPairOut) and rows [y0, y1) of the
// new state.  A (the first wave) reads rows pa0 .. pa1, one per iteration; B
// (the second) takes the rows in between from jb0, lag iterations later: a
// row of the ring is complete 4 rows after its first population was written;
// B reads it in the next iteration (walled: one later still, since a wall row
// is formed from the row after it) and marches it in the one after.  One
// barrier per iteration.  While A writes rows p (the rest population), p - 2,
// p - 3 and p - 4, B reads row p - 5 (walled: p - 6, at the walls the interior
// row beside them, past the top wall the slot of row p - 9, which is that of
// p - 1): never a slot of the eight that A writes.  kWalls: the piece may
// reach wall nodes, or nodes next to a wall.
template <bool kForce, bool kWalls>
__device__ __forceinline__ void march_piece(const StepParams& p, const double* wy16, double* hand,
                                            int lane, int role, int x0, int x1, int y0, int y1) {
  using Real = double;
  const int nx = p.nx, ny = p.ny;
  const bool per_x = !kWalls || p.per_x, per_y = !kWalls || p.per_y;
  const unsigned long long plane_bytes = static_cast<unsigned long long>(p.plane) * sizeof(Real);
  const unsigned long long pitch_bytes = static_cast<unsigned long long>(p.pitch) * sizeof(Real);
  const Real* __restrict__ src = static_cast<const Real*>(p.src);
  Real* __restrict__ dst = static_cast<Real*>(p.dst);
  const int c = x0 - kPairHalo + lane;
  const int cm = per_x ? wrap(c, nx) : clampi(c, 0, nx - 1);
  Real wx[kWeightsPerNode];
#pragma unroll
  for (int k = 0; k < kWeightsPerNode; ++k) wx[k] = p.wx[cm * kWeightsPerNode + k];
  mirror_weights<kWalls>(wx);
  const int src_lane = per_x ? lane : lane + clampi(c, 1, nx - 2) - c;
  const WallLanes wl{!per_x && x0 - kPairHalo <= 0, !per_x && x0 - kPairHalo + kLanes > nx - 1,
                     c, nx - 1};

  Stage<Real> st;
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
#pragma unroll
    for (int k = 0; k < 4; ++k) st.P[q][k] = st.acc[q][k] = Real(0);
  }

  // Rows in between: [jlo, jhi); those B needs of a walled axis are the
  // interior ones.
  const int jlo = y0 - kHalo, jhi = y1 + kHalo;
  const int pa0 = per_y ? jlo - kHalo : max(jlo - kHalo, 0);
  const int pa1 = (per_y ? jhi - 1 : min(jhi - 1, ny - 2)) + kHalo;
  const int jb0 = per_y ? jlo : max(jlo, 0);
  const int jb1 = jhi - 1;
  const int lag = (kWalls ? 7 : 6) + jb0 - pa0;
  const int niter = (jb1 - jb0 + lag + 1 + 3) & ~3;

  if (role == 0) {
    // ---- A: rows from memory, two iterations ahead in two buffers.
    unsigned voff = static_cast<unsigned>(cm) * static_cast<unsigned>(sizeof(Real));
    // The next row to load, in the grid; rows past pa1 repeat it.
    int nl = pa0, nlm = per_y ? wrap(pa0, ny) : min(pa0, ny - 1);
    auto load_row = [&](Real (&gb)[kQ]) {
      asm volatile("" : "+v"(voff));  // keeps the scalar-base form (see load_planes)
      load_planes(reinterpret_cast<const Real*>(reinterpret_cast<const char*>(src) +
                                                nlm * pitch_bytes),
                  plane_bytes, voff, gb);
      if (nl < pa1) {
        ++nl;
        nlm = nlm + 1 < ny ? nlm + 1 : (per_y ? 0 : nlm);
      }
    };
    // With walls one buffer: a second one does not fit the registers.
    Real gA[kQ], gB2[kQ];
    Real(&gB)[kQ] = kWalls ? gA : gB2;
    load_row(gA);
    if (!kWalls) load_row(gB);
    int rm = per_y ? wrap(pa0 - 2, ny) : 0;  // row pr - 2, in the grid
    auto row = [&](auto phase, int it, Real (&gb)[kQ]) {
      constexpr int I = decltype(phase)::value;
      const int pr = pa0 + it, r = pr - 2;
      // Every iteration forms a row, also past the last that is needed: those
      // go nowhere, and a branch around the row costs registers.
      const bool mid = r >= jlo - 2 && r < jhi + 2 && r >= 1 && r <= ny - 2;
      if (!per_y) rm = clampi(r, 0, ny - 1);
      stage_row<I, kForce, kWalls>(
          p, wy16, st, gb, wx, per_y || mid, rm, !per_y && r == 1, !per_y && r == ny - 2, wl,
          [&]() { load_row(gb); },
          [&](int q, int d, Real v) {
            hand[(((pr - d) & (kHandRows - 1)) * kQ + q) * kLanes + lane] = v;
          });
      rm = rm + 1 < ny ? rm + 1 : 0;
      __syncthreads();
    };
    for (int it = 0; it < niter; it += 4) {
      row(std::integral_constant<int, 0>{}, it, gA);
      row(std::integral_constant<int, 1>{}, it + 1, gB);
      row(std::integral_constant<int, 2>{}, it + 2, gA);
      row(std::integral_constant<int, 3>{}, it + 3, gB);
    }
  } else {
    // ---- B: rows from the ring, the new state to memory.
    const bool lane_o = lane >= kPairHalo && c < x1 && lane < kLanes - kPairHalo &&
                        (per_x || (c >= 1 && c <= nx - 2));
    // (Rows are read at the nearest interior node; a wall node's state is
    // extrapolated from it below.)
    int rm = per_y ? wrap(jb0 - lag - 2, ny) : 0;  // row j - 2, in the grid
    // A row of the ring is read in the iteration before its use.
    Real g[kQ];
    auto read_row = [&](int j) {
      // (Rows past the top wall enter with weight zero: any finite row that A
      // does not write meanwhile will do, and it skips the slot of row j - 3.)
      const int js = per_y ? j : (j < ny ? clampi(j, 1, ny - 2) : j - 3);
      const Real* slot = hand + (js & (kHandRows - 1)) * kQ * kLanes + src_lane;
#pragma unroll
      for (int q = 0; q < kQ; ++q) g[q] = slot[q * kLanes];
    };
#pragma unroll
    for (int q = 0; q < kQ; ++q) g[q] = Real(0);
    // Stores go through a buffer descriptor of their row, whose bounds check
    // drops the lanes and rows that are not this piece's outputs: no branch
    // and no change of the execution mask in the march.
    const int voff = lane_o ? c * static_cast<int>(sizeof(Real)) : INT_MIN;
    auto row = [&](auto phase, int it) {
      constexpr int I = decltype(phase)::value;
      const int j = jb0 + it - lag;
      if (kWalls) {
        if (!per_y && j < jb0) {  // below the bottom wall: any finite values
#pragma unroll
          for (int q = 0; q < kQ; ++q) g[q] = Real(0);
        }
        if (__builtin_expect(wl.has_l || wl.has_r || (!per_y && (j < 1 || j > ny - 2)), 0)) {
          double s, jx, jy;
          moment_sums(g, s, jx, jy);
          const double rho = 1.0 + s;
          const double ir = recip(rho);
          const double ux = fma_of(jx, ir, p.half_dt * p.Fx);
          const double uy = fma_of(jy, ir, p.half_dt * p.Fy);
          double ub, vb;
          wall_velocity(p, c, j, ub, vb);
          Real shift[kQ];
          nee_shift(rho, ux, uy, ub, vb, shift);
          const bool wall = (!per_y && (j < 1 || j > ny - 2)) || src_lane != lane;
#pragma unroll
          for (int q = 0; q < kQ; ++q) g[q] = wall ? g[q] + shift[q] : g[q];
        }
      }
      const int r = j - 2;
      const bool mid = r >= y0 - 2 && r < y1 + 2 && r >= 1 && r <= ny - 2;
      if (!per_y) rm = clampi(r, 0, ny - 1);
      stage_row<I, kForce, kWalls>(
          p, wy16, st, g, wx, per_y || mid, rm, !per_y && r == 1, !per_y && r == ny - 2, wl,
          [&] { read_row(j + 1); },
          [&](int q, int d, Real v) {
            const int o = j - d;
            const bool ok = o >= y0 && o < y1 && (per_y || (o >= 1 && o <= ny - 2));
            const unsigned long long base =
                reinterpret_cast<unsigned long long>(dst) + (q * plane_bytes + o * pitch_bytes);
            const unsigned lo = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(base));
            const unsigned hi = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(base >> 32));
            const int bytes =
                __builtin_amdgcn_readfirstlane(ok ? static_cast<int>(pitch_bytes) : 0);
            const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
                reinterpret_cast<void*>((static_cast<unsigned long long>(hi) << 32) | lo), 0,
                bytes, 0x00020000);
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U32x2, v), rsrc, voff, 0,
                                                  kNonTemporal);
          });
      rm = rm + 1 < ny ? rm + 1 : 0;
      __syncthreads();
    };
    for (int it = 0; it < niter; it += 4) {
      row(std::integral_constant<int, 0>{}, it);
      row(std::integral_constant<int, 1>{}, it + 1);
      row(std::integral_constant<int, 2>{}, it + 2);
      row(std::integral_constant<int, 3>{}, it + 3);
    }
  }
}

// Main pieces: work order and XCD-aware block map as in step_kernel, over
// the strips of kPairOut columns from plan.x0 and the rows from plan.y0.
// With walls (kFrame) these stay 8 nodes clear of them, and run the code
// without wall paths; the frame around them (the strips along the x walls,
// the rows along the y walls) goes to the grid's first plan.frame blocks, one
// piece each, whose pieces are shorter because the wall paths are slower
// (hundreds of scalar spills; in the main march they would slow every row).
template <bool kForce, bool kFrame>
__global__ __launch_bounds__(kPairWaves * kLanes, 2) void pair_step_kernel(StepParams p,
                                                                           PairPlan plan) {
  __shared__ double hand[kHandRows * kQ * kLanes];  // [slot][q][lane]
  const int lane = threadIdx.x & (kLanes - 1);
  const int role = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  int block = blockIdx.x;
  if (kFrame) {
    if (block < plan.frame) {
      const int nedge = plan.edge * plan.chunks;
      int x0, y0, y1;
      if (block < nedge) {
        // Along an x wall: edge strip 0 is the left one, the others the right.
        const int e = block / plan.chunks, k = block % plan.chunks;
        x0 = e == 0 ? 0 : plan.x0 + (plan.nunits + e - 1) * kPairOut;
        y0 = static_cast<int>(static_cast<long long>(p.ny) * k / plan.chunks);
        y1 = static_cast<int>(static_cast<long long>(p.ny) * (k + 1) / plan.chunks);
      } else {
        // Along a y wall: the bottom, then the top, of each main strip.
        const int k = block - nedge;
        if (p.per_y || k >= 2 * plan.nunits) return;  // padding block
        x0 = plan.x0 + (k >> 1) * kPairOut;
        y0 = (k & 1) == 0 ? 0 : plan.y0 + plan.rows;
        y1 = (k & 1) == 0 ? plan.y0 : p.ny;
      }
      if (y0 >= y1) return;  // empty piece (few rows): whole block, before any barrier
      const int x1 = min(x0 + kPairOut, p.nx);
      march_piece<kForce, true>(p, plan.wy16, hand, lane, role, x0, x1, y0, y1);
      __syncthreads();  // the piece's stores are visible to the block
      piece_walls<true, false>(p, static_cast<double*>(p.dst), x0, x1, y0, y1, threadIdx.x,
                               kPairWaves * kLanes, [&](int, int, int side, double& u, double& v) {
                                 u = p.uw[side][0];
                                 v = p.uw[side][1];
                               });
      return;
    }
    block -= plan.frame;
  }
  const int G = gridDim.x - (kFrame ? plan.frame : 0);
  const int L = (block % 8) * (G / 8) + block / 8;
  if (L >= plan.nblocks) return;  // padding block: whole block, before any barrier
  const long long total = static_cast<long long>(plan.nunits) * plan.rows;
  const long long band_pieces = static_cast<long long>(plan.nunits) * plan.band;
  long long beg = total * L / plan.nblocks;
  const long long end = total * (L + 1) / plan.nblocks;
  while (beg < end) {  // uniform per block
    const int b = static_cast<int>(beg / band_pieces);
    const long long rem = beg - b * band_pieces;
    const int r0 = b * plan.band;
    const int hb = min(plan.band, plan.rows - r0);
    const int strip = static_cast<int>(rem / hb);
    const int y0 = r0 + static_cast<int>(rem % hb);
    const int y1 = static_cast<int>(min(static_cast<long long>(r0 + hb), y0 + (end - beg)));
    beg += y1 - y0;
    const int x0 = plan.x0 + strip * kPairOut;
    march_piece<kForce, false>(p, plan.wy16, hand, lane, role, x0, min(x0 + kPairOut, p.nx),
                               plan.y0 + y0, plan.y0 + y1);
  }
}

template <typename F>
hipError_t with_pair_kernel(bool force, bool walls, F f) {
  if (force) return walls ? f(pair_step_kernel<true, true>) : f(pair_step_kernel<true, false>);
  return walls ? f(pair_step_kernel<false, true>) : f(pair_step_kernel<false, false>);
}

}  // namespace

hipError_t launch_pair_step(const StepParams& p, const PairPlan& plan, int grid, hipStream_t s) {
  return with_pair_kernel(p.has_force != 0, !p.per_x || !p.per_y, [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kPairWaves * kLanes), 0, s, p, plan);
    return hipGetLastError();
  });
}

int pair_blocks_per_cu(bool force, bool walls) {
  int n = 0;
  const hipError_t e = with_pair_kernel(force, walls, [&](auto kernel) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, kPairWaves * kLanes, 0);
  });
  return e == hipSuccess ? n : -1;
}

}  // namespace t2s2
