// C-ABI of the t2s2 library (declared in include/t2s2.h): argument checks,
// time step and stencil coefficients on the host, launch plan, ping-pong
// state.  The library allocates no device memory: the caller provides the
// two state buffers and the workspace.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/t2s2.h"
#include "t2s2_internal.h"

using namespace t2s2;

namespace {

thread_local std::string g_last_error;

int fail(int code, const std::string& msg) {
  g_last_error = msg;
  return code;
}

int hip_fail(hipError_t e, const char* where) {
  return fail(T2S2_ERR_HIP, std::string(where) + ": " + hipGetErrorString(e));
}

size_t align256(size_t b) { return (b + 255) & ~static_cast<size_t>(255); }

// Metric 1/x'(i) with x'(i) = (x[i+1] - x[i-1]) / 2 (period added across a
// periodic seam); zero on wall nodes, which are never differentiated.
std::vector<double> metric(const std::vector<double>& c, bool per, double period) {
  const int n = static_cast<int>(c.size());
  std::vector<double> m(n, 0.0);
  for (int i = 0; i < n; ++i) {
    double cm, cp;
    if (per) {
      cm = i == 0 ? c[n - 1] - period : c[i - 1];
      cp = i == n - 1 ? c[0] + period : c[i + 1];
    } else {
      if (i == 0 || i == n - 1) continue;
      cm = c[i - 1];
      cp = c[i + 1];
    }
    m[i] = 2.0 / (cp - cm);
  }
  return m;
}

// Row table of the two-step kernel from the y weights w (PairPlan::wy16).
std::vector<double> scatter_weights(const std::vector<double>& w, int n, bool per) {
  std::vector<double> t(static_cast<size_t>(n) * 16, 0.0);
  for (int r = 0; r < n; ++r) {
    double* o = &t[static_cast<size_t>(r) * 16];
    for (int k = 0; k < kWeightsPerNode; ++k)
      o[k] = w[static_cast<size_t>(r) * kWeightsPerNode + k];
    for (int s = 0; s < 2; ++s)
      for (int k = 0; k < kTaps; ++k) {
        int i = r - (s == 0 ? k - 2 : k - 1);  // the output whose tap k is row r
        if (per)
          i = (i % n + n) % n;
        else if (i < 0 || i >= n)
          continue;
        o[8 + s * kTaps + k] = w[static_cast<size_t>(i) * kWeightsPerNode + s * kTaps + k];
      }
  }
  return t;
}

// Trapezoid measure of each node (diagnostics).
std::vector<double> measure(const std::vector<double>& c, bool per, double period) {
  const int n = static_cast<int>(c.size());
  std::vector<double> J(n);
  for (int i = 0; i < n; ++i) {
    if (per) {
      const double cm = i == 0 ? c[n - 1] - period : c[i - 1];
      const double cp = i == n - 1 ? c[0] + period : c[i + 1];
      J[i] = 0.5 * (cp - cm);
    } else if (i == 0) {
      J[i] = 0.5 * (c[1] - c[0]);
    } else if (i == n - 1) {
      J[i] = 0.5 * (c[n - 1] - c[n - 2]);
    } else {
      J[i] = 0.5 * (c[i + 1] - c[i - 1]);
    }
  }
  return J;
}

// dt-scaled stencil weights of -xi_a d/dx_a per node: for each sign of the
// velocity component, the 4 taps of the mixed difference (eqs 2.36-2.38 with
// eta the upwind weight) times the metric.  sign > 0 taps at offsets
// (-2,-1,0,+1), sign < 0 at (-1,0,+1,+2).  At the first interior node of a
// walled axis the upwind point outside the domain is replaced by quadratic
// extrapolation, which turns that upwind difference into the central one.
std::vector<double> stencil_weights(const std::vector<double>& m, bool per, double eta,
                                    double dt) {
  const int n = static_cast<int>(m.size());
  std::vector<double> w(static_cast<size_t>(n) * kWeightsPerNode, 0.0);
  const double up_pos[kTaps] = {eta / 2.0, -(1.0 + 3.0 * eta) / 2.0, 3.0 * eta / 2.0,
                                (1.0 - eta) / 2.0};
  const double up_neg[kTaps] = {-(1.0 - eta) / 2.0, -3.0 * eta / 2.0, (1.0 + 3.0 * eta) / 2.0,
                                -eta / 2.0};
  const double cen_pos[kTaps] = {0.0, -0.5, 0.0, 0.5};
  const double cen_neg[kTaps] = {-0.5, 0.0, 0.5, 0.0};
  for (int i = 0; i < n; ++i) {
    if (!per && (i == 0 || i == n - 1)) continue;
    const double* ap = (!per && i == 1) ? cen_pos : up_pos;
    const double* an = (!per && i == n - 2) ? cen_neg : up_neg;
    for (int k = 0; k < kTaps; ++k) {
      w[static_cast<size_t>(i) * kWeightsPerNode + k] = -dt * m[i] * ap[k];
      w[static_cast<size_t>(i) * kWeightsPerNode + kTaps + k] = dt * m[i] * an[k];
    }
  }
  return w;
}

bool check_axis(const double* c, int n, int per, double period, std::string& why) {
  for (int i = 0; i < n; ++i)
    if (!std::isfinite(c[i])) {
      why = "non-finite coordinate";
      return false;
    }
  for (int i = 1; i < n; ++i)
    if (!(c[i] > c[i - 1])) {
      why = "coordinates must be strictly increasing";
      return false;
    }
  if (per && !(std::isfinite(period) && period > c[n - 1] - c[0])) {
    why = "period must exceed the coordinate span";
    return false;
  }
  return true;
}

// Strip plan of the step kernel that p selects: strips of 56 output columns
// grouped into units of the kernel's strips per block.  The block count is
// set at bind time (plan_blocks).
void plan_strips(StepParams& p, int storage) {
  p.nstrips = (p.nx + kStripOut - 1) / kStripOut;
  const int spb = strips_per_block(storage, p.single ? 0 : p.scheme);
  p.nunits = (p.nstrips + spb - 1) / spb;
  p.nblocks = 8;
  p.band = p.ny;
}

// Band height of the march's split of nunits x ny unit-rows over nb blocks:
// one block's share, so that away from the last band a block owns one unit
// of one band.
int band_of(long long nunits, int ny, long long nb) {
  const long long rows = nunits * ny;
  return static_cast<int>(std::min<long long>(ny, std::max<long long>(1, (rows + nb - 1) / nb)));
}

// Work of the busiest block under that split, in unit-rows: the rows of its
// range plus kPieceWork for each piece the range is cut into at unit and
// band ends (a piece refills the march's pipeline: it loads the four rows
// above and below its range again and runs its leading and trailing
// iterations).  The ranges and pieces are enumerated as the step kernels
// cut them.  A last band of a few rows cuts each range that covers it into
// one piece per unit: on a 4060^2 grid in FP64 the default 512 blocks leave
// a last band of 7 rows and 74 pieces in the busiest range.
constexpr long long kPieceWork = 4;  // fitted to step times at 1101^2 - 4060^2
// The search stops at `limit` (a count already known to be worse), from the
// last range down, since the short last band is where the pieces are.
long long busiest_block_work(long long nunits, int ny, long long nb, long long piece_work,
                             long long limit) {
  const int band = band_of(nunits, ny, nb);
  const long long total = nunits * ny, band_rows = nunits * band;
  long long worst = 0;
  for (long long L = nb - 1; L >= 0 && worst < limit; --L) {
    long long beg = total * L / nb;
    const long long end = total * (L + 1) / nb;
    long long work = end - beg;
    while (beg < end) {
      const long long b = beg / band_rows, rem = beg - b * band_rows;
      const long long r0 = b * band, hb = std::min<long long>(band, ny - r0);
      const long long y0 = r0 + rem % hb;
      const long long y1 = std::min(r0 + hb, y0 + (end - beg));
      beg += y1 - y0;
      work += piece_work;
    }
    worst = std::max(worst, work);
  }
  return worst;
}

// Sets p's split of nunits x ny unit-rows to about nb blocks (a multiple of 8;
// unless forced, fewer where that makes the busiest block's work at least 3%
// less) and returns the block count.
template <typename Plan>  // StepParams or PairPlan
int set_blocks(Plan& p, int ny, long long nb, bool forced, long long piece_work) {
  const long long rows = static_cast<long long>(p.nunits) * ny;
  nb = std::max<long long>(8, nb / 8 * 8);
  nb = std::min<long long>(nb, std::max<long long>(8, rows / 8 * 8));
  if (!forced) {
    const long long w0 = busiest_block_work(p.nunits, ny, nb, piece_work, LLONG_MAX);
    long long best = nb, wbest = w0;
    for (long long c = nb - 8; c >= std::max<long long>(8, nb - nb / 4); c -= 8) {
      // No count below this one can do better: its equal share alone is more.
      if ((static_cast<long long>(p.nunits) * ny + c - 1) / c + piece_work >= wbest) break;
      const long long w = busiest_block_work(p.nunits, ny, c, piece_work, wbest);
      if (w < wbest) {
        wbest = w;
        best = c;
      }
    }
    if (wbest * 100 < w0 * 97) nb = best;
  }
  p.nblocks = static_cast<int>(nb);
  // The blocks of neighbouring units in a band march the same rows at the
  // same time, so the halo lines they share are fetched once.
  p.band = band_of(p.nunits, ny, nb);
  return static_cast<int>(nb);
}

// One block per resident slot (CUs x blocks per CU), so every block runs in
// a single wave of the grid with an equal share of the unit-rows (a unit is
// the block's group of neighbouring strips), as long as a share keeps at
// least 8 unit-rows.  Smaller meshes, where a block's march is a few
// latency-bound iterations, use one block per CU (equal work on every CU)
// while a share keeps at least 4 unit-rows, and below that one block per 4
// unit-rows.  A multiple of 8 for the XCD-aware block order.  Where that
// count cuts the ranges into many pieces, a count up to a quarter smaller
// whose busiest block does at least 3% less work (busiest_block_work) is
// taken instead: a step lasts as long as its busiest block, since with
// fewer blocks than slots each block marches at about the same rate.
// Returns the grid size, or -1 if the kernel cannot be resident.
int plan_blocks(StepParams& p, int storage, int cus) {
  const bool walls = !p.per_x || !p.per_y;
  // Kernel scheme codes: 0 the single-stencil step, 4 the family with
  // collision weights other than (1/2, 0, 1/2).
  const int kscheme = p.single ? 0 : (p.scheme == 3 && p.gen_bbar ? 4 : p.scheme);
  const int per_cu = step_blocks_per_cu(storage, p.has_force != 0, walls, kscheme);
  if (per_cu < 1) return -1;
  const long long rows = static_cast<long long>(p.nunits) * p.ny;
  const long long slots = static_cast<long long>(cus) * per_cu;
  long long nb = rows >= 8 * slots ? slots : (rows >= 4LL * cus ? cus : rows / 4);
  const char* forced = std::getenv("T2S2_BLOCKS");
  if (forced) nb = std::atoll(forced);
  return set_blocks(p, p.ny, nb, forced != nullptr, kPieceWork);
}

// Rows that a piece costs the two-step kernel beyond its own: eight above
// and eight below it are read again, and the second wave starts ten
// iterations after the first.
constexpr long long kPairPieceWork = 25;
// Time of a row of the frame's pieces (the wall paths) over a main row's:
// along the x walls, where every row takes them, and along the y walls.
// (Cavity 2049^2: 115.9 us per step at 1.5 / 1.5, 116.2 at 2 / 2, 118.4 at
// 3 / 2.5; 4097^2: 375.8 at 2 / 1.5, 381.7 at 3 / 2.)
constexpr double kPairEdgeCost = 2.0, kPairTopCost = 1.5;
// Estimated us of a step by the march, W unit-rows (pieces included) in the
// busiest of nb blocks per CU, march[0] + W (march[1] + march[2] nb); by n
// one-row tiles per CU (two at a time), one[0] + one[1] n + one[2] ceil(n / 2);
// and by n two-row tiles per CU, two[0] + two[1] n + two[2] ceil(n).
struct StepTimes {
  double march[3], one[3], two[3];
};
// Fitted by walls and force to 900 measured cases of 2 to 12 one-row tiles per
// CU, with sides up to 1 : 13 (residuals 3 to 6%, two-row tiles of the narrower
// forms with walls 5 to 9%).
constexpr StepTimes kTimes64[2][2] = {  // [walls][force]
    {{{8.53, 0.39, 0.21}, {1.96, 5.36, 2.65}, {0.34, 3.10, 7.47}},
     {{7.49, 0.86, 0.04}, {1.98, 5.79, 2.66}, {0.30, 3.05, 8.00}}},
    {{{11.22, 0.37, 0.24}, {5.08, 5.53, 1.89}, {3.80, 3.95, 6.14}},
     {{12.39, 0.56, 0.19}, {4.71, 5.59, 2.60}, {2.94, 3.67, 7.25}}}};
constexpr StepTimes kTimes32[2][2] = {
    {{{9.32, 0.13, 0.34}, {4.84, 2.19, 1.18}, {3.51, 4.95, 3.52}},
     {{8.68, 0.40, 0.20}, {6.21, 2.51, 0.81}, {3.33, 5.49, 4.27}}},
    {{{8.60, 0.33, 0.29}, {6.61, 2.02, 0.88}, {4.01, 4.16, 4.25}},
     {{10.28, 0.45, 0.16}, {7.15, 2.64, 0.39}, {3.81, 4.71, 4.86}}}};
constexpr StepTimes kTimes16[2][2] = {
    {{{8.69, 0.23, 0.14}, {5.96, 1.51, 1.34}, {5.44, 2.47, 4.03}},
     {{8.00, 0.27, 0.17}, {6.33, 1.32, 2.27}, {4.95, 1.03, 6.34}}},
    {{{9.51, 0.32, 0.13}, {7.15, 1.35, 1.42}, {5.24, 2.37, 4.43}},
     {{9.78, 0.37, 0.14}, {6.97, 1.63, 1.64}, {6.44, 2.05, 5.34}}}};

// Which kernel takes single steps of scheme 1 with A > 0: the march (0) or
// tiles of one row per wave (1) or two (2).  A CU holds one tile of either shape
// in FP64, two one-row tiles or one two-row tile in the narrower forms; the
// two-row tiles spend less on halo rows, but fewer of them may leave CUs idle.
// One-row tiles while each CU gets at most one (FP64 cavity 321^2 10.6 / 12.4
// us, one row / two), two in the narrower forms; FP64 then two-row tiles while
// they take about one round (385^2 16.1 / 12.9), the narrower forms while they
// take one (FP32 cavity 470^2 13.6 / 12.4); beyond, up to twelve one-row tiles
// per CU, the least estimate, the march's counted 2 to 5% less: of those 900
// cases 14 are then more than 1% slower than the march, and the choice is 0.9%
// above the best on average.  By counts of tiles alone FP32 on periodic grids
// took the march from six tiles per CU (879 x 883 26.9 us per step, 22.8 by
// tiles), and FP64 with walls two-row tiles up to four (channel 848 x 840 42.8,
// 36.1 by the march).  sp holds the march's plan.
int plan_tile(const StepParams& sp, int storage, int cus) {
  const int walls = !sp.per_x || !sp.per_y ? 1 : 0, force = sp.has_force ? 1 : 0;
  auto per_cu = [&](int kind) {
    const int rows = step_tile_rows(storage, kind);
    return static_cast<double>(sp.nstrips) * ((sp.ny + rows - 1) / rows) / cus;
  };
  const double n1 = per_cu(1), n2 = per_cu(2);
  const bool fp64 = storage == kF64;
  if (n1 <= 1.0) return 1;
  if (!fp64 && n1 <= 2.01) return 1;
  if (n2 <= (fp64 ? 1.1 : 1.0)) return 2;
  if (n1 > 12.0) return 0;
  const StepTimes& t = fp64              ? kTimes64[walls][force]
                       : storage == kF32 ? kTimes32[walls][force]
                                         : kTimes16[walls][force];
  const double w = static_cast<double>(
      busiest_block_work(sp.nunits, sp.ny, sp.nblocks, kPieceWork, LLONG_MAX));
  const double less = fp64 ? 0.98 : (storage == kF32 ? 0.95 : 0.97);
  const double march =
      less * (t.march[0] + w * (t.march[1] + t.march[2] * static_cast<double>(sp.nblocks) / cus));
  const double one = t.one[0] + t.one[1] * n1 + t.one[2] * std::ceil(n1 / 2);
  // (Two-row tiles that also store S cost the narrower forms more.)
  const double two =
      (fp64 ? 1.0 : 1.03) * (t.two[0] + t.two[1] * n2 + t.two[2] * std::ceil(n2));
  if (march <= std::min(one, two)) return 0;
  return one <= two ? 1 : 2;
}

// The two-step kernel takes meshes whose busiest block marches at least this
// many rows (piece work included); on smaller ones the rows read again cost
// more than the saved pass (Taylor-Green 1101^2, 50 rows, 52.1 us per step by
// single steps, 54.7).
constexpr long long kPairMinWork = 52;
// Beyond that, meshes where two single steps march at least this many times the
// rows of a two-step launch, each counted for the busiest block of its split,
// pieces included: what a row of the two-step march takes over one of the
// single step's, in blocks half as wide and twice as many per CU, by walls and
// force (a force costs the two-step march more, whose vector units are the
// busier).  Of 217 meshes from 800 x 1800 to 4096^2 and 60 x 20000 that its
// first rule took, none is slower by more than 0.3% than by single steps under
// this one, and it leaves gains of at most 6.7%; that rule, kPairMinWork alone,
// lost up to 33%.  us per step, single steps / two-step (ratio): Taylor-Green
// 1200^2 57 / 43 (2.33), 1300^2 62 / 64 (1.50), 4096^2 495 / 343 (2.88); with a
// force 300 x 4000 53 / 70 (1.38), 2500^2 221 / 192 (2.3); cavity 1200^2 61 / 65
// (1.24), 2049^2 151 / 114 (2.12); forced channel 1300^2 69 / 82 (1.52), 2500^2
// 224 / 200 (2.8).
constexpr double kPairRows[2][2] = {{1.52, 1.95}, {1.385, 1.82}};  // [walls][force]

// Steps of one launch of the one-block kernel: about a millisecond.
constexpr int64_t kMeshSteps = 256;

// Steps of a call from which one block takes them all, 0 if it never does.
// Meshes that fit one block, where a launch per step is mostly the launch;
// against the tile kernel, us per call (one block / tiles):
//   up to 512 nodes from two steps (FP64 forced channel 10 x 21, 2 steps 7 / 15,
//     20 steps 34 / 152; walled 16 x 32 14.7 / 18.2, 111 / 182);
//   beyond, where a thread holds half the registers, FP64 on periodic grids so
//     too (Taylor-Green 32^2, 2 steps 12.0 / 13.0, 20 steps 81 / 129); with walls
//     it spills, so only from 8 steps and up to 800 nodes (784 nodes, 8 steps
//     69.9 / 71.7, 20 steps 165 / 179; 900 nodes, 20 steps 183 / 178); with a
//     force never (channel 31 x 33, 20 steps 288 / 157);
//   the reduced forms with walls from three steps (1024 nodes, BF16, 2 steps 14.4
//     / 14.7, 3 steps 19.9 / 22.1, 20 steps 113 / 147).  Not on periodic grids,
//     where the compiler fuses the FP32 products of a step without a force in
//     another way than in the tile kernel, and stochastic rounding would turn
//     last-bit differences into whole units of the 16-bit forms.
int plan_mesh(const StepParams& sp, int storage) {
  const bool walls = !sp.per_x || !sp.per_y;
  const long long nodes = static_cast<long long>(sp.nx) * sp.ny;
  if (nodes > kMeshNodes || (storage != kF64 && !walls)) return 0;
  if (nodes <= kMeshNodes / 2) return 2;
  if (storage != kF64) return 3;
  if (sp.has_force || (walls && nodes > 800)) return 0;
  return walls ? 8 : 2;
}

// The two-step kernel's plan: the frame of a walled mesh and the main strips
// and rows inside it, over one block per resident slot, so that a frame
// piece and a main block's share take about the same time.  p holds the single
// step's plan.  Returns the grid, 0 if the mesh does not take the kernel.
// T2S2_PAIR_BLOCKS=n forces it with n main blocks (a hook for checking small
// meshes and ragged splits against single steps).
int plan_pair(const StepParams& p, PairPlan& plan, int cus) {
  const bool walls = !p.per_x || !p.per_y;
  const int per_cu = pair_blocks_per_cu(p.has_force != 0, walls);
  if (per_cu < 1) return 0;
  const long long slots = static_cast<long long>(cus) * per_cu / 8 * 8;
  const char* forced = std::getenv("T2S2_PAIR_BLOCKS");
  // Columns: the main strips keep 8 columns clear of a wall.
  plan.x0 = p.per_x ? 0 : kPairOut;
  plan.nunits = p.per_x ? (p.nx + kPairOut - 1) / kPairOut
                     : std::max(0, (p.nx - kPairOut - 2 * kHalo) / kPairOut);
  const int right = p.nx - plan.x0 - plan.nunits * kPairOut;  // columns right of the main strips
  plan.edge = p.per_x ? 0 : 1 + (right > 0 ? (right + kPairOut - 1) / kPairOut : 0);
  // Frame pieces of hx rows along the x walls and hy rows along the y
  // walls; returns the rows a main block marches over nb main blocks.
  auto split = [&](long long hx, long long hy, long long& nb) {
    plan.chunks = static_cast<int>((p.ny + hx - 1) / hx);
    plan.y0 = p.per_y ? 0 : static_cast<int>(std::max<long long>(2 * kHalo, hy));
    plan.rows = p.per_y ? p.ny : p.ny - 2 * plan.y0;
    if (plan.rows < 1) {  // few rows: the bottom pieces take them all
      plan.y0 = p.ny;
      plan.rows = 0;
    }
    const int pieces = plan.edge * plan.chunks + (p.per_y ? 0 : 2 * plan.nunits);
    plan.frame = (pieces + 7) / 8 * 8;
    nb = slots - plan.frame;
    const long long rows = static_cast<long long>(plan.nunits) * plan.rows;
    return nb < 8 ? -1 : (rows + nb - 1) / nb + kPairPieceWork;
  };
  long long nb = slots;
  if (forced) {
    split(17, 17, nb);
    nb = std::atoll(forced);
  } else {
    long long work = 0;
    for (long long t = kPairMinWork;; ++t) {
      if (t > p.ny + kPairPieceWork) return 0;
      auto rows = [&](double cost) {
        return std::max<long long>(2 * kHalo, static_cast<long long>(t / cost) - kPairPieceWork);
      };
      work = split(rows(kPairEdgeCost), rows(kPairTopCost), nb);
      if (work >= 0 && work <= t) break;
    }
    if (work < kPairMinWork) return 0;
  }
  if (static_cast<long long>(plan.nunits) * plan.rows == 0) {
    plan.nblocks = 0;
    plan.band = 1;
    return forced ? plan.frame : 0;
  }
  const int grid = plan.frame + set_blocks(plan, plan.rows, nb, forced != nullptr, kPairPieceWork);
  if (forced) return grid;
  const long long rows2 =
      busiest_block_work(plan.nunits, plan.rows, plan.nblocks, kPairPieceWork, LLONG_MAX);
  const long long rows1 = busiest_block_work(p.nunits, p.ny, p.nblocks, kPieceWork, LLONG_MAX);
  const double least = kPairRows[walls ? 1 : 0][p.has_force ? 1 : 0];
  return 2.0 * static_cast<double>(rows1) >= least * static_cast<double>(rows2) ? grid : 0;
}

}  // namespace

// Reduction partials of t2s2_diagnostics_noalloc: a file-scope device array
// (one copy per device, held until the process ends) instead of workspace
// memory.  In host code `scratch` names a host-side stand-in, not device
// memory; its device address comes from hipGetSymbolAddress, once per device
// (scratch_address), and only that address reaches the kernels.
constexpr int kNoAllocDoubles = kDiagBlocks * kDiagSlots;  // 32 KiB
static __device__ __align__(256) double scratch[kNoAllocDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_dev[kMaxDevices] = {};

// Device address of `scratch` on device dev, which must be current; looked
// up on the first call for that device (t2s2_bind) and kept.
hipError_t scratch_address(int dev, double** out) {
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_dev[dev] = static_cast<double*>(p);
  }
  *out = g_scratch_dev[dev];
  return hipSuccess;
}
}  // namespace

struct t2s2_ctx {
  t2s2_config cfg;
  int device = -1;  // device current at bind
  int nx = 0, ny = 0;
  long long pitch = 0;
  double dt = 0, tau = 0, omega = 0;
  std::vector<double> wx, wy, wy16, jx, jy;
  std::vector<float> wx32, wy32;
  size_t off_wx = 0, off_wy = 0, off_wy16 = 0, off_wx32 = 0, off_wy32 = 0, off_jx = 0, off_jy = 0,
         off_part = 0, off_res = 0, ws_bytes = 0;
  void* state[2] = {nullptr, nullptr};
  char* ws = nullptr;
  hipStream_t stream = nullptr;
  bool bound = false;
  int cur = 0;
  int64_t steps = 0;
  StepParams sp{};
  AuxParams ap{};
  int grid = 0;
  // The two-stencil kernels' plan of the same step (their own occupancy),
  // for the adjoint's recompute, which stores S, formed only by step_kernel
  // and tile_step_kernel; equal to sp unless sp.single.
  StepParams sp_gen{};
  int grid_gen = 0;
  // Plan of the two-step kernel; grid_pair 0: this context does not take it.
  PairPlan pair{};
  int grid_pair = 0;
  // One block takes all steps of a call of this many steps or more (0: never).
  int mesh_from = 0;
  // adjoint
  AdjParams adj{};
  bool adj_bound = false;
  double* adj_partial = nullptr;
  size_t adj_state_bytes = 0;
  // captured multi-step graph
  hipGraphExec_t graph = nullptr;
  int graph_steps = 0;
  int graph_cur = 0;  // buffer holding the state when the graph starts
  ~t2s2_ctx() {
    if (graph) (void)hipGraphExecDestroy(graph);
  }
};

namespace {
void drop_graph(t2s2_ctx* c) {
  if (c->graph) (void)hipGraphExecDestroy(c->graph);
  c->graph = nullptr;
  c->graph_steps = 0;
}
}  // namespace

extern "C" {

const char* t2s2_last_error(void) { return g_last_error.c_str(); }

int t2s2_create(const t2s2_config* cfg, const double* x, int nx, const double* y, int ny,
                t2s2_ctx** out) {
  g_last_error.clear();
  if (!out) return fail(T2S2_ERR_INVALID_ARG, "out is NULL");
  *out = nullptr;
  if (!cfg || !x || !y) return fail(T2S2_ERR_INVALID_ARG, "NULL config or coordinates");
  if (nx < 5 || ny < 5) return fail(T2S2_ERR_INVALID_ARG, "nx and ny must be >= 5");
  if (nx > (1 << 20) || ny > (1 << 20) || static_cast<long long>(nx) * ny > (1LL << 31))
    return fail(T2S2_ERR_INVALID_ARG, "mesh too large");
  std::string why;
  if (!check_axis(x, nx, cfg->periodic_x, cfg->period_x, why))
    return fail(T2S2_ERR_INVALID_ARG, "x: " + why);
  if (!check_axis(y, ny, cfg->periodic_y, cfg->period_y, why))
    return fail(T2S2_ERR_INVALID_ARG, "y: " + why);
  if (!(cfg->nu > 0.0)) return fail(T2S2_ERR_INVALID_ARG, "nu must be > 0 (or +INFINITY)");
  if (!(cfg->dt > 0.0) && !(cfg->cfl > 0.0 && cfg->cfl <= 1.0))
    return fail(T2S2_ERR_INVALID_ARG, "cfl must be in (0, 1] when dt <= 0");
  if (cfg->dt > 0.0 && !std::isfinite(cfg->dt)) return fail(T2S2_ERR_INVALID_ARG, "dt not finite");
  if (!(cfg->eta >= 0.0 && cfg->eta <= 1.0)) return fail(T2S2_ERR_INVALID_ARG, "eta not in [0,1]");
  if (!(cfg->A >= 0.0 && cfg->A <= 1.0)) return fail(T2S2_ERR_INVALID_ARG, "A not in [0,1]");
  if (cfg->storage < T2S2_F64 || cfg->storage > T2S2_F16_SR_DEV)
    return fail(T2S2_ERR_INVALID_ARG, "unknown storage");
  if (cfg->scheme != 0 && cfg->scheme != T2S2_FDLBM1 && cfg->scheme != T2S2_FDLBM2 &&
      cfg->scheme != T2S2_FAMILY)
    return fail(T2S2_ERR_INVALID_ARG, "unknown scheme");
  if ((cfg->storage == T2S2_BF16_SR_DEV || cfg->storage == T2S2_F16_SR_DEV) &&
      cfg->scheme != 0 && cfg->scheme != T2S2_FDLBM1)
    return fail(T2S2_ERR_UNSUPPORTED, "stochastically rounded storage runs T2S2_FDLBM1 only");
  if (cfg->scheme == T2S2_FAMILY) {
    const double* b = cfg->btilde;
    for (int k = 0; k < 3; ++k)
      if (!(b[k] >= 0.0 && b[k] <= (k == 2 ? 0.5 : 1.0)))
        return fail(T2S2_ERR_INVALID_ARG, "btilde: B~0, B~1 in [0,1], B~2 in [0,1/2]");
    if (!(std::fabs(b[0] + b[1] + b[2] - 1.0) <= 1e-12))
      return fail(T2S2_ERR_INVALID_ARG, "btilde must sum to 1 (eq 2.14a)");
    const double* bb = cfg->bbar;
    if (!(bb[0] == 0.0 && bb[1] == 0.0 && bb[2] == 0.0)) {
      for (int k = 0; k < 3; ++k)
        if (!(bb[k] >= 0.0 && bb[k] <= (k == 2 ? 0.5 : 1.0)))
          return fail(T2S2_ERR_INVALID_ARG, "bbar: B-0, B-1 in [0,1], B-2 in [0,1/2]");
      if (!(std::fabs(bb[0] + bb[1] + bb[2] - 1.0) <= 1e-12))
        return fail(T2S2_ERR_INVALID_ARG, "bbar must sum to 1 (eq 2.14a)");
    }
  }
  // The step kernel addresses a population plane with 32-bit byte offsets.
  if (static_cast<long long>(ny) * ((nx + 63) / 64 * 64) *
          static_cast<long long>(storage_bytes(cfg->storage)) >= (1LL << 32))
    return fail(T2S2_ERR_UNSUPPORTED, "one population plane (ny * pitch elements) must be under 4 GiB");
  if (!std::isfinite(cfg->force[0]) || !std::isfinite(cfg->force[1]))
    return fail(T2S2_ERR_INVALID_ARG, "force not finite");
  for (int s = 0; s < 4; ++s)
    if (!std::isfinite(cfg->u_wall[s][0]) || !std::isfinite(cfg->u_wall[s][1]))
      return fail(T2S2_ERR_INVALID_ARG, "wall velocity not finite");

  t2s2_ctx* c = new t2s2_ctx();
  c->cfg = *cfg;
  c->nx = nx;
  c->ny = ny;
  c->pitch = (nx + 63) / 64 * 64;
  std::vector<double> xs(x, x + nx), ys(y, y + ny);

  // eq 3.1 with xi = 1 and dx = the smallest node spacing over both axes.
  double dmin = INFINITY;
  for (int i = 1; i < nx; ++i) dmin = std::fmin(dmin, xs[i] - xs[i - 1]);
  for (int i = 1; i < ny; ++i) dmin = std::fmin(dmin, ys[i] - ys[i - 1]);
  if (cfg->periodic_x) dmin = std::fmin(dmin, xs[0] + cfg->period_x - xs[nx - 1]);
  if (cfg->periodic_y) dmin = std::fmin(dmin, ys[0] + cfg->period_y - ys[ny - 1]);
  c->dt = cfg->dt > 0.0 ? cfg->dt : cfg->cfl * dmin;
  c->tau = 3.0 * cfg->nu;
  c->omega = std::isinf(cfg->nu) ? 0.0 : c->dt / c->tau;

  const int scheme = cfg->scheme == T2S2_FDLBM2 ? 2 : (cfg->scheme == T2S2_FAMILY ? 3 : 1);
  c->cfg.scheme = scheme;
  // T2S2-FDLBM2 predicts with a full step (h = dt, A = 1 in the maps below)
  // and needs the physical f^n, which is P at A = 0.
  const double A = scheme == 2 ? 1.0 : cfg->A, Ap = scheme == 2 ? 0.0 : A;
  const double w = c->omega, dt = c->dt;
  StepParams& p = c->sp;
  p.scheme = scheme;
  // At A = 0 the half step is the identity and one stencil remains (T1S2).
  p.single = (scheme == 1 && A == 0.0) ? 1 : 0;
  p.nx = nx;
  p.ny = ny;
  p.pitch = c->pitch;
  p.plane = c->pitch * ny;
  p.per_x = cfg->periodic_x ? 1 : 0;
  p.per_y = cfg->periodic_y ? 1 : 0;
  p.A = A;
  // Closed forms of the pointwise maps in terms of w = dt / tau:
  //   P = fbar^{+,h} = [(2 - A w) f~ + (1 + A) w f^eq + (1 + A) dt F] / (2 + w)
  //   Q = f~^+       = [(2 - w) f~ + 2 w f^eq + 2 dt F] / (2 + w)
  //   R = f(t*)      = [2 S + A w f^eq* + A dt F*] / (2 + A w)
  p.cPg = (2.0 - Ap * w) / (2.0 + w);
  p.cPe = (1.0 + Ap) * w / (2.0 + w);
  p.cPF = (1.0 + Ap) * dt / (2.0 + w);
  p.cQg = (2.0 - w) / (2.0 + w);
  p.cQe = 2.0 * w / (2.0 + w);
  p.cQF = 2.0 * dt / (2.0 + w);
  p.cRs = 2.0 / (2.0 + A * w);
  p.cRe = A * w / (2.0 + A * w);
  p.cRF = A * dt / (2.0 + A * w);
  // The family (scheme 3) also takes f at h = dt from f~ or from fbar(t_{n+1}):
  //   U = [2 X + w f^eq + dt F] / (2 + w)  (f^n from f~^n, f^{n+1} from S2),
  // and weighs the three gradients by btilde.
  p.cUg = 2.0 / (2.0 + w);
  p.cUe = w / (2.0 + w);
  p.cUF = dt / (2.0 + w);
  for (int k = 0; k < 3; ++k) p.b[k] = scheme == 3 ? cfg->btilde[k] : (k == 1 ? 1.0 : 0.0);
  // Collision weights of the family (all zero: (1/2, 0, 1/2)).  Other than
  // (1/2, 0, 1/2), with w = dt / tau and Omega(f) dt = w (f^eq - f) + dt F:
  //   Q2 = f^n + B-0 dt Omega(f^n), f^n = cUg f~ + cUe f^eq + cUF F:
  //     cQ2g = (1 - B-0 w) cUg, cQ2e = (1 - B-0 w) cUe + B-0 w,
  //     cQ2F = (1 - B-0 w) cUF + B-0 dt;
  //   V = B-1 dt Omega(f*): cV = B-1 w, cVF = B-1 dt;
  //   f^{n+1} = [Y + B-2 (w f^eq + dt F)] / (1 + B-2 w) and
  //   f~ = f^{n+1} + (w/2) (f^{n+1} - f^eq) - (dt/2) F (eq 2.19):
  //     aY = (1 + w/2) / (1 + B-2 w), aE = w (B-2 - 1/2) / (1 + B-2 w),
  //     aF = dt (B-2 - 1/2) / (1 + B-2 w).
  {
    const double* bb = cfg->bbar;
    const bool zero = bb[0] == 0.0 && bb[1] == 0.0 && bb[2] == 0.0;
    const double b0 = zero ? 0.5 : bb[0], b1 = zero ? 0.0 : bb[1], b2 = zero ? 0.5 : bb[2];
    p.gen_bbar = (scheme == 3 && !(b0 == 0.5 && b1 == 0.0 && b2 == 0.5)) ? 1 : 0;
    p.bbar[0] = b0;
    p.bbar[1] = b1;
    p.bbar[2] = b2;
    p.cQ2g = (1.0 - b0 * w) * p.cUg;
    p.cQ2e = (1.0 - b0 * w) * p.cUe + b0 * w;
    p.cQ2F = (1.0 - b0 * w) * p.cUF + b0 * dt;
    p.cV = b1 * w;
    p.cVF = b1 * dt;
    p.aY = (1.0 + 0.5 * w) / (1.0 + b2 * w);
    p.aE = w * (b2 - 0.5) / (1.0 + b2 * w);
    p.aF = dt * (b2 - 0.5) / (1.0 + b2 * w);
    p.b2dt = b2 * dt;
    c->cfg.bbar[0] = b0;
    c->cfg.bbar[1] = b1;
    c->cfg.bbar[2] = b2;
  }
  {
    const double wc[3] = {4.0 / 9.0, 1.0 / 9.0, 1.0 / 36.0};
    p.c64.cPg = p.cPg;
    p.c64.cQg = p.cQg;
    p.c64.cRs = p.cRs;
    p.c64.A = A;
    p.c64.cU = p.cUg;
    for (int k = 0; k < 3; ++k) {
      p.c64.kP[k] = p.cPe * wc[k];
      p.c64.kQ[k] = p.cQe * wc[k];
      p.c64.kR[k] = p.cRe * wc[k];
      p.c64.kU[k] = p.cUe * wc[k];
      p.c64.b[k] = p.b[k];
      p.c64.kQ2[k] = p.cQ2e * wc[k];
      p.c64.kV[k] = p.cV * wc[k];
      p.c64.kA[k] = p.aE * wc[k];
    }
    p.c64.cQ2g = p.cQ2g;
    p.c64.cV = p.cV;
    p.c64.aY = p.aY;
    p.c32.cPg = static_cast<float>(p.c64.cPg);
    p.c32.cQg = static_cast<float>(p.c64.cQg);
    p.c32.cRs = static_cast<float>(p.c64.cRs);
    p.c32.A = static_cast<float>(A);
    p.c32.cU = static_cast<float>(p.c64.cU);
    for (int k = 0; k < 3; ++k) {
      p.c32.kP[k] = static_cast<float>(p.c64.kP[k]);
      p.c32.kQ[k] = static_cast<float>(p.c64.kQ[k]);
      p.c32.kR[k] = static_cast<float>(p.c64.kR[k]);
      p.c32.kU[k] = static_cast<float>(p.c64.kU[k]);
      p.c32.b[k] = static_cast<float>(p.c64.b[k]);
      p.c32.kQ2[k] = static_cast<float>(p.c64.kQ2[k]);
      p.c32.kV[k] = static_cast<float>(p.c64.kV[k]);
      p.c32.kA[k] = static_cast<float>(p.c64.kA[k]);
    }
    p.c32.cQ2g = static_cast<float>(p.c64.cQ2g);
    p.c32.cV = static_cast<float>(p.c64.cV);
    p.c32.aY = static_cast<float>(p.c64.aY);
  }
  p.half_dt = 0.5 * dt;
  p.half_h = 0.5 * A * dt;
  p.Fx = cfg->force[0];
  p.Fy = cfg->force[1];
  p.has_force = (cfg->force[0] != 0.0 || cfg->force[1] != 0.0) ? 1 : 0;
  for (int s = 0; s < 4; ++s) {
    p.uw[s][0] = cfg->u_wall[s][0];
    p.uw[s][1] = cfg->u_wall[s][1];
    // D2Q9 velocities in the paper's order (Sec. 3).
    static const int ex[kQ] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
    static const int ey[kQ] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
    const double ux = p.uw[s][0], uy = p.uw[s][1], uu = 1.5 * (ux * ux + uy * uy);
    for (int q = 0; q < kQ; ++q) {
      const double e = ex[q] * ux + ey[q] * uy;
      p.xb[s][q] = e * (3.0 + 4.5 * e) - uu;
      p.xb32[s][q] = static_cast<float>(p.xb[s][q]);
    }
  }

  c->wx = stencil_weights(metric(xs, cfg->periodic_x, cfg->period_x), cfg->periodic_x, cfg->eta, dt);
  c->wy = stencil_weights(metric(ys, cfg->periodic_y, cfg->period_y), cfg->periodic_y, cfg->eta, dt);
  c->wy16 = scatter_weights(c->wy, ny, cfg->periodic_y);
  c->wx32.assign(c->wx.begin(), c->wx.end());
  c->wy32.assign(c->wy.begin(), c->wy.end());
  c->jx = measure(xs, cfg->periodic_x, cfg->period_x);
  c->jy = measure(ys, cfg->periodic_y, cfg->period_y);

  // Launch plans; the block counts are set at bind time from the device's
  // CU count and the kernels' occupancy.
  plan_strips(p, cfg->storage);
  c->grid = 8;
  c->sp_gen = p;
  c->sp_gen.single = 0;
  plan_strips(c->sp_gen, cfg->storage);
  c->grid_gen = 8;

  size_t off = 0;
  c->off_wx = off;
  off = align256(off + c->wx.size() * sizeof(double));
  c->off_wy = off;
  off = align256(off + c->wy.size() * sizeof(double));
  c->off_wy16 = off;
  off = align256(off + c->wy16.size() * sizeof(double));
  c->off_wx32 = off;
  off = align256(off + c->wx32.size() * sizeof(float));
  c->off_wy32 = off;
  off = align256(off + c->wy32.size() * sizeof(float));
  c->off_jx = off;
  off = align256(off + c->jx.size() * sizeof(double));
  c->off_jy = off;
  off = align256(off + c->jy.size() * sizeof(double));
  c->off_part = off;
  off = align256(off + static_cast<size_t>(kDiagBlocks) * kDiagSlots * sizeof(double));
  c->off_res = off;
  off = align256(off + kDiagSlots * sizeof(double));
  c->ws_bytes = off;

  AuxParams& a = c->ap;
  a.nx = nx;
  a.ny = ny;
  a.pitch = c->pitch;
  a.plane = c->pitch * ny;
  a.tau = c->tau;
  a.dt = dt;
  a.half_dt = 0.5 * dt;
  a.Fx = cfg->force[0];
  a.Fy = cfg->force[1];
  *out = c;
  return T2S2_OK;
}

size_t t2s2_state_bytes(const t2s2_ctx* c) {
  if (!c) return 0;
  return static_cast<size_t>(kQ) * c->ny * c->pitch * storage_bytes(c->cfg.storage);
}

size_t t2s2_workspace_bytes(const t2s2_ctx* c) { return c ? c->ws_bytes : 0; }

int t2s2_bind(t2s2_ctx* c, void* state_a, void* state_b, void* workspace, void* stream) {
  g_last_error.clear();
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (!state_a || !state_b || !workspace || state_a == state_b)
    return fail(T2S2_ERR_INVALID_ARG, "need two distinct state buffers and a workspace");
  if ((reinterpret_cast<uintptr_t>(state_a) | reinterpret_cast<uintptr_t>(state_b) |
       reinterpret_cast<uintptr_t>(workspace)) & 255)
    return fail(T2S2_ERR_INVALID_ARG, "buffers must be 256-byte aligned");
  drop_graph(c);  // a captured graph holds the previous buffer addresses
  c->state[0] = state_a;
  c->state[1] = state_b;
  c->ws = static_cast<char*>(workspace);
  c->stream = static_cast<hipStream_t>(stream);
  hipError_t e;
  struct {
    size_t off;
    const void* src;
    size_t bytes;
  } up[] = {{c->off_wx, c->wx.data(), c->wx.size() * sizeof(double)},
            {c->off_wy, c->wy.data(), c->wy.size() * sizeof(double)},
            {c->off_wy16, c->wy16.data(), c->wy16.size() * sizeof(double)},
            {c->off_wx32, c->wx32.data(), c->wx32.size() * sizeof(float)},
            {c->off_wy32, c->wy32.data(), c->wy32.size() * sizeof(float)},
            {c->off_jx, c->jx.data(), c->jx.size() * sizeof(double)},
            {c->off_jy, c->jy.data(), c->jy.size() * sizeof(double)}};
  for (auto& u : up) {
    e = hipMemcpyAsync(c->ws + u.off, u.src, u.bytes, hipMemcpyHostToDevice, c->stream);
    if (e != hipSuccess) return hip_fail(e, "bind: upload");
  }
  e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return hip_fail(e, "bind: synchronize");
  c->sp.wx = reinterpret_cast<const double*>(c->ws + c->off_wx);
  c->sp.wy = reinterpret_cast<const double*>(c->ws + c->off_wy);
  c->pair.wy16 = reinterpret_cast<const double*>(c->ws + c->off_wy16);
  c->sp.wx32 = reinterpret_cast<const float*>(c->ws + c->off_wx32);
  c->sp.wy32 = reinterpret_cast<const float*>(c->ws + c->off_wy32);
  c->ap.jx = reinterpret_cast<const double*>(c->ws + c->off_jx);
  c->ap.jy = reinterpret_cast<const double*>(c->ws + c->off_jy);
  c->sp_gen.wx = c->sp.wx;
  c->sp_gen.wy = c->sp.wy;
  c->sp_gen.wx32 = c->sp.wx32;
  c->sp_gen.wy32 = c->sp.wy32;
  int dev = 0, cus = 0;
  e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return hip_fail(e, "bind: device query");
  c->device = dev;
  // The no-allocation diagnostics' scratch: its device address is looked up
  // here, at set-up with the device current, so that the entry point itself
  // (possibly under graph capture) makes no such call.
  if (dev < kMaxDevices) {
    double* scratch_dev = nullptr;
    e = scratch_address(dev, &scratch_dev);
    if (e != hipSuccess) return hip_fail(e, "bind: scratch address");
  }
  c->grid = plan_blocks(c->sp, c->cfg.storage, cus);
  c->grid_gen = c->sp.single ? plan_blocks(c->sp_gen, c->cfg.storage, cus) : c->grid;
  // Small meshes take the tile kernel (scheme 1, A > 0); not when the block
  // count is forced (T2S2_BLOCKS), which selects the march.  T2S2_TILE=0, 1 or
  // 2 forces the march or a tile shape.
  c->sp.tile = 0;
  if (c->sp.scheme == 1 && !c->sp.single && !std::getenv("T2S2_BLOCKS")) {
    c->sp.tile = plan_tile(c->sp, c->cfg.storage, cus);
    if (const char* t = std::getenv("T2S2_TILE"))
      if (t[0] >= '0' && t[0] <= '2') c->sp.tile = t[0] - '0';
  }
  if (!c->sp.single) c->sp_gen = c->sp;
  // T2S2_TILE selects single steps, T2S2_PAIR_BLOCKS the two-step kernel.
  const bool single_steps = std::getenv("T2S2_TILE") != nullptr;
  const bool two_steps = std::getenv("T2S2_PAIR_BLOCKS") != nullptr;
  c->mesh_from =
      c->sp.tile && !single_steps && !two_steps ? plan_mesh(c->sp, c->cfg.storage) : 0;
  c->grid_pair = 0;
  if (c->cfg.storage == T2S2_F64 && c->sp.scheme == 1 && !c->sp.single &&
      !std::getenv("T2S2_BLOCKS") && (!single_steps || two_steps))
    c->grid_pair = plan_pair(c->sp, c->pair, cus);
  if (c->grid < 1 || c->grid_gen < 1) return fail(T2S2_ERR_HIP, "bind: step kernel cannot be resident");
  c->bound = true;
  c->cur = 0;
  c->steps = 0;
  return T2S2_OK;
}

// Whether one block takes all nsteps steps of a call.
static bool takes_mesh(const t2s2_ctx* c, int64_t nsteps) {
  return c->mesh_from > 0 && nsteps >= c->mesh_from;
}

// Launches nsteps steps from buffer cur, which ends as the buffer that holds
// the result.  Where the two-step kernel applies, four steps at a time go as
// two launches of it, which end in the buffer they began in, as four single
// steps do.
static hipError_t launch_steps(t2s2_ctx* c, int64_t nsteps, int& cur, int64_t* taken) {
  if (takes_mesh(c, nsteps)) {
    // All of them in one block, at most kMeshSteps to a launch, which ends in
    // the buffer that as many single steps end in.
    for (int64_t left = nsteps; left > 0;) {
      const int n = static_cast<int>(std::min<int64_t>(left, kMeshSteps));
      c->sp.src = c->state[cur];
      if (n & 1) cur = 1 - cur;
      c->sp.dst = c->state[cur];
      const hipError_t e = launch_mesh_steps(c->cfg.storage, c->sp, n, c->stream);
      if (e != hipSuccess) {
        if (n & 1) cur = 1 - cur;
        return e;
      }
      left -= n;
      if (taken) *taken += n;
    }
    return hipSuccess;
  }
  const int64_t pairs = c->grid_pair > 0 ? 2 * (nsteps / 4) : 0;
  for (int64_t k = 0; k < pairs; ++k) {
    c->sp.src = c->state[cur];
    c->sp.dst = c->state[1 - cur];
    const hipError_t e = launch_pair_step(c->sp, c->pair, c->grid_pair, c->stream);
    if (e != hipSuccess) return e;
    cur = 1 - cur;
    if (taken) *taken += 2;
  }
  for (int64_t k = 2 * pairs; k < nsteps; ++k) {
    c->sp.src = c->state[cur];
    c->sp.dst = c->state[1 - cur];
    const hipError_t e = launch_step(c->cfg.storage, c->sp, c->grid, c->stream);
    if (e != hipSuccess) return e;
    cur = 1 - cur;
    if (taken) ++*taken;
  }
  return hipSuccess;
}

const char* t2s2_step_kernel(const t2s2_ctx* c, int64_t nsteps) {
  if (!c || !c->bound) return "";
  if (takes_mesh(c, nsteps)) return "mesh_steps_kernel";
  if (c->grid_pair > 0 && nsteps >= 4) return "pair_step_kernel";
  if (c->sp.tile) return "tile_step_kernel";
  return c->sp.single ? "single_step_kernel" : "step_kernel";
}

int t2s2_init_macro(t2s2_ctx* c, const double* rho, const double* ux, const double* uy,
                    const double* grad) {
  g_last_error.clear();
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (!c->bound) return fail(T2S2_ERR_NOT_BOUND, "context not bound");
  if (!rho || !ux || !uy) return fail(T2S2_ERR_INVALID_ARG, "NULL field");
  if (grad && std::isinf(c->cfg.nu))
    return fail(T2S2_ERR_INVALID_ARG, "eq 3.5 correction needs a finite tau");
  hipError_t e = launch_init_macro(c->cfg.storage, c->ap, c->state[c->cur], rho, ux, uy, grad,
                                   c->stream);
  if (e != hipSuccess) return hip_fail(e, "init_macro");
  c->steps = 0;
  return T2S2_OK;
}

int t2s2_init_distributions(t2s2_ctx* c, const double* g) {
  g_last_error.clear();
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (!c->bound) return fail(T2S2_ERR_NOT_BOUND, "context not bound");
  if (!g) return fail(T2S2_ERR_INVALID_ARG, "NULL distributions");
  hipError_t e = launch_load_dist(c->cfg.storage, c->ap, c->state[c->cur], g, c->stream);
  if (e != hipSuccess) return hip_fail(e, "init_distributions");
  c->steps = 0;
  return T2S2_OK;
}

int t2s2_step(t2s2_ctx* c, int64_t nsteps) {
  g_last_error.clear();
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (!c->bound) return fail(T2S2_ERR_NOT_BOUND, "context not bound");
  if (nsteps < 0) return fail(T2S2_ERR_INVALID_ARG, "nsteps < 0");
  const hipError_t e = launch_steps(c, nsteps, c->cur, &c->steps);
  if (e != hipSuccess) return hip_fail(e, "step");
  return T2S2_OK;
}

int t2s2_graph_capture(t2s2_ctx* c, int steps_per_graph) {
  g_last_error.clear();
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (!c->bound) return fail(T2S2_ERR_NOT_BOUND, "context not bound");
  if (steps_per_graph < 2 || (steps_per_graph & 1))
    return fail(T2S2_ERR_INVALID_ARG, "steps_per_graph must be even and >= 2");
  if (c->stream == nullptr)
    return fail(T2S2_ERR_UNSUPPORTED, "graph capture needs a non-default stream");
  drop_graph(c);
  hipError_t e = hipStreamBeginCapture(c->stream, hipStreamCaptureModeRelaxed);
  if (e != hipSuccess) return hip_fail(e, "graph capture: begin");
  // Record the launches of steps_per_graph steps; nothing executes, so the
  // host-side buffer index is advanced on a copy only.
  int cur = c->cur;
  const hipError_t le = launch_steps(c, steps_per_graph, cur, nullptr);
  hipGraph_t g = nullptr;
  e = hipStreamEndCapture(c->stream, &g);
  if (le != hipSuccess || e != hipSuccess) {
    if (g) (void)hipGraphDestroy(g);
    return hip_fail(le != hipSuccess ? le : e, "graph capture: launches");
  }
  hipGraphExec_t exec = nullptr;
  e = hipGraphInstantiate(&exec, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e != hipSuccess) return hip_fail(e, "graph capture: instantiate");
  c->graph = exec;
  c->graph_steps = steps_per_graph;
  c->graph_cur = c->cur;
  return T2S2_OK;
}

int t2s2_graph_step(t2s2_ctx* c, int64_t nsteps) {
  g_last_error.clear();
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (!c->bound) return fail(T2S2_ERR_NOT_BOUND, "context not bound");
  if (!c->graph) return fail(T2S2_ERR_NOT_BOUND, "no graph captured");
  if (nsteps < 0) return fail(T2S2_ERR_INVALID_ARG, "nsteps < 0");
  int64_t left = nsteps;
  int rc = T2S2_OK;
  // The graph reads the buffer that held the state at capture; an odd
  // number of plain steps since then is evened out with one plain step.
  if (left > 0 && c->cur != c->graph_cur) {
    if ((rc = t2s2_step(c, 1)) != T2S2_OK) return rc;
    --left;
  }
  while (left >= c->graph_steps) {
    hipError_t e = hipGraphLaunch(c->graph, c->stream);
    if (e != hipSuccess) return hip_fail(e, "graph launch");
    c->steps += c->graph_steps;  // an even count leaves c->cur unchanged
    left -= c->graph_steps;
  }
  return left > 0 ? t2s2_step(c, left) : T2S2_OK;
}

int t2s2_current(const t2s2_ctx* c) { return c ? c->cur : -1; }

int64_t t2s2_steps_taken(const t2s2_ctx* c) { return c ? c->steps : -1; }

double t2s2_dt(const t2s2_ctx* c) { return c ? c->dt : 0.0; }

int t2s2_moments(t2s2_ctx* c, double* drho, double* ux, double* uy) {
  g_last_error.clear();
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (!c->bound) return fail(T2S2_ERR_NOT_BOUND, "context not bound");
  hipError_t e =
      launch_moments(c->cfg.storage, c->ap, c->state[c->cur], drho, ux, uy, c->stream);
  if (e != hipSuccess) return hip_fail(e, "moments");
  return T2S2_OK;
}

int t2s2_read_distributions(t2s2_ctx* c, double* g) {
  g_last_error.clear();
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (!c->bound) return fail(T2S2_ERR_NOT_BOUND, "context not bound");
  if (!g) return fail(T2S2_ERR_INVALID_ARG, "NULL output");
  hipError_t e = launch_read_dist(c->cfg.storage, c->ap, c->state[c->cur], g, c->stream);
  if (e != hipSuccess) return hip_fail(e, "read_distributions");
  return T2S2_OK;
}

int t2s2_diagnostics(t2s2_ctx* c, double out[T2S2_NDIAG]) {
  g_last_error.clear();
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (!c->bound) return fail(T2S2_ERR_NOT_BOUND, "context not bound");
  if (!out) return fail(T2S2_ERR_INVALID_ARG, "NULL output");
  double* part = reinterpret_cast<double*>(c->ws + c->off_part);
  double* res = reinterpret_cast<double*>(c->ws + c->off_res);
  hipError_t e = launch_diagnostics(c->cfg.storage, c->ap, c->state[c->cur], part, res,
                                    kDiagSlots, c->stream);
  if (e != hipSuccess) return hip_fail(e, "diagnostics");
  double host[kDiagSlots];
  e = hipMemcpyAsync(host, res, sizeof(host), hipMemcpyDeviceToHost, c->stream);
  if (e != hipSuccess) return hip_fail(e, "diagnostics: copy");
  e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return hip_fail(e, "diagnostics: synchronize");
  for (int k = 0; k < T2S2_NDIAG; ++k) out[k] = host[k];
  if (host[3] > 0.0) return fail(T2S2_ERR_NONFINITE, "non-finite populations in the state");
  return T2S2_OK;
}

int t2s2_diagnostics_noalloc(t2s2_ctx* c, double* out) {
  g_last_error.clear();
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (!c->bound) return fail(T2S2_ERR_NOT_BOUND, "context not bound");
  if (!out || (reinterpret_cast<uintptr_t>(out) & 7))
    return fail(T2S2_ERR_INVALID_ARG, "out must be an 8-byte aligned device pointer");
  // The partials take kDiagBlocks * kDiagSlots doubles for any mesh (a
  // fixed grid of partial blocks), which the array holds.
  static_assert(kDiagBlocks * kDiagSlots <= kNoAllocDoubles, "scratch too small");
  if (c->device < 0 || c->device >= kMaxDevices)
    return fail(T2S2_ERR_UNSUPPORTED, "device index beyond the scratch table");
  int cur = -1;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return hip_fail(e, "diagnostics_noalloc: device query");
  if (cur != c->device && (e = hipSetDevice(c->device)) != hipSuccess)
    return hip_fail(e, "diagnostics_noalloc: set device");
  double* part = nullptr;
  e = scratch_address(c->device, &part);
  if (e == hipSuccess)
    e = launch_diagnostics(c->cfg.storage, c->ap, c->state[c->cur], part, out, T2S2_NDIAG,
                           c->stream);
  if (cur != c->device) (void)hipSetDevice(cur);
  if (e != hipSuccess) return hip_fail(e, "diagnostics_noalloc");
  return T2S2_OK;
}

int t2s2_velocity_error(t2s2_ctx* c, const double* ux_ref, const double* uy_ref,
                        double out[T2S2_NGRE]) {
  g_last_error.clear();
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (!c->bound) return fail(T2S2_ERR_NOT_BOUND, "context not bound");
  if (!ux_ref || !uy_ref || !out) return fail(T2S2_ERR_INVALID_ARG, "NULL reference or output");
  double* part = reinterpret_cast<double*>(c->ws + c->off_part);
  double* res = reinterpret_cast<double*>(c->ws + c->off_res);
  hipError_t e = launch_velocity_error(c->cfg.storage, c->ap, c->state[c->cur], ux_ref, uy_ref,
                                       part, res, c->stream);
  if (e != hipSuccess) return hip_fail(e, "velocity_error");
  double host[kDiagSlots];
  e = hipMemcpyAsync(host, res, sizeof(host), hipMemcpyDeviceToHost, c->stream);
  if (e != hipSuccess) return hip_fail(e, "velocity_error: copy");
  e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return hip_fail(e, "velocity_error: synchronize");
  out[0] = host[0];
  out[1] = host[1];
  out[2] = host[3];
  // E(u) of eq 3.6 (normalised by the reference) and the residual form of
  // Sec. 3C (normalised by the current field).
  out[3] = host[1] > 0.0 ? std::sqrt(host[0] / host[1]) : NAN;
  out[4] = host[3] > 0.0 ? std::sqrt(host[0] / host[3]) : NAN;
  return T2S2_OK;
}

int t2s2_stencil_weights(const t2s2_ctx* c, double* wx, double* wy) {
  g_last_error.clear();
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (wx) std::copy(c->wx.begin(), c->wx.end(), wx);
  if (wy) std::copy(c->wy.begin(), c->wy.end(), wy);
  return T2S2_OK;
}

double t2s2_omega(const t2s2_ctx* c) { return c ? c->omega : 0.0; }

size_t t2s2_adjoint_state_bytes(const t2s2_ctx* c) {
  if (!c) return 0;
  return static_cast<size_t>(kQ) * c->sp.plane * adjoint_real_bytes(c->cfg.storage);
}

size_t t2s2_adjoint_scratch_bytes(const t2s2_ctx* c) {
  if (!c) return 0;
  return 2 * align256(t2s2_adjoint_state_bytes(c)) + align256(t2s2_state_bytes(c)) +
         align256(kAdjMaxBlocks * sizeof(double));
}

int t2s2_bind_adjoint(t2s2_ctx* c, void* scratch) {
  g_last_error.clear();
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (!c->bound) return fail(T2S2_ERR_NOT_BOUND, "context not bound");
  if (c->sp.has_force) return fail(T2S2_ERR_UNSUPPORTED, "the adjoint covers unforced flows");
  if (c->sp.scheme != 1) return fail(T2S2_ERR_UNSUPPORTED, "the adjoint covers T2S2-FDLBM1 / T1S2");
  if (c->cfg.storage == T2S2_BF16_SR_DEV || c->cfg.storage == T2S2_F16_SR_DEV)
    return fail(T2S2_ERR_UNSUPPORTED, "the adjoint covers the storage forms rounded to nearest");
  if (!scratch || (reinterpret_cast<uintptr_t>(scratch) & 255))
    return fail(T2S2_ERR_INVALID_ARG, "scratch must be a 256-byte aligned device pointer");
  // The adjoint kernels address a plane of its arithmetic-type buffers
  // (twice the storage's bytes for the 16-bit forms) with 32-bit byte offsets.
  if (static_cast<long long>(c->sp.plane) * static_cast<long long>(adjoint_real_bytes(c->cfg.storage)) >=
      (1LL << 32))
    return fail(T2S2_ERR_UNSUPPORTED, "one plane of the adjoint's buffers must be under 4 GiB");
  AdjParams& a = c->adj;
  a.nx = c->nx;
  a.ny = c->ny;
  a.pitch = c->pitch;
  a.plane = c->sp.plane;
  a.per_x = c->sp.per_x;
  a.per_y = c->sp.per_y;
  a.wx = c->sp.wx;
  a.wy = c->sp.wy;
  a.wx32 = c->sp.wx32;
  a.wy32 = c->sp.wy32;
  const double A = c->cfg.A, w = c->omega;
  a.A = A;
  a.cPg = c->sp.cPg;
  a.cPe = c->sp.cPe;
  a.cQg = c->sp.cQg;
  a.cQe = c->sp.cQe;
  a.cRs = c->sp.cRs;
  a.cRe = c->sp.cRe;
  // d/d omega of (2 - A w)/(2 + w), (2 - w)/(2 + w) and 2/(2 + A w); the
  // equilibrium coefficients are one minus these.
  a.dcPg = -2.0 * (1.0 + A) / ((2.0 + w) * (2.0 + w));
  a.dcQg = -4.0 / ((2.0 + w) * (2.0 + w));
  a.dcRs = -2.0 * A / ((2.0 + A * w) * (2.0 + A * w));
  // omega = dt / tau = dt c_s^2 / nu at a fixed dt: d omega / d nu = -omega / nu.
  a.dnu_per_domega = std::isinf(c->cfg.nu) ? 0.0 : -w / c->cfg.nu;
  for (int k = 0; k < 4; ++k) {
    a.uw[k][0] = c->sp.uw[k][0];
    a.uw[k][1] = c->sp.uw[k][1];
  }
  char* p = static_cast<char*>(scratch);
  const size_t ab = align256(t2s2_adjoint_state_bytes(c));
  a.S = p;
  a.mu = p + ab;
  a.next = p + 2 * ab;
  c->adj_partial = reinterpret_cast<double*>(p + 2 * ab + align256(t2s2_state_bytes(c)));
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = plan_adjoint_march(c->cfg.storage, a, cus);
  if (e != hipSuccess) return hip_fail(e, "bind_adjoint: march plan");
  c->adj_bound = true;
  return T2S2_OK;
}

static int adj_ready(t2s2_ctx* c) {
  if (!c) return fail(T2S2_ERR_INVALID_ARG, "NULL context");
  if (!c->bound || !c->adj_bound) return fail(T2S2_ERR_NOT_BOUND, "adjoint scratch not bound");
  return T2S2_OK;
}

int t2s2_adjoint_seed_velocity(t2s2_ctx* c, const void* state, const double* gu,
                               const double* gv, void* lam) {
  g_last_error.clear();
  if (int rc = adj_ready(c)) return rc;
  if (!state || !lam) return fail(T2S2_ERR_INVALID_ARG, "NULL state or adjoint");
  hipError_t e = launch_adjoint_seed(c->cfg.storage, c->adj, state, gu, gv, lam, c->stream);
  if (e != hipSuccess) return hip_fail(e, "adjoint_seed_velocity");
  return T2S2_OK;
}

int t2s2_adjoint_step(t2s2_ctx* c, const void* state_n, const void* lam_np1, void* lam_n,
                      double* dnu_accum) {
  g_last_error.clear();
  if (int rc = adj_ready(c)) return rc;
  if (!state_n || !lam_np1 || !lam_n || lam_np1 == lam_n)
    return fail(T2S2_ERR_INVALID_ARG, "need a state and two distinct adjoint buffers");
  hipError_t e = launch_adjoint_step(c->cfg.storage, c->adj, c->sp_gen, c->grid_gen, state_n, lam_np1,
                                     lam_n, c->adj_partial, dnu_accum, c->stream);
  if (e != hipSuccess) return hip_fail(e, "adjoint_step");
  return T2S2_OK;
}

int t2s2_step_save_s(t2s2_ctx* c, const void* src, void* dst, void* s_out) {
  g_last_error.clear();
  if (int rc = adj_ready(c)) return rc;
  if (!src || !dst || !s_out || src == dst || dst == s_out || src == s_out)
    return fail(T2S2_ERR_INVALID_ARG, "need three distinct buffers");
  StepParams fwd = c->sp_gen;
  fwd.src = src;
  fwd.dst = dst;
  fwd.save_s = s_out;
  hipError_t e = launch_step_save_s(c->cfg.storage, fwd, c->grid_gen, c->stream);
  if (e != hipSuccess) return hip_fail(e, "step_save_s");
  return T2S2_OK;
}

int t2s2_adjoint_step_stored(t2s2_ctx* c, const void* state_n, const void* state_np1,
                             const void* s_n, const void* lam_np1, void* lam_n,
                             double* dnu_accum) {
  g_last_error.clear();
  if (int rc = adj_ready(c)) return rc;
  if (!state_n || !state_np1 || !s_n || !lam_np1 || !lam_n || lam_np1 == lam_n)
    return fail(T2S2_ERR_INVALID_ARG, "need the stored step and two distinct adjoint buffers");
  hipError_t e = launch_adjoint_step_stored(c->cfg.storage, c->adj, state_n, state_np1, s_n,
                                            lam_np1, lam_n, c->adj_partial, dnu_accum,
                                            c->stream);
  if (e != hipSuccess) return hip_fail(e, "adjoint_step_stored");
  return T2S2_OK;
}

int t2s2_adjoint_init_macro(t2s2_ctx* c, const void* lam0, const double* rho, const double* ux,
                            const double* uy, double* grho, double* gux, double* guy) {
  g_last_error.clear();
  if (int rc = adj_ready(c)) return rc;
  if (!lam0 || !rho || !ux || !uy) return fail(T2S2_ERR_INVALID_ARG, "NULL input");
  hipError_t e = launch_adjoint_init(c->cfg.storage, c->adj, lam0, rho, ux, uy, grho, gux, guy,
                                     c->stream);
  if (e != hipSuccess) return hip_fail(e, "adjoint_init_macro");
  return T2S2_OK;
}

int t2s2_adjoint_read(t2s2_ctx* c, const void* lam, double* out) {
  g_last_error.clear();
  if (int rc = adj_ready(c)) return rc;
  if (!lam || !out) return fail(T2S2_ERR_INVALID_ARG, "NULL buffer");
  hipError_t e = launch_adjoint_convert(c->cfg.storage, c->adj, lam, out, nullptr, nullptr,
                                        c->stream);
  if (e != hipSuccess) return hip_fail(e, "adjoint_read");
  return T2S2_OK;
}

int t2s2_adjoint_load(t2s2_ctx* c, const double* in, void* lam) {
  g_last_error.clear();
  if (int rc = adj_ready(c)) return rc;
  if (!lam || !in) return fail(T2S2_ERR_INVALID_ARG, "NULL buffer");
  hipError_t e = launch_adjoint_convert(c->cfg.storage, c->adj, nullptr, nullptr, in, lam,
                                        c->stream);
  if (e != hipSuccess) return hip_fail(e, "adjoint_load");
  return T2S2_OK;
}

int t2s2_copy_probe(const void* src, void* dst, int64_t plane_elems, int elem_bytes,
                    void* stream) {
  g_last_error.clear();
  if (!src || !dst) return fail(T2S2_ERR_INVALID_ARG, "NULL buffer");
  if (plane_elems <= 0) return fail(T2S2_ERR_INVALID_ARG, "plane_elems must be > 0");
  if (elem_bytes != 8 && elem_bytes != 4 && elem_bytes != 2)
    return fail(T2S2_ERR_INVALID_ARG, "elem_bytes must be 8, 4 or 2");
  if ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) %
      static_cast<uintptr_t>(elem_bytes))
    return fail(T2S2_ERR_INVALID_ARG, "buffers must be aligned to elem_bytes");
  const uintptr_t bytes = static_cast<uintptr_t>(kQ) * static_cast<uintptr_t>(plane_elems) *
                          static_cast<uintptr_t>(elem_bytes);
  const uintptr_t a = reinterpret_cast<uintptr_t>(src), b = reinterpret_cast<uintptr_t>(dst);
  if (a < b + bytes && b < a + bytes) return fail(T2S2_ERR_INVALID_ARG, "buffers overlap");
  hipError_t e = launch_copy_probe(src, dst, static_cast<long long>(plane_elems), elem_bytes,
                                   static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_fail(e, "copy_probe");
  return T2S2_OK;
}

int t2s2_stability_map(const t2s2_stability_params* prm, const double* omega, const double* r,
                       int npoints, double* radius, void* stream) {
  g_last_error.clear();
  if (!prm) return fail(T2S2_ERR_INVALID_ARG, "NULL parameters");
  if (prm->model < T2S2_STAB_PAPER || prm->model > T2S2_STAB_FAMILY)
    return fail(T2S2_ERR_INVALID_ARG, "unknown stability model");
  if (!(prm->eta >= 0.0 && prm->eta <= 1.0)) return fail(T2S2_ERR_INVALID_ARG, "eta not in [0,1]");
  if (!(prm->A >= 0.0 && prm->A <= 1.0)) return fail(T2S2_ERR_INVALID_ARG, "A not in [0,1]");
  if (!std::isfinite(prm->b2bar) || !std::isfinite(prm->b2tilde) || !std::isfinite(prm->u[0]) ||
      !std::isfinite(prm->u[1]))
    return fail(T2S2_ERR_INVALID_ARG, "non-finite parameter");
  if (prm->model == T2S2_STAB_FAMILY && !(std::isfinite(prm->btilde[0]) &&
                                          std::isfinite(prm->btilde[1]) &&
                                          std::isfinite(prm->btilde[2])))
    return fail(T2S2_ERR_INVALID_ARG, "non-finite btilde");
  if (prm->model == T2S2_STAB_FAMILY && !(std::isfinite(prm->bbar[0]) &&
                                          std::isfinite(prm->bbar[1]) &&
                                          std::isfinite(prm->bbar[2])))
    return fail(T2S2_ERR_INVALID_ARG, "non-finite bbar");
  if (prm->nk < 2 || prm->nk > 257) return fail(T2S2_ERR_INVALID_ARG, "nk not in [2, 257]");
  if (prm->squarings < 1 || prm->squarings > 60)
    return fail(T2S2_ERR_INVALID_ARG, "squarings not in [1, 60]");
  if (npoints < 0) return fail(T2S2_ERR_INVALID_ARG, "npoints < 0");
  if (npoints == 0) return T2S2_OK;
  if (!omega || !r || !radius) return fail(T2S2_ERR_INVALID_ARG, "NULL array");
  StabArgs a{};
  a.model = prm->model;
  a.eta = prm->eta;
  a.A = prm->A;
  a.b2bar = prm->b2bar;
  a.b2tilde = prm->b2tilde;
  a.ux = prm->u[0];
  a.uy = prm->u[1];
  const double pi = 3.14159265358979323846;
  a.nky = prm->nk;
  a.dthy = pi / (prm->nk - 1);
  a.dthx = a.dthy;
  a.nkx = prm->full_kx ? 2 * prm->nk - 1 : prm->nk;
  a.thx0 = prm->full_kx ? -pi : 0.0;
  a.squarings = prm->squarings;
  for (int k = 0; k < 3; ++k) a.bt[k] = prm->model == T2S2_STAB_FAMILY ? prm->btilde[k] : 0.0;
  {
    const double* bb = prm->bbar;
    const bool zero = bb[0] == 0.0 && bb[1] == 0.0 && bb[2] == 0.0;
    a.bb[0] = zero ? 0.5 : bb[0];
    a.bb[1] = zero ? 0.0 : bb[1];
    a.bb[2] = zero ? 0.5 : bb[2];
    a.gen_bb = prm->model == T2S2_STAB_FAMILY &&
               !(a.bb[0] == 0.5 && a.bb[1] == 0.0 && a.bb[2] == 0.5);
  }
  hipError_t e = launch_stability(a, omega, r, npoints, radius, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_fail(e, "stability map");
  return T2S2_OK;
}

void t2s2_destroy(t2s2_ctx* c) { delete c; }

}  // extern "C"
