// Multi-step march kernel (lks_march.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "lks_march.hpp"
#include "lks_march_wave.hpp"

namespace lks {

namespace {

template <typename S, typename C, int BC, int NL>
__global__ __launch_bounds__(64 * kMarchWaves, 2) void k_march(
    Geom g, Coef<C> k, const S *__restrict__ src, S *__restrict__ dst, int width, int nstrips,
    int chunk, int side, int xcds, uint32_t *__restrict__ ctr, int parity) {
  const uint32_t step = ctr[parity];
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) ctr[parity ^ 1] = step + (uint32_t)NL;
  // a block's waves: `side` strips next to each other, kMarchWaves / side
  // chunks of rows.  xcds = 3: all blocks of such a group of chunks on one
  // XCD (the hardware deals blocks round-robin to the 8 XCDs, gridDim.x is a
  // multiple of 8); xcds = 0: blocks in dispatch order.
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wc = side == 1 ? wave : (side == 2 ? wave >> 1 : 0);
  const int ws = wave & (side - 1);
  const int sw = ((int)blockIdx.x >> xcds) * side + ws;
  const int gi = ((int)blockIdx.y << xcds) + ((int)blockIdx.x & ((1 << xcds) - 1));
  const int ci = gi * (kMarchWaves / side) + wc;
  const int si = min(sw, nstrips - 1);
  const int nx = g.nx, ny = g.ny;
  const int y0 = min(ny, ci * chunk), y1 = sw < nstrips ? min(ny, y0 + chunk) : y0;
  // columns: lane NL - 1 holds the strip's first column
  const int col = ((int)threadIdx.x & 63) - (NL - 1);
  const int x0 = si * width;
  int x = (x0 + col) % nx;
  if (x < 0) x += nx;
  const bool keep = col >= 0 && col < width && x0 + col < nx;
  march<S, C, BC, NL, false>(g, k, src, dst, x, keep, y0, y1, chunk + 2 * (NL - 1), step);
}

// A chunk of n rows updates n + NL - 1 rows a level on average (some its
// neighbours update too) and fills its pipeline for about one more.  The
// blocks run in rounds of as many as the device holds at once.  What r rounds
// cost was fitted to chunks of 16 to 103 rows on 4096^2, 2048^2 and 5000 x
// 1111 and of 3 to 10 rows on 1023 x 513 to 2500 x 300 nodes: a partly empty
// round costs a fifth of a round more than its share, at most a whole one; a
// few blocks over one round cost half a round; from four rounds on the blocks
// even out (4096^2 FP64, four steps a launch: 1.97 rounds of 74 rows 299 us a
// step, 4.5 of 32 rows 299, 1.69 of 86 rows 333; 2048^2 FP32 0.66 of 37 rows
// 83, 1.03 of 24 rows 94).  The cut with the shortest product is taken.
// From 16 groups on they come in eights, one per XCD: the lines that
// neighbouring strips share are then in one L2 (4096^2, two steps a launch:
// FP32 329 against 336 us a step, FP64 556 against 566).
double rounds_cost(double r) {
  if (r > 4.0) return 0.96 * r;
  if (r > 1.0 && r < 1.2) return 1.5;
  return std::min(std::ceil(r), r + 0.2);
}

constexpr int kMostRounds = 12, kLeastRows = 3;
RowCut cut_rows(int ny, int chunks_per_group, int blocks_x, int slots, int lead) {
  RowCut best{(ny + chunks_per_group - 1) / chunks_per_group, 1, false};
  double best_cost = 1e300;
  for (int groups = 1; groups <= ny; groups += groups < 16 ? 1 : 8) {
    const int rows = (ny + groups * chunks_per_group - 1) / (groups * chunks_per_group);
    const double rounds = (double)groups * blocks_x / slots;
    if (groups > 1 && (rows < kLeastRows || rounds > kMostRounds)) break;
    const double cost = rounds_cost(rounds) * (rows + lead);
    if (cost < best_cost) {
      best_cost = cost;
      const int used = (ny + rows * chunks_per_group - 1) / (rows * chunks_per_group);
      best = RowCut{rows, used, groups >= 16};
    }
  }
  return best;
}

int strips_of(int nx, int steps) {
  const int most = 64 - 2 * (steps - 1);
  return (nx + most - 1) / most;
}

template <typename S, int BC, int NL>
hipError_t launch(MarchPlan &plan, const MarchArgs &a) {
  const int nx = a.geom.nx, ny = a.geom.ny;
  const int nstrips = strips_of(nx, NL);
  const int width = (nx + nstrips - 1) / nstrips;
  const int side = nstrips >= 3 ? 4 : nstrips;
  const int bx = (nstrips + side - 1) / side;
  // blocks of 4 wavefronts a compute unit holds: 2 or 3 wavefronts per SIMD,
  // by the registers of the variant
  static const int per_cu = [] {
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &n, k_march<S, double, BC, NL>, 64 * kMarchWaves, 0);
    return e == hipSuccess && n > 0 ? n : 2;
  }();
  RowCut &cut = plan.cut[NL - 2];
  if (cut.rows == 0) cut = cut_rows(ny, kMarchWaves / side, bx, plan.units * per_cu, NL);
  const dim3 grid = cut.by_xcd ? dim3(8u * (unsigned)bx, (unsigned)((cut.groups + 7) / 8))
                               : dim3((unsigned)bx, (unsigned)cut.groups);
  hipLaunchKernelGGL((k_march<S, double, BC, NL>), grid, dim3(64 * kMarchWaves), 0, a.stream,
                     a.geom, *a.kd, static_cast<const S *>(a.src), static_cast<S *>(a.dst), width,
                     nstrips, cut.rows, side, cut.by_xcd ? 3 : 0, a.ctr, a.parity);
  return hipGetLastError();
}

template <typename S, int NL>
hipError_t launch_bgk_trt(MarchPlan &plan, const MarchArgs &a) {
  switch (a.scheme) {
  case BC_LINK: return launch<S, BC_LINK, NL>(plan, a);
  case BC_MOMENT: return launch<S, BC_MOMENT, NL>(plan, a);
  case BC_LINK | COLL_TRT: return launch<S, BC_LINK | COLL_TRT, NL>(plan, a);
  case BC_MOMENT | COLL_TRT: return launch<S, BC_MOMENT | COLL_TRT, NL>(plan, a);
  default: return hipErrorInvalidValue;
  }
}

template <typename S, int NL>
hipError_t launch_scheme(MarchPlan &plan, const MarchArgs &a) {
  switch (a.scheme) {
  case BC_LINK | COLL_MRT: return launch<S, BC_LINK | COLL_MRT, NL>(plan, a);
  case BC_MOMENT | COLL_MRT: return launch<S, BC_MOMENT | COLL_MRT, NL>(plan, a);
  default: return launch_bgk_trt<S, NL>(plan, a);
  }
}

} // namespace

// Steps per launch.  More steps move the state less often, but each loses two
// more columns of a wavefront's 64 and two more rows of a chunk, and needs 19
// more values per lane.  Measured at 4096^2 (us a step; single steps: FP32
// 427, FP64 921): FP32, bound by its arithmetic, 2 steps 310, 3 282-289, 4
// 285; FP64, bound by memory, 2 steps 560, 3 384, 4 302.  FP64 with the MRT
// collision spills at 4: 422 against 381 at 3.
// Small channels fill too few wavefronts, and short chunks compute more rows
// twice, the more so the more steps a launch takes.  FP64 (us a step, BGK with
// moment walls: single steps; 2, 3, 4 steps a launch): 300 x 1000 25.5; 11.2,
// 10.4, 11.5; 128 x 1250 10.7; 8.1, 9.4, 10.6; 256 x 512 8.7; 7.5, 8.1, 11.6; 300
// x 333 10.4; 6.3, 9.0, 9.7.  Below 125k nodes only two steps win, and not where
// the width is a power of two: single steps then fill their blocks and lines (64
// x 1796 7.8; 8.3, 9.0, 9.7; 256 x 449 8.3; 8.8, 8.0, 9.7), save wide BGK and TRT
// channels (512 x 224 9.0; 7.3, 7.2, 7.8; with MRT 512 x 195 8.5; 9.0, 8.7).
// FP32 (single steps against the march): 512 x 512 9.8, 11.3 (its rows are
// aligned to cache lines, which helps single steps), 200 x 1500 13.7, 11.5, 1023
// x 513 21.1, 16.8; 2 steps a launch there, as chunks are short: 1023 x 513 16.8
// (3 steps: 17.7), 1024 x 1024 29.6 (29.4).  And a strip of few columns leaves
// the other lanes idle, which FP32 can afford less.
int march_most(const Channel &c) {
  const bool f64 = c.p.precision == LKS_FP64;
  if (!f64 && c.p.precision != LKS_FP32) return 1;
  const int sch = scheme_of(c.p);
  if (sch & ~(3 | COLL_TRT | COLL_MRT)) return 1; // x walls, cut walls, solid bodies
  const long long nodes = (long long)c.p.nx * c.p.ny;
  if (nodes < (f64 ? 100000 : 400000)) return 1;
  int most = f64 ? (mrt_of(sch) || nodes < 350000 ? 3 : 4) : (nodes < 1000000 ? 2 : 3);
  if (f64 && nodes < 125000) {
    const bool full = (c.p.nx & (c.p.nx - 1)) == 0;
    if (full && (c.p.nx < 512 || mrt_of(sch))) return 1;
    most = 2;
  }
  const long long lanes = 64LL * strips_of(c.p.nx, most);
  return 10LL * c.p.nx < (f64 ? 4 : 7) * lanes ? 1 : most;
}

hipError_t launch_march(MarchPlan &plan, const MarchArgs &a) {
  if (a.precision == LKS_FP64) {
    switch (a.steps) {
    case 2: return launch_scheme<double, 2>(plan, a);
    case 3: return launch_scheme<double, 3>(plan, a);
    case 4: return launch_bgk_trt<double, 4>(plan, a);
    default: return hipErrorInvalidValue;
    }
  }
  switch (a.steps) {
  case 2: return launch_scheme<float, 2>(plan, a);
  case 3: return launch_scheme<float, 3>(plan, a);
  default: return hipErrorInvalidValue;
  }
}

} // namespace lks
