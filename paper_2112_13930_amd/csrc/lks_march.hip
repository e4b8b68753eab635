// Multi-step march kernel (lks_march.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "lks_march.hpp"

namespace lks {

namespace {

// Planes by their motion along y: along the row, up (from row y - 1) and
// down (from row y + 1).
constexpr int kAlong[9] = {0, 1, 3, 9, 10, 12, 14, 15, 17};
constexpr int kUp[5] = {2, 5, 6, 11, 16};
constexpr int kDown[5] = {4, 7, 8, 13, 18};
// x component of each plane's velocity
constexpr int kEx[19] = {0, 1, 0, -1, 0, 1, -1, -1, 1, 0, 1, 0, -1, 0, 0, 1, 0, -1, 0};
constexpr int kEy[19] = {0, 0, 1, 0, -1, 1, 1, -1, -1, 0, 0, 1, 0, -1, 0, 0, 1, 0, -1};

// The value of the lane to the left (EX = 1) or right (EX = -1): a plane
// moving along x is pulled from the column it comes from.  The lanes at
// the wavefront's ends get zeros of no use; they belong to the columns a
// level loses.
template <int EX> __device__ __forceinline__ uint32_t lane_pull(uint32_t v) {
  if constexpr (EX == 1) return __builtin_amdgcn_mov_dpp(v, 0x138, 0xf, 0xf, true); // wave_shr:1
  else if constexpr (EX == -1) return __builtin_amdgcn_mov_dpp(v, 0x130, 0xf, 0xf, true); // wave_shl:1
  else return v;
}
template <int EX> __device__ __forceinline__ float lane_pull(float v) {
  return __builtin_bit_cast(float, lane_pull<EX>(__builtin_bit_cast(uint32_t, v)));
}
template <int EX> __device__ __forceinline__ double lane_pull(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint64_t lo = lane_pull<EX>((uint32_t)b), hi = lane_pull<EX>((uint32_t)(b >> 32));
  return __builtin_bit_cast(double, (hi << 32) | lo);
}

// What level j + 1 needs of level j's rows, beyond the newest one: the
// planes along the row and up of the last row p, and the planes moving up of
// row p - 1 (where p = 0 there is no such row: the planes moving down of row
// 0, which the link closure of the lower wall takes).
template <typename S> struct Carry {
  S along[9], up[5], up_prev[5];
};

constexpr int kMarchWaves = 4; // wavefronts of a block

template <int I, int N, typename F> __device__ __forceinline__ void unrolled(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unrolled<I + 1, N>(f);
  }
}

template <typename S, typename C, int BC, int NL>
__global__ __launch_bounds__(64 * kMarchWaves, 2) void k_march(
    Geom g, Coef<C> k, const S *__restrict__ src, S *__restrict__ dst, int width, int nstrips,
    int chunk, int side, int xcds, uint32_t *__restrict__ ctr, int parity) {
  constexpr bool SR = kUseSR<S, C>;
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
  const int lane = (int)threadIdx.x & 63;
  const int col = lane - (NL - 1);
  const int x0 = si * width;
  int x = (x0 + col) % nx;
  if (x < 0) x += nx;
  const bool store = col >= 0 && col < width && x0 + col < nx;
  const int xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
  const uint32_t o0 = (uint32_t)x * (uint32_t)sizeof(S), om = (uint32_t)xm * (uint32_t)sizeof(S),
                 op = (uint32_t)xp * (uint32_t)sizeof(S);
  const uint32_t xseed = (uint32_t)x * kNodeSeedFactor; // a node's seed hashes its index times this
  const long long P = g.plane;

  auto load_row = [&](int r, S(&raw)[19]) {
    const bool lo = r == 0, hi = r == ny - 1;
    const S *plane = sbase(src + (long long)r * g.pitch);
    // (pinned here, in the block of the loads, so that they stay the loads'
    // 32-bit vector offsets)
    uint32_t b0 = o0, bm = om, bp = op;
    asm("" : "+v"(b0), "+v"(bm), "+v"(bp));
    unrolled<0, 19>([&](auto qi) {
      constexpr int q = decltype(qi)::value;
      // a row off the channel's end is read from the row itself (unused: the
      // wall closure replaces it)
      const S *row = plane - (kEy[q] > 0 ? (lo ? 0 : g.pitch) : (kEy[q] < 0 ? (hi ? 0 : -g.pitch) : 0));
      const char *base = reinterpret_cast<const char *>(sbase(row));
      raw[q] = *(gptr<const S>)(base + (kEx[q] > 0 ? bm : (kEx[q] < 0 ? bp : b0)));
      if (q < 18) plane = sbase(plane + P);
    });
  };

  Carry<S> cy[NL - 1];
#pragma unroll
  for (int j = 0; j < NL - 1; ++j) {
#pragma unroll
    for (int i = 0; i < 9; ++i) cy[j].along[i] = S(0);
#pragma unroll
    for (int i = 0; i < 5; ++i) cy[j].up[i] = cy[j].up_prev[i] = S(0);
  }

  // level j (1-based) updates the rows y0 - (NL - j) .. y1 - 1 + (NL - j)
  // of the channel, one row behind level j - 1
  const int rb = y1 > y0 ? y1 - 1 + (NL - 1) : -1;
  S raw[19];
  load_row(max(0, min(ny - 1, y0 - (NL - 1))), raw);
  for (int it = 0; it < chunk + 2 * (NL - 1); ++it) {
    // the block's waves stay within a few rows of each other, so that the
    // cache lines that neighbouring strips share are in the L2 when the
    // second one comes
    __builtin_amdgcn_s_barrier();
    const int r = y0 - (NL - 1) + it;
    if (r < 0 || r > rb) continue;
    S fresh[19]; // the newest row of the level below
    {
      // (past the channel's last row the last row again, which no level uses)
      const int rr = min(r, ny - 1);
      C f[9], gx[5], gy[5];
#pragma unroll
      for (int q = 0; q < 9; ++q) f[q] = (C)raw[q];
#pragma unroll
      for (int q = 0; q < 5; ++q) gx[q] = (C)raw[9 + q], gy[q] = (C)raw[14 + q];
      NodeObs<C> o;
      const uint32_t rseed = (uint32_t)rr * (uint32_t)nx * kNodeSeedFactor;
      node_finish<S, C, BC, MODE_STEP, SR>(
          g, k, src, (const C *)nullptr, x, rr, f, gx, gy, o,
          SR ? mix32((xseed + rseed) ^ step_seed(step)) : 0u, fresh);
    }
    // (computed here: sunk past the next level's arithmetic, the inputs they
    // are formed from would stay in registers across it)
#pragma unroll
    for (int q = 0; q < 19; ++q) asm volatile("" : "+v"(fresh[q]));
    // the next row's values arrive while the further levels work
    if (r < rb) load_row(min(r + 1, ny - 1), raw);
#pragma unroll
    for (int j = 1; j < NL; ++j) {
      Carry<S> &c = cy[j - 1];
      const int p = r - j; // row of this level; the level below has just given row p + 1
      S next[19];
      if (p >= max(0, y0 - (NL - 1 - j)) && p <= min(ny - 1, y1 - 1 + (NL - 1 - j))) {
        C f[9], gx[5], gy[5];
        S v[19];
        unrolled<0, 9>([&](auto i) {
          constexpr int q = kAlong[decltype(i)::value];
          v[q] = lane_pull<kEx[q]>(c.along[decltype(i)::value]);
        });
        unrolled<0, 5>([&](auto i) {
          constexpr int q = kUp[decltype(i)::value];
          v[q] = lane_pull<kEx[q]>(c.up_prev[decltype(i)::value]);
        });
        unrolled<0, 5>([&](auto i) {
          constexpr int q = kDown[decltype(i)::value];
          v[q] = lane_pull<kEx[q]>(fresh[q]);
        });
#pragma unroll
        for (int q = 0; q < 9; ++q) f[q] = (C)v[q];
#pragma unroll
        for (int q = 0; q < 5; ++q) gx[q] = (C)v[9 + q], gy[q] = (C)v[14 + q];
        NodeObs<C> o;
        const uint32_t rseed = (uint32_t)p * (uint32_t)nx * kNodeSeedFactor;
        node_finish<S, C, BC, MODE_STEP, SR, false, true>(
            g, k, src, (const C *)nullptr, x, p, f, gx, gy, o,
            SR ? mix32((xseed + rseed) ^ step_seed(step + (uint32_t)j)) : 0u, next, c.up_prev,
            c.up);
        if (j < NL - 1) {
#pragma unroll
          for (int q = 0; q < 19; ++q) asm volatile("" : "+v"(next[q]));
        } else if (store) {
          S *plane = sbase(dst + (long long)p * g.pitch);
          uint32_t b0 = o0;
          asm("" : "+v"(b0));
          unrolled<0, 19>([&](auto qi) {
            constexpr int q = decltype(qi)::value;
            *(gptr<S>)(reinterpret_cast<char *>(plane) + b0) = next[q];
            if (q < 18) plane = sbase(plane + P);
          });
        }
      } else {
#pragma unroll
        for (int q = 0; q < 19; ++q) next[q] = S(0);
      }
      // the level below moves on by one row
      if (p + 1 == 0) {
        asm volatile("");
#pragma unroll
        for (int i = 0; i < 5; ++i) c.up_prev[i] = fresh[kDown[i]];
      } else {
#pragma unroll
        for (int i = 0; i < 5; ++i) c.up_prev[i] = c.up[i];
      }
#pragma unroll
      for (int i = 0; i < 5; ++i) c.up[i] = fresh[kUp[i]];
#pragma unroll
      for (int i = 0; i < 9; ++i) c.along[i] = fresh[kAlong[i]];
      if (j < NL - 1) {
#pragma unroll
        for (int q = 0; q < 19; ++q) fresh[q] = next[q];
      }
    }
  }
}

// How a launch cuts the rows: groups of chunks, rows per chunk, and whether
// a group's blocks stay on one XCD.
struct RowCut {
  int rows, groups;
  bool by_xcd;
};

// A chunk of n rows takes n + 2 (NL - 1) turns of the row loop (the rows its
// neighbours compute too) and about two more to fill its pipeline.  The
// blocks run in rounds of as many as the device holds at once; the last,
// partly empty round costs about a third of one on average over the sizes
// measured, and less than one round takes as long as one.  The cut with the
// shortest sum is taken.  From 16 groups on they come in eights, one per XCD:
// the lines that neighbouring strips share are then in one L2 (4096^2, two
// steps a launch: FP32 329 against 336 us a step, FP64 556 against 566).
constexpr int kMostRounds = 12, kLeastRows = 3;
RowCut cut_rows(int ny, int chunks_per_group, int blocks_x, int slots, int lead) {
  RowCut best{(ny + chunks_per_group - 1) / chunks_per_group, 1, false};
  double best_cost = 1e300;
  for (int groups = 1; groups <= ny; groups += groups < 16 ? 1 : 8) {
    const int rows = (ny + groups * chunks_per_group - 1) / (groups * chunks_per_group);
    const double rounds = (double)groups * blocks_x / slots;
    if (groups > 1 && (rows < kLeastRows || rounds > kMostRounds)) break;
    const double cost = std::max(1.0, rounds + 0.35) * (rows + lead);
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
hipError_t launch(const MarchArgs &a) {
  const int nx = a.geom.nx, ny = a.geom.ny;
  const int nstrips = strips_of(nx, NL);
  const int width = (nx + nstrips - 1) / nstrips;
  const int side = nstrips >= 3 ? 4 : nstrips;
  const int bx = (nstrips + side - 1) / side;
  // blocks of 4 wavefronts a device of 256 CUs holds: 2 or 3 wavefronts per
  // SIMD, by the registers of the variant
  static const int per_cu = [] {
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &n, k_march<S, double, BC, NL>, 64 * kMarchWaves, 0);
    return e == hipSuccess && n > 0 ? n : 2;
  }();
  const RowCut cut = cut_rows(ny, kMarchWaves / side, bx, 256 * per_cu, 2 * (NL - 1) + 2);
  const dim3 grid = cut.by_xcd ? dim3(8u * (unsigned)bx, (unsigned)((cut.groups + 7) / 8))
                               : dim3((unsigned)bx, (unsigned)cut.groups);
  hipLaunchKernelGGL((k_march<S, double, BC, NL>), grid, dim3(64 * kMarchWaves), 0, a.stream,
                     a.geom, *a.kd, static_cast<const S *>(a.src), static_cast<S *>(a.dst), width,
                     nstrips, cut.rows, side, cut.by_xcd ? 3 : 0, a.ctr, a.parity);
  return hipGetLastError();
}

template <typename S, int NL>
hipError_t launch_bgk_trt(const MarchArgs &a) {
  switch (a.scheme) {
  case BC_LINK: return launch<S, BC_LINK, NL>(a);
  case BC_MOMENT: return launch<S, BC_MOMENT, NL>(a);
  case BC_LINK | COLL_TRT: return launch<S, BC_LINK | COLL_TRT, NL>(a);
  case BC_MOMENT | COLL_TRT: return launch<S, BC_MOMENT | COLL_TRT, NL>(a);
  default: return hipErrorInvalidValue;
  }
}

template <typename S, int NL>
hipError_t launch_scheme(const MarchArgs &a) {
  switch (a.scheme) {
  case BC_LINK | COLL_MRT: return launch<S, BC_LINK | COLL_MRT, NL>(a);
  case BC_MOMENT | COLL_MRT: return launch<S, BC_MOMENT | COLL_MRT, NL>(a);
  default: return launch_bgk_trt<S, NL>(a);
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
// twice; the sizes where the march starts to win (us a step, single steps
// against the march): FP64 384 x 384 12.4, 7.1; FP32 512 x 512 9.8, 11.3 (its
// rows are aligned to cache lines, which helps single steps), 200 x 1500
// 13.7, 11.5, 1023 x 513 21.1, 16.8.  FP32 takes 2 steps a launch there, as
// chunks are short: 1023 x 513 16.8 (3 steps: 17.7), 1024 x 1024 29.6 (29.4).
// And a strip of few columns leaves the other lanes idle, which FP32 can
// afford less.
int march_most(const Channel &c) {
  const bool f64 = c.p.precision == LKS_FP64;
  if (!f64 && c.p.precision != LKS_FP32) return 1;
  const int sch = scheme_of(c.p);
  if (sch & ~(3 | COLL_TRT | COLL_MRT)) return 1; // x walls, cut walls, solid bodies
  const long long nodes = (long long)c.p.nx * c.p.ny;
  if (nodes < (f64 ? 100000 : 400000)) return 1;
  const int most = f64 ? (mrt_of(sch) ? 3 : 4) : (nodes < 1000000 ? 2 : 3);
  const long long lanes = 64LL * strips_of(c.p.nx, most);
  return 10LL * c.p.nx < (f64 ? 4 : 7) * lanes ? 1 : most;
}

hipError_t launch_march(const MarchArgs &a) {
  if (a.precision == LKS_FP64) {
    switch (a.steps) {
    case 2: return launch_scheme<double, 2>(a);
    case 3: return launch_scheme<double, 3>(a);
    case 4: return launch_bgk_trt<double, 4>(a);
    default: return hipErrorInvalidValue;
    }
  }
  switch (a.steps) {
  case 2: return launch_scheme<float, 2>(a);
  case 3: return launch_scheme<float, 3>(a);
  default: return hipErrorInvalidValue;
  }
}

} // namespace lks
