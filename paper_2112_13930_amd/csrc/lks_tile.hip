// Multi-step kernel of small channels (lks_tile.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "lks_tile.hpp"

namespace lks {

namespace {

// Velocity of each stored plane.
constexpr int kEx[19] = {0, 1, 0, -1, 0, 1, -1, -1, 1, 0, 1, 0, -1, 0, 0, 1, 0, -1, 0};
constexpr int kEy[19] = {0, 0, 1, 0, -1, 1, 1, -1, -1, 0, 0, 1, 0, -1, 0, 0, 1, 0, -1};
// The planes that move (the three rest populations stay in registers).
constexpr int kMoving[16] = {1, 2, 3, 4, 5, 6, 7, 8, 10, 11, 12, 13, 15, 16, 17, 18};

template <typename S, typename C, int BC, int T>
__global__ __launch_bounds__(T) void k_tile(Geom g, Coef<C> k, const S *__restrict__ src,
                                            S *__restrict__ dst, const C *__restrict__ ref,
                                            TilePlan pl, int steps, uint32_t *__restrict__ ctr,
                                            int parity) {
  constexpr bool SR = kUseSR<S, C>;
  constexpr bool XA = kXA<S, C>;
  __shared__ S lds[2][16][T];
  const uint32_t step0 = ctr[parity];
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
    ctr[parity ^ 1] = step0 + (uint32_t)steps;
  const int nx = g.nx, ny = g.ny;
  const int t = (int)threadIdx.x;
  const int ly = t / pl.rw, lx = t - ly * pl.rw;
  const int cx = (int)blockIdx.x * pl.ow + lx - pl.ox; // column, before the wrap
  int x = cx % nx;
  if (x < 0) x += nx;
  const int y = (int)blockIdx.y * pl.oh + ly - pl.oy;
  const bool in = ly < pl.rh && y >= 0 && y < ny;
  const long long P = g.plane;
  const long long o = in ? (long long)y * g.pitch + x : 0;
  // LDS index of the node each moving plane is pulled from; past the region's
  // edge the node's own (out of date from the first step on, and not kept)
  const bool wide = pl.rw == nx;
  const int xl = lx > 0 ? t - 1 : (wide ? t + nx - 1 : t);
  const int xr = lx < pl.rw - 1 ? t + 1 : (wide ? t - nx + 1 : t);
  const int below = in && ly > 0 ? -pl.rw : 0, above = in && ly < pl.rh - 1 ? pl.rw : 0;

  S cur[19];
#pragma unroll
  for (int q = 0; q < 19; ++q) cur[q] = in ? src[q * P + o] : S(0);
  // binary16: references of the rows a population comes from
  const int yy = in ? y : 0;
  const C *Dy = ref + (long long)yy * kRefRow;
  const C *Dm = yy == 0 ? Dy : Dy - kRefRow, *Dp = yy == ny - 1 ? Dy : Dy + kRefRow;
  const uint32_t index = (uint32_t)(yy * nx + x);

  for (int i = 0; i < steps; ++i) {
    S(*buf)[T] = lds[i & 1];
#pragma unroll
    for (int m = 0; m < 16; ++m) buf[m][t] = cur[kMoving[m]];
    __syncthreads();
    if (in) {
      S pulled[19];
      pulled[0] = cur[0], pulled[9] = cur[9], pulled[14] = cur[14];
#pragma unroll
      for (int m = 0; m < 16; ++m) {
        const int q = kMoving[m];
        const int at = (kEx[q] > 0 ? xl : (kEx[q] < 0 ? xr : t)) +
                       (kEy[q] > 0 ? below : (kEy[q] < 0 ? above : 0));
        pulled[q] = buf[m][at];
      }
      const S own_lo[5] = {cur[4], cur[7], cur[8], cur[13], cur[18]};
      const S own_hi[5] = {cur[2], cur[5], cur[6], cur[11], cur[16]};
      NodeObs<C> obs;
      const uint32_t nseed = SR ? node_seed(step_seed(step0 + (uint32_t)i), index) : 0u;
      if constexpr (XA) {
        const XTabs tab = xtabs_of(const_cast<C *>(ref), ny);
        const long long row = (long long)yy * kRefRow;
        F16Words ew(nseed);
        S next[19];
        node_finish_x<S, BC, MODE_STEP, true>(g, k, cur, tab, tab.V + row, tab.K + row, x, yy,
                                              pulled, obs,
                                              [&](int q, float zq) { next[q] = sr_f16(zq, ew.word(q)); },
                                              own_lo, own_hi);
#pragma unroll
        for (int q = 0; q < 19; ++q) cur[q] = next[q];
      } else {
        C f[9], gx[5], gy[5];
#pragma unroll
        for (int q = 0; q < 9; ++q)
          f[q] = dec<S>((C)pulled[q], kEy[q] > 0 ? Dm : (kEy[q] < 0 ? Dp : Dy), q);
#pragma unroll
        for (int q = 0; q < 5; ++q) {
          gx[q] = dec<S>((C)pulled[9 + q], kEy[9 + q] > 0 ? Dm : (kEy[9 + q] < 0 ? Dp : Dy), 9 + q);
          gy[q] = dec<S>((C)pulled[14 + q], kEy[14 + q] > 0 ? Dm : (kEy[14 + q] < 0 ? Dp : Dy), 14 + q);
        }
        S next[19];
        node_finish<S, C, BC, MODE_STEP, SR, false, true>(g, k, cur, ref, x, yy, f, gx, gy, obs,
                                                          nseed, next, own_lo, own_hi);
#pragma unroll
        for (int q = 0; q < 19; ++q) cur[q] = next[q];
      }
    }
  }
  const bool keep = in && lx >= pl.ox && lx < pl.ox + pl.ow && cx < nx && ly >= pl.oy &&
                    ly < pl.oy + pl.oh;
  if (keep) {
#pragma unroll
    for (int q = 0; q < 19; ++q) dst[q * P + o] = cur[q];
  }
}

template <typename S, typename C, int BC>
hipError_t launch(const TilePlan &pl, const TileArgs &a) {
  const Coef<C> *k;
  if constexpr (sizeof(C) == 8) k = a.kd;
  else k = a.kf;
  const dim3 grid((unsigned)pl.tiles_x, (unsigned)pl.tiles_y);
  if (pl.threads == 256)
    hipLaunchKernelGGL((k_tile<S, C, BC, 256>), grid, dim3(256), 0, a.stream, a.geom, *k,
                       static_cast<const S *>(a.src), static_cast<S *>(a.dst),
                       static_cast<const C *>(a.ref), pl, a.steps, a.ctr, a.parity);
  else
    hipLaunchKernelGGL((k_tile<S, C, BC, 512>), grid, dim3(512), 0, a.stream, a.geom, *k,
                       static_cast<const S *>(a.src), static_cast<S *>(a.dst),
                       static_cast<const C *>(a.ref), pl, a.steps, a.ctr, a.parity);
  return hipGetLastError();
}

} // namespace

// The plan with the shortest time a step, by a model fitted to all of T = 256
// and 512, w = 16, 32 and 64 and k = 2 to 8 on channels of 8 x 64 to 64 x 2048
// nodes: a launch and its trips to memory take 3.5 us plus 1.5 us for every
// block a compute unit gets, a step of one block 1.2 us (256 threads, one
// wavefront per SIMD) or 2.15 us (512), of a further one on the same compute
// unit 1.0 or 2.0 us.  Single steps take 5.2 us or more, so that is where the
// line lies: from about 50k nodes on the overlap costs more than launches do
// (FP64 256 x 256: 5.5 us a step in regions, 6.1 to 6.4 in single steps; 512 x
// 512: 13.0 to 19.9 against 8.7 to 11.7).
constexpr double kSingleStepUs = 5.2;

// Whether plans of two steps per launch pay, which the model puts at 4.65 us.
// It is that of FP64 steps; the others compute more per step: regions take 5.9
// to 6.6 us a step with FP32 storage, 5.9 to 6.3 with binary16 (6.5 to 7.0 with
// moment walls and TRT or MRT) and, computed in FP64, 6.4 to 6.7 (BGK 6.8 to
// 7.6).  Single steps are at their best where rows are whole wavefronts and
// cache lines: 256 x 256 5.8, 5.4 to 5.9 and 5.4 us, against 6.6, 6.6 and 7.0 for
// 100 x 655; FP32 loses that from 70k nodes on (128 x 625 6.4 against 5.9).
// Regions as wide as the channel overlap in one direction only and always pay
// (64 x 1024 FP32 4.6 against 5.6).
bool two_steps_pay(const Channel &c, int region_width) {
  if (c.p.precision == LKS_FP64 || region_width == c.p.nx) return true;
  const bool full = c.p.nx % 128 == 0, bgk = !(scheme_of(c.p) & (COLL_TRT | COLL_MRT));
  if (c.p.precision == LKS_FP32) return !full || (long long)c.p.nx * c.p.ny >= 70000;
  if (c.p.precision == LKS_FP16_STORE) return !full && (bgk || c.p.bc == LKS_BC_LINK);
  return !full && !bgk;
}

TilePlan plan_tiles(const Channel &c, int units) {
  TilePlan best;
  if (scheme_of(c.p) & ~(3 | COLL_TRT | COLL_MRT | WALLS_X)) return best; // cut walls, solid bodies
  const int nx = c.p.nx, ny = c.p.ny;
  if ((long long)nx * ny > 300000) return best;
  double best_us = kSingleStepUs;
  for (int T : {256, 512}) {
    for (int w : {nx, 16, 32, 64}) {
      if (w > T || w > nx) continue;
      const int h = std::min(ny, T / w);
      for (int k = two_steps_pay(c, w) ? 2 : 3; k <= 32; ++k) {
        TilePlan p;
        p.threads = T, p.steps = k, p.rw = w, p.rh = h;
        p.ox = w == nx ? 0 : k, p.ow = w - 2 * p.ox;
        p.oy = h == ny ? 0 : k, p.oh = h - 2 * p.oy;
        if (p.ow < 1 || p.oh < 1) break;
        p.tiles_x = (nx + p.ow - 1) / p.ow, p.tiles_y = (ny + p.oh - 1) / p.oh;
        const double more = (p.tiles_x * p.tiles_y + units - 1) / units - 1;
        const double us = (5.0 + 1.5 * more) / k + (T == 256 ? 1.2 + more : 2.15 + 2.0 * more);
        if (us < best_us) best_us = us, best = p;
      }
    }
  }
  return best;
}

hipError_t launch_tiles(const TilePlan &pl, const TileArgs &a) {
  return dispatch_precision(a.precision, [&](auto t) -> hipError_t {
    using S = typename decltype(t)::S;
    using C = typename decltype(t)::C;
    switch (a.scheme) {
    case BC_LINK: return launch<S, C, BC_LINK>(pl, a);
    case BC_MOMENT: return launch<S, C, BC_MOMENT>(pl, a);
    case BC_LINK | COLL_TRT: return launch<S, C, BC_LINK | COLL_TRT>(pl, a);
    case BC_MOMENT | COLL_TRT: return launch<S, C, BC_MOMENT | COLL_TRT>(pl, a);
    case BC_LINK | COLL_MRT: return launch<S, C, BC_LINK | COLL_MRT>(pl, a);
    case BC_MOMENT | COLL_MRT: return launch<S, C, BC_MOMENT | COLL_MRT>(pl, a);
    case BC_LINK | WALLS_X: return launch<S, C, BC_LINK | WALLS_X>(pl, a);
    case BC_LINK | COLL_TRT | WALLS_X: return launch<S, C, BC_LINK | COLL_TRT | WALLS_X>(pl, a);
    case BC_LINK | COLL_MRT | WALLS_X: return launch<S, C, BC_LINK | COLL_MRT | WALLS_X>(pl, a);
    default: return hipErrorInvalidValue;
    }
  });
}

} // namespace lks
