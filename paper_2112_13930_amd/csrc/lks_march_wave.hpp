// The march of one wavefront (see lks_march.hpp), shared by the
// single-channel and the batched kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "lks_node.hpp"

namespace lks {

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

// One wavefront's march: lane -> column x (already wrapped; keep: the lane's
// column is stored), rows y0 .. y1 - 1 kept, `turns` turns of the row loop
// (at least the rows kept plus 2 (NL - 1), the same in every wavefront of a
// block: there is a barrier in each).
// LANES: y0 and y1 differ between the lanes (narrow channels: groups of lanes
// take chunks of rows of their own).  Row addresses are then formed per lane;
// otherwise they are scalar.
template <typename S, typename C, int BC, int NL, bool LANES>
__device__ __forceinline__ void march(const Geom &g, const Coef<C> &k, const S *__restrict__ src,
                                      S *__restrict__ dst, int x, bool keep, int y0, int y1,
                                      int turns, uint32_t step) {
  constexpr bool SR = kUseSR<S, C>;
  const int nx = g.nx, ny = g.ny;
  const int xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
  const uint32_t o0 = (uint32_t)x * (uint32_t)sizeof(S), om = (uint32_t)xm * (uint32_t)sizeof(S),
                 op = (uint32_t)xp * (uint32_t)sizeof(S);
  const uint32_t pitch = (uint32_t)g.pitch * (uint32_t)sizeof(S); // bytes
  // a node's seed hashes its index times this factor
  const uint32_t rseed = (uint32_t)nx * kNodeSeedFactor;
  const uint32_t xseed = (uint32_t)x * kNodeSeedFactor;
  const long long P = g.plane;

  // (offsets are pinned in the block of the accesses, so that they stay
  // their 32-bit vector offsets against a scalar base)
  auto load_row = [&](int r, S(&raw)[19]) {
    // a row off the channel's end is read from the row itself (unused: the
    // wall closure replaces it)
    const bool lo = r == 0, hi = r == ny - 1;
    if constexpr (LANES) {
      const uint32_t mid = (uint32_t)r * pitch;
      const uint32_t from[3] = {hi ? mid : mid + pitch, mid, lo ? mid : mid - pitch};
      uint32_t at[3][3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        at[i][0] = from[i] + op, at[i][1] = from[i] + o0, at[i][2] = from[i] + om;
        asm("" : "+v"(at[i][0]), "+v"(at[i][1]), "+v"(at[i][2]));
      }
      const S *plane = sbase(src);
      unrolled<0, 19>([&](auto qi) {
        constexpr int q = decltype(qi)::value;
        raw[q] = *(gptr<const S>)(reinterpret_cast<const char *>(plane) +
                                  at[1 + kEy[q]][1 + kEx[q]]);
        if (q < 18) plane = sbase(plane + P);
      });
    } else {
      const S *plane = sbase(src + (long long)r * g.pitch);
      uint32_t b0 = o0, bm = om, bp = op;
      asm("" : "+v"(b0), "+v"(bm), "+v"(bp));
      unrolled<0, 19>([&](auto qi) {
        constexpr int q = decltype(qi)::value;
        const S *row =
            plane - (kEy[q] > 0 ? (lo ? 0 : g.pitch) : (kEy[q] < 0 ? (hi ? 0 : -g.pitch) : 0));
        const char *base = reinterpret_cast<const char *>(sbase(row));
        raw[q] = *(gptr<const S>)(base + (kEx[q] > 0 ? bm : (kEx[q] < 0 ? bp : b0)));
        if (q < 18) plane = sbase(plane + P);
      });
    }
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
  for (int it = 0; it < turns; ++it) {
    // the block's waves stay within a row of each other, so that the cache
    // lines that neighbouring strips share are in the L2 when the second one
    // comes
    __builtin_amdgcn_s_barrier();
    const int r = y0 - (NL - 1) + it;
    // (with LANES every turn is computed, rows off the channel to no use)
    if constexpr (!LANES)
      if (r < 0 || r > rb) continue;
    S fresh[19]; // the newest row of the level below
    {
      // (off the channel's rows the nearest one, which no level uses)
      const int rr = LANES ? max(0, min(r, ny - 1)) : min(r, ny - 1);
      C f[9], gx[5], gy[5];
#pragma unroll
      for (int q = 0; q < 9; ++q) f[q] = (C)raw[q];
#pragma unroll
      for (int q = 0; q < 5; ++q) gx[q] = (C)raw[9 + q], gy[q] = (C)raw[14 + q];
      NodeObs<C> o;
      node_finish<S, C, BC, MODE_STEP, SR>(
          g, k, src, (const C *)nullptr, x, rr, f, gx, gy, o,
          SR ? mix32((xseed + (uint32_t)r * rseed) ^ step_seed(step)) : 0u, fresh);
    }
    // (computed here: sunk past the next level's arithmetic, the inputs they
    // are formed from would stay in registers across it)
#pragma unroll
    for (int q = 0; q < 19; ++q) asm volatile("" : "+v"(fresh[q]));
    // the next row's values arrive while the further levels work
    if constexpr (LANES) {
      if (it + 1 < turns) load_row(max(0, min(r + 1, ny - 1)), raw);
    } else {
      if (r < rb) load_row(min(r + 1, ny - 1), raw);
    }
#pragma unroll
    for (int j = 1; j < NL; ++j) {
      Carry<S> &c = cy[j - 1];
      const int p = r - j; // row of this level; the level below has just given row p + 1
      S next[19];
      const bool turn = LANES ? it >= 2 * j
                              : p >= max(0, y0 - (NL - 1 - j)) &&
                                    p <= min(ny - 1, y1 - 1 + (NL - 1 - j));
      if (turn) {
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
        node_finish<S, C, BC, MODE_STEP, SR, false, true>(
            g, k, src, (const C *)nullptr, x, p, f, gx, gy, o,
            SR ? mix32((xseed + (uint32_t)p * rseed) ^ step_seed(step + (uint32_t)j)) : 0u, next,
            c.up_prev, c.up);
        if (j < NL - 1) {
#pragma unroll
          for (int q = 0; q < 19; ++q) asm volatile("" : "+v"(next[q]));
        } else if (LANES ? keep && p >= y0 && p < y1 : keep) {
          S *plane = sbase(LANES ? dst : dst + (long long)p * g.pitch);
          uint32_t b0 = LANES ? (uint32_t)p * pitch + o0 : o0;
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

} // namespace lks
