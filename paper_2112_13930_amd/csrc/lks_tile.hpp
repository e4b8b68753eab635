// Several time steps of a small channel in one launch.
//
// A step of a small channel takes as long as launching it and one trip to
// memory, whatever its arithmetic: 4 to 6 us on MI355X, of which the update
// itself is about one.  Here a block holds a region of the channel in
// registers and LDS, one node per thread, and advances it several steps.
// Each step makes one more ring of the region's nodes out of date (their
// neighbours outside the region are not there), so a block keeps the inner
// part, and neighbouring blocks' regions overlap: the redundant updates run
// on compute units that would have been idle.  Within a step a thread writes
// its populations to LDS, and after one barrier pulls its neighbours' (two
// buffers, taken in turn).  Regions as wide as the channel wrap in x, and
// the channel's walls end a region without loss.
//
// Measured on MI355X (us a step, single steps against this kernel): 8 x 64
// FP64 5.3 -> 1.24, 64 x 64 FP32 5.1 -> 1.8, 128 x 128 FP64 5.6 -> 2.4, 257 x
// 65 FP32 5.8 -> 2.9, 128 x 128 binary16 5.8 -> 2.3.  What is left is the
// arithmetic of one wavefront per SIMD (about 1 us a step) and the launch.
//
// Every step rounds its values to the storage type (with the random words
// of its own step index) and calls node_finish (node_finish_x), as the
// single-step kernels do, so the result is that of single steps bit for bit.
#pragma once

#include <hip/hip_runtime.h>

#include "lks_common.hpp"

namespace lks {

// How a small channel is cut into regions.
struct TilePlan {
  int threads = 0;     // threads of a block, one per node of a region; 0: not for this channel
  int steps = 1;       // most steps a launch takes
  int rw = 0, rh = 0;  // region
  int ow = 0, oh = 0;  // the part of it a block keeps
  int ox = 0, oy = 0;  // offset of that part in the region
  int tiles_x = 0, tiles_y = 0;
};

// units: compute units of the device.
TilePlan plan_tiles(const Channel &c, int units);

struct TileArgs {
  Geom geom;
  const Coef<double> *kd;
  const Coef<float> *kf;
  const void *ref; // row references (binary16)
  int precision, scheme;
  const void *src;
  void *dst;
  uint32_t *ctr;
  int parity;
  int steps; // 1..plan.steps
  hipStream_t stream;
};

hipError_t launch_tiles(const TilePlan &plan, const TileArgs &a);

} // namespace lks
