// sk_grid.h -- one-dimensional grids of any number of 256-thread workgroups.
#pragma once

#include <stdint.h>

namespace sk {

// HIP refuses a grid of 2^32 threads or more; a launch takes half of that.
constexpr int64_t kGridBlocks = 1ll << 23;

// part(first workgroup, workgroups) for launches that cover [0, blocks) in order.
template <class F>
void grid_parts(int64_t blocks, F part) {
  for (int64_t b = 0; b < blocks; b += kGridBlocks)
    part((uint32_t)b, (uint32_t)(blocks - b < kGridBlocks ? blocks - b : kGridBlocks));
}

}  // namespace sk
