// Grid sizes, host arithmetic only.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace ep {

// HIP supports fewer than 2^32 threads along a dimension of a grid. A launch
// over the elements or rows of a matrix that device memory can hold may want
// more (3 million rows of 1000 labels: 4.6e9 dwords of split planes), so its
// kernel walks its blocks in steps of the grid, which is capped here; below
// the cap each block takes one step.
constexpr int64_t kMaxLaunchThreads = (int64_t(1) << 32) - 1;

inline unsigned stride_grid(int64_t blocks, int threads) {
    return (unsigned)std::min<int64_t>(std::max<int64_t>(blocks, 0), kMaxLaunchThreads / threads);
}

}  // namespace ep
