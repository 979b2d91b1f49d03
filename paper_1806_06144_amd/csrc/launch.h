// Grid sizes and split counts, host arithmetic only.
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

// Visits (splits, items per split) for every way to cut `items` into at most
// `most` contiguous ranges of equal length of which none is empty, fewest
// splits first. There are at most 2 sqrt(items) of them; trying every count
// instead took the host 79 us for 10000 centre panels, per chunk of a call.
template <class Visit>
inline void each_split(int64_t items, int64_t most, Visit visit) {
    for (int64_t splits = 1; splits <= items && splits <= most;) {
        const int64_t per = (items + splits - 1) / splits;
        visit(splits, per);
        if (per == 1) return;
        splits = (items + per - 2) / (per - 1);      // the fewest of length per - 1
    }
}

}  // namespace ep
