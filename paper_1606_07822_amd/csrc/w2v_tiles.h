// Index arithmetic of the kernels' tiles that does not depend on the device, so that it can be checked on the host.
#pragma once

#include <stdint.h>

namespace w2v {

// Distance of the 64 probes of a search step over [lo, hi), lo < hi (any two values of that kind: the sum of their
// distance and 63 may pass 2^31).
constexpr int32_t probe_step(int32_t lo, int32_t hi) {
    return static_cast<int32_t>((static_cast<uint32_t>(hi) - static_cast<uint32_t>(lo) + 63u) / 64u);
}

// The log-likelihood's tiles: rows of up to `columns` floats take `tiles` tiles of 64 columns, of which the first
// `full` lie within every such row, and 4 `groups` window words a step; wider rows go in panels of that many tiles.
struct LoglikTiles {
    int columns, tiles, groups, full;
    bool panels;
};
constexpr LoglikTiles kLoglikTiles[] = {{64, 1, 3, 0, false},  {128, 2, 3, 1, false}, {256, 4, 2, 2, false},
                                        {320, 5, 2, 4, false}, {512, 8, 2, 5, false}, {1024, 8, 2, 0, true}};

// First of the four columns that a lane reads in tile t of the panel that starts at column c0: its own, or column 0
// where its own lie past a row of dim floats (every row has four columns from 0 on: strides are multiples of 4; the
// caller drops what it reads there). The first `full` tiles lie within the row.
constexpr int quad_column(int full, int c0, int t, int lane, int dim) {
    return t < full || c0 + t * 64 + (lane >> 2) * 4 < dim ? c0 + t * 64 + (lane >> 2) * 4 : 0;
}

}  // namespace w2v
