// The launch grid of `blocks` 256-thread blocks that take tiles by their linear number
// blockIdx.y kTileGridRow + blockIdx.x.  A dimension's threads must stay below 2^32 (a launch
// above that silently starts the number modulo 2^32), so the number is cut into rows; x is a
// multiple of 8 in either case, which keeps block b on XCD b % 8.  May start up to a row of blocks
// too many: each tests its number against the tile count.
// Usable from host code without HIP (for tests).
#pragma once

#include <stdint.h>

namespace elb {

constexpr int kTileGridRow = 1 << 23;  // blocks of a row: 2^31 threads

struct TileGrid {
    unsigned x, y;
};

inline TileGrid tile_grid(int64_t blocks) {
    const int64_t n = (blocks + 7) / 8 * 8;
    if (n <= kTileGridRow) return {(unsigned)n, 1u};
    return {(unsigned)kTileGridRow, (unsigned)((n + kTileGridRow - 1) / kTileGridRow)};
}

}  // namespace elb
