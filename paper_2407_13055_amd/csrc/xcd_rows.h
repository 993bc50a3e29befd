// Work-group order of KeyMult over hoisted rotations (plain C++, so that the
// host can check it).
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define CKKS_HD __host__ __device__ __forceinline__
#else
#define CKKS_HD inline
#endif

namespace ckks {

// Every rotation of a row reads the row's shared ModUp rows (256 KB each at
// N = 2^16), so a row's work-groups all run on one XCD (work-groups go to the
// 8 XCDs in turn), one rotation after the other, and its L2 serves all but the
// first.  Rows past the last multiple of 8 would leave XCDs without work: each
// of them is shared by 8, 4 or 2 XCDs (every p-th tile of all its rotations),
// so that every XCD has the same share at every number of rows.  P rows, the
// longer ones, are the first rows.
// 32 hoisted rotations at N = 2^16, by (tile, row, rotation) -> whole rows only
// -> this order: 32 rows 1048 -> 953 -> 955 us, 25 rows 822 -> 797 -> 753,
// 19 rows 539 -> 544 -> 516, 9 rows 221 -> 265 -> 220, 3 rows 101 -> 150 -> 102;
// their weighted sum 500 -> 398 -> 399, 421 -> 373 -> 364, 222 -> 252 -> 197,
// 117 -> 125 -> 117, 119 -> 130 -> 119.
// The order takes all three grid dimensions: the work-items along one of them
// have to stay below 2^32, which rows, tiles and the 65535 rotations of a call
// in one dimension would pass.
struct XcdGrid {
    uint32_t x, y, z;
};
struct XcdRows {
    int row, rot, tile;  // row < 0: nothing to do

    // Along x a step's 8 XCDs times the tiles of a row; steps along y, and z
    // past 65535 of them.
    static XcdGrid grid(uint32_t rows, uint32_t tiles, uint32_t n_rot)
    {
        const uint32_t rest = rows % 8, p = parts(rest), len = (n_rot * tiles + p - 1) / p;
        const uint32_t steps = rows / 8 * n_rot + (rest * p / 8 * len + tiles - 1) / tiles;
        const uint32_t z = (steps + 65534) / 65535;
        return XcdGrid{8 * tiles, (steps + z - 1) / z, z};
    }
    CKKS_HD XcdRows(XcdGrid block, uint32_t grid_y, uint32_t rows, uint32_t tiles, uint32_t n_rot)
    {
        const uint32_t step = block.y + grid_y * block.z, xcd = block.x & 7u, slot = block.x >> 3;
        const uint32_t full = rows / 8 * n_rot;  // steps of the rows that fill all XCDs
        if (step < full) {
            const uint32_t g = step / n_rot;
            row = (int)(8 * g + xcd), rot = (int)(step - g * n_rot), tile = (int)slot;
            return;
        }
        const uint32_t rest = rows % 8, p = parts(rest), items = n_rot * tiles, len = (items + p - 1) / p;
        const uint32_t i = slot + tiles * (step - full), m = i / len, u = 8 * m + xcd;
        const uint32_t item = (i - m * len) * p + u % p;  // rotation by rotation, every p-th tile
        row = u < rest * p && item < items ? (int)(rows - rest + u / p) : -1;
        rot = (int)(item / tiles), tile = (int)(item % tiles);
    }

private:
    CKKS_HD static uint32_t parts(uint32_t rest) { return rest & 1 ? 8 : rest & 2 ? 4 : 2; }
};

}  // namespace ckks
