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
// first: 32 hoisted rotations' KeyMult at N = 2^16, 24 limbs 464 -> 403 us with
// the 16-byte gathers, and 380 us with the key rows loaded past the L2
// (load_once).
// The order takes all three grid dimensions: the work-items along one of them
// have to stay below 2^32, which rows, tiles and the 65535 rotations of a call
// in one dimension would pass.
struct XcdGrid {
    uint32_t x, y, z;
};
struct XcdRows {
    int row, rot, tile;  // row < 0: nothing to do
    static XcdGrid grid(uint32_t rows, uint32_t tiles, uint32_t n_rot) { return XcdGrid{8 * tiles, n_rot, (rows + 7) / 8}; }
    CKKS_HD XcdRows(XcdGrid block, uint32_t rows, uint32_t /* tiles */, uint32_t /* n_rot */)
    {
        const uint32_t r = block.z * 8 + (block.x & 7u);
        row = r < rows ? (int)r : -1;
        rot = (int)block.y;
        tile = (int)(block.x >> 3);
    }
};

}  // namespace ckks
