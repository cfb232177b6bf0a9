// Where the attention kernel's fetches start, in elements.  Plain integer functions, so that they can be checked on the host at sizes no
// test can allocate.
#pragma once

#include <stdint.h>

namespace sp {

// Keys: a tile begins at key kt0 of the sequence (its first tile up to seven in front of it), in rows of ld elements.  The tile's start is
// the same for the whole workgroup and 64 bits wide; within the tile (up to 64 rows of at most 3072 elements) 32 bits are enough.
constexpr int64_t key_tile_offset(int kt0, int ld) { return (int64_t)kt0 * ld; }
// row i of the tile; what lies outside the sequence's L keys repeats its first or last one
constexpr uint32_t key_row_offset(int kt0, int i, int L, int ld)
{
    const int key = kt0 + i < 0 ? 0 : (kt0 + i < L ? kt0 + i : L - 1);
    return (uint32_t)(key - kt0) * (uint32_t)ld;
}
// Values: dimension d of a head, in rows of all token rows of a student (63 of them pass 2^32 elements from 68.2 M token rows on).
constexpr int64_t value_row_offset(int d, int rows) { return (int64_t)d * rows; }

}  // namespace sp
