// Buffer offsets of a 2 x 2 tile's outputs, for the fast-filtering kernels.
// Plain constexpr functions, so that host code can check them.
#pragma once

#include <stdint.h>

namespace miconv {

constexpr uint32_t kOob = 0x80000000u;  // beyond any buffer of < 2^31 bytes

// Byte offsets of the outputs (0, 0), (0, 1), (1, 0), (1, 1) of a tile whose
// first one is at byte o, rows row_bytes apart; kOob for what does not exist
// (in: the tile, two_p: its second row, two_q: its second column).  An offset
// is replaced as a whole: kOob plus a row can pass 2^32 and come back inside.
struct TileOffsets {
    uint32_t at[4];
};
constexpr TileOffsets tile_offsets(uint32_t o, uint32_t row_bytes, bool in, bool two_p, bool two_q)
{
    return TileOffsets{{in ? o : kOob, in && two_q ? o + 4u : kOob, in && two_p ? o + row_bytes : kOob,
                        in && two_p && two_q ? o + row_bytes + 4u : kOob}};
}

}  // namespace miconv
