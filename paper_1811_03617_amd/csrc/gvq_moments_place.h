// How the int8 moments kernel cuts slices into panels, and where a thread of it finds and leaves its numbers.  Plain C++: nothing
// here needs HIP.
#pragma once

#define INT_NS 64                    // samples per block

// Panels of a slice of d elements, and tiles of 16 elements per panel.
constexpr int int_panels(int d) { const int t = (d + 15) / 16; return t <= 8 ? 1 : (t + 5) / 6; }
constexpr int int_tiles(int d) { const int np = int_panels(d); return ((d + 15) / 16 + np - 1) / np; }

// A thread parks 16 samples of one column.  Its item in one word: from bit 13 on, where its first sample lies in a block's
// memory; below, in units of 16 bytes, where its first digits go in LDS, which also says its column (bits 0 to 3 and, the tile, 6 to 9)
// and its samples (bits 4 and 5).
constexpr unsigned int int_place(unsigned int from, int column, int quarter)
{
    return from << 13 | (unsigned int)((column >> 4) * 64 + quarter * 16 + (column & 15));
}
constexpr unsigned int int_place_from(unsigned int p) { return p >> 13; }
constexpr unsigned int int_place_lds(unsigned int p) { return (p & 0x3ffu) << 4; }
constexpr int int_place_column(unsigned int p) { return (int)((p >> 6 & 15u) * 16 + (p & 15u)); }
constexpr int int_place_quarter(unsigned int p) { return (int)(p >> 4 & 3u); }

// A column past the slice's end starts where the largest block (1024 elements of four bytes) is over: whatever the rows' distances
// add, it is out of every block's buffer resource and reads as zeros.
#define INT_MOST_D 1024
#define INT_NOWHERE ((unsigned int)(INT_NS * INT_MOST_D * 4))
// Element e of sample 16 * quarter of a block, in bytes from its start.
constexpr unsigned int int_from(int e, int quarter, int d, int bytes)
{
    return e < d ? (unsigned int)((16 * quarter * d + e) * bytes) : INT_NOWHERE;
}
static_assert(INT_NOWHERE < 1u << 19, "19 bits for it");
