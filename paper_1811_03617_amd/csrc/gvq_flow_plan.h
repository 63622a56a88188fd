// How the kernels of gvq_flow.h cut a range of slices into tiles and deal them out.  Plain C++: nothing here needs HIP.
#pragma once
#include <cstdint>

// Tiles of `rows` slices that cover the slices of `bases` bases, none of them holding slices of two
// (offs: [bases + 1] first slice of each).
inline int64_t flow_tiles(const int64_t* offs, int64_t bases, int rows)
{
    int64_t n = 0;
    for (int64_t b = 0; b < bases; ++b) n += (offs[b + 1] - offs[b] + rows - 1) / rows;
    return n;
}

// Slices per tile: as many as there is room for (`most`), as long as that leaves nobody idle.  All work-groups that run
// at once (`slots`) start together and a tile is far more than a start, so what counts is the number of tiles the busiest
// one gets; the rows are spread evenly over that number.  `unit`: slices that occupy every wave.
// A fixed number of rows left the last of few rounds nearly empty (24 M elements in 24 bases, d = 160, k = 40, compress: 39.2
// -> 31.8 us, with runs as below; d = 400, k = 100, decompress 59 -> 44) and small ranges on a fraction of the chip (0.5 M
// elements, d = 12, k = 3, 65 tiles of 640 rows: 9.2 -> 8.0 us).
inline int flow_tile_rows(const int64_t* offs, int64_t bases, int most, int unit, int64_t slots)
{
    int64_t longest = 0;
    for (int64_t b = 0; b < bases; ++b)
        if (offs[b + 1] - offs[b] > longest) longest = offs[b + 1] - offs[b];
    if (most > longest) most = (int)(longest + 15) / 16 * 16;
    if (unit > most) unit = 16;
    const int64_t each = (flow_tiles(offs, bases, most) + slots - 1) / slots;
    int lo = 1, hi = (most + unit - 1) / unit;   // in units; `hi` does
    while (lo < hi) {
        const int mid = (lo + hi) / 2;
        if (flow_tiles(offs, bases, mid * unit < most ? mid * unit : most) <= each * slots) hi = mid; else lo = mid + 1;
    }
    return lo * unit < most ? lo * unit : most;
}

// Consecutive tiles a work-group takes before it jumps ahead by the width of the grid: the more, the fewer changes of
// basis (each reloads U with nothing in flight), up to `most`, as long as the busiest work-group gets hardly more tiles
// than it must: `each` tiles, and what a run of r makes of that.  (The number of tiles per work-group, rounded down and cut
// off at `most`, dealt 633 runs of 3 to 512 work-groups: 6 tiles for some, 3 for most.)
inline int flow_run(int64_t tiles, int64_t slots, int most)
{
    const int64_t each = (tiles + slots - 1) / slots;
    for (int r = most < each ? most : (int)each; r > 1; --r) {
        const int64_t runs = (tiles + r - 1) / r, got = (runs + slots - 1) / slots * r;
        if (8 * got <= 9 * each) return r;
    }
    return 1;
}

// What flow_divide multiplies by in place of a division by n: i / n = (2 i * flow_divisor(n)) >> 32 for i < 4096, n < 4096.
inline unsigned int flow_divisor(int n) { return (0x80000000u + (unsigned int)n - 1) / (unsigned int)n; }
