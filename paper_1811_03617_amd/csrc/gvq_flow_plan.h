// How the kernels of gvq_flow.h take a shape, and how they cut a range of slices into tiles and deal them out.  Plain C++:
// nothing here needs HIP.
#pragma once
#include <cstddef>
#include <cstdint>
#include <initializer_list>
#include <type_traits>

constexpr int flow_words(int waves) { return waves == 4 ? 8 : 6; }   // most words per thread and tile
// bytes of a row of `steps` 32-number steps in LDS: fp32, or the first bf16 terms and then the second ones; an odd number of
// 16-byte words, so that the 16 rows an operand is read from start in different banks
constexpr int flow_row(int steps) { return 128 * steps + 16; }
// The rows of x in LDS, `len` numbers each: 16 lanes write 16 rows at a time, so rows of an even number of 16-byte words get
// one more (48 M elements, decompress: d = 96 65.7 -> 59.0 us, d = 160 59.6 -> 50.5, d = 160 to bf16 47.4 -> 41.2).
constexpr int flow_out_row(int len) { return len % 8 == 0 ? len + 4 : len; }

// How a kernel takes a shape (0 waves: not at all).
struct FlowPlan {
    bool exact = false;               // fp32 products, else the bf16 split
    int waves = 0, rows = 0, per_cu = 1;
    int wn = 1, ntw = 0, steps = 0;   // compress: waves over the comps, comp tiles per wave, steps of 32 elements
    int etw = 0, kst = 0;             // decompress: element tiles per wave, steps of 32 comps
    size_t words = 0;                 // 128-bit words of the packed U per basis
    size_t row_bytes = 0, fixed_bytes = 0;   // LDS per row of a tile, and besides
    size_t lds(int tile_rows) const { return tile_rows * row_bytes + fixed_bytes + 16; }
};

// Default products of a shape (gvq_long_split without options): the split from 10 flop/B up.
inline bool flow_exact(int d, int k) { return 2.0 * d * k / (4.0 * (d + k)) < 10.0; }

inline int flow_round_up(int v, std::initializer_list<int> allowed)
{
    for (int s : allowed)
        if (v <= s) return s;
    return 0;
}

// Most rows of a tile: as many whole 16-slice groups (a multiple of `unit` groups if there are that many) as the waves'
// words and a work-group's share of the 160 KB of LDS hold.
inline int flow_most_rows(int most_words, int words, const FlowPlan& q, int unit)
{
    const size_t lds = 160 * 1024 / q.per_cu;
    int g = most_words / words / 16;
    const int fit = (int)((lds - 512 - q.fixed_bytes) / (16 * q.row_bytes));
    if (g > fit) g = fit;
    if (g > 64) g = 64;
    if (g > unit) g = g / unit * unit;
    return 16 * g;
}

inline FlowPlan flow_compress_plan(int d, int k)
{
    FlowPlan best;
    if (d < 4 || k > 128) return best;
    const int NT = (k + 15) / 16, words = (d + 3) / 4, steps = flow_round_up((d + 31) / 32, {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16});
    if (!steps) return best;
    for (int W = 4; W <= 8 && !best.waves; W *= 2)
        for (int wn = 1; wn <= W; wn *= 2) {
            FlowPlan q;
            q.exact = flow_exact(d, k);
            q.wn = wn; q.ntw = (NT + wn - 1) / wn; q.steps = steps; q.waves = W;
            q.per_cu = 8 / W;   // three of four waves: d = 63 gains 2 %, d = 96 and 100 lose 20 % to the smaller tiles
            if (wn > 1 && wn / 2 >= NT) break;                        // waves with nothing to do
            if (W == 4 && (q.ntw > 4 || q.ntw * steps > 16)) continue;   // 128 registers of U per wave
            if (W == 8 && q.ntw > 1) continue;
            q.fixed_bytes = 16 * (size_t)words;
            q.row_bytes = flow_row(steps) + 4 * (size_t)k;
            q.rows = flow_most_rows(64 * W * flow_words(W), words, q, W / wn);
            if (q.rows < 16) continue;
            q.words = (size_t)wn * q.ntw * steps * 128;
            best = q;
            if (q.rows / 16 >= W / wn) break;   // every wave has a slice group; else share out the comps further
        }
    return best;
}

inline FlowPlan flow_decompress_plan(int d, int k)
{
    FlowPlan best;
    if (k > 128) return best;
    const int words = (k + 3) / 4, kst = (k + 31) / 32, ET = (d + 15) / 16;
    for (int W = 4; W <= 8 && !best.waves; W *= 2)
        for (int wn = 1; wn <= W; wn *= 2) {
            FlowPlan q;
            q.exact = flow_exact(d, k);
            q.waves = W; q.kst = kst; q.wn = wn;
            if (wn > 1 && wn / 2 >= ET) break;   // waves with nothing to do
            q.etw = flow_round_up((ET + wn - 1) / wn, {1, 2, 3, 4, 5, 6, 7, 8, 10, 12});
            const int most = W == 4 ? (kst == 1 ? 12 : kst == 2 ? 8 : kst == 3 ? 5 : 4) : (kst <= 2 ? 8 : kst == 3 ? 7 : 5);   // registers
            if (!q.etw || q.etw > most) continue;
            if (W == 8 && wn < 8) continue;      // what is compiled for eight waves
            q.per_cu = 8 / W;
            q.fixed_bytes = 4 * (size_t)(16 * wn * q.etw);
            q.row_bytes = flow_row(kst) + 4 * (size_t)flow_out_row(d);
            q.rows = flow_most_rows(64 * W * 4, words, q, W / wn);
            if (q.rows < 16) continue;
            q.words = (size_t)wn * q.etw * kst * 128;
            best = q;
            if (q.rows / 16 >= W / wn) break;    // every wave has a slice group; else share out the elements further
        }
    return best;
}

// The instances of the kernels, all that a plan can ask for and no more: f(tiles per wave, steps, exact, waves) as constants
// (compress: comp tiles, steps of elements; decompress: steps of comps, element tiles).  False: there is none.
template <int... S> struct FlowSteps {};
template <int T, bool EXACT, int W, typename F, int... S> bool flow_instance(int s, FlowSteps<S...>, F f)
{
    bool found = false;
    ((s == S ? (f(std::integral_constant<int, T>{}, std::integral_constant<int, S>{}, std::integral_constant<bool, EXACT>{},
                  std::integral_constant<int, W>{}),
                (void)(found = true))
             : (void)0),
     ...);
    return found;
}
template <typename F> bool flow_compress_instance(const FlowPlan& p, F f)
{
    if (p.waves == 8) return !p.exact && p.ntw == 1 && flow_instance<1, false, 8>(p.steps, FlowSteps<10, 12, 16>{}, f);
    if (p.waves != 4) return false;
    if (p.exact) {
        // fewer than 10 flop/B: more than 16 comps only with short slices
        if (p.ntw == 1) return flow_instance<1, true, 4>(p.steps, FlowSteps<1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16>{}, f);
        if (p.ntw == 2) return flow_instance<2, true, 4>(p.steps, FlowSteps<1, 2, 3, 4>{}, f);
        return p.ntw == 3 && flow_instance<3, true, 4>(p.steps, FlowSteps<2>{}, f);
    }
    if (p.ntw == 1) return flow_instance<1, false, 4>(p.steps, FlowSteps<5, 6, 7, 8, 10, 12, 16>{}, f);
    if (p.ntw == 2) return flow_instance<2, false, 4>(p.steps, FlowSteps<2, 3, 4, 5, 6, 7, 8>{}, f);
    if (p.ntw == 3) return flow_instance<3, false, 4>(p.steps, FlowSteps<2, 3, 4, 5>{}, f);
    return p.ntw == 4 && flow_instance<4, false, 4>(p.steps, FlowSteps<2, 3, 4>{}, f);
}
template <typename F> bool flow_decompress_instance(const FlowPlan& p, F f)
{
    if (p.waves == 8) {
        if (p.kst == 1) return p.exact ? flow_instance<1, true, 8>(p.etw, FlowSteps<7, 8>{}, f) : flow_instance<1, false, 8>(p.etw, FlowSteps<7, 8>{}, f);
        if (p.exact) return false;
        if (p.kst == 2) return flow_instance<2, false, 8>(p.etw, FlowSteps<5, 6, 7, 8>{}, f);
        if (p.kst == 3) return flow_instance<3, false, 8>(p.etw, FlowSteps<3, 4, 5, 6, 7>{}, f);
        return p.kst == 4 && flow_instance<4, false, 8>(p.etw, FlowSteps<3, 4, 5>{}, f);
    }
    if (p.waves != 4) return false;
    if (p.exact) {
        // fewer than 10 flop/B: more than 32 comps only with slices of 33 to 50
        if (p.kst == 1) return flow_instance<1, true, 4>(p.etw, FlowSteps<1, 2, 3, 4, 5, 6, 7, 8, 10, 12>{}, f);
        return p.kst == 2 && flow_instance<2, true, 4>(p.etw, FlowSteps<3, 4>{}, f);
    }
    if (p.kst == 1) return flow_instance<1, false, 4>(p.etw, FlowSteps<4, 5, 6, 7, 8, 10, 12>{}, f);
    if (p.kst == 2) return flow_instance<2, false, 4>(p.etw, FlowSteps<3, 4, 5, 6, 7, 8>{}, f);
    if (p.kst == 3) return flow_instance<3, false, 4>(p.etw, FlowSteps<3, 4, 5>{}, f);
    return p.kst == 4 && flow_instance<4, false, 4>(p.etw, FlowSteps<3, 4>{}, f);
}

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

// Which kernels take a shape: these, or the LDS-tiled ones of gvq_codec_long.hip where those are faster.  Their word-wide
// path needs slices (and, for decompress, comps) of whole words; lengths of any other kind always come here, but for the
// smallest ranges.  It depends on the handle alone, never on the range of a call: a segment has the bits of the whole.
//
// Measured on 67 lengths x up to 11 numbers of comps, 0.5 to 100 M elements, one basis, 24 and thousands, both storage types
// (here / there, geometric mean over the lengths named, 1 = level): 22499 pairs with everything here 0.64, 8.3 % of them more
// than 5 % slower; 21556 with these rules 0.71, 2.4 % slower, nearly all of them by 1 - 2 us of at most 30.
struct FlowShape {
    int d, k, bases;
    bool bf16;       // storage of the gradient (compress) or of the result (decompress)
    int64_t slices;
    int cus;
};

// Tiles per work-group of the whole gradient.
inline double flow_tiles_each(const FlowShape& s, const FlowPlan& p)
{
    return (double)s.slices / p.rows / ((double)s.cus * p.per_cu);
}

// Short slices and few tiles: such a call is a few microseconds of latency, and a tile's phases make more of it.  Exact
// products, one basis, f32, 0.5 M elements: d = 13 compress 7.5 us against 6.0, d = 24 decompress 5.6 against 4.4; from a
// tile per work-group on 0.65 - 0.9.
inline bool flow_too_small(const FlowShape& s, const FlowPlan& p)
{
    const double each = flow_tiles_each(s, p);
    return p.exact && ((s.d <= 48 && each < 0.25) || (s.d % 4 == 0 && s.d <= 64 && each < 1));
}

// The register-resident kernels of gvq_codec.hip keep a shape of theirs whose comps are whole words.  Of the others, which go
// through their bounds-checked loop, compress of many short slices comes here, with enough tiles (8192 elements) for every
// work-group of the chip and, with several bases, enough of them per basis: each basis ends with a tile that is partly empty,
// and a work-group loads U anew for it.  Here / there, 1 = level, 1 to 100 M elements, one basis down to 3000 elements per basis:
//   d = 16: f32 from 16 M elements on 0.72 - 1.0, 6000 a basis 0.8 - 1.07, 3000 1.0 - 1.4, 8 M elements 1.07 - 1.2; bf16 from 16 M on
//     0.55 - 0.99 down to 6000 a basis, 3000 k = 2 and 5 0.86 - 0.91, 11 and 15 1.0 - 1.25, 8 M elements 0.83 - 1.0 and 0.95 - 1.1;
//   d = 32, k <= 16: f32 from 32 M on 0.85 - 0.97, 15000 a basis 0.92 - 0.95, 20000 0.95 - 1.07, 10000 1.06 - 1.16; bf16 from 16 M
//     on 0.56 - 0.96 down to 20000 a basis, 6000 and 10000 0.74 - 1.1, 8 M elements one basis 0.85, several 1.07 - 1.3;
//   d = 32, k > 16: f32 from 32 M on and bf16 from 6.4 M on 0.5 - 0.9 down to 6000 a basis, 3000 k = 22 1.0 - 1.1, 30 0.83 - 0.95;
//   d = 64, from 32 M on: f32 k = 17 1.0 - 1.1, 19 to 29 0.7 - 0.99, 15000 a basis 0.85 - 0.91, 20000 0.85 - 1.08, 10000 1.0 - 1.25; bf16
//     k = 17 and 19 1.0 - 1.25, 21 0.9 - 1.06 (from 48 M on 0.87 - 0.98), 26 and 29 0.75 - 0.97, 10000 a basis 1.02 - 1.16.
// d = 128 (k = 13, 21: 0.96 - 1.5), fewer comps at d = 64 and decompress (d = 16, k = 5 78 / 72 us) stay there.
inline bool flow_resident_shape(int d, int k) { return k <= 32 && (d == 16 || d == 32 || d == 64 || d == 128); }

inline bool flow_takes_resident_compress(const FlowShape& s)
{
    double each, per_basis;   // fewest tiles per work-group, two on a unit, and per basis
    if (s.d == 16) {
        each = s.bf16 && s.k < 8 ? 1.9 : 3.8;
        per_basis = s.bf16 && s.k < 8 ? 0.3 : 0.6;
    } else if (s.d == 32 && s.k <= 16) {
        each = !s.bf16 ? 7.6 : s.bases > 1 ? 3.8 : 1.5;
        per_basis = s.bf16 ? 0.6 : 1.5;
    } else if (s.d == 32) {
        each = s.bf16 ? 1.5 : 7.6;
        per_basis = s.k > 24 ? 0.3 : 0.6;
    } else if (s.d == 64 && s.k > (s.bf16 ? 20 : 18)) {
        each = s.bf16 && s.k <= 24 ? 11 : 7.6;
        per_basis = 1.5;
    } else {
        return false;
    }
    const double tiles = (double)s.slices * s.d / 8192;
    return s.k % 4 != 0 && tiles >= each * 2 * s.cus && (s.bases == 1 || tiles >= per_basis * s.bases);
}

inline bool flow_takes_compress(const FlowShape& s)
{
    const FlowPlan p = flow_compress_plan(s.d, s.k);
    if (!p.waves) return false;
    if (flow_resident_shape(s.d, s.k)) return p.exact && flow_takes_resident_compress(s);
    if (!s.bf16 && flow_too_small(s, p)) return false;
    if (s.d % 4) return true;
    // U over eight waves (f32 d = 400, k = 100 1.18, bf16 d = 500, k = 128 1.24); above 256 elements with bf16 storage or
    // several bases (d = 512, k = 20 bf16 1.6; d = 400, k = 60 24 bases 1.3)
    if (p.waves != 4 || (s.d > 256 && (s.bf16 || s.bases > 1))) return false;
    // one tile of comps and long slices: a tile's rows do not give every wave a group of slices (f32 257 - 512 elements 1.1 -
    // 1.2, bf16 161 - 256 1.05 - 1.2), which does not matter (0.4 - 0.8) while there is less than a tile for each
    return !(s.k <= 16 && s.d > (s.bf16 ? 160 : 256) && flow_tiles_each(s, p) >= 1);
}

inline bool flow_takes_decompress(const FlowShape& s)
{
    const FlowPlan p = flow_decompress_plan(s.d, s.k);
    const int d = s.d, k = s.k;
    if (!p.waves) return false;
    if (flow_resident_shape(d, k)) return false;
    if (flow_too_small(s, p)) return false;
    if (d % 4) return true;
    const double each = flow_tiles_each(s, p);
    if (d % 256 == 0) return false;   // 24 bases 1.1, to bf16 1.27
    // few comps: little to read per number written, where those kernels' ordinary stores are at their best (f32 129 - 256
    // elements 1.1 - 1.28, to bf16 65 - 192 1.0 - 1.3; below a tile each 0.5 - 0.9)
    if (k <= 16 && d > (s.bf16 ? 64 : 128) && each >= (d > 768 ? 2 : 1)) return false;
    // between one tile and two: the second waits for the first, and the smaller tiles there come out more evenly (1.05 - 1.2)
    if (!p.exact && d > 64 && d <= 320 && k <= 64 && each > 1 && each <= 2) return false;
    if (!s.bf16) return true;
    // to bf16, where half the bytes are written: what is left is what their narrow reads of comps that are no whole words,
    // or the padding to 64 elements, cost there
    if (d < 64) return k % 4 != 0;                  // otherwise 1.0 - 1.2
    if (d <= 128) return k > 16 && (k % 4 != 0 || k <= 32);   // 0.77 - 0.97, otherwise 1.0 - 1.1
    if (d <= 160) return k > 32 || each < 1;        // otherwise 1.05 - 1.15
    if (d < 200) return true;                       // 0.85 - 0.95
    if (d <= 768) return k % 4 != 0 && k > 32;      // 0.8 - 0.9, otherwise 0.95 - 1.3
    return true;                                    // 0.5 - 0.95
}
