// Moments of the basis refresh (GradiVeQ Section 2, PCA paragraph after Eq. 4) from many samples, slices longer than 64
// elements: sum x and sum x x^T as gvq_moments.hip gives them, with the products on the int8 matrix pipe
// (v_mfma_i32_16x16x64_i8, 4.2 to 4.4 PFLOP/s at the 2.0 to 2.1 GHz that this load leaves) instead of the fp64 one (77.5 TFLOP/s).
//
// A number becomes a whole number of 48 bits in units of its column's scale and that a sum of six digits in base 256, -128 to
// 127 each.  A product of two digits summed over up to 20480 samples is exact in int32.  Seven levels of products have sums of
// their own; the eighth is added up over a block and then goes into the seventh, less its lower byte; the others count 2^-64 of
// the largest product and less and are left out.  Scales have room for 2 to 4 times a column's largest number so far, so that
// an fp32 number is exact if it is above 2^-24 of that room (bf16: 2^-40).
//
// What keeps the sums as good as float64 sums of exact products (INT_LOW, INT_MANY): no 16 numbers of a column that a thread
// converts are all below 2^-6 of the room, unless they are zeros or fewer (the last of a task's samples of a gradient), and no more than an eighth of these items have a number below
// 2^-16.  A block for which that is not so, or that holds a number out of range, gets new scales; where new scales do not help,
// it is multiplied on the fp64 pipe (int_exactly), as are the blocks behind it if new scales are asked for too often.  Difference to
// long double sums over sqrt(C_aa C_bb), rms, fp64 pipe -> here: planted model, 200 000 samples of 96 elements at 64 scales
// 1.1e-16 -> 4.9e-17, 100 000 of 80 4.4e-17 -> 4.2e-17, 78 000 of 256 7.7e-17 -> 3.9e-17; 40 000 of 128, products of three normal
// numbers 1.4e-17 -> 1.3e-17, columns from 1 to 1e-8 4.0e-17 -> 1.1e-17; ten draws of 16 400 samples of 96 and 128: normal 1.6e-17 ->
// 1.3e-17, lognormal (sigma = 3) 2.0e-17 -> 1.9e-17 (bf16 1.9e-17 -> 1.7e-17), fourth powers of normal numbers 2.3e-17 both (bf16 too),
// one in a hundred a thousand times larger 1.5e-17 -> 1.3e-17 (1.4e-17 both), repeated numbers with an outlier 9.9e-16 -> 6.4e-16.
// (Without the eighth level and these conditions lognormal numbers 1.7e-16, bf16 1.3e-14, fourth powers 1.1e-16 and 1.3e-14.)
//
// Digits come from float64: x * scale + 1.5 * 2^52 + 0x80..80 has them, plus 128 each, as its lower bytes (one conversion and one
// v_fma_f64; with fp32 arithmetic alone it took seven instructions a number and the kernel a sixth longer).  The last digit
// (bf16: the last three) is 0 in nearly every number: its products are made only for tiles of a block that have another one
// (bf16: of the fourth digit, and rarer yet the last two apart: 139 bases of d = 128, 32 gradients 5.20 -> 5.04 ms).
//
// What bounds it: instruction issue.  A wave issues a vector instruction every 5 cycles, every 7.8 while another wave of its SIMD
// has products in flight, and its own products do not overlap with its own vector instructions.  Hence twelve waves of 168
// registers, three a SIMD: of up to three pairs of tiles each, 28 registers a pair, some of which park the next block before their
// products and some behind them; for eight tiles with themselves (36 pairs) two pairs for the four that park first, three
// for the four that park behind their products and four for those that do not park, a few of whose registers are in scratch.
// 32 gradients of 138 M elements, d = 128, with the eigensolver: fp64 pipe 9.9 ms, here 7.0 (without the eighth level 6.2; three pairs
// for every wave 7.9, spills; eight waves of 256 registers and every wave parking between its own products were slower yet);
// 8 gradients of d = 768 16.5 -> 12.9 ms.  Data that go to the fp64 pipe after all take up to a
// tenth longer than in its own kernel, whose tasks are cut finer (60 M elements, 8 gradients, Student's t with three degrees of freedom, or lognormal with
// sigma = 1): d = 128 1.55 -> 1.58 ms, in bf16 1.54 -> 1.55, d = 160 2.04 -> 2.18, d = 768 8.8 -> 9.8 (with twice as many tries of
// new scales, and blocks parked whole between two barriers, 1.75, 1.70, 2.45 and 10.6); sizes that change by orders of
// magnitude every block 1.56 -> 1.57, where new scales every time took twice as long.
#include <math.h>

#include "gvq_moments.h"
#include "gvq_moments_place.h"

typedef int i4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));

#define INT_THREADS 768
#define INT_WAVES 12
#define INT_SLOTS 2
#define INT_ND 6                      // digits of a number
#define INT_LEVELS 7                  // with sums of their own
#define INT_LOW 6                     // bits
#define INT_MANY 8                    // items of a wave's 64
#define INT_FLUSH 320                // blocks between flushes: 6 products of 2^14 a sample stay below 2^31 for 21845 samples

static_assert(INT_MOST_D >= GVQ_MAX_D, "columns past a slice's end");

template <int NT, bool OFF> struct IntShape {
    using Mom = MomShape<NT, OFF>;
    static constexpr int TILES = Mom::TILES, NPAIR = Mom::NPAIR, COLS = 16 * TILES;
    // The threads of this wave park an item each: 16 samples of one column.
    static_assert(COLS * 4 <= INT_THREADS, "an item per thread");
    static constexpr bool parks(int w) { return 64 * w < COLS * 4; }
    static constexpr int PLANE = TILES * 1024, BUF = INT_ND * PLANE;           // bytes: one digit, one block
    // a block in float64, where the two blocks of digits are otherwise: doubles per sample
    static constexpr int ROW = 16 * (TILES | 1);
    static_assert(INT_NS * ROW * 8 <= 2 * BUF, "a block in float64");
    static constexpr int LDS = 2 * BUF + 8 * COLS + 2 * 16 * 4 + (OFF ? 0 : 32 * COLS);
    // the pairs in the order in which the waves share them out: 2 x 2 tiles at a time
    struct Order { int p[NPAIR]; };
    static constexpr Order make_order()
    {
        Order o{};
        int n = 0;
        constexpr int SB = (NT + 1) / 2;
        for (int R = 0; R < SB; ++R)
            for (int q = OFF ? 0 : R; q < SB; ++q) {
                const int C = R & 1 ? SB - 1 - (q - (OFF ? 0 : R)) : q;
                for (int k = 0; k < 4; ++k) {
                    const int r = 2 * R + (k >> 1), c = 2 * C + ((k ^ (k >> 1)) & 1);
                    if (r >= NT || c >= NT || (!OFF && c < r)) continue;
                    for (int p = 0; p < NPAIR; ++p)
                        if (Mom::row(p) == r && Mom::col(p) == (OFF ? NT + c : c)) o.p[n++] = p;
                }
            }
        return o;
    }
    static constexpr Order order = make_order();
    // of eight tiles with themselves, the waves that do not park take a pair from those that park first
    static constexpr int extra(int w) { return (INT_WAVES - 1 - w < NPAIR % INT_WAVES ? 1 : 0) + (!OFF && NT == 8 ? (w < 4 ? -1 : w < 8 ? 0 : 1) : 0); }
    static_assert(NPAIR >= INT_WAVES, "a pair for every wave");
    static constexpr int first(int w)
    {
        int p = 0;
        for (int i = 0; i < w; ++i) p += NPAIR / INT_WAVES + extra(i);
        return p;
    }
    static constexpr int row(int i) { return Mom::row(order.p[i]); }
    static constexpr int col(int i) { return Mom::col(order.p[i]); }
    // Which tiles a wave's two sets of operand registers hold when pair i is multiplied (phase 1: once its own tiles are
    // there; phase 2: with the tile that the next pair wants, where a set is free for it; phase 0: before either).
    struct Slots { int t[INT_SLOTS]; };
    static constexpr int slot(const Slots& s, int tile)   // INT_SLOTS: in none
    {
        int q = 0;
        while (q < INT_SLOTS && s.t[q] != tile) ++q;
        return q;
    }
    static constexpr bool holds(const Slots& s, int tile) { return slot(s, tile) < INT_SLOTS; }
    static constexpr Slots slots(int p0, int p1, int i, int phase)
    {
        Slots s{};
        for (int q = 0; q < INT_SLOTS; ++q) s.t[q] = -1;
        for (int p = p0; p <= i; ++p) {
            const int need[2] = {row(p), col(p)};
            if (p == i && phase == 0) return s;
            for (int k = 0; k < 2; ++k) {
                if (holds(s, need[k])) continue;
                for (int q = 0; q < INT_SLOTS; ++q)
                    if (s.t[q] != need[0] && s.t[q] != need[1]) { s.t[q] = need[k]; break; }
            }
            if (p == i && phase == 1) return s;
            if (p + 1 == p1) continue;
            const int then[2] = {row(p + 1), col(p + 1)};
            for (int k = 0; k < 2; ++k) {
                if (holds(s, then[k])) continue;
                for (int q = 0; q < INT_SLOTS; ++q)
                    if (s.t[q] != need[0] && s.t[q] != need[1] && s.t[q] != then[0] && s.t[q] != then[1]) { s.t[q] = then[k]; break; }
            }
        }
        return s;
    }
};

// Four samples of one column -> four bytes (one dword) per digit.  Bytes 0 to 3 of lo hold digits 5 to 2, the two lowest
// bytes of hi the others, all biased by 128, which the exclusive or turns into two's complement.
__device__ __forceinline__ void pack_digits(const unsigned int (&hi)[4], const unsigned int (&lo)[4], unsigned int (&out)[INT_ND])
{
    const auto perm = [](unsigned int high, unsigned int low, unsigned int sel) { return __builtin_amdgcn_perm(high, low, sel); };
    const unsigned int p = perm(lo[1], lo[0], 0x05010400u), q = perm(lo[3], lo[2], 0x05010400u);
    const unsigned int r = perm(lo[1], lo[0], 0x07030602u), s = perm(lo[3], lo[2], 0x07030602u);
    const unsigned int t = perm(hi[1], hi[0], 0x05010400u), u = perm(hi[3], hi[2], 0x05010400u);
    out[5] = perm(q, p, 0x05040100u) ^ 0x80808080u;
    out[4] = perm(q, p, 0x07060302u) ^ 0x80808080u;
    out[3] = perm(s, r, 0x05040100u) ^ 0x80808080u;
    out[2] = perm(s, r, 0x07060302u) ^ 0x80808080u;
    out[1] = perm(u, t, 0x05040100u) ^ 0x80808080u;
    out[0] = perm(u, t, 0x07060302u) ^ 0x80808080u;
}

// A task's samples: rows j0 .. j0 + n of every gradient in `blocks` blocks.
struct IntRange {
    int64_t j0;
    int n, blocks;
    int tail;   // rows of the gradient behind them, less a block (no more than an int holds)
};

// A block: 64 slices from src on, of which only those from `skip` on and no more than `rows` count.  One that ends a task's
// samples, or lies at the gradient's end, is read with its neighbours, so that every load is whole.
struct IntBlock { uintptr_t src; int skip, rows; };

// The blocks of all gradients one after the other, from number `done` on.
struct IntBlocks {
    IntBlock ahead;   // the one to request next
    int left, rows_left, l;
    __device__ __forceinline__ IntBlocks(const MomArgs& a, const IntRange& r, int done, int step)
    {
        left = r.blocks * a.L - done;
        l = r.blocks ? done / r.blocks : 0;
        const int i = done - l * r.blocks;
        rows_left = 0;
        ahead = IntBlock{0, 0, INT_NS};
        if (i > 0) {   // as if the block before had been requested
            ahead.src = (uintptr_t)a.grads.p[l++] + r.j0 * step + (int64_t)(i - 1) * (INT_NS * step);
            rows_left = r.n - (i - 1) * INT_NS;
        }
    }
    __device__ __forceinline__ void next(const MomArgs& a, const IntRange& r, int step)
    {
        if (left == 0) return;   // the last block is requested again: loads stay unconditional
        --left;
        rows_left -= INT_NS;
        ahead.src += INT_NS * step;
        if (rows_left < INT_NS) {
            if (rows_left <= 0) {
                ahead.src = (uintptr_t)a.grads.p[l++] + r.j0 * step;
                rows_left = r.n;
            }
            ahead.rows = rows_left < INT_NS ? rows_left : INT_NS;
            const int past = -rows_left - r.tail;   // slices that the block's 64 would reach past the gradient's last
            ahead.skip = past > 0 ? past : 0;
            ahead.src -= ahead.skip * step;
        }
    }
};

// Hides a value's origin, so that what is made from it is not kept in registers from one block to the next.
template <typename T> __device__ __forceinline__ T fresh(T v)
{
    asm("" : "+v"(v));
    return v;
}

// Four of an item's 16 samples.  Loads through a buffer resource: the rows' distances are uniform offsets, which a lane's address
// would have to add up.
template <bool BF16, bool OFF>
__device__ __forceinline__ void int_load_quad(float (&x)[16], int q, const IntBlock& k, unsigned int place, int step)
{
    auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)k.src, 0, INT_NS * step, 0x00027000);
    const unsigned int at = int_place_from(fresh(place)) + (q >= 2 ? 8u * step : 0u);
#pragma unroll
    for (int i = 4 * q; i < 4 * q + 4; ++i) {
        const int row = __builtin_amdgcn_readfirstlane((i & 7) * step);
        if (BF16) x[i] = __uint_as_float((unsigned int)__builtin_amdgcn_raw_buffer_load_b16(rsrc, at, row, 0) << 16);
        else x[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, at, row, OFF ? 0 : 2));
    }
}
template <bool BF16, bool OFF>
__device__ __forceinline__ void int_load(float (&x)[16], const IntBlock& k, unsigned int place, int step)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) int_load_quad<BF16, OFF>(x, q, k, place, step);
}
template <int I0 = 0, int I1 = 16>
__device__ __forceinline__ void int_mask(float (&x)[16], const IntBlock& k, unsigned int place)   // samples that do not count become zeros
{
    if (k.rows < INT_NS) {
        const int r = 16 * int_place_quarter(fresh(place)) - k.skip;
#pragma unroll
        for (int i = I0; i < I1; ++i) x[i] = (unsigned int)(r + i) < (unsigned int)k.rows ? x[i] : 0.f;
    }
}

// A uniform value, or the thread, of which nothing is worked out ahead of the loops around this.
template <typename T> __device__ __forceinline__ T here(T v)
{
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ int int_thread()
{
    int v = threadIdx.x;
    asm volatile("" : "+v"(v));
    return v;
}

// This thread's item.
template <int NT, bool BF16, bool OFF> __device__ __forceinline__ unsigned int int_item(const MomArgs& a, int tid, int pa, int pb)
{
    constexpr int COLS = IntShape<NT, OFF>::COLS;
    const int c = tid % COLS, q = tid / COLS;
    const int e = OFF && c >= 16 * NT ? pb * a.pw + c - 16 * NT : pa * a.pw + c;
    return int_place(int_from(e, q, a.d, BF16 ? 2 : 4), c, q);
}

// What lies in LDS behind the blocks.
template <int NT, bool OFF> struct IntLds {
    using Sh = IntShape<NT, OFF>;
    unsigned int* colmax;   // [COLS]
    int* cexp;              // [COLS] x 2^cexp is what the digits hold
    // [2][16], a word per wave: 1 a number is out of its column's range, 2 an item's are all far below it, 4 too many items have
    // last digits; from bit 3 on, the tiles whose first digit of those that are nearly always 0 is not, from bit 15 on, the others
    unsigned int* flags;
    double* sums;           // [4][COLS] of x
    __device__ __forceinline__ explicit IntLds(unsigned char* lds)
        : colmax((unsigned int*)(lds + 2 * Sh::BUF)), cexp((int*)(colmax + Sh::COLS)), flags((unsigned int*)(cexp + Sh::COLS)),
          sums((double*)(flags + 32))
    {
    }
};

// Blocks from number `done` on; returns the first that it leaves undone because digits will not do for it (but its samples are in
// the sums of x).
template <int NT, bool BF16, bool OFF, int WAVE>
__device__ __forceinline__ int int_task(const MomArgs& a, unsigned char* lds, int pa, int pb, const IntRange& range, int done, int patience, double* out,
                                        unsigned int& taken)
{
    using Sh = IntShape<NT, OFF>;
    constexpr int P0 = Sh::first(WAVE), NA = Sh::first(WAVE + 1) - P0;
    constexpr int NB = BF16 ? 3 : 5;   // digits of every number; the others are nearly always zero
    constexpr int COLS = Sh::COLS, ND = INT_ND, BITS = 8 * ND;
    constexpr bool PARKS = Sh::parks(WAVE);
    const int tid = int_thread(), lane = tid & 63;
    const IntLds<NT, OFF> at(lds);
    const int step = a.d * (BF16 ? 2 : 4);
    unsigned int place = 0u;
    if constexpr (PARKS) place = int_item<NT, BF16, OFF>(a, tid, pa, pb);
    auto col_of = [](unsigned int p) { return int_place_column(p); };
    auto quarter_of = [](unsigned int p) { return int_place_quarter(p); };

    float x[16];
    auto load_quad = [&](int q, const IntBlock& k) { int_load_quad<BF16, OFF>(x, q, k, place, step); };
    auto load = [&](const IntBlock& k) { int_load<BF16, OFF>(x, k, place, step); };
    auto mask = [&](const IntBlock& k) { int_mask(x, k, place); };
    IntBlocks blocks(a, range, done, step);
    int todo = blocks.left;
    auto next_block = [&]() { blocks.next(a, range, step); };

    int by = 0;                // x * 2^by is the whole number that the digits hold, for numbers below 2^(BITS - 1 - by)
    unsigned int marks = 0u;   // of the block just parked, see flags
    bool stale = false;        // ... and whether this thread's item asks for another scale
    auto sum_at = [&]() {
        const unsigned int p = fresh(place);
        return quarter_of(p) * COLS + col_of(p);
    };
    // Block k, which x holds.  `then(q)` follows the last use of four samples' registers; `count`: the samples are new to the sums of x.
    auto park = [&](const IntBlock& k, unsigned char* buf, bool count, auto then) {
        // 1.5 * 2^52 makes the sum's unit 1: its lower bits are the whole number, biased so that every byte is a digit + 128
        constexpr double BIAS = 0x1.8p52 + 0x808080808080p0;
        const double scale = __builtin_bit_cast(double, (unsigned long long)(1023 + fresh(by)) << 52);
        double sum[2] = {0.0, 0.0};
        float most = 0.f;
        unsigned int last = 0u, deep = 0u;
        i4 out4[ND];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            unsigned int hi[4], lo[4], dig[ND];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float f = x[4 * q + i];
                const double v = (double)f;
                const unsigned long long t = __builtin_bit_cast(unsigned long long, __builtin_fma(v, scale, BIAS));
                hi[i] = (unsigned int)(t >> 32);
                lo[i] = (unsigned int)t;
                most = __builtin_fmaxf(most, __builtin_fabsf(f));
                if (!OFF) sum[i & 1] += v;
            }
            pack_digits(hi, lo, dig);
#pragma unroll
            for (int g = 0; g < ND; ++g) {
                out4[g][q] = (int)dig[g];
                if (g == NB) last |= dig[g];
                if (g > NB) deep |= dig[g];
            }
            then(q);
        }
        unsigned char* o = buf + int_place_lds(fresh(place));
#pragma unroll
        for (int g = 0; g < ND; ++g) *(i4*)(o + g * Sh::PLANE) = out4[g];
        const int room = BITS - 1 - fresh(by);
        const bool low = most > 0.f && most < ldexpf(0.98f, room - INT_LOW);
        const unsigned long long some = __ballot((last | deep) != 0u);
        const bool many = __builtin_popcountll(some) > INT_MANY;
        stale = low || (many && (last | deep) != 0u);
        // fewer than 16 samples say little about their column
        constexpr int Q0 = 64 * WAVE / COLS, Q1 = (64 * WAVE + 63) / COLS;
        const bool whole = k.skip <= 16 * Q0 && k.skip + k.rows >= 16 * Q1 + 16;
        marks = (__any(!(most < ldexpf(0.98f, room))) ? 1u : 0u)   // 0x7f7f.. of 0x8000..: every byte's digit is at most 127
                | (__any(low) && whole ? 2u : 0u) | (many ? 4u : 0u);
        // a wave has four tiles' columns, side by side or around the end
        auto tiles = [](unsigned long long items) {
            const unsigned int t = (items & 0xffffull ? 1u : 0u) | (items & 0xffff0000ull ? 2u : 0u)
                                   | (items & 0xffff00000000ull ? 4u : 0u) | (items & 0xffff000000000000ull ? 8u : 0u);
            const unsigned int at_tile = t << 64 * WAVE % COLS / 16;
            return (at_tile | at_tile >> Sh::TILES) & ((1u << Sh::TILES) - 1u);
        };
        if (some != 0ull) {
            marks |= tiles(__ballot(last != 0u)) << 3;
            if constexpr (NB + 1 < ND) marks |= tiles(__ballot(deep != 0u)) << 15;
        }
        if (!OFF && count) unsafeAtomicAdd(&at.sums[sum_at()], sum[0] + sum[1]);
    };

    bool stored = a.accumulate != 0 || done > 0;   // the partials hold something to add to
    // accumulators -> float64
    auto flush = [&](i4 (&acc)[NA > 0 ? NA : 1][INT_LEVELS]) {
        double* const first = here(out) + (lane >> 4) * 64 + (lane & 15);
        static_for<NA>([&](auto ii) {
            constexpr int I = decltype(ii)::value, R = Sh::row(P0 + I), C = Sh::col(P0 + I), P = Sh::order.p[P0 + I];
            double* o = first + P * 256;
            const int ec = at.cexp[16 * C + (lane & 15)];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int er = at.cexp[16 * R + 4 * (lane >> 4) + r];
                double v = (double)acc[I][INT_LEVELS - 1][r];
#pragma unroll
                for (int s = INT_LEVELS - 2; s >= 0; --s) v = __builtin_fma(v, 0x1p-8, (double)acc[I][s][r]);
                // level 0 is the product of two top digits
                v = ldexp(v, 16 * (ND - 1) - er - ec);
                o[r * 16] = stored ? o[r * 16] + v : v;
            }
        });
        stored = true;
    };
    // What the waves found in the block they have parked; returns once it is all there.
    unsigned int found = 0u;
    int parity = 0;   // of the exchange: a slow wave may still read the last one's words
    auto exchange = [&]() {
        parity ^= 1;
        const int self = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, fresh(0u)));   // the lane
        if (PARKS && self == 0) at.flags[parity * 16 + WAVE] = marks;
        __syncthreads();
        found = at.flags[parity * 16 + (self & 15)];
    };
    // ... all waves' findings in one word
    auto findings = [&]() {
        unsigned int f = found;
        f |= __builtin_amdgcn_mov_dpp(f, 0xb1, 0xf, 0xf, true);    // lane ^ 1
        f |= __builtin_amdgcn_mov_dpp(f, 0x4e, 0xf, 0xf, true);    // lane ^ 2
        f |= __builtin_amdgcn_mov_dpp(f, 0x141, 0xf, 0xf, true);   // 7 - lane of 8
        f |= __builtin_amdgcn_mov_dpp(f, 0x140, 0xf, 0xf, true);   // 15 - lane of 16
        return (unsigned int)__builtin_amdgcn_readfirstlane(f);
    };
    next_block();
    IntBlock parked_block = blocks.ahead;   // in LDS ...
    next_block();
    IntBlock req = blocks.ahead;            // in registers, or on its way
    next_block();
    // New scales, for the columns' largest numbers so far (`all`, and columns that asked for it: of this block) and in block k,
    // which is then parked with them.
    bool counted = false;   // ... whose samples are in the sums of x
    auto refresh = [&](const IntBlock& k, bool all, unsigned char* buf) {
        const unsigned int p = fresh(place);
        if constexpr (PARKS) {
            if (all || stale) at.colmax[col_of(p)] = 0u;
        }
        __syncthreads();   // (also: all flushes have read cexp)
        if constexpr (PARKS) {
            load(k);
            mask(k);
            float most = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) most = __builtin_fmaxf(most, __builtin_fabsf(x[i]));
            most = __builtin_fminf(most, 3.4028235e38f);
            atomicMax(&at.colmax[col_of(p)], __float_as_uint(most));
        }
        __syncthreads();
        if constexpr (PARKS) {
            // room for 2 to 4 times the column's largest number; a column of zeros has none, so that its first other number
            // asks for new scales
            const unsigned int m = at.colmax[col_of(p)];
            const double f = (double)__uint_as_float(m ? m : 1u);
            by = BITS - 1 - ((int)(__builtin_bit_cast(unsigned long long, f) >> 52) - 1023 + 2);
            if (quarter_of(p) == 0) at.cexp[col_of(p)] = by;
            park(k, buf, !counted, [](int) {});
        }
        counted = true;
        exchange();
    };
    const unsigned char* mine = lds + lane * 16;
    int flip = 0;
    bool all = done == 0;     // no column's largest number so far is known
    bool again = done > 0;    // they are, but may be of samples much larger than this block's; its columns then say so
    // New scales take as long as a block and a half, a block on the fp64 pipe as long as 1.4: not worth it for fewer than four blocks.
    int spent = 0;
    while (todo > 0) {
        if (spent > patience) break;
        spent += 4;
        // blocks until the scales no longer fit, or the accumulators might overflow; the first, which the last round has
        // parked with the scales it had, is parked again
        refresh(parked_block, all, lds + flip * Sh::BUF);
        all = false;
        if (findings() & 7u) {
            if (!again) break;   // nor do new scales fit
            again = false;
            continue;
        }
        again = false;
        if constexpr (PARKS) load(req);
        i4 acc[NA > 0 ? NA : 1][INT_LEVELS];
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int s = 0; s < INT_LEVELS; ++s) acc[i][s] = i4{0, 0, 0, 0};
        for (int since = 1;; ++since, flip ^= 1) {
            unsigned char* const next = lds + (flip ^ 1) * Sh::BUF;
            const unsigned char* const buf = mine + flip * Sh::BUF;
            i4 op[INT_SLOTS][NB];
            auto fetch_digit = [&](int g, int tile) {
                return *(const i4*)(buf + g * Sh::PLANE + tile * 1024);
            };
            auto fetch_for = [&](auto ii, auto phase) {   // the tiles that change from a phase of pair i to the next
                constexpr int I = decltype(ii)::value, PH = decltype(phase)::value;
                constexpr auto before = Sh::slots(P0, P0 + NA, P0 + I, PH), now = Sh::slots(P0, P0 + NA, P0 + I, PH + 1);
                static_for<NB * INT_SLOTS>([&](auto gi) {   // digit by digit: the first products need the first ones only
                    constexpr int G = decltype(gi)::value / INT_SLOTS, Q = decltype(gi)::value % INT_SLOTS;
                    if constexpr (now.t[Q] != before.t[Q]) op[Q][G] = fetch_digit(G, now.t[Q]);
                });
            };
            // The three waves of a SIMD park at different times, one of them before its products and the others behind, or not at
            // all: while one converts the others have the matrix pipe.
            constexpr bool EARLY = WAVE < 4;
            if constexpr (!EARLY && NA > 0) fetch_for(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
            __builtin_amdgcn_sched_barrier(0);
            const unsigned int known = findings(), rare = known >> 3, deep = known >> 15;
            if (since > INT_FLUSH || (known & 7u)) break;   // (not the first)
            if (!OFF && WAVE == 0) taken += parked_block.rows;
            parked_block = req;
            req = blocks.ahead;
            auto park_next = [&]() {
                if constexpr (PARKS) {
                    mask(parked_block);
                    // the next block as soon as registers are free; the late waves of a panel with itself have none to spare
                    park(parked_block, next, todo > 1, [&](int q) { if (OFF || EARLY) load_quad(q, req); });
                    if (!OFF && !EARLY) load(req);
                }
            };
            if constexpr (EARLY) {
                park_next();
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (NA > 0) fetch_for(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
            }
            // Two panels: who parks behind its products goes first (6060 -> 5660 cycles a block, before the eighth level).  A panel with itself has waves
            // that do not park, and gains nothing (21 pairs of tiles lose 3 %).
            constexpr int PRIORITY = !OFF || EARLY ? 0 : WAVE < 8 ? 2 : 1;
            if constexpr (PRIORITY > 0) __builtin_amdgcn_s_setprio(PRIORITY);
            static_for<NA>([&](auto ii) {
                constexpr int I = decltype(ii)::value;
                __builtin_amdgcn_sched_barrier(0);
                constexpr auto now = Sh::slots(P0, P0 + NA, P0 + I, 1);
                constexpr int R = Sh::row(P0 + I), C = Sh::col(P0 + I), A = Sh::slot(now, R), B = Sh::slot(now, C);
                if constexpr (I > 0) fetch_for(ii, std::integral_constant<int, 0>{});
                fetch_for(ii, std::integral_constant<int, 1>{});
                __builtin_amdgcn_sched_barrier(0);
                i4 rest = i4{0, 0, 0, 0};   // the level below the last
                auto product = [&](const i4& x, int i, const i4& y, int j) {
                    if (i + j < INT_LEVELS) acc[I][i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(x, y, acc[I][i + j], 0, 0, 0);
                    else if (i + j == INT_LEVELS) rest = __builtin_amdgcn_mfma_i32_16x16x64_i8(x, y, rest, 0, 0, 0);
                };
                auto add_rest = [&]() {
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[I][INT_LEVELS - 1][r] += rest[r] >> 8;
                };
#pragma unroll
                for (int top = 0; top < NB; ++top) {   // in the order in which digits arrive, the rest early
                    product(op[A][top], top, op[B][top], top);
#pragma unroll
                    for (int i = top - 1; i >= 0; --i) {
                        product(op[A][top], top, op[B][i], i);
                        product(op[A][i], i, op[B][top], top);
                    }
                }
                if (NB == 5) add_rest();
                if constexpr (PARKS && !EARLY && I == 0) next_block();   // scalar work, between products
                if ((rare >> R | rare >> C) & 1u) {
                    if (NB + NB - 1 >= INT_LEVELS) rest = i4{0, 0, 0, 0};
                    const i4 a_last = fetch_digit(NB, R);
#pragma unroll
                    for (int i = 0; i < NB; ++i) product(a_last, NB, op[B][i], i);
                    const i4 b_last = fetch_digit(NB, C);
                    if (2 * NB < INT_LEVELS) product(a_last, NB, b_last, NB);
#pragma unroll
                    for (int i = 0; i < NB; ++i) product(op[A][i], i, b_last, NB);
                    if (NB + NB - 1 >= INT_LEVELS) add_rest();
                }
                if constexpr (NB + 1 < ND) {
                    if ((deep >> R | deep >> C) & 1u) {
                        rest = i4{0, 0, 0, 0};
#pragma unroll
                        for (int g = NB + 1; g < ND; ++g) {
                            const i4 a_last = fetch_digit(g, R);
#pragma unroll
                            for (int i = 0; i < ND; ++i)
                                if (g + i <= INT_LEVELS) product(a_last, g, i < NB ? op[B][i < NB ? i : 0] : fetch_digit(i, C), i);
                            const i4 b_last = fetch_digit(g, C);
#pragma unroll
                            for (int i = 0; i <= NB; ++i)
                                if (g + i <= INT_LEVELS) product(i < NB ? op[A][i < NB ? i : 0] : fetch_digit(i, R), i, b_last, g);
                        }
                        add_rest();
                    }
                }
            });
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (PRIORITY > 0) __builtin_amdgcn_s_setprio(0);
            if constexpr (!EARLY) park_next();
            --todo;
            spent -= spent > 0 ? 1 : 0;
            if (todo == 0) break;
            if constexpr (EARLY) next_block();
            exchange();   // also: everyone is done with this block's buffer
        }
        flush(acc);
    }
    return range.blocks * a.L - todo;
}

template <int NT, bool BF16, bool OFF>
__device__ __forceinline__ int int_waves(const MomArgs& a, unsigned char* lds, int pa, int pb, const IntRange& range, int done, int patience, double* out,
                                         unsigned int& taken)
{
    switch (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {   // uniform: the cases hold barriers
    case 0: return int_task<NT, BF16, OFF, 0>(a, lds, pa, pb, range, done, patience, out, taken);
    case 1: return int_task<NT, BF16, OFF, 1>(a, lds, pa, pb, range, done, patience, out, taken);
    case 2: return int_task<NT, BF16, OFF, 2>(a, lds, pa, pb, range, done, patience, out, taken);
    case 3: return int_task<NT, BF16, OFF, 3>(a, lds, pa, pb, range, done, patience, out, taken);
    case 4: return int_task<NT, BF16, OFF, 4>(a, lds, pa, pb, range, done, patience, out, taken);
    case 5: return int_task<NT, BF16, OFF, 5>(a, lds, pa, pb, range, done, patience, out, taken);
    case 6: return int_task<NT, BF16, OFF, 6>(a, lds, pa, pb, range, done, patience, out, taken);
    case 7: return int_task<NT, BF16, OFF, 7>(a, lds, pa, pb, range, done, patience, out, taken);
    case 8: return int_task<NT, BF16, OFF, 8>(a, lds, pa, pb, range, done, patience, out, taken);
    case 9: return int_task<NT, BF16, OFF, 9>(a, lds, pa, pb, range, done, patience, out, taken);
    case 10: return int_task<NT, BF16, OFF, 10>(a, lds, pa, pb, range, done, patience, out, taken);
    default: return int_task<NT, BF16, OFF, 11>(a, lds, pa, pb, range, done, patience, out, taken);
    }
}

// Blocks `done` to done + n on the fp64 pipe: 32 rows of float64 in either half of the LDS.  The first block's samples are in the sums of x.
template <int NT, bool BF16, bool OFF>
__device__ __forceinline__ void int_exactly(const MomArgs& a, unsigned char* lds, int pa, int pb, const IntRange& range, int done, int n, double* out,
                                            unsigned int& taken)
{
    using Sh = IntShape<NT, OFF>;
    // a wave has pairs wave, wave + 12, ...: the waves of a SIMD differ by four, so that no SIMD has more than one pair above its share
    constexpr int NF = Sh::NPAIR / INT_WAVES, MORE = Sh::NPAIR % INT_WAVES, NP = NF + (MORE ? 1 : 0);
    const int tid = int_thread(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool parks = wave * 64 < Sh::COLS * 4;
    const IntLds<NT, OFF> at(lds);
    const int step = a.d * (BF16 ? 2 : 4);
    const unsigned int place = parks ? int_item<NT, BF16, OFF>(a, tid, pa, pb) : 0u;
    const bool more = wave < MORE;   // it has NP pairs, not NF
    int row[NP], col[NP];   // first elements of the pairs' tiles
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int p = wave + INT_WAVES * i < Sh::NPAIR ? wave + INT_WAVES * i : 0;
        int r = 0, c = p;
        if (OFF) {
            r = p / NT;
            c = NT + p - r * NT;
        } else {
            for (; c >= NT - r; ++r) c -= NT - r;
            c += r;
        }
        row[i] = 16 * r;
        col[i] = 16 * c;
    }
    // Half a block at a time, in turn in either half of the rows: every thread parks eight of its item's 16 samples for the next
    // products while other waves multiply.  Samples s and s + 4 of eight side by side: a lane reads its operands of two products at once
    // (a product leaves no vector instruction room beside it; one by one: 138 M elements, d = 128, 32 gradients 11.1 ms).
    constexpr int HALF = INT_NS / 4 * Sh::ROW;   // pairs of doubles
    d2* const rows = (d2*)lds;
    d2* const to = rows + 4 * int_place_quarter(place) * Sh::ROW + int_place_column(place);
    const d2* const from = rows + (lane >> 4) * Sh::ROW + (lane & 15);
    IntBlocks blocks(a, range, done, step);
    blocks.next(a, range, step);
    IntBlock block = blocks.ahead;
    float x[16];
    double sum = 0.0;   // of this thread's samples, but the first block's
    if (parks) int_load<BF16, OFF>(x, block, place, step);
    auto park = [&](auto half, const IntBlock& k, bool count) {
        constexpr int H = decltype(half)::value;
        int_mask<8 * H, 8 * H + 8>(x, k, place);
        double part[2] = {0.0, 0.0};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int s = 8 * H + i;
            const d2 v = {(double)x[s], (double)x[s + 4]};
            to[H * HALF + i * Sh::ROW] = v;
            part[0] += v[0];
            part[1] += v[1];
        }
        if (!OFF && count) sum += part[0] + part[1];
    };
    auto load = [&](auto half, const IntBlock& k) {
        constexpr int H = decltype(half)::value;
        int_load_quad<BF16, OFF>(x, 2 * H, k, place, step);
        int_load_quad<BF16, OFF>(x, 2 * H + 1, k, place, step);
    };
    constexpr std::integral_constant<int, 0> lower;
    constexpr std::integral_constant<int, 1> upper;
    // two sums a pair, half as long: the work-groups of gvq_moments.hip, two a compute unit, have half as many samples
    d4 acc[NP][2];
#pragma unroll
    for (int i = 0; i < NP; ++i) acc[i][0] = acc[i][1] = d4{0.0, 0.0, 0.0, 0.0};
    auto multiply = [&](auto half) {
        auto pairs_of = [&](auto pairs) {
#pragma unroll
            for (int g = 0; g < INT_NS / 16; ++g) {
#pragma unroll
                for (int i = 0; i < decltype(pairs)::value; ++i) {
                    if (i > 0) __builtin_amdgcn_sched_barrier(6);   // pair by pair: 10.6 -> 10.4 ms
                    const d2* const at = from + decltype(half)::value * HALF + 4 * g * Sh::ROW;
                    const d2 u = at[row[i]], v = at[col[i]];
                    acc[i][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(u[0], v[0], acc[i][0], 0, 0, 0);
                    acc[i][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(u[1], v[1], acc[i][1], 0, 0, 0);
                }
            }
        };
        if (MORE && more) pairs_of(std::integral_constant<int, NP>{});
        else pairs_of(std::integral_constant<int, NF>{});
    };
    blocks.next(a, range, step);
    IntBlock req = blocks.ahead;
    if (parks) {
        park(lower, block, false);
        load(lower, req);
    }
    __syncthreads();
    for (int k = 0; k < n; ++k) {
        if (parks) {
            park(upper, block, k > 0);
            load(upper, req);
        }
        multiply(lower);
        if (!OFF && wave == 0) taken += block.rows;
        block = req;
        blocks.next(a, range, step);
        req = blocks.ahead;
        __syncthreads();   // the upper half is there, everyone is done with the lower one
        if (parks) {
            park(lower, block, k + 1 < n);
            load(lower, req);
        }
        multiply(upper);
        __syncthreads();
    }
    if (!OFF && parks) unsafeAtomicAdd(&at.sums[int_place_quarter(place) * Sh::COLS + int_place_column(place)], sum);
    const bool stored = a.accumulate != 0 || done > 0;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        if (i >= NF && !more) break;
        double* o = here(out) + (wave + INT_WAVES * i) * 256 + lane;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double v = acc[i][0][r] + acc[i][1][r];
            o[r * 64] = stored ? o[r * 64] + v : v;
        }
    }
}

// Blocks go to the fp64 pipe when digits will not do for one with scales of its own, or new scales are asked for too often: that one,
// and while the ones behind it are no better eight times as many each time, up to 512.
template <int NT, bool BF16, bool OFF>
__device__ __forceinline__ void int_chunk(const MomArgs& a, unsigned char* lds, int pa, int pb, int chunk, int chunks, double* out)
{
    using Sh = IntShape<NT, OFF>;
    const int tid = threadIdx.x, b = blockIdx.y;
    const IntLds<NT, OFF> at(lds);
    const int64_t full = a.M / a.d;
    int64_t lo = a.offs[b], hi = a.offs[b + 1] < full ? a.offs[b + 1] : full;
    if (hi < lo) hi = lo;
    const int64_t cnt = hi - lo;
    IntRange range;
    range.j0 = lo + cnt * chunk / chunks;
    const int64_t j1 = lo + cnt * (chunk + 1) / chunks, tail = full - INT_NS - j1;
    range.n = (int)(j1 - range.j0);
    range.blocks = (range.n + INT_NS - 1) / INT_NS;
    range.tail = tail < (1 << 30) ? (int)tail : 1 << 30;
    if (tid < 32) at.flags[tid] = 0u;
    if (!OFF)
        for (int i = tid; i < 4 * Sh::COLS; i += INT_THREADS) at.sums[i] = 0.0;
    __syncthreads();
    const int total = range.blocks * a.L;
    unsigned int taken = 0u;   // samples, counted by the first wave
    for (int done = 0, spell = 1; done < total;) {
        const int before = done;
        done = int_waves<NT, BF16, OFF>(a, lds, pa, pb, range, done, spell > 1 ? 4 : 8, out, taken);
        if (done == total) break;
        if (done - before >= 32) spell = 1;
        const int n = spell < total - done ? spell : total - done;
        int_exactly<NT, BF16, OFF>(a, lds, pa, pb, range, done, n, out, taken);
        done += n;
        spell = spell < 512 ? 8 * spell : 512;
    }
    if (total == 0 && !a.accumulate)
        for (int i = tid; i < Sh::NPAIR * 256; i += INT_THREADS) out[i] = 0.0;
    if (OFF) return;
    __syncthreads();
    if (tid < Sh::COLS) {
        double v = 0.0;
        for (int o = 0; o < 4; ++o) v += at.sums[o * Sh::COLS + tid];
        double* p = out + Sh::NPAIR * 256 + tid;
        *p = a.accumulate ? *p + v : v;
    }
    if (tid == 0 && pa == 0 && taken) atomicAdd(a.nsamp + b, (unsigned long long)taken);
}

template <int NT, bool BF16, bool MULTI>
__global__ __launch_bounds__(INT_THREADS, 3) void moments_int_kernel(MomArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char int_lds[];
    using Diag = MomShape<NT, false>;
    double* part = a.part + (size_t)blockIdx.y * a.part_basis;
    int task = blockIdx.x;
    if constexpr (MULTI) {
        using Off = MomShape<NT, true>;
        const int npairs = a.np * (a.np - 1) / 2;
        if (task < npairs * a.chunks_off) {
            int chunk = task / npairs, q = task - chunk * npairs, pa = 0;
            if (chunk < (a.chunks_off & ~7)) {   // the pairs of one chunk on one XCD: they share its samples
                const int s = task >> 3;
                chunk = (s / npairs) * 8 + (task & 7);
                q = s % npairs;
            }
            double* out = part + (size_t)a.np * a.chunks_diag * Diag::PART + ((size_t)q * a.chunks_off + chunk) * Off::PART;
            while (q >= a.np - 1 - pa) { q -= a.np - 1 - pa; ++pa; }
            int_chunk<NT, BF16, true>(a, int_lds, pa, pa + 1 + q, chunk, a.chunks_off, out);
            return;
        }
        task -= npairs * a.chunks_off;
    }
    const int chunk = task / a.np, p = task - chunk * a.np;
    int_chunk<NT, BF16, false>(a, int_lds, p, p, chunk, a.chunks_diag, part + ((size_t)p * a.chunks_diag + chunk) * Diag::PART);
}

// ======================================================================================
template <typename F> static int by_int_tiles(int nt, F f)
{
    switch (nt) {
    case 5: return f(std::integral_constant<int, 5>{});
    case 6: return f(std::integral_constant<int, 6>{});
    case 7: return f(std::integral_constant<int, 7>{});
    default: return f(std::integral_constant<int, 8>{});
    }
}

// It reads 64 slices at a time, and counts a task's slices and blocks of 32 gradients in an int.
bool gvq_moments_int_shape(const gvq_basis* h) { return h->d > 64 && h->M / h->d >= INT_NS && h->M / h->d < 1 << 30; }

// From 16384 samples of the longest basis on.  Of 90 refreshes from there to a million samples a basis (65 to 1024 elements, both
// storages, 1 to 100 bases, normal numbers) none takes longer than with the fp64 pipe, by more than 0.2 %: up to 30 000
// samples 0.97 to 1.0 of its time, where the eigensolver takes most of it, down to 0.58 with 100 bases or 430 000 samples in
// bf16.  Below, there is little to gain.
bool gvq_moments_int_takes(const gvq_basis* h, int L)
{
    if (!gvq_moments_int_shape(h)) return false;
    int64_t longest = 0;
    for (int b = 0; b < h->B; ++b) longest = h->h_offs[b + 1] - h->h_offs[b] > longest ? h->h_offs[b + 1] - h->h_offs[b] : longest;
    return longest * L >= 16384;
}

// Sample chunks per task: as in gvq_moments_plan, with one work-group per compute unit and whole blocks of samples.  What a block
// takes, in units that balance the two kinds of task best: alone, panels with themselves take less of it (2740 cycles of 80 elements, 3300 of
// 96, where two panels take 4520 and 5990), but with these figures d = 250 takes 4.36 instead of 3.98 ms, d = 768 13.2 instead of 12.9.
size_t gvq_moments_int_plan(gvq_basis* h, int64_t longest)
{
    const int np = int_panels(h->d), poff = np * (np - 1) / 2;
    size_t basis = 0;
    by_int_tiles(int_tiles(h->d), [&](auto nt) {
        using Diag = MomShape<decltype(nt)::value, false>;
        using Off = MomShape<decltype(nt)::value, true>;
        const double slots = h->num_cu, start = 20000.0;
        auto task = [&](int cycles, int64_t chunks) {   // of about eight gradients
            return (double)cycles * 8.0 * (double)((longest + chunks * INT_NS - 1) / (chunks * INT_NS)) + start;
        };
        const int64_t most = (longest + INT_NS - 1) / INT_NS;
        double best = 0.0;
        const int cycles_d = 2100 + 75 * Diag::NPAIR, cycles_o = 2950 + 75 * Off::NPAIR;
        for (int64_t c = 1; c <= most && c <= (int64_t)(2.0 * slots); ++c) {
            // A panel with itself in as many chunks as make its tasks no longer than the others, or one fewer: 1,023 splits
            // looked at where all of c/2 .. c are 66,048 (d = 160, 312,500 samples), for the same estimate within 0.2 %.
            const int64_t even = poff ? (c * cycles_d + cycles_o - 1) / cycles_o : c;
            for (int64_t cd = poff && even > 1 ? even - 1 : even; cd <= even; ++cd) {
                const double td = task(cycles_d, cd), to = poff ? task(cycles_o, c) : 0.0;
                const double tasks = (double)h->B * (np * cd + (poff ? poff * c : 0));
                const double work = (double)h->B * (np * cd * td + (poff ? poff * c * to : 0.0));
                const double longest_task = td > to ? td : to;
                const double t = tasks <= slots ? longest_task : work / slots + 0.5 * longest_task;
                if (best == 0.0 || t < best) { best = t; h->mom_idiag = (int)cd; h->mom_ioff = poff ? (int)c : 0; }
            }
            if ((double)h->B * (np * (c + 1) / 2 + poff * c) > 8.0 * slots) break;   // past what could help; the partials take memory
        }
        basis = (size_t)np * h->mom_idiag * Diag::PART + (size_t)poff * h->mom_ioff * Off::PART;
        return GVQ_OK;
    });
    return basis;
}

int gvq_launch_moments_int(gvq_basis* h, const void* const* grads, int L, hipStream_t st)
{
    MomArgs a;
    a.offs = h->d_offs; a.M = h->M; a.d = h->d; a.np = int_panels(h->d); a.pw = 16 * int_tiles(h->d);
    a.chunks_diag = h->mom_idiag; a.chunks_off = h->mom_ioff;
    a.part = h->d_part; a.part_basis = h->mom_part; a.nsamp = h->d_nsamp;
    const int poff = a.np * (a.np - 1) / 2;
    return by_int_tiles(int_tiles(h->d), [&](auto nt) -> int {
        constexpr int NT = decltype(nt)::value;
        const dim3 grid((unsigned)(a.np * a.chunks_diag + poff * a.chunks_off), (unsigned)h->B);
        static gvq_once_per_device once[4];
        auto launch = [&](auto kern, int lds) -> int {
            const int ready = once[(h->dtype == GVQ_BF16 ? 1 : 0) + (a.np > 1 ? 2 : 0)].call(h->device, [&]() -> int {
                GVQ_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
                return GVQ_OK;
            });
            if (ready != GVQ_OK) return ready;
            for (int l0 = 0; l0 < L; l0 += GVQ_MAX_PTRS) {
                a.L = L - l0 < GVQ_MAX_PTRS ? L - l0 : GVQ_MAX_PTRS;
                for (int i = 0; i < a.L; ++i) a.grads.p[i] = grads[l0 + i];
                a.accumulate = l0 > 0;
                hipLaunchKernelGGL(kern, grid, dim3(INT_THREADS), lds, st, a);
                GVQ_HIP(hipGetLastError());
            }
            return GVQ_OK;
        };
        int rc = GVQ_EINVAL;
        const bool bf = h->dtype == GVQ_BF16;
        if (a.np > 1) {
            if constexpr (NT <= 6)
                rc = bf ? launch(moments_int_kernel<NT, true, true>, IntShape<NT, true>::LDS)
                        : launch(moments_int_kernel<NT, false, true>, IntShape<NT, true>::LDS);
        } else {
            rc = bf ? launch(moments_int_kernel<NT, true, false>, IntShape<NT, false>::LDS)
                    : launch(moments_int_kernel<NT, false, false>, IntShape<NT, false>::LDS);
        }
        if (rc != GVQ_OK) return rc;
        return gvq_launch_moments_reduce(h, NT, a.np, a.pw, a.chunks_diag, a.chunks_off, st);
    });
}
