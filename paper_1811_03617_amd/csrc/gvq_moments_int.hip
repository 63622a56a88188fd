// Moments of the basis refresh (GradiVeQ Section 2, PCA paragraph after Eq. 4) from many samples, slices longer than 64
// elements: sum x and sum x x^T as gvq_moments.hip gives them, with the products on the int8 matrix pipe
// (v_mfma_i32_16x16x64_i8, 4.2 to 4.4 PFLOP/s at the 2.0 to 2.1 GHz that this load leaves) instead of the fp64 one (77.5 TFLOP/s).
//
// A number becomes a whole number of 48 bits (bf16 storage: 40) in units of its column's scale and that a sum of six (five)
// digits in base 256, -128 to 127 each.  A product of two digits summed over up to 20480 samples is exact in int32; the
// products of two digits that count 2^-56 of the largest product and less are left out (INT_LEVELS), which is what float64 rounds
// away of a single sum of a few terms.  Scales have room for 2 to 4 times a column's largest number so far, so that an fp32
// number is exact if it is above 2^-23 of that room, one in 500 000 of a normal distribution's; a block with a number
// out of range, or with all of them below 2^-8 of it, gets new scales first.  Difference to long double sums over
// sqrt(C_aa C_bb), rms, fp64 pipe -> here: planted model, a million samples of 96 elements at 64 scales 1.2e-16 -> 3.6e-17,
// 200 000 of 100 1.0e-16 -> 3.2e-17, 78 000 of 256 6.6e-17 -> 2.9e-17, 100 000 of 80 3.1e-17 -> 3.7e-17 (what rounding the result leaves);
// 40 000 of 128, products of three normal numbers 1.2e-17 -> 2.0e-17, columns from 1 to 1e-8 1.6e-17 -> 2.0e-17.
//
// Digits come from float64: x * scale + 1.5 * 2^52 + 0x80..80 has them, plus 128 each, as its lower bytes (one conversion and one
// v_fma_f64; with fp32 arithmetic alone it took seven instructions a number and the kernel a sixth longer).  The last digit
// (bf16: the last two) is 0 in nearly every number: its products are made only for tiles of a block that have another one.
//
// What bounds it: instruction issue.  A wave issues a vector instruction every 5 cycles, every 7.8 while another wave of its SIMD
// has products in flight, and its own products do not overlap with its own vector instructions.  Hence twelve waves, three a
// SIMD, the most that have room for their share of the accumulators (seven levels a pair of tiles, 84 of 168 registers for
// three pairs), of which one parks the next block before its products, the others behind them.  A block of 64 samples
// of 128 elements takes 4820 cycles at 1.8 to 1.85 GHz, 3400 of them products (eight waves 5300, all of them parking between their products 6400);
// with the eigensolver 32 gradients of 138 M elements 10.1 -> 6.37 ms, 8 gradients of
// d = 768 16.9 -> 12.6 ms.
#include <math.h>

#include "gvq_moments.h"
#include "gvq_moments_place.h"

typedef int i4 __attribute__((ext_vector_type(4)));

#define INT_THREADS 768
#define INT_WAVES 12
#define INT_SLOTS 2
#define INT_LEVELS 7
#define INT_FLUSH 320                // blocks between flushes: 6 products of 2^14 a sample stay below 2^31 for 21845 samples

static_assert(INT_MOST_D >= GVQ_MAX_D, "columns past a slice's end");

template <int NT, bool OFF, int ND> struct IntShape {
    using Mom = MomShape<NT, OFF>;
    static constexpr int TILES = Mom::TILES, NPAIR = Mom::NPAIR, COLS = 16 * TILES;
    // The threads of this wave park an item each: 16 samples of one column.
    static_assert(COLS * 4 <= INT_THREADS, "an item per thread");
    static constexpr bool parks(int w) { return 64 * w < COLS * 4; }
    static constexpr int PLANE = TILES * 1024, BUF = ND * PLANE;               // bytes: one digit, one block
    static constexpr int LDS = 2 * BUF + 8 * COLS + 2 * 16 * 4 + (OFF ? 0 : 64 * COLS);
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
    static constexpr int first(int w)
    {
        int p = 0;
        for (int i = 0; i < w; ++i) p += NPAIR / INT_WAVES + extra(i);
        return p;
    }
    static constexpr int row(int i) { return Mom::row(order.p[i]); }
    static constexpr int col(int i) { return Mom::col(order.p[i]); }
    // Which tiles a wave's three sets of operand registers hold when pair i is multiplied (phase 1: once its own tiles are
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

// Four samples of one column -> four bytes (one dword) per digit.  Bytes 0 to 3 of lo hold digits ND - 1 to ND - 4, the lowest
// bytes of hi the others, all biased by 128, which the exclusive or turns into two's complement.
template <int ND> __device__ __forceinline__ void pack_digits(const unsigned int (&hi)[4], const unsigned int (&lo)[4], unsigned int (&out)[ND])
{
    const auto perm = [](unsigned int high, unsigned int low, unsigned int sel) { return __builtin_amdgcn_perm(high, low, sel); };
    const unsigned int p = perm(lo[1], lo[0], 0x05010400u), q = perm(lo[3], lo[2], 0x05010400u);
    const unsigned int r = perm(lo[1], lo[0], 0x07030602u), s = perm(lo[3], lo[2], 0x07030602u);
    out[ND - 1] = perm(q, p, 0x05040100u) ^ 0x80808080u;
    out[ND - 2] = perm(q, p, 0x07060302u) ^ 0x80808080u;
    out[ND - 3] = perm(s, r, 0x05040100u) ^ 0x80808080u;
    out[ND - 4] = perm(s, r, 0x07060302u) ^ 0x80808080u;
    if constexpr (ND == 6) {
        const unsigned int t = perm(hi[1], hi[0], 0x05010400u), u = perm(hi[3], hi[2], 0x05010400u);
        out[1] = perm(u, t, 0x05040100u) ^ 0x80808080u;
        out[0] = perm(u, t, 0x07060302u) ^ 0x80808080u;
    } else {
        out[0] = (perm(hi[1], hi[0], 0x0c0c0400u) | perm(hi[3], hi[2], 0x04000c0cu)) ^ 0x80808080u;
    }
}

template <int NT, bool BF16, bool OFF, int ND, int WAVE>
__device__ __forceinline__ void int_task(const MomArgs& a, unsigned char* lds, int pa, int pb, int chunk, int chunks, double* out)
{
    using Sh = IntShape<NT, OFF, ND>;
    constexpr int P0 = Sh::first(WAVE), NA = Sh::first(WAVE + 1) - P0;
    constexpr int NB = BF16 ? 3 : 5;   // digits of every number; the others are nearly always zero
    constexpr int ES = BF16 ? 2 : 4, COLS = Sh::COLS, BITS = 8 * ND;
    constexpr bool PARKS = Sh::parks(WAVE);
    const int tid = threadIdx.x, lane = tid & 63;
    const int b = blockIdx.y, d = a.d;
    unsigned int* const colmax = (unsigned int*)(lds + 2 * Sh::BUF);
    int* const cexp = (int*)(colmax + COLS);                    // x 2^cexp is what the digits hold
    // [2][waves]: 1 a number is out of its column's range, 2 one is not small, 4 one is not 0; from bit 4 on, the tiles whose
    // last digits are not all zero
    unsigned int* const flags = (unsigned int*)(cexp + COLS);
    double* const sums = (double*)(flags + 32);   // [4][COLS] of x; then of x over the block that is parked

    const int64_t full = a.M / d;
    int64_t lo = a.offs[b], hi = a.offs[b + 1] < full ? a.offs[b + 1] : full;
    if (hi < lo) hi = lo;
    const int64_t cnt = hi - lo;
    const int64_t j0 = lo + cnt * chunk / chunks, j1 = lo + cnt * (chunk + 1) / chunks;
    const int64_t nblk = (j1 - j0 + INT_NS - 1) / INT_NS;

    unsigned int place = 0u;   // this thread's item
    if constexpr (PARKS) {
        const int c = tid % COLS, q = tid / COLS;
        const int e = OFF && c >= 16 * NT ? pb * a.pw + c - 16 * NT : pa * a.pw + c;
        place = int_place(int_from(e, q, d, ES), c, q);
    }
    auto col_of = [](unsigned int p) { return int_place_column(p); };
    auto quarter_of = [](unsigned int p) { return int_place_quarter(p); };
    // Hides a value's origin, so that what is made from it is not kept in registers from one block to the next.
    auto fresh = [](auto v) { asm("" : "+v"(v)); return v; };

    float x[16];
    int64_t left = nblk * a.L;   // blocks not yet requested
    // A block: 64 slices from src on, of which only those from `skip` on and no more than `rows` count.  One that ends a task's
    // samples, or lies at the gradient's end, is read with its neighbours, so that every load is whole.
    struct Block { uintptr_t src; int skip, rows; } ahead{0, 0, 0};   // the one to request next
    const int step = d * ES, stride = INT_NS * step;
    int64_t rows_left = 0;   // this task's samples of the gradient from that block on
    int l = 0;
    unsigned long long taken = 0;
    auto next_block = [&]() {
        if (left == 0) return;   // the last block is requested again: loads stay unconditional
        --left;
        rows_left -= INT_NS;
        ahead.src += stride;
        if (rows_left < INT_NS) {
            if (rows_left <= 0) {
                ahead.src = (uintptr_t)a.grads.p[l++] + j0 * step;
                rows_left = j1 - j0;
            }
            ahead.rows = rows_left < INT_NS ? (int)rows_left : INT_NS;
            const int64_t past = j1 - rows_left - (full - INT_NS);   // slices that the block's 64 would reach past the last
            ahead.skip = past > 0 ? (int)past : 0;
            ahead.src -= ahead.skip * step;
        }
    };
    // Loads through a buffer resource: the rows' distances are uniform offsets, which a lane's address would have to add up.
    int row_at[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) row_at[i] = __builtin_amdgcn_readfirstlane(i * step);
    auto load_quad = [&](int q, const Block& k) {
        auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)k.src, 0, stride, 0x00027000);
        const unsigned int at = int_place_from(fresh(place)) + (q >= 2 ? 8u * step : 0u);
#pragma unroll
        for (int i = 4 * q; i < 4 * q + 4; ++i) {
            if (BF16) x[i] = __uint_as_float((unsigned int)__builtin_amdgcn_raw_buffer_load_b16(rsrc, at, row_at[i & 7], 0) << 16);
            else x[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, at, row_at[i & 7], OFF ? 0 : 2));
        }
    };
    auto load = [&](const Block& k) {
#pragma unroll
        for (int q = 0; q < 4; ++q) load_quad(q, k);
    };

    int by = 0;                // x * 2^by is the whole number that the digits hold, for numbers below 2^(BITS - 1 - by)
    unsigned int marks = 0u;   // of the block just parked, see flags
    auto sum_at = [&]() {
        const unsigned int p = fresh(place);
        return quarter_of(p) * COLS + col_of(p);
    };
    auto mask = [&](const Block& k) {   // samples that do not count become zeros
        if (k.rows < INT_NS) {
            const int r = 16 * quarter_of(fresh(place)) - k.skip;
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = (unsigned int)(r + i) < (unsigned int)k.rows ? x[i] : 0.f;
        }
    };
    // `then(q)` follows the last use of four samples' registers.
    auto park = [&](unsigned char* buf, auto then) {
        // 1.5 * 2^52 makes the sum's unit 1: its lower bits are the whole number, biased so that every byte is a digit + 128
        constexpr double BIAS = 0x1.8p52 + (ND == 6 ? 0x808080808080p0 : 0x8080808080p0);
        const double scale = __builtin_bit_cast(double, (unsigned long long)(1023 + fresh(by)) << 52);
        double sum[2] = {0.0, 0.0};
        float most = 0.f;
        unsigned int last = 0u;
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
            pack_digits<ND>(hi, lo, dig);
#pragma unroll
            for (int g = 0; g < ND; ++g) {
                out4[g][q] = (int)dig[g];
                if (g >= NB) last |= dig[g];
            }
            then(q);
        }
        unsigned char* o = buf + int_place_lds(fresh(place));
#pragma unroll
        for (int g = 0; g < ND; ++g) *(i4*)(o + g * Sh::PLANE) = out4[g];
        const float limit = ldexpf(0.98f, BITS - 1 - fresh(by));   // 0x7f7f.. of 0x8000..: every byte's digit is at most 127
        marks = (__any(!(most < limit)) ? 1u : 0u) | (__any(most > limit * 0x1p-8f) ? 2u : 0u) | (__any(most > 0.f) ? 4u : 0u);
        // a wave has four tiles' columns, side by side or around the end
        const unsigned long long some = __ballot(last != 0u);
        if (some != 0ull) {
            const unsigned int tiles = (some & 0xffffull ? 1u : 0u) | (some & 0xffff0000ull ? 2u : 0u)
                                       | (some & 0xffff00000000ull ? 4u : 0u) | (some & 0xffff000000000000ull ? 8u : 0u);
            const unsigned int at_tile = tiles << 64 * WAVE % COLS / 16;
            marks |= ((at_tile | at_tile >> Sh::TILES) & ((1u << Sh::TILES) - 1u)) << 4;
        }
        if (!OFF) sums[4 * COLS + sum_at()] = sum[0] + sum[1];
    };

    bool stored = a.accumulate != 0;   // the partials hold something to add to
    // accumulators and sums -> float64
    auto flush = [&](i4 (&acc)[NA > 0 ? NA : 1][INT_LEVELS]) {
        static_for<NA>([&](auto ii) {
            constexpr int I = decltype(ii)::value, R = Sh::row(P0 + I), C = Sh::col(P0 + I), P = Sh::order.p[P0 + I];
            double* o = out + P * 256 + (lane >> 4) * 64 + (lane & 15);
            const int ec = cexp[16 * C + (lane & 15)];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int er = cexp[16 * R + 4 * (lane >> 4) + r];
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
        if (PARKS && self == 0) flags[parity * 16 + WAVE] = marks;
        __syncthreads();
        found = flags[parity * 16 + (self & 15)];
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
    // New scales, for the columns' largest numbers since `forget` and in block k, which is then parked with them.
    auto refresh = [&](const Block& k, bool forget, unsigned char* buf) {
        if (forget)
            for (int i = tid; i < COLS; i += INT_THREADS) colmax[i] = 0u;
        __syncthreads();   // (also: all flushes have read cexp)
        const unsigned int p = fresh(place);
        if constexpr (PARKS) {
            load(k);
            mask(k);
            float most = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) most = __builtin_fmaxf(most, __builtin_fabsf(x[i]));
            most = __builtin_fminf(most, 3.4028235e38f);
            atomicMax(&colmax[col_of(p)], __float_as_uint(most));
        }
        __syncthreads();
        if constexpr (PARKS) {
            // room for 2 to 4 times the column's largest number; a column of zeros has none, so that its first other number
            // asks for new scales
            const unsigned int m = colmax[col_of(p)];
            const double f = (double)__uint_as_float(m ? m : 1u);
            by = BITS - 1 - ((int)(__builtin_bit_cast(unsigned long long, f) >> 52) - 1023 + 2);
            if (quarter_of(p) == 0) cexp[col_of(p)] = by;
            park(buf, [](int) {});
        }
        exchange();
    };

    if (tid < 32) flags[tid] = 0u;
    if (!OFF)
        for (int i = tid; i < 4 * COLS; i += INT_THREADS) sums[i] = 0.0;
    const unsigned char* mine = lds + lane * 16;
    int64_t todo = left;
    int flip = 0;
    next_block();
    Block parked_block = ahead;   // in LDS
    next_block();
    Block req = ahead;            // in registers, or on its way
    next_block();
    bool forget = true;   // the columns' largest numbers so far
    while (todo > 0) {
        // blocks until the scales no longer fit, or the accumulators might overflow; the first, which the last round has
        // parked with the scales it had, is parked again
        refresh(parked_block, forget, lds + flip * Sh::BUF);
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
            // The two waves of a SIMD park at different times, one of them before its products and one behind: while one
            // converts the other has the matrix pipe.
            constexpr bool EARLY = WAVE < 4;
            if constexpr (!EARLY && NA > 0) fetch_for(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
            __builtin_amdgcn_sched_barrier(0);
            const unsigned int known = findings(), rare = known >> 4;
            forget = (known & 6u) == 4u;
            if (since > INT_FLUSH || (known & 1u) || forget) {
                if (since > 1) break;   // with the scales just made all is well, or cannot be helped
            }
            if (!OFF && WAVE == 0) taken += parked_block.rows;
            parked_block = req;
            req = ahead;
            auto park_next = [&]() {
                if constexpr (PARKS) {
                    double sum = 0.0;
                    if (!OFF) sum = sums[4 * COLS + sum_at()];   // of the block that was parked last
                    mask(parked_block);
                    // the next block as soon as registers are free; the late waves of a panel with itself have none to spare
                    park(next, [&](int q) { if (OFF || EARLY) load_quad(q, req); });
                    if (!OFF && !EARLY) load(req);
                    if (!OFF) unsafeAtomicAdd(&sums[sum_at()], sum);
                }
            };
            if constexpr (EARLY) {
                park_next();
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (NA > 0) fetch_for(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
            }
            // Two panels: who parks behind its products goes first (6060 -> 5660 cycles a block).  A panel with itself has waves
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
                auto multiply = [&](int i, int j) {
                    if (i + j < INT_LEVELS)
                        acc[I][i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(op[A][i], op[B][j], acc[I][i + j], 0, 0, 0);
                };
#pragma unroll
                for (int top = 0; top < NB; ++top) {   // in the order in which digits arrive
#pragma unroll
                    for (int i = 0; i < top; ++i) multiply(top, i);
#pragma unroll
                    for (int i = 0; i <= top; ++i) multiply(i, top);
                }
                if constexpr (PARKS && !EARLY && I == 0) next_block();   // scalar work, between products
                if ((rare >> R | rare >> C) & 1u) {
#pragma unroll
                    for (int g = NB; g < ND; ++g) {
                        const i4 a_last = fetch_digit(g, R), b_last = fetch_digit(g, C);
#pragma unroll
                        for (int i = 0; i < NB; ++i)
                            if (i + g < INT_LEVELS) {
                                acc[I][i + g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a_last, op[B][i], acc[I][i + g], 0, 0, 0);
                                acc[I][i + g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(op[A][i], b_last, acc[I][i + g], 0, 0, 0);
                            }
                        if (2 * g < INT_LEVELS) acc[I][2 * g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a_last, b_last, acc[I][2 * g], 0, 0, 0);
                    }
                }
            });
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (PRIORITY > 0) __builtin_amdgcn_s_setprio(0);
            if constexpr (!EARLY) park_next();
            --todo;
            if (todo == 0) break;
            if constexpr (EARLY) next_block();
            exchange();   // also: everyone is done with this block's buffer
        }
        flush(acc);
    }
    if (!stored) {
        static_for<NA>([&](auto ii) {
            constexpr int P = Sh::order.p[P0 + decltype(ii)::value];
#pragma unroll
            for (int r = 0; r < 4; ++r) out[P * 256 + r * 64 + lane] = 0.0;
        });
    }
    if (OFF) return;
    __syncthreads();
    if (tid < COLS) {
        double v = 0.0;
        for (int o = 0; o < 4; ++o) v += sums[o * COLS + tid];
        double* p = out + Sh::NPAIR * 256 + tid;
        *p = a.accumulate ? *p + v : v;
    }
    if (tid == 0 && pa == 0 && taken) atomicAdd(a.nsamp + b, taken);
}

template <int NT, bool BF16, bool OFF, int ND>
__device__ __forceinline__ void int_waves(const MomArgs& a, unsigned char* lds, int pa, int pb, int chunk, int chunks, double* out)
{
    switch (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {   // uniform: the cases hold barriers
    case 0: int_task<NT, BF16, OFF, ND, 0>(a, lds, pa, pb, chunk, chunks, out); break;
    case 1: int_task<NT, BF16, OFF, ND, 1>(a, lds, pa, pb, chunk, chunks, out); break;
    case 2: int_task<NT, BF16, OFF, ND, 2>(a, lds, pa, pb, chunk, chunks, out); break;
    case 3: int_task<NT, BF16, OFF, ND, 3>(a, lds, pa, pb, chunk, chunks, out); break;
    case 4: int_task<NT, BF16, OFF, ND, 4>(a, lds, pa, pb, chunk, chunks, out); break;
    case 5: int_task<NT, BF16, OFF, ND, 5>(a, lds, pa, pb, chunk, chunks, out); break;
    case 6: int_task<NT, BF16, OFF, ND, 6>(a, lds, pa, pb, chunk, chunks, out); break;
    case 7: int_task<NT, BF16, OFF, ND, 7>(a, lds, pa, pb, chunk, chunks, out); break;
    case 8: int_task<NT, BF16, OFF, ND, 8>(a, lds, pa, pb, chunk, chunks, out); break;
    case 9: int_task<NT, BF16, OFF, ND, 9>(a, lds, pa, pb, chunk, chunks, out); break;
    case 10: int_task<NT, BF16, OFF, ND, 10>(a, lds, pa, pb, chunk, chunks, out); break;
    default: int_task<NT, BF16, OFF, ND, 11>(a, lds, pa, pb, chunk, chunks, out); break;
    }
}

template <int NT, bool BF16, bool MULTI>
__global__ __launch_bounds__(INT_THREADS, 3) void moments_int_kernel(MomArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char int_lds[];
    constexpr int ND = BF16 ? 5 : 6;
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
            int_waves<NT, BF16, true, ND>(a, int_lds, pa, pa + 1 + q, chunk, a.chunks_off, out);
            return;
        }
        task -= npairs * a.chunks_off;
    }
    const int chunk = task / a.np, p = task - chunk * a.np;
    int_waves<NT, BF16, false, ND>(a, int_lds, p, p, chunk, a.chunks_diag, part + ((size_t)p * a.chunks_diag + chunk) * Diag::PART);
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

bool gvq_moments_int_shape(const gvq_basis* h) { return h->d > 64 && h->M / h->d >= INT_NS; }   // it reads 64 slices at a time

// From 16384 samples of the longest basis on.  Of 70 refreshes from 2000 to a million samples a basis (65 to 1024 elements,
// both storages, 1 to 100 bases) none is more than 1 % slower than with the fp64 pipe; from 16384 to 100 000 samples they
// take 0.96 of its time where the eigensolver takes most of it and down to 0.56 with 100 bases, from 100 000 on 0.49 to
// 0.97.  Below, there is little to gain and fewer samples over which the products left out average.
bool gvq_moments_int_takes(const gvq_basis* h, int L)
{
    if (!gvq_moments_int_shape(h)) return false;
    int64_t longest = 0;
    for (int b = 0; b < h->B; ++b) longest = h->h_offs[b + 1] - h->h_offs[b] > longest ? h->h_offs[b + 1] - h->h_offs[b] : longest;
    return longest * L >= 16384;
}

// Sample chunks per task: as in gvq_moments_plan, with one work-group per compute unit and whole blocks of samples.  Cycles a
// block measured: 4820 (36 pairs of tiles) and 3570 (21) for a panel with itself, 5660 (36) for two panels.
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
                rc = bf ? launch(moments_int_kernel<NT, true, true>, IntShape<NT, true, 5>::LDS)
                        : launch(moments_int_kernel<NT, false, true>, IntShape<NT, true, 6>::LDS);
        } else {
            rc = bf ? launch(moments_int_kernel<NT, true, false>, IntShape<NT, false, 5>::LDS)
                    : launch(moments_int_kernel<NT, false, false>, IntShape<NT, false, 6>::LDS);
        }
        if (rc != GVQ_OK) return rc;
        return gvq_launch_moments_reduce(h, NT, a.np, a.pw, a.chunks_diag, a.chunks_off, st);
    });
}
