// Eqs. (2) and (4) for the slice lengths and numbers of comps that the register-resident and the basis-stationary kernels
// do not take: lengths from 4 to 512, any number of bases, up to 128 comps; decompress up to 640, up to 896 with 96 comps
// and up to 1024 with 64, as the registers have room for U (gvq_flow_plan.h, which also says where others are faster).
//
// Bound: memory.  What kept the LDS-tiled kernels (gvq_codec_long.hip) at 1.4 - 3.6 TB/s on these shapes was how they
// touched it: lanes walked down 16 slices 64 bytes at a time, and a slice length that is no multiple of 4 (three lengths out
// of four) went number by number.  48 M elements, compress / decompress in us, there -> here: d = 13, k = 3 167 / 190 ->
// 70 / 87; d = 63, k = 16 124 / 112 -> 48 / 59; d = 100, k = 25 74 / 70 -> 46 / 49 (5.2 TB/s); d = 201, k = 67 129 / 140 ->
// 65 / 67; bf16 d = 401, k = 60 182 / 91 -> 50 / 48.  Short of memory (bf16 storage, eight waves) it is the chain of a
// tile's phases: words -> LDS, barrier, products, barrier, results.
//
// A tile is a run of whole slices, moved in words of four numbers in memory order: global_load_dwordx4 takes any 4-byte
// address, and the last word of a slice that is no whole number of words is simply its last four numbers, whose repeated
// entries meet zeros in the packed copy of U.  U stays in registers, shared out over the waves of a work-group by comps
// (compress) or by elements (decompress); results leave through LDS as one run.
//
//   compress    x (registers, a tile ahead) -> x - mu/N, split in two bf16 terms once per number -> LDS -> products -> LDS -> y
//   decompress  y (registers, a tile ahead) -> two bf16 terms -> LDS -> products, + mu -> LDS -> x
//
// Two barriers a tile; two work-groups of four waves per compute unit (or one of eight where U needs the registers) keep
// memory busy across them.  Products as in the LDS-tiled kernels: fp32 on v_mfma_f32_16x16x4_f32 (EXACT) below 10 flop/B,
// else x1 u1 + x1 u2 + x2 u1 of two-term bf16 splits on v_mfma_f32_16x16x32_bf16, fp32 accumulation.
#pragma once
#include "gvq_device.h"
#include "gvq_flow_plan.h"

// a word of four numbers at any address
typedef float fw4 __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned short hw4 __attribute__((ext_vector_type(4), aligned(2)));
typedef unsigned int hu4 __attribute__((ext_vector_type(4), aligned(2)));

// A tile of a handle with several bases: `rows` slices of basis b from `first` on.
struct FlowTile {
    int64_t first;
    int rows, b;
};

struct FlowArgs {
    const void* in;
    void* out;
    const float* acc_in;     // compress only, may be null: added to the result
    const u4* Upack;
    const float* mu;         // [B][d]
    const FlowTile* tiles;   // the handle's tiles (B > 1 only)
    int64_t M, S, seg_begin, seg_end, t0, t1;
    int64_t whole;           // rows of the input that can be read word by word: whole ones, of at least four numbers
    int B, d, k;
    int words;               // words of a row of the input: ceil(d/4) (compress) or ceil(k/4) (decompress)
    unsigned int by_words, by_out;   // flow_divide by that, and by the words of a padded row of the result
    int rows;                // slices per tile
    int wn;                  // waves that share out the comps (compress) or the elements; the rest share out the slices
    int run;                 // consecutive tiles a work-group takes before it jumps ahead by the width of the grid
    int out_bf16, keep;      // decompress: storage of the result; compress: ordinary instead of non-temporal stores
    size_t upack_stride;     // words from one basis to the next
    float n_workers;
};

// The tiles of one work-group: runs of a.run consecutive ones, runs interleaved across the grid.  With several bases a tile
// comes out of a table that the host made: one scalar load, asked for a tile ahead.  (Found by searching the bases' offsets
// for every tile it cost 10 - 30 % with 24 bases; walking from one basis to the next, which a work-group with few tiles of
// thousands of short bases does hundreds of times between two of its tiles, a millisecond: 24 M elements in 16216 bases,
// d = 40, k = 10 968 us, now 88.)  With one basis none of that is touched: the next tile's number carried along for both
// kinds, and the products of a tile bounded by its own rows there too, cost decompress up to 4 % (48 M elements, d = 13, k = 3
// 89.8 -> 87.0 us; d = 24, k = 6 72.7 -> 69.7; d = 127, k = 32 55.3 -> 53.9; d = 201, k = 50 52.9 -> 51.6).
struct FlowIter {
    int64_t tile;
    int pos;               // of `tile` in its run
    FlowTile rec, next;    // B > 1: the entries of this tile and of the one after it (past the last one: this one's again)
    static __device__ __forceinline__ FlowTile entry(const FlowArgs& a, int64_t i)
    {
        return __builtin_bit_cast(FlowTile, uniform_load((const u4*)(a.tiles + i)));
    }
    __device__ __forceinline__ void prefetch(const FlowArgs& a)
    {
        int64_t i = tile + 1;
        if (pos + 1 == a.run) i += (int64_t)(gridDim.x - 1) * a.run;
        next = entry(a, i < a.t1 ? i : tile);
    }
    __device__ __forceinline__ FlowIter(const FlowArgs& a)
    {
        tile = a.t0 + (int64_t)blockIdx.x * a.run;
        pos = 0;
        if (a.B > 1 && tile < a.t1) {
            rec = entry(a, tile);
            prefetch(a);
        }
    }
    // To the next tile; false: none is left.
    __device__ __forceinline__ bool advance(const FlowArgs& a)
    {
        ++tile;
        if (++pos == a.run) {
            pos = 0;
            tile += (int64_t)(gridDim.x - 1) * a.run;
        }
        if (tile >= a.t1) return false;
        if (a.B > 1) {
            rec = next;
            prefetch(a);
        }
        return true;
    }
    // What of it lies in the requested range.
    __device__ __forceinline__ FlowTile get(const FlowArgs& a) const
    {
        FlowTile t;
        t.b = 0;
        t.first = a.seg_begin + tile * a.rows;
        int64_t end = t.first + a.rows;
        if (a.B > 1) {
            t.b = rec.b;
            t.first = rec.first;
            end = rec.first + rec.rows;
        }
        if (t.first < a.seg_begin) t.first = a.seg_begin;
        if (end > a.seg_end) end = a.seg_end;
        t.rows = (int)(end - t.first);
        return t;
    }
};

// i / n for i < 4096, n < 4096 and by = flow_divisor(n): one instruction.  (A division by a number that is not a constant
// takes about 40 instructions, and a thread starts with a dozen of them.  0.5 M elements, d = 12, k = 3: compress 8.0 -> 7.6 us,
// decompress 7.2 -> 6.7.)
__device__ __forceinline__ int flow_divide(int i, unsigned int by) { return (int)__umulhi(2u * (unsigned int)i, by); }

// Four numbers -> their two bf16 terms.
__device__ __forceinline__ void split4(const f4& v, u2& hi, u2& lo)
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const unsigned int h = pack_bf16x2(v[2 * i], v[2 * i + 1]);
        hi[i] = h;
        lo[i] = pack_bf16x2(v[2 * i] - __uint_as_float(h << 16), v[2 * i + 1] - __uint_as_float(h & 0xffff0000u));
    }
}

// A tile's results as one run of words of V numbers (V divides a padded row's length): f(word, its numbers in LDS).
template <int V, int NTHR>
struct FlowRun {
    int row0, col0, dr, dc, words;
    bool padded;
    __device__ __forceinline__ FlowRun(int len, unsigned int by)
    {
        padded = flow_out_row(len) != len;
        words = padded ? len / V : 1;
        row0 = flow_divide((int)threadIdx.x, by); col0 = (int)threadIdx.x - row0 * words;
        dr = flow_divide(NTHR, by); dc = NTHR - dr * words;
    }
    template <typename F> __device__ __forceinline__ void each(const float* lds, int len, int total, F f) const
    {
        if (!padded) {
            for (int j = threadIdx.x; j < total / V; j += NTHR) f(j, lds + V * j);
            return;
        }
        int row = row0, col = col0;
        for (int j = threadIdx.x; j < total / V; j += NTHR) {
            f(j, lds + row * (len + 4) + V * col);
            row += dr;
            col += dc;
            if (col >= words) { col -= words; ++row; }
        }
    }
    // number i of the run
    __device__ __forceinline__ const float* number(const float* lds, int len, int i) const
    {
        return padded ? lds + i / len * (len + 4) + i % len : lds + i;
    }
};

// The input side of both kernels: the words of a tile of `rows` rows of `len` numbers, NTHR threads, at most U words each.
// Word (row, c) holds the numbers from min(4 c, len - 4) on.
template <int U, int NTHR, bool BF16>
struct FlowInput {
    static constexpr int ES = BF16 ? 2 : 4;
    typedef typename std::conditional<BF16, hw4, fw4>::type word;
    word raw[U];
    unsigned int off[U], rc[U];   // byte offset in the tile; row << 16 | c
    __device__ __forceinline__ void init(const FlowArgs& a, int len)
    {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int i = threadIdx.x + NTHR * u;
            if (i >= a.rows * a.words) i = a.rows * a.words - 1;   // a word twice does no harm
            const int row = flow_divide(i, a.by_words), c = i - row * a.words, e = 4 * c < len - 4 ? 4 * c : len < 4 ? 0 : len - 4;
            off[u] = (unsigned int)((row * len + e) * ES);
            rc[u] = (unsigned int)(row << 16 | c);
        }
    }
    // Word u of a plain tile; of any other nothing that is used (the load itself stays unconditional): load_rest follows.
    __device__ __forceinline__ void load(const FlowArgs& a, const FlowTile& t, int len, bool plain_tile, int u)
    {
        const char* src = plain_tile ? (const char*)a.in + t.first * len * ES : (const char*)a.Upack;
        unsigned int o = off[u];
        if (t.rows < a.rows || !plain_tile) {
            const int row = (int)(rc[u] >> 16);
            if (row >= t.rows) o -= (unsigned int)(row * len * ES);   // a row that is not there: the first one's word
            if (!plain_tile) o = 0;
        }
        raw[u] = __builtin_nontemporal_load((const word*)(src + o));
    }
    // The words of a tile that is not plain, number by number; zeros past a short row and past the input (`total` numbers).
    __device__ __forceinline__ void load_rest(const FlowArgs& a, const FlowTile& t, int len, int64_t total)
    {
        typedef typename std::conditional<BF16, unsigned short, float>::type num;
        const num* src = (const num*)a.in + t.first * len;
        const int valid = len < 4 ? len : 4;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = (int)(rc[u] >> 16);
            const int64_t e = off[u] / ES;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                num v = 0;
                if (row < t.rows && i < valid && t.first * len + e + i < total) v = src[e + i];
                raw[u][i] = v;
            }
        }
        drain_memory();
    }
    // Zeros in the place of the numbers that the last word of a row repeats.  They meet zeros of U, which is enough but
    // for an infinity; the split turns those into NaN anyway.
    static __device__ __forceinline__ void drop_repeats(const FlowArgs& a, int len, int c, f4& v)
    {
        if ((len & 3) == 0 || len < 4) return;
        const int n = c == a.words - 1 ? 4 * a.words - len : 0;
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = i < n ? 0.f : v[i];
    }
    __device__ __forceinline__ f4 value(int u) const
    {
        f4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (BF16) v[i] = __uint_as_float((unsigned int)raw[u][i] << 16);
            else v[i] = raw[u][i];
        }
        return v;
    }
};

// --------------------------------------------------------------------------------------
// compress.  Wave (wn, ws): comp tiles wn NTW .. + NTW - 1 of slice groups ws, ws + W/wn, ...  Step st of 32 numbers:
//   EXACT  word i: A lane (m, kk) U[32 st + 16 i + 4 kk + j][16 nt + m], B lane (n, kk) x[n][same], j = 0..3, one product each
//   split  A lane (m, kk) U[32 st + 8 kk + j][16 nt + m], j = 0..7, B likewise
// Upack[b][nt][st][2: word i or term][64 lanes].  Result register r of lane (n, kk): comp 16 nt + 4 kk + r of slice n.
// LDS: x, mu/N [4 words], y [rows][k].
// --------------------------------------------------------------------------------------
template <int NTW, int STEPS, bool BF16, bool EXACT, int W>
__global__ __launch_bounds__(64 * W, 8 / W) void compress_flow_kernel(FlowArgs a)
{
    constexpr int NTHR = 64 * W, U = flow_words(W), RB = flow_row(STEPS);
    extern __shared__ f4 smem[];
    char* xs = (char*)smem;
    float* mus = (float*)(xs + a.rows * RB);
    float* ys = mus + 4 * a.words;
    const int tid = threadIdx.x, lane = tid & 63, n_ = lane & 15, kk = lane >> 4, d = a.d, k = a.k;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wn = wave % a.wn, ws = wave / a.wn, WS = W / a.wn;

    for (int i = tid; i < a.rows * RB / 16; i += NTHR) smem[i] = f4{0.f, 0.f, 0.f, 0.f};   // past a row's words: zeros
    FlowInput<U, NTHR, BF16> in;
    in.init(a, d);

    FlowIter it(a);
    if (it.tile >= a.t1) return;
    FlowTile t = it.get(a), before = t;
    bool plain = t.first + t.rows <= a.whole;
#pragma unroll
    for (int u = 0; u < U; ++u)
        in.load(a, t, d, plain, u);
    if (!plain) in.load_rest(a, t, d, a.M);

    u4 us[NTW][STEPS][2];
    int cur = -1;
    auto store_y = [&](const FlowTile& q) {
        // the tile's y is one run
        const int total = q.rows * k;
        float* Y = (float*)a.out + q.first * k;
        const float* prev = a.acc_in ? a.acc_in + q.first * k : nullptr;
        if (prev) {
            for (int j = tid; j < total / 4; j += NTHR)
                __builtin_nontemporal_store((fw4)(*(const f4*)(ys + 4 * j) + (f4)*(const fw4*)(prev + 4 * j)), (fw4*)(Y + 4 * j));
        } else if (a.keep) {
            for (int j = tid; j < total / 4; j += NTHR) *(fw4*)(Y + 4 * j) = (fw4)*(const f4*)(ys + 4 * j);
        } else {
            for (int j = tid; j < total / 4; j += NTHR) __builtin_nontemporal_store((fw4)*(const f4*)(ys + 4 * j), (fw4*)(Y + 4 * j));
        }
        const int j = (total & ~3) + tid;
        if (j < total) Y[j] = prev ? ys[j] + prev[j] : ys[j];
    };

    for (bool first = true;; first = false) {
        if (t.b != cur) {
            cur = t.b;
            const u4* Ub = a.Upack + (size_t)cur * a.upack_stride + (size_t)wn * NTW * STEPS * 128 + lane;
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
                for (int st = 0; st < STEPS; ++st)
#pragma unroll
                    for (int p = 0; p < 2; ++p) us[nt][st][p] = Ub[((nt * STEPS + st) * 2 + p) * 64];
            for (int e = tid; e < 4 * a.words; e += NTHR) {
                const int at = e < 4 * (a.words - 1) ? e : d - 4 + (e & 3);
                mus[e] = a.mu[(size_t)cur * d + at] / a.n_workers;
            }
            drain_memory();
            __syncthreads();
        }
        const bool more = it.advance(a);
        const FlowTile tn = more ? it.get(a) : t;   // this one again at the end: the loads stay unconditional
        plain = tn.first + tn.rows <= a.whole;
        f4 mw[U / 2];   // a few words of mu at a time: the LDS answers once for all of them
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u % (U / 2) == 0) {
#pragma unroll
                for (int q = 0; q < U / 2; ++q) mw[q] = *(const f4*)(mus + 4 * (int)(in.rc[u + q] & 0xffffu));
                __builtin_amdgcn_sched_barrier(0);
            }
            const int row = (int)(in.rc[u] >> 16), c = (int)(in.rc[u] & 0xffffu);
            f4 v = in.value(u) - mw[u % (U / 2)];
            if (EXACT) in.drop_repeats(a, d, c, v);
            in.load(a, tn, d, plain, u);
            if constexpr (EXACT) {
                *(f4*)(xs + row * RB + 16 * c) = v;
            } else {
                u2 h, l;
                split4(v, h, l);
                *(u2*)(xs + row * RB + 8 * c) = h;
                *(u2*)(xs + row * RB + 8 * c + 64 * STEPS) = l;
            }
        }
        if (!plain) in.load_rest(a, tn, d, a.M);
        if (!first) store_y(before);
        __syncthreads();
        // (short bases leave most of a tile empty)
        const int groups = a.B > 1 ? (t.rows + 15) / 16 : a.rows / 16;
        for (int g = ws; g < groups; g += WS) {
            f4 acc[NTW];
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt) acc[nt] = f4{0.f, 0.f, 0.f, 0.f};
            const char* xr = xs + (16 * g + n_) * RB + 16 * kk;
            if constexpr (EXACT) {
                f4 x[2];   // a word is read ahead of the products of the one before
                x[0] = *(const f4*)xr;
#pragma unroll
                for (int w = 0; w < 2 * STEPS; ++w) {
                    if (w + 1 < 2 * STEPS) x[(w + 1) & 1] = *(const f4*)(xr + 64 * (w + 1));
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int nt = 0; nt < NTW; ++nt)
                            acc[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(us[nt][w >> 1][w & 1][j]), x[w & 1][j], acc[nt], 0, 0, 0);
                }
            } else {
                constexpr int AT = NTW * STEPS <= 8 ? 4 : 2;   // steps whose operands are read together
#pragma unroll
                for (int s0 = 0; s0 < STEPS; s0 += AT) {
                    u4 xh[AT], xl[AT];
#pragma unroll
                    for (int q = 0; q < AT; ++q) {
                        if (s0 + q >= STEPS) break;
                        xh[q] = *(const u4*)(xr + 64 * (s0 + q));
                        xl[q] = *(const u4*)(xr + 64 * (STEPS + s0 + q));
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int q = 0; q < AT; ++q) {
                        if (s0 + q >= STEPS) break;
                        const lbf8 bh = __builtin_bit_cast(lbf8, xh[q]), bl = __builtin_bit_cast(lbf8, xl[q]);
#pragma unroll
                        for (int nt = 0; nt < NTW; ++nt)
                            acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lbf8, us[nt][s0 + q][0]), bl, acc[nt], 0, 0, 0);
#pragma unroll
                        for (int nt = 0; nt < NTW; ++nt)
                            acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lbf8, us[nt][s0 + q][1]), bh, acc[nt], 0, 0, 0);
#pragma unroll
                        for (int nt = 0; nt < NTW; ++nt)
                            acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lbf8, us[nt][s0 + q][0]), bh, acc[nt], 0, 0, 0);
                    }
                }
            }
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt) {
                const int c0 = 16 * (wn * NTW + nt) + 4 * kk;
                float* y = ys + (16 * g + n_) * k + c0;
                if ((k & 3) == 0) {
                    if (c0 < k) *(f4*)y = acc[nt];
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (c0 + r < k) y[r] = acc[nt][r];
                }
            }
        }
        __syncthreads();
        before = t;
        if (!more) break;
        t = tn;
    }
    store_y(before);
}

// --------------------------------------------------------------------------------------
// decompress.  Wave (wn, ws): element tiles wn ETW .. + ETW - 1 of slice groups ws, ws + W/wn, ...  Step ks of 32 comps, operands as in compress with
// elements in the place of comps: A lane (m, kk) U[16 et + m][32 ks + 8 kk + j] (split) or [32 ks + 16 i + 4 kk + j] (EXACT).
// Upack[b][et][ks][2][64].  LDS: y, mu [16 wn ETW], x [rows][d] fp32 (flow_out_row).
// --------------------------------------------------------------------------------------
template <int ETW, int KST, bool EXACT, int W>
__global__ __launch_bounds__(64 * W, 8 / W) void decompress_flow_kernel(FlowArgs a)
{
    constexpr int NTHR = 64 * W, U = 4, RB = flow_row(KST);
    extern __shared__ f4 smem[];
    char* yh = (char*)smem;
    float* mus = (float*)(yh + a.rows * RB);
    float* os = mus + 16 * a.wn * ETW;
    const int tid = threadIdx.x, lane = tid & 63, n_ = lane & 15, kk = lane >> 4, d = a.d, k = a.k;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wn = wave % a.wn, ws = wave / a.wn, WS = W / a.wn;

    for (int i = tid; i < a.rows * RB / 16; i += NTHR) smem[i] = f4{0.f, 0.f, 0.f, 0.f};
    FlowInput<U, NTHR, false> in;
    in.init(a, k);

    FlowIter it(a);
    if (it.tile >= a.t1) return;
    FlowTile t = it.get(a), before = t;
    bool plain = t.first + t.rows <= a.whole;
#pragma unroll
    for (int u = 0; u < U; ++u)
        in.load(a, t, k, plain, u);
    if (!plain) in.load_rest(a, t, k, a.S * k);

    u4 us[ETW][KST][2];
    int cur = -1;
    const FlowRun<4, NTHR> run4(d, a.by_out);
    const FlowRun<8, NTHR> run8(d, a.by_out);
    const int xrow = flow_out_row(d);
    auto store_x = [&](const FlowTile& q) {
        const int64_t at = q.first * d, room = a.M - at;
        const int total = (int64_t)q.rows * d < room ? q.rows * d : (int)room;
        if (a.out_bf16) {
            unsigned short* X = (unsigned short*)a.out + at;
            run8.each(os, d, total, [&](int j, const float* x) {
                const f4 v0 = *(const f4*)x, v1 = *(const f4*)(x + 4);
                const hu4 w = {pack_bf16x2(v0[0], v0[1]), pack_bf16x2(v0[2], v0[3]), pack_bf16x2(v1[0], v1[1]), pack_bf16x2(v1[2], v1[3])};
                __builtin_nontemporal_store(w, (hu4*)(X + 8 * j));
            });
            const int j = (total & ~7) + tid;
            if (j < total) X[j] = (unsigned short)f32_to_bf16_rne(*run8.number(os, d, j));
        } else {
            float* X = (float*)a.out + at;
            run4.each(os, d, total, [&](int j, const float* x) {
                __builtin_nontemporal_store((fw4)*(const f4*)x, (fw4*)(X + 4 * j));
            });
            const int j = (total & ~3) + tid;
            if (j < total) X[j] = *run4.number(os, d, j);
        }
    };

    for (bool first = true;; first = false) {
        if (t.b != cur) {
            cur = t.b;
            const u4* Ub = a.Upack + (size_t)cur * a.upack_stride + (size_t)wn * ETW * KST * 128 + lane;
#pragma unroll
            for (int et = 0; et < ETW; ++et)
#pragma unroll
                for (int ks = 0; ks < KST; ++ks)
#pragma unroll
                    for (int p = 0; p < 2; ++p) us[et][ks][p] = Ub[((et * KST + ks) * 2 + p) * 64];
            for (int e = tid; e < 16 * a.wn * ETW; e += NTHR) mus[e] = e < d ? a.mu[(size_t)cur * d + e] : 0.f;
            drain_memory();
            __syncthreads();
        }
        const bool more = it.advance(a);
        const FlowTile tn = more ? it.get(a) : t;
        plain = tn.first + tn.rows <= a.whole;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = (int)(in.rc[u] >> 16), c = (int)(in.rc[u] & 0xffffu);
            f4 v = in.value(u);
            if (EXACT) in.drop_repeats(a, k, c, v);
            in.load(a, tn, k, plain, u);
            if constexpr (EXACT) {
                *(f4*)(yh + row * RB + 16 * c) = v;
            } else {
                u2 h, l;
                split4(v, h, l);
                *(u2*)(yh + row * RB + 8 * c) = h;
                *(u2*)(yh + row * RB + 8 * c + 64 * KST) = l;
            }
        }
        if (!plain) in.load_rest(a, tn, k, a.S * k);
        if (!first) store_x(before);
        __syncthreads();
        const int groups = a.B > 1 ? (t.rows + 15) / 16 : a.rows / 16;
        for (int g = ws; g < groups; g += WS) {
            const char* yr = yh + (16 * g + n_) * RB + 16 * kk;
            f4 acc[ETW];
#pragma unroll
            for (int et = 0; et < ETW; ++et) acc[et] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KST; ++ks) {
                if constexpr (EXACT) {
#pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        const f4 y = *(const f4*)(yr + 128 * ks + 64 * w);
#pragma unroll
                        for (int j = 0; j < 4; ++j)
#pragma unroll
                            for (int et = 0; et < ETW; ++et)
                                acc[et] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(us[et][ks][w][j]), y[j], acc[et], 0, 0, 0);
                    }
                } else {
                    const lbf8 bh = __builtin_bit_cast(lbf8, *(const u4*)(yr + 64 * ks));
                    const lbf8 bl = __builtin_bit_cast(lbf8, *(const u4*)(yr + 64 * (KST + ks)));
#pragma unroll
                    for (int et = 0; et < ETW; ++et)
                        acc[et] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lbf8, us[et][ks][0]), bl, acc[et], 0, 0, 0);
#pragma unroll
                    for (int et = 0; et < ETW; ++et)
                        acc[et] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lbf8, us[et][ks][1]), bh, acc[et], 0, 0, 0);
#pragma unroll
                    for (int et = 0; et < ETW; ++et)
                        acc[et] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lbf8, us[et][ks][0]), bh, acc[et], 0, 0, 0);
                }
            }
#pragma unroll
            for (int et = 0; et < ETW; ++et) {
                const int e0 = 16 * (wn * ETW + et) + 4 * kk;
                const f4 v = acc[et] + *(const f4*)(mus + e0);
                float* x = os + (16 * g + n_) * xrow + e0;
                if ((d & 3) == 0) {
                    if (e0 < d) *(f4*)x = v;
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (e0 + r < d) x[r] = v[r];
                }
            }
        }
        __syncthreads();
        before = t;
        if (!more) break;
        t = tn;
    }
    store_x(before);
}

// ---- host side --------------------------------------------------------------------------------------------------------
typedef void (*flow_kernel)(FlowArgs);
flow_kernel gvq_flow_compress_f32(const FlowPlan& p);    // null: there is no instance for the plan
flow_kernel gvq_flow_compress_bf16(const FlowPlan& p);
flow_kernel gvq_flow_decompress(const FlowPlan& p);
