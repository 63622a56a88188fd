// Shared by the two kernels that sum x x^T (gvq_moments.hip: float64 matrix pipe, gvq_moments_int.hip: int8 matrix pipe): their
// arguments and how a task's tile pairs are numbered in the partials.
#pragma once
#include <type_traits>
#include <utility>

#include "gvq_internal.h"

// f(0) .. f(N - 1) with the index as a compile-time constant (which tiles a pair names decides which registers are used).
template <typename F, int... I>
__device__ __forceinline__ void static_for_seq(F f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void static_for(F f)
{
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}

struct MomArgs {
    gvq_ptrs grads;
    int L;
    const int64_t* offs;
    int64_t M;
    int d, np, pw;                // np panels of pw elements, the last one shorter
    int chunks_diag, chunks_off;  // sample chunks of the two kinds of task
    int accumulate;               // 0: overwrite the partials, 1: add to them
    double* part;                 // [B][part_basis]: the diagonal tasks' partials, then the others'
    size_t part_basis;
    unsigned long long* nsamp;    // [B] += the sample slices this launch took in (counted by the tasks of panel 0)
};

// Words of four numbers: WORDS per row (sample) in LDS, RPS rows per 256 threads, four words per thread and block.
// SPLIT: the tile pairs are shared out among the four waves, which then all read every sample; with few pairs each wave
// has all of them and takes every fourth group of four samples.  Rows of an even number of tiles get one tile of
// padding where all waves read them, so that the rows of a group start 32 banks apart.
template <int NT, bool OFF> struct MomShape {
    static constexpr bool SPLIT = OFF || NT >= 6;
    static constexpr int NPAIR = OFF ? NT * NT : NT * (NT + 1) / 2;
    static constexpr int TILES = OFF ? 2 * NT : NT;
    static constexpr int U = 4;                                    // words per thread and block
    static constexpr int WORDS = 4 * TILES, RPS = SPLIT ? 256 / WORDS : 256 / WORDS / 4 * 4, NS = U * RPS;
    static constexpr int STRIDE = SPLIT ? 1 : 4, NGW = NS / 4 / STRIDE;   // groups of four samples per wave and block
    static constexpr int NACC = SPLIT ? (NPAIR + 3) / 4 : NPAIR;
    static constexpr int ROW = 16 * (SPLIT ? (TILES | 1) : TILES);
    static constexpr int PART = NPAIR * 256 + (OFF ? 0 : 16 * NT);
    static constexpr int BUF = NS * ROW;       // doubles per buffer
    static constexpr int LDS = 2 * BUF * 8;    // bytes
    static __host__ __device__ constexpr int row(int p)
    {
        if (OFF) return p / NT;
        int t = 0;
        while (p >= NT - t) { p -= NT - t; ++t; }
        return t;
    }
    static __host__ __device__ constexpr int col(int p)   // tile index in the LDS row
    {
        if (OFF) return NT + p % NT;
        int t = 0;
        while (p >= NT - t) { p -= NT - t; ++t; }
        return t + p;
    }
    static constexpr bool needs(int p0, int p1, int tile)   // one of the pairs p0 .. p1 - 1 has this tile
    {
        for (int p = p0; p < p1; ++p)
            if (row(p) == tile || col(p) == tile) return true;
        return false;
    }
};
