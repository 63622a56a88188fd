// The covariance of a first-slice refresh's samples, which its own kernel (gvq_sample.hip) and, behind the work-groups of its
// matrices, the tridiagonalisation (gvq_eigen.hip) make.
#pragma once
#include "gvq_eigen.h"

struct SampleCov {
    const double* X;       // [B][L][d], x_stride apart: the centred samples
    size_t x_stride;
    double* cov;           // [B][d][d]
    int L, d, blocks, total;   // 64 x 64 blocks of one matrix's upper triangle, of all
};

// C = X^T X / L: block `at` of all by one wave, with its mirror image.  Returns the largest |entry|, or a NaN among them.
__device__ __forceinline__ double sample_cov_block(const SampleCov& a, int at)
{
    typedef double d4 __attribute__((ext_vector_type(4)));
    const int b = at / a.blocks, lane = threadIdx.x & 63, m = lane & 15, kk = lane >> 4, d = a.d;
    const int ng = (d + 63) / 64;
    int g1 = 0, rem = at - b * a.blocks;
    while (rem >= ng - g1) { rem -= ng - g1; ++g1; }
    const int g2 = g1 + rem;
    const double* X = a.X + (size_t)b * a.x_stride;
    d4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
    double na[4], nb[4];
    auto fetch = [&](int l) {   // one group of four samples ahead, from inside the array; zero past the last sample
        const double* row = X + (size_t)(l + kk < a.L ? l + kk : a.L - 1) * d;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int e1 = 64 * g1 + 16 * t + m, e2 = 64 * g2 + 16 * t + m;
            na[t] = row[e1 < d ? e1 : d - 1];
            nb[t] = row[e2 < d ? e2 : d - 1];
        }
    };
    fetch(0);
    for (int l = 0; l < a.L; l += 4) {
        double va[4], vb[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            va[t] = l + kk < a.L ? na[t] : 0.0;
            vb[t] = nb[t];
        }
        fetch(l + 4);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(va[i], vb[j], acc[i][j], 0, 0, 0);
    }
    double* cov = a.cov + (size_t)b * d * d;
    double big = 0.0, bad = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 64 * g1 + 16 * i + 4 * r + kk, col = 64 * g2 + 16 * j + m;
                if (row >= d || col >= d) continue;
                const double v = acc[i][j][r] / (double)a.L;
                cov[(size_t)row * d + col] = v;
                if (g1 != g2) cov[(size_t)col * d + row] = v;
                big = fmax(big, fabs(v));
                if (v != v) bad = v;
            }
    return bad != bad ? bad : big;
}
