// Gradient flattening of GradiVeQ (Section 2, first paragraphs, and Fig. 2a): the gradient of a
// convolution layer with F filters of depth D, height H, width W is laid out so that the F
// gradients at the same (depth, row, column) position of the F filters are adjacent; these
// groups follow each other along the depth first, then the width, then the height:
//     flat[((h*W + w)*D + d)*F + f] = grad[f][d][h][w]          (grad stored [F][D][H][W])
// That is the order in which neighbouring numbers are linearly correlated, which is what the
// slice-wise PCA lives on.  Pure permutation; bound by HBM.
//
// One work-group moves a tile of TF filters x a run of consecutive numbers of each filter (TD depths x all H*W
// positions, or one depth x a piece of H*W when that alone is longer than a tile) through LDS, tile[row][filter] with
// row = hw * nd + dd the order of the flat side.
//   [F][D][H][W] side: a thread takes GV consecutive numbers of VT = 16 / sizeof(T) neighbouring filters (VT accesses),
//     transposes them in registers and exchanges GV whole 16-byte words with LDS.  GV = VT where runs are 16-byte
//     aligned (D*H*W and the pieces multiples of VT), else 1.
//   flat side: a thread moves FV neighbouring filters of one row; FV = VT where F is a multiple of VT (and both arrays are
//     16-byte aligned), else one 32-bit word at whatever address: one fp32 number or two bf16 (a bf16 number at a time, two
//     lanes shared a bank: 4097 x 4096 unflatten 68 us, 19 now, 51 before the words of LDS were permuted).
// A thread's accesses of a side are all requested before the first of them is waited for (up to eight 16-byte words):
// with one at a time, as before, a tile took a memory latency per word.  The 16-byte words of a row are permuted by
// x -> x ^ (row ^ row >> 2): words of one filter group in rows 4 c + i, c = 0, 1, 2 .., then sit in different banks, and so
// does a whole row; no padding.
// Every access is 256 bytes or more in one piece; what is left is how the pieces in flight lie in memory.  A layer of 32 MB
// and more takes its tiles with the filter groups fastest (whole rows of the flat side at a time; fully connected 4096 x 25088
// fp32 5.1 TB/s read + written against 4.65 along the runs), a smaller one along the runs (1000 x 4096 4.1 against 3.7).  With
// the filter groups fastest, work-groups side by side read the same columns of rows D*H*W numbers apart; where that is close to
// a multiple of 8 KB they meet in the same channels, and each filter group starts one run further on instead (the diagonals of
// the grid of tiles: 4096 x 16384 flatten 3.7 -> 5.0, 4096 x 4112 3.6 -> 4.7, 4096 x 16448 4.1 -> 4.8; 4096 x 25088 would lose
// 1 - 2 %).  Tiles of 128 filters are no faster (4096 x 4096: 5.6 against 6.3), nor are non-temporal accesses.
// fp32 / bf16, flatten, TB/s: 4096 x 25088 5.1 / 4.8 (one access at a time and LDS rows of odd length: 4.4 / 3.7), 4096 x 16384
// 5.0 / 5.0 (4.4 / 3.5), 4096 x 4096 4.9 / 4.4 (6.3 / 6.0 out of the last-level cache), 512 x 4096 x 3 x 3 4.4 / 4.2, 512 x 512
// x 3 x 3 3.1 / 2.1 (6 and 4.5 us: a tile's latency).
#include <type_traits>

#include "gvq_internal.h"

#define LAYOUT_THREADS 256
#define LAYOUT_TF 64
#define LAYOUT_TILE 32768   // bytes of LDS per work-group

struct LayoutArgs {
    const void* src;
    void* dst;
    int F, D, HW;
    int TD, HWT;               // depths and positions per tile (TD = 1 or HWT = H*W)
    int n_ftiles, n_dtiles, n_hwtiles;
    unsigned int magic;        // n / H*W = n * magic >> 16 for the positions of a tile (TD > 1)
    int filters_fast;          // order of the tiles: the filter groups, or the runs, fastest
    int skew;                  // filter groups fastest: runs that each group starts after the one before it
};

typedef unsigned int lu4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned int first_of(unsigned int x) { return x; }
__device__ __forceinline__ unsigned int first_of(lu4 x) { return x[0]; }

template <typename T, int N> union LayoutVec {
    lu4 v;
    T e[N];
};

template <typename T, bool FLATTEN, int GV, int FV>
__global__ __launch_bounds__(LAYOUT_THREADS) void conv_layout_kernel(LayoutArgs a)
{
    extern __shared__ lu4 tile[];                         // [rows][TF / VT] 16-byte words, permuted within a row
    constexpr int TF = LAYOUT_TF, VT = 16 / sizeof(T), QF = TF / VT;
    constexpr int GI = GV > 1 ? LAYOUT_TILE / 16 / VT / LAYOUT_THREADS : 2;   // items in flight on the [F][D][H][W] side
    constexpr int FI = 8;                                                     // accesses in flight on the flat side
    typedef typename std::conditional<FV == VT, lu4, unsigned int>::type FVec;
    static_assert(FV * sizeof(T) == sizeof(FVec), "an access of the flat side");
    typedef LayoutVec<T, VT> Vec;
    const int tid = threadIdx.x;
    const int nr = a.n_dtiles * a.n_hwtiles;              // runs of a filter
    const int ft = a.filters_fast ? (int)blockIdx.x % a.n_ftiles : (int)blockIdx.x / nr;
    int rt = a.filters_fast ? (int)blockIdx.x / a.n_ftiles : (int)blockIdx.x - ft * nr;
    if (a.skew) rt = (rt + a.skew * ft) % nr;
    const int dt = rt / a.n_hwtiles, ht = rt - dt * a.n_hwtiles;
    const int f0 = ft * TF, d0 = dt * a.TD, hw0 = ht * a.HWT;
    const int nf = a.F - f0 < TF ? a.F - f0 : TF;
    const int nd = a.D - d0 < a.TD ? a.D - d0 : a.TD;
    const int nhw = a.HW - hw0 < a.HWT ? a.HW - hw0 : a.HWT;
    const int run = nd * nhw;                             // consecutive numbers of a filter
    const size_t fstride = (size_t)a.D * a.HW;
    T* const gside = (T*)(FLATTEN ? a.src : a.dst) + (size_t)f0 * fstride + (size_t)d0 * a.HW + hw0;
    T* const fside = (T*)(FLATTEN ? a.dst : a.src) + ((size_t)hw0 * a.D + d0) * a.F + f0;
    const auto word = [](int row, int q) { return row * QF + (q ^ ((row ^ (row >> 2)) & (QF - 1))); };

    // [F][D][H][W] side: item = (group of VT filters, GV consecutive numbers)
    const auto g_side = [&]() {
        const int rq = run / GV, nq = (nf + VT - 1) / VT, items = rq * nq;
        for (int it0 = tid; it0 < items; it0 += GI * LAYOUT_THREADS) {
            int q[GI], r0[GI];
            T x[GI][VT][GV];       // [item][filter][number]
#pragma unroll
            for (int n = 0; n < GI; ++n) {
                const int it = it0 + n * LAYOUT_THREADS;
                q[n] = it < items ? it / rq : -1;
                r0[n] = GV * (it - q[n] * rq);
            }
            if (FLATTEN) {
#pragma unroll
                for (int n = 0; n < GI; ++n) {
                    if (q[n] < 0) continue;
                    const T* p = gside + (size_t)(VT * q[n]) * fstride + r0[n];
#pragma unroll
                    for (int u = 0; u < VT; ++u, p += fstride) {
                        if (FV < VT && VT * q[n] + u >= nf) continue;     // F a multiple of VT otherwise
                        if constexpr (GV > 1) {
                            const lu4 w = *(const lu4*)p;
                            __builtin_memcpy(x[n][u], &w, 16);
                        } else {
                            x[n][u][0] = *p;
                        }
                    }
                }
            }
#pragma unroll
            for (int n = 0; n < GI; ++n) {
                if (q[n] < 0) continue;
#pragma unroll
                for (int i = 0; i < GV; ++i) {
                    int row = r0[n] + i;
                    if (nd > 1) {
                        const int dd = (int)((unsigned int)row * a.magic >> 16);
                        row = (row - dd * nhw) * nd + dd;
                    }
                    Vec w;
                    if (FLATTEN) {
#pragma unroll
                        for (int u = 0; u < VT; ++u) w.e[u] = x[n][u][i];
                        tile[word(row, q[n])] = w.v;
                    } else {
                        w.v = tile[word(row, q[n])];
#pragma unroll
                        for (int u = 0; u < VT; ++u) x[n][u][i] = w.e[u];
                    }
                }
            }
            if (!FLATTEN) {
#pragma unroll
                for (int n = 0; n < GI; ++n) {
                    if (q[n] < 0) continue;
                    T* p = gside + (size_t)(VT * q[n]) * fstride + r0[n];
#pragma unroll
                    for (int u = 0; u < VT; ++u, p += fstride) {
                        if (FV < VT && VT * q[n] + u >= nf) continue;
                        if constexpr (GV > 1) {
                            lu4 w;
                            __builtin_memcpy(&w, x[n][u], 16);
                            *(lu4*)p = w;
                        } else {
                            *p = x[n][u][0];
                        }
                    }
                }
            }
        }
    };
    // flat side: rows of the tile, FV filters per access; a row of the tile is TF / FV accesses wide
    const auto f_side = [&]() {
        constexpr int W = TF / FV, ROWS = LAYOUT_THREADS / W;
        const int c = tid % W;                            // this thread's access within every row
        if (c * FV >= nf) return;
        const bool single = FV == 2 && c * FV + 1 >= nf;  // the last of an odd number of filters
        for (int row0 = tid / W; row0 < run; row0 += FI * ROWS) {
            FVec x[FI];
            T* p[FI];
#pragma unroll
            for (int n = 0; n < FI; ++n) {
                const int row = row0 + n * ROWS;
                const int hw = nhw == 1 ? 0 : nd == 1 ? row : row / nd, dd = row - hw * nd;   // row = hw * nd + dd
                p[n] = fside + ((size_t)hw * a.D + dd) * a.F + FV * c;
                if (!FLATTEN && row < run) {
                    if (single) x[n] = FVec{} + *p[n];
                    else if constexpr (FV == VT) x[n] = *(const FVec*)p[n];
                    else __builtin_memcpy(&x[n], p[n], sizeof(FVec));   // of any alignment
                }
            }
#pragma unroll
            for (int n = 0; n < FI; ++n) {
                const int row = row0 + n * ROWS;
                if (row >= run) break;
                // FVec is the type of the 16-byte words' parts here, whose address is a multiple of its size
                FVec& w = ((FVec*)&tile[word(row, c * FV / VT)])[c % (VT / FV)];
                if (FLATTEN) x[n] = w;
                else w = x[n];
            }
            if (FLATTEN) {
#pragma unroll
                for (int n = 0; n < FI; ++n) {
                    if (row0 + n * ROWS >= run) break;
                    if (single) *p[n] = (T)first_of(x[n]);
                    else if constexpr (FV == VT) *(FVec*)p[n] = x[n];
                    else __builtin_memcpy(p[n], &x[n], sizeof(FVec));
                }
            }
        }
    };
    if (FLATTEN) {
        g_side();
        __syncthreads();
        f_side();
    } else {
        f_side();
        __syncthreads();
        g_side();
    }
}

// Layers whose two orders are the same (a bias: D = H*W = 1, or one filter with D or H*W = 1): a copy, 16 bytes per
// thread where both sides are aligned.  Through the tiles a bias took 3.6 us on average instead of 2.6, all of it latency.
template <typename T>
__global__ __launch_bounds__(LAYOUT_THREADS) void layout_copy_kernel(const T* src, T* dst, size_t n, int words)
{
    constexpr int VT = 16 / sizeof(T);
    const size_t i0 = (size_t)blockIdx.x * LAYOUT_THREADS + threadIdx.x, step = (size_t)gridDim.x * LAYOUT_THREADS;
    const size_t w = words ? n / VT : 0;
    for (size_t i = i0; i < w; i += step) ((lu4*)dst)[i] = ((const lu4*)src)[i];
    for (size_t i = w * VT + i0; i < n; i += step) dst[i] = src[i];
}

template <typename T, bool FLATTEN, int GV, int FV>
static int launch_tiles(const LayoutArgs& a, int64_t grid, size_t lds, hipStream_t st)
{
    hipLaunchKernelGGL((conv_layout_kernel<T, FLATTEN, GV, FV>), dim3((unsigned)grid), dim3(LAYOUT_THREADS), lds, st, a);
    GVQ_HIP(hipGetLastError());
    return GVQ_OK;
}

template <typename T, bool FLATTEN>
static int launch_layout(const void* src, void* dst, int F, int D, int HW, hipStream_t st)
{
    constexpr int VT = 16 / sizeof(T), F1 = 4 / sizeof(T);
    const bool aligned = (((uintptr_t)src | (uintptr_t)dst) & 15) == 0;
    if (D * (int64_t)HW == 1 || (F == 1 && (D == 1 || HW == 1))) {
        const size_t n = (size_t)F * D * HW, per = (size_t)LAYOUT_THREADS * (aligned ? VT : 1);
        const size_t grid = (n + per - 1) / per;
        hipLaunchKernelGGL((layout_copy_kernel<T>), dim3((unsigned)(grid < 2048 ? grid : 2048)), dim3(LAYOUT_THREADS), 0, st,
                           (const T*)src, (T*)dst, n, aligned ? 1 : 0);
        GVQ_HIP(hipGetLastError());
        return GVQ_OK;
    }
    const bool fv = aligned && F % VT == 0;
    bool gv = aligned && ((int64_t)D * HW) % VT == 0;
    const int max_run = LAYOUT_TILE / LAYOUT_TF / (int)sizeof(T);   // numbers of one filter, a multiple of VT
    const int n_ftiles = (F + LAYOUT_TF - 1) / LAYOUT_TF;
    LayoutArgs a;
    a.src = src; a.dst = dst; a.F = F; a.D = D; a.HW = HW;
    // a small layer is cut into shorter runs, down to 32 numbers, so that its tiles reach more of the chip
    int most = max_run;
    while (most > 32 && (int64_t)n_ftiles * (((int64_t)D * HW + most - 1) / most) < 512) most /= 2;
    a.HWT = HW;
    a.TD = 1;
    if (HW > most && HW > max_run) {
        if (HW % VT) gv = false;
        a.HWT = most;
    } else {
        const int fit = HW > most ? HW : most;
        int step = 1;                                         // depths whose run is a multiple of VT
        if (gv) while ((HW * step) % VT) step *= 2;
        int td = fit / HW / step * step;
        if (td < step) {                                      // not one such group of depths in a tile
            td = max_run / HW / step * step;
            if (td < step) { td = max_run / HW; gv = false; }
            else td = step;
        }
        a.TD = td < D ? td : D;
    }
    a.n_dtiles = (D + a.TD - 1) / a.TD;
    a.n_hwtiles = (HW + a.HWT - 1) / a.HWT;
    a.magic = (65536u + (unsigned int)a.HWT - 1) / (unsigned int)a.HWT;
    a.n_ftiles = n_ftiles;
    a.filters_fast = (size_t)F * D * HW * sizeof(T) >= (32u << 20);
    a.skew = a.filters_fast && (size_t)D * HW * sizeof(T) % 8192 < 1024;
    const size_t lds = sizeof(T) * (size_t)a.TD * a.HWT * LAYOUT_TF;
    const int64_t grid = (int64_t)n_ftiles * a.n_dtiles * a.n_hwtiles;
    if (grid > 0x7fffffff) return GVQ_EINVAL;
    if (gv && fv) return launch_tiles<T, FLATTEN, VT, VT>(a, grid, lds, st);
    if (gv) return launch_tiles<T, FLATTEN, VT, F1>(a, grid, lds, st);
    if (fv) return launch_tiles<T, FLATTEN, 1, VT>(a, grid, lds, st);
    return launch_tiles<T, FLATTEN, 1, F1>(a, grid, lds, st);
}

int gvq_launch_layout(const void* src, void* dst, int F, int D, int HW, gvq_dtype_t dtype, bool flatten,
                      hipStream_t st)
{
    if (dtype == GVQ_BF16)
        return flatten ? launch_layout<unsigned short, true>(src, dst, F, D, HW, st)
                       : launch_layout<unsigned short, false>(src, dst, F, D, HW, st);
    return flatten ? launch_layout<unsigned int, true>(src, dst, F, D, HW, st)
                   : launch_layout<unsigned int, false>(src, dst, F, D, HW, st);
}
