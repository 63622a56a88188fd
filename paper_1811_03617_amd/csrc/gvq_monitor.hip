// Eq. (6) of GradiVeQ, the local compression loss, for one basis with 17 to 32 comps and slices of 64 or 128 elements:
// per slice y = U^T (x - mu/N), then |x - mu/N - U y|^2, summed over all slices.
//
// 4 d k flop per slice, twice what Eq. (2) needs, and on the fp32 matrix pipe they take longer than the gradient takes to
// arrive (138 M elements, d = 128, k = 32: 113 against 90 us; 161 - 190 us measured, the products and the rest of a wave's
// work hardly overlapped).  So both contractions run on v_mfma_f32_16x16x32_bf16, with every fp32 number as three bf16 terms
// that add up to it exactly (x and y cut off at 8 bits, U rounded to nearest): of the nine products of two numbers the six
// with i + j <= 4 are taken, what is left out is below 2^-24 of the product, and the large ones are added to the sum of the
// small ones.  Six products take 100 matrix cycles where the fp32 pipe takes 256.  138 M elements, d = 128, k = 32, the whole call:
// 161 -> 118 - 124 us (its kernels in a trace 190 -> 121; bf16 storage 158 -> 110; 60 M elements, d = 64, k = 24 78 -> 60), relative error against float64 over 18 draws of
// sizes and noise levels 1.7e-7 -> 1.6e-7 rms.  What bounds it now is a wave's own instructions: splitting, products and residuals of a tile
// of 16 slices take 4000 cycles of a SIMD, of which the matrix pipe is busy 1700; the gradient alone would take 90 us.
//
// Every wave sums its residuals in float64; one number per work-group leaves (the sum over slices used to be a launch of its own,
// 7 us, over one float per slice).
//
// Operand orders, lane l, n = l%16, kk = l/16.  The order of a contraction is free, and so is the order of the rows of a
// product's result; they are chosen so that nothing moves between lanes:
//   y:  A[row 16 nt + l%16 = comp][8 kk + j] = U[32 st + 8 kk + j][comp], B = x[slice n][32 st + 8 kk + j]
//   U y: row m of result tile (st, h) is element 32 st + 8 (m / 4) + 4 h + m % 4, so that result register r of lane (n, kk) is
//       the element 8 kk + 4 h + r of step st that the same lane holds for the first product; contraction slot 8 kk + j is
//       comp 16 (j / 4) + 4 kk + j % 4, which is where the first product's result registers are.
#include "gvq_device.h"

struct LossArgs {
    const void* in;
    const u4* pack;        // [d/32][3][2][64] then [2 d/32][3][64], see pack_loss_kernel
    const float* mu;
    double* part;          // [grid]
    int64_t M, n_super, T; // super-tiles (2048 elements each, whole slices), 16-slice tiles in all
    float n_workers;
    int il;                // super-tiles whose 1 KB rows interleave (CodecArgs::il)
};

// 8 floats -> three bf16 terms in operand order; each term is the upper half of what the ones before leave, so that the sum is
// exact and no finite number turns infinite.
__device__ __forceinline__ void split8x3(const f4& v0, const f4& v1, u4 (&t)[3])
{
    unsigned int r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = __float_as_uint(i < 4 ? v0[i & 3] : v1[i & 3]);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
#pragma unroll
        for (int i = 0; i < 4; ++i) t[p][i] = __builtin_amdgcn_perm(r[2 * i + 1], r[2 * i], 0x07060302u);
        if (p < 2) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                r[i] = __float_as_uint(__uint_as_float(r[i]) - __uint_as_float(r[i] & 0xffff0000u));
        }
    }
}

__device__ __forceinline__ f4 mfma_bf16(const u4& a, const u4& b, const f4& c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lbf8, a), __builtin_bit_cast(lbf8, b), c, 0, 0, 0);
}

template <int D, bool BF16>
__global__ __launch_bounds__(WG_THREADS, 2) void loss_split_kernel(LossArgs a)
{
    constexpr int G = 128 / D, ST = D / 32, CPS = D / 4, ES = BF16 ? 2 : 4;
    constexpr int EPL = BF16 ? 8 : 4, LCPS = D / EPL, NL = 2048 / EPL / 64, NLT = NL / G;   // loads per super-tile and tile
    __shared__ f4 lds_all[WAVES_PER_WG][512];
    __shared__ u4 ud[2 * ST * 3 * 64];
    __shared__ double red[WAVES_PER_WG];
    const int lane = threadIdx.x & 63, n_ = lane & 15, kk = lane >> 4, wave = threadIdx.x >> 6;
    f4* lds = lds_all[wave];

    for (int i = threadIdx.x; i < 2 * ST * 3 * 64; i += WG_THREADS) ud[i] = a.pack[ST * 3 * 2 * 64 + i];
    u4 uf[ST][2][2];   // the third terms are used once per step: in LDS, for the registers' sake
    __shared__ u4 u3_lds[ST * 2 * 64];
    for (int i = threadIdx.x; i < ST * 2 * 64; i += WG_THREADS) u3_lds[i] = a.pack[(i / 128 * 3 + 2) * 128 + i % 128];
#pragma unroll
    for (int st = 0; st < ST; ++st)
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) uf[st][p][nt] = a.pack[((st * 3 + p) * 2 + nt) * 64 + lane];
    const int lc = lane % LCPS;
    float mun[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) mun[i] = a.mu[lc * EPL + i] / a.n_workers;
    int in_slot[NL];
#pragma unroll
    for (int r = 0; r < NL; ++r) {
        const int row = (r * 64 + lane) / LCPS;
        in_slot[r] = row * CPS + ((BF16 ? 2 * lc : lc) ^ swz<D>(row & 15));
    }
    __syncthreads();

    auto park = [&](int r, const u4& v) {
        if (BF16) {
            const f4 lo = {bf16_to_f32(v.x & 0xffffu) - mun[0], bf16_to_f32(v.x >> 16) - mun[1],
                           bf16_to_f32(v.y & 0xffffu) - mun[2], bf16_to_f32(v.y >> 16) - mun[3]};
            const f4 hi = {bf16_to_f32(v.z & 0xffffu) - mun[4 % EPL], bf16_to_f32(v.z >> 16) - mun[5 % EPL],
                           bf16_to_f32(v.w & 0xffffu) - mun[6 % EPL], bf16_to_f32(v.w >> 16) - mun[7 % EPL]};
            lds[in_slot[r]] = lo;
            lds[in_slot[r] ^ 1] = hi;
        } else {
            lds[in_slot[r]] = f4{__uint_as_float(v.x) - mun[0], __uint_as_float(v.y) - mun[1],
                                 __uint_as_float(v.z) - mun[2], __uint_as_float(v.w) - mun[3]};
        }
    };
    double total = 0.0;
    // the 16 slices parked as tile g; elements from `end` on (counted from the tile's first) are padding
    auto residual = [&](int g, auto checked, int64_t end) {
        f4 x[ST][2], hi[2], lo[2];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) hi[nt] = lo[nt] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int st = 0; st < ST; ++st) {
#pragma unroll
            for (int h = 0; h < 2; ++h) x[st][h] = lds[(g * 16 + n_) * CPS + ((2 * (4 * st + kk) + h) ^ swz<D>(n_))];
        }
#pragma unroll
        for (int st = 0; st < ST; ++st) {
            u4 t[3];
            __builtin_amdgcn_sched_barrier(0);   // the terms of one step at a time: all at once do not fit the registers
            split8x3(x[st][0], x[st][1], t);
            // neighbours in the order do not depend on each other
            const u4 w0 = u3_lds[(st * 2) * 64 + lane], w1 = u3_lds[(st * 2 + 1) * 64 + lane];
            lo[0] = mfma_bf16(uf[st][0][0], t[2], lo[0]);
            lo[1] = mfma_bf16(uf[st][0][1], t[2], lo[1]);
            hi[0] = mfma_bf16(uf[st][0][0], t[0], hi[0]);
            hi[1] = mfma_bf16(uf[st][0][1], t[0], hi[1]);
            lo[0] = mfma_bf16(uf[st][1][0], t[1], lo[0]);
            lo[1] = mfma_bf16(uf[st][1][1], t[1], lo[1]);
            lo[0] = mfma_bf16(w0, t[0], lo[0]);
            lo[1] = mfma_bf16(w1, t[0], lo[1]);
            lo[0] = mfma_bf16(uf[st][0][0], t[1], lo[0]);
            lo[1] = mfma_bf16(uf[st][0][1], t[1], lo[1]);
            lo[0] = mfma_bf16(uf[st][1][0], t[0], lo[0]);
            lo[1] = mfma_bf16(uf[st][1][1], t[0], lo[1]);
        }
        u4 y[3];
        split8x3(hi[0] + lo[0], hi[1] + lo[1], y);
        float sq = 0.f;
#pragma unroll
        for (int st = 0; st < ST; ++st) {
            f4 rec[2];
            __builtin_amdgcn_sched_barrier(0);
            const u4* u = ud + 2 * st * 3 * 64 + lane;
            const u4 u1[2] = {u[0], u[192]}, u2[2] = {u[64], u[256]}, u3[2] = {u[128], u[320]};
            for (int h = 0; h < 2; ++h) rec[h] = mfma_bf16(u1[h], y[2], f4{0.f, 0.f, 0.f, 0.f});
            for (int h = 0; h < 2; ++h) rec[h] = mfma_bf16(u3[h], y[0], rec[h]);
            for (int h = 0; h < 2; ++h) rec[h] = mfma_bf16(u2[h], y[1], rec[h]);
            for (int h = 0; h < 2; ++h) rec[h] = mfma_bf16(u1[h], y[1], rec[h]);
            for (int h = 0; h < 2; ++h) rec[h] = mfma_bf16(u2[h], y[0], rec[h]);
            for (int h = 0; h < 2; ++h) rec[h] = mfma_bf16(u1[h], y[0], rec[h]);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float df = x[st][h][r] - rec[h][r];
                    if (!decltype(checked)::value || n_ * D + 32 * st + 8 * kk + 4 * h + r < end) sq = fmaf(df, df, sq);
                }
        }
        total += (double)sq;
    };

    // super-tiles: as in compress_fast_phase, no branch around a memory instruction
    SuperIter it;
    if (it.init(a.n_super, 1)) {
        const int64_t n_il = a.n_super / a.il * a.il;
        u4 regs[NL];
        auto load = [&](int64_t p, bool rows) {
            const bool group = p < n_il;
            const int64_t g = p / a.il, row = group ? g * a.il * NL + (p - g * a.il) : p * NL;
            const char* base = (const char*)a.in + row * 1024 + lane * 16;
            const int64_t stride = !rows ? 0 : group ? (int64_t)a.il * 1024 : 1024;
#pragma unroll
            for (int r = 0; r < NL; ++r) regs[r] = stream_load((const u4*)(base + r * stride));
        };
        int64_t cur = it.p;
        load(cur, true);
        bool more;
        do {
            wave_lds_sync();
#pragma unroll
            for (int r = 0; r < NL; ++r) park(r, regs[r]);
            more = it.advance();
            cur = more ? it.p : cur;
            load(cur, more);   // one row again when there is no next one
            wave_lds_sync();
            __builtin_amdgcn_s_setprio(3);
#pragma unroll
            for (int g = 0; g < G; ++g) residual(g, std::false_type{}, 0);
            __builtin_amdgcn_s_setprio(0);
        } while (more);
        drain_memory();
    }
    // the tiles behind them: bounds checked, the waves with the fewest super-tiles first
    for (int64_t t = a.n_super * G + (grid_waves() - 1 - grid_wave()); t < a.T; t += grid_waves()) {
        const int64_t base = t * TILE_SLICES * D;
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < NLT; ++r) {
            const int64_t e0 = base + (int64_t)(r * 64 + lane) * EPL;
            u4 v = {0u, 0u, 0u, 0u};
            if (e0 + EPL <= a.M) v = *(const u4*)((const char*)a.in + e0 * ES);
            else
#pragma unroll
                for (int i = 0; i < EPL; ++i)
                    if (e0 + i < a.M) {
                        if (BF16) v[i / 2] |= (unsigned int)((const unsigned short*)a.in)[e0 + i] << (16 * (i & 1));
                        else v[i & 3] = ((const unsigned int*)a.in)[e0 + i];
                    }
            park(r, v);
        }
        wave_lds_sync();
        residual(0, std::true_type{}, a.M - base);
    }
    // the work-group's sum, in a fixed order
    for (int o = 32; o > 0; o >>= 1) total += __shfl_xor(total, o, 64);
    if (lane == 0) red[wave] = total;
    __syncthreads();
    if (threadIdx.x == 0) a.part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// U as three bf16 terms, each the rounding to nearest of what the ones before leave, in the orders of the two products (zero
// past column k).
__global__ __launch_bounds__(256) void pack_loss_kernel(const float* U, unsigned short* out, int d, int k)
{
    const int half = d / 32 * 3 * 2 * 512;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < 2 * half; i += gridDim.x * 256) {
        const int j = i & 7, lane = (i >> 3) & 63, n = lane & 15, kk = lane >> 4, at = (i < half ? i : i - half) >> 9;
        int e, c, p;
        if (i < half) {
            const int st = at / 6;
            p = at / 2 % 3;
            e = 32 * st + 8 * kk + j;
            c = 16 * (at & 1) + n;
        } else {
            const int et = at / 3;
            p = at % 3;
            e = 32 * (et >> 1) + 8 * (n >> 2) + 4 * (et & 1) + (n & 3);
            c = 16 * (j >> 2) + 4 * kk + (j & 3);
        }
        unsigned int term = 0u;
        if (c < k) {
            float rest = U[(size_t)e * k + c];
            for (int t = 0; t <= p; ++t) {
                term = f32_to_bf16_rne(rest);
                rest -= bf16_to_f32(term);
            }
        }
        out[i] = (unsigned short)term;
    }
}

// ======================================================================================
// With several bases every wave would need its own copy of the second product's U; with up to 16 comps the fp32 pipe's products
// take half as long, less than the gradient takes to arrive (d = 128, k = 16: 112 us).
bool gvq_loss_split_shape(const gvq_basis* h) { return h->B == 1 && (h->d == 64 || h->d == 128) && h->k > 16 && h->k <= 32; }

size_t gvq_loss_split_pack_halves(int d) { return (size_t)d / 32 * 3 * 2 * 512 * 2; }

int gvq_launch_pack_loss(const gvq_basis* h, hipStream_t st)
{
    hipLaunchKernelGGL(pack_loss_kernel, dim3((unsigned)(gvq_loss_split_pack_halves(h->d) / 1024)), dim3(256), 0, st, h->d_U, h->d_Uls, h->d, h->k);
    GVQ_HIP(hipGetLastError());
    return GVQ_OK;
}

int gvq_launch_loss_split(const gvq_basis* h, const void* grad, int n_workers, double* part, int* parts, hipStream_t st)
{
    LossArgs a;
    const int G = 128 / h->d;
    a.in = grad; a.pack = (const u4*)h->d_Uls; a.mu = h->d_mu; a.part = part;
    a.M = h->M; a.n_workers = (float)n_workers;
    a.T = (h->S + TILE_SLICES - 1) / TILE_SLICES;
    a.n_super = gvq_opt_no_fast() & 1 ? 0 : h->M / (2048);
    a.il = gvq_opt_interleave() > 0 ? gvq_opt_interleave() : 64;
    const int64_t items = a.n_super + (a.T - a.n_super * G), want = (items + WAVES_PER_WG - 1) / WAVES_PER_WG;
    int64_t cap = (int64_t)h->num_cu * (gvq_opt_wg_per_cu() > 0 ? gvq_opt_wg_per_cu() : 2);
    if (cap > GVQ_LOSS_MAX_PARTS) cap = GVQ_LOSS_MAX_PARTS;
    const dim3 grid((unsigned)(want < cap ? want : cap)), threads(WG_THREADS);
    const bool bf = h->dtype == GVQ_BF16;
    if (h->d == 64) {
        if (bf) hipLaunchKernelGGL((loss_split_kernel<64, true>), grid, threads, 0, st, a);
        else hipLaunchKernelGGL((loss_split_kernel<64, false>), grid, threads, 0, st, a);
    } else {
        if (bf) hipLaunchKernelGGL((loss_split_kernel<128, true>), grid, threads, 0, st, a);
        else hipLaunchKernelGGL((loss_split_kernel<128, false>), grid, threads, 0, st, a);
    }
    GVQ_HIP(hipGetLastError());
    *parts = (int)grid.x;
    return GVQ_OK;
}
