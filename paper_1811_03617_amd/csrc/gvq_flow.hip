// Plans, packed U and launches of the codec kernels of gvq_flow.h.
#include "gvq_flow.h"

static FlowPlan compress_plan(const gvq_basis* h) { return flow_compress_plan(h->d, h->k); }
static FlowPlan decompress_plan(const gvq_basis* h) { return flow_decompress_plan(h->d, h->k); }

static flow_kernel compress_kernel(const gvq_basis* h, const FlowPlan& p)
{
    return h->dtype == GVQ_BF16 ? gvq_flow_compress_bf16(p) : gvq_flow_compress_f32(p);
}

static FlowShape shape_of(const gvq_basis* h, bool bf16) { return FlowShape{h->d, h->k, h->B, bf16, h->S, h->num_cu}; }

bool gvq_flow_takes_compress(const gvq_basis* h) { return h->d_Ufc && flow_takes_compress(shape_of(h, h->dtype == GVQ_BF16)); }
bool gvq_flow_takes_decompress(const gvq_basis* h, bool out_bf16) { return h->d_Ufd && flow_takes_decompress(shape_of(h, out_bf16)); }

int gvq_flow_alloc(gvq_basis* h)
{
    const FlowPlan c = compress_plan(h), e = decompress_plan(h);
    const size_t B = (size_t)h->B;
    auto allow_lds = [](flow_kernel kern) {   // the most any plan of the kernel takes
        return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    };
    // nothing for a direction that no call takes here
    if (flow_takes_compress(shape_of(h, h->dtype == GVQ_BF16))) {
        h->flow_rows_c = c.rows;
        GVQ_HIP(allow_lds(compress_kernel(h, c)));
        GVQ_HIP(hipMalloc((void**)&h->d_Ufc, sizeof(u4) * B * c.words));
    }
    if (flow_takes_decompress(shape_of(h, false)) || flow_takes_decompress(shape_of(h, true))) {
        h->flow_rows_d = e.rows;
        GVQ_HIP(allow_lds(gvq_flow_decompress(e)));
        GVQ_HIP(hipMalloc((void**)&h->d_Ufd, sizeof(u4) * B * e.words));
    }
    if (h->B == 1) return GVQ_OK;
    if (h->flow_rows_c) h->flow_rows_c = flow_tile_rows(h->h_offs, (int64_t)B, c.rows, 16 * (c.waves / c.wn), (int64_t)h->num_cu * c.per_cu);
    if (h->flow_rows_d) h->flow_rows_d = flow_tile_rows(h->h_offs, (int64_t)B, e.rows, 16 * (e.waves / e.wn), (int64_t)h->num_cu * e.per_cu);
    // first tile of each basis, and the tiles themselves, for compress and then for decompress
    h->h_ftile = (int64_t*)malloc(sizeof(int64_t) * 2 * (B + 1));
    if (!h->h_ftile) return GVQ_ENOMEM;
    for (int which = 0; which < 2; ++which) {
        const int rows = which ? h->flow_rows_d : h->flow_rows_c;
        int64_t* t = h->h_ftile + which * (B + 1);
        t[0] = which ? h->h_ftile[B] : 0;
        for (size_t b = 0; b < B; ++b) t[b + 1] = t[b] + (rows ? (h->h_offs[b + 1] - h->h_offs[b] + rows - 1) / rows : 0);
    }
    const int64_t n = h->h_ftile[2 * B + 1];
    if (n == 0) return GVQ_OK;
    FlowTile* tiles = (FlowTile*)malloc(sizeof(FlowTile) * (size_t)n);
    if (!tiles) return GVQ_ENOMEM;
    FlowTile* t = tiles;
    for (int which = 0; which < 2; ++which) {
        const int rows = which ? h->flow_rows_d : h->flow_rows_c;
        for (size_t b = 0; rows && b < B; ++b)
            for (int64_t s = h->h_offs[b], end = h->h_offs[b + 1]; s < end; s += rows)
                *t++ = FlowTile{s, (int)(end - s < rows ? end - s : rows), (int)b};
    }
    hipError_t err = hipMalloc(&h->d_ftile, sizeof(FlowTile) * (size_t)n);
    if (err == hipSuccess) err = hipMemcpy(h->d_ftile, tiles, sizeof(FlowTile) * (size_t)n, hipMemcpyHostToDevice);
    free(tiles);
    return err == hipSuccess ? GVQ_OK : gvq_hip_fail(err, "table of tiles");
}

// One 128-bit word of either packed copy per thread.  rows_of: what the A operand's rows are (comps for compress, elements
// for decompress), `len` the length of the contraction, `steps` its steps of 32, tiles rows of tiles.  Positions past the
// last whole word hold the last four numbers' places: those already met are zero.
template <bool EXACT, bool COMPRESS>
__global__ __launch_bounds__(256) void pack_flow_kernel(const float* U, u4* out, int d, int k, int steps, int tiles)
{
    const int b = blockIdx.y, len = COMPRESS ? d : k, rows = COMPRESS ? k : d, words = (len + 3) / 4;
    const size_t n = (size_t)tiles * steps * 128;
    const float* Ub = U + (size_t)b * d * k;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const int lane = (int)(i & 63), m = lane & 15, kk = lane >> 4, w = (int)(i >> 6) & 1;
        const int st = (int)((i >> 7) % steps), row = 16 * (int)((i >> 7) / steps) + m;
        auto at = [&](int pos) -> float {
            int e = pos;
            if (pos >= 4 * words) return 0.f;
            if (pos >= 4 * (words - 1)) {
                e = len < 4 ? pos : len - 4 + (pos & 3);
                if (e < 4 * (words - 1) || e >= len) return 0.f;
            }
            if (row >= rows) return 0.f;
            return COMPRESS ? Ub[(size_t)e * k + row] : Ub[(size_t)row * k + e];
        };
        u4 v;
        if (EXACT) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = __float_as_uint(at(32 * st + 16 * w + 4 * kk + j));
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                unsigned int half[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float u = at(32 * st + 8 * kk + 2 * j + q);
                    const unsigned int t0 = f32_to_bf16_rne(u);
                    half[q] = w == 0 ? t0 : f32_to_bf16_rne(u - bf16_to_f32(t0));
                }
                v[j] = half[0] | half[1] << 16;
            }
        }
        out[(size_t)b * n + i] = v;
    }
}

int gvq_launch_pack_flow(const gvq_basis* h, hipStream_t st)
{
    const bool exact = flow_exact(h->d, h->k);
    auto grid = [&](size_t words) { return dim3((unsigned)(words / 256 < 64 ? (words + 255) / 256 : 64), (unsigned)h->B); };
    if (h->d_Ufc) {
        const FlowPlan p = compress_plan(h);
        auto kern = exact ? pack_flow_kernel<true, true> : pack_flow_kernel<false, true>;
        hipLaunchKernelGGL(kern, grid(p.words), dim3(256), 0, st, h->d_U, (u4*)h->d_Ufc, h->d, h->k, p.steps, p.wn * p.ntw);
        GVQ_HIP(hipGetLastError());
    }
    if (h->d_Ufd) {
        const FlowPlan p = decompress_plan(h);
        auto kern = exact ? pack_flow_kernel<true, false> : pack_flow_kernel<false, false>;
        hipLaunchKernelGGL(kern, grid(p.words), dim3(256), 0, st, h->d_U, (u4*)h->d_Ufd, h->d, h->k, p.kst, p.wn * p.etw);
        GVQ_HIP(hipGetLastError());
    }
    return GVQ_OK;
}

static int launch_flow(const gvq_basis* h, flow_kernel kern, const FlowPlan& p, FlowArgs& a, int which, int64_t first_slice,
                       int64_t n_slices, hipStream_t st)
{
    a.mu = h->d_mu; a.M = h->M; a.S = h->S; a.B = h->B; a.d = h->d; a.k = h->k;
    a.seg_begin = first_slice; a.seg_end = first_slice + n_slices;
    a.wn = p.wn; a.upack_stride = p.words;
    const int per_cu = gvq_opt_wg_per_cu() > 0 ? gvq_opt_wg_per_cu() : p.per_cu;
    const int64_t cap = (int64_t)h->num_cu * per_cu;
    const int64_t range[2] = {0, n_slices};
    a.rows = h->B > 1 ? (which ? h->flow_rows_d : h->flow_rows_c) : flow_tile_rows(range, 1, p.rows, 16 * (p.waves / p.wn), cap);
    a.tiles = (const FlowTile*)h->d_ftile;
    a.run = 1;
    a.t0 = 0;
    a.t1 = (n_slices + a.rows - 1) / a.rows;
    if (h->B > 1) {
        const int64_t* ft = h->h_ftile + which * (h->B + 1);
        auto tile_of = [&](int64_t s) {
            int lo = 0, hi = h->B;
            while (hi - lo > 1) {
                const int mid = (lo + hi) / 2;
                if (h->h_offs[mid] <= s) lo = mid; else hi = mid;
            }
            return ft[lo] + (s - h->h_offs[lo]) / a.rows;
        };
        a.t0 = tile_of(first_slice);
        a.t1 = tile_of(first_slice + n_slices - 1) + 1;
        // (24 bases, compress: d = 160 60.0 us with runs of 4, 57.5 with 8, 63.4 in one run; decompress 67.9, 80.3, 78.8)
        a.run = flow_run(a.t1 - a.t0, cap, which == 0 && p.ntw * p.steps > 2 ? 8 : 4);
        if (gvq_opt_run_tiles() > 0) a.run = gvq_opt_run_tiles();
    }
    const int64_t runs = (a.t1 - a.t0 + a.run - 1) / a.run;
    const int grid = (int)(runs < cap ? runs : cap);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * p.waves), p.lds(a.rows), st, a);
    GVQ_HIP(hipGetLastError());
    return GVQ_OK;
}

int gvq_launch_compress_flow(const gvq_basis* h, const void* grad, int n_workers, int64_t first_slice, int64_t n_slices,
                             const float* comp_in, float* out, hipStream_t st)
{
    const FlowPlan p = compress_plan(h);
    FlowArgs a;
    a.in = grad; a.out = out; a.acc_in = comp_in; a.Upack = (const u4*)h->d_Ufc; a.n_workers = (float)n_workers;
    a.words = (h->d + 3) / 4; a.by_words = flow_divisor(a.words); a.by_out = 0; a.out_bf16 = 0;
    a.whole = h->M / h->d;
    // as for the register-resident kernels: results that are summed next stay in the last-level cache if they all fit it
    a.keep = !comp_in && (int64_t)n_workers * n_slices * h->k * 4 <= (224ll << 20);
    return launch_flow(h, compress_kernel(h, p), p, a, 0, first_slice, n_slices, st);
}

int gvq_launch_decompress_flow(const gvq_basis* h, const float* comp, int64_t first_slice, int64_t n_slices, void* out,
                               bool out_bf16, hipStream_t st)
{
    const FlowPlan p = decompress_plan(h);
    FlowArgs a;
    a.in = comp; a.out = out; a.acc_in = nullptr; a.Upack = (const u4*)h->d_Ufd; a.n_workers = 1.f;
    a.words = (h->k + 3) / 4; a.by_words = flow_divisor(a.words); a.out_bf16 = out_bf16 ? 1 : 0; a.keep = 0;
    a.by_out = flow_divisor(flow_out_row(h->d) == h->d ? 1 : out_bf16 ? h->d / 8 : h->d / 4);
    a.whole = h->k >= 4 ? h->S : 0;
    return launch_flow(h, gvq_flow_decompress(p), p, a, 1, first_slice, n_slices, st);
}
