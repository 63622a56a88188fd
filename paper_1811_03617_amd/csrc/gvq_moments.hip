// Moments of the basis refresh (GradiVeQ Section 2, PCA paragraph after Eq. 4): per basis, sum x and sum x x^T over the
// sample slices, in float64 (fp32 and bf16 inputs widen exactly and their products are exact in float64), for every
// slice length up to GVQ_MAX_D.  Many samples of slices longer than 64 elements: gvq_moments_int.hip.
//
// sum x x^T is a (d x n)(n x d) product with the samples as the contraction index, on v_mfma_f64_16x16x4_f64: A lane l =
// (row l%16, step l/16), B lane l = (step l/16, column l%16), result register r of lane l = (row 4r + l/16, column l%16).
// A and B have the same lane layout, so both operands of a pair of 16-element tiles come from the same place.
//
// What bounds it: the fp64 matrix pipe (77.5 TFLOP/s measured with nothing else), and while an fp64 product runs its SIMD
// issues no vector instruction at all (9 products alone 585 cycles, with 72 v_fma_f32 in between 905): every conversion,
// address and select is paid for in full.  So a work-group converts each number once, on its way into LDS, from where
// its four waves read float64 operands that need nothing done to them, and a lane's addresses are a uniform pointer
// plus an offset that never changes.  d = 24 and 16, 8 gradients of
// 10 M elements, 0.98 -> 0.15 ms and 0.23 -> 0.12 ms with the sum over the partials.
//
// Where the rest of the matrix pipe's time goes at d = 128 (9 700 to 10 700 cycles per block of 32 samples for two
// work-groups, 9 360 of them products): conversions and sums about 5 %, waiting at the block's barrier 5 %; at d = 768 the
// clock also falls to 2.25 GHz under the load.
//
// A slice is cut into np panels of at most 128 elements (NT tiles each).  A task is one sample chunk of either a panel
// with itself (tile pairs T1 <= T2 only, the matrix is symmetric) or of two different panels (all NT^2 pairs).
#include <math.h>

#include "gvq_moments.h"

typedef double d4 __attribute__((ext_vector_type(4)));
// a word of four numbers: slices of any length start anywhere, so it need not be aligned
typedef unsigned int mw4 __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned short mh4 __attribute__((ext_vector_type(4), aligned(2)));

template <int NT, bool BF16, bool OFF, int WAVE>
__device__ __forceinline__ void moments_task(const MomArgs& a, double* lds, int pa, int pb, int chunk, int chunks,
                                             double* out)
{
    using Sh = MomShape<NT, OFF>;
    constexpr int P0 = Sh::SPLIT ? WAVE * Sh::NACC : 0;
    constexpr int P1 = Sh::SPLIT ? (P0 + Sh::NACC < Sh::NPAIR ? P0 + Sh::NACC : Sh::NPAIR) : Sh::NPAIR;
    constexpr int NA = P1 - P0;
    constexpr int ES = BF16 ? 2 : 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, m = lane & 15, kk = lane >> 4;
    const int b = blockIdx.y, d = a.d;

    const int64_t full = a.M / d;
    int64_t lo = a.offs[b], hi = a.offs[b + 1] < full ? a.offs[b + 1] : full;
    if (hi < lo) hi = lo;
    const int64_t cnt = hi - lo;
    const int64_t j0 = lo + cnt * chunk / chunks, j1 = lo + cnt * (chunk + 1) / chunks;   // this task's samples
    const int64_t nblk = (j1 - j0 + Sh::NS - 1) / Sh::NS;

    // this thread's word of every row it moves
    const int c = tid % Sh::WORDS, r0 = tid / Sh::WORDS;
    const int panel = OFF && c >= 4 * NT ? pb : pa, p0 = panel * a.pw, p1 = p0 + a.pw < d ? p0 + a.pw : d;
    const int e = p0 + 4 * (OFF && c >= 4 * NT ? c - 4 * NT : c);   // its first element
    const bool active = r0 < Sh::RPS && e < p1;
    // the last word of a slice whose length is no multiple of 4 is read as the slice's last four numbers (read one by one
    // where the slice has not as many)
    const int e_read = !active ? 0 : d >= 4 && e > d - 4 ? d - 4 : e;
    const int shift = active ? e - e_read : 0;
    const unsigned int voff0 = (unsigned int)(e_read * ES), voff = voff0 + (unsigned int)(active ? r0 * d * ES : 0);

    float stage[Sh::U][4];
    int64_t left = nblk * a.L;   // blocks not yet requested
    int64_t rows_left = 0;       // rows of the current gradient from the next block on
    const char *base = nullptr, *src = nullptr;   // the next block, the block being requested
    int l = 0, rows_src = 0;     // next gradient, rows of the requested block inside the range
    unsigned long long taken = 0;
    const int step = Sh::RPS * d * ES;   // bytes from one of a thread's rows to the next
    auto next_block = [&]() {
        if (left == 0) return;   // the last block is requested again: loads stay unconditional
        --left;
        if (rows_left <= 0) {
            base = (const char*)a.grads.p[l] + j0 * d * ES;
            rows_left = j1 - j0;
            ++l;
        }
        rows_src = rows_left < Sh::NS ? (int)rows_left : Sh::NS;
        taken += rows_src;
        src = base;
        base += (int64_t)Sh::NS * d * ES;
        rows_left -= Sh::NS;
    };
    auto load_row = [&](int u) {
        // rows past the range read the block's first row instead, and are parked as zeros
        const bool whole = rows_src == Sh::NS;
        const char* p = whole ? src + (int64_t)u * step : src;
        unsigned int v = voff;
        if (!whole) v = u * Sh::RPS + r0 < rows_src ? voff + (unsigned int)(u * step) : voff0;
        if (NT == 1 && d < 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int at = i < d ? i * ES : 0;
                stage[u][i] = BF16 ? __uint_as_float((unsigned int)*(const unsigned short*)(p + v + at) << 16)
                                   : *(const float*)(p + v + at);
                if (i >= d) stage[u][i] = 0.f;
            }
        } else if (BF16) {
            const mh4 w = __builtin_nontemporal_load((const mh4*)(p + v));
#pragma unroll
            for (int i = 0; i < 4; ++i) stage[u][i] = __uint_as_float((unsigned int)w[i] << 16);
        } else {
            const mw4 w = OFF ? *(const mw4*)(p + v) : __builtin_nontemporal_load((const mw4*)(p + v));
#pragma unroll
            for (int i = 0; i < 4; ++i) stage[u][i] = __uint_as_float(w[i]);
        }
    };
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    const bool ragged = d >= 4 && (d & 3) != 0;
    double* mine_out = lds + r0 * Sh::ROW + 4 * c;
    auto park_row = [&](int at, int u, int rows) {
        if (!active) return;
        float* x = stage[u];
        if (ragged) {
            const float y0 = shift & 1 ? x[1] : x[0], y1 = shift & 1 ? x[2] : x[1], y2 = shift & 1 ? x[3] : x[2];
            const float y3 = shift & 1 ? 0.f : x[3];
            x[0] = shift & 2 ? y2 : y0;
            x[1] = shift & 2 ? y3 : y1;
            x[2] = shift & 2 ? 0.f : y2;
            x[3] = shift & 2 ? 0.f : y3;
        }
        if (rows < Sh::NS) {
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = u * Sh::RPS + r0 < rows ? x[i] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double v = (double)x[i];
            mine_out[at + u * Sh::RPS * Sh::ROW + i] = v;
            if (!OFF) sum[i] += v;
        }
    };

    d4 acc[NA > 0 ? NA : 1];
#pragma unroll
    for (int i = 0; i < NA; ++i) acc[i] = d4{0.0, 0.0, 0.0, 0.0};
    // the columns past a panel's elements stay zero
    for (int i = tid; i < 2 * Sh::BUF; i += 256) lds[i] = 0.0;

    const double* mine = lds + kk * Sh::ROW + m;
    auto fetch = [&](const double* buf, int g, double (&x)[Sh::TILES]) {
        static_for<Sh::TILES>([&](auto t) {
            constexpr int T = decltype(t)::value;
            if constexpr (Sh::needs(P0, P1, T)) x[T] = buf[4 * g * Sh::ROW + 16 * T];
        });
    };
    auto multiply = [&](const double (&x)[Sh::TILES]) {
        static_for<NA>([&](auto i) {
            constexpr int I = decltype(i)::value, R = Sh::row(P0 + I), C = Sh::col(P0 + I);
            acc[I] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[R], x[C], acc[I], 0, 0, 0);
        });
    };

    int64_t todo = left;
    const int g0 = Sh::SPLIT ? 0 : wave;
    __syncthreads();
    if (todo > 0) {
        next_block();
#pragma unroll
        for (int u = 0; u < Sh::U; ++u) load_row(u);
#pragma unroll
        for (int u = 0; u < Sh::U; ++u) park_row(0, u, rows_src);
        next_block();
#pragma unroll
        for (int u = 0; u < Sh::U; ++u) load_row(u);
    }
    for (int flip = 0; todo > 0; --todo, flip ^= 1) {
        __syncthreads();      // this block is parked; everyone is done with the buffer that takes the next one
        const int rows_parked = rows_src, next = (flip ^ 1) * Sh::BUF;
        const bool more = todo > 1;
        next_block();
        const double* buf = mine + flip * Sh::BUF;
        double x[2][Sh::TILES];   // a group's operands are read ahead of the products of the group before
        fetch(buf, g0, x[0]);
        // The next block is parked row by row between this one's products, each row's registers taking the block after
        // it.  Parked before the products, the two work-groups of a compute unit end up parking at the same time, with the
        // matrix pipe idle: whichever the pipe favours on one SIMD waits at the barrier for the SIMDs that favour the other.
        static_for<Sh::NGW>([&](auto gi) {
            constexpr int G = decltype(gi)::value;
            if constexpr (G + 1 < Sh::NGW) fetch(buf, g0 + (G + 1) * Sh::STRIDE, x[(G + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            multiply(x[G & 1]);
            static_for<Sh::U>([&](auto ui) {
                constexpr int V = decltype(ui)::value, AT = (V + 1) * Sh::NGW / (Sh::U + 1) - 1;
                if constexpr ((AT < 0 ? 0 : AT) == G) {
                    if (more) park_row(next, V, rows_parked);
                    load_row(V);
                }
            });
        });
    }

    __syncthreads();
    if constexpr (Sh::SPLIT) {
        double* o = out + P0 * 256 + lane;
        if (a.accumulate) {
#pragma unroll
            for (int i = 0; i < NA; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][r] += o[i * 256 + r * 64];
        }
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) o[i * 256 + r * 64] = acc[i][r];
    } else {
        // the four waves' sums, added in order
        for (int w = 0; w < 4; ++w) {
            if (wave == w) {
#pragma unroll
                for (int i = 0; i < NA; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int at = i * 256 + r * 64 + lane;
                        lds[at] = w == 0 ? acc[i][r] : lds[at] + acc[i][r];
                    }
            }
            __syncthreads();
        }
        for (int i = tid; i < NA * 256; i += 256) out[i] = a.accumulate ? out[i] + lds[i] : lds[i];
        __syncthreads();
    }
    if (OFF) return;
    // sums of x over the threads that share a word
    double* ss = lds;                                        // [RPS][16 NT]
    if (r0 < Sh::RPS) {
#pragma unroll
        for (int i = 0; i < 4; ++i) ss[r0 * 16 * NT + 4 * c + i] = sum[i];
    }
    __syncthreads();
    if (tid < 16 * NT) {
        double v = 0.0;
        for (int r = 0; r < Sh::RPS; ++r) v += ss[r * 16 * NT + tid];
        double* o = out + Sh::NPAIR * 256 + tid;
        *o = a.accumulate ? *o + v : v;
    }
    if (tid == 0 && pa == 0 && taken) atomicAdd(a.nsamp + b, taken);
}

template <int NT, bool BF16, bool OFF>
__device__ __forceinline__ void moments_waves(const MomArgs& a, double* lds, int pa, int pb, int chunk, int chunks, double* out)
{
    if constexpr (MomShape<NT, OFF>::SPLIT) {
        switch (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {   // uniform: the cases hold barriers
        case 0: moments_task<NT, BF16, OFF, 0>(a, lds, pa, pb, chunk, chunks, out); break;
        case 1: moments_task<NT, BF16, OFF, 1>(a, lds, pa, pb, chunk, chunks, out); break;
        case 2: moments_task<NT, BF16, OFF, 2>(a, lds, pa, pb, chunk, chunks, out); break;
        default: moments_task<NT, BF16, OFF, 3>(a, lds, pa, pb, chunk, chunks, out); break;
        }
    } else {
        moments_task<NT, BF16, OFF, 0>(a, lds, pa, pb, chunk, chunks, out);
    }
}

// Two work-groups per compute unit (LDS).  MULTI: more than one panel; the longer tasks start first.
template <int NT, bool BF16, bool MULTI>
__global__ __launch_bounds__(256, 2) void moments_kernel(MomArgs a)
{
    extern __shared__ __attribute__((aligned(16))) double mom_lds[];
    using Diag = MomShape<NT, false>;
    double* part = a.part + (size_t)blockIdx.y * a.part_basis;
    int task = blockIdx.x;
    if constexpr (MULTI) {
        using Off = MomShape<NT, true>;
        const int npairs = a.np * (a.np - 1) / 2;
        if (task < npairs * a.chunks_off) {
            const int chunk = task / npairs;       // the pairs of one chunk side by side: they share its samples
            int q = task - chunk * npairs, pa = 0;
            double* out = part + (size_t)a.np * a.chunks_diag * Diag::PART + ((size_t)q * a.chunks_off + chunk) * Off::PART;
            while (q >= a.np - 1 - pa) { q -= a.np - 1 - pa; ++pa; }
            moments_waves<NT, BF16, true>(a, mom_lds, pa, pa + 1 + q, chunk, a.chunks_off, out);
            return;
        }
        task -= npairs * a.chunks_off;
    }
    const int chunk = task / a.np, p = task - chunk * a.np;
    moments_waves<NT, BF16, false>(a, mom_lds, p, p, chunk, a.chunks_diag,
                                   part + ((size_t)p * a.chunks_diag + chunk) * Diag::PART);
}

// mom [B][d*d + d] (sum x x^T, both triangles, then sum x) from the partials: 64 entries per work-group, 16 threads per
// entry that each add a sixteenth of the chunks in order, then those sums in order.  (One thread per entry walking
// through all chunks took 0.5 ms for a 24 x 24 matrix in 512 chunks.)  Up to 16 chunks, with many bases, one thread per entry
// and a wave per work-group: the same sums (4000 bases of 16 x 16 48 -> 12 us).
template <int NT>
__global__ __launch_bounds__(1024) void moments_reduce_kernel(const double* part_all, size_t part_basis, double* mom, int d,
                                                              int np, int pw, int chunks_diag, int chunks_off)
{
    using Diag = MomShape<NT, false>;
    using Off = MomShape<NT, true>;
    __shared__ double sub[16][64];
    const int b = blockIdx.z, lane = threadIdx.x & 63, s = threadIdx.x >> 6;
    const int at = blockIdx.x * 64 + lane, parts = blockDim.x > 64 ? 16 : 1;
    int q = blockIdx.y;
    const bool off = q >= np;
    const int width = off ? Off::PART : Diag::PART, chunks = off ? chunks_off : chunks_diag;
    if (blockIdx.x * 64 >= width) return;   // the grid is as wide as the widest kind; uniform
    int pa = q, pb = q;
    const double* src = part_all + (size_t)b * part_basis;
    if (off) {
        q -= np;
        src += (size_t)np * chunks_diag * Diag::PART + (size_t)q * chunks_off * Off::PART;
        pa = 0;
        while (q >= np - 1 - pa) { q -= np - 1 - pa; ++pa; }
        pb = pa + 1 + q;
    } else {
        src += (size_t)q * chunks_diag * Diag::PART;
    }
    double v = 0.0;
    if (at < width) {
        const int c1 = (int)((int64_t)chunks * (s + 1) / parts);
#pragma unroll 8
        for (int c = (int)((int64_t)chunks * s / parts); c < c1; ++c) v += src[(size_t)c * width + at];
    }
    if (parts > 1) {
        sub[s][lane] = v;
        __syncthreads();
        if (s != 0) return;
        v = 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) v += sub[i][lane];
    }
    if (at >= width) return;
    double* o = mom + (size_t)b * ((size_t)d * d + d);
    const int npair = off ? Off::NPAIR : Diag::NPAIR;
    if (at >= npair * 256) {
        const int t = at - npair * 256, e = pa * pw + t;
        if (t < pw && e < d) o[(size_t)d * d + e] = v;
        return;
    }
    const int p = at >> 8, r = (at >> 6) & 3, ln = at & 63;
    const int t1 = off ? Off::row(p) : Diag::row(p), t2 = off ? Off::col(p) - NT : Diag::col(p);
    const int e1 = pa * pw + 16 * t1 + 4 * r + (ln >> 4), e2 = pb * pw + 16 * t2 + (ln & 15);
    if (e1 >= d || e2 >= d) return;
    o[(size_t)e1 * d + e2] = v;
    if (pa != pb || t1 != t2) o[(size_t)e2 * d + e1] = v;   // a tile with itself holds both of its triangles
}

// ======================================================================================
static int panels(int d) { return (d + 127) / 128; }
static int panel_tiles(int d) { const int np = panels(d); return (d + 16 * np - 1) / (16 * np); }

// Calls f with the shape's number of tiles per panel as a compile-time constant.
template <typename F>
static int by_tiles(int nt, F f)
{
    switch (nt) {
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    case 3: return f(std::integral_constant<int, 3>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 5: return f(std::integral_constant<int, 5>{});
    case 6: return f(std::integral_constant<int, 6>{});
    case 7: return f(std::integral_constant<int, 7>{});
    default: return f(std::integral_constant<int, 8>{});
    }
}

// Sample chunks per task: what finishes first, counting matrix-pipe time (a pair of tiles is 64 cycles per four
// samples) and about 6000 cycles to start a task and store its result, when every task that fits runs at once (two
// work-groups per compute unit) and a surplus queues for the slots.  Never fewer than one block of samples each.
size_t gvq_moments_plan(gvq_basis* h, int64_t longest)
{
    const int np = panels(h->d), poff = np * (np - 1) / 2;
    size_t basis = 0;
    by_tiles(panel_tiles(h->d), [&](auto nt) {
        using Diag = MomShape<decltype(nt)::value, false>;
        using Off = MomShape<decltype(nt)::value, true>;
        const double slots = 2.0 * h->num_cu, start = 6000.0;
        const double samples = 8.0 * (double)longest;   // of about eight gradients
        const double td = 64.0 * (Diag::SPLIT ? Diag::NACC : Diag::NPAIR / 4.0) * samples / 4.0;
        const double to = 64.0 * Off::NACC * samples / 4.0;
        const int64_t most_d = (longest + Diag::NS - 1) / Diag::NS, most_o = (longest + Off::NS - 1) / Off::NS;
        double best = 0.0;
        const int64_t top = poff ? most_o : most_d;
        for (int64_t c = 1; c <= top && c <= (int64_t)slots; ++c) {
            // as many diagonal chunks as make those tasks no longer than the others
            int64_t cd = poff ? (int64_t)ceil((double)c * td / to) : c;
            if (cd > most_d) cd = most_d;
            const double longest_task = poff ? fmax(to / c, td / cd) : td / c;
            const double tasks = (double)h->B * (np * cd + (poff ? poff * c : 0));
            const double work = (double)h->B * (np * td + poff * to) + tasks * start;
            const double t = tasks <= slots ? longest_task + start : work / slots + 0.5 * longest_task;
            if (best == 0.0 || t < best) { best = t; h->mom_diag = (int)cd; h->mom_off = poff ? (int)c : 0; }
            if (tasks > 3.0 * slots) break;   // past what could help, and the partials take memory (75 KB a task at d = 128)
        }
        basis = (size_t)np * h->mom_diag * Diag::PART + (size_t)poff * h->mom_off * Off::PART;
        return GVQ_OK;
    });
    if (gvq_moments_int_shape(h)) {
        const size_t other = gvq_moments_int_plan(h, longest);
        if (other > basis) basis = other;
    }
    return basis;
}

int gvq_launch_moments_reduce(const gvq_basis* h, int nt, int np, int pw, int chunks_diag, int chunks_off, hipStream_t st)
{
    return by_tiles(nt, [&](auto t) -> int {
        constexpr int NT = decltype(t)::value;
        const int width = np > 1 ? MomShape<NT, true>::PART : MomShape<NT, false>::PART;
        hipLaunchKernelGGL((moments_reduce_kernel<NT>), dim3((unsigned)((width + 63) / 64), (unsigned)(np + np * (np - 1) / 2), (unsigned)h->B),
                           dim3(chunks_diag > 16 || chunks_off > 16 ? 1024 : 64), 0, st, h->d_part, h->mom_part, h->d_mom, h->d,
                           np, pw, chunks_diag, chunks_off);
        GVQ_HIP(hipGetLastError());
        return GVQ_OK;
    });
}

int gvq_launch_moments(gvq_basis* h, const void* const* grads, int L, hipStream_t st)
{
    if (gvq_moments_int_takes(h, L)) return gvq_launch_moments_int(h, grads, L, st);
    MomArgs a;
    a.offs = h->d_offs; a.M = h->M; a.d = h->d; a.np = panels(h->d); a.pw = 16 * panel_tiles(h->d);
    a.chunks_diag = h->mom_diag; a.chunks_off = h->mom_off;
    a.part = h->d_part; a.part_basis = h->mom_part; a.nsamp = h->d_nsamp;
    const int poff = a.np * (a.np - 1) / 2;
    return by_tiles(panel_tiles(h->d), [&](auto nt) -> int {
        constexpr int NT = decltype(nt)::value;
        using Diag = MomShape<NT, false>;
        using Off = MomShape<NT, true>;
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
                hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, a);
                GVQ_HIP(hipGetLastError());
            }
            return GVQ_OK;
        };
        int rc;
        const bool bf = h->dtype == GVQ_BF16;
        if constexpr (NT >= 5) {
            constexpr int lds = Diag::LDS > Off::LDS ? Diag::LDS : Off::LDS;
            if (a.np > 1) rc = bf ? launch(moments_kernel<NT, true, true>, lds) : launch(moments_kernel<NT, false, true>, lds);
            else rc = bf ? launch(moments_kernel<NT, true, false>, Diag::LDS) : launch(moments_kernel<NT, false, false>, Diag::LDS);
        } else {
            rc = bf ? launch(moments_kernel<NT, true, false>, Diag::LDS) : launch(moments_kernel<NT, false, false>, Diag::LDS);
        }
        if (rc != GVQ_OK) return rc;
        return gvq_launch_moments_reduce(h, NT, a.np, a.pw, a.chunks_diag, a.chunks_off, st);
    });
}
