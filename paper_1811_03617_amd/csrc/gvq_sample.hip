// Basis refresh from the first slice of every basis (GradiVeQ Section 3, "compressor reuse": L time samples of one slice,
// slices of hundreds of elements).
//
// The covariance C = Xc^T Xc / L (Xc: the L centred samples as rows) has rank < L, and its non-zero eigenpairs are those
// of the L x L matrix K = Xc Xc^T / L: K v = lambda v  =>  C (Xc^T v) = lambda (Xc^T v).  With 2 L <= d the eigensolver
// therefore runs on K, and the kept directions are Xc^T v, made orthonormal.  Directions beyond the rank of the data
// (eigenvalue <= 1e-12 of the largest) are not determined by it: random vectors take their place and the same
// orthonormalisation completes U.  C itself is formed for gvq_basis_export_cov only, by compute units that the
// tridiagonalisation of K leaves idle.
//
// One work-group per basis did all of this in one kernel before (26 bases, d = 768, k = 96, L = 100: 17.8 ms, and
// 1.4 ms for the moments, which read two elements from memory per product); spread over the chip in products on the
// fp64 matrix pipe the same refresh takes 0.8 ms.
#include "gvq_sample.h"

typedef double d4 __attribute__((ext_vector_type(4)));

struct SampleArgs {
    gvq_ptrs grads[GVQ_SAMPLE_MAX_L / GVQ_MAX_PTRS];
    int L;
    const int64_t* offs;
    int64_t M;
    int d, k, bf16;
    double* X;             // [B][L][d], x_stride apart: the centred samples
    size_t x_stride;
    double* K;             // [B][L][L], x_stride apart
    const double* V;       // [B][min(k, L)][L], x_stride apart: eigenvectors of K
    float* mu;             // [B][d]
    double* Z;             // [B][k][d]
    const double* eig;     // [B][d]
    unsigned long long* nsamp;   // [B] samples, then [B] norms
    int B;
    int* solves;           // [B]
};

__device__ __forceinline__ float load_elem(const void* g, bool bf16, int64_t idx)
{
    if (bf16) return __uint_as_float((unsigned int)((const unsigned short*)g)[idx] << 16);
    return ((const float*)g)[idx];
}

// mu and the centred samples: 64 elements per work-group, its four waves a quarter of the samples each, which are read once
// and together (26 bases of d = 768, L = 100: 30 -> 25 us against eight at a time, twice).
__global__ __launch_bounds__(256) void centre_kernel(SampleArgs a)
{
    __shared__ double part[4][64];
    const int b = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + lane;
    const int64_t j = a.offs[b];
    const bool full = (j + 1) * a.d <= a.M;   // the first slice must be a full one
    const int l0 = a.L * wave / 4, l1 = a.L * (wave + 1) / 4;
    float v[GVQ_SAMPLE_MAX_L / 4];
    const int64_t at = full ? j * a.d + (e < a.d ? e : a.d - 1) : 0;
    static_assert(GVQ_SAMPLE_MAX_L / 4 == 32, "two halves of 16");
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        if (l0 + 16 * half >= l1) break;
#pragma unroll
        for (int i = 16 * half; i < 16 * half + 16; ++i) {
            const int l = l0 + i < l1 ? l0 + i : l1 - 1;
            v[i] = full ? load_elem(a.grads[l / GVQ_MAX_PTRS].p[l % GVQ_MAX_PTRS], a.bf16 != 0, at) : 0.f;
        }
    }
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < GVQ_SAMPLE_MAX_L / 4; ++i)
        if (l0 + i < l1) s += (double)v[i];
    part[wave][lane] = s;
    __syncthreads();
    // true division: identical samples then give exactly C = 0
    const double mean = ((part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane])) / (double)a.L;
    double* X = a.X + (size_t)b * a.x_stride;
    if (e < a.d) {
#pragma unroll
        for (int i = 0; i < GVQ_SAMPLE_MAX_L / 4; ++i)
            if (l0 + i < l1) X[(size_t)(l0 + i) * a.d + e] = full ? (double)v[i] - mean : 0.0;
        if (wave == 0) a.mu[(size_t)b * a.d + e] = (float)mean;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.nsamp[b] = full ? (unsigned long long)a.L : 0ull;
        a.solves[b] = 0;   // the solver raises it
    }
}

// v_mfma_f64_16x16x4_f64: A lane l = (row l%16, step l/16), B lane l = (step l/16, column l%16), result register r of
// lane l = (row 4r + l/16, column l%16).

// K = X X^T / L, one 16 x 16 block (and its mirror image) per work-group, its four waves a quarter of the elements each.
__global__ __launch_bounds__(256) void sample_gram_kernel(SampleArgs a)
{
    __shared__ double part[3][256];
    const int b = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = lane & 15, kk = lane >> 4;
    const int nt = (a.L + 15) / 16;
    int t1 = 0, rem = blockIdx.x;
    while (rem >= nt - t1) { rem -= nt - t1; ++t1; }
    const int t2 = t1 + rem;
    const double* X = a.X + (size_t)b * a.x_stride;
    const int r1 = 16 * t1 + m, r2 = 16 * t2 + m;
    const double* x1 = X + (size_t)(r1 < a.L ? r1 : 0) * a.d;
    const double* x2 = X + (size_t)(r2 < a.L ? r2 : 0) * a.d;
    const int steps = (a.d + 3) / 4, s0 = steps * wave / 4, s1 = steps * (wave + 1) / 4;
    d4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int s = s0; s < s1; s += 8) {
        double va[8], vb[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = 4 * (s + u) + kk, at = e < a.d ? e : a.d - 1;   // unconditional loads, all eight in flight
            const bool in = s + u < s1 && e < a.d;
            const double la = x1[at], lb = x2[at];
            va[u] = in && r1 < a.L ? la : 0.0;
            vb[u] = in && r2 < a.L ? lb : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(va[u], vb[u], acc, 0, 0, 0);
    }
    if (wave > 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) part[wave - 1][64 * r + lane] = acc[r];
    }
    __syncthreads();
    if (wave > 0) return;
    double* K = a.K + (size_t)b * a.x_stride;
    double big = 0.0, bad = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const double v = ((acc[r] + part[0][64 * r + lane]) + (part[1][64 * r + lane] + part[2][64 * r + lane])) / (double)a.L;
        const int row = 16 * t1 + 4 * r + kk, col = 16 * t2 + m;
        if (row < a.L && col < a.L) {
            K[(size_t)row * a.L + col] = v;
            if (t1 != t2) K[(size_t)col * a.L + row] = v;
            big = fmax(big, fabs(v));
            if (v != v) bad = v;   // fmax drops a NaN
        }
    }
    eig_norm_max(bad != bad ? bad : big, a.nsamp + a.B + b);
}

// C = X^T X / L in 64 x 64 blocks, one wave each (and its mirror image).
__global__ __launch_bounds__(64) void sample_cov_kernel(SampleCov c, unsigned long long* norm)
{
    const double v = sample_cov_block(c, blockIdx.x);
    eig_norm_max(v, norm + blockIdx.x / c.blocks);
}

// The raw directions X^T v (random numbers where the data determines none), 16 columns x 64 elements per wave.
__global__ __launch_bounds__(256) void sample_lift_kernel(SampleArgs a)
{
    const int b = blockIdx.z, lane = threadIdx.x & 63, m = lane & 15, kk = lane >> 4, d = a.d;
    if (eig_skip(a.nsamp[a.B + b])) return;
    const int c0 = blockIdx.y * 16, e0 = blockIdx.x * 256 + (threadIdx.x >> 6) * 64;
    const int kv = a.k < a.L ? a.k : a.L;
    const double* X = a.X + (size_t)b * a.x_stride;
    const double* V = a.V + (size_t)b * a.x_stride;
    const double* eig = a.eig + (size_t)b * d;
    d4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = d4{0.0, 0.0, 0.0, 0.0};
    const double* v = V + (size_t)(c0 + m < kv ? c0 + m : kv - 1) * a.L;
    for (int l = 0; l < a.L; l += 8) {
        double va[2], vb[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int at = l + 4 * u + kk, in = at < a.L ? at : a.L - 1;   // unconditional loads
            va[u] = v[in];
            if (at >= a.L || c0 + m >= kv) va[u] = 0.0;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int e = e0 + 16 * t + m;
                vb[u][t] = X[(size_t)in * d + (e < d ? e : d - 1)];
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(va[u], vb[u][t], acc[t], 0, 0, 0);
    }
    const double floor_eig = 1e-12 * eig[0];
    double* Z = a.Z + (size_t)b * a.k * d;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = c0 + 4 * r + kk;
        if (c >= a.k) continue;
        const bool determined = c < kv && eig[c] > floor_eig;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int e = e0 + 16 * t + m;
            if (e < d) Z[(size_t)c * d + e] = determined ? acc[t][r] : hash_unit((unsigned int)e, (unsigned int)c);
        }
    }
}

// ======================================================================================
// The centred samples fit the eigensolver's work space (d + 1) d.
bool gvq_sample_shape(int d, int L) { return L >= 2 && L <= GVQ_SAMPLE_MAX_L && L <= d; }

// The small-matrix route: samples, K with its reflectors and K's vectors fit that work space together
// (L d + (L + 1) L + L min(k, L) <= (d + 1) d).
static bool gram_shape(int d, int L) { return 2 * L <= d; }

int gvq_launch_fit_samples(const gvq_basis* h, const void* const* grads, int L, hipStream_t st)
{
    const int d = h->d, k = h->k, B = h->B;
    SampleArgs a;
    for (int l = 0; l < L; ++l) a.grads[l / GVQ_MAX_PTRS].p[l % GVQ_MAX_PTRS] = grads[l];
    EigenArgs e = gvq_eigen_args(h);
    a.L = L; a.offs = h->d_offs; a.M = h->M; a.d = d; a.k = k; a.bf16 = h->dtype == GVQ_BF16 ? 1 : 0;
    a.X = h->d_eA; a.x_stride = e.A_stride;
    double* work = h->d_eA + (size_t)L * d;       // K's work space: a spare row, then K
    a.K = work + L;
    a.V = work + (size_t)(L + 1) * L;
    a.mu = h->d_mu; a.Z = h->d_eZ; a.eig = h->d_eig; a.nsamp = h->d_nsamp; a.B = B;
    a.solves = h->d_solves;
    const bool gram = gram_shape(d, L);
    hipLaunchKernelGGL(centre_kernel, dim3((unsigned)((d + 63) / 64), B), dim3(256), 0, st, a);
    GVQ_HIP(hipGetLastError());
    const int ng = (d + 63) / 64, blocks = ng * (ng + 1) / 2;
    const SampleCov cov{a.X, a.x_stride, h->d_cov, L, d, blocks, B * blocks};
    if (!gram) {
        hipLaunchKernelGGL(sample_cov_kernel, dim3((unsigned)cov.total), dim3(64), 0, st, cov, a.nsamp + B);
        GVQ_HIP(hipGetLastError());
        return gvq_launch_eigen(h, false, st);
    }
    const int nt = (L + 15) / 16;
    hipLaunchKernelGGL(sample_gram_kernel, dim3((unsigned)(nt * (nt + 1) / 2), B), dim3(256), 0, st, a);
    GVQ_HIP(hipGetLastError());
    e.n = L; e.k = k < L ? k : L; e.clamp = 1;   // a negative eigenvalue of K is rounding noise around zero
    e.src = a.K; e.src_stride = e.A_stride;
    e.A = work;
    e.Z = const_cast<double*>(a.V); e.Z_stride = e.A_stride;
    int rc = gvq_launch_sym_eigen(h, e, false, st, &cov);
    if (rc != GVQ_OK) return rc;
    hipLaunchKernelGGL(sample_lift_kernel, dim3((unsigned)((d + 255) / 256), (unsigned)((k + 15) / 16), B), dim3(256), 0, st, a);
    GVQ_HIP(hipGetLastError());
    rc = gvq_launch_orthonormalise(h, h->d_eZ, (size_t)k * d, k, d, st);
    return rc != GVQ_OK ? rc : gvq_launch_basis_out(h, st);
}
