// Basis refresh kernels for gfx950 (GradiVeQ Section 2, PCA paragraph after Eq. 4):
//   1. moments:  per basis, sum x and sum x x^T over the sample slices, in float64: gvq_moments.hip, and here those of
//                a first-slice refresh from many samples (from few: gvq_sample.hip);
//   2. covariance and its eigendecomposition: gvq_eigen.hip.
#include "gvq_internal.h"

__device__ __forceinline__ float load_elem(const void* g, bool bf16, int64_t idx)
{
    if (bf16) return __uint_as_float((unsigned int)((const unsigned short*)g)[idx] << 16);
    return ((const float*)g)[idx];
}

// Section 3, "compressor reuse": moments of the first slice of every basis only -- L samples of d
// numbers per basis, a few KB; one thread per matrix entry.  For more samples than gvq_sample.hip takes.
__global__ void first_slice_moments_kernel(gvq_ptrs grads, int L, const int64_t* offs, int64_t M, int d, int bf16,
                                           int accumulate, double* mom, unsigned long long* nsamp)
{
    const int b = blockIdx.x, W = d * d + d;
    const int64_t j = offs[b];
    const bool ok = (j + 1) * d <= M;     // the first slice must be a full one
    if (blockIdx.y == 0 && threadIdx.x == 0 && ok) atomicAdd(nsamp + b, (unsigned long long)L);
    for (int i = blockIdx.y * blockDim.x + threadIdx.x; i < W; i += gridDim.y * blockDim.x) {
        const int r = i < d * d ? i / d : i - d * d, c = i < d * d ? i % d : -1;
        double acc = 0.0;
        if (ok)
            for (int l = 0; l < L; ++l) {
                const double xr = (double)load_elem(grads.p[l], bf16 != 0, j * d + r);
                acc += c >= 0 ? xr * (double)load_elem(grads.p[l], bf16 != 0, j * d + c) : xr;
            }
        double* o = mom + (size_t)b * W + i;
        *o = accumulate ? *o + acc : acc;
    }
}

// Section 3, Eq. (5): smallest k with (eig[0] + .. + eig[k-1]) / sum(eig) >= 1 - lambda; one
// thread per basis, partial sums from the largest eigenvalue down, in double.
__global__ void select_k_kernel(const double* eig, int d, int B, double lambda, int* k_out)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const double* e = eig + (size_t)b * d;
    double total = 0.0;
    for (int i = 0; i < d; ++i) total += e[i];
    int k = d;
    if (!(total > 0.0)) {
        k = 1;
    } else {
        double cum = 0.0;
        for (int i = 1; i <= d; ++i) {
            cum += e[i - 1];
            if (cum / total >= 1.0 - lambda) { k = i; break; }
        }
    }
    k_out[b] = k;
}

int gvq_launch_select_k(const gvq_basis* h, double lambda, hipStream_t st)
{
    hipLaunchKernelGGL(select_k_kernel, dim3((h->B + 63) / 64), dim3(64), 0, st, h->d_eig, h->d, h->B, lambda,
                       h->d_ksel);
    GVQ_HIP(hipGetLastError());
    return GVQ_OK;
}

// ======================================================================================
// A fill kernel rather than a memset, so that a fit can be captured into a HIP graph.
__global__ void zero_counts_kernel(unsigned long long* p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

int gvq_launch_fit(gvq_basis* h, const void* const* grads, int L, bool first_slice_only, hipStream_t st)
{
    const int d = h->d, W = d * d + d;
    hipLaunchKernelGGL(zero_counts_kernel, dim3((2 * h->B + 255) / 256), dim3(256), 0, st, h->d_nsamp, 2 * h->B);
    GVQ_HIP(hipGetLastError());
    if (first_slice_only && gvq_sample_shape(d, L)) {
        const int rc = gvq_launch_fit_samples(h, grads, L, st);
        return rc != GVQ_OK ? rc : gvq_launch_pack(h, st);
    }
    if (first_slice_only) {
        for (int l0 = 0; l0 < L; l0 += GVQ_MAX_PTRS) {
            gvq_ptrs p;
            const int n = L - l0 < GVQ_MAX_PTRS ? L - l0 : GVQ_MAX_PTRS;
            for (int i = 0; i < n; ++i) p.p[i] = grads[l0 + i];
            hipLaunchKernelGGL(first_slice_moments_kernel, dim3(h->B, (W + 4095) / 4096), dim3(256), 0, st, p, n,
                               h->d_offs, h->M, d,
                               h->dtype == GVQ_BF16 ? 1 : 0, l0 > 0 ? 1 : 0, h->d_mom, h->d_nsamp);
            GVQ_HIP(hipGetLastError());
        }
    } else {
        const int rc = gvq_launch_moments(h, grads, L, st);
        if (rc != GVQ_OK) return rc;
    }

    const int rc = gvq_launch_eigen(h, true, st);
    return rc != GVQ_OK ? rc : gvq_launch_pack(h, st);
}
