// The symmetric eigensolver of the basis refresh (gvq_eigen.hip), as its callers see it.
#pragma once
#include "gvq_internal.h"

#define EIG_INF_BITS 0x7FF0000000000000ull
#define EIG_MOST_SOLVES 5   // most solves for an eigenvector; two do but for a start that hardly has it

struct EigenArgs {
    int n;                      // matrix size
    int k;                      // wanted eigenvectors
    const double* src;          // [B] matrices n x n, src_stride apart
    size_t src_stride;
    double* A;                  // [B][(n+1) n], A_stride apart: one spare row, then the working matrix / reflectors
    size_t A_stride;
    double* T;                  // [B][5 t_ld]: diagonal, off-diagonal, tau, p of even steps, p of odd steps
    int t_ld;
    const unsigned long long* norm;   // [B] largest |entry| of src, as bits
    double* eig;                // [B][eig_ld] eigenvalues in decreasing order
    int eig_ld;
    double* Z;                  // [B][k][n], Z_stride apart: eigenvectors
    size_t Z_stride;
    unsigned long long* xchg;   // n > 128: [B][4][2 n], then a word, xchg_stride apart: what the work-groups of one matrix tell each other
    size_t xchg_stride;
    double* wy;                 // n > 128: [B][(n - 2) / 32 rounded up][32][32], wy_stride apart: T of each block of reflectors
    size_t wy_stride;
    double* lu;                 // n > 128: factors, 5 n 64 doubles per 64 vectors
    int lanes;                  // bisect: lanes per eigenvalue
    int clamp;                  // 1: negative eigenvalues become 0
    int* solves;                // [B] most solves any vector took, GVQ_NO_CONVERGENCE if one did not converge
};

// A zero or a not finite matrix: nothing to decompose.
__device__ __forceinline__ bool eig_skip(unsigned long long norm) { return norm == 0 || norm >= EIG_INF_BITS; }

// Largest |entry| of a wave's lanes into a basis' norm, as the bits of a positive double (NaN and Inf sort above all).
__device__ __forceinline__ void eig_norm_max(double v, unsigned long long* norm)
{
    unsigned long long big = (unsigned long long)__double_as_longlong(fabs(v));
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long m = __shfl_xor(big, o, 64);
        if (m > big) big = m;
    }
    if ((threadIdx.x & 63) == 0 && big) atomicMax(norm, big);
}

// A number in (-1, 1) from two indices (murmur3's finaliser as the mixing step).
__device__ __forceinline__ double hash_unit(unsigned int i, unsigned int j)
{
    unsigned int x = i * 0x9E3779B1u ^ (j + 0x7F4A7C15u) * 0x85EBCA77u;
    x ^= x >> 16; x *= 0x85EBCA6Bu;
    x ^= x >> 13; x *= 0xC2B2AE35u;
    x ^= x >> 16;
    return ((double)x + 0.5) * (2.0 / 4294967296.0) - 1.0;
}

// The solver's arguments for a handle's covariance matrices; other matrices change what differs.
EigenArgs gvq_eigen_args(const gvq_basis* h);
// Eigenvalues and the k leading eigenvectors of B matrices; the vectors orthonormal to float64 precision if `ortho`,
// else as the inverse iteration leaves them.
// Matrices of up to GVQ_EIGEN_SMALL rows: `side` is done along with them.
struct SampleCov;
int gvq_launch_sym_eigen(const gvq_basis* h, EigenArgs a, bool ortho, hipStream_t st, const SampleCov* side = nullptr);
int gvq_launch_orthonormalise(const gvq_basis* h, double* Z, size_t Z_stride, int k, int n, hipStream_t st);
// h->d_eZ (k columns of d) -> h->d_U, with order and sign settled.
int gvq_launch_basis_out(const gvq_basis* h, hipStream_t st);
