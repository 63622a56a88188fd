// Eigensolver of the basis refresh (GradiVeQ Section 2, PCA paragraph: "applies SVD to obtain the eigen matrix U
// and eigen vector s"), float64, any slice length and any number of bases side by side:
//
//   tridiagonal    A = Q T Q^T by Householder reflections.  Up to 128 rows one work-group holds the whole matrix in
//                  its registers; a larger matrix is first cut down to its trailing 128 x 128 block by one launch over
//                  the chip for all columns, or one per column.
//   bisect         every eigenvalue of T by multisection on Sturm counts, a group of lanes per eigenvalue.
//   inverse        the k wanted eigenvectors of T by inverse iteration from random vectors, one lane each.
//   orthonormalise modified Gram-Schmidt over those k vectors (eigenvalues of the noise lie so close together that
//                  their vectors come out of the iteration correct but not orthogonal to float64 precision).
//   back           Q z for each of them.
//   out            order, sign and conversion to the fp32 basis.
//
// It replaces Jacobi methods, which compute all d eigenvectors and need 12 - 14 sweeps over the matrix whatever k is:
// d = 128 4.0 -> 0.39 ms, d = 768 (k = 96) 22 -> 3.0 ms.  What bounds it is the chain of dependent steps (d reflections,
// each needing the whole of the one before), not arithmetic or memory.
//
// Every kernel returns at once for a basis whose matrix is zero (unit vectors, eigenvalues 0) or not finite
// (eigenvalues NaN, reported by gvq_fit_status), which the largest |entry| says (EigenArgs::norm).
#include "gvq_sample.h"

#include <mutex>
#include <type_traits>

// ---- helpers ----------------------------------------------------------------------------------------------------

template <int CTRL> __device__ __forceinline__ double dpp_move(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
#define DPP_XOR1 0xB1          // quad_perm [1,0,3,2]
#define DPP_XOR2 0x4E          // quad_perm [2,3,0,1]
#define DPP_HALF_MIRROR 0x141  // lane i of 8 -> 7 - i
#define DPP_MIRROR 0x140       // lane i of 16 -> 15 - i
#define DPP_ROR4 0x124
#define DPP_ROR8 0x128

__device__ __forceinline__ double lane_value(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// v of this lane plus v of lane ^ 16 (^ 32), the same bits in both.
__device__ __forceinline__ double add_xor16(double v)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double add_xor32(double v)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

// Sum over the 64 lanes, the same bits in every lane.
__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_move<DPP_XOR1>(v);
    v += dpp_move<DPP_XOR2>(v);
    v += dpp_move<DPP_HALF_MIRROR>(v);
    v += dpp_move<DPP_MIRROR>(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Four of them: each exchange with a neighbour halves the sums a lane holds.
__device__ __forceinline__ void wave_sum4(double (&v)[4])
{
    const bool o1 = threadIdx.x & 1, o2 = threadIdx.x & 2;
    const double a0 = (o1 ? v[2] : v[0]) + dpp_move<DPP_XOR1>(o1 ? v[0] : v[2]);
    const double a1 = (o1 ? v[3] : v[1]) + dpp_move<DPP_XOR1>(o1 ? v[1] : v[3]);
    double b = (o2 ? a1 : a0) + dpp_move<DPP_XOR2>(o2 ? a0 : a1);
    b += dpp_move<DPP_ROR4>(b);
    b += dpp_move<DPP_ROR8>(b);
    b = add_xor32(add_xor16(b));
    v[0] = lane_value(b, 0);
    v[1] = lane_value(b, 2);
    v[2] = lane_value(b, 1);
    v[3] = lane_value(b, 3);
}

// Largest of the 64 lanes' values, in every lane.
__device__ __forceinline__ double wave_max(double v)
{
    v = fmax(v, dpp_move<DPP_XOR1>(v));
    v = fmax(v, dpp_move<DPP_XOR2>(v));
    v = fmax(v, dpp_move<DPP_HALF_MIRROR>(v));
    v = fmax(v, dpp_move<DPP_MIRROR>(v));
    return fmax(fmax(lane_value(v, 0), lane_value(v, 16)), fmax(lane_value(v, 32), lane_value(v, 48)));
}

// 1/x to the last bit or two for normal x and 1/x: the hardware's approximation and two Newton steps.
__device__ __forceinline__ double fast_rcp(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    y = fma(fma(-x, y, 1.0), y, y);
    return y;
}

// sqrt(x) and 1/sqrt(x) likewise, x > 0 and far from the ends of the range (squares of what fp32 numbers' products leave).
__device__ __forceinline__ double fast_sqrt(double x, double& inverse)
{
    double y = __builtin_amdgcn_rsq(x);
    y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    const double r = x * y;
    inverse = y;
    return fma(0.5 * y, fma(-r, r, x), r);
}

// The reflector that takes (x0, rest) to (beta, 0), n2 = |rest|^2: v = (1, rest * sc), H = I - t v v^T.  Every wave of a
// work-group forms it for itself, so what counts is the number of instructions: with the library's square root and
// divisions a step of tri_small_kernel, at four waves to a SIMD, took 2.4 us, 2.2 with these.
__device__ __forceinline__ void reflector(double x0, double n2, double& beta, double& t, double& sc)
{
    beta = x0; t = 0.0; sc = 0.0;
    if (n2 > 0.0) {
        double inv;
        beta = fast_sqrt(fma(x0, x0, n2), inv);
        if (x0 > 0.0) { beta = -beta; inv = -inv; }
        t = (beta - x0) * inv;
        sc = fast_rcp(x0 - beta);
    }
}

typedef double d4 __attribute__((ext_vector_type(4)));

#define EIG_E_FLOOR 1e-20     // smallest off-diagonal entry of T relative to the matrix: decoupled blocks stay coupled
                              // by far less than rounding, which spares every recurrence its special cases
#define EIG_PIVOT 2.3e-16     // smallest pivot relative to the matrix

// Power of two that brings the largest entry below 1.
__device__ __forceinline__ int eig_scale_exp(unsigned long long norm)
{
    return -(__builtin_amdgcn_frexp_exp(__longlong_as_double((long long)norm)));
}

// ---- covariance from the moments ----------------------------------------------------------------------------------

// cov = G/n - mu mu^T, mu, and the largest |entry| (as the bits of a positive double: NaN and Inf sort above all).
__global__ __launch_bounds__(256) void cov_kernel(const double* mom_all, const unsigned long long* nsamp, int d,
                                                  double* cov_all, float* mu, unsigned long long* norm, int* solves)
{
    const int b = blockIdx.y;
    const size_t W = (size_t)d * d + d;
    const double* mom = mom_all + (size_t)b * W;
    double* cov = cov_all + (size_t)b * d * d;
    const double ns = (double)nsamp[b];
    double big = 0.0, bad = 0.0;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < d * d; i += gridDim.x * 256) {
        const int r = i / d, c = i - r * d;
        // upper and lower halves of the Gram sum are bit-identical (same products, same order);
        // true divisions: a constant gradient then gives exactly C = 0
        const double v = ns > 0.0 ? mom[i] / ns - (mom[(size_t)d * d + r] / ns) * (mom[(size_t)d * d + c] / ns) : 0.0;
        cov[i] = v;
        big = fmax(big, fabs(v));
        if (v != v) bad = v;   // fmax drops a NaN
    }
    for (int i = blockIdx.x * 256 + threadIdx.x; i < d; i += gridDim.x * 256)
        mu[(size_t)b * d + i] = ns > 0.0 ? (float)(mom[(size_t)d * d + i] / ns) : 0.0f;
    eig_norm_max(bad != bad ? bad : big, norm + b);
    if (blockIdx.x == 0 && threadIdx.x == 0) solves[b] = 0;   // the solver raises it
}

// ---- tridiagonal ----------------------------------------------------------------------------------------------------
//
// Step i reflects the entries i+1.. of column i onto its first: H = I - tau v v^T with v[i+1] = 1, and A <- H A H is the
// rank-two update A - v w^T - w v^T, w = p - (tau/2)(p.v) v, p = tau A v.  Row r of the working matrix is
// a.A + (r+1) n; the reflector of step i goes to row i-1, which nobody needs any more.

// The update of one entry.  Written out, so that the compiler has nothing to contract: a column as a launch of its own and all of
// them in one launch give the same bits.
__device__ __forceinline__ double tri_update(double x, double vr, double wc, double wr, double vc)
{
    return fma(-vr, wc, fma(-wr, vc, x));
}

// One column of a matrix with more than 128 rows.  Every work-group repeats the O(n) part (the previous step's w, the
// column, its reflector) and then takes eight rows: the rank-two update of the step before, in place, and their
// entries of p for this step -- so a step is one launch, whose end is the only synchronisation it needs.  NE = number of
// 64-column pieces of a row.  Bound by that chain (launch, two block-wide sums, one dot product: about 5 us a
// column); its memory traffic is a few per cent of that.
template <int NE> struct TriShared {
    double vp[NE * 64], wp[NE * 64], vn[NE * 64], red[2][4], first;
};

// ALL: by one work-group, which takes all the rows.
template <int NE, bool ALL> __device__ __forceinline__ void tri_column(const EigenArgs& a, int i, TriShared<NE>& sh)
{
    double (&vp)[NE * 64] = sh.vp, (&wp)[NE * 64] = sh.wp, (&vn)[NE * 64] = sh.vn, (&red)[2][4] = sh.red, &first = sh.first;
    const int b = blockIdx.y, n = a.n, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double* A = a.A + (size_t)b * a.A_stride;
    const double* cur = i == 0 ? a.src + (size_t)b * a.src_stride : A + n;   // the matrix before the pending update
    double* T = a.T + (size_t)b * 5 * a.t_ld;
    const double* p_old = T + (size_t)(3 + ((i + 1) & 1)) * a.t_ld;
    double* p_new = T + (size_t)(3 + (i & 1)) * a.t_ld;

    // this wave's two rows, requested first
    int r0 = i + 1 + (blockIdx.x * 4 + wave) * 2;
    double x[2][NE];
    auto fetch = [&]() {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int q = 0; q < NE; ++q) {
                const int c = 64 * q + lane;
                x[u][q] = (r0 + u < n && c > i && c < n) ? cur[(size_t)(r0 + u) * n + c] : 0.0;
            }
    };
    fetch();

    // column i (row i, the matrix is symmetric) with the previous step's update; at most four entries per thread, always the
    // same ones: tri_chain_kernel adds in this order too
    constexpr int NT = (NE + 3) / 4;
    double col[NT], v[NT], p[NT];
    double tau = 0.0, s = 0.0, pi = 0.0;
    const double* v_old = A + (size_t)(i - 1) * n;   // not touched at i = 0
    if (i > 0) { tau = T[2 * a.t_ld + i - 1]; pi = p_old[i]; }
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        const int c = tid + 256 * u;
        const bool on = c >= i && c < n;
        col[u] = on ? cur[(size_t)i * n + c] : 0.0;
        v[u] = i > 0 && on ? v_old[c] : 0.0;
        p[u] = i > 0 && on ? p_old[c] : 0.0;
        s = fma(p[u], v[u], s);
    }
    s = wave_sum(s);
    if (lane == 0) red[0][wave] = s;
    __syncthreads();
    s = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    const double half = 0.5 * tau * s, wi = fma(-0.5 * tau, s, pi);   // v[i] of the previous step is 1
    double n2 = 0.0;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        const int c = tid + 256 * u;
        const double w = fma(-half, v[u], p[u]);
        col[u] -= fma(v[u], wi, w);
        if (c < n) { vp[c] = v[u]; wp[c] = w; }
        if (c > i + 1) n2 = fma(col[u], col[u], n2);
        if (c == i + 1) first = col[u];
    }
    n2 = wave_sum(n2);
    if (lane == 0) red[1][wave] = n2;
    __syncthreads();
    n2 = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
    const double x0 = first;
    double beta, t, sc;
    reflector(x0, n2, beta, t, sc);
    double* R = A + (size_t)i * n;   // row i-1 of the matrix
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        const int c = tid + 256 * u;
        if (c < i || c >= n) continue;
        const double h = c == i + 1 ? 1.0 : c > i ? col[u] * sc : 0.0;
        vn[c] = h;
        if (blockIdx.x == 0) {
            if (c > i) R[c] = h;
            else { T[i] = col[u]; T[a.t_ld + i] = beta; T[2 * a.t_ld + i] = t; }
        }
    }
    __syncthreads();
    for (;;) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = r0 + u;
            if (r >= n) continue;   // uniform over the wave
            const double vr = vp[r], wr = wp[r];
            double dot = 0.0;
#pragma unroll
            for (int q = 0; q < NE; ++q) {
                const int c = 64 * q + lane;
                if (c <= i || c >= n) continue;
                const double y = tri_update(x[u][q], vr, wp[c], wr, vp[c]);
                A[(size_t)(r + 1) * n + c] = y;
                dot = fma(y, vn[c], dot);
            }
            dot = wave_sum(dot);
            if (lane == 0) p_new[r] = t * dot;
        }
        r0 += 8;
        if (!ALL || r0 >= n) break;
        fetch();
    }
}

template <int NE>
__global__ __launch_bounds__(256) void tri_step_kernel(EigenArgs a, int i)
{
    __shared__ TriShared<NE> sh;
    if (eig_skip(a.norm[blockIdx.y])) return;
    tri_column<NE, false>(a, i, sh);
}

// All of those steps in one launch, where the matrices' rows find a place in the registers of the chip at once (eight rows
// per work-group and at most one work-group per compute unit, gvq_launch_sym_eigen).  What a step needs from the others are p of
// the step before and its own column: both are published as plain 64-bit words, and a word that still holds the mark
// (all bits set, which no arithmetic on finite numbers gives) has not arrived.  Waiting for the words themselves takes one way
// through memory per step, where a counter takes three (the data, the count, the data again) and the end of a launch about
// five microseconds: d = 768 6.4 -> 2.9 us a column, 4.2 -> 1.85 ms for all of them.
//
// Slots: p of step i and row i + 1 go to slot i % 4.  Who has seen all of p of step i - 1 knows that every work-group which
// still takes part is done with slot (i - 2) % 4; those that will write it in step i + 2 put the mark back at the end of step i,
// and wait for that before they publish p of step i + 1, which every later reader of that slot has to see first.  (With three slots
// the mark goes back within the step, and a step waited for it: 3.6 against 3.0 us.)  A work-group leaves when its rows are
// reflected away, so nobody who no longer publishes still reads.
//
// The wait is bounded: a poll takes 0.27 us, the bound 0.14 s, which is about what doing the matrix over takes, and longer than
// most kernels that may hold up part of the grid.  A work-group whose words do not come, because another process or such a kernel
// keeps the others off the chip, gives up, says so behind the slots, and the rest stop too, at the latest when they look there;
// tri_redo_kernel then does the matrix over, with one work-group that waits for nobody.
#define TRI_CHAIN_MARK 0xFFFFFFFFFFFFFFFFull
#define TRI_CHAIN_POLLS (1 << 19)

__global__ __launch_bounds__(256) void tri_chain_clear_kernel(unsigned long long* x, size_t stride, int n)
{
    x += (size_t)blockIdx.y * stride;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) x[i] = TRI_CHAIN_MARK;
}

__device__ __forceinline__ unsigned long long chain_load(const unsigned long long* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void chain_store(unsigned long long* p, unsigned long long v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void chain_publish(unsigned long long* p, double v)
{
    const unsigned long long bits = (unsigned long long)__double_as_longlong(v);
    chain_store(p, bits == TRI_CHAIN_MARK ? 0x7FF8000000000000ull : bits);
}

template <int NE>
__global__ __launch_bounds__(256) void tri_chain_kernel(EigenArgs a, int steps, int polls)
{
    constexpr int NT = (NE + 3) / 4;
    __shared__ double cb[NE * 64], wp[NE * 64], red[2][4], pi_s, first_s;
    __shared__ int lost;
    const int b = blockIdx.y, n = a.n, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (eig_skip(a.norm[b])) return;
    const double* src = a.src + (size_t)b * a.src_stride;
    double* A = a.A + (size_t)b * a.A_stride;
    double* T = a.T + (size_t)b * 5 * a.t_ld;
    unsigned long long* X = a.xchg + (size_t)b * a.xchg_stride;   // [4][2 n]: p, row; then the mark while nobody has given up
    const int r0 = (blockIdx.x * 4 + wave) * 2, r_last = blockIdx.x * 8 + 7;
    const bool writer = blockIdx.x == gridDim.x - 1;   // takes part to the end: it keeps the reflectors

    double x[2][NE], vl[NE], v[NT], vr[2] = {0.0, 0.0};
#pragma unroll
    for (int q = 0; q < NE; ++q) {
        vl[q] = 0.0;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int c = 64 * q + lane;
            x[u][q] = r0 + u < n && c < n ? src[(size_t)(r0 + u) * n + c] : 0.0;
        }
    }
#pragma unroll
    for (int u = 0; u < NT; ++u) v[u] = 0.0;
    if (tid == 0) lost = chain_load(X + 8 * n) != TRI_CHAIN_MARK;
    __syncthreads();
    if (lost) return;   // uniform: nobody polls, and sets it, before the barriers of step 0

    double tau = 0.0;   // of the step before
    bool gone = false;
    for (int i = 0; i < steps; ++i) {
        if (r_last <= i) { gone = true; break; }
        double col[NT], p[NT], s = 0.0;
        if (i == 0) {
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                const int c = tid + 256 * u;
                col[u] = c < n ? src[c] : 0.0;
                p[u] = 0.0;
            }
        } else {
            const unsigned long long* from = X + (size_t)((i - 1) % 4) * 2 * n;
            unsigned long long pw[NT], rw[NT];
            int spins = 0;
            for (;;) {
                bool missing = false;
#pragma unroll
                for (int u = 0; u < NT; ++u) {
                    const int c = tid + 256 * u;
                    const bool on = c >= i && c < n;
                    pw[u] = on ? chain_load(from + c) : 0ull;
                    rw[u] = on ? chain_load(from + n + c) : 0ull;
                }
#pragma unroll
                for (int u = 0; u < NT; ++u) missing |= pw[u] == TRI_CHAIN_MARK || rw[u] == TRI_CHAIN_MARK;
                if (!missing) break;
                if (++spins >= polls || (spins % 64 == 0 && chain_load(X + 8 * n) != TRI_CHAIN_MARK)) { lost = 1; break; }
            }
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                p[u] = __longlong_as_double((long long)pw[u]);
                col[u] = __longlong_as_double((long long)rw[u]);
                s = fma(p[u], v[u], s);
                if (tid + 256 * u == i) pi_s = p[u];
            }
        }
        s = wave_sum(s);
        if (lane == 0) red[0][wave] = s;
        __syncthreads();
        if (lost) break;   // uniform
        s = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
        const double half = 0.5 * tau * s, wi = i > 0 ? fma(-0.5 * tau, s, pi_s) : 0.0;   // v[i] of the previous step is 1
        double n2 = 0.0;
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            const int c = tid + 256 * u;
            const double w = fma(-half, v[u], p[u]);
            col[u] -= fma(v[u], wi, w);
            if (c < NE * 64) {
                cb[c] = c > i ? col[u] : 0.0;
                wp[c] = w;
            }
            if (c > i + 1) n2 = fma(col[u], col[u], n2);
            if (c == i + 1) first_s = col[u];
        }
        n2 = wave_sum(n2);
        if (lane == 0) red[1][wave] = n2;
        __syncthreads();
        n2 = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
        double beta, t, sc;
        reflector(first_s, n2, beta, t, sc);
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            const int c = tid + 256 * u;
            const double h = c == i + 1 ? 1.0 : c > i ? col[u] * sc : 0.0;
            v[u] = c < n ? h : 0.0;
        }
        tau = t;

        // the previous step's update of this wave's rows, and their entries of p
        double hl[NE], wl[NE];
#pragma unroll
        for (int q = 0; q < NE; ++q) {
            const int c = 64 * q + lane;
            hl[q] = c == i + 1 ? 1.0 : cb[c] * sc;   // zero up to column i
            wl[q] = wp[c];
        }
        unsigned long long* to = X + (size_t)(i % 4) * 2 * n;
        double dot[2] = {0.0, 0.0};
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the marks of the step before are back before this wave's p says so
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = r0 + u;
            if (r <= i || r >= n) continue;   // uniform over the wave
            const double wr = wp[r], vo = vr[u];
            vr[u] = r == i + 1 ? 1.0 : cb[r] * sc;
#pragma unroll
            for (int q = 0; q < NE; ++q) {
                x[u][q] = tri_update(x[u][q], vo, wl[q], wr, vl[q]);
                dot[u] = fma(x[u][q], hl[q], dot[u]);
            }
            if (r == i + 1) {
#pragma unroll
                for (int q = 0; q < NE; ++q) {
                    const int c = 64 * q + lane;
                    if (c > i && c < n) chain_publish(to + n + c, x[u][q]);
                }
            }
        }
        const double d0 = wave_sum(dot[0]), d1 = wave_sum(dot[1]);
#pragma unroll
        for (int q = 0; q < NE; ++q) vl[q] = hl[q];
        const int r = r0 + (lane & 1);
        const double pr = t * (lane & 1 ? d1 : d0);
        if (lane < 2 && r > i && r < n) {
            chain_publish(to + r, pr);
            if (i == steps - 1) T[(size_t)(3 + (i & 1)) * a.t_ld + r] = pr;
        }
        // slot (i + 2) % 4 takes the mark back: by whoever writes it in step i + 2
        {
            unsigned long long* next = X + (size_t)((i + 2) % 4) * 2 * n;
            if (lane < 2 && r0 + lane >= i + 3 && r0 + lane < n) chain_store(next + r0 + lane, TRI_CHAIN_MARK);
            if (r0 == i + 3 || r0 + 1 == i + 3) {
#pragma unroll
                for (int q = 0; q < NE; ++q)
                    if (64 * q + lane < n) chain_store(next + n + 64 * q + lane, TRI_CHAIN_MARK);
            }
        }
        if (writer) {
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                const int c = tid + 256 * u;
                if (c > i && c < n) A[(size_t)i * n + c] = v[u];
                if (c == i) { T[i] = col[u]; T[a.t_ld + i] = beta; T[2 * a.t_ld + i] = t; }
            }
        }
    }
    if (lost) {
        if (tid == 0) chain_store(X + 8 * n, 0ull);
        return;
    }
    if (gone) return;
    // what is left, as tri_step_kernel leaves it: the last step's update pending
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int q = 0; q < NE; ++q) {
            const int r = r0 + u, c = 64 * q + lane;
            if (r >= steps && r < n && c >= steps && c < n) A[(size_t)(r + 1) * n + c] = x[u][q];
        }
}

// The matrices whose chain was given up (none, as a rule), from the start: the same operations in the same order, hence the same bits,
// a column at a time by one work-group (d = 520 37 ms, 768 93, 1024 220).
// The launch that waits inside is over when this one starts: `note` says so to the host.
template <int NE>
__global__ __launch_bounds__(256) void tri_redo_kernel(EigenArgs a, int steps, unsigned long long* note, unsigned long long ticket)
{
    __shared__ TriShared<NE> sh;
    if (blockIdx.y == 0 && threadIdx.x == 0) __hip_atomic_store(note, ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (eig_skip(a.norm[blockIdx.y]) || chain_load(a.xchg + (size_t)blockIdx.y * a.xchg_stride + 8 * a.n) == TRI_CHAIN_MARK) return;
    for (int i = 0; i < steps; ++i) {
        tri_column<NE, true>(a, i, sh);
        __syncthreads();   // this column's rows and entries of p, before the next one reads them
    }
}

// The whole matrix (n <= 128), or what is left of a larger one from row i0 on, in the registers of one work-group:
// thread (ti, tj) holds the R x R entries of rows R ti.. and columns R tj...  Per step: the column goes through LDS
// (one barrier), every wave forms the reflector for itself, multiplies its tiles with it, sums over tj inside the wave,
// the entries of p go through LDS (second barrier), update.  About 4500 cycles a step, most of it the
// instructions that every wave repeats and the two passes through LDS; hence R = 8 and one wave per SIMD above 64 rows (16 waves
// of 4 x 4: d = 128 270 -> 245 us, 1000 bases 2450 -> 1960 for the whole refresh).  The matrix never leaves the
// registers (in LDS, 128 x 128 doubles would take 1000 cycles to read once).
//
// SIDE: the work-groups behind those of the `mats` matrices take a block of `side` per wave.  A refresh from first slices has one
// matrix a work-group and needs its full covariances only when it is over: 26 bases of d = 768, L = 100 84 us as a launch of their own.
template <int TJ, int R, bool SIDE>
__global__ __launch_bounds__(TJ * TJ) void tri_small_kernel(EigenArgs a, int i0, int mats, SampleCov side)
{
    if (SIDE && (int)blockIdx.x >= mats) {
        const int at = ((int)blockIdx.x - mats) * (TJ * TJ / 64) + (int)(threadIdx.x >> 6);
        if (at < side.total) (void)sample_cov_block(side, at);
        return;
    }
    constexpr int N = R * TJ, PL = N > 64 ? N / 64 : 1;   // entries of a vector per lane
    __shared__ double colb[2][N], pb[N];
    const int b = blockIdx.x, n = a.n, nl = n - i0, tid = threadIdx.x, lane = tid & 63;
    const int ti = tid / TJ, tj = tid % TJ;
    if (eig_skip(a.norm[b])) return;
    double* A = a.A + (size_t)b * a.A_stride;
    const double* cur = i0 == 0 ? a.src + (size_t)b * a.src_stride : A + n;
    double* T = a.T + (size_t)b * 5 * a.t_ld;

    double x[R][R];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < R; ++c) {
            const int gr = i0 + R * ti + r, gc = i0 + R * tj + c;
            x[r][c] = gr < n && gc < n ? cur[(size_t)gr * n + gc] : 0.0;
        }
    if (i0 > 0) {
        // the update that the last of the steps before this kernel left pending
        const double* p_old = T + (size_t)(3 + ((i0 + 1) & 1)) * a.t_ld;
        const double* v_old = A + (size_t)(i0 - 1) * n;
        const double tau = T[2 * a.t_ld + i0 - 1];
        double s = 0.0;
        for (int c = i0 + lane; c < n; c += 64) s = fma(p_old[c], v_old[c], s);
        const double half = 0.5 * tau * wave_sum(s);
        double vr[R], wr[R], vc[R], wc[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int r = i0 + R * ti + u, c = i0 + R * tj + u;
            vr[u] = r < n ? v_old[r] : 0.0;
            wr[u] = r < n ? fma(-half, vr[u], p_old[r]) : 0.0;
            vc[u] = c < n ? v_old[c] : 0.0;
            wc[u] = c < n ? fma(-half, vc[u], p_old[c]) : 0.0;
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < R; ++c) x[r][c] -= fma(vr[r], wc[c], wr[r] * vc[c]);
    }

    __builtin_amdgcn_s_waitcnt(0);   // the reflectors overwrite rows of the matrix: every thread's loads have come back
    __syncthreads();
    for (int ib = 0; ib < nl; ib += R) {
#pragma unroll
        for (int cb = 0; cb < R; ++cb) {
            const int i = ib + cb;
            if (i >= nl) break;
            double* col = colb[cb & 1];
            if (tj == ib / R) {
#pragma unroll
                for (int r = 0; r < R; ++r) col[R * ti + r] = x[r][cb];
            }
            __syncthreads();
            // nothing to reflect in the last two columns
            if (i >= nl - 2) {
                if (tid == 0) {
                    T[i0 + i] = col[i];
                    T[a.t_ld + i0 + i] = i + 1 < nl ? col[i + 1] : 0.0;
                    T[2 * a.t_ld + i0 + i] = 0.0;
                }
                continue;
            }
            double xl[PL], n2 = 0.0;
#pragma unroll
            for (int u = 0; u < PL; ++u) {
                const int c = PL * lane + u;
                xl[u] = c < N ? col[c] : 0.0;   // entries past the matrix are zero
                if (c > i + 1) n2 = fma(xl[u], xl[u], n2);
            }
            n2 = wave_sum(n2);
            const double x0 = col[i + 1];
            double beta, t, sc;
            reflector(x0, n2, beta, t, sc);
            if (tid < 64) {
#pragma unroll
                for (int u = 0; u < PL; ++u) {
                    const int c = PL * lane + u;
                    if (c > i && c < nl) A[(size_t)(i0 + i) * n + i0 + c] = c == i + 1 ? 1.0 : xl[u] * sc;
                }
                if (lane == 0) {
                    T[i0 + i] = col[i];
                    T[a.t_ld + i0 + i] = beta;
                    T[2 * a.t_ld + i0 + i] = t;
                }
            }
            if (t == 0.0) continue;   // uniform over the work-group; the next column takes the other buffer
            double vr[R], vc[R], y[R];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int r = R * ti + u, c = R * tj + u;
                vr[u] = r == i + 1 ? 1.0 : r > i ? col[r] * sc : 0.0;
                vc[u] = c == i + 1 ? 1.0 : c > i ? col[c] * sc : 0.0;
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                y[r] = x[r][0] * vc[0];
#pragma unroll
                for (int c = 1; c < R; ++c) y[r] = fma(x[r][c], vc[c], y[r]);
            }
            // sum over tj: every exchange with a neighbour halves the rows a lane keeps
            {
                const bool o1 = lane & 1, o2 = lane & 2;
                double h[R / 2], z[R / 4];
#pragma unroll
                for (int q = 0; q < R / 2; ++q)
                    h[q] = (o1 ? y[q + R / 2] : y[q]) + dpp_move<DPP_XOR1>(o1 ? y[q] : y[q + R / 2]);
#pragma unroll
                for (int q = 0; q < R / 4; ++q) {
                    z[q] = (o2 ? h[q + R / 4] : h[q]) + dpp_move<DPP_XOR2>(o2 ? h[q] : h[q + R / 4]);
                    if (TJ >= 16) {
                        z[q] += dpp_move<DPP_ROR4>(z[q]);
                        z[q] += dpp_move<DPP_ROR8>(z[q]);
                    } else {
                        z[q] += __shfl_xor(z[q], 4, 64);
                    }
                }
                if (tj < 4) {
#pragma unroll
                    for (int q = 0; q < R / 4; ++q) pb[R * ti + R / 2 * (lane & 1) + R / 4 * ((lane >> 1) & 1) + q] = t * z[q];
                }
            }
            __syncthreads();
            double s = 0.0;
#pragma unroll
            for (int u = 0; u < PL; ++u) {
                const int c = PL * lane + u;
                const double v = c == i + 1 ? 1.0 : c > i ? xl[u] * sc : 0.0;
                if (c < N) s = fma(pb[c], v, s);
            }
            const double half = 0.5 * t * wave_sum(s);
            double wr[R], wc[R];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                wr[u] = fma(-half, vr[u], pb[R * ti + u]);
                wc[u] = fma(-half, vc[u], pb[R * tj + u]);
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int c = 0; c < R; ++c) x[r][c] = fma(-vr[r], wc[c], fma(-wr[r], vc[c], x[r][c]));
        }
    }
}

// ---- eigenvalues of T -----------------------------------------------------------------------------------------------
//
// The number of eigenvalues below s is the number of sign changes in p_0 = 1, p_1 = d_0 - s, p_{i+1} = (d_i - s) p_i -
// e_{i-1}^2 p_{i-1}.  The three-term form (one dependent fused multiply-add a step, rescaled every eight steps) is a
// quarter of the latency of the quotient form with its division.  A group of `lanes` lanes cuts the interval of its
// eigenvalue into lanes + 1 pieces per pass.  All eigenvalues start from one interval and follow one tree of cuts, so
// they come out ordered.
__global__ __launch_bounds__(256) void bisect_kernel(EigenArgs a)
{
    extern __shared__ double2 t[];   // [n] d_i, e_{i-1}^2
    __shared__ double bound[2];
    const int b = blockIdx.y, n = a.n, tid = threadIdx.x, nthr = blockDim.x;
    const unsigned long long norm = a.norm[b];
    double* eig = a.eig + (size_t)b * a.eig_ld;
    const int g = blockIdx.x * (nthr / a.lanes) + tid / a.lanes;   // this group's eigenvalue, in increasing order
    const int l = tid % a.lanes;
    if (blockIdx.x == 0)
        for (int i = n + tid; i < a.eig_ld; i += nthr) eig[i] = norm >= EIG_INF_BITS ? __longlong_as_double(-1ll) : 0.0;
    if (eig_skip(norm)) {
        if (l == 0 && g < n) eig[g] = norm ? __longlong_as_double(-1ll) : 0.0;   // NaN where the input was not finite
        return;
    }
    const double* T = a.T + (size_t)b * 5 * a.t_ld;
    const int ex = eig_scale_exp(norm);
    double lo = 0.0, hi = 0.0;
    for (int i = tid; i < n; i += nthr) {
        const double d = ldexp(T[i], ex);
        const double e0 = i ? fmax(fabs(ldexp(T[a.t_ld + i - 1], ex)), EIG_E_FLOOR) : 0.0;
        const double e1 = i + 1 < n ? fmax(fabs(ldexp(T[a.t_ld + i], ex)), EIG_E_FLOOR) : 0.0;
        t[i] = make_double2(d, e0 * e0);
        lo = fmin(lo, d - e0 - e1);
        hi = fmax(hi, d + e0 + e1);
    }
    if (tid == 0) { bound[0] = 0.0; bound[1] = 0.0; }
    __syncthreads();
    // One LDS atomic per wave and bound; from every thread they queued up at one address (n = 4, one matrix: 10.4 us a launch,
    // 4.4 now).  |bounds| as integers: positive doubles order like their bits.
    lo = wave_max(fabs(lo));
    hi = wave_max(fabs(hi));
    if ((tid & 63) == 0) {
        atomicMax((unsigned long long*)&bound[0], (unsigned long long)__double_as_longlong(lo));
        atomicMax((unsigned long long*)&bound[1], (unsigned long long)__double_as_longlong(hi));
    }
    __syncthreads();
    const double slack = 1e-15 * (bound[0] + bound[1]) + 1e-18;
    lo = -bound[0] - slack;
    hi = bound[1] + slack;

    const double step = 1.0 / (a.lanes + 1);
    const int passes = a.lanes == 64 ? 9 : a.lanes == 16 ? 14 : a.lanes == 8 ? 18 : 24;   // (lanes + 1)^passes > 2^54
    for (int pass = 0; pass < passes; ++pass) {
        const double w = (hi - lo) * step, s = fma(w, (double)(l + 1), lo);
        double p0 = 1.0, p1 = t[0].x - s;
        unsigned int below = (unsigned int)__double2hiint(p1) >> 31;
        int i = 1;
        for (; i + 8 <= n; i += 8) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const double2 q = t[i + u];
                const double p2 = fma(q.x - s, p1, -(q.y * p0));
                below += (unsigned int)(__double2hiint(p2) ^ __double2hiint(p1)) >> 31;
                p0 = p1;
                p1 = p2;
            }
            const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
            p0 = ldexp(p0, -e);
            p1 = ldexp(p1, -e);
        }
        for (; i < n; ++i) {
            const double2 q = t[i];
            const double p2 = fma(q.x - s, p1, -(q.y * p0));
            below += (unsigned int)(__double2hiint(p2) ^ __double2hiint(p1)) >> 31;
            p0 = p1;
            p1 = p2;
        }
        // cut points with at most g eigenvalues below them are at or left of eigenvalue g
        const unsigned long long left = __ballot(below <= (unsigned int)g);
        const int cut = a.lanes == 64 ? __popcll(left)
                                      : __popcll((left >> ((tid & 63) / a.lanes * a.lanes)) & ((1ull << a.lanes) - 1));
        const double base = lo;
        lo = cut > 0 ? fma(w, (double)cut, base) : base;
        if (cut < a.lanes) hi = fma(w, (double)(cut + 1), base);
    }
    if (l == 0 && g < n) {
        const double v = ldexp(0.5 * (lo + hi), -ex);
        eig[n - 1 - g] = a.clamp && v < 0.0 ? 0.0 : v;
    }
}

// ---- eigenvectors of T ------------------------------------------------------------------------------------------------
//
// One lane per vector: LU with partial pivoting of T - s I (s the eigenvalue), then two solves, the first with a random
// right-hand side of U alone (more, up to EIG_MOST_SOLVES, while a solve does not make the vector grow).  A solve multiplies what other eigenvectors contribute by (rounding / gap), so two leave
// nothing of any whose eigenvalue can be told apart.  Vectors of eigenvalues that cannot are independent random
// members of their common space, which the orthonormalisation sorts out.  NV vectors per work-group (one wave); the
// factors sit in LDS, up to n = 128 of 16 vectors, above that of four or two while the chip has a compute unit for every
// work-group (d = 768, k = 96 415 -> 321 us), else in global memory; entry-major, so that a step's access is one contiguous run.
// Bound by the chain of dependent steps: n divisions and 3 n multiply-adds per vector.
#define EIG_LDS4_ROWS 896   // four vectors' factors, 160 bytes a row, and 16 KB for T fit a compute unit's LDS
template <int NV, bool IN_LDS>
__global__ __launch_bounds__(64) void inverse_kernel(EigenArgs a)
{
    extern __shared__ double lu_lds[];
    constexpr int ROWS = IN_LDS && NV == 16 ? GVQ_EIGEN_SMALL : GVQ_MAX_D;
    __shared__ double td[ROWS], te[ROWS];
    const int b = blockIdx.y, n = a.n, lane = threadIdx.x;
    const unsigned long long norm = a.norm[b];
    if (eig_skip(norm)) return;
    const double* T = a.T + (size_t)b * 5 * a.t_ld;
    const int ex = eig_scale_exp(norm);
    for (int i = lane; i < n; i += 64) {
        td[i] = ldexp(T[i], ex);
        const double e = i + 1 < n ? ldexp(T[a.t_ld + i], ex) : 0.0;
        te[i] = i + 1 < n && fabs(e) < EIG_E_FLOOR ? EIG_E_FLOOR : e;   // 0 past the last
    }
    __syncthreads();
    double* base = IN_LDS ? lu_lds : a.lu + ((size_t)b * gridDim.x + blockIdx.x) * 5 * n * NV;
    const size_t plane = (size_t)n * NV;
    const int j = blockIdx.x * NV + lane;
    int used = 0;
    if (lane < NV && j < a.k) {
        double* ip = base + lane;        // 1 / pivot
        double* u1 = ip + plane;         // U's first and second superdiagonal
        double* u2 = u1 + plane;
        double* lm = u2 + plane;         // multipliers
        double* z = lm + plane;          // right-hand side, solution
        const double s = ldexp(a.eig[(size_t)b * a.eig_ld + j], ex);
        double c = td[0] - s, sup = te[0];
#pragma unroll 4
        for (int i = 0; i < n - 1; ++i) {
            const double e = te[i], d1 = td[i + 1] - s, e1 = te[i + 1];
            // no swap for an off-diagonal entry below rounding: the block ends here, and its pivot is what is floored
            const bool swap = fabs(e) > fmax(fabs(c), EIG_PIVOT);
            double piv = swap ? e : c;
            if (fabs(piv) < EIG_PIVOT) piv = piv < 0.0 ? -EIG_PIVOT : EIG_PIVOT;
            const double r = fast_rcp(piv), f = (swap ? c : e) * r;
            ip[(size_t)i * NV] = r;
            u1[(size_t)i * NV] = swap ? d1 : sup;
            u2[(size_t)i * NV] = swap ? (i + 2 < n ? e1 : 1.0) : 0.0;   // non-zero marks a swap
            lm[(size_t)i * NV] = f;
            c = swap ? fma(-f, d1, sup) : fma(-f, sup, d1);
            sup = swap ? -f * e1 : e1;
        }
        if (fabs(c) < EIG_PIVOT) c = c < 0.0 ? -EIG_PIVOT : EIG_PIVOT;
        const double r_last = fast_rcp(c);

        // Both sweeps work on blocks of eight steps: a block's operands are read before the block ahead of it is
        // worked through, so that the chain waits for arithmetic only.
        constexpr int K = 8;
        double big = 1.0;
        auto solve = [&](auto first) {   // a constant: as a number that is looked at in the loops it cost 420 -> 730 us at d = 768
            constexpr bool FIRST = decltype(first)::value;
            double y = hash_unit((unsigned int)(n - 1), (unsigned int)j);
            if constexpr (!FIRST) {
                // forward, on the first solution scaled to its largest entry
                const double sc = 1.0 / big;
                double zc[K], lc[K], uc[K], zn[K], ln[K], un[K];
                auto fetch = [&](int i, double (&zz)[K], double (&ll)[K], double (&uu)[K]) {
#pragma unroll
                    for (int u = 0; u < K; ++u) {
                        const int at = i + u < n - 1 ? i + u : n - 2;
                        zz[u] = z[(size_t)(at + 1) * NV];
                        ll[u] = lm[(size_t)at * NV];
                        uu[u] = u2[(size_t)at * NV];
                    }
                };
                y = z[0] * sc;
                fetch(0, zc, lc, uc);
                for (int i = 0; i < n - 1; i += K) {
                    fetch(i + K, zn, ln, un);
#pragma unroll
                    for (int u = 0; u < K; ++u) {
                        if (i + u >= n - 1) break;
                        const double t = zc[u] * sc, f = lc[u];
                        const bool swap = uc[u] != 0.0;
                        z[(size_t)(i + u) * NV] = swap ? t : y;
                        y = swap ? fma(-f, t, y) : fma(-f, y, t);
                    }
#pragma unroll
                    for (int u = 0; u < K; ++u) { zc[u] = zn[u]; lc[u] = ln[u]; uc[u] = un[u]; }
                }
            }
            // backward
            double x2 = 0.0, x1 = y * r_last;
            big = fabs(x1);
            z[(size_t)(n - 1) * NV] = x1;
            double rc[K], ac[K], bc[K], zc[K], rn[K], an[K], bn[K], zn[K];
            auto fetch = [&](int i, double (&rr)[K], double (&aa)[K], double (&bb)[K], double (&zz)[K]) {
#pragma unroll
                for (int u = 0; u < K; ++u) {
                    const int at = i - u > 0 ? i - u : 0;
                    rr[u] = ip[(size_t)at * NV];
                    aa[u] = u1[(size_t)at * NV];
                    bb[u] = at == n - 2 ? 0.0 : u2[(size_t)at * NV];
                    zz[u] = FIRST ? hash_unit((unsigned int)at, (unsigned int)j) : z[(size_t)at * NV];
                }
            };
            fetch(n - 2, rc, ac, bc, zc);
            for (int i = n - 2; i >= 0; i -= K) {
                fetch(i - K, rn, an, bn, zn);
#pragma unroll
                for (int u = 0; u < K; ++u) {
                    if (i - u < 0) break;
                    const double v = fma(-ac[u], x1, fma(-bc[u], x2, zc[u])) * rc[u];
                    z[(size_t)(i - u) * NV] = v;
                    x2 = x1;
                    x1 = v;
                    big = fmax(big, fabs(v));
                }
#pragma unroll
                for (int u = 0; u < K; ++u) { rc[u] = rn[u]; ac[u] = an[u]; bc[u] = bn[u]; zc[u] = zn[u]; }
            }
        };
        solve(std::true_type{});
        used = 1;
        do {
            solve(std::false_type{});
            ++used;
            // a vector that has converged grows by about 1 / (rounding) in a solve
        } while (!(big > 1e9) && used < EIG_MOST_SOLVES);
        if (!(big > 1e9)) used = GVQ_NO_CONVERGENCE;
        lm[0] = 1.0 / big;   // this vector's scale, for the copy below
    }
    __syncthreads();
    for (int o = 32; o > 0; o >>= 1) used = max(used, __shfl_xor(used, o, 64));
    if (lane == 0) atomicMax(a.solves + b, used);
    for (int v = 0; v < NV; ++v) {
        const int jv = blockIdx.x * NV + v;
        if (jv >= a.k) break;
        const double sc = base[3 * plane + v];
        double* o = a.Z + (size_t)b * a.Z_stride + (size_t)jv * n;
        for (int i = lane; i < n; i += 64) o[i] = base[4 * plane + (size_t)i * NV + v] * sc;
    }
}

// ---- orthonormalise -----------------------------------------------------------------------------------------------------
//
// Modified Gram-Schmidt over k columns of length n, one work-group per basis, panels of 32 columns in registers (four
// per wave, NE numbers per lane each).  A panel first sheds its components along the finished columns, then along its
// own, column by column through LDS.
//
// One work-group per basis is a 256th of the chip, and what many columns take is the first part: more than 256 columns are
// finished panel by panel, each in a launch of its own (FINISH), and after each the later panels shed their components along
// it, a work-group each (SHED): the same operations in the same order (d = k = 1024 20.6 -> 2.8 ms; the whole refresh 29.4 -> 11.6, d = k = 512 6.4 -> 3.9).
// A column's sums over the wave, four at a time, and its reciprocal square root are what a step waits for, and the finished
// columns arrive while the one before them is worked through (d = 768, k = 96: 193 -> 158 us).  At NE = 16 ORTHO_ALL keeps 64 of
// its registers in scratch for that, and gains all the same (d = 1024, k = 128: 392 -> 333 us; 26 bases of d = 900, k = 96 237 -> 212).
enum OrthoPart { ORTHO_ALL, ORTHO_FINISH, ORTHO_SHED };
template <int NE, OrthoPart PART>
__global__ __launch_bounds__(512) void orthonormalise_kernel(double* Z, size_t Z_stride, int k, int n, int panel,
                                                             const unsigned long long* norm)
{
    __shared__ double q[2][NE * 64];
    const int b = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (eig_skip(norm[b])) return;
    Z += (size_t)b * Z_stride;
    const int first = PART == ORTHO_ALL ? 0 : 32 * (PART == ORTHO_FINISH ? panel : panel + 1 + (int)blockIdx.x);
    const int end = PART == ORTHO_ALL ? k : first + 32;
    for (int c0 = first; c0 < end; c0 += 32) {
        double x[4][NE];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const int c = c0 + 8 * s + wave, i = 64 * e + lane;
                x[s][e] = c < k && i < n ? Z[(size_t)c * n + i] : 0.0;
            }
        const int done0 = PART == ORTHO_SHED ? 32 * panel : 0, done1 = PART == ORTHO_ALL ? c0 : PART == ORTHO_SHED ? done0 + 32 : 0;
        double next[NE];   // the finished column after this one is on its way while this one is worked through
        auto fetch = [&](int done) {
#pragma unroll
            for (int e = 0; e < NE; ++e) next[e] = Z[(size_t)done * n + (64 * e + lane < n ? 64 * e + lane : n - 1)];
        };
        if (done0 < done1) fetch(done0);
        for (int done = done0; done < done1; ++done) {
            double y[NE], dot[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int e = 0; e < NE; ++e) y[e] = 64 * e + lane < n ? next[e] : 0.0;
            fetch(done + 1 < done1 ? done + 1 : done);
#pragma unroll
            for (int e = 0; e < NE; ++e)
#pragma unroll
                for (int s = 0; s < 4; ++s) dot[s] = fma(y[e], x[s][e], dot[s]);
            wave_sum4(dot);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int e = 0; e < NE; ++e) x[s][e] = fma(-dot[s], y[e], x[s][e]);
        }
        if (PART == ORTHO_SHED) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int e = 0; e < NE; ++e) {
                    const int c = c0 + 8 * s + wave, i = 64 * e + lane;
                    if (c < k && i < n) Z[(size_t)c * n + i] = x[s][e];
                }
            return;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            for (int w = 0; w < 8; ++w) {
                const int c = c0 + 8 * s + w;
                if (c >= k) break;   // uniform
                double* buf = q[w & 1];
                if (wave == w) {
                    double n2 = 0.0;
#pragma unroll
                    for (int e = 0; e < NE; ++e) n2 = fma(x[s][e], x[s][e], n2);
                    n2 = wave_sum(n2);
                    double inv = 0.0;
                    if (n2 > 0.0) (void)fast_sqrt(n2, inv);
#pragma unroll
                    for (int e = 0; e < NE; ++e) {
                        x[s][e] *= inv;
                        buf[64 * e + lane] = x[s][e];
                        if (64 * e + lane < n) Z[(size_t)c * n + 64 * e + lane] = x[s][e];
                    }
                }
                __syncthreads();
                double y[NE], dot[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int e = 0; e < NE; ++e) y[e] = buf[64 * e + lane];
#pragma unroll
                for (int e = 0; e < NE; ++e)
#pragma unroll
                    for (int s2 = 0; s2 < 4; ++s2)
                        if (s2 >= s) dot[s2] = fma(y[e], x[s2][e], dot[s2]);
                wave_sum4(dot);
#pragma unroll
                for (int s2 = 0; s2 < 4; ++s2) {
                    if (s2 < s || (s2 == s && wave <= w)) continue;
#pragma unroll
                    for (int e = 0; e < NE; ++e) x[s2][e] = fma(-dot[s2], y[e], x[s2][e]);
                }
            }
        }
        __syncthreads();   // the finished panel is visible to every wave
    }
}

// ---- back ---------------------------------------------------------------------------------------------------------------
//
// z <- H_0 H_1 ... H_{n-3} z, one wave per vector held in registers.  A step is a dot product and an update of a few numbers
// per lane, far less than the time its reflector takes to arrive, so PF of them are in flight (d = 128 55 us with one in
// flight, 29 with four).  Up to 128 rows.
template <int NE>
__global__ __launch_bounds__(256) void back_kernel(EigenArgs a)
{
    constexpr int PF = 4;
    const int b = blockIdx.y, n = a.n, lane = threadIdx.x & 63;
    const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (eig_skip(a.norm[b]) || j >= a.k) return;
    const double* R = a.A + (size_t)b * a.A_stride;   // reflector i is row i (row i-1 of the matrix)
    const double* tau = a.T + (size_t)b * 5 * a.t_ld + 2 * a.t_ld;
    double* Z = a.Z + (size_t)b * a.Z_stride + (size_t)j * n;
    double z[NE], v[PF][NE], t[PF];
#pragma unroll
    for (int e = 0; e < NE; ++e) z[e] = 64 * e + lane < n ? Z[64 * e + lane] : 0.0;
    auto fetch = [&](int i, double (&w)[NE], double& tw) {
        const int at = i > 0 ? i : 0;   // past the last: its words again, unused
        tw = tau[at];
#pragma unroll
        for (int e = 0; e < NE; ++e) w[e] = R[(size_t)at * n + (64 * e + lane < n ? 64 * e + lane : n - 1)];
    };
#pragma unroll
    for (int u = 0; u < PF; ++u) fetch(n - 3 - u, v[u], t[u]);
    for (int i = n - 3; i >= 0; i -= PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            double cur[NE], dot = 0.0;
            const double tc = t[u];
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const int c = 64 * e + lane;
                cur[e] = c > i - u && c < n ? v[u][e] : 0.0;
            }
            fetch(i - u - PF, v[u], t[u]);
            if (i - u < 0 || tc == 0.0) continue;   // none, or its vector was not written
#pragma unroll
            for (int e = 0; e < NE; ++e) dot = fma(cur[e], z[e], dot);
            dot = tc * wave_sum(dot);
#pragma unroll
            for (int e = 0; e < NE; ++e) z[e] = fma(-dot, cur[e], z[e]);
        }
    }
#pragma unroll
    for (int e = 0; e < NE; ++e)
        if (64 * e + lane < n) Z[64 * e + lane] = z[e];
}

// More than 128 rows: the same reflectors 32 at a time, H_i .. H_{i+31} = I - V^T T V (rows of V: the reflectors, T upper triangular).
// One at a time a vector goes through n dependent steps, each a sum over a wave, and every wave reads every reflector
// (d = 768, k = 96: 374 us, 490 ns a step; a compute unit's four waves fetched 24 KB each step).  Here the chain is n / 32 steps, and
// the four waves of a vector fetch eight reflectors of a block each, once, into registers that serve both products.
// d = 768, k = 96: 374 -> 91 us and 22 for T; at 128 rows and below 28 + 13 against 30 us, and thousands of small matrices lose a tenth.
#define WY_ROWS 32

// T of every block, and zeros where V has none (a reflector's row holds old entries up to its column; all of it if tau is 0).
// T(0..j-1, j) = -tau_j T(0..j-1, 0..j-1) G(0..j-1, j), G = V V^T: products on the fp64 matrix pipe, a quarter of the columns per wave.
__global__ __launch_bounds__(256) void wy_kernel(EigenArgs a)
{
    __shared__ double part[4][3][256], G[WY_ROWS][WY_ROWS + 1];
    const int b = blockIdx.y, n = a.n, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, m = lane & 15, kk = lane >> 4;
    if (eig_skip(a.norm[b])) return;
    double* A = a.A + (size_t)b * a.A_stride;
    const double* tau = a.T + (size_t)b * 5 * a.t_ld + 2 * a.t_ld;
    double* out = a.wy + (size_t)b * a.wy_stride + (size_t)blockIdx.x * WY_ROWS * WY_ROWS;
    const int nref = n - 2, i0 = WY_ROWS * blockIdx.x;
    for (int r = wave; r < WY_ROWS && i0 + r < nref; r += 4) {
        const int i = i0 + r, end = tau[i] == 0.0 ? n : i + 1;
        for (int c = lane; c < end; c += 64) A[(size_t)i * n + c] = 0.0;
    }
    __syncthreads();   // also orders the stores above before the loads below: one work-group, one compute unit
    d4 g[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) g[t] = d4{0.0, 0.0, 0.0, 0.0};
    // columns 16 at a time from the block's first; the order of a contraction is free, so a lane takes four that are neighbours
    const double* row0 = A + (size_t)(i0 + m < nref ? i0 + m : nref - 1) * n;
    const double* row1 = A + (size_t)(i0 + 16 + m < nref ? i0 + 16 + m : nref - 1) * n;
    for (int c0 = i0 / 16 * 16 + 16 * wave; c0 < n; c0 += 64) {
        double x0[4], x1[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + 4 * kk + u, at = c < n ? c : n - 1;
            x0[u] = row0[at];
            x1[u] = row1[at];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool in = c0 + 4 * kk + u < n;
            x0[u] = in && i0 + m < nref ? x0[u] : 0.0;
            x1[u] = in && i0 + 16 + m < nref ? x1[u] : 0.0;
            g[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0[u], x0[u], g[0], 0, 0, 0);
            g[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0[u], x1[u], g[1], 0, 0, 0);
            g[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(x1[u], x1[u], g[2], 0, 0, 0);
        }
    }
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[wave][t][(4 * r + kk) * 16 + m] = g[t][r];
    __syncthreads();
    for (int e = tid; e < 3 * 256; e += 256) {
        const int t = e >> 8, r = (e >> 4) & 15, c = e & 15;
        G[r + (t == 2 ? 16 : 0)][c + (t == 0 ? 0 : 16)] =
            (part[0][t][e & 255] + part[1][t][e & 255]) + (part[2][t][e & 255] + part[3][t][e & 255]);
    }
    __syncthreads();
    if (tid >= WY_ROWS) return;
    double row[WY_ROWS];   // row tid of T: each depends on itself and G alone
#pragma unroll
    for (int j = 0; j < WY_ROWS; ++j) {
        const double t = i0 + j < nref ? tau[i0 + j] : 0.0;
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < j; ++q) s = fma(row[q], G[q][j], s);
        row[j] = tid == j ? t : tid < j ? -t * s : 0.0;
        out[tid * WY_ROWS + j] = row[j];
    }
}

template <int NE>
__global__ __launch_bounds__(256) void back_wy_kernel(EigenArgs a)
{
    constexpr int RW = WY_ROWS / 4;   // reflectors of a block per wave
    __shared__ double part[4][NE * 64], ws[WY_ROWS];
    const int b = blockIdx.y, n = a.n, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (eig_skip(a.norm[b])) return;
    const double* R = a.A + (size_t)b * a.A_stride;   // reflector i is row i
    const double* TW = a.wy + (size_t)b * a.wy_stride;
    double* Z = a.Z + (size_t)b * a.Z_stride + (size_t)blockIdx.x * n;
    const int nref = n - 2, blocks = (nref + WY_ROWS - 1) / WY_ROWS;
    double z[NE], v[RW][NE], t[4];
    int at[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int c = 64 * e + lane;
        at[e] = c < n ? c : n - 1;   // past the row: its last entry, which meets zeros of z
        z[e] = c < n ? Z[c] : 0.0;
    }
    auto fetch = [&](int blk) {
        const int i0 = WY_ROWS * blk;
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = TW[(size_t)blk * WY_ROWS * WY_ROWS + (RW * wave + (lane >> 3)) * WY_ROWS + 4 * (lane & 7) + u];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const int i = i0 + RW * wave + r;
            const double* row = R + (size_t)(i < nref ? i : nref - 1) * n;   // past the last: meets zeros of T
#pragma unroll
            for (int e = 0; e < NE; ++e) v[r][e] = 64 * e + 63 > i0 ? row[at[e]] : 0.0;   // uniform: nothing up to column i0
        }
    };
    fetch(blocks - 1);
    for (int blk = blocks - 1; blk >= 0; --blk) {
        double d8[RW];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            d8[r] = 0.0;
#pragma unroll
            for (int e = 0; e < NE; ++e) d8[r] = fma(v[r][e], z[e], d8[r]);
        }
        // eight sums over the 64 lanes: each exchange halves the sums a lane holds
        double s4[4], s2[2], d1;
        const bool o1 = lane & 1, o2 = lane & 2, o4 = lane & 4;
#pragma unroll
        for (int r = 0; r < 4; ++r) s4[r] = (o1 ? d8[r + 4] : d8[r]) + dpp_move<DPP_XOR1>(o1 ? d8[r] : d8[r + 4]);
#pragma unroll
        for (int r = 0; r < 2; ++r) s2[r] = (o2 ? s4[r + 2] : s4[r]) + dpp_move<DPP_XOR2>(o2 ? s4[r] : s4[r + 2]);
        d1 = (o4 ? s2[1] : s2[0]) + __shfl_xor(o4 ? s2[0] : s2[1], 4, 64);
        d1 += dpp_move<DPP_ROR8>(d1);
        d1 = add_xor32(add_xor16(d1));
        if (lane < RW) ws[RW * wave + 4 * (lane & 1) + 2 * ((lane >> 1) & 1) + (lane >> 2)] = d1;
        __syncthreads();
        double y = 0.0;   // T w, eight lanes a row
#pragma unroll
        for (int u = 0; u < 4; ++u) y = fma(t[u], ws[4 * (lane & 7) + u], y);
        y += dpp_move<DPP_XOR1>(y);
        y += dpp_move<DPP_XOR2>(y);
        y += dpp_move<DPP_HALF_MIRROR>(y);
        double f[RW];
#pragma unroll
        for (int r = 0; r < RW; ++r) f[r] = lane_value(y, 8 * r);
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            double s = 0.0;
#pragma unroll
            for (int r = 0; r < RW; ++r) s = fma(v[r][e], f[r], s);
            part[wave][64 * e + lane] = s;
        }
        fetch(blk > 0 ? blk - 1 : 0);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int c = 64 * e + lane;
            const double s = (part[0][c] + part[1][c]) + (part[2][c] + part[3][c]);
            z[e] = c < n ? z[e] - s : 0.0;
        }
    }
#pragma unroll
    for (int e = 0; e < NE; ++e)
        if (e % 4 == wave && 64 * e + lane < n) Z[64 * e + lane] = z[e];
}

// ---- out ----------------------------------------------------------------------------------------------------------------
//
// U = the k columns of Z as float, each negated if needed so that its largest-magnitude entry (lowest index on ties) is
// positive; unit vectors for a zero matrix, NaN for one that is not finite.  One wave per column.
__global__ __launch_bounds__(256) void basis_out_kernel(const double* Z, size_t Z_stride, int k, int d,
                                                        const unsigned long long* norm, float* U, int* solves)
{
    const int b = blockIdx.y, lane = threadIdx.x & 63, c = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (c >= k) return;
    U += (size_t)b * d * k;
    const unsigned long long nb = norm[b];
    if (eig_skip(nb)) {
        for (int i = lane; i < d; i += 64) U[(size_t)i * k + c] = nb ? __int_as_float(0x7FC00000) : i == c ? 1.f : 0.f;
        if (c == 0 && lane == 0) solves[b] = nb ? GVQ_NO_CONVERGENCE : 0;
        return;
    }
    const double* z = Z + (size_t)b * Z_stride + (size_t)c * d;
    double big = -1.0;
    int arg = GVQ_MAX_D;
    bool neg = false;
    for (int i = lane; i < d; i += 64) {
        const double v = z[i], m = fabs(v);
        if (m > big) { big = m; arg = i; neg = v < 0.0; }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double m = __shfl_xor(big, o, 64);
        const int at = __shfl_xor(arg, o, 64);
        const int ng = __shfl_xor((int)neg, o, 64);
        if (m > big || (m == big && at < arg)) { big = m; arg = at; neg = ng != 0; }
    }
    for (int i = lane; i < d; i += 64) U[(size_t)i * k + c] = (float)(neg ? -z[i] : z[i]);
}

// What gvq_fit_status reports, into host memory: the most solves, whether any vector did not converge, whether any eigenvalue
// is not finite (the whole call 13 - 16 us, with copies of both arrays instead 38 - 48; 1 basis of 768 to 26 of 900 eigenvalues).
__global__ __launch_bounds__(1024) void fit_status_kernel(const int* solves, int B, const double* eig, size_t n,
                                                          unsigned long long* out)
{
    __shared__ int most, flags;
    if (threadIdx.x == 0) most = flags = 0;
    __syncthreads();
    int mx = 0, fl = 0;
    for (int b = threadIdx.x; b < B; b += 1024) {
        const int s = solves[b];
        if (s >= GVQ_NO_CONVERGENCE) fl |= 1;
        else if (s > mx) mx = s;
    }
#pragma unroll 8
    for (size_t i = threadIdx.x; i < n; i += 1024)
        if (((unsigned long long)__double_as_longlong(eig[i]) & EIG_INF_BITS) == EIG_INF_BITS) fl |= 2;
    if (mx) atomicMax(&most, mx);
    if (fl) atomicOr(&flags, fl);
    __syncthreads();
    if (threadIdx.x == 0) *out = (unsigned long long)(unsigned int)flags << 32 | (unsigned int)most;
}

// ======================================================================================
int gvq_launch_fit_status(const gvq_basis* h, hipStream_t st)
{
    hipLaunchKernelGGL(fit_status_kernel, dim3(1), dim3(1024), 0, st, h->d_solves, h->B, h->d_eig, (size_t)h->B * h->d, h->h_notes);
    GVQ_HIP(hipGetLastError());
    return GVQ_OK;
}

size_t gvq_eigen_lu_doubles(int d, int k)   // per basis
{
    return d <= GVQ_EIGEN_SMALL ? 0 : (size_t)((k + 63) / 64) * 5 * d * 64;
}

template <template <int> class F, typename... Args>
static void by_long_pieces(int n, Args... args)   // n > 128
{
    if (n <= 256) F<4>::go(args...);
    else if (n <= 512) F<8>::go(args...);
    else if (n <= 768) F<12>::go(args...);
    else F<16>::go(args...);
}
template <template <int> class F, typename... Args>
static void by_pieces(int n, Args... args)
{
    if (n <= 64) F<1>::go(args...);
    else if (n <= 128) F<2>::go(args...);
    else by_long_pieces<F>(n, args...);
}
template <int NE> struct go_step {
    static void go(dim3 grid, EigenArgs a, int i, hipStream_t st) { hipLaunchKernelGGL((tri_step_kernel<NE>), grid, dim3(256), 0, st, a, i); }
};
template <int NE> struct go_chain {
    static void go(dim3 grid, EigenArgs a, int steps, int polls, hipStream_t st) { hipLaunchKernelGGL((tri_chain_kernel<NE>), grid, dim3(256), 0, st, a, steps, polls); }
};
template <int NE> struct go_redo {
    static void go(dim3 grid, EigenArgs a, int steps, unsigned long long* note, unsigned long long ticket, hipStream_t st)
    {
        hipLaunchKernelGGL((tri_redo_kernel<NE>), grid, dim3(256), 0, st, a, steps, note, ticket);
    }
};
template <int NE> struct go_ortho {
    static void go(double* Z, size_t stride, int k, int n, int B, const unsigned long long* norm, hipStream_t st)
    {
        const dim3 threads(64 * (k < 8 ? k : 8));   // a wave per column of eight
        if (k <= 256) {
            hipLaunchKernelGGL((orthonormalise_kernel<NE, ORTHO_ALL>), dim3(1, B), threads, 0, st, Z, stride, k, n, 0, norm);
            return;
        }
        for (int p = 0; 32 * p < k; ++p) {
            const int later = (k - 1) / 32 - p;
            hipLaunchKernelGGL((orthonormalise_kernel<NE, ORTHO_FINISH>), dim3(1, B), threads, 0, st, Z, stride, k, n, p, norm);
            if (later) hipLaunchKernelGGL((orthonormalise_kernel<NE, ORTHO_SHED>), dim3(later, B), threads, 0, st, Z, stride, k, n, p, norm);
        }
    }
};
template <int NE> struct go_back_wy {
    static void go(dim3 grid, EigenArgs a, hipStream_t st) { hipLaunchKernelGGL((back_wy_kernel<NE>), grid, dim3(256), 0, st, a); }
};

int gvq_launch_orthonormalise(const gvq_basis* h, double* Z, size_t Z_stride, int k, int n, hipStream_t st)
{
    by_pieces<go_ortho>(n, Z, Z_stride, k, n, h->B, (const unsigned long long*)(h->d_nsamp + h->B), st);
    GVQ_HIP(hipGetLastError());
    return GVQ_OK;
}

// Whether the stream may use every compute unit (hipExtStreamCreateWithCUMask gives it fewer).
static bool whole_chip(const gvq_basis* h, hipStream_t st)
{
    uint32_t mask[32] = {0};
    if (hipExtStreamGetCUMask(st, 32, mask) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    int units = 0;
    for (uint32_t m : mask) units += __builtin_popcount(m);
    return units >= h->num_cu;
}

// The last launch on a device whose work-groups wait for each other: it is over when its handle's note holds the ticket.
struct ChainTurn {
    const gvq_basis* owner = nullptr;
    hipStream_t stream = nullptr;
    unsigned long long ticket = 0;
};
static std::mutex g_chain_lock;
static ChainTurn g_chain_last[GVQ_MAX_DEVICES];

void gvq_chain_forget(const gvq_basis* h)
{
    std::lock_guard<std::mutex> guard(g_chain_lock);
    for (ChainTurn& t : g_chain_last)
        if (t.owner == h) t = ChainTurn();
}

// All columns up to the trailing block in one launch (*done), where every work-group (8 rows) has a compute unit to itself;
// more matrices than that take turns, and a launch per column serves them all at once.  Work-groups that wait for each other
// have to be on the chip together, so two such launches must not run side by side, each half resident.  A stream keeps its
// own apart; while another stream's is queued or running, this refresh takes the launches per column, which wait for nobody
// (an event between the streams would make it wait for all that the other stream had queued before).  So do two kinds of
// stream: one that is being captured, as the graph may be replayed beside anything, and one that may not use every compute
// unit, as work-groups are dealt to the eight parts of the chip in turn, however many units of each the mask leaves.
static int launch_chain(const gvq_basis* h, const EigenArgs& a, int steps, hipStream_t st, bool* done)
{
    static unsigned long long tickets = 0;
    const int wgs = (a.n + 7) / 8;
    if ((int64_t)wgs * h->B > h->num_cu || h->device < 0 || h->device >= GVQ_MAX_DEVICES) return GVQ_OK;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        return GVQ_OK;
    }
    if (!whole_chip(h, st)) return GVQ_OK;
    std::lock_guard<std::mutex> guard(g_chain_lock);
    ChainTurn& last = g_chain_last[h->device];
    const bool same = last.stream == st && st != hipStreamPerThread;   // that handle names another stream in each thread
    if (last.owner && !same && ((const volatile unsigned long long*)last.owner->h_notes)[1] != last.ticket) return GVQ_OK;
    hipLaunchKernelGGL(tri_chain_clear_kernel, dim3((unsigned)((8 * a.n + 1 + 255) / 256), h->B), dim3(256), 0, st, a.xchg, a.xchg_stride, 8 * a.n + 1);
    GVQ_HIP(hipGetLastError());
    by_long_pieces<go_chain>(a.n, dim3((unsigned)wgs, h->B), a, steps, gvq_opt_chain_polls() > 0 ? gvq_opt_chain_polls() : TRI_CHAIN_POLLS, st);
    GVQ_HIP(hipGetLastError());
    last = ChainTurn{h, st, ++tickets};
    by_long_pieces<go_redo>(a.n, dim3(1, h->B), a, steps, h->h_notes + 1, last.ticket, st);
    GVQ_HIP(hipGetLastError());
    *done = true;
    return GVQ_OK;
}

int gvq_launch_sym_eigen(const gvq_basis* h, EigenArgs a, bool ortho, hipStream_t st, const SampleCov* side)
{
    const int n = a.n, B = h->B, i0 = n > GVQ_EIGEN_SMALL ? n - GVQ_EIGEN_SMALL : 0;
    bool chain = false;
    if (i0 > 0) {
        const int rc = launch_chain(h, a, i0, st, &chain);
        if (rc != GVQ_OK) return rc;
    }
    for (int i = 0; i < i0 && !chain; ++i) {
        by_long_pieces<go_step>(n, dim3((unsigned)((n - 1 - i + 7) / 8), B), a, i, st);
        GVQ_HIP(hipGetLastError());
    }
    auto small = [&](auto kern, auto kern_side, int threads) {
        const int per = threads / 64;
        if (side) hipLaunchKernelGGL(kern_side, dim3((unsigned)(B + (side->total + per - 1) / per)), dim3(threads), 0, st, a, i0, B, *side);
        else hipLaunchKernelGGL(kern, dim3(B), dim3(threads), 0, st, a, i0, B, SampleCov{});
    };
    if (side && i0 > 0) return GVQ_EINVAL;   // no caller does
    if (n - i0 <= 32) small(tri_small_kernel<8, 4, false>, tri_small_kernel<8, 4, true>, 64);
    else if (n - i0 <= 64) small(tri_small_kernel<16, 4, false>, tri_small_kernel<16, 4, true>, 256);
    else small(tri_small_kernel<16, 8, false>, tri_small_kernel<16, 8, true>, 256);
    GVQ_HIP(hipGetLastError());
    // a wave per eigenvalue while that leaves the chip's 1024 SIMDs a handful each, fewer lanes for many small matrices (the
    // passes that more lanes spare are fewer than the lanes: 16 x 16, 4000 of them 69 us with 16 lanes, 36 with 4 and a wave each)
    a.lanes = (int64_t)n * B <= 4096 ? 64 : (int64_t)n * B <= 16384 ? 16 : (int64_t)n * B <= 32768 ? 8 : 4;
    const int bisect_threads = n * a.lanes >= 256 ? 256 : (n * a.lanes + 63) / 64 * 64;
    hipLaunchKernelGGL(bisect_kernel, dim3((unsigned)((n * a.lanes + bisect_threads - 1) / bisect_threads), B), dim3(bisect_threads),
                       sizeof(double2) * n, st, a);
    GVQ_HIP(hipGetLastError());
    if (n <= GVQ_EIGEN_SMALL) {
        const size_t lds = sizeof(double) * 5 * n * 16;
        static gvq_once_per_device once;
        const int rc = once.call(h->device, [&]() -> int {
            GVQ_HIP(hipFuncSetAttribute((const void*)(inverse_kernel<16, true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)(sizeof(double) * 5 * GVQ_EIGEN_SMALL * 16)));
            return GVQ_OK;
        });
        if (rc != GVQ_OK) return rc;
        hipLaunchKernelGGL((inverse_kernel<16, true>), dim3((unsigned)((a.k + 15) / 16), B), dim3(64), lds, st, a);
    } else if (const int nv = n <= EIG_LDS4_ROWS ? 4 : 2; (int64_t)((a.k + nv - 1) / nv) * B <= h->num_cu) {
        static gvq_once_per_device once;
        const int rc = once.call(h->device, [&]() -> int {
            GVQ_HIP(hipFuncSetAttribute((const void*)(inverse_kernel<4, true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)(sizeof(double) * 5 * EIG_LDS4_ROWS * 4)));
            GVQ_HIP(hipFuncSetAttribute((const void*)(inverse_kernel<2, true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)(sizeof(double) * 5 * GVQ_MAX_D * 2)));
            return GVQ_OK;
        });
        if (rc != GVQ_OK) return rc;
        const dim3 grid((unsigned)((a.k + nv - 1) / nv), B);
        if (nv == 4) hipLaunchKernelGGL((inverse_kernel<4, true>), grid, dim3(64), sizeof(double) * 5 * n * 4, st, a);
        else hipLaunchKernelGGL((inverse_kernel<2, true>), grid, dim3(64), sizeof(double) * 5 * n * 2, st, a);
    } else {
        hipLaunchKernelGGL((inverse_kernel<64, false>), dim3((unsigned)((a.k + 63) / 64), B), dim3(64), 0, st, a);
    }
    GVQ_HIP(hipGetLastError());
    if (ortho) {
        const int rc = gvq_launch_orthonormalise(h, a.Z, a.Z_stride, a.k, n, st);
        if (rc != GVQ_OK) return rc;
    }
    if (n > GVQ_EIGEN_SMALL) {
        hipLaunchKernelGGL(wy_kernel, dim3((unsigned)((n - 2 + WY_ROWS - 1) / WY_ROWS), B), dim3(256), 0, st, a);
        GVQ_HIP(hipGetLastError());
        by_long_pieces<go_back_wy>(n, dim3((unsigned)a.k, B), a, st);
        GVQ_HIP(hipGetLastError());
    } else if (n > 2) {
        const dim3 grid((unsigned)((a.k + 3) / 4), B);
        if (n <= 64) hipLaunchKernelGGL((back_kernel<1>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((back_kernel<2>), grid, dim3(256), 0, st, a);
        GVQ_HIP(hipGetLastError());
    }
    return GVQ_OK;
}

EigenArgs gvq_eigen_args(const gvq_basis* h)
{
    EigenArgs a;
    const size_t d = (size_t)h->d;
    a.n = h->d; a.k = h->k;
    a.src = h->d_cov; a.src_stride = d * d;
    a.A = h->d_eA; a.A_stride = (d + 1) * d;
    a.T = h->d_eT; a.t_ld = h->d;
    a.norm = h->d_nsamp + h->B;
    a.eig = h->d_eig; a.eig_ld = h->d;
    a.Z = h->d_eZ; a.Z_stride = (size_t)h->k * d;
    a.wy = h->d_mom; a.wy_stride = d * d + d;   // the covariance is made: the moments are not needed any more
    a.xchg = h->d_eX; a.xchg_stride = 8 * d + 8;
    a.lu = h->d_eLU; a.lanes = 64; a.clamp = 0; a.solves = h->d_solves;
    return a;
}

int gvq_launch_basis_out(const gvq_basis* h, hipStream_t st)
{
    hipLaunchKernelGGL(basis_out_kernel, dim3((unsigned)((h->k + 3) / 4), h->B), dim3(256), 0, st, h->d_eZ,
                       (size_t)h->k * h->d, h->k, h->d, h->d_nsamp + h->B, h->d_U, h->d_solves);
    GVQ_HIP(hipGetLastError());
    return GVQ_OK;
}

int gvq_launch_eigen(const gvq_basis* h, bool from_moments, hipStream_t st)
{
    if (from_moments) {
        int g = (int)(((int64_t)h->d * h->d + 1023) / 1024);
        if (g > 256) g = 256;
        hipLaunchKernelGGL(cov_kernel, dim3(g, h->B), dim3(256), 0, st, h->d_mom, h->d_nsamp, h->d, h->d_cov, h->d_mu,
                           h->d_nsamp + h->B, h->d_solves);
        GVQ_HIP(hipGetLastError());
    }
    const int rc = gvq_launch_sym_eigen(h, gvq_eigen_args(h), true, st);
    return rc != GVQ_OK ? rc : gvq_launch_basis_out(h, st);
}
