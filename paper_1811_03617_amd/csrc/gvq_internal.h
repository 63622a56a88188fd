// Internal declarations shared by the translation units of libgvq (host side only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gvq.h"
#include "gvq_once.h"

#define GVQ_MAX_PTRS 32  // device pointers passed by value in one kernel launch
#define GVQ_EIGEN_SMALL 128      // largest matrix one work-group tridiagonalises in its registers
#define GVQ_NO_CONVERGENCE (1 << 20)   // in place of a number of solves
#define GVQ_SAMPLE_MAX_L 128     // most samples of a first-slice refresh that keeps them centred in memory
#define GVQ_MAX_DEVICES 64       // devices a per-device table of this process has room for

// Many bases: the split of the gradient's 16-slice tiles into super-tiles (G consecutive tiles of
// whole slices of one basis, for the branch-free fast phase of the register-resident codec kernels)
// and the rest, made once per handle.
struct gvq_plan {
    int64_t n_super = 0, n_rest = 0;
    int64_t* d_sup_tile = nullptr;   // [n_super] first 16-slice tile
    int* d_sup_basis = nullptr;      // [n_super] basis
    int64_t* d_rest = nullptr;       // [n_rest] the tiles no super-tile covers
};

struct gvq_basis {
    int64_t M = 0, S = 0;       // elements, slices
    int d = 0, k = 0, B = 0;    // slice length, kept components, number of bases
    gvq_dtype_t dtype = GVQ_F32;
    int device = 0;
    int num_cu = 0;
    int64_t* h_offs = nullptr;  // host [B+1]
    int64_t* d_offs = nullptr;  // device [B+1]
    int* d_tile_block = nullptr;  // device [ceil(S/16)]: basis of the first slice of each 16-slice tile (B > 1)
    gvq_plan plan[2];             // B > 1, register-resident shapes: G = 128/d, and the bf16-pipe compress's G
    int64_t* h_ltile = nullptr; // host [B+1]: first 128-slice tile of each basis (long slices, B > 1)
    int64_t* d_ltile = nullptr; // device copy
    float* d_U = nullptr;       // [B][d][k]
    float* d_mu = nullptr;      // [B][d]
    float* d_Upc = nullptr;     // [B][d][KP] U in compress-MFMA operand order (MFMA shapes only; long slices:
                                // d rounded up to 64, KP = 16 * gvq_long_nt(k))
    float* d_Upd = nullptr;     // [B][d][KP] U in decompress-MFMA operand order
    unsigned short* d_Upb = nullptr;  // [B][d/32][3][NT][64][8] bf16 three-term split of U (bf16 gradients);
                                      // long slices: the two-term copies, compress order then decompress order
    unsigned short* d_Uws = nullptr;  // basis-stationary compress kernel (gvq_ws_shape): two-term bf16 copy of U in its
                                      // operand order, per wave
    float* d_Umu = nullptr;     // [B][KP] U^T mu (bf16 gradients)
    unsigned short* d_Uls = nullptr;  // gvq_monitor.hip: three-term bf16 copies of U for the two products of Eq. 6
    void* d_Ufc = nullptr;      // gvq_flow.h: packed U of its compress kernel (null: no call goes there)
    void* d_Ufd = nullptr;      // ... and of its decompress kernel
    int flow_rows_c = 0, flow_rows_d = 0;   // slices per tile of the two
    int64_t* h_ftile = nullptr; // host [2][B+1]: first tile of each basis, compress then decompress (B > 1)
    void* d_ftile = nullptr;    // those tiles (FlowTile), compress then decompress
    double* d_eig = nullptr;    // [B][d]
    double* d_cov = nullptr;    // [B][d][d]
    double* d_part = nullptr;   // moment partials: [B][mom_part]
    size_t mom_part = 0;        // doubles per basis
    int mom_diag = 1, mom_off = 0;   // sample chunks per panel, and per pair of different panels, of the moments kernel
    int mom_idiag = 1, mom_ioff = 0; // ... and of the int8 moments kernel
    double* d_mom = nullptr;    // [B][d*d+d] reduced moments (sum x x^T, then sum x)
    unsigned long long* d_nsamp = nullptr;  // [B] sample slices the moment kernels of the last fit took in, counted by
                                // them; then [B] largest |entry| of the decomposed matrix, as bits
    double* d_eA = nullptr;     // eigensolver: [B][(d+1) d] matrix, then its reflectors (first-slice refresh: samples too)
    double* d_eT = nullptr;     // [B][5 d] tridiagonal matrix and work vectors
    double* d_eZ = nullptr;     // [B][k][d] eigenvectors
    unsigned long long* d_eX = nullptr;   // d > GVQ_EIGEN_SMALL: [B][8 d + 8] exchange between the work-groups of one matrix
    double* d_eLU = nullptr;    // d > GVQ_EIGEN_SMALL: factors of the inverse iteration
    int* d_solves = nullptr;    // [B] most solves any eigenvector took (0 = zero matrix), or GVQ_NO_CONVERGENCE
    int* d_ksel = nullptr;      // [B] result of the last gvq_select_k
    unsigned long long* h_notes = nullptr;  // pinned host memory that kernels write (null until needed): [0] gvq_fit_status's answer in one word (calls
                                            // that overlap on the same fit write the same one), [1] ticket of the last
                                            // launch that waits inside (gvq_eigen.hip)
    float* d_loss_slice = nullptr;  // [S] per-slice squared residual of the last gvq_local_loss (gvq_monitor.hip: its sums)
    double* d_loss_part = nullptr;  // [B][loss_groups] partial sums of those
    int loss_groups = 1;
    int fit_L = 0;              // gradients of the last fit
    bool fit_first_slice = false;  // the last fit sampled only the first slice of every basis
    bool fitted = false;        // basis usable (fit or import)
    bool has_cov = false;       // d_cov / d_eig hold a fit's results
};

struct gvq_ptrs {
    const void* p[GVQ_MAX_PTRS];
};

// Records the HIP error text for gvq_strerror and returns GVQ_EHIP.
int gvq_hip_fail(hipError_t e, const char* what);

#define GVQ_HIP(call)                                         \
    do {                                                      \
        hipError_t e__ = (call);                              \
        if (e__ != hipSuccess) return gvq_hip_fail(e__, #call); \
    } while (0)

// Workgroups per compute unit for the streaming kernels (0 = pick from occupancy).
int gvq_opt_wg_per_cu();
// Tiles per run in the MFMA kernels' schedule (0 = default).
int gvq_opt_run_tiles();
// LDS-tiled codec kernels: 0 = pick the matrix pipe from the shape, 1 = fp32 products, 2 = the bf16 split,
// 3 = the bf16 split without the basis-stationary compress kernel.
int gvq_opt_long_mode();
// Bit mask: send every tile through the bounds-checked general phase (1: fp32-pipe compress, 2: bf16-pipe
// compress, 4: decompress).
int gvq_opt_no_fast();
// Pacing of the fast phase (CodecArgs::pace), -1 = each kernel's default.
int gvq_opt_pace();
// Super-tiles whose 1 KB rows interleave in the fast phase (CodecArgs::il), 0 = each kernel's default, 1 = none.
int gvq_opt_interleave();
// Polls of the one-launch tridiagonalisation before it gives up, 0 = its default.
int gvq_opt_chain_polls();

// Kernel launchers (each only enqueues on `st`; returns GVQ_OK or GVQ_EHIP).
int gvq_launch_compress(const gvq_basis* h, const void* grad, int n_workers, int64_t first_slice,
                        int64_t n_slices, const float* comp_in, float* out, hipStream_t st);
int gvq_launch_aggregate(const gvq_basis* h, const float* const* comps, int N, float* out,
                         hipStream_t st);
int gvq_launch_decompress(const gvq_basis* h, const float* comp, int64_t first_slice, int64_t n_slices,
                          void* out, gvq_dtype_t odt, hipStream_t st);
int gvq_launch_fit(gvq_basis* h, const void* const* grads, int L, bool first_slice_only, hipStream_t st);
int gvq_launch_local_loss(const gvq_basis* h, const void* grad, int n_workers, double* loss_out,
                          hipStream_t st);
int gvq_launch_local_loss_static(const gvq_basis* h, const void* grad, int n_workers, double* loss_out,
                                 hipStream_t st);
// Eq. 6 on the bf16 matrix pipe (gvq_monitor.hip): one sum per work-group into part [GVQ_LOSS_MAX_PARTS], *parts of them.
#define GVQ_LOSS_MAX_PARTS 1024
bool gvq_loss_split_shape(const gvq_basis* h);
size_t gvq_loss_split_pack_halves(int d);
int gvq_launch_pack_loss(const gvq_basis* h, hipStream_t st);
int gvq_launch_loss_split(const gvq_basis* h, const void* grad, int n_workers, double* part, int* parts, hipStream_t st);
int gvq_launch_layout(const void* src, void* dst, int F, int D, int HW, gvq_dtype_t dtype, bool flatten,
                      hipStream_t st);
int gvq_launch_select_k(const gvq_basis* h, double lambda, hipStream_t st);
// Refresh the operand-order copies of U after d_U changed (no-op for non-MFMA shapes).
int gvq_launch_pack(const gvq_basis* h, hipStream_t st);
bool gvq_mfma_shape(int d, int k);
int gvq_build_plans(gvq_basis* h);   // fills h->plan (needs h_offs; no-op for one basis or other shapes)
bool gvq_bf16_pipe_shape(const gvq_basis* h);
// Moments: chooses the sample chunks (`longest`: slices of the longest basis), returns the partials' doubles per basis.
size_t gvq_moments_plan(gvq_basis* h, int64_t longest);
int gvq_launch_moments(gvq_basis* h, const void* const* grads, int L, hipStream_t st);   // -> d_mom, d_nsamp
// The same on the int8 matrix pipe (gvq_moments_int.hip): whether it can take the handle's slices, and takes a refresh from
// L gradients.
bool gvq_moments_int_shape(const gvq_basis* h);
bool gvq_moments_int_takes(const gvq_basis* h, int L);
size_t gvq_moments_int_plan(gvq_basis* h, int64_t longest);
int gvq_launch_moments_int(gvq_basis* h, const void* const* grads, int L, hipStream_t st);
// Partials -> d_mom.
int gvq_launch_moments_reduce(const gvq_basis* h, int nt, int np, int pw, int chunks_diag, int chunks_off, hipStream_t st);
bool gvq_long_shape(int d, int k);            // codec: the LDS-tiled MFMA kernels take this shape (d > 128, or any
                                              // shape with k <= 128 that the register-resident kernels do not)
size_t gvq_long_pack_floats(int d, int k);    // floats per basis in either operand-order copy of U
size_t gvq_long_split_pack_halves(int d, int k);   // bf16 values per basis in either two-term copy of U
int64_t gvq_long_tiles(int64_t slices);       // 128-slice tiles that cover this many slices of one basis
int gvq_launch_pack_long(const gvq_basis* h, hipStream_t st);
int gvq_launch_compress_long(const gvq_basis* h, const void* grad, int n_workers, int64_t first_slice,
                             int64_t n_slices, const float* comp_in, float* out, hipStream_t st);
int gvq_launch_loss_long(const gvq_basis* h, const void* grad, int n_workers, float* loss_slice, hipStream_t st);
int gvq_launch_decompress_long(const gvq_basis* h, const float* comp, int64_t first_slice, int64_t n_slices,
                               void* out, gvq_dtype_t odt, hipStream_t st);
// The codec kernels of gvq_flow.h; whether they are the ones to take the handle's shape.
bool gvq_flow_takes_compress(const gvq_basis* h);
bool gvq_flow_takes_decompress(const gvq_basis* h, bool out_bf16);
int gvq_flow_alloc(gvq_basis* h);
int gvq_launch_pack_flow(const gvq_basis* h, hipStream_t st);
int gvq_launch_compress_flow(const gvq_basis* h, const void* grad, int n_workers, int64_t first_slice, int64_t n_slices,
                             const float* comp_in, float* out, hipStream_t st);
int gvq_launch_decompress_flow(const gvq_basis* h, const float* comp, int64_t first_slice, int64_t n_slices, void* out,
                               bool out_bf16, hipStream_t st);
// Basis-stationary compress kernel (gvq_codec_ws.hip): U stays in registers, the gradient streams past in tiles
// of 16 whole slices.  The launcher reports the slices done (the whole range, as far as the gradient has slices).
bool gvq_ws_shape(const gvq_basis* h);   // it can take this handle's shape
size_t gvq_ws_pack_halves(int d, int k);   // bf16 values of its operand-order copy of U
bool gvq_wsd_shape(const gvq_basis* h);  // the decompress kernel of the same kind can take the shape
size_t gvq_ws_alloc_halves(const gvq_basis* h);   // bf16 values of d_Uws: both kernels' copies
int gvq_launch_decompress_ws(const gvq_basis* h, const float* comp, int64_t first_slice, int64_t n_slices, void* out,
                             bool out_bf16, bool exact, hipStream_t st, int64_t* done);
int gvq_launch_pack_ws(const gvq_basis* h, hipStream_t st);
int gvq_launch_compress_ws(const gvq_basis* h, const void* grad, int n_workers, int64_t first_slice, int64_t n_slices,
                           const float* comp_in, float* out, bool exact, hipStream_t st, int64_t* done);
size_t gvq_eigen_lu_doubles(int d, int k);   // doubles per basis of d_eLU
// d_cov (made from d_mom first if from_moments) -> d_eig, d_U.
int gvq_launch_eigen(const gvq_basis* h, bool from_moments, hipStream_t st);
void gvq_chain_forget(const gvq_basis* h);   // before the handle goes: nothing of it is queued any more
int gvq_launch_fit_status(const gvq_basis* h, hipStream_t st);   // -> h_notes[0]: most solves, 1 << 32 no convergence, 2 << 32 not finite
bool gvq_sample_shape(int d, int L);         // first-slice refresh: gvq_launch_fit_samples takes it
int gvq_launch_fit_samples(const gvq_basis* h, const void* const* grads, int L, hipStream_t st);
