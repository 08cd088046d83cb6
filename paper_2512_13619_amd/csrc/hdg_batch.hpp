// Internal declarations for batched independent instances.
#pragma once

#include <algorithm>
#include <vector>

#include "hdg_internal.hpp"

// Per-instance descriptor (device copy). Offsets are in elements of each concatenated array.
struct InstDesc {
    int M, D, P, PF, L, nu, nq, nt, nb, S, R, C, NW, KD, ne, nf;
    int64_t e0, f0;                 // first global element / face of the instance
    int64_t off[11];                // Minv, Bd, Cd, D, E, F, G, H, J, ru, rt
    int64_t kbar_off, rbar_off, local_off, du_off, dq_off;
    int64_t K_off, nbr_off, vec_off, f2e_off, e2f_off, binv_off;
};

struct BatchElemPtrs {
    const double *Minv, *Bd, *Cd, *D, *E, *F, *G, *H, *J, *ru, *rt;
};

// Per-instance GMRES state (device). 48 bytes: beta sits at a multiple of 8 bytes.
struct BatchCtl {
    int done, k, nonfinite, pad;
    double beta, est, pad2, pad3;
};

// One block of the face operator: 256 >> lteam faces of instance inst from instance-local face f0,
// 1 << lteam threads a face.
struct FaceBlk {
    int32_t inst, f0, lteam, pad;
};

// Threads of a face with blocks of edge nb (log2): 8, 16 or 32, the fewest that are at least 4 nb and half
// its S*nb columns, or 32: the block's gathered x fits 512 doubles (S*nb <= 64), and a thread has at most 16
// entries (nb = 7, nlfe = 5).
inline int batch_team(int nb, int S) {
    int l = 3;
    while (l < 5 && ((1 << l) < 4 * nb || 2 << l < S * nb)) ++l;
    return l;
}

// Whether an element's condensation is better off with its product in tiles: more than 64 multiply-adds a
// thread of 256 by entries (R rows and columns, depth KD; both sides in k_batch.hip).
inline bool cond_tiles(int R, int KD) { return (R * R + 255) / 256 * KD > 64; }

// Entries of a reduction chunk. 96 instances of 270,000 unknowns in all give 580 blocks.
constexpr int SEG_CHUNK = 512;

// Chunks times columns above which an instance's partial inner products are added up once for all its
// blocks, by a kernel of its own, instead of by every block: the blocks' reads grow with the square of
// the instance's size. One instance, time of a step with both CGS2 passes: 100,000 unknowns (196
// chunks), 30 columns 49.5 us by every block, 52.2 once; 100 columns 79.2 and 76.3; 272,000, 30
// columns 84.0 and 83.6; 10^6, 30 columns 271 and 225; 8 10^6 5490 and 1690.
constexpr int SEG_DIRECT = 8192;

// One Gram-Schmidt sweep (k_seg_sweep): w against the J basis vectors V. part_in: the sweep's
// coefficients as the partials of the sweep before (coef: their sums, ld_coef per instance, for instances
// above SEG_DIRECT); col: this step's Hessenberg column (stride ld_col per instance), set or added to. The
// index arrays are the launcher's to fill in.
struct SegSweep {
    const double* V;
    size_t ldv;
    int J;
    double* w;
    const double* part_in;
    double* coef;
    int ld_coef;
    double* part_out;
    double* col;
    int ld_col, add;
    const BatchCtl* ctl;
    const int32_t *blk_inst, *ib0, *ib1;
    const int64_t *blk_lo, *blk_hi;
    int nblk;
};

struct BatchDev {
    InstDesc* desc = nullptr;
    int32_t* eid = nullptr;         // [total_ne] instance of each element
    int32_t* fid = nullptr;         // [total_nf]
    FaceBlk* fblk = nullptr;        // [nfblk] blocks of the face operator
    int32_t* dof_inst = nullptr;    // [total_dof]
    int32_t* blk_inst = nullptr;    // [nblk] reduction chunks (never straddle instances)
    int64_t* blk_lo = nullptr;
    int64_t* blk_hi = nullptr;
    int32_t* ib0 = nullptr;         // [n_inst] first / one-past-last chunk of each instance
    int32_t* ib1 = nullptr;
    int n_inst = 0, nblk = 0, nfblk = 0, max_chunks = 0;
    int64_t total_ne = 0, total_nf = 0, total_dof = 0;
    size_t max_cond_lds = 0, max_rec_lds = 0;
    bool tiles = false;             // condensation by tiles: one kernel for all elements: the one for most of the multiply-adds
    int max_nb = 0, max_snb = 0, max_R = 0;
};

// Batched element residuals / Jacobian blocks (scalar convection-diffusion models): per
// instance its sizes, the offsets of its parts of the concatenated geometry arrays and of
// the batch arrays it reads and writes, and its model coefficients.
struct ElemInst {
    int P, PF, L, D, Qv, Qf;
    int64_t e0;
    int64_t g_wdet, g_dphix, g_phi, g_phif, g_psi, g_ndA, g_dA, g_src, g_uD;
    int64_t e2f_off, u_off, uh_off, q_off;
    int64_t out_off[11];            // Minv, Bd, Cd, D, E, F, G, H, J, ru, rt
    double nu, tau, beta[3], gamma[3];
    double c;                       // time-term factor of the instance (0: steady)
};

struct ElemBatchArgs {
    hdg_elem_geom g;                // concatenated arrays (nqv, nqf unused)
    const int32_t* e2f;
    const double *u, *uhat, *u_prev;   // u_prev: batch array like u (read where c != 0)
    const double* r_extra;             // batch array like u, or null (known stage term)
    hdg_elem_arrays out;
    int* bad;
    int residual_only, keep_mass;
};

size_t element_batch_lds_bytes(int P, int PF, int L, int D, int nqv, int nqf);
hdg_status element_blocks_batch_run(hdg_ctx ctx, int64_t total_ne, const ElemInst* inst_dev, const int32_t* eid,
                                    const ElemBatchArgs& a, size_t lds);
hdg_status residual_norm_batch_run(hdg_ctx ctx, int n_inst, const InstDesc* desc, const double* ru, const double* rt,
                                   const int32_t* f2e, double* norms);
hdg_status newton_update_batch_run(hdg_ctx ctx, int n_inst, const InstDesc* desc, const double* alpha,
                                   const double* du, double* u, const double* x, double* uhat);

hdg_status batch_launch_condense(hdg_ctx ctx, const BatchDev& b, const BatchElemPtrs& in, double* Kbar, double* rbar,
                                 double* local, int* bad, int grid);
hdg_status batch_launch_assemble(hdg_ctx ctx, const BatchDev& b, const int32_t* f2e, const int32_t* e2f,
                                 const double* Kbar, const double* rbar, double* K64, float* K32, int32_t* nbr,
                                 double* r);
hdg_status batch_launch_face(hdg_ctx ctx, const BatchDev& b, const void* M1, bool fp32, const int32_t* nbr,
                             bool bj_only, double* x, double* out, double s0, const double* X, double a0,
                             const double* denom, int ld_denom, const BatchCtl* ctl);
hdg_status batch_launch_bj(hdg_ctx ctx, const BatchDev& b, const double* K64, double* B64, float* B32, int* bad);
hdg_status seg_sweep(hdg_ctx ctx, const BatchDev& b, SegSweep a, bool axpy, bool dot);
hdg_status seg_reduce(hdg_ctx ctx, const BatchDev& b, const double* part, double* out, int ldo);
hdg_status seg_update(hdg_ctx ctx, const BatchDev& b, const double* Z, size_t ldz, const double* y, int ldy, double* x,
                      const BatchCtl* ctl);
hdg_status seg_sumsq(hdg_ctx ctx, const BatchDev& b, const double* w, double* part, const BatchCtl* ctl);
hdg_status seg_scale(hdg_ctx ctx, const BatchDev& b, double* v, const double* denom, int ld_denom,
                     const BatchCtl* ctl);
hdg_status seg_cycle_init(hdg_ctx ctx, const BatchDev& b, const double* part, BatchCtl* ctl, double* g, int ldg,
                          int jmax, const double* target);
hdg_status seg_givens(hdg_ctx ctx, const BatchDev& b, const double* part, BatchCtl* ctl, double* H, int ldh, int mcols,
                      double* cs, double* sn, double* g, int ldg, int j, int jmax, const double* target);
hdg_status seg_backsolve(hdg_ctx ctx, const BatchDev& b, const BatchCtl* ctl, const double* H, int ldh, int mcols,
                         const double* g, int ldg, double* y);
hdg_status batch_launch_recover(hdg_ctx ctx, const BatchDev& b, const double* local, const double* Minv,
                                const double* Bd, const double* Cd, const int32_t* e2f, const double* xhat,
                                double* du, double* dq);
