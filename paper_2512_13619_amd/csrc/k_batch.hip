// Batched independent instances (many small uneven meshes, degrees and element
// types in one set of launches): condensation in one persistent launch with the
// whole element system in LDS, face-parallel assembly, a face-block operator
// whose faces carry their instance's block size, and segmented Krylov kernels
// with per-instance reductions, Givens updates and convergence masks.
//
// The arithmetic per element/face/instance is the same as in the single-instance
// kernels (Section 4.1 eq. w15-w19, Section 4.2 eq. w21-w22, Section 4.3-4.5);
// only the indexing differs: every element, face and vector entry looks up its
// instance descriptor.
#include <cmath>

#include "hdg_batch.hpp"
#include "wave_ops.hpp"

namespace {

constexpr int BS = 256;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// ---- condensation: one element per workgroup iteration, all in LDS ------------------------
// Bound by the elimination's chain of pivots: three barriers a pivot, the update in a 16 x 16 grid of
// threads (entries numbered through cost a division each, and the multipliers a barrier of their own), and
// by the latency of the element's arrays, which are read once. The product with W: 16x16 tiles on the
// matrix cores, or an entry per thread for small elements (cond_tiles), where few waves have a tile and the
// tiles' 112 registers let only four waves share a SIMD (seven by entries). 8000 elements, us by tiles and by
// entries (multiply-adds a thread): p = 1 quads 119, 97 (8); p = 2 quads 217, 207 (36); p = 1 quads with three
// components 285, 246 (48); p = 1 hexes 240, 301 (96); p = 4 triangles 382, 467 (120); p = 4 quads 1066, 1820
// (400). 96 mixed instances: 4.05 ms by entries, 2.6 by tiles.
template <bool TILES>
__global__ __launch_bounds__(BS) void k_batch_condense(const InstDesc* __restrict__ desc,
                                                       const int32_t* __restrict__ eid, int64_t total_ne,
                                                       BatchElemPtrs in, double* __restrict__ Kbar,
                                                       double* __restrict__ rbar, double* __restrict__ local,
                                                       int* bad_elem) {
    extern __shared__ double sm[];
    __shared__ int pidx;
    __shared__ double pval;
    for (int64_t g = blockIdx.x; g < total_ne; g += gridDim.x) {
        const InstDesc& q = desc[eid[g]];
        const int64_t le = g - q.e0;
        const int P = q.P, D = q.D, M = q.M, PF = q.PF, L = q.L;
        const int nu = q.nu, nq = q.nq, nt = q.nt, R = q.R, C = q.C, NW = q.NW, KD = q.KD, LPF = L * PF;
        double* T = sm;                        // R x C (row stride C)
        double* W = sm + (size_t)R * C;        // KD x NW
        const double* Mi = in.Minv + q.off[0] + le * P * P;
        const double* Bd = in.Bd + q.off[1] + le * D * P * P;
        const double* Cd = in.Cd + q.off[2] + le * D * P * LPF;
        const double* Dm = in.D + q.off[3] + le * nu * nq;
        const double* Em = in.E + q.off[4] + le * nu * nu;
        const double* Fm = in.F + q.off[5] + le * nu * nt;
        const double* Gm = in.G + q.off[6] + le * nt * nq;
        const double* Hm = in.H + q.off[7] + le * nt * nu;
        const double* Jm = in.J + q.off[8] + le * nt * nt;
        const double* ru = in.ru + q.off[9] + le * nu;
        const double* rt = in.rt + q.off[10] + le * nt;
        const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
        // W = Minv [B_d | C_d]
        {
            const int dr = BS / NW, dc = BS - dr * NW;
            for (int idx = threadIdx.x, r = idx / NW, c = idx - r * NW; idx < KD * NW; idx += BS, r += dr, c += dc) {
                if (c >= NW) {
                    c -= NW;
                    ++r;
                }
                const int d = (r >= P) + (r >= 2 * P), i = r - d * P;
                const double* b = c < P ? Bd + (size_t)d * P * P + c : Cd + (size_t)d * P * LPF + (c - P);
                const int ldb = c < P ? P : LPF;
                double acc = 0.0;
                for (int k = 0; k < P; ++k) acc += Mi[(size_t)i * P + k] * b[(size_t)k * ldb];
                W[idx] = acc;
            }
        }
        __syncthreads();
        // T = T0 - X W, column-mapped per component
        const int NC = nu + nt;
        auto x_row = [&](int r) { return r < nu ? Dm + (size_t)r * nq : Gm + (size_t)(r - nu) * nq; };
        auto t0_at = [&](int r, int t) {          // t < nu: columns of u, then of the trace
            if (t < nu) return r < nu ? Em[(size_t)r * nu + t] : Hm[(size_t)(r - nu) * nu + t];
            return r < nu ? Fm[(size_t)r * nt + t - nu] : Jm[(size_t)(r - nu) * nt + t - nu];
        };
        if constexpr (!TILES) {
            const int dr = BS / NC, dc = BS - dr * NC;
            for (int idx = threadIdx.x, r = idx / NC, t = idx - r * NC; idx < R * NC; idx += BS, r += dr, t += dc) {
                if (t >= NC) {
                    t -= NC;
                    ++r;
                }
                const int l = (t - nu) / (M * PF), tr = t - nu - l * M * PF;
                const int m = t < nu ? t / P : tr / PF, c = t < nu ? t - m * P : P + l * PF + tr - m * PF;
                const double* X = x_row(r) + m * KD;
                const double t0 = t0_at(r, t);
                double acc = 0.0;
                for (int k = 0; k < KD; ++k) acc += X[k] * W[k * NW + c];
                T[r * C + t] = t0 - acc;
            }
        } else {
            const int wave = threadIdx.x >> 6, l16 = threadIdx.x & 15, lq = (threadIdx.x & 63) >> 4;
            int job = 0;
            for (int m = 0; m < M; ++m)
                for (int r0 = 0; r0 < R; r0 += 16)
                    for (int c0 = 0; c0 < NW; c0 += 16) {
                        if ((job++ & (BS / 64 - 1)) != wave) continue;
                        const int r = r0 + l16 < R ? r0 + l16 : R - 1, c = c0 + l16 < NW ? c0 + l16 : NW - 1;
                        const int l = (c - P) / PF, t = c < P ? m * P + c : nu + (l * M + m) * PF + (c - P - l * PF);
                        double t0[4];                 // on its way with the product's operands
#pragma unroll
                        for (int q4 = 0; q4 < 4; ++q4) t0[q4] = t0_at(r0 + 4 * q4 + lq < R ? r0 + 4 * q4 + lq : R - 1, t);
                        wave_ops::d4 acc = {};
                        wave_ops::mma16s<false, false>(KD, wave_ops::seq(x_row(r) + m * KD, 1), wave_ops::seq(W + c, NW), acc);
                        if (c0 + l16 >= NW) continue;
#pragma unroll
                        for (int q4 = 0; q4 < 4; ++q4)
                            if (r0 + 4 * q4 + lq < R) T[(r0 + 4 * q4 + lq) * C + t] = t0[q4] - acc[q4];
                    }
        }
        for (int r = threadIdx.x; r < R; r += BS) T[(size_t)r * C + C - 1] = r < nu ? ru[r] : rt[r - nu];
        __syncthreads();
        // eliminate the first nu columns, pivots among the Ebar rows; the multipliers of column k that are
        // stored (the Ebar rows') are written back while wave 0 looks for the next pivot
        bool singular = false;
        double inv = 0.0;
        for (int k = 0; k < nu; ++k) {
            if (threadIdx.x >= 64 && k > 0) {
                for (int i = k + threadIdx.x - 64; i < nu; i += BS - 64) T[i * C + k - 1] *= inv;
            } else if (threadIdx.x < 64) {
                double best = -1.0;
                int bi = k;
                for (int i = k + threadIdx.x; i < nu; i += 64) {
                    const double v = fabs(T[i * C + k]);
                    if (v > best || (v == best && i < bi)) { best = v; bi = i; }
                }
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) {
                    const double ob = __shfl_xor(best, off, 64);
                    const int oi = __shfl_xor(bi, off, 64);
                    if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
                }
                if (threadIdx.x == 0) { pidx = bi; pval = T[bi * C + k]; }
            }
            __syncthreads();
            const int p = pidx;
            double pv = pval;
            if (!(fabs(pv) > 0.0) || !isfinite(pv)) { singular = true; pv = 1.0; }
            if (p != k)
                for (int c = k + threadIdx.x; c < C; c += BS) {
                    const double t = T[k * C + c];
                    T[k * C + c] = T[p * C + c];
                    T[p * C + c] = t;
                }
            __syncthreads();
            inv = 1.0 / pv;
            for (int i = k + 1 + ty; i < R; i += BS / 16) {
                const double f = T[i * C + k] * inv;
                for (int c = k + 1 + tx; c < C; c += 16) T[i * C + c] -= f * T[k * C + c];
            }
            __syncthreads();
        }
        if (singular && threadIdx.x == 0) atomicMin(bad_elem, (int)g);
        double* lo = local + q.local_off + le * nu * C;
        for (int idx = threadIdx.x; idx < nu * C; idx += BS) lo[idx] = T[idx];
        double* Ko = Kbar + q.kbar_off + le * nt * nt;
        for (int idx = threadIdx.x; idx < nt * nt; idx += BS) {
            const int i = idx / nt, j = idx - i * nt;
            Ko[idx] = T[(size_t)(nu + i) * C + nu + j];
        }
        for (int i = threadIdx.x; i < nt; i += BS) rbar[q.rbar_off + le * nt + i] = T[(size_t)(nu + i) * C + C - 1];
        __syncthreads();
    }
}

// ---- assembly --------------------------------------------------------------------------------
__global__ __launch_bounds__(BS) void k_batch_assemble(const InstDesc* __restrict__ desc,
                                                       const int32_t* __restrict__ fid, int64_t total_nf,
                                                       const int32_t* __restrict__ f2e, const int32_t* __restrict__ e2f,
                                                       const double* __restrict__ Kbar, const double* __restrict__ rbar,
                                                       double* __restrict__ K64, float* __restrict__ K32,
                                                       int32_t* __restrict__ nbr, double* __restrict__ r) {
    __shared__ int se[16], slr[16], slc[16];
    for (int64_t g = blockIdx.x; g < total_nf; g += gridDim.x) {
        const InstDesc& q = desc[fid[g]];
        const int64_t f = g - q.f0;
        const int M = q.M, PF = q.PF, L = q.L, nb = q.nb, S = q.S, nt = q.nt;
        const int32_t* f2 = f2e + q.f2e_off + 4 * f;
        const int e1 = f2[0], l1 = f2[1], e2 = f2[2], l2 = f2[3];
        if (threadIdx.x == 0) {
            int s = 0;
            se[s] = e1; slr[s] = l1; slc[s] = l1; ++s;
            for (int l = 0; l < L; ++l)
                if (l != l1) { se[s] = e1; slr[s] = l1; slc[s] = l; ++s; }
            for (int l = 0; l < L; ++l) {
                if (e2 >= 0) {
                    if (l != l2) { se[s] = e2; slr[s] = l2; slc[s] = l; ++s; }
                } else if (l != 0) {
                    se[s] = -1; slr[s] = 0; slc[s] = 0; ++s;
                }
            }
        }
        __syncthreads();
        for (int s = threadIdx.x; s < S; s += BS) {
            int gg = -1;
            if (s == 0) gg = (int)f;
            else if (se[s] >= 0) gg = e2f[q.e2f_off + (int64_t)se[s] * L + slc[s]];
            nbr[q.nbr_off + f * S + s] = gg;
        }
        const int64_t blk = (int64_t)nb * nb;
        for (int s = 0; s < S; ++s) {
            const int e = se[s];
            double* out = K64 + q.K_off + (f * S + s) * blk;
            float* out32 = K32 ? K32 + q.K_off + (f * S + s) * blk : nullptr;
            for (int idx = threadIdx.x; idx < (int)blk; idx += BS) {
                const int c = idx / nb, rr = idx - c * nb;
                double v = 0.0;
                if (e >= 0) {
                    const int mr = rr / PF, jr = rr - mr * PF, mc = c / PF, jc = c - mc * PF;
                    const double* Ke = Kbar + q.kbar_off + (int64_t)e * nt * nt;
                    v = Ke[(int64_t)((slr[s] * M + mr) * PF + jr) * nt + (slc[s] * M + mc) * PF + jc];
                    if (s == 0 && e2 >= 0) {
                        const double* K2 = Kbar + q.kbar_off + (int64_t)e2 * nt * nt;
                        v += K2[(int64_t)((l2 * M + mr) * PF + jr) * nt + (l2 * M + mc) * PF + jc];
                    }
                }
                out[idx] = v;
                if (out32) out32[idx] = (float)v;
            }
        }
        for (int rr = threadIdx.x; rr < nb; rr += BS) {
            const int m = rr / PF, j = rr - m * PF;
            double v = rbar[q.rbar_off + (int64_t)e1 * nt + (l1 * M + m) * PF + j];
            if (e2 >= 0) v += rbar[q.rbar_off + (int64_t)e2 * nt + (l2 * M + m) * PF + j];
            r[q.vec_off + f * nb + rr] = v;
        }
        __syncthreads();
    }
}

// ---- face-block operator -----------------------------------------------------------------------
// u_f = sum_s M1[f][s] x_{nbr[f][s]} (or the block-diagonal product when bj_only), then
// out_f = s0 u_f + a0 X_f (X may be null); faces of finished instances are skipped.
// bj_only with denom: x_f is first divided by its instance's denom[inst * ld_denom] and written back
// (the normalisation of a new basis vector, which only its own face reads here).
// Bound by latency at these sizes (a face is 0.1 to 1.4 KB of FP32 blocks): a block's faces are of
// one instance, whose descriptor then comes by scalar loads, a face has the fewest threads that
// leave each a handful of entries (batch_team), so that fewer waves pass through the chain of
// dependent loads, and the first FU block entries of every thread are on their way before the
// neighbour numbers and x are gathered (96 instances: 9.3 us a launch; 32 threads for every face and
// a descriptor looked up per face 16.8).
template <typename T>
__global__ __launch_bounds__(BS) void k_batch_face(const InstDesc* __restrict__ desc,
                                                   const FaceBlk* __restrict__ fblk,
                                                   const T* __restrict__ M1, const int32_t* __restrict__ nbr,
                                                   int bj_only, double* x, double* out,
                                                   double s0, const double* X, double a0,
                                                   const double* denom, int ld_denom, const BatchCtl* ctl) {
    constexpr int FU = 8;
    __shared__ double sm[512], red[BS];
    const FaceBlk fb = fblk[blockIdx.x];
    const int inst = fb.inst;
    if (ctl && ctl[inst].done) return;
    const InstDesc& q = desc[inst];
    const int lteam = fb.lteam, TEAM = 1 << lteam, team = threadIdx.x >> lteam, t = threadIdx.x & (TEAM - 1);
    const int nb = q.nb, S = bj_only ? 1 : q.S, L = q.L, cols = S * nb;
    const int fl = fb.f0 + team;
    const bool live = fl < q.nf;
    const int64_t f = live ? fl : q.nf - 1;
    double* xs = sm + team * q.S * nb;         // BS / TEAM faces of S*nb <= 2 TEAM entries
    const int G = TEAM / nb, grp = t / nb, row = t - grp * nb;
    const bool mine = grp < G;
    const T* Mf = M1 + (bj_only ? q.binv_off : q.K_off) + f * cols * nb;
    T a[FU];
#pragma unroll
    for (int u = 0; u < FU; ++u) {
        const int k = grp + u * G;
        a[u] = (mine && k < cols) ? Mf[k * nb + row] : (T)0;        // an empty slot's entries are not used
    }
    // a boundary face's empty slots are its last: entries past ncols are neither gathered nor used
    bool empty = false;
    for (int i = t; i < cols; i += TEAM) {
        const int s = i / nb, c = i - s * nb;
        const int64_t gg = bj_only ? f : nbr[q.nbr_off + f * S + s];
        double v = 0.0;
        if (gg >= 0) {
            double* xp = x + q.vec_off + gg * nb + c;
            v = *xp;
            if (denom) {
                v /= denom[(size_t)inst * ld_denom];
                if (live) *xp = v;
            }
        } else {
            empty = empty || s >= L;
        }
        xs[i] = v;
    }
    const uint64_t any = __ballot(empty) >> (threadIdx.x & 63 & ~(TEAM - 1)) & ((TEAM < 64 ? 1ull << TEAM : 0ull) - 1);
    const int ncols = any ? L * nb : cols;
    __syncthreads();
    double acc = 0.0;
    if (mine) {
#pragma unroll
        for (int u = 0; u < FU; ++u) {
            const int k = grp + u * G;
            if (k < ncols) acc += (double)a[u] * xs[k];
        }
        for (int k = grp + FU * G; k < ncols; k += G) acc += (double)Mf[k * nb + row] * xs[k];
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    if (live && t < nb) {
        double u = 0.0;
        for (int g2 = 0; g2 < G; ++g2) u += red[team * TEAM + g2 * nb + t];
        const int64_t idx = q.vec_off + f * nb + t;
        double v = s0 * u;
        if (X) v += a0 * X[idx];
        out[idx] = v;
    }
}

// ---- block-Jacobi inverses (Gauss-Jordan, partial pivoting), one face per workgroup -------------
__global__ __launch_bounds__(BS) void k_batch_bj(const InstDesc* __restrict__ desc, const int32_t* __restrict__ fid,
                                                 int64_t total_nf, const double* __restrict__ K, double* B64,
                                                 float* B32, int* bad_face) {
    __shared__ double A[16 * 33];
    __shared__ int ps;
    for (int64_t g = blockIdx.x; g < total_nf; g += gridDim.x) {
        const InstDesc& q = desc[fid[g]];
        const int64_t f = g - q.f0;
        const int nb = q.nb, lda = 2 * nb + 1;
        const double* Kf = K + q.K_off + f * q.S * nb * nb;
        for (int idx = threadIdx.x; idx < nb * nb; idx += BS) {
            const int c = idx / nb, r = idx - c * nb;
            A[r * lda + c] = Kf[idx];
            A[r * lda + nb + c] = (r == c) ? 1.0 : 0.0;
        }
        __syncthreads();
        bool singular = false;
        for (int k = 0; k < nb; ++k) {
            if (threadIdx.x == 0) {
                int p = k;
                for (int r = k + 1; r < nb; ++r)
                    if (fabs(A[r * lda + k]) > fabs(A[p * lda + k])) p = r;
                ps = p;
            }
            __syncthreads();
            const int p = ps;
            if (p != k)
                for (int c = threadIdx.x; c < 2 * nb; c += BS) {
                    const double t = A[k * lda + c];
                    A[k * lda + c] = A[p * lda + c];
                    A[p * lda + c] = t;
                }
            __syncthreads();
            double pv = A[k * lda + k];
            if (!(fabs(pv) > 0.0) || !isfinite(pv)) { singular = true; pv = 1.0; }
            __syncthreads();
            for (int c = threadIdx.x; c < 2 * nb; c += BS) A[k * lda + c] /= pv;
            __syncthreads();
            for (int idx = threadIdx.x; idx < nb * 2 * nb; idx += BS) {
                const int r = idx / (2 * nb), c = idx - r * (2 * nb);
                if (r == k || c == k) continue;
                A[r * lda + c] -= A[r * lda + k] * A[k * lda + c];
            }
            __syncthreads();
            for (int r = threadIdx.x; r < nb; r += BS)
                if (r != k) A[r * lda + k] = 0.0;
            __syncthreads();
        }
        if (singular && threadIdx.x == 0) atomicMin(bad_face, (int)g);
        for (int idx = threadIdx.x; idx < nb * nb; idx += BS) {
            const int c = idx / nb, r = idx - c * nb;
            B64[q.binv_off + f * nb * nb + idx] = A[r * lda + nb + c];
            if (B32) B32[q.binv_off + f * nb * nb + idx] = (float)A[r * lda + nb + c];
        }
        __syncthreads();
    }
}

// ---- segmented Krylov kernels -------------------------------------------------------------------
// Block b covers entries [blk_lo[b], blk_hi[b]) of instance blk_inst[b] (at most SEG_CHUNK; chunks
// never straddle two instances). part[i * nblk + b].
// One Gram-Schmidt sweep over an instance's basis: the coefficients h_i = sum_b part_in[i][b] of the
// sweep before (AXPY; every block of the instance adds them up in the same order, or k_seg_coef has
// done it in that order for all, see SEG_DIRECT; its first block puts them into the Hessenberg
// column), w -= V h, then the partial inner products V^T w (DOT) or
// ||w||^2. A wave takes four columns at a time with all their loads in flight; a sweep by one column
// after another, with reductions in kernels of their own, took 31 + 4 + 7 us a sweep for 96
// instances (270,000 unknowns, up to 30 columns, averages over cycles in which ever fewer are
// active); this one 7 (DOT), 11 (both) and 8 us (AXPY).
constexpr int SEG_U = SEG_CHUNK / 64, SEG_C = 4;
template <bool AXPY, bool DOT>
__global__ __launch_bounds__(BS) void k_seg_sweep(SegSweep a) {
    __shared__ double hs[AXPY ? 200 : 1], ws[SEG_CHUNK], red[BS / 64];
    const int b = blockIdx.x, inst = a.blk_inst[b];
    if (a.ctl[inst].done) return;
    const int64_t k0 = a.blk_lo[b];
    const int len = (int)(a.blk_hi[b] - k0), J = a.J, nblk = a.nblk;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double* V = a.V + k0;
    double* w = a.w + k0;
    if constexpr (AXPY) {
        const int b0 = a.ib0[inst], b1 = a.ib1[inst];
        if ((int64_t)(b1 - b0) * J > SEG_DIRECT) {
            for (int i = threadIdx.x; i < J; i += BS) hs[i] = a.coef[(size_t)inst * a.ld_coef + i];
        } else {
            for (int i = wave * SEG_C; i < J; i += (BS / 64) * SEG_C) {
                double s[SEG_C] = {};
                for (int q = b0 + lane; q < b1; q += 64)
#pragma unroll
                    for (int c = 0; c < SEG_C; ++c) s[c] += a.part_in[(size_t)(i + c < J ? i + c : i) * nblk + q];
#pragma unroll
                for (int c = 0; c < SEG_C; ++c) {
                    const double h = wave_ops::wave_sum_all(s[c]);
                    if (lane == 0 && i + c < J) hs[i + c] = h;
                }
            }
        }
        __syncthreads();
        if (b == b0) {
            double* col = a.col + (size_t)inst * a.ld_col;
            for (int i = threadIdx.x; i < J; i += BS) col[i] = a.add ? col[i] + hs[i] : hs[i];
        }
        constexpr int E = SEG_CHUNK / BS;
        double acc[E] = {};
        for (int i = 0; i < J; i += 8) {
            double v[8][E];
#pragma unroll
            for (int c = 0; c < 8; ++c)
#pragma unroll
                for (int u = 0; u < E; ++u) {
                    const int k = threadIdx.x + u * BS;
                    v[c][u] = V[(size_t)(i + c < J ? i + c : i) * a.ldv + (k < len ? k : 0)];
                }
#pragma unroll
            for (int c = 0; c < 8; ++c)
#pragma unroll
                for (int u = 0; u < E; ++u)
                    if (i + c < J) acc[u] += v[c][u] * hs[i + c];
        }
        double ss = 0.0;
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const int k = threadIdx.x + u * BS;
            const double r = k < len ? w[k] - acc[u] : 0.0;
            if (k < len) w[k] = r;
            if constexpr (DOT) ws[k] = r;
            ss += r * r;
        }
        if constexpr (!DOT) {
            ss = wave_ops::wave_sum_all(ss);
            if (lane == 0) red[wave] = ss;
            __syncthreads();
            if (threadIdx.x == 0) a.part_out[b] = (red[0] + red[1]) + (red[2] + red[3]);
            return;
        }
    } else {
        for (int k = threadIdx.x; k < SEG_CHUNK; k += BS) ws[k] = k < len ? w[k] : 0.0;
    }
    if constexpr (DOT) {
        __syncthreads();
        double wr[SEG_U];
#pragma unroll
        for (int u = 0; u < SEG_U; ++u) wr[u] = ws[lane + 64 * u];
        for (int i = wave * SEG_C; i < J; i += (BS / 64) * SEG_C) {
            double v[SEG_C][SEG_U];
#pragma unroll
            for (int c = 0; c < SEG_C; ++c)
#pragma unroll
                for (int u = 0; u < SEG_U; ++u) {
                    const int k = lane + 64 * u;
                    v[c][u] = V[(size_t)(i + c < J ? i + c : i) * a.ldv + (k < len ? k : 0)];
                }
#pragma unroll
            for (int c = 0; c < SEG_C; ++c) {
                double s = 0.0;
#pragma unroll
                for (int u = 0; u < SEG_U; ++u)
                    if (lane + 64 * u < len) s += v[c][u] * wr[u];
                s = wave_ops::wave_sum_all(s);
                if (lane == 0 && i + c < J) a.part_out[(size_t)(i + c) * nblk + b] = s;
            }
        }
    }
}

// coef[inst][i] = sum of part_in[i] over the instance's blocks, for instances above SEG_DIRECT; one wave
// per sum
__global__ void k_seg_coef(SegSweep a, int n_inst) {
    const int64_t w = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (w >= (int64_t)n_inst * a.J) return;
    const int inst = (int)(w / a.J), i = (int)(w - (int64_t)inst * a.J), lane = threadIdx.x & 63;
    const int b0 = a.ib0[inst], b1 = a.ib1[inst];
    if ((int64_t)(b1 - b0) * a.J <= SEG_DIRECT || a.ctl[inst].done) return;
    double s = 0.0;
    for (int q = b0 + lane; q < b1; q += 64) s += a.part_in[(size_t)i * a.nblk + q];
    s = wave_ops::wave_sum_all(s);
    if (lane == 0) a.coef[(size_t)inst * a.ld_coef + i] = s;
}

// out[inst * ldo] = sum of part[b] over the instance's blocks; one wave per instance
__global__ void k_seg_reduce(const int32_t* __restrict__ ib0, const int32_t* __restrict__ ib1, int n_inst,
                             const double* __restrict__ part, double* out, int ldo) {
    const int inst = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (inst >= n_inst) return;
    double s = 0.0;
    for (int b = ib0[inst] + lane; b < ib1[inst]; b += 64) s += part[b];
    s = wave_sum(s);
    if (lane == 0) out[(size_t)inst * ldo] = s;
}

// x[k] += sum_{i<k_inst} Z[i][k] y[inst(k)][i] with k_inst the instance's steps this cycle
__global__ __launch_bounds__(BS) void k_seg_update(const int32_t* __restrict__ dof_inst, const double* __restrict__ Z,
                                                   size_t ldz, const double* __restrict__ y, int ldy, double* x,
                                                   size_t n, const BatchCtl* ctl) {
    const size_t k = (size_t)blockIdx.x * BS + threadIdx.x;
    if (k >= n) return;
    const int inst = dof_inst[k];
    const int J = ctl[inst].k;
    const double* yy = y + (size_t)inst * ldy;
    double acc = 0.0;
    for (int i = 0; i < J; i += 8) {
        double z[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) z[c] = Z[(size_t)(i + c < J ? i + c : i) * ldz + k];
#pragma unroll
        for (int c = 0; c < 8; ++c)
            if (i + c < J) acc += z[c] * yy[i + c];
    }
    x[k] += acc;
}

__global__ __launch_bounds__(BS) void k_seg_sumsq(const int32_t* __restrict__ blk_inst,
                                                  const int64_t* __restrict__ blk_lo, const int64_t* __restrict__ blk_hi,
                                                  const double* __restrict__ w, double* part, const BatchCtl* ctl) {
    __shared__ double red[BS / 64];
    const int b = blockIdx.x;
    if (ctl && ctl[blk_inst[b]].done) return;
    double acc = 0.0;
    for (int64_t k = blk_lo[b] + threadIdx.x; k < blk_hi[b]; k += BS) acc += w[k] * w[k];
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) part[b] = red[0] + red[1] + red[2] + red[3];
}

__global__ __launch_bounds__(BS) void k_seg_scale(const int32_t* __restrict__ dof_inst, double* v, size_t n,
                                                  const double* denom, int ld_denom, const BatchCtl* ctl) {
    const size_t k = (size_t)blockIdx.x * BS + threadIdx.x;
    if (k >= n) return;
    const int inst = dof_inst[k];
    if (ctl[inst].done) return;
    v[k] /= denom[(size_t)inst * ld_denom];
}

// per instance: beta from the residual partials, cycle state
__global__ void k_seg_cycle_init(const int32_t* __restrict__ ib0, const int32_t* __restrict__ ib1, int n_inst,
                                 const double* part, BatchCtl* ctl, double* g, int ldg, int jmax,
                                 const double* target) {
    const int inst = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (inst >= n_inst) return;
    double s = 0.0;
    for (int b = ib0[inst] + lane; b < ib1[inst]; b += 64) s += part[b];
    s = wave_sum(s);
    if (lane == 0) {
        BatchCtl& c = ctl[inst];
        const double beta = sqrt(s);
        c.beta = beta;
        c.est = beta;
        c.k = 0;
        c.nonfinite = !isfinite(beta);
        c.done = (beta <= target[inst] || !isfinite(beta) || jmax <= 0) ? 1 : 0;
        g[(size_t)inst * ldg] = beta;
    }
}

// One wave per instance: ||w|| from the sweep's partials, the earlier rotations on the new column (the
// column and the rotations staged in LDS: the chain of dependent updates then waits on no memory),
// the new rotation and the residual estimate.
__global__ __launch_bounds__(64) void k_seg_givens(const int32_t* __restrict__ ib0, const int32_t* __restrict__ ib1,
                                                   const double* part, BatchCtl* ctl, double* H, int ldh, int mcols,
                                                   double* cs, double* sn, double* g, int ldg, int j, int jmax,
                                                   const double* target) {
    __shared__ double sc[201], cc_s[200], ss_s[200];
    const int inst = blockIdx.x, lane = threadIdx.x;
    BatchCtl& c = ctl[inst];
    if (c.done) return;
    double* col = H + (size_t)inst * ldh * mcols + (size_t)j * ldh;
    double* csi = cs + (size_t)inst * ldg;
    double* sni = sn + (size_t)inst * ldg;
    double* gi = g + (size_t)inst * ldg;
    const double gj = gi[j], tgt = target[inst];
    for (int i = lane; i <= j; i += 64) sc[i] = col[i];
    for (int i = lane; i < j; i += 64) {
        cc_s[i] = csi[i];
        ss_s[i] = sni[i];
    }
    double s = 0.0;
    for (int b = ib0[inst] + lane; b < ib1[inst]; b += 64) s += part[b];
    s = wave_sum(s);
    __syncthreads();
    const double hn = sqrt(s);
    if (lane == 0) {
        double h = sc[0];
        for (int i = 0; i < j; ++i) {
            const double nx = sc[i + 1];
            sc[i] = cc_s[i] * h + ss_s[i] * nx;
            h = -ss_s[i] * h + cc_s[i] * nx;
        }
        double ct = 1.0, st = 0.0;
        if (hn != 0.0) {
            const double r = hypot(h, hn);
            ct = h / r;
            st = hn / r;
        }
        csi[j] = ct;
        sni[j] = st;
        sc[j] = ct * h + st * hn;
        col[j + 1] = hn;
        gi[j + 1] = -st * gj;
        gi[j] = ct * gj;
        const double est = fabs(-st * gj);
        c.est = est;
        c.k = j + 1;
        if (!isfinite(est)) c.nonfinite = 1;
        if (est <= tgt || hn == 0.0 || j + 1 >= jmax || !isfinite(est)) c.done = 1;
    }
    __syncthreads();
    for (int i = lane; i <= j; i += 64) col[i] = sc[i];
}

// R y = g by columns, one wave per instance: the unknowns still to come stay in LDS and the next
// column of R is loaded while the current one is applied.
__global__ __launch_bounds__(64) void k_seg_backsolve(const BatchCtl* ctl, const double* H, int ldh, int mcols,
                                                      const double* g, int ldg, double* y) {
    __shared__ double ys[201];
    const int inst = blockIdx.x, lane = threadIdx.x;
    const int k = ctl[inst].k;
    const double* Hi = H + (size_t)inst * ldh * mcols;
    for (int i = lane; i < k; i += 64) ys[i] = g[(size_t)inst * ldg + i];
    __syncthreads();
    double nx[4];
    auto load = [&](int c) {
#pragma unroll
        for (int u = 0; u < 4; ++u) nx[u] = (c >= 0 && lane + 64 * u <= c) ? Hi[(size_t)c * ldh + lane + 64 * u] : 0.0;
    };
    load(k - 1);
    for (int c = k - 1; c >= 0; --c) {
        double r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) r[u] = nx[u];
        load(c - 1);
        const int du = c >> 6;
        const double rd = du == 0 ? r[0] : du == 1 ? r[1] : du == 2 ? r[2] : r[3];
        const double yc = ys[c] / wave_ops::read_lane(rd, c & 63);
        __syncthreads();
        if (lane == 0) ys[c] = yc;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (lane + 64 * u < c) ys[lane + 64 * u] -= r[u] * yc;
        __syncthreads();
    }
    for (int i = lane; i < k; i += 64) y[(size_t)inst * ldg + i] = ys[i];
}

// ---- recovery ------------------------------------------------------------------------------------
__global__ __launch_bounds__(BS) void k_batch_recover(const InstDesc* __restrict__ desc,
                                                      const int32_t* __restrict__ eid, int64_t total_ne,
                                                      const double* __restrict__ local, const double* __restrict__ Minv,
                                                      const double* __restrict__ Bd, const double* __restrict__ Cd,
                                                      const int32_t* __restrict__ e2f, const double* __restrict__ xhat,
                                                      double* __restrict__ du, double* __restrict__ dq) {
    extern __shared__ double sm[];
    for (int64_t g = blockIdx.x; g < total_ne; g += gridDim.x) {
        const InstDesc& q = desc[eid[g]];
        const int64_t le = g - q.e0;
        const int P = q.P, D = q.D, M = q.M, PF = q.PF, L = q.L, nu = q.nu, nt = q.nt, nb = q.nb, C = q.C;
        const int LPF = L * PF;
        double* xe = sm;
        double* t = xe + nt;
        double* s = t + nu;
        for (int idx = threadIdx.x; idx < nt; idx += BS) {
            const int l = idx / nb, rem = idx - l * nb;
            xe[idx] = xhat[q.vec_off + (int64_t)e2f[q.e2f_off + le * L + l] * nb + rem];
        }
        __syncthreads();
        const double* Le = local + q.local_off + le * nu * C;
        for (int i = threadIdx.x; i < nu; i += BS) {
            const double* row = Le + (size_t)i * C + nu;
            double acc = 0.0;
            for (int k = 0; k < nt; ++k) acc += row[k] * xe[k];
            t[i] = row[nt] - acc;
        }
        __syncthreads();
        for (int i = nu - 1; i >= 0; --i) {
            const double ui = t[i] / Le[(size_t)i * C + i];
            __syncthreads();
            if (threadIdx.x == 0) t[i] = ui;
            for (int k = threadIdx.x; k < i; k += BS) t[k] -= Le[(size_t)k * C + i] * ui;
            __syncthreads();
        }
        for (int i = threadIdx.x; i < nu; i += BS) du[q.du_off + le * nu + i] = t[i];
        const double* Mi = Minv + q.off[0] + le * P * P;
        for (int m = 0; m < M; ++m)
            for (int d = 0; d < D; ++d) {
                const double* B = Bd + q.off[1] + (le * D + d) * P * P;
                const double* Cm = Cd + q.off[2] + (le * D + d) * P * LPF;
                for (int i = threadIdx.x; i < P; i += BS) {
                    double acc = 0.0;
                    for (int j = 0; j < P; ++j) acc += B[(size_t)i * P + j] * t[m * P + j];
                    for (int l = 0; l < L; ++l)
                        for (int j = 0; j < PF; ++j) acc += Cm[(size_t)i * LPF + l * PF + j] * xe[(l * M + m) * PF + j];
                    s[i] = acc;
                }
                __syncthreads();
                for (int i = threadIdx.x; i < P; i += BS) {
                    double acc = 0.0;
                    for (int k = 0; k < P; ++k) acc += Mi[(size_t)i * P + k] * s[k];
                    dq[q.dq_off + le * q.nq + (int64_t)(m * D + d) * P + i] = -acc;
                }
                __syncthreads();
            }
        __syncthreads();
    }
}

}  // namespace

// ---- launchers ---------------------------------------------------------------------------------------
hdg_status batch_launch_condense(hdg_ctx ctx, const BatchDev& b, const BatchElemPtrs& in, double* Kbar, double* rbar,
                                 double* local, int* bad, int grid) {
    const size_t lds = sizeof(double) * b.max_cond_lds;
    const void* k = b.tiles ? (const void*)k_batch_condense<true> : (const void*)k_batch_condense<false>;
    if (lds > 64 * 1024)
        HDG_HIP_CHECK(ctx, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    void* args[] = {(void*)&b.desc, (void*)&b.eid, (void*)&b.total_ne, (void*)&in, (void*)&Kbar, (void*)&rbar,
                    (void*)&local, (void*)&bad};
    HDG_HIP_CHECK(ctx, hipLaunchKernel(k, dim3(grid), dim3(BS), args, lds, ctx->stream));
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status batch_launch_assemble(hdg_ctx ctx, const BatchDev& b, const int32_t* f2e, const int32_t* e2f,
                                 const double* Kbar, const double* rbar, double* K64, float* K32, int32_t* nbr,
                                 double* r) {
    const int grid = (int)std::min<int64_t>(b.total_nf, 65536);
    hipLaunchKernelGGL(k_batch_assemble, dim3(grid), dim3(BS), 0, ctx->stream, b.desc, b.fid, b.total_nf, f2e, e2f,
                       Kbar, rbar, K64, K32, nbr, r);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status batch_launch_face(hdg_ctx ctx, const BatchDev& b, const void* M1, bool fp32, const int32_t* nbr,
                             bool bj_only, double* x, double* out, double s0, const double* X, double a0,
                             const double* denom, int ld_denom, const BatchCtl* ctl) {
    if (fp32)
        hipLaunchKernelGGL(k_batch_face<float>, dim3(b.nfblk), dim3(BS), 0, ctx->stream, b.desc, b.fblk, (const float*)M1,
                           nbr, bj_only ? 1 : 0, x, out, s0, X, a0, denom, ld_denom, ctl);
    else
        hipLaunchKernelGGL(k_batch_face<double>, dim3(b.nfblk), dim3(BS), 0, ctx->stream, b.desc, b.fblk,
                           (const double*)M1, nbr, bj_only ? 1 : 0, x, out, s0, X, a0, denom, ld_denom, ctl);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status batch_launch_bj(hdg_ctx ctx, const BatchDev& b, const double* K64, double* B64, float* B32, int* bad) {
    const int grid = (int)std::min<int64_t>(b.total_nf, 65536);
    hipLaunchKernelGGL(k_batch_bj, dim3(grid), dim3(BS), 0, ctx->stream, b.desc, b.fid, b.total_nf, K64, B64, B32,
                       bad);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status seg_sweep(hdg_ctx ctx, const BatchDev& b, SegSweep a, bool axpy, bool dot) {
    a.blk_inst = b.blk_inst;
    a.blk_lo = b.blk_lo;
    a.blk_hi = b.blk_hi;
    a.ib0 = b.ib0;
    a.ib1 = b.ib1;
    a.nblk = b.nblk;
    if (axpy && (int64_t)b.max_chunks * a.J > SEG_DIRECT) {
        hipLaunchKernelGGL(k_seg_coef, dim3(div_up((long long)b.n_inst * a.J, 4)), dim3(256), 0, ctx->stream, a, b.n_inst);
        HDG_LAUNCH_CHECK(ctx);
    }
    const void* k = !axpy ? (const void*)k_seg_sweep<false, true>
                    : dot ? (const void*)k_seg_sweep<true, true>
                          : (const void*)k_seg_sweep<true, false>;
    void* args[] = {(void*)&a};
    HDG_HIP_CHECK(ctx, hipLaunchKernel(k, dim3(b.nblk), dim3(BS), args, 0, ctx->stream));
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status seg_reduce(hdg_ctx ctx, const BatchDev& b, const double* part, double* out, int ldo) {
    hipLaunchKernelGGL(k_seg_reduce, dim3(div_up(b.n_inst, 4)), dim3(256), 0, ctx->stream, b.ib0, b.ib1, b.n_inst, part,
                       out, ldo);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status seg_update(hdg_ctx ctx, const BatchDev& b, const double* Z, size_t ldz, const double* y, int ldy, double* x,
                      const BatchCtl* ctl) {
    hipLaunchKernelGGL(k_seg_update, dim3(div_up((long long)b.total_dof, BS)), dim3(BS), 0, ctx->stream, b.dof_inst, Z,
                       ldz, y, ldy, x, (size_t)b.total_dof, ctl);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status seg_sumsq(hdg_ctx ctx, const BatchDev& b, const double* w, double* part, const BatchCtl* ctl) {
    hipLaunchKernelGGL(k_seg_sumsq, dim3(b.nblk), dim3(BS), 0, ctx->stream, b.blk_inst, b.blk_lo, b.blk_hi, w, part,
                       ctl);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status seg_scale(hdg_ctx ctx, const BatchDev& b, double* v, const double* denom, int ld_denom,
                     const BatchCtl* ctl) {
    hipLaunchKernelGGL(k_seg_scale, dim3(div_up((long long)b.total_dof, BS)), dim3(BS), 0, ctx->stream, b.dof_inst, v,
                       (size_t)b.total_dof, denom, ld_denom, ctl);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status seg_cycle_init(hdg_ctx ctx, const BatchDev& b, const double* part, BatchCtl* ctl, double* g, int ldg,
                          int jmax, const double* target) {
    hipLaunchKernelGGL(k_seg_cycle_init, dim3(div_up(b.n_inst, 4)), dim3(256), 0, ctx->stream, b.ib0, b.ib1, b.n_inst,
                       part, ctl, g, ldg, jmax, target);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status seg_givens(hdg_ctx ctx, const BatchDev& b, const double* part, BatchCtl* ctl, double* H, int ldh, int mcols,
                      double* cs, double* sn, double* g, int ldg, int j, int jmax, const double* target) {
    hipLaunchKernelGGL(k_seg_givens, dim3(b.n_inst), dim3(64), 0, ctx->stream, b.ib0, b.ib1, part, ctl, H, ldh, mcols, cs, sn, g, ldg, j, jmax, target);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status seg_backsolve(hdg_ctx ctx, const BatchDev& b, const BatchCtl* ctl, const double* H, int ldh, int mcols,
                         const double* g, int ldg, double* y) {
    hipLaunchKernelGGL(k_seg_backsolve, dim3(b.n_inst), dim3(64), 0, ctx->stream, ctl, H, ldh, mcols, g, ldg, y);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status batch_launch_recover(hdg_ctx ctx, const BatchDev& b, const double* local, const double* Minv,
                                const double* Bd, const double* Cd, const int32_t* e2f, const double* xhat,
                                double* du, double* dq) {
    const int grid = (int)std::min<int64_t>(b.total_ne, 65536);
    const size_t lds = sizeof(double) * b.max_rec_lds;
    hipLaunchKernelGGL(k_batch_recover, dim3(grid), dim3(BS), lds, ctx->stream, b.desc, b.eid, b.total_ne, local, Minv,
                       Bd, Cd, e2f, xhat, du, dq);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}
