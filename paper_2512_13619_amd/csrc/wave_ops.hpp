// Wave-level helpers shared by the recovery, condensation and block-Jacobi kernels (64-lane waves).
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

namespace wave_ops {

template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v) {
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(v), __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(v), __double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// v of lane N of this lane's row of 16.
template <int N>
__device__ __forceinline__ double row_bcast(double v) {
    return dpp_mov<0x150 + N>(v);    // row_newbcast:N
}

__device__ __forceinline__ double read_lane(double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

// Largest v over the wave (ties: smallest i), returned in every lane. Within each row of
// 16 lanes the partners come through DPP (xor 1, xor 2, half-row and row mirrors, no LDS
// round trip); the four row results are then read as uniform values.
template <int CTRL>
__device__ __forceinline__ void argmax_dpp_step(double& v, int& i) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    const int olo = __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false);
    const int ohi = __builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false);
    const int oi = __builtin_amdgcn_update_dpp(i, i, CTRL, 0xF, 0xF, false);
    const double ov = __hiloint2double(ohi, olo);
    if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; }
}

__device__ __forceinline__ void wave_argmax(double& v, int& i) {
    argmax_dpp_step<0xB1>(v, i);   // quad_perm [1,0,3,2]
    argmax_dpp_step<0x4E>(v, i);   // quad_perm [2,3,0,1]
    argmax_dpp_step<0x141>(v, i);  // row_half_mirror
    argmax_dpp_step<0x140>(v, i);  // row_mirror
    const int lo = __double2loint(v), hi = __double2hiint(v);
#pragma unroll
    for (int r = 1; r < 4; ++r) {
        const double ov = __hiloint2double(__builtin_amdgcn_readlane(hi, 16 * r), __builtin_amdgcn_readlane(lo, 16 * r));
        const int oi = __builtin_amdgcn_readlane(i, 16 * r);
        if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; }
    }
    // row 0's lanes started from their own row value; make every lane agree on the result
    const double v0 = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 0),
                                       __builtin_amdgcn_readlane(__double2loint(v), 0));
    i = __builtin_amdgcn_readlane(i, 0);
    v = v0;
}

// Sum over the wave, the same value in every lane: within each row of 16 lanes the
// partners come through DPP (xor 1, xor 2, half-row and row mirrors), then the four row
// sums are added in a fixed order.
__device__ __forceinline__ double wave_sum_all(double v) {
    v += dpp_mov<0xB1>(v);    // quad_perm [1,0,3,2]
    v += dpp_mov<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp_mov<0x141>(v);   // row_half_mirror
    v += dpp_mov<0x140>(v);   // row_mirror
    return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// Copies `bytes` (a multiple of 4) from global memory to LDS without a round trip through registers;
// wave `wave` of `nw` takes every nw-th piece of 256 bytes. Both sides need 4-byte alignment only.
// Complete for the whole block after copies_done() and a barrier.
__device__ __forceinline__ void copy_to_lds(const void* g, void* lds, int bytes, int wave, int nw) {
    const int lane = threadIdx.x & 63;
    for (int o = wave * 256; o < bytes; o += nw * 256)
        if (o + lane * 4 < bytes)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) uint32_t*)((const char*)g + o + lane * 4),
                (__attribute__((address_space(3))) uint32_t*)((char*)lds + o), 4, 0, 0);
}
__device__ __forceinline__ void copies_done() { __builtin_amdgcn_s_waitcnt(0x0F70); }    // vmcnt(0)

// acc += A B for one 16 x 16 tile over K terms on the FP64 matrix cores (v_mfma_f64_16x16x4f64:
// A[i][k] in lane i+16k, B[k][j] in lane j+16k; the result's entry (i, j) in lane
// j+16(i mod 4), register i div 4). fa(k) gives this lane's A[lane mod 16][k], fb(k) its
// B[k][lane mod 16], with k in [0, K); terms past K are zero on both sides. U steps' loads
// are issued together.
typedef double d4 __attribute__((ext_vector_type(4)));
template <int U, class FA, class FB>
__device__ __forceinline__ void mma16(int K, const FA& fa, const FB& fb, d4& acc) {
    const int kq = (threadIdx.x & 63) >> 4;
    int k0 = 0;
    for (; k0 + 4 * U <= K; k0 += 4 * U) {
        double a[U], b[U];
#pragma unroll
        for (int s = 0; s < U; ++s) {
            a[s] = fa(k0 + 4 * s + kq);
            b[s] = fb(k0 + 4 * s + kq);
        }
#pragma unroll
        for (int s = 0; s < U; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
    }
    for (; k0 < K; k0 += 4) {
        const int k = k0 + kq, kc = k < K ? k : K - 1;
        double a = fa(kc), b = fb(kc);
        a = k < K ? a : 0.0;
        b = k < K ? b : 0.0;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
    }
}

// This lane's entries of an operand: entry k at p[k s], times w[k ws] where weighted.
struct Seq {
    const double* p;
    int s;
    const double* w;
    int ws;
};
__device__ __forceinline__ Seq seq(const double* p, int s) { return {p, s, nullptr, 0}; }
__device__ __forceinline__ Seq seq(const double* p, int s, const double* w, int ws) { return {p, s, w, ws}; }

// mma16 over strided operands: running pointers instead of an index product per load, and all steps
// of a remainder below 16 terms in flight together.
template <bool WA, bool WB>
__device__ __forceinline__ void mma16s(int K, const Seq& A, const Seq& B, d4& acc) {
    const int kq = (threadIdx.x & 63) >> 4;
    const double *pa = A.p + __mul24(kq, A.s), *pb = B.p + __mul24(kq, B.s);
    const double *wa = WA ? A.w + __mul24(kq, A.ws) : nullptr, *wb = WB ? B.w + __mul24(kq, B.ws) : nullptr;
    int left = K;
    for (; left >= 16; left -= 16) {
        double a[4], b[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            a[s] = *pa;
            b[s] = *pb;
            if (WA) a[s] *= *wa;
            if (WB) b[s] *= *wb;
            pa += 4 * A.s;
            pb += 4 * B.s;
            if (WA) wa += 4 * A.ws;
            if (WB) wb += 4 * B.ws;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
    }
    if (left > 0) {
        double a[4], b[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (4 * s >= left) break;
            const bool in = 4 * s + kq < left;
            const int o = in ? 4 * s : left - 1 - kq;          // past the end: the last entry, then zeroed
            a[s] = pa[__mul24(o, A.s)];
            b[s] = pb[__mul24(o, B.s)];
            if (WA) a[s] *= wa[__mul24(o, A.ws)];
            if (WB) b[s] *= wb[__mul24(o, B.ws)];
            a[s] = in ? a[s] : 0.0;
            b[s] = in ? b[s] : 0.0;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (4 * s >= left) break;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
        }
    }
}

// res[r] = sum_{k<n} A[(i0+r)*lda + k] v[k] for r < nr (nr <= 4), v in LDS; the loads of
// the four rows are issued together (row and column indices clamped to valid entries).
__device__ __forceinline__ void rows_dot4(const double* __restrict__ A, int lda, int i0, int nr,
                                          const double* v, int n, double (&res)[4]) {
    const int lane = threadIdx.x & 63;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = 0; k0 < n; k0 += 64) {
        const int k = k0 + lane;
        const bool ok = k < n;
        const int kc = ok ? k : 0;
        double a[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) a[r] = A[(size_t)(i0 + (r < nr ? r : 0)) * lda + kc];
        const double xv = v[kc];
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] += ok ? a[r] * xv : 0.0;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) res[r] = wave_sum_all(acc[r]);
}

}  // namespace wave_ops

namespace wave_ops {

// Solves U x = y in place for the n x n upper triangle of U (row stride ld, global memory;
// entries below the diagonal are not read into the result), with y in LDS. All NT threads
// of the block call it. Diagonal blocks of 64 rows from the bottom: the block's rows first
// take the unknowns already solved below them (four rows per wave at a time), then one wave
// solves the 64 x 64 triangle with one unknown per lane. Rows above row 0 in the top block
// are padding (identity rows that take nothing from the rows below).
template <int NT>
__device__ void upper_solve_lds(const double* __restrict__ U, int ld, int n, double* y) {
    constexpr int NW = NT / 64;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int top = n; top > 0; top -= 64) {
        const int base = top - 64;
        const int lo = base > 0 ? base : 0;
        if (top < n) {
            for (int i0 = lo + 4 * wave; i0 < top; i0 += 4 * NW) {
                const int nr = top - i0 < 4 ? top - i0 : 4;
                double res[4];
                rows_dot4(U + top, ld, i0, nr, y + top, n - top, res);
                if (lane < nr) {
                    double rr = res[0];
#pragma unroll
                    for (int r = 1; r < 4; ++r) rr = lane == r ? res[r] : rr;
                    y[i0 + lane] -= rr;
                }
            }
        }
        __syncthreads();
        if (wave == 0) {
            const int g = base + lane;
            double x = g >= 0 ? y[g] : 0.0;
            double ub[64];                 // column g of the block: ub[i] = U[base + i][g]
#pragma unroll
            for (int i = 0; i < 64; ++i) {
                const int gr = base + i;
                const bool in = gr >= 0 && g >= 0;
                const double v = U[in ? (size_t)gr * ld + g : 0];
                ub[i] = in ? v : (i == lane ? 1.0 : 0.0);
            }
#pragma unroll
            for (int i = 63; i >= 0; --i) {
                const double s = wave_sum_all(lane > i ? ub[i] * x : 0.0);
                const double xi = (read_lane(x, i) - s) / read_lane(ub[i], i);
                x = lane == i ? xi : x;
            }
            if (g >= 0) y[g] = x;
        }
        __syncthreads();
    }
}

}  // namespace wave_ops
