// Element residuals and Jacobian blocks on the device for M-component models in 3D
// (Section 2.1, Section 2.2's weak form and numerical flux, Section 4.1's element matrices):
//   linear elasticity (M = 3)   F = -sigma(q), sigma = lam tr(eps) I + 2 mu eps, eps = sym(q);
//   compressible Navier-Stokes  F = F_c(u) - F_v(u, q), conservative u = (rho, rho v, rho E),
//   (M = 5)                     mu = 1/Re, Stokes hypothesis, heat flux (mu gamma / Pr) grad e.
// fhat = F(uhat, q).n + tau (u - uhat); Dirichlet trace rows uhat - u_D on boundary faces.
//
// Two kernels per chunk of elements, every sum over quadrature points on the FP64 matrix cores:
//   1. k_sys_points: per element, the mass matrix and its inverse, B_d and C_d, the consistent
//      q = -M^{-1}(B_d u_m + C_d uhat_m) (eq. w16, r_q = 0), the state at the volume and face
//      quadrature points, per point the flux (residual rows ru, rt) and, unless residual-only,
//      its derivatives with respect to u and q by forward-mode dual numbers, stored weighted
//      (volume) or contracted with the scaled normal (faces) in a point workspace;
//   2. k_sys_blocks: every matrix entry as one sum over the points of that workspace times
//      the basis values -- the products of per-point flux data with the basis tables that
//      Section 4.1 forms (E = Psi U), evaluated per element.
// Residual rows (trace rows negated on interior faces), with an implicit stage's time term
// (c = 1/(a_ii dt), u_n, r_x):
//   R_u[m,i]   = -(F_m, grad phi_i) + <fhat_m, phi_i> - (s_m, phi_i) + c (u_m - u_n,m, phi_i) + r_x
//   R_t[l,m,j] = -<fhat_m, psi_j>_l (interior),  <uhat_m - u_D,m, psi_j>_l (Dirichlet)
// ru = -R_u, rt = -R_t; D..J their derivatives with respect to q, u and uhat.
#include <cmath>

#include "hdg_internal.hpp"
#include "wave_ops.hpp"

namespace {

constexpr int SBS = 256;
constexpr int BBS = 512;     // k_sys_blocks
constexpr int SD = 3;        // space dimension of both models
using wave_ops::d4;
using wave_ops::mma16;

// Value and N directional derivatives.
template <int N>
struct Dual {
    double v, d[N];
};
#define HDG_DUAL_EACH for (int n_ = 0; n_ < N; ++n_)
template <int N>
__device__ __forceinline__ Dual<N> operator+(Dual<N> a, const Dual<N>& b) {
    a.v += b.v;
    HDG_DUAL_EACH a.d[n_] += b.d[n_];
    return a;
}
template <int N>
__device__ __forceinline__ Dual<N> operator-(Dual<N> a, const Dual<N>& b) {
    a.v -= b.v;
    HDG_DUAL_EACH a.d[n_] -= b.d[n_];
    return a;
}
template <int N>
__device__ __forceinline__ Dual<N> operator*(const Dual<N>& a, const Dual<N>& b) {
    Dual<N> r;
    r.v = a.v * b.v;
    HDG_DUAL_EACH r.d[n_] = a.d[n_] * b.v + a.v * b.d[n_];
    return r;
}
template <int N>
__device__ __forceinline__ Dual<N> operator/(const Dual<N>& a, const Dual<N>& b) {
    const double s = 1.0 / b.v;
    Dual<N> r;
    r.v = a.v * s;
    HDG_DUAL_EACH r.d[n_] = (a.d[n_] - a.v * s * b.d[n_]) * s;
    return r;
}
template <int N>
__device__ __forceinline__ Dual<N> operator*(double s, Dual<N> a) {
    a.v *= s;
    HDG_DUAL_EACH a.d[n_] *= s;
    return a;
}
#undef HDG_DUAL_EACH
__device__ __forceinline__ double neg(double a) { return -a; }
template <int N>
__device__ __forceinline__ Dual<N> neg(Dual<N> a) {
    return -1.0 * a;
}

struct SysParams {
    int kind;
    double tau, lam, mu, Re, Pr, gamma;
};

// F[a][x] of linear elasticity (u is not used)
template <class T>
__device__ __forceinline__ void flux_elasticity(const SysParams& p, const T (&u)[3], const T (&q)[3][SD],
                                                T (&F)[3][SD]) {
    (void)u;
    const T tr = q[0][0] + q[1][1] + q[2][2];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int x = 0; x < SD; ++x) {
            T s = p.mu * (q[a][x] + q[x][a]);
            if (a == x) s = s + p.lam * tr;
            F[a][x] = neg(s);
        }
}

// F[a][x] of the compressible Navier-Stokes equations
template <class T>
__device__ __forceinline__ void flux_navier_stokes(const SysParams& p, const T (&u)[5], const T (&q)[5][SD],
                                                   T (&F)[5][SD]) {
    const double g = p.gamma, mu = 1.0 / p.Re, kappa = mu * g / p.Pr;
    const T rho = u[0], rE = u[4];
    T v[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) v[a] = u[1 + a] / rho;
    const T pr = (g - 1.0) * (rE - 0.5 * (u[1] * v[0] + u[2] * v[1] + u[3] * v[2]));
    const T E = rE / rho;
    T gv[3][SD];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int x = 0; x < SD; ++x) gv[a][x] = (q[1 + a][x] - v[a] * q[0][x]) / rho;
    const T div = gv[0][0] + gv[1][1] + gv[2][2];
#pragma unroll
    for (int x = 0; x < SD; ++x) {
        const T ge = (q[4][x] - E * q[0][x]) / rho - (v[0] * gv[0][x] + v[1] * gv[1][x] + v[2] * gv[2][x]);
        F[0][x] = u[1 + x];
        T work = {};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            T tv = mu * (gv[a][x] + gv[x][a]);
            if (a == x) tv = tv - (2.0 / 3.0) * mu * div;
            T f = u[1 + a] * v[x] - tv;
            if (a == x) f = f + pr;
            F[1 + a][x] = f;
            work = work + tv * v[a];
        }
        F[4][x] = (rE + pr) * v[x] - work - kappa * ge;
    }
}

template <int M, class T>
__device__ __forceinline__ void flux(const SysParams& p, const T (&u)[M], const T (&q)[M][SD], T (&F)[M][SD]) {
    if constexpr (M == 3) flux_elasticity(p, u, q, F);
    else flux_navier_stokes(p, u, q, F);
}

// Per-element point workspace (doubles): for every component pair (a, b)
//   vol  [a*M+b][Qv][12]  w dF[a][xi]/dq_bd at d*3 + xi (d < 3), w dF[a][xi]/du_b at 9 + xi
//   face [a*M+b][LQf][4]  sum_xi dF[a][xi]/dq_bd n_xi (d < 3), sum_xi dF[a][xi]/duhat_b n_xi
// A pair's points are contiguous, so the wave that forms the pair's blocks reads one stream and
// a thread's stores of a point are whole 16-byte pieces.
struct PointWs {
    int face, per_elem;
};
__host__ __device__ inline PointWs point_ws(int M, int Qv, int LQf) {
    PointWs w;
    w.face = M * M * Qv * 12;
    w.per_elem = w.face + M * M * LQf * 4;
    return w;
}

// LDS of k_sys_points (doubles)
struct PtsLds {
    int Mm, un, up, uh, qn, t, uq, duq, qq, uf, uhf, qf, total;
};
__host__ __device__ inline PtsLds pts_lds(int M, int P, int PF, int L, int Qv, int Qf) {
    PtsLds o;
    int k = 0;
    o.Mm = k; k += P * P;
    o.un = k; k += M * P;
    o.up = k; k += M * P;
    o.uh = k; k += L * M * PF;
    o.qn = k; k += M * SD * P;
    o.t = k;  k += M * SD * P;
    o.uq = k; k += Qv * M;
    o.duq = k; k += Qv * M;
    o.qq = k; k += Qv * M * SD;
    o.uf = k; k += L * Qf * M;
    o.uhf = k; k += L * Qf * M;
    o.qf = k; k += L * Qf * M * SD;
    o.total = k;
    return o;
}

struct SysArgs {
    hdg_elem_geom g;        // src [ne][nqv][M], uD [ne][nlfe][nqf][M]
    SysParams pm;
    const int32_t* e2f;
    const double* u;        // [ne][M][P]
    const double* uhat;     // [nf][M][PF]
    const double* u_prev;   // [ne][M][P] when c != 0
    const double* r_extra;  // [ne][M*P] or null
    double c;
    hdg_elem_arrays out;
    double* ws;             // point workspace of the chunk
    int* bad;
    int e0, P, PF, L, Qv, Qf, residual_only, keep_mass;
};

// One block per element. Bound by the element's data (geometry read once) when residual-only; every
// sum over points or basis functions is a 16x16 matrix-core tile shared out over the four waves
// (a point evaluation has the points as rows and the M or 3M fields as columns; a test-function
// sum the fields as rows and the basis functions as columns), where a thread-per-entry loop spent
// two loads on every multiply-add (24,480 Navier-Stokes p = 2 tets, residual only: 2.04 ms so, with
// k_sys_blocks' sums; 0.61 ms now, 1.3 TB/s).
// JAC: the flux derivatives too. Without them the Navier-Stokes kernel holds 107 registers, four blocks a CU,
// instead of 165 and three; elasticity's derivatives cost nothing (65 and 69, seven).
template <int M, bool JAC>
__global__ void __launch_bounds__(SBS, JAC ? 2 : 4) k_sys_points(SysArgs a) {
    extern __shared__ double sm[];
    const int el = blockIdx.x;
    const size_t e = (size_t)a.e0 + el;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
    constexpr int NW = SBS / 64, MD = M * SD;
    const int P = a.P, PF = a.PF, L = a.L, Qv = a.Qv, Qf = a.Qf, LQf = L * Qf, LPF = L * PF;
    const PtsLds o = pts_lds(M, P, PF, L, Qv, Qf);
    double *Mm = sm + o.Mm, *un = sm + o.un, *up = sm + o.up, *uh = sm + o.uh, *qn = sm + o.qn, *t = sm + o.t;
    double *uq = sm + o.uq, *duq = sm + o.duq, *qq = sm + o.qq, *uf = sm + o.uf, *uhf = sm + o.uhf, *qf = sm + o.qf;
    const double* wdet = a.g.wdet + e * Qv;
    const double* dphix = a.g.dphix + e * Qv * P * SD;
    const double* phi = a.g.phi;
    const double* phif = a.g.phif + e * LQf * P;
    const double* psi = a.g.psi;
    const double* ndA = a.g.ndA + e * LQf * SD;
    const double* dA = a.g.dA + e * LQf;
    const double* src = a.g.src + e * Qv * M;
    const double* uD = a.g.uD + e * LQf * M;
    const int32_t* e2f = a.e2f + e * L;
    const int32_t* bnd = a.g.bnd + e * L;
    const double cdt = a.c;
    const int tP = (P + 15) >> 4, tPF = (PF + 15) >> 4, tQv = (Qv + 15) >> 4, tQf = (Qf + 15) >> 4;
    const int tLQf = (LQf + 15) >> 4;

    // 1. nodal state
    for (int k = tid; k < M * P; k += SBS) {
        un[k] = a.u[e * M * P + k];
        up[k] = cdt != 0.0 ? a.u_prev[e * M * P + k] : 0.0;
    }
    for (int k = tid; k < L * M * PF; k += SBS) {
        const int l = k / (M * PF), r = k - l * M * PF;
        uh[k] = a.uhat[(size_t)e2f[l] * M * PF + r];
    }
    // 2. mass matrix and its inverse (Gauss-Jordan in place; M is SPD), or the kept inverse
    if (a.keep_mass) {
        for (int k = tid; k < P * P; k += SBS) Mm[k] = a.out.Minv[e * P * P + k];
        __syncthreads();
    } else {
        for (int it = wave; it < tP * tP; it += NW) {
            const int i0 = (it / tP) * 16, j0 = (it % tP) * 16;
            const int i = i0 + l16 < P ? i0 + l16 : P - 1, j = j0 + l16 < P ? j0 + l16 : P - 1;
            d4 acc = {};
            mma16<4>(Qv, [&](int x) { return wdet[x] * phi[x * P + i]; }, [&](int x) { return phi[x * P + j]; }, acc);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (i0 + 4 * r + lq < P && j0 + l16 < P) Mm[(i0 + 4 * r + lq) * P + j0 + l16] = acc[r];
        }
        __syncthreads();
        const int gi = tid >> 4, gj = tid & 15;
        for (int k = 0; k < P; ++k) {
            const double piv = Mm[k * P + k];
            if (!(piv > 0.0) || !isfinite(piv)) {
                if (tid == 0) atomicMin(a.bad, (int)e);
                return;    // uniform across the workgroup: every thread read the same pivot
            }
            const double rp = 1.0 / piv;
            for (int i = gi; i < P; i += SBS / 16) {
                if (i == k) continue;
                const double f = Mm[i * P + k] * rp;
                for (int j = gj; j < P; j += 16)
                    if (j != k) Mm[i * P + j] -= f * Mm[k * P + j];
            }
            __syncthreads();
            for (int idx = tid; idx < P; idx += SBS) {
                if (idx != k) {
                    Mm[idx * P + k] = -Mm[idx * P + k] * rp;
                    Mm[k * P + idx] *= rp;
                }
            }
            if (tid == 0) Mm[k * P + k] = rp;
            __syncthreads();
        }
        if (a.out.Minv)
            for (int k = tid; k < P * P; k += SBS) a.out.Minv[e * P * P + k] = Mm[k];
    }
    // B_d [d][i][j] and C_d [d][i][(l,j)] (geometry only)
    if (JAC && !a.keep_mass) {
        for (int it = wave; it < SD * tP * tP; it += NW) {
            const int d = it / (tP * tP), r0 = it - d * tP * tP, i0 = (r0 / tP) * 16, j0 = (r0 % tP) * 16;
            const int i = i0 + l16 < P ? i0 + l16 : P - 1, j = j0 + l16 < P ? j0 + l16 : P - 1;
            d4 acc = {};
            mma16<4>(Qv, [&](int x) { return wdet[x] * dphix[(x * P + i) * SD + d]; },
                     [&](int x) { return phi[x * P + j]; }, acc);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (i0 + 4 * r + lq < P && j0 + l16 < P)
                    a.out.Bd[e * SD * P * P + ((size_t)d * P + i0 + 4 * r + lq) * P + j0 + l16] = acc[r];
        }
        for (int it = wave; it < SD * L * tP * tPF; it += NW) {
            int q = it;
            const int j0 = (q % tPF) * 16; q /= tPF;
            const int i0 = (q % tP) * 16; q /= tP;
            const int l = q % L, d = q / L;
            const int i = i0 + l16 < P ? i0 + l16 : P - 1, j = j0 + l16 < PF ? j0 + l16 : PF - 1;
            d4 acc = {};
            mma16<4>(Qf, [&](int x) { return -ndA[(l * Qf + x) * SD + d] * phif[(l * Qf + x) * P + i]; },
                     [&](int x) { return psi[x * PF + j]; }, acc);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (i0 + 4 * r + lq < P && j0 + l16 < PF)
                    a.out.Cd[e * SD * P * LPF + ((size_t)d * P + i0 + 4 * r + lq) * LPF + l * PF + j0 + l16] = acc[r];
        }
    }
    // 3. u and u_n at the volume points (columns m and M + m); u and uhat at the face points
    for (int it = wave; it < tQv + L * tQf; it += NW) {
        if (it < tQv) {
            const int x0 = it * 16, x = x0 + l16 < Qv ? x0 + l16 : Qv - 1;
            const double* st = l16 < M ? un + l16 * P : up + (l16 < 2 * M ? l16 - M : 0) * P;
            d4 acc = {};
            mma16<4>(P, [&](int i) { return phi[x * P + i]; }, [&](int i) { return st[i]; }, acc);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int xr = x0 + 4 * r + lq;
                if (xr < Qv && l16 < M) uq[xr * M + l16] = acc[r];
                if (xr < Qv && l16 >= M && l16 < 2 * M) duq[xr * M + l16 - M] = acc[r];
            }
        } else {
            const int l = (it - tQv) / tQf, x0 = (it - tQv - l * tQf) * 16, x = x0 + l16 < Qf ? x0 + l16 : Qf - 1;
            const int m = l16 < M ? l16 : 0;
            d4 au = {}, ah = {};
            mma16<4>(P, [&](int i) { return phif[(l * Qf + x) * P + i]; }, [&](int i) { return un[m * P + i]; }, au);
            mma16<4>(PF, [&](int j) { return psi[x * PF + j]; }, [&](int j) { return uh[(l * M + m) * PF + j]; }, ah);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int xr = x0 + 4 * r + lq;
                if (xr < Qf && l16 < M) {
                    uf[(l * Qf + xr) * M + l16] = au[r];
                    uhf[(l * Qf + xr) * M + l16] = ah[r];
                }
            }
        }
    }
    __syncthreads();
    // 4. q = -M^{-1} (B_d u_m + C_d uhat_m): the volume sums in t, the face sums in qn, then both
    // as one operand of the product with M^{-1}
    const int tDP = (SD * P + 15) >> 4;
    for (int it = wave; it < 2 * tDP; it += NW) {
        const int c0 = (it >> 1) * 16, c = c0 + l16 < SD * P ? c0 + l16 : SD * P - 1, d = c / P, i = c - d * P;
        const int m = l16 < M ? l16 : 0;
        d4 acc = {};
        if (it & 1)
            mma16<4>(LQf, [&](int x) { return -uhf[x * M + m]; },
                     [&](int x) { return ndA[x * SD + d] * phif[x * P + i]; }, acc);
        else
            mma16<4>(Qv, [&](int x) { return uq[x * M + m]; },
                     [&](int x) { return wdet[x] * dphix[(x * P + i) * SD + d]; }, acc);
        double* dst = (it & 1) ? qn : t;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * r + lq < M && c0 + l16 < SD * P) dst[(4 * r + lq) * SD * P + c0 + l16] = acc[r];
    }
    __syncthreads();
    for (int k = tid; k < MD * P; k += SBS) t[k] += qn[k];
    __syncthreads();
    for (int it = wave; it < tP; it += NW) {
        const int i0 = it * 16, i = i0 + l16 < P ? i0 + l16 : P - 1, md = l16 < MD ? l16 : 0;
        d4 acc = {};
        mma16<4>(P, [&](int j) { return -t[md * P + j]; }, [&](int j) { return Mm[i * P + j]; }, acc);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * r + lq < MD && i0 + l16 < P) {
                qn[(4 * r + lq) * P + i0 + l16] = acc[r];
                if (a.out.q) a.out.q[(e * MD + 4 * r + lq) * P + i0 + l16] = acc[r];
            }
    }
    __syncthreads();
    // q at the points
    for (int it = wave; it < tQv + tLQf; it += NW) {
        const bool vol = it < tQv;
        const int n = vol ? Qv : LQf, x0 = (vol ? it : it - tQv) * 16, x = x0 + l16 < n ? x0 + l16 : n - 1;
        const double* tab = (vol ? phi : phif) + (size_t)x * P;
        const int md = l16 < MD ? l16 : 0;
        d4 acc = {};
        mma16<4>(P, [&](int i) { return tab[i]; }, [&](int i) { return qn[md * P + i]; }, acc);
        double* dst = vol ? qq : qf;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (x0 + 4 * r + lq < n && l16 < MD) dst[(x0 + 4 * r + lq) * MD + l16] = acc[r];
    }
    __syncthreads();
    // 5. flux derivatives: one work item per point, component b and pair of directions
    // (q_b0, q_b1) or (q_b2, u_b)
    if constexpr (JAC) {
        const PointWs W = point_ws(M, Qv, LQf);
        double* ws = a.ws + (size_t)el * W.per_elem;
        const int npt = Qv + LQf;
        for (int it = tid; it < npt * M * 2; it += SBS) {
            const int pb = it / npt, k = it - pb * npt, b = pb >> 1, half = pb & 1;
            const bool vol = k < Qv;
            const int lx = vol ? 0 : k - Qv;
            Dual<2> uu[M], qd[M][SD], F[M][SD];
            const double* us = vol ? uq + k * M : uhf + lx * M;
            const double* qs = vol ? qq + k * MD : qf + lx * MD;
#pragma unroll
            for (int m = 0; m < M; ++m) {
                uu[m] = {us[m], {0.0, (half && m == b) ? 1.0 : 0.0}};
#pragma unroll
                for (int d = 0; d < SD; ++d)
                    qd[m][d] = {qs[m * SD + d], {(m == b && d == 2 * half) ? 1.0 : 0.0,
                                                 (m == b && d == 1 && !half) ? 1.0 : 0.0}};
            }
            flux<M>(a.pm, uu, qd, F);
            if (vol) {
                const double w = wdet[k];
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    double2* dst = (double2*)(ws + ((size_t)(m * M + b) * Qv + k) * 12 + 6 * half);
                    dst[0] = make_double2(w * F[m][0].d[0], w * F[m][1].d[0]);
                    dst[1] = make_double2(w * F[m][2].d[0], w * F[m][0].d[1]);
                    dst[2] = make_double2(w * F[m][1].d[1], w * F[m][2].d[1]);
                }
            } else {
                double n[SD];
#pragma unroll
                for (int x = 0; x < SD; ++x) n[x] = ndA[lx * SD + x];
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    double s0 = 0.0, s1 = 0.0;
#pragma unroll
                    for (int x = 0; x < SD; ++x) {
                        s0 += F[m][x].d[0] * n[x];
                        s1 += F[m][x].d[1] * n[x];
                    }
                    *(double2*)(ws + W.face + ((size_t)(m * M + b) * LQf + lx) * 4 + 2 * half) = make_double2(s0, s1);
                }
            }
        }
        __syncthreads();
    }
    // 6. the flux per point, in place of the state it was formed from: w F over q and
    // w (s - c (u - u_n)) over u_n at the volume points, fhat over u and dA (uhat - u_D) over uhat
    // at the face points
    for (int k = tid; k < Qv + LQf; k += SBS) {
        const bool vol = k < Qv;
        const int lx = vol ? 0 : k - Qv;
        double uu[M], qd[M][SD], F[M][SD];
        const double* us = vol ? uq + k * M : uhf + lx * M;
        const double* qs = vol ? qq + k * MD : qf + lx * MD;
#pragma unroll
        for (int m = 0; m < M; ++m) {
            uu[m] = us[m];
#pragma unroll
            for (int d = 0; d < SD; ++d) qd[m][d] = qs[m * SD + d];
        }
        flux<M>(a.pm, uu, qd, F);
        if (vol) {
            const double w = wdet[k];
#pragma unroll
            for (int m = 0; m < M; ++m) {
#pragma unroll
                for (int x = 0; x < SD; ++x) qq[k * MD + m * SD + x] = w * F[m][x];
                duq[k * M + m] = w * (src[k * M + m] - cdt * (uu[m] - duq[k * M + m]));
            }
        } else {
            double n[SD];
#pragma unroll
            for (int x = 0; x < SD; ++x) n[x] = ndA[lx * SD + x];
            const double da = dA[lx];
#pragma unroll
            for (int m = 0; m < M; ++m) {
                double fn = 0.0;
#pragma unroll
                for (int x = 0; x < SD; ++x) fn += F[m][x] * n[x];
                uf[lx * M + m] = fn + a.pm.tau * (uf[lx * M + m] - uu[m]) * da;
                uhf[lx * M + m] = da * (uu[m] - uD[lx * M + m]);
            }
        }
    }
    __syncthreads();
    // 7. ru = -R_u: waves 0..2 take the three dimensions of (F, grad phi), wave 3 the source, time and
    // face sums; the four partial sums (over the room of qn and t) are added in that order.
    // rt = -R_t per face.
    double* part = sm + (o.qn < o.t ? o.qn : o.t);      // M*P per wave: 4 M P <= 2 * 3 M P
    const int mr = l16 < M ? l16 : 0;
    for (int it = 0; it < tP; ++it) {
        const int i0 = it * 16, i = i0 + l16 < P ? i0 + l16 : P - 1;
        d4 acc = {};
        if (wave < SD) {
            mma16<4>(Qv, [&](int x) { return qq[x * MD + mr * SD + wave]; },
                     [&](int x) { return dphix[(x * P + i) * SD + wave]; }, acc);
        } else {
            mma16<4>(Qv, [&](int x) { return duq[x * M + mr]; }, [&](int x) { return phi[x * P + i]; }, acc);
            mma16<4>(LQf, [&](int x) { return -uf[x * M + mr]; }, [&](int x) { return phif[x * P + i]; }, acc);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * r + lq < M && i0 + l16 < P) part[(wave * M + 4 * r + lq) * P + i0 + l16] = acc[r];
    }
    for (int it = wave; it < L * tPF; it += NW) {
        const int l = it / tPF, j0 = (it - l * tPF) * 16, j = j0 + l16 < PF ? j0 + l16 : PF - 1;
        const bool bd = bnd[l] != 0;
        d4 acc = {};
        mma16<4>(Qf, [&](int x) { return bd ? -uhf[(l * Qf + x) * M + mr] : uf[(l * Qf + x) * M + mr]; },
                 [&](int x) { return psi[x * PF + j]; }, acc);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * r + lq < M && j0 + l16 < PF)
                a.out.rt[e * L * M * PF + (size_t)(l * M + 4 * r + lq) * PF + j0 + l16] = acc[r];
    }
    __syncthreads();
    for (int k = tid; k < M * P; k += SBS) {
        double s = ((part[k] + part[M * P + k]) + part[2 * M * P + k]) + part[3 * M * P + k];
        if (a.r_extra) s -= a.r_extra[e * M * P + k];
        a.out.ru[e * M * P + k] = s;
    }
}

// Points of one LDS stage of k_sys_blocks: xc volume points (phi and dphix, 4 P doubles each) and fc
// face points (phif, P doubles each); resident when the element's whole tables fit side by side.
// face_staged: one face's point values and tables fit in LDS.
struct BlkStage {
    int xc, fc, resident, doubles, face_staged;
};
inline BlkStage blk_stage(int M, int P, int PF, int Qv, int L, int Qf) {
    constexpr int ROOM = 9984;         // 78 KiB: two blocks share a CU's 160 KiB
    const int LQf = L * Qf;
    BlkStage s;
    s.resident = 4 * P * Qv + P * LQf <= ROOM;
    if (s.resident) {
        s.xc = Qv;
        s.fc = LQf;
        s.doubles = 4 * P * Qv + P * LQf;
    } else {
        const int xc = ROOM / (4 * P) & ~3, fc = ROOM / P & ~3;
        s.xc = xc < 4 ? 4 : xc < Qv ? xc : Qv;
        s.fc = fc < 4 ? 4 : fc < LQf ? fc : LQf;
        const int dv = 4 * P * s.xc, df = P * s.fc;
        s.doubles = dv > df ? dv : df;
    }
    const int face = Qf * (4 * M * M + P + PF + 1);
    s.face_staged = face <= 2 * ROOM;
    if (s.face_staged && face > s.doubles) s.doubles = face;
    return s;
}

// Matrix blocks D, E, F, G, H, J of one element per blockIdx.x; blockIdx.y of gridDim.y shares the
// element's work items (several blocks an element only where the mesh alone leaves the chip idle).
//
// D and E of a component pair (a, b) are four products A_s phi over the volume points plus A_s phif
// over the face points (s < 3: D's dimension, s = 3: E), A_s[i][x] formed in registers from the
// pair's 12 (or 4) point values, which one load per four points brings to each row of 16 lanes and
// row broadcasts hand to every lane. A wave owns TI row tiles of all four slots, so a point's basis
// gradients serve 4 TI products; TI = 1 where P <= 16 (a second tile would be padding). Two row tiles
// and one column tile, held to 128 VGPRs with 13 to 17 spilled (none with TI = 1), let four waves share a
// SIMD, which hide the operand chain and the stores (2 x 2 tiles at two waves a SIMD: 6.5 ms below, this
// 5.5). G, F and J share per (face, b) the operand rows (a, j).
// Bound by its stores: 16^3 Navier-Stokes p = 2 hexes write 10.7 GB, 4.2 ms with every product left
// out (rows of 27 or 9 doubles at 8-byte alignment reach 3.1 TB/s in a store-only loop, whole lines
// 4.5 to 5.8) and 2.9 ms of products with the stores left out; 5.5 ms together (1.9 TB/s), where the
// thread-per-entry loop took 78.6 ms.
template <int M, int TI, bool FS>
__global__ void __launch_bounds__(BBS, 4) k_sys_blocks(SysArgs a, BlkStage st) {
    extern __shared__ double sm[];
    const int el = blockIdx.x;
    const size_t e = (size_t)a.e0 + el;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int NW = BBS / 64;
    const int first = blockIdx.y * NW + wave, stride = gridDim.y * NW;
    const int P = a.P, PF = a.PF, L = a.L, Qv = a.Qv, Qf = a.Qf, LQf = L * Qf, MPF = M * PF;
    const int nu = M * P, nq = M * SD * P, nt = L * MPF;
    const PointWs W = point_ws(M, Qv, LQf);
    const double* ws = a.ws + (size_t)el * W.per_elem;
    const double* wdet = a.g.wdet + e * Qv;
    const double* dphix = a.g.dphix + e * Qv * P * SD;
    const double* phi = a.g.phi;
    const double* phif = a.g.phif + e * LQf * P;
    const double* psi = a.g.psi;
    const double* dA = a.g.dA + e * LQf;
    const int32_t* bnd = a.g.bnd + e * L;
    const double tau = a.pm.tau, cdt = a.c;
    double* sphi = sm;                                  // [xc][P]
    double* sdph = sm + st.xc * P;                      // [xc][P][3]
    double* sphf = sm + (st.resident ? 4 * st.xc * P : 0);

    auto stage_vol = [&](int x0, int n) {
        for (int k = tid; k < n * P; k += BBS) sphi[k] = phi[x0 * P + k];
        for (int k = tid; k < n * P * SD; k += BBS) sdph[k] = dphix[(size_t)x0 * P * SD + k];
    };
    auto stage_face = [&](int f0, int n) {
        for (int k = tid; k < n * P; k += BBS) sphf[k] = phif[(size_t)f0 * P + k];
    };
    auto volume_blocks = [&]() {
        if (st.resident) {
            __syncthreads();
            stage_vol(0, Qv);
            stage_face(0, LQf);
            __syncthreads();
        }
        // D[(a,i)][(b,d,j)] and E[(a,i)][(b,j)]
        const int nblk = (P + 16 * TI - 1) / (16 * TI), tPj = (P + 15) >> 4, nitem = M * M * nblk * tPj;
        for (int r0 = blockIdx.y * NW; r0 < nitem; r0 += stride) {     // the same trips for every wave
            const bool act = r0 + wave < nitem;
            const int item = act ? r0 + wave : nitem - 1;
            const int ab = item / (nblk * tPj), tt = item - ab * nblk * tPj;
            const int am = ab / M, b = ab - am * M, i0 = (tt / tPj) * 16 * TI, j0 = (tt % tPj) * 16;
            const bool diag = am == b;
            const int jc = j0 + l16 < P ? j0 + l16 : P - 1;
            int ic[TI];
#pragma unroll
            for (int t = 0; t < TI; ++t) ic[t] = i0 + 16 * t + l16 < P ? i0 + 16 * t + l16 : P - 1;
            d4 acc[4][TI] = {};
            const double* vp = ws + (size_t)ab * Qv * 12 + (l16 < 12 ? l16 : 11);
            for (int x0 = 0; x0 < Qv; x0 += st.xc) {
                const int n = Qv - x0 < st.xc ? Qv - x0 : st.xc;
                if (!st.resident) {
                    __syncthreads();
                    stage_vol(x0, n);
                    __syncthreads();
                }
                if (!act) continue;
                double nxt = vp[(size_t)(x0 + (lq < n ? lq : n - 1)) * 12];
                for (int k0 = 0; k0 < n; k0 += 4) {
                    const int xk = k0 + lq, x = xk < n ? xk : n - 1, xn = xk + 4 < n ? xk + 4 : n - 1;
                    const double v = xk < n ? nxt : 0.0;
                    nxt = vp[(size_t)(x0 + xn) * 12];
                    double A[4][TI];
                    const double B = sphi[x * P + jc];
#pragma unroll
                    for (int t = 0; t < TI; ++t) {
                        const double* g = sdph + (x * P + ic[t]) * SD;
                        const double g0 = g[0], g1 = g[1], g2 = g[2];
                        A[0][t] = -(wave_ops::row_bcast<0>(v) * g0 + wave_ops::row_bcast<1>(v) * g1 + wave_ops::row_bcast<2>(v) * g2);
                        A[1][t] = -(wave_ops::row_bcast<3>(v) * g0 + wave_ops::row_bcast<4>(v) * g1 + wave_ops::row_bcast<5>(v) * g2);
                        A[2][t] = -(wave_ops::row_bcast<6>(v) * g0 + wave_ops::row_bcast<7>(v) * g1 + wave_ops::row_bcast<8>(v) * g2);
                        A[3][t] = -(wave_ops::row_bcast<9>(v) * g0 + wave_ops::row_bcast<10>(v) * g1 + wave_ops::row_bcast<11>(v) * g2);
                    }
                    if (diag && cdt != 0.0) {
                        const double w = xk < n ? cdt * wdet[x0 + x] : 0.0;
#pragma unroll
                        for (int t = 0; t < TI; ++t) A[3][t] += w * sphi[x * P + ic[t]];
                    }
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int ti = 0; ti < TI; ++ti)
                            acc[s][ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[s][ti], B, acc[s][ti], 0, 0, 0);
                }
            }
            const double* fp = ws + W.face + (size_t)ab * LQf * 4 + (l16 < 4 ? l16 : 3);
            for (int f0 = 0; f0 < LQf; f0 += st.fc) {
                const int n = LQf - f0 < st.fc ? LQf - f0 : st.fc;
                if (!st.resident) {
                    __syncthreads();
                    stage_face(f0, n);
                    __syncthreads();
                }
                if (!act) continue;
                double nxt = fp[(size_t)(f0 + (lq < n ? lq : n - 1)) * 4];
                for (int k0 = 0; k0 < n; k0 += 4) {
                    const int xk = k0 + lq, x = xk < n ? xk : n - 1, xn = xk + 4 < n ? xk + 4 : n - 1;
                    const double v = xk < n ? nxt : 0.0;
                    nxt = fp[(size_t)(f0 + xn) * 4];
                    const double da = (diag && xk < n) ? tau * dA[f0 + x] : 0.0;
                    double pi[TI];
                    const double B = sphf[x * P + jc];
#pragma unroll
                    for (int t = 0; t < TI; ++t) pi[t] = sphf[x * P + ic[t]];
                    const double y[3] = {wave_ops::row_bcast<0>(v), wave_ops::row_bcast<1>(v), wave_ops::row_bcast<2>(v)};
#pragma unroll
                    for (int s = 0; s < 3; ++s)
#pragma unroll
                        for (int ti = 0; ti < TI; ++ti)
                            acc[s][ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(y[s] * pi[ti], B, acc[s][ti], 0, 0, 0);
                    if (diag)
#pragma unroll
                        for (int ti = 0; ti < TI; ++ti)
                            acc[3][ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(da * pi[ti], B, acc[3][ti], 0, 0, 0);
                }
            }
            if (!act) continue;
#pragma unroll
            for (int ti = 0; ti < TI; ++ti)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = i0 + 16 * ti + 4 * r + lq;
                    if (i >= P) continue;
                    double* dr = a.out.D + e * nu * nq + (size_t)(am * P + i) * nq + b * SD * P;
                    double* er = a.out.E + e * nu * nu + (size_t)(am * P + i) * nu + b * P;
                    const int j = j0 + l16;
                    if (j >= P) continue;
#pragma unroll
                    for (int s = 0; s < SD; ++s) dr[s * P + j] = acc[s][ti][r];
                    er[j] = acc[3][ti][r];
                }
        }
    };
    auto face_blocks = [&]() {
        // Face by face, the face's point values, phif, psi and dA staged in LDS (FS; the values were
        // written by the kernel before and come back from HBM, a latency that the short products below
        // cannot hide): per component b, rows (a, j): G[(l,a,j)][(b,d,k)] over two column tiles of k and
        // F[(a,k)][(l,b,j)] from the same operands with their sides exchanged; J[(l,a,j)][(l,b,k)];
        // H[(l,a,j)][(a,k)], the same block for every component.
        const int tP = (P + 15) >> 4, CP = (tP + 1) >> 1, RT = (MPF + 15) >> 4, tPF = (PF + 15) >> 4;
        const int nG = M * RT * CP, nJ = M * RT * tPF, nH = tPF * tP;
        for (int l = 0; l < L; ++l) {
            const double *fY = ws + W.face + (size_t)l * Qf * 4, *fF = phif + (size_t)l * Qf * P, *fA = dA + l * Qf, *fS = psi;
            int ldy = LQf * 4;
            if constexpr (FS) {
                double *sY = sm, *sF = sY + M * M * Qf * 4, *sA = sF + Qf * P, *sS = sA + Qf;
                __syncthreads();
                for (int ab = wave; ab < M * M; ab += NW)
                    for (int k = lane; k < 2 * Qf; k += 64)
                        ((double2*)sY)[ab * Qf * 2 + k] = ((const double2*)(fY + (size_t)ab * ldy))[k];
                for (int k = tid; k < Qf * P; k += BBS) sF[k] = fF[k];
                for (int k = tid; k < Qf; k += BBS) sA[k] = fA[k];
                for (int k = tid; k < Qf * PF; k += BBS) sS[k] = psi[k];
                __syncthreads();
                fY = sY; fF = sF; fA = sA; fS = sS;
                ldy = Qf * 4;
            }
            const bool inner = bnd[l] == 0;
            for (int it = first; it < nG + nJ + nH; it += stride) {
                int q = it < nG ? it : it < nG + nJ ? it - nG : it - nG - nJ;
                if (it < nG) {
                    const int c0 = (q % CP) * 32; q /= CP;
                    const int r0 = (q % RT) * 16, b = q / RT;
                    const int row = r0 + l16 < MPF ? r0 + l16 : MPF - 1, ar = row / PF, jr = row - ar * PF;
                    const int k1 = c0 + l16 < P ? c0 + l16 : P - 1, k2 = c0 + 16 + l16 < P ? c0 + 16 + l16 : P - 1;
                    const double* fv = fY + (size_t)(ar * M + b) * ldy;
                    const double td = ar == b ? tau : 0.0;
                    const bool two = c0 + 16 < P;
                    d4 g[SD][2] = {}, f[2] = {};
                    for (int x0 = 0; x0 < Qf; x0 += 4) {
                        const int xk = x0 + lq, x = xk < Qf ? xk : Qf - 1;
                        const double2 ya = *(const double2*)(fv + x * 4), yb = *(const double2*)(fv + x * 4 + 2);
                        double ps = fS[x * PF + jr], p1 = fF[x * P + k1], p2 = fF[x * P + k2];
                        const double z = xk < Qf ? (yb.y - td * fA[x]) * ps : 0.0;
                        f[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(p1, z, f[0], 0, 0, 0);
                        if (two) f[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(p2, z, f[1], 0, 0, 0);
                        if (inner) {
                            const double y[SD] = {ya.x, ya.y, yb.x};
#pragma unroll
                            for (int d = 0; d < SD; ++d) {
                                const double av = xk < Qf ? -y[d] * ps : 0.0;
                                g[d][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, p1, g[d][0], 0, 0, 0);
                                if (two) g[d][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, p2, g[d][1], 0, 0, 0);
                            }
                        }
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int gr = r0 + 4 * r + lq;
                        if (gr < MPF) {
                            double* dst = a.out.G + e * nt * nq + (size_t)(l * MPF + gr) * nq + b * SD * P;
#pragma unroll
                            for (int d = 0; d < SD; ++d) {
                                if (c0 + l16 < P) dst[d * P + c0 + l16] = g[d][0][r];
                                if (c0 + 16 + l16 < P) dst[d * P + c0 + 16 + l16] = g[d][1][r];
                            }
                        }
                        if (r0 + l16 < MPF) {
                            double* dst = a.out.F + e * nu * nt + (size_t)ar * P * nt + l * MPF + b * PF + jr;
                            const int i = c0 + 4 * r + lq;
                            if (i < P) dst[(size_t)i * nt] = f[0][r];
                            if (i + 16 < P) dst[(size_t)(i + 16) * nt] = f[1][r];
                        }
                    }
                } else if (it < nG + nJ) {
                    const int c0 = (q % tPF) * 16; q /= tPF;
                    const int r0 = (q % RT) * 16, b = q / RT;
                    const int row = r0 + l16 < MPF ? r0 + l16 : MPF - 1, ar = row / PF, jr = row - ar * PF;
                    const int kc = c0 + l16 < PF ? c0 + l16 : PF - 1;
                    const double* fv = fY + (size_t)(ar * M + b) * ldy + 3;
                    const double td = ar == b ? (inner ? tau : 1.0) : 0.0;
                    d4 acc = {};
                    mma16<2>(Qf, [&](int x) { return ((inner ? -fv[x * 4] : 0.0) + td * fA[x]) * fS[x * PF + jr]; },
                             [&](int x) { return fS[x * PF + kc]; }, acc);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r0 + 4 * r + lq < MPF && c0 + l16 < PF)
                            a.out.J[e * nt * nt + (size_t)(l * MPF + r0 + 4 * r + lq) * nt + l * MPF + b * PF + c0 + l16] = acc[r];
                } else {
                    const int c0 = (q % tP) * 16, j0 = (q / tP) * 16;
                    const int jc = j0 + l16 < PF ? j0 + l16 : PF - 1, kc = c0 + l16 < P ? c0 + l16 : P - 1;
                    d4 acc = {};
                    mma16<2>(Qf, [&](int x) { return fA[x] * fS[x * PF + jc]; }, [&](int x) { return fF[x * P + kc]; }, acc);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (j0 + 4 * r + lq < PF && c0 + l16 < P)
#pragma unroll
                            for (int m = 0; m < M; ++m)
                                a.out.H[e * nt * nu + (size_t)(l * MPF + m * PF + j0 + 4 * r + lq) * nu + m * P + c0 + l16] =
                                    inner ? -tau * acc[r] : 0.0;
                }
            }
        }
        // zeros: H off the component diagonal, J off the face diagonal, a row per wave
        for (int row = first; row < nt; row += stride) {
            const int l = row / MPF, m = (row - l * MPF) / PF;
            double* hr = a.out.H + (e * nt + row) * nu;
            for (int c = lane; c < nu; c += 64)
                if (c < m * P || c >= (m + 1) * P) hr[c] = 0.0;
            double* jr = a.out.J + (e * nt + row) * nt;
            for (int c = lane; c < nt; c += 64)
                if (c < l * MPF || c >= (l + 1) * MPF) jr[c] = 0.0;
        }
    };
    // Half the blocks take the faces first, so that some blocks store G, F, H and J while others are
    // in the products of D and E (16^3 Navier-Stokes p = 2 hexes: 3% faster than all in one order).
    if ((el >> 8) & 1) {
        face_blocks();
        volume_blocks();
    } else {
        volume_blocks();
        face_blocks();
    }
}

}  // namespace

size_t element_sys_lds_bytes(const hdg_dims* d, int nqv, int nqf) {
    return sizeof(double) * (size_t)pts_lds(d->ncomp, d->npe, d->npf, d->nlfe, nqv, nqf).total;
}

size_t element_sys_ws_doubles(const hdg_dims* d, int nqv, int nqf) {
    return (size_t)point_ws(d->ncomp, nqv, d->nlfe * nqf).per_elem;
}

// The two kernels over elements [e0, e0 + n) with the point workspace `ws` (not read, may be null,
// when residual-only).
hdg_status element_sys_run(hdg_ctx ctx, const hdg_dims* d, const hdg_elem_geom* g, const hdg_sys_model* m,
                           const hdg_time_term* tt, const int32_t* e2f, const double* u, const double* uhat,
                           int32_t flags, const hdg_elem_arrays* out, int* bad, double* ws, int64_t e0, int64_t n) {
    if (n <= 0) return HDG_OK;
    SysArgs a;
    a.g = *g;
    a.pm.kind = m->kind;
    a.pm.tau = m->tau;
    a.pm.lam = m->lam;
    a.pm.mu = m->mu;
    a.pm.Re = m->Re;
    a.pm.Pr = m->Pr;
    a.pm.gamma = m->gamma;
    a.e2f = e2f;
    a.u = u;
    a.uhat = uhat;
    a.c = tt ? tt->c : 0.0;
    a.u_prev = tt ? tt->u_prev : nullptr;
    a.r_extra = tt ? tt->r_extra : nullptr;
    a.out = *out;
    a.ws = ws;
    a.bad = bad;
    a.e0 = (int)e0;
    a.P = d->npe;
    a.PF = d->npf;
    a.L = d->nlfe;
    a.Qv = g->nqv;
    a.Qf = g->nqf;
    a.residual_only = (flags & HDG_ELEM_RESIDUAL_ONLY) != 0;
    a.keep_mass = (flags & HDG_ELEM_KEEP_MASS) != 0;
    const size_t lds = element_sys_lds_bytes(d, g->nqv, g->nqf);
    const void* kp;
    if (a.residual_only) kp = d->ncomp == 3 ? (const void*)k_sys_points<3, false> : (const void*)k_sys_points<5, false>;
    else kp = d->ncomp == 3 ? (const void*)k_sys_points<3, true> : (const void*)k_sys_points<5, true>;
    if (lds > 64 * 1024) HDG_HIP_CHECK(ctx, hipFuncSetAttribute(kp, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    void* args[] = {(void*)&a};
    HDG_HIP_CHECK(ctx, hipLaunchKernel(kp, dim3((unsigned)n), dim3(SBS), args, lds, ctx->stream));
    HDG_LAUNCH_CHECK(ctx);
    if (a.residual_only) return HDG_OK;
    const BlkStage st = blk_stage(d->ncomp, d->npe, d->npf, g->nqv, d->nlfe, g->nqf);
    const bool one = d->npe <= 16;
    const void* kb;
    if (st.face_staged)
        kb = d->ncomp == 3 ? (one ? (const void*)k_sys_blocks<3, 1, true> : (const void*)k_sys_blocks<3, 2, true>)
                           : (one ? (const void*)k_sys_blocks<5, 1, true> : (const void*)k_sys_blocks<5, 2, true>);
    else
        kb = d->ncomp == 3 ? (one ? (const void*)k_sys_blocks<3, 1, false> : (const void*)k_sys_blocks<3, 2, false>)
                           : (one ? (const void*)k_sys_blocks<5, 1, false> : (const void*)k_sys_blocks<5, 2, false>);
    const size_t bl = sizeof(double) * (size_t)st.doubles;
    if (bl > 64 * 1024) HDG_HIP_CHECK(ctx, hipFuncSetAttribute(kb, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bl));
    // 256 CUs hold 512 blocks, two each: a mesh of fewer elements shares an element's items out over
    // up to seven blocks: the 50 products of D and E of a Navier-Stokes p = 2 hex are seven rounds of eight
    // waves (27 of them: one block 363 us, four 197, seven 168, twelve 167; thread-per-entry loop 8260). Over
    // one to twelve blocks of twelve shapes with 8 to 64 elements seven is within 5% of the best, but for
    // p = 3 hexes (192 and 400 products, nine blocks: 27 elements 434 us, seven 502). 125 to 300 elements,
    // where the bound of 512 gives five to two blocks, would be up to 20% faster with four to eight.
    const int64_t parts = n >= 512 ? 1 : (512 + n - 1) / n < 7 ? (512 + n - 1) / n : 7;
    void* bargs[] = {(void*)&a, (void*)&st};
    HDG_HIP_CHECK(ctx, hipLaunchKernel(kb, dim3((unsigned)n, (unsigned)parts), dim3(BBS), bargs, bl, ctx->stream));
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}
