// Element residuals and Jacobian blocks on the device (Section 4.1, Section 4.4's residual
// evaluation) for scalar convection-diffusion models
//   F(u, q) = beta u^2/2 + gamma u - nu q,   fhat = F(uhat, q).n + tau (u - uhat),
// which cover Poisson (beta = gamma = 0, nu = 1) and viscous Burgers. Each element is one
// workgroup: its quadrature geometry and state are staged in LDS, the state is evaluated at
// the quadrature points (the Phi/Psi products of Section 4.1 as per-point sums), the flux
// and its derivatives are formed per point, and every output entry is one sum over the
// volume or face points, taken as 16x16 tiles on the FP64 matrix cores. q is derived from the
// q-equation (M q_d + B_d u + C_d uhat = 0), so r_q = 0.
//
// Residual rows (the sign of the trace rows as everywhere in the library), with the time
// term of an implicit stage (c = 1/(a_ii dt), u_n, r_x; c = 0 and no r_x: steady):
//   R_u[i]   = -(F, grad phi_i) + <fhat, phi_i> - (s, phi_i) + c (u - u_n, phi_i) + r_x[i]
//   R_t[l,j] = -<fhat, psi_j>_l (interior face), <uhat - u_D, psi_j>_l (Dirichlet face)
// and ru = -R_u, rt = -R_t; D..J are their derivatives with respect to q, u and uhat.
#include "hdg_batch.hpp"
#include "wave_ops.hpp"

namespace {

constexpr int EBS = 256;
using wave_ops::d4;
using wave_ops::mma16s;
using wave_ops::seq;

// One element's inputs and outputs, every pointer already at that element (phi and psi:
// the reference tables; uhat: the face values of the element's mesh, indexed by e2f).
struct ElemView {
    const double *wdet, *dphix, *phi, *phif, *psi, *ndA, *dA, *src, *uD;
    const int32_t *bnd, *e2f;
    const double *u, *uhat, *u_prev, *r_extra;
    double *Minv, *Bd, *Cd, *D, *E, *F, *G, *H, *J, *ru, *rt, *q;
    int P, PF, L, Dm, Qv, Qf, residual_only, keep_mass, eid;
    double nu, tau, beta[3], gamma[3], c;
    int* bad;              // first element with a non-positive mass pivot
};

struct ElemArgs {
    hdg_elem_geom g;
    hdg_conv_diff m;
    const int32_t* e2f;
    const double* u;       // [ne][P]
    const double* uhat;    // [nf][PF]
    hdg_elem_arrays out;
    double c;              // implicit-stage mass factor 1/(a_ii dt); 0: steady
    const double* u_prev;  // [ne][P], read when c != 0
    const double* r_extra; // [ne][P] or null
    int* bad;
    int ne, P, PF, L, D, residual_only, keep_mass;
};

// Threads of an element's block: as few waves as still keep a CU busy, since a phase of one or two tiles
// leaves the others at its barrier. A CU of 160 KiB holds 160 KiB / lds elements, and no more than its
// share of the mesh; 12 of one wave are enough, 6 of two, fewer take four. us with 64, 128 and 256 threads,
// 16,384 elements, Jacobian with kept mass matrices, then residual only:
//   quads p = 2 (19 a CU)  183 222 312, 124 151 205     triangles p = 3 (13)  250 256 333, 170 177 225
//   quads p = 3 (8)        367 300 386, 233 195 245     hexes p = 1 (8)       544 437 546, 290 237 299
//   quads p = 4 (4)       1035 770 586, 589 434 346     tets p = 2 (4)        966 737 659, 612 460 369
// quads p = 1 (48) by the size of the mesh: 256 elements 65 61 59, 2048 71 71 81, 4096 83 92 110.
inline int elem_threads(size_t lds, int64_t ne) {
    const int64_t held = (int64_t)(160 * 1024 / lds), share = (ne + 255) / 256;
    const int64_t per_cu = held < share ? held : share;
    return per_cu >= 12 ? 64 : per_cu >= 6 ? 128 : EBS;
}

// LDS offsets (in doubles) of the element's staged arrays
struct ElemLds {
    int phi, dphi, wdet, phif, psi, ndA, dA, src, uD, u, uh, up, M, t, q, uq, duq, qq, uf, qf, uhf, wF, wFu, fhat, Z,
        total;
};

__host__ __device__ inline ElemLds elem_lds(int P, int PF, int L, int D, int Qv, int Qf) {
    ElemLds o;
    int p = 0;
    o.phi = p;  p += Qv * P;
    o.dphi = p; p += Qv * P * D;
    o.wdet = p; p += Qv;
    o.phif = p; p += L * Qf * P;
    o.psi = p;  p += Qf * PF;
    o.ndA = p;  p += L * Qf * D;
    o.dA = p;   p += L * Qf;
    o.src = p;  p += Qv;
    o.uD = p;   p += L * Qf;
    o.u = p;    p += P;
    o.uh = p;   p += L * PF;
    o.up = p;   p += P;
    o.M = p;    p += P * P;
    o.t = p;    p += D * P;
    o.q = p;    p += D * P;
    o.uq = p;   p += Qv;
    o.duq = p;  p += Qv;
    o.qq = p;   p += Qv * D;
    o.uf = p;   p += L * Qf;
    o.qf = p;   p += L * Qf * D;
    o.uhf = p;  p += L * Qf;
    o.wF = p;   p += Qv * D;
    o.wFu = p;  p += Qv * D;
    o.fhat = p; p += L * Qf;
    o.Z = p;    p += L * Qf;
    o.total = p;
    return o;
}

// v[d] for d < 3 without dynamic indexing (which would put v in scratch memory)
__device__ __forceinline__ double sel3(const double (&v)[3], int d) { return d == 0 ? v[0] : d == 1 ? v[1] : v[2]; }

// Bound by the matrix-core tiles and by the element's arrays (each read and written once); every sum is
// an mma16 tile with its operands in LDS, the tiles shared out over the waves, where a thread per
// entry spent two LDS loads on each multiply-add. Tiles are 16 wide, so P = 25 works at 61% of its
// products. 16384 Burgers p = 4 quads, Jacobian with kept mass matrices: 0.87 ms by entries, 0.58 so
// (1.7 TB/s; the copies to LDS alone 0.15 ms, the rest matrix-core and vector instructions in near
// equal parts); 14400 p = 1 quads 0.26 and 0.16 ms.
template <int D>
__device__ __forceinline__ void element_body(const ElemView& a, double* sm) {
    const int e = a.eid;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), BS = blockDim.x, NW = BS >> 6;
    const int P = a.P, PF = a.PF, L = a.L, Qv = a.Qv, Qf = a.Qf;
    const int nt = L * PF;
    const ElemLds o = elem_lds(P, PF, L, D, Qv, Qf);
    double *phi = sm + o.phi, *dphi = sm + o.dphi, *wdet = sm + o.wdet, *phif = sm + o.phif, *psi = sm + o.psi;
    double *ndA = sm + o.ndA, *dA = sm + o.dA, *src = sm + o.src, *uD = sm + o.uD, *u = sm + o.u, *uh = sm + o.uh;
    double *up = sm + o.up, *duq = sm + o.duq;
    double *Mm = sm + o.M, *t = sm + o.t, *q = sm + o.q, *uq = sm + o.uq, *qq = sm + o.qq, *uf = sm + o.uf;
    double *qf = sm + o.qf, *uhf = sm + o.uhf, *wF = sm + o.wF, *wFu = sm + o.wFu, *fhat = sm + o.fhat, *Z = sm + o.Z;

    // 1. stage geometry, reference tables and state: every copy in flight at once
    const double cdt = a.c;
    const int LQf = L * Qf;
    auto stage = [&](const double* g, double* dst, int n) { wave_ops::copy_to_lds(g, dst, 8 * n, wave, NW); };
    stage(a.dphix, dphi, Qv * P * D);
    stage(a.phif, phif, LQf * P);
    if (a.keep_mass) stage(a.Minv, Mm, P * P);
    stage(a.phi, phi, Qv * P);
    stage(a.ndA, ndA, LQf * D);
    stage(a.wdet, wdet, Qv);
    stage(a.src, src, Qv);
    stage(a.psi, psi, Qf * PF);
    stage(a.dA, dA, LQf);
    stage(a.uD, uD, LQf);
    stage(a.u, u, P);
    if (cdt != 0.0) stage(a.u_prev, up, P);
    for (int l = wave; l < L; l += NW) wave_ops::copy_to_lds(a.uhat + (size_t)a.e2f[l] * PF, uh + l * PF, 8 * PF, 0, 1);
    wave_ops::copies_done();
    __syncthreads();

    // 2. mass matrix and its inverse (Gauss-Jordan in place; M is SPD, no interchanges), or
    //    the inverse kept from an earlier evaluation on the same mesh (state-independent)
    // tiles go round the waves: job counts them, NW is a power of two
    int job = 0;
    auto mine = [&]() { return (job++ & (NW - 1)) == wave; };
    if (!a.keep_mass) {
        for (int i0 = 0; i0 < P; i0 += 16)
            for (int j0 = 0; j0 < P; j0 += 16) {
                if (!mine()) continue;
                const int i = i0 + l16 < P ? i0 + l16 : P - 1, j = j0 + l16 < P ? j0 + l16 : P - 1;
                d4 acc = {};
                mma16s<true, false>(Qv, seq(phi + i, P, wdet, 1), seq(phi + j, P), acc);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (i0 + 4 * r + lq < P && j0 + l16 < P) Mm[(i0 + 4 * r + lq) * P + j0 + l16] = acc[r];
            }
        __syncthreads();
        const int gi = tid >> 4, gj = tid & 15;
        for (int k = 0; k < P; ++k) {
            const double piv = Mm[k * P + k];
            if (!(piv > 0.0) || !isfinite(piv)) {
                if (tid == 0) atomicMin(a.bad, e);
                return;    // uniform across the workgroup: every thread read the same pivot
            }
            const double rp = 1.0 / piv;
            // row k scaled (entry k becomes 1/piv), other rows updated with the old column k
            for (int i = gi; i < P; i += BS / 16) {
                if (i == k) continue;
                const double f = Mm[i * P + k] * rp;
                for (int j = gj; j < P; j += 16)
                    if (j != k) Mm[i * P + j] -= f * Mm[k * P + j];
            }
            __syncthreads();
            for (int idx = tid; idx < P; idx += BS) {
                if (idx != k) {
                    Mm[idx * P + k] = -Mm[idx * P + k] * rp;
                    Mm[k * P + idx] *= rp;
                }
            }
            if (tid == 0) Mm[k * P + k] = rp;
            __syncthreads();
        }
    }

    // 3. u and u_n (columns 0 and 1) at the volume points, u at the face points, uhat at the points
    //    of every face (a column per face)
    for (int vol = 1; vol >= 0; --vol) {
        const int n = vol ? Qv : LQf;
        for (int x0 = 0; x0 < n; x0 += 16) {
            if (!mine()) continue;
            const int x = x0 + l16 < n ? x0 + l16 : n - 1;
            d4 acc = {};
            mma16s<false, false>(P, seq((vol ? phi : phif) + x * P, 1), seq(l16 == 1 && cdt != 0.0 ? up : u, 1), acc);
            double* dst = !vol ? uf : l16 == 0 ? uq : duq;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (x0 + 4 * r + lq < n && l16 <= vol) dst[x0 + 4 * r + lq] = acc[r];
        }
    }
    for (int x0 = 0; x0 < Qf; x0 += 16) {                // L <= 6 columns
        if (!mine()) continue;
        const int x = x0 + l16 < Qf ? x0 + l16 : Qf - 1, l = l16 < L ? l16 : L - 1;
        d4 acc = {};
        mma16s<false, false>(PF, seq(psi + x * PF, 1), seq(uh + l * PF, 1), acc);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (x0 + 4 * r + lq < Qf && l16 < L) uhf[l16 * Qf + x0 + 4 * r + lq] = acc[r];
    }
    __syncthreads();

    // 4. q = -M^{-1} (B_d u + C_d uhat): -B_d u in t, the face sums in q, both then one operand of the
    //    product with M^{-1}
    const int DP = D * P;
    for (int d = 0; d < D; ++d)
        for (int i0 = 0; i0 < P; i0 += 16)
            for (int fc = 0; fc < 2; ++fc) {
                if (!mine()) continue;
                const int i = i0 + l16 < P ? i0 + l16 : P - 1;
                d4 acc = {};
                if (fc)
                    mma16s<false, true>(LQf, seq(uhf, 1), seq(phif + i, P, ndA + d, D), acc);
                else
                    mma16s<false, true>(Qv, seq(uq, 1), seq(dphi + i * D + d, DP, wdet, 1), acc);
                // all 16 rows are alike
                if (lq == 0 && i0 + l16 < P) (fc ? q : t)[d * P + i0 + l16] = fc ? acc[0] : -acc[0];
            }
    __syncthreads();
    for (int k = tid; k < DP; k += BS) t[k] += q[k];
    __syncthreads();
    for (int i0 = 0; i0 < P; i0 += 16) {
        if (!mine()) continue;
        const int i = i0 + l16 < P ? i0 + l16 : P - 1, d = l16 < D ? l16 : 0;
        d4 acc = {};
        mma16s<false, false>(P, seq(t + d * P, 1), seq(Mm + i * P, 1), acc);
        if (lq < D && i0 + l16 < P) {                    // D <= 3 < 4 rows: register 0
            q[lq * P + i0 + l16] = acc[0];
            if (a.q) a.q[lq * P + i0 + l16] = acc[0];
        }
    }
    __syncthreads();

    // 5. q at the points, then the flux and its derivatives per point
    for (int vol = 1; vol >= 0; --vol) {
        const int n = vol ? Qv : LQf;
        for (int x0 = 0; x0 < n; x0 += 16) {
            if (!mine()) continue;
            const int x = x0 + l16 < n ? x0 + l16 : n - 1, d = l16 < D ? l16 : 0;
            d4 acc = {};
            mma16s<false, false>(P, seq((vol ? phi : phif) + x * P, 1), seq(q + d * P, 1), acc);
            double* dst = vol ? qq : qf;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (x0 + 4 * r + lq < n && l16 < D) dst[(x0 + 4 * r + lq) * D + l16] = acc[r];
        }
    }
    __syncthreads();
    const double nu = a.nu, tau = a.tau;
    for (int x = tid; x < Qv; x += BS) {
        const double v = uq[x], w = wdet[x];
        for (int d = 0; d < D; ++d) {
            const double bt = sel3(a.beta, d), gm = sel3(a.gamma, d);
            wF[x * D + d] = w * (bt * 0.5 * v * v + gm * v - nu * qq[x * D + d]);
            wFu[x * D + d] = w * (bt * v + gm);
        }
        // the source and time term, over u_n at the points
        duq[x] = w * (src[x] - (cdt != 0.0 ? cdt * (v - duq[x]) : 0.0));
    }
    for (int lx = tid; lx < LQf; lx += BS) {
        const double v = uhf[lx];
        double fn = 0.0, zn = 0.0;
        for (int d = 0; d < D; ++d) {
            const double n = ndA[lx * D + d];
            const double bt = sel3(a.beta, d), gm = sel3(a.gamma, d);
            fn += (bt * 0.5 * v * v + gm * v - nu * qf[lx * D + d]) * n;
            zn += (bt * v + gm) * n;
        }
        fhat[lx] = fn + tau * (uf[lx] - v) * dA[lx];
        Z[lx] = zn - tau * dA[lx];    // d fhat / d uhat per unit trace value
    }
    __syncthreads();

    // 6. right-hand sides ru = -R_u, rt = -R_t. The D + 2 sums of ru (a dimension of (F, grad phi) each,
    //    the source and time term, the faces) go to min(4, 2 D) partials over the room of t and q,
    //    added in order.
    const int np = 2 * D < 4 ? 2 * D : 4;
    for (int slot = 0; slot < np; ++slot)
        for (int i0 = 0; i0 < P; i0 += 16) {
            if (!mine()) continue;
            const int i = i0 + l16 < P ? i0 + l16 : P - 1;
            d4 acc = {}, fc = {};
            for (int sum = slot; sum < D + 2; sum += np) {
                if (sum < D) mma16s<false, false>(Qv, seq(wF + sum, D), seq(dphi + i * D + sum, DP), acc);
                else if (sum == D) mma16s<false, false>(Qv, seq(duq, 1), seq(phi + i, P), acc);
                else mma16s<false, false>(LQf, seq(fhat, 1), seq(phif + i, P), fc);
            }
            if (lq == 0 && i0 + l16 < P) t[slot * P + i0 + l16] = acc[0] - fc[0];
        }
    for (int k = tid; k < nt; k += BS) {
        const int l = k / PF, j = k - l * PF;
        const bool bd = a.bnd[l] != 0;
        double s = 0.0;
        for (int x = 0; x < Qf; ++x) {
            const int lx = l * Qf + x;
            s += (bd ? -dA[lx] * (uhf[lx] - uD[lx]) : fhat[lx]) * psi[x * PF + j];
        }
        a.rt[k] = s;
    }
    __syncthreads();
    for (int i = tid; i < P; i += BS) {
        double s = t[i];
        for (int w = 1; w < np; ++w) s += t[w * P + i];
        if (a.r_extra) s -= a.r_extra[i];
        a.ru[i] = s;
    }
    if (a.residual_only) return;

    // 7. matrices. With dF/dq = -nu I: the volume part of D is nu B_d, and G on an interior
    // face is -nu C_d^T.
    const bool put_mass = !a.keep_mass;      // Minv, Bd, Cd: written unless kept
    if (put_mass)
        for (int k = tid; k < P * P; k += BS) a.Minv[k] = Mm[k];
    for (int i0 = 0; i0 < P; i0 += 16)                      // Bd, D, E
        for (int j0 = 0; j0 < P; j0 += 16) {
            if (!mine()) continue;
            const int i = i0 + l16 < P ? i0 + l16 : P - 1, j = j0 + l16 < P ? j0 + l16 : P - 1;
            d4 bd[D] = {}, ev = {};
            auto vol = [&](const double* pw, const double* pj, const double* pi, const double* pd, const double* pf, bool in) {
                const double w = in ? *pw : 0.0;
                double g = cdt * w * *pi;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    g -= in ? pf[d] * pd[d] : 0.0;
                    bd[d] = __builtin_amdgcn_mfma_f64_16x16x4f64(w * pd[d], *pj, bd[d], 0, 0, 0);
                }
                ev = __builtin_amdgcn_mfma_f64_16x16x4f64(g, *pj, ev, 0, 0, 0);
            };
            int left = Qv;
            {
                const int k = lq * P;
                const double *pw = wdet + lq, *pj = phi + k + j, *pi = phi + k + i, *pd = dphi + (k + i) * D, *pf = wFu + lq * D;
                for (; left >= 4; left -= 4, pw += 4, pj += 4 * P, pi += 4 * P, pd += 4 * DP, pf += 4 * D)
                    vol(pw, pj, pi, pd, pf, true);
                if (left > 0) {
                    const bool in = lq < left;
                    const int o = in ? 0 : left - 1 - lq;
                    vol(pw + o, pj + o * P, pi + o * P, pd + o * DP, pf + o * D, in);
                }
            }
            if (put_mass)
#pragma unroll
                for (int d = 0; d < D; ++d)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (i0 + 4 * r + lq < P && j0 + l16 < P)
                            a.Bd[(size_t)(d * P + i0 + 4 * r + lq) * P + j0 + l16] = bd[d][r];
            auto face = [&](const double* pa, const double* pi, const double* pj, const double* pn, bool in) {
                const double v = in ? *pi : 0.0;
#pragma unroll
                for (int d = 0; d < D; ++d)
                    bd[d] = __builtin_amdgcn_mfma_f64_16x16x4f64(-pn[d] * v, *pj, bd[d], 0, 0, 0);
                ev = __builtin_amdgcn_mfma_f64_16x16x4f64(tau * *pa * v, *pj, ev, 0, 0, 0);
            };
            left = LQf;
            {
                const double *pa = dA + lq, *pi = phif + lq * P + i, *pj = phif + lq * P + j, *pn = ndA + lq * D;
                for (; left >= 4; left -= 4, pa += 4, pi += 4 * P, pj += 4 * P, pn += 4 * D) face(pa, pi, pj, pn, true);
                if (left > 0) {
                    const bool in = lq < left;
                    const int o = in ? 0 : left - 1 - lq;
                    face(pa + o, pi + o * P, pj + o * P, pn + o * D, in);
                }
            }
            const int jr = j0 + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int ir = i0 + 4 * r + lq;
                if (ir >= P || jr >= P) continue;
#pragma unroll
                for (int d = 0; d < D; ++d)
                    a.D[ir * DP + d * P + jr] = nu * bd[d][r];
                a.E[ir * P + jr] = ev[r];
            }
        }
    for (int l = 0; l < L; ++l) {
        const bool interior = a.bnd[l] == 0;
        for (int j0 = 0; j0 < PF; j0 += 16) {
            const int j = j0 + l16 < PF ? j0 + l16 : PF - 1;
            for (int i0 = 0; i0 < P; i0 += 16) {            // rows j, columns i: Cd, F, G, H
                if (!mine()) continue;
                const int i = i0 + l16 < P ? i0 + l16 : P - 1;
                d4 cd[D] = {}, f = {}, h = {};
                for (int x0 = 0; x0 < Qf; x0 += 4) {
                    const int xk = x0 + lq, x = xk < Qf ? xk : Qf - 1, lx = l * Qf + x;
                    const double ps = xk < Qf ? psi[x * PF + j] : 0.0, pi = phif[lx * P + i];
#pragma unroll
                    for (int d = 0; d < D; ++d)
                        cd[d] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ndA[lx * D + d] * ps, pi, cd[d], 0, 0, 0);
                    f = __builtin_amdgcn_mfma_f64_16x16x4f64(xk < Qf ? Z[lx] * ps : 0.0, pi, f, 0, 0, 0);
                    h = __builtin_amdgcn_mfma_f64_16x16x4f64(dA[lx] * ps, pi, h, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int jr = j0 + 4 * r + lq, ir = i0 + l16, c = l * PF + jr;
                    if (jr >= PF || ir >= P) continue;
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                        if (put_mass) a.Cd[(d * P + ir) * nt + c] = cd[d][r];
                        a.G[c * DP + d * P + ir] = interior ? -nu * cd[d][r] : 0.0;
                    }
                    a.F[ir * nt + c] = f[r];
                    a.H[c * P + ir] = interior ? -tau * h[r] : 0.0;
                }
            }
            for (int k0 = 0; k0 < PF; k0 += 16) {           // J[(l,j)][(l,j')]
                if (!mine()) continue;
                const int k = k0 + l16 < PF ? k0 + l16 : PF - 1;
                d4 acc = {};
                mma16s<true, false>(Qf, seq(psi + j, PF, (interior ? Z : dA) + l * Qf, 1), seq(psi + k, PF), acc);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (j0 + 4 * r + lq < PF && k0 + l16 < PF)
                        a.J[(l * PF + j0 + 4 * r + lq) * nt + l * PF + k0 + l16] = interior ? -acc[r] : acc[r];
            }
        }
    }
    // J is block diagonal in l
    for (int row = wave, lo = 0; row < nt; row += NW) {
        while (row >= lo + PF) lo += PF;
        for (int c = lane; c < nt; c += 64)
            if (c < lo || c >= lo + PF) a.J[row * nt + c] = 0.0;
    }
}

template <int D>
__global__ void __launch_bounds__(EBS, 4) k_element_blocks(ElemArgs a) {
    extern __shared__ double sm[];
    const size_t E = blockIdx.x;
    const int P = a.P, PF = a.PF, L = a.L, Qv = a.g.nqv, Qf = a.g.nqf, nt = L * PF;
    ElemView v;
    v.wdet = a.g.wdet + E * Qv;
    v.dphix = a.g.dphix + E * Qv * P * D;
    v.phi = a.g.phi;
    v.phif = a.g.phif + E * L * Qf * P;
    v.psi = a.g.psi;
    v.ndA = a.g.ndA + E * L * Qf * D;
    v.dA = a.g.dA + E * L * Qf;
    v.src = a.g.src + E * Qv;
    v.uD = a.g.uD + E * L * Qf;
    v.bnd = a.g.bnd + E * L;
    v.e2f = a.e2f + E * L;
    v.u = a.u + E * P;
    v.uhat = a.uhat;
    v.u_prev = a.u_prev ? a.u_prev + E * P : nullptr;
    v.r_extra = a.r_extra ? a.r_extra + E * P : nullptr;
    const bool mats = !a.residual_only;
    v.Minv = (mats || a.keep_mass) ? a.out.Minv + E * P * P : nullptr;
    v.Bd = mats ? a.out.Bd + E * D * P * P : nullptr;
    v.Cd = mats ? a.out.Cd + E * D * P * nt : nullptr;
    v.D = mats ? a.out.D + E * P * D * P : nullptr;
    v.E = mats ? a.out.E + E * P * P : nullptr;
    v.F = mats ? a.out.F + E * P * nt : nullptr;
    v.G = mats ? a.out.G + E * nt * D * P : nullptr;
    v.H = mats ? a.out.H + E * nt * P : nullptr;
    v.J = mats ? a.out.J + E * nt * nt : nullptr;
    v.ru = a.out.ru + E * P;
    v.rt = a.out.rt + E * nt;
    v.q = a.out.q ? a.out.q + E * D * P : nullptr;
    v.P = P; v.PF = PF; v.L = L; v.Dm = D; v.Qv = Qv; v.Qf = Qf;
    v.residual_only = a.residual_only;
    v.keep_mass = a.keep_mass;
    v.eid = (int)E;
    v.nu = a.m.nu; v.tau = a.m.tau; v.c = a.c;
    for (int d = 0; d < 3; ++d) { v.beta[d] = a.m.beta[d]; v.gamma[d] = a.m.gamma[d]; }
    v.bad = a.bad;
    element_body<D>(v, sm);
}

// Batched instances: element e belongs to instance eid[e]; its arrays sit at the instance's
// offsets plus its instance-local index times the per-element sizes.
// 128 registers, two of them spilled: four waves a SIMD (eight p = 4 quad instances, 8000 elements, residual:
// 266 us with 131 registers and three waves, 236 so).
__global__ void __launch_bounds__(EBS, 4) k_element_blocks_batch(const ElemInst* __restrict__ inst,
                                                               const int32_t* __restrict__ eid, ElemBatchArgs a) {
    extern __shared__ double sm[];
    const int64_t e = blockIdx.x;
    const ElemInst& q = inst[eid[e]];
    const int64_t E = e - q.e0;
    const int P = q.P, PF = q.PF, L = q.L, D = q.D, Qv = q.Qv, Qf = q.Qf, nt = L * PF;
    ElemView v;
    v.wdet = a.g.wdet + q.g_wdet + E * Qv;
    v.dphix = a.g.dphix + q.g_dphix + E * Qv * P * D;
    v.phi = a.g.phi + q.g_phi;
    v.phif = a.g.phif + q.g_phif + E * L * Qf * P;
    v.psi = a.g.psi + q.g_psi;
    v.ndA = a.g.ndA + q.g_ndA + E * L * Qf * D;
    v.dA = a.g.dA + q.g_dA + E * L * Qf;
    v.src = a.g.src + q.g_src + E * Qv;
    v.uD = a.g.uD + q.g_uD + E * L * Qf;
    v.bnd = a.g.bnd + q.e2f_off + E * L;
    v.e2f = a.e2f + q.e2f_off + E * L;
    v.u = a.u + q.u_off + E * P;
    v.uhat = a.uhat + q.uh_off;
    v.u_prev = (q.c != 0.0) ? a.u_prev + q.u_off + E * P : nullptr;
    v.r_extra = a.r_extra ? a.r_extra + q.u_off + E * P : nullptr;
    const bool mats = !a.residual_only;
    v.Minv = (mats || a.keep_mass) ? a.out.Minv + q.out_off[0] + E * P * P : nullptr;
    v.Bd = mats ? a.out.Bd + q.out_off[1] + E * D * P * P : nullptr;
    v.Cd = mats ? a.out.Cd + q.out_off[2] + E * D * P * nt : nullptr;
    v.D = mats ? a.out.D + q.out_off[3] + E * P * D * P : nullptr;
    v.E = mats ? a.out.E + q.out_off[4] + E * P * P : nullptr;
    v.F = mats ? a.out.F + q.out_off[5] + E * P * nt : nullptr;
    v.G = mats ? a.out.G + q.out_off[6] + E * nt * D * P : nullptr;
    v.H = mats ? a.out.H + q.out_off[7] + E * nt * P : nullptr;
    v.J = mats ? a.out.J + q.out_off[8] + E * nt * nt : nullptr;
    v.ru = a.out.ru + q.out_off[9] + E * P;
    v.rt = a.out.rt + q.out_off[10] + E * nt;
    v.q = a.out.q ? a.out.q + q.q_off + E * D * P : nullptr;
    v.P = P; v.PF = PF; v.L = L; v.Dm = D; v.Qv = Qv; v.Qf = Qf;
    v.residual_only = a.residual_only;
    v.keep_mass = a.keep_mass;
    v.eid = (int)e;
    v.nu = q.nu; v.tau = q.tau; v.c = q.c;
    for (int d = 0; d < 3; ++d) { v.beta[d] = q.beta[d]; v.gamma[d] = q.gamma[d]; }
    v.bad = a.bad;
    if (v.Dm == 2) element_body<2>(v, sm);
    else if (v.Dm == 3) element_body<3>(v, sm);
    else element_body<1>(v, sm);
}

// ||R|| of instance blockIdx.x: its element u-rows and its faces' summed trace rows.
__global__ void __launch_bounds__(EBS) k_residual_norm_batch(const InstDesc* __restrict__ desc,
                                                             const double* __restrict__ ru,
                                                             const double* __restrict__ rt,
                                                             const int32_t* __restrict__ f2e, double* norms) {
    __shared__ double red[EBS / 64];
    const InstDesc& q = desc[blockIdx.x];
    double acc = 0.0;
    const int64_t nuu = (int64_t)q.ne * q.nu;
    for (int64_t k = threadIdx.x; k < nuu; k += EBS) {
        const double v = ru[q.off[9] + k];
        acc += v * v;
    }
    const int64_t nfe = (int64_t)q.nf * q.nb;
    for (int64_t k = threadIdx.x; k < nfe; k += EBS) {
        const int64_t f = k / q.nb;
        const int j = (int)(k - f * q.nb);
        const int32_t* fe = f2e + q.f2e_off + 4 * f;
        double v = rt[q.off[10] + (int64_t)fe[0] * q.nt + (int64_t)fe[1] * q.nb + j];
        if (fe[2] >= 0) v += rt[q.off[10] + (int64_t)fe[2] * q.nt + (int64_t)fe[3] * q.nb + j];
        acc += v * v;
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < EBS / 64; ++w) s += red[w];
        norms[blockIdx.x] = sqrt(s);
    }
}

// u += alpha_i du and uhat += alpha_i x over instance i = blockIdx.x (nothing when alpha_i = 0).
__global__ void __launch_bounds__(EBS) k_newton_update_batch(const InstDesc* __restrict__ desc,
                                                             const double* __restrict__ alpha,
                                                             const double* __restrict__ du, double* u,
                                                             const double* __restrict__ x, double* uhat) {
    const InstDesc& q = desc[blockIdx.x];
    const double al = alpha[blockIdx.x];
    if (al == 0.0) return;
    const int64_t nuu = (int64_t)q.ne * q.nu, nfe = (int64_t)q.nf * q.nb;
    for (int64_t k = threadIdx.x; k < nuu; k += EBS) u[q.du_off + k] += al * du[q.du_off + k];
    for (int64_t k = threadIdx.x; k < nfe; k += EBS) uhat[q.vec_off + k] += al * x[q.vec_off + k];
}

}  // namespace

size_t element_batch_lds_bytes(int P, int PF, int L, int D, int nqv, int nqf) {
    return sizeof(double) * (size_t)elem_lds(P, PF, L, D, nqv, nqf).total;
}

hdg_status element_blocks_batch_run(hdg_ctx ctx, int64_t total_ne, const ElemInst* inst_dev, const int32_t* eid,
                                    const ElemBatchArgs& a, size_t lds) {
    if (total_ne == 0) return HDG_OK;
    // lds is the largest instance's
    hipLaunchKernelGGL(k_element_blocks_batch, dim3((unsigned)total_ne), dim3(elem_threads(lds, total_ne)), lds, ctx->stream,
                       inst_dev, eid, a);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status residual_norm_batch_run(hdg_ctx ctx, int n_inst, const InstDesc* desc, const double* ru, const double* rt,
                                   const int32_t* f2e, double* norms) {
    if (n_inst == 0) return HDG_OK;
    hipLaunchKernelGGL(k_residual_norm_batch, dim3(n_inst), dim3(EBS), 0, ctx->stream, desc, ru, rt, f2e, norms);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

hdg_status newton_update_batch_run(hdg_ctx ctx, int n_inst, const InstDesc* desc, const double* alpha,
                                   const double* du, double* u, const double* x, double* uhat) {
    if (n_inst == 0) return HDG_OK;
    hipLaunchKernelGGL(k_newton_update_batch, dim3(n_inst), dim3(EBS), 0, ctx->stream, desc, alpha, du, u, x, uhat);
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}

size_t element_blocks_lds_bytes(const hdg_dims* d, int nqv, int nqf) {
    const ElemLds o = elem_lds(d->npe, d->npf, d->nlfe, d->dim, nqv, nqf);
    return sizeof(double) * (size_t)o.total;
}

hdg_status element_blocks_run(hdg_ctx ctx, const hdg_dims* d, const hdg_elem_geom* g, const hdg_conv_diff* m,
                              const hdg_time_term* tt, const int32_t* e2f, const double* u, const double* uhat,
                              int flags, const hdg_elem_arrays* out, int* bad) {
    if (d->ne == 0) return HDG_OK;
    ElemArgs a;
    a.g = *g;
    a.m = *m;
    a.e2f = e2f;
    a.u = u;
    a.uhat = uhat;
    a.out = *out;
    a.c = tt ? tt->c : 0.0;
    a.u_prev = tt ? tt->u_prev : nullptr;
    a.r_extra = tt ? tt->r_extra : nullptr;
    a.bad = bad;
    a.ne = d->ne;
    a.P = d->npe;
    a.PF = d->npf;
    a.L = d->nlfe;
    a.D = d->dim;
    a.residual_only = (flags & HDG_ELEM_RESIDUAL_ONLY) != 0;
    a.keep_mass = (flags & HDG_ELEM_KEEP_MASS) != 0;
    const size_t lds = element_blocks_lds_bytes(d, g->nqv, g->nqf);
    const void* k = d->dim == 2   ? (const void*)k_element_blocks<2>
                    : d->dim == 3 ? (const void*)k_element_blocks<3>
                                  : (const void*)k_element_blocks<1>;
    void* args[] = {(void*)&a};
    HDG_HIP_CHECK(ctx, hipLaunchKernel(k, dim3(d->ne), dim3(elem_threads(lds, d->ne)), args, lds, ctx->stream));
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}
