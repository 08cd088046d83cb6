// Batched independent instances: descriptor tables, a small autotuner for the
// persistent condensation launch, and the segmented FGMRES driver (per-instance
// Arnoldi, Givens and convergence masks; one host synchronisation per cycle,
// optionally replayed as one captured hipGraph). Same arithmetic as the
// single-instance path (Sections 3.1-3.2, 4.1-4.5).
#include <chrono>
#include <cmath>
#include <cstring>
#include <map>
#include <new>
#include <string>

#include "hdg_batch.hpp"

struct hdg_batch_s {
    int device = 0;
    std::vector<hdg_dims> dims;
    std::vector<InstDesc> host;
    std::vector<std::vector<int64_t>> offs;   // [array id][n_inst + 1]
    BatchDev dev;
    std::vector<void*> allocs;
    int tuned_grid = 0;
};

namespace {

enum {
    A_MINV, A_BD, A_CD, A_D, A_E, A_F, A_G, A_H, A_J, A_RU, A_RT,
    A_KBAR, A_RBAR, A_LOCAL, A_DU, A_DQ, A_K, A_NBR, A_VEC, A_F2E, A_E2F, A_BINV, A_NARR
};

template <typename T>
T* dev_upload(hdg_batch b, const std::vector<T>& v, hipError_t* err) {
    void* p = nullptr;
    const size_t bytes = std::max<size_t>(sizeof(T) * v.size(), 16);
    *err = hipMalloc(&p, bytes);
    if (*err != hipSuccess) return nullptr;
    b->allocs.push_back(p);
    if (!v.empty()) *err = hipMemcpy(p, v.data(), sizeof(T) * v.size(), hipMemcpyHostToDevice);
    return (T*)p;
}

double now_s() {
    return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

}  // namespace

extern "C" {

hdg_status hdg_batch_create(hdg_ctx ctx, int32_t n_inst, const hdg_dims* dims_h, hdg_batch* out) {
    if (!ctx || !out) return HDG_ERR_ARG;
    *out = nullptr;
    if (n_inst < 1 || !dims_h) {
        ctx->err = "hdg_batch_create: need n_inst >= 1 and dims";
        return HDG_ERR_ARG;
    }
    hdg_batch b = new (std::nothrow) hdg_batch_s();
    if (!b) return HDG_ERR_NOMEM;
    b->device = ctx->device;
    b->dims.assign(dims_h, dims_h + n_inst);
    b->offs.assign(A_NARR, std::vector<int64_t>(n_inst + 1, 0));
    std::vector<int32_t> eid, fid, dof_inst, blk_inst, ib0(n_inst), ib1(n_inst);
    std::vector<int64_t> blk_lo, blk_hi;
    std::vector<FaceBlk> fblk;
    int64_t e0 = 0, f0 = 0;
    size_t max_cond = 0, max_rec = 0;
    double tile_work = 0.0;
    for (int i = 0; i < n_inst; ++i) {
        const hdg_dims& d = dims_h[i];
        if (d.ne < 1 || d.nf < 1 || d.ncomp < 1 || d.dim < 1 || d.dim > 3 || d.npe < 1 || d.npf < 1 || d.nlfe < 2 ||
            d.nlfe > 6) {
            ctx->err = "hdg_batch_create: bad dims for instance " + std::to_string(i);
            delete b;
            return HDG_ERR_SHAPE;
        }
        InstDesc q;
        std::memset(&q, 0, sizeof(q));
        q.M = d.ncomp; q.D = d.dim; q.P = d.npe; q.PF = d.npf; q.L = d.nlfe;
        q.nu = q.M * q.P; q.nq = q.M * q.D * q.P; q.nt = q.L * q.M * q.PF; q.nb = q.M * q.PF;
        q.S = 2 * q.L - 1; q.R = q.nu + q.nt; q.C = q.R + 1; q.NW = q.P + q.L * q.PF; q.KD = q.D * q.P;
        q.ne = d.ne; q.nf = d.nf;
        if (q.nb > 8 || q.S * q.nb > 64) {
            ctx->err = "hdg_batch_create: batched instances need M*P_F <= 8 and S*M*P_F <= 64 (instance " +
                       std::to_string(i) + ")";
            delete b;
            return HDG_ERR_SHAPE;
        }
        const size_t cond = (size_t)q.R * q.C + (size_t)q.KD * q.NW;
        if (cond * 8 > 150 * 1024) {
            ctx->err = "hdg_batch_create: element system of instance " + std::to_string(i) + " exceeds LDS";
            delete b;
            return HDG_ERR_SHAPE;
        }
        max_cond = std::max(max_cond, cond);
        const double madds = (double)q.ne * q.R * q.R * q.KD;
        tile_work += cond_tiles(q.R, q.KD) ? madds : -madds;
        max_rec = std::max(max_rec, (size_t)q.nt + q.nu + q.P);
        const int64_t per[A_NARR] = {
            (int64_t)q.ne * q.P * q.P, (int64_t)q.ne * q.D * q.P * q.P, (int64_t)q.ne * q.D * q.P * q.L * q.PF,
            (int64_t)q.ne * q.nu * q.nq, (int64_t)q.ne * q.nu * q.nu, (int64_t)q.ne * q.nu * q.nt,
            (int64_t)q.ne * q.nt * q.nq, (int64_t)q.ne * q.nt * q.nu, (int64_t)q.ne * q.nt * q.nt,
            (int64_t)q.ne * q.nu, (int64_t)q.ne * q.nt,
            (int64_t)q.ne * q.nt * q.nt, (int64_t)q.ne * q.nt, (int64_t)q.ne * q.nu * q.C,
            (int64_t)q.ne * q.nu, (int64_t)q.ne * q.nq,
            (int64_t)q.nf * q.S * q.nb * q.nb, (int64_t)q.nf * q.S, (int64_t)q.nf * q.nb,
            (int64_t)q.nf * 4, (int64_t)q.ne * q.L, (int64_t)q.nf * q.nb * q.nb};
        for (int a = 0; a < A_NARR; ++a) b->offs[a][i + 1] = b->offs[a][i] + per[a];
        for (int a = 0; a < 11; ++a) q.off[a] = b->offs[a][i];
        q.kbar_off = b->offs[A_KBAR][i]; q.rbar_off = b->offs[A_RBAR][i]; q.local_off = b->offs[A_LOCAL][i];
        q.du_off = b->offs[A_DU][i]; q.dq_off = b->offs[A_DQ][i]; q.K_off = b->offs[A_K][i];
        q.nbr_off = b->offs[A_NBR][i]; q.vec_off = b->offs[A_VEC][i]; q.f2e_off = b->offs[A_F2E][i];
        q.e2f_off = b->offs[A_E2F][i]; q.binv_off = b->offs[A_BINV][i];
        q.e0 = e0; q.f0 = f0;
        e0 += q.ne;
        f0 += q.nf;
        b->host.push_back(q);
        eid.insert(eid.end(), q.ne, i);
        fid.insert(fid.end(), q.nf, i);
        const int64_t n = (int64_t)q.nf * q.nb;
        dof_inst.insert(dof_inst.end(), n, i);
        const int lteam = batch_team(q.nb, q.S);
        for (int f = 0; f < q.nf; f += 256 >> lteam) fblk.push_back({i, f, lteam, 0});
        ib0[i] = (int32_t)blk_inst.size();
        for (int64_t k = 0; k < n; k += SEG_CHUNK) {
            blk_inst.push_back(i);
            blk_lo.push_back(q.vec_off + k);
            blk_hi.push_back(q.vec_off + std::min<int64_t>(n, k + SEG_CHUNK));
        }
        ib1[i] = (int32_t)blk_inst.size();
        b->dev.max_chunks = std::max(b->dev.max_chunks, ib1[i] - ib0[i]);
        b->dev.max_nb = std::max(b->dev.max_nb, q.nb);
        b->dev.max_R = std::max(b->dev.max_R, q.R);
    }
    hipError_t err = hipSetDevice(ctx->device);
    BatchDev& dv = b->dev;
    dv.n_inst = n_inst;
    dv.total_ne = e0;
    dv.total_nf = f0;
    dv.total_dof = b->offs[A_VEC][n_inst];
    dv.nblk = (int)blk_inst.size();
    dv.max_cond_lds = max_cond;
    dv.tiles = tile_work > 0.0;
    dv.max_rec_lds = max_rec;
    if (err == hipSuccess) dv.desc = dev_upload(b, b->host, &err);
    if (err == hipSuccess) dv.eid = dev_upload(b, eid, &err);
    if (err == hipSuccess) dv.fid = dev_upload(b, fid, &err);
    dv.nfblk = (int)fblk.size();
    if (err == hipSuccess) dv.fblk = dev_upload(b, fblk, &err);
    if (err == hipSuccess) dv.dof_inst = dev_upload(b, dof_inst, &err);
    if (err == hipSuccess) dv.blk_inst = dev_upload(b, blk_inst, &err);
    if (err == hipSuccess) dv.blk_lo = dev_upload(b, blk_lo, &err);
    if (err == hipSuccess) dv.blk_hi = dev_upload(b, blk_hi, &err);
    if (err == hipSuccess) dv.ib0 = dev_upload(b, ib0, &err);
    if (err == hipSuccess) dv.ib1 = dev_upload(b, ib1, &err);
    if (err != hipSuccess) {
        ctx->err = std::string("hdg_batch_create: ") + hipGetErrorString(err);
        for (void* p : b->allocs) (void)hipFree(p);
        delete b;
        return HDG_ERR_HIP;
    }
    *out = b;
    return HDG_OK;
}

hdg_status hdg_batch_destroy(hdg_batch b) {
    if (!b) return HDG_ERR_ARG;
    (void)hipSetDevice(b->device);
    (void)hipDeviceSynchronize();
    for (void* p : b->allocs) (void)hipFree(p);
    delete b;
    return HDG_OK;
}

hdg_status hdg_batch_offsets(hdg_batch b, int32_t array_id, int64_t* off_h) {
    if (!b || !off_h || array_id < 0 || array_id >= A_NARR) return HDG_ERR_ARG;
    std::memcpy(off_h, b->offs[array_id].data(), sizeof(int64_t) * b->offs[array_id].size());
    return HDG_OK;
}

int32_t hdg_batch_tuned_grid(hdg_batch b) { return b ? b->tuned_grid : 0; }

hdg_status hdg_element_blocks_batch(hdg_ctx ctx, hdg_batch b, const int32_t* nqv_h, const int32_t* nqf_h,
                                    const hdg_elem_geom* g, const hdg_conv_diff* models_h, const double* c_h,
                                    const double* u_prev, const double* r_extra, const int32_t* e2f,
                                    const double* u, const double* uhat, int32_t flags,
                                    const hdg_elem_arrays* out) {
    if (!ctx || !b) return HDG_ERR_ARG;
    if (!nqv_h || !nqf_h || !g || !models_h || !e2f || !u || !uhat || !out || !out->ru || !out->rt || !g->wdet ||
        !g->dphix || !g->phi || !g->phif || !g->psi || !g->ndA || !g->dA || !g->src || !g->uD || !g->bnd) {
        ctx->err = "hdg_element_blocks_batch: NULL pointer";
        return HDG_ERR_ARG;
    }
    const bool residual_only = (flags & HDG_ELEM_RESIDUAL_ONLY) != 0;
    if ((flags & ~(HDG_ELEM_RESIDUAL_ONLY | HDG_ELEM_KEEP_MASS)) ||
        ((flags & HDG_ELEM_KEEP_MASS) && !out->Minv)) {
        ctx->err = "hdg_element_blocks_batch: unknown flags, or HDG_ELEM_KEEP_MASS without the kept Minv";
        return HDG_ERR_ARG;
    }
    if (!residual_only && (!out->Minv || !out->Bd || !out->Cd || !out->D || !out->E || !out->F || !out->G ||
                           !out->H || !out->J)) {
        ctx->err = "hdg_element_blocks_batch: NULL matrix output (residual_only = 0)";
        return HDG_ERR_ARG;
    }
    const int n = b->dev.n_inst;
    std::vector<ElemInst> inst(n);
    int64_t gw = 0, gdp = 0, gph = 0, gpf = 0, gps = 0, gn = 0, gda = 0, gs = 0, gud = 0;
    size_t lds = 0;
    for (int i = 0; i < n; ++i) {
        const InstDesc& q = b->host[i];
        const int Qv = nqv_h[i], Qf = nqf_h[i];
        if (q.M != 1 || Qv < 1 || Qf < 1) {
            ctx->err = "hdg_element_blocks_batch: instance " + std::to_string(i) +
                       " is not a scalar model with nqv, nqf >= 1";
            return HDG_ERR_ARG;
        }
        const size_t li = element_batch_lds_bytes(q.P, q.PF, q.L, q.D, Qv, Qf);
        if (li > 65536) {
            ctx->err = "hdg_element_blocks_batch: element data of instance " + std::to_string(i) +
                       " exceed 64 KiB of LDS";
            return HDG_ERR_SHAPE;
        }
        lds = std::max(lds, li);
        const double nu_ = models_h[i].nu, tau_ = models_h[i].tau;
        ElemInst& E = inst[i];
        E.P = q.P; E.PF = q.PF; E.L = q.L; E.D = q.D; E.Qv = Qv; E.Qf = Qf;
        E.e0 = q.e0;
        E.g_wdet = gw;  gw += (int64_t)q.ne * Qv;
        E.g_dphix = gdp; gdp += (int64_t)q.ne * Qv * q.P * q.D;
        E.g_phi = gph;  gph += (int64_t)Qv * q.P;
        E.g_phif = gpf; gpf += (int64_t)q.ne * q.L * Qf * q.P;
        E.g_psi = gps;  gps += (int64_t)Qf * q.PF;
        E.g_ndA = gn;   gn += (int64_t)q.ne * q.L * Qf * q.D;
        E.g_dA = gda;   gda += (int64_t)q.ne * q.L * Qf;
        E.g_src = gs;   gs += (int64_t)q.ne * Qv;
        E.g_uD = gud;   gud += (int64_t)q.ne * q.L * Qf;
        E.e2f_off = q.e2f_off;
        E.u_off = q.du_off;
        E.uh_off = q.vec_off;
        E.q_off = q.dq_off;
        for (int a = 0; a < 11; ++a) E.out_off[a] = q.off[a];
        E.nu = nu_; E.tau = tau_;
        E.c = c_h ? c_h[i] : 0.0;
        if (!std::isfinite(E.c) || (E.c != 0.0 && !u_prev)) {
            ctx->err = "hdg_element_blocks_batch: instance " + std::to_string(i) +
                       " has a non-finite time-term factor or no u_prev";
            return HDG_ERR_ARG;
        }
        for (int d = 0; d < 3; ++d) { E.beta[d] = models_h[i].beta[d]; E.gamma[d] = models_h[i].gamma[d]; }
    }
    HDG_HIP_CHECK(ctx, hipSetDevice(ctx->device));
    hdg_status st;
    char* base = (char*)ws_get(ctx, WS_NEWTON_BATCH, sizeof(ElemInst) * (size_t)n + 2 * sizeof(double) * n + 256,
                               &st);
    if (!base) return st;
    int* status = (int*)ws_get(ctx, WS_STATUS, 64, &st);
    if (!status) return st;
    const int big = 0x7fffffff;
    HDG_HIP_CHECK(ctx, hipMemcpyAsync(status, &big, sizeof(int), hipMemcpyHostToDevice, ctx->stream));
    HDG_HIP_CHECK(ctx, hipMemcpyAsync(base, inst.data(), sizeof(ElemInst) * (size_t)n, hipMemcpyHostToDevice,
                                      ctx->stream));
    ElemBatchArgs a;
    a.g = *g;
    a.e2f = e2f;
    a.u = u;
    a.uhat = uhat;
    a.u_prev = u_prev;
    a.r_extra = r_extra;
    a.out = *out;
    a.bad = status;
    a.residual_only = residual_only ? 1 : 0;
    a.keep_mass = (flags & HDG_ELEM_KEEP_MASS) ? 1 : 0;
    if (lds > 64 * 1024) lds = 64 * 1024;
    if ((st = element_blocks_batch_run(ctx, b->dev.total_ne, (const ElemInst*)base, b->dev.eid, a, lds)) != HDG_OK)
        return st;
    int bad = big;
    HDG_HIP_CHECK(ctx, hipMemcpyAsync(&bad, status, sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
    HDG_HIP_CHECK(ctx, hipStreamSynchronize(ctx->stream));
    if (bad != big) {
        ctx->err = "hdg_element_blocks_batch: non-positive mass-matrix pivot in (global) element " +
                   std::to_string(bad);
        return HDG_ERR_SINGULAR;
    }
    return HDG_OK;
}

hdg_status hdg_residual_norm_batch(hdg_ctx ctx, hdg_batch b, const int32_t* f2e, const double* ru, const double* rt,
                                   double* norms_h) {
    if (!ctx || !b) return HDG_ERR_ARG;
    if (!f2e || !ru || !rt || !norms_h) {
        ctx->err = "hdg_residual_norm_batch: NULL pointer";
        return HDG_ERR_ARG;
    }
    const int n = b->dev.n_inst;
    HDG_HIP_CHECK(ctx, hipSetDevice(ctx->device));
    hdg_status st;
    char* base = (char*)ws_get(ctx, WS_NEWTON_BATCH, sizeof(ElemInst) * (size_t)n + 2 * sizeof(double) * n + 256,
                               &st);
    if (!base) return st;
    double* norms = (double*)(base + sizeof(ElemInst) * (size_t)n);
    if ((st = residual_norm_batch_run(ctx, n, b->dev.desc, ru, rt, f2e, norms)) != HDG_OK) return st;
    HDG_HIP_CHECK(ctx, hipMemcpyAsync(norms_h, norms, sizeof(double) * n, hipMemcpyDeviceToHost, ctx->stream));
    HDG_HIP_CHECK(ctx, hipStreamSynchronize(ctx->stream));
    return HDG_OK;
}

hdg_status hdg_newton_update_batch(hdg_ctx ctx, hdg_batch b, const double* alpha_h, const double* du, double* u,
                                   const double* x, double* uhat) {
    if (!ctx || !b) return HDG_ERR_ARG;
    if (!alpha_h || !du || !u || !x || !uhat) {
        ctx->err = "hdg_newton_update_batch: NULL pointer";
        return HDG_ERR_ARG;
    }
    const int n = b->dev.n_inst;
    HDG_HIP_CHECK(ctx, hipSetDevice(ctx->device));
    hdg_status st;
    char* base = (char*)ws_get(ctx, WS_NEWTON_BATCH, sizeof(ElemInst) * (size_t)n + 2 * sizeof(double) * n + 256,
                               &st);
    if (!base) return st;
    double* alpha = (double*)(base + sizeof(ElemInst) * (size_t)n) + n;
    HDG_HIP_CHECK(ctx, hipMemcpyAsync(alpha, alpha_h, sizeof(double) * n, hipMemcpyHostToDevice, ctx->stream));
    if ((st = newton_update_batch_run(ctx, n, b->dev.desc, alpha, du, u, x, uhat)) != HDG_OK) return st;
    // the host array is read by the copy above: keep the call synchronous for the caller
    HDG_HIP_CHECK(ctx, hipStreamSynchronize(ctx->stream));
    return HDG_OK;
}

hdg_status hdg_condense_batch(hdg_ctx ctx, hdg_batch b, const hdg_elem_blocks* in, double* Kbar, double* rbar,
                              double* local) {
    if (!ctx || !b) return HDG_ERR_ARG;
    if (!in || !in->Minv || !in->Bd || !in->Cd || !in->D || !in->E || !in->F || !in->G || !in->H || !in->J ||
        !in->ru || !in->rt || !Kbar || !rbar || !local) {
        ctx->err = "hdg_condense_batch: NULL pointer";
        return HDG_ERR_ARG;
    }
    HDG_HIP_CHECK(ctx, hipSetDevice(ctx->device));
    hdg_status st;
    int* status = (int*)ws_get(ctx, WS_STATUS, 64, &st);
    if (!status) return st;
    const int big = 0x7fffffff;
    HDG_HIP_CHECK(ctx, hipMemcpyAsync(status, &big, sizeof(int), hipMemcpyHostToDevice, ctx->stream));
    BatchElemPtrs p{in->Minv, in->Bd, in->Cd, in->D, in->E, in->F, in->G, in->H, in->J, in->ru, in->rt};
    if (b->tuned_grid == 0) {
        // autotune the persistent grid: time each candidate once on the real data (the
        // kernel is a pure function of its inputs, so repeated runs write the same outputs)
        const int cands[5] = {256, 512, 1024, 2048, 4096};
        double best = 1e300;
        int pick = 1024;
        hipEvent_t e0, e1;
        HDG_HIP_CHECK(ctx, hipEventCreate(&e0));
        HDG_HIP_CHECK(ctx, hipEventCreate(&e1));
        for (int c : cands) {
            const int grid = (int)std::min<int64_t>(c, b->dev.total_ne);
            HDG_HIP_CHECK(ctx, hipEventRecord(e0, ctx->stream));
            if ((st = batch_launch_condense(ctx, b->dev, p, Kbar, rbar, local, status, grid)) != HDG_OK) return st;
            HDG_HIP_CHECK(ctx, hipEventRecord(e1, ctx->stream));
            HDG_HIP_CHECK(ctx, hipEventSynchronize(e1));
            float ms = 0.f;
            HDG_HIP_CHECK(ctx, hipEventElapsedTime(&ms, e0, e1));
            if (ms < best) { best = ms; pick = grid; }
            if (grid == b->dev.total_ne) break;
        }
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        b->tuned_grid = pick;
    } else {
        if ((st = batch_launch_condense(ctx, b->dev, p, Kbar, rbar, local, status, b->tuned_grid)) != HDG_OK)
            return st;
    }
    int bad = big;
    HDG_HIP_CHECK(ctx, hipMemcpyAsync(&bad, status, sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
    HDG_HIP_CHECK(ctx, hipStreamSynchronize(ctx->stream));
    if (bad != big) {
        int inst = 0;
        while (inst + 1 < b->dev.n_inst && b->host[inst + 1].e0 <= bad) ++inst;
        ctx->err = "condensation: zero or non-finite pivot in Ebar of instance " + std::to_string(inst) +
                   " element " + std::to_string(bad - b->host[inst].e0);
        return HDG_ERR_SINGULAR;
    }
    return HDG_OK;
}

hdg_status hdg_assemble_batch(hdg_ctx ctx, hdg_batch b, const int32_t* f2e, const int32_t* e2f, const double* Kbar,
                              const double* rbar, double* K64, float* K32, int32_t* nbr, double* r) {
    if (!ctx || !b) return HDG_ERR_ARG;
    if (!f2e || !e2f || !Kbar || !rbar || !K64 || !nbr || !r) {
        ctx->err = "hdg_assemble_batch: NULL pointer";
        return HDG_ERR_ARG;
    }
    HDG_HIP_CHECK(ctx, hipSetDevice(ctx->device));
    return batch_launch_assemble(ctx, b->dev, f2e, e2f, Kbar, rbar, K64, K32, nbr, r);
}

hdg_status hdg_recover_batch(hdg_ctx ctx, hdg_batch b, const double* local, const double* Minv, const double* Bd,
                             const double* Cd, const int32_t* e2f, const double* xhat, double* du, double* dq) {
    if (!ctx || !b) return HDG_ERR_ARG;
    if (!local || !Minv || !Bd || !Cd || !e2f || !xhat || !du || !dq) {
        ctx->err = "hdg_recover_batch: NULL pointer";
        return HDG_ERR_ARG;
    }
    HDG_HIP_CHECK(ctx, hipSetDevice(ctx->device));
    return batch_launch_recover(ctx, b->dev, local, Minv, Bd, Cd, e2f, xhat, du, dq);
}

hdg_status hdg_gmres_solve_batch(hdg_ctx ctx, hdg_batch b, const double* K64, const float* K32, const int32_t* nbr,
                                 const double* rhs, double* x, const hdg_solve_opts* o, hdg_solve_stats* stats) {
    if (!ctx || !b) return HDG_ERR_ARG;
    if (!o || !stats || !K64 || !nbr || !rhs || !x) {
        ctx->err = "hdg_gmres_solve_batch: NULL pointer";
        return HDG_ERR_ARG;
    }
    if (o->restart < 1 || o->restart > 200 || o->max_iters < 0 || !(o->rtol >= 0.0) || !(o->atol >= 0.0)) {
        ctx->err = "hdg_gmres_solve_batch: bad restart/max_iters/rtol/atol";
        return HDG_ERR_ARG;
    }
    if (o->prec != HDG_PREC_NONE && o->prec != HDG_PREC_BJ) {
        ctx->err = "hdg_gmres_solve_batch: only HDG_PREC_NONE and HDG_PREC_BJ are batched";
        return HDG_ERR_ARG;
    }
    if (o->orth != HDG_ORTH_CGS2 && o->orth != HDG_ORTH_CGS) {
        ctx->err = "hdg_gmres_solve_batch: orth must be CGS2 or CGS";
        return HDG_ERR_ARG;
    }
    const bool mixed = o->precision == HDG_MIXED;
    if (o->precision != HDG_FP64 && !mixed) return HDG_ERR_ARG;
    if (mixed && !K32) {
        ctx->err = "mixed precision needs K32";
        return HDG_ERR_ARG;
    }
    HDG_HIP_CHECK(ctx, hipSetDevice(ctx->device));
    const double t0 = now_s();
    CaptureStreamScope cap;
    if (o->use_graph) HDG_HIP_CHECK(ctx, cap.begin(ctx));
    const BatchDev& dv = b->dev;
    const int ni = dv.n_inst, m = o->restart, ldh = m + 1, ldg = m + 2;
    const size_t N = (size_t)dv.total_dof;
    const size_t ld = (N + 63) / 64 * 64;
    hdg_status st;
    double* V = (double*)ws_get(ctx, WS_KRYLOV_V, sizeof(double) * ld * (m + 1), &st);
    if (!V) return st;
    double* Z = (double*)ws_get(ctx, WS_KRYLOV_Z, sizeof(double) * ld * m, &st);
    if (!Z) return st;
    double* part = (double*)ws_get(ctx, WS_PART, sizeof(double) * (size_t)dv.nblk * (m + 1) * 2, &st);
    if (!part) return st;
    double* part2 = part + (size_t)dv.nblk * (m + 1);     // a sweep reads the partials of the one before
    const size_t nctl = (size_t)ni * ((size_t)ldh * m + 6 * (size_t)ldg + 2);
    char* base = (char*)ws_get(ctx, WS_CTL, sizeof(BatchCtl) * ni + sizeof(double) * nctl, &st);
    if (!base) return st;
    BatchCtl* ctl = (BatchCtl*)base;
    double* H = (double*)(base + sizeof(BatchCtl) * ni);
    double* cs = H + (size_t)ni * ldh * m;
    double* sn = cs + (size_t)ni * ldg;
    double* g = sn + (size_t)ni * ldg;
    double* y = g + (size_t)ni * ldg;
    double* bn = y + (size_t)ni * ldg;       // ||b||^2 per instance
    double* coef = bn + (size_t)ni * ldg;
    double* target = coef + (size_t)ni * ldg;   // per-instance absolute target
    const void* Kop = mixed ? (const void*)K32 : (const void*)K64;
    const void* Bop = nullptr;
    double* B64 = nullptr;
    float* B32 = nullptr;
    if (o->prec == HDG_PREC_BJ) {
        const int64_t nbinv = b->offs[A_BINV][ni];
        ctx->bj_key.valid = false;   // the batch's inverses go to the same workspace
        B64 = (double*)ws_get(ctx, WS_BINV64, sizeof(double) * nbinv, &st);
        if (!B64) return st;
        if (mixed) {
            B32 = (float*)ws_get(ctx, WS_BINV32, sizeof(float) * nbinv, &st);
            if (!B32) return st;
        }
        int* status = (int*)ws_get(ctx, WS_STATUS, 64, &st);
        if (!status) return st;
        const int big = 0x7fffffff;
        HDG_HIP_CHECK(ctx, hipMemcpyAsync(status, &big, sizeof(int), hipMemcpyHostToDevice, ctx->stream));
        if ((st = batch_launch_bj(ctx, dv, K64, B64, B32, status)) != HDG_OK) return st;
        int bad = big;
        HDG_HIP_CHECK(ctx, hipMemcpyAsync(&bad, status, sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
        HDG_HIP_CHECK(ctx, hipStreamSynchronize(ctx->stream));
        if (bad != big) {
            ctx->err = "block-Jacobi: singular diagonal block of face " + std::to_string(bad) + " (batch index)";
            return HDG_ERR_SINGULAR;
        }
        Bop = mixed ? (const void*)B32 : (const void*)B64;
    }
    // per-instance ||b||
    if ((st = seg_sumsq(ctx, dv, rhs, part, nullptr)) != HDG_OK) return st;
    if ((st = seg_reduce(ctx, dv, part, bn, ldg)) != HDG_OK) return st;
    std::vector<double> bn_h((size_t)ni * ldg), tg_h((size_t)ni * ldg, 0.0);
    HDG_HIP_CHECK(ctx, hipMemcpyAsync(bn_h.data(), bn, sizeof(double) * bn_h.size(), hipMemcpyDeviceToHost,
                                      ctx->stream));
    HDG_HIP_CHECK(ctx, hipStreamSynchronize(ctx->stream));
    std::vector<double> bnorm(ni);
    for (int i = 0; i < ni; ++i) {
        bnorm[i] = std::sqrt(bn_h[(size_t)i * ldg]);
        if (!std::isfinite(bnorm[i])) {
            ctx->err = "right-hand side of instance " + std::to_string(i) + " contains NaN or Inf";
            return HDG_ERR_NONFINITE;
        }
        tg_h[i] = std::max(o->rtol * bnorm[i], o->atol);
    }
    HDG_HIP_CHECK(ctx, hipMemcpy(target, tg_h.data(), sizeof(double) * ni, hipMemcpyHostToDevice));
    for (int i = 0; i < ni; ++i) std::memset(&stats[i], 0, sizeof(hdg_solve_stats));
    const int ld_beta = (int)(sizeof(BatchCtl) / sizeof(double));
    auto enqueue_cycle = [&](int jmax) -> hdg_status {
        hdg_status s2;
        if ((s2 = batch_launch_face(ctx, dv, K64, false, nbr, false, x, V, -1.0, rhs, 1.0, nullptr, 0, nullptr)) != HDG_OK)
            return s2;
        if ((s2 = seg_sumsq(ctx, dv, V, part, nullptr)) != HDG_OK) return s2;
        if ((s2 = seg_cycle_init(ctx, dv, part, ctl, g, ldg, jmax, target)) != HDG_OK) return s2;
        for (int j = 0; j < jmax; ++j) {
            double* vj = V + (size_t)j * ld;
            double* zj = Z + (size_t)j * ld;
            double* wv = V + (size_t)(j + 1) * ld;
            double* col = H + (size_t)j * ldh;
            // v_j arrives not yet normalised: its norm is beta or the last column's subdiagonal entry
            const double* denom = j == 0 ? &ctl[0].beta : col - ldh + j;
            const int ld_denom = j == 0 ? ld_beta : ldh * m;
            if (Bop) {
                if ((s2 = batch_launch_face(ctx, dv, Bop, mixed, nullptr, true, vj, zj, 1.0, nullptr, 0.0, denom, ld_denom,
                                            ctl)) != HDG_OK)
                    return s2;
            } else {
                if ((s2 = seg_scale(ctx, dv, vj, denom, ld_denom, ctl)) != HDG_OK) return s2;
                if ((s2 = vec_lincomb(ctx, N, zj, 1.0, vj, 0.0, nullptr, nullptr)) != HDG_OK) return s2;
            }
            if ((s2 = batch_launch_face(ctx, dv, Kop, mixed, nbr, false, zj, wv, 1.0, nullptr, 0.0, nullptr, 0, ctl)) !=
                HDG_OK)
                return s2;
            SegSweep sw{};
            sw.V = V; sw.ldv = ld; sw.J = j + 1; sw.w = wv; sw.part_out = part;
            sw.col = col; sw.ld_col = ldh * m; sw.ctl = ctl;
            sw.coef = coef; sw.ld_coef = ldg;
            if ((s2 = seg_sweep(ctx, dv, sw, false, true)) != HDG_OK) return s2;
            if (o->orth == HDG_ORTH_CGS2) {
                sw.part_in = part; sw.part_out = part2;
                if ((s2 = seg_sweep(ctx, dv, sw, true, true)) != HDG_OK) return s2;
                sw.add = 1;
            }
            sw.part_in = sw.part_out;
            sw.part_out = sw.part_in == part ? part2 : part;
            if ((s2 = seg_sweep(ctx, dv, sw, true, false)) != HDG_OK) return s2;
            if ((s2 = seg_givens(ctx, dv, sw.part_out, ctl, H, ldh, m, cs, sn, g, ldg, j, jmax, target)) != HDG_OK) return s2;
        }
        if ((s2 = seg_backsolve(ctx, dv, ctl, H, ldh, m, g, ldg, y)) != HDG_OK) return s2;
        return seg_update(ctx, dv, Z, ld, y, ldg, x, ctl);
    };
    hipGraph_t graph = nullptr;
    hipGraphExec_t gexec = nullptr;
    auto drop_graph = [&]() {
        if (gexec) (void)hipGraphExecDestroy(gexec);
        if (graph) (void)hipGraphDestroy(graph);
        gexec = nullptr;
        graph = nullptr;
    };
    std::vector<BatchCtl> hc(ni);
    // stagnation: an instance whose inner estimate met its target at every restart while its
    // true residual stayed above the target and above 0.9 times the best true residual it had
    // shown, five cycles in a row, has reached the accuracy its FP64 residual can show; it
    // stops (not converged, flagged)
    std::vector<double> best_beta(ni, INFINITY), prev_est(ni, INFINITY);
    std::vector<int> stalls(ni, 0);
    int iters = 0;
    hdg_status result = HDG_NOT_CONVERGED;
    while (true) {
        const int jmax = std::max(0, std::min(m, o->max_iters - iters));
        if (o->use_graph && jmax == m) {
            if (!gexec) {
                HDG_HIP_CHECK(ctx, hipStreamBeginCapture(ctx->stream, hipStreamCaptureModeThreadLocal));
                st = enqueue_cycle(jmax);
                hipGraph_t gr = nullptr;
                const hipError_t ec = hipStreamEndCapture(ctx->stream, &gr);
                if (st != HDG_OK) { if (gr) (void)hipGraphDestroy(gr); return st; }
                if (ec != hipSuccess) {
                    ctx->err = std::string("graph capture failed: ") + hipGetErrorString(ec);
                    return HDG_ERR_HIP;
                }
                graph = gr;
                if (hipGraphInstantiate(&gexec, graph, nullptr, nullptr, 0) != hipSuccess) {
                    drop_graph();
                    ctx->err = "graph instantiation failed";
                    return HDG_ERR_HIP;
                }
            }
            if (hipGraphLaunch(gexec, ctx->stream) != hipSuccess) {
                drop_graph();
                ctx->err = "graph launch failed";
                return HDG_ERR_HIP;
            }
        } else if ((st = enqueue_cycle(jmax)) != HDG_OK) {
            drop_graph();
            return st;
        }
        const hipError_t e1 = hipMemcpyAsync(hc.data(), ctl, sizeof(BatchCtl) * ni, hipMemcpyDeviceToHost, ctx->stream);
        const hipError_t e2 = hipStreamSynchronize(ctx->stream);
        if (e1 != hipSuccess || e2 != hipSuccess) {
            drop_graph();
            ctx->err = "reading the batched GMRES status failed";
            return HDG_ERR_HIP;
        }
        bool any_active = false, bad = false;
        for (int i = 0; i < ni; ++i) {
            stats[i].rel_resid_true = bnorm[i] > 0 ? hc[i].beta / bnorm[i] : 0.0;
            if (hc[i].nonfinite) bad = true;
            if (hc[i].k > 0) {
                stats[i].iters += hc[i].k;
                stats[i].cycles += 1;
                stats[i].rel_resid_est = bnorm[i] > 0 ? hc[i].est / bnorm[i] : 0.0;
                any_active = true;
            }
        }
        iters += any_active ? m : 0;
        for (int i = 0; i < ni; ++i) {
            if (hc[i].k == 0) continue;
            const bool stall = prev_est[i] <= tg_h[i] && hc[i].beta > tg_h[i] && hc[i].beta > 0.9 * best_beta[i];
            stalls[i] = stall ? stalls[i] + 1 : 0;
            best_beta[i] = std::min(best_beta[i], hc[i].beta);
            prev_est[i] = hc[i].est;
            if (stalls[i] >= 5) {
                stats[i].fallback_flags |= HDG_FALLBACK_STAGNATED;
                const double stop = INFINITY;     // the next cycle's start marks it done
                HDG_HIP_CHECK(ctx, hipMemcpyAsync(target + i, &stop, sizeof(double), hipMemcpyHostToDevice,
                                                  ctx->stream));
                HDG_HIP_CHECK(ctx, hipStreamSynchronize(ctx->stream));
            }
        }
        if (bad) {
            ctx->err = "batched solve: residual or Arnoldi data became NaN or Inf";
            result = HDG_ERR_NONFINITE;
            break;
        }
        if (!any_active) {
            bool all = true;
            for (int i = 0; i < ni; ++i) {
                stats[i].converged = hc[i].beta <= tg_h[i];
                all = all && stats[i].converged;
            }
            result = all ? HDG_OK : HDG_NOT_CONVERGED;
            break;
        }
    }
    drop_graph();
    const double t1 = now_s();
    for (int i = 0; i < ni; ++i) stats[i].t_total = t1 - t0;
    return result;
}

}  // extern "C"
