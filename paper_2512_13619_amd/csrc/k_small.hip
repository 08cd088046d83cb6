// One restart cycle of GMRES on a small system in one workgroup (Sections 4.3-4.5): FP64 residual,
// Arnoldi steps with classical Gram-Schmidt (one pass or two), Givens rotations, back substitution
// and the update, with block-Jacobi or no preconditioner.
//
// A step of the general path is four to ten launches of 2 to 3 us each whatever the size; here a step
// is a chain of barriers in one block: 16 waves take the operator rows, the inner products by columns
// (four per wave at a time) and the updates by rows, the new vector and the rotations stay in LDS,
// and only the basis and the operator come from L2. Where it stops to pay is where one CU's share of
// the L2 bandwidth (the basis is read four times a CGS2 step, twice a CGS step) costs more than the
// launches. Time of a step (us) here and in the general path, in cycles that run their whole length (FP64,
// block-Jacobi, blocks of 4 on quads, 28 entries of K a row; blocks of 1 are further ahead):
//              CGS2, 10 columns   50          100         200         CGS, 50     100         200
//   N =  256       16.2/33.3   16.0/39.6   19.2/56.9   27.2/91.4   12.2/34.2   14.0/42.8   18.9/61.4
//   N = 1024       24.1/40.6   29.5/42.6   40.9/59.3   66.3/92.3   20.6/35.1   26.5/43.8   39.9/62.3
//   N = 1408       31.6/41.4   40.3/43.3   56.9/60.5   93.7/94.7   27.9/36.1   36.4/44.6   55.7/63.5
//   N = 1664       35.1/42.1   45.0/43.4   64.0/60.9  105.6/94.9   31.0/36.2   40.7/44.8   62.5/63.6
//   N = 1792       36.1/43.5   46.3/44.8   65.4/61.5  107.8/95.0   31.9/36.3   41.6/45.1   63.8/63.9
//   N = 1920       39.0/42.2   50.7/43.7   72.1/61.4  119.4/94.8   34.8/36.2   45.6/44.8   70.3/63.9
// and whole Newton solves of a Poisson problem (GMRES(50), CGS2): 1.6 ms here and 5.4 with 432 unknowns,
// 6.1 and 6.9 with 1440, 6.5 and 6.5 with 1680, 9.2 and 8.4 with 1920. Hence the limits of
// small_cycle_fits. (1024 threads leave a thread 128 registers; 18 are spilled.)
#include <cmath>

#include "hdg_internal.hpp"
#include "wave_ops.hpp"

namespace {

constexpr int BS = 1024, NW = BS / 64;
constexpr int NBR_LDS = 2304;

struct Shared {
    double w[SMALL_CYCLE_MAX], z[SMALL_CYCLE_MAX], red[SMALL_CYCLE_MAX];
    double h[201], cs[201], sn[201], g[202];
    double wred[NW], scal[2];
    int stop;
    int nbr[NBR_LDS];
};

// Rows of this thread: row and, for systems above BS, row + BS; grp of G shares a row's terms.
struct Rows {
    int row, grp, G, RW;
    int f[2], r[2];
};

// sum over the block; every thread gets it
__device__ __forceinline__ double block_sum(double v, Shared& s) {
    v = wave_ops::wave_sum_all(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s.wred[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) t += s.wred[i];
    return t;
}

// acc[p] = the group's part of row p of the block rows M (cols column blocks a face, S stored) times z.
template <class T>
__device__ __forceinline__ void mul_rows(const SmallCycle& a, const Rows& R, const T* __restrict__ M, int S, bool diag,
                                         const int* nbr, const double* z, double (&acc)[2]) {
    const int nb = a.nb;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        acc[p] = 0.0;
        if (R.row + p * BS >= a.N) continue;
        const int f = R.f[p];
        const int se = (!diag && S > a.L && nbr[f * S + a.L] < 0) ? a.L : S;
        const int Q = se * nb, q0 = R.grp * Q / R.G, q1 = (R.grp + 1) * Q / R.G;
        int s = q0 / nb, c = q0 - s * nb;
        const T* m = M + ((size_t)f * S * nb + q0) * nb + R.r[p];
        int base = q0 < q1 ? (diag ? f : nbr[f * S + s]) * nb : 0;
        for (int q = q0; q < q1; q += 8, m += 8 * nb) {
            T v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = m[(q + u < q1 ? u : 0) * nb];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (q + u >= q1) break;
                acc[p] += (double)v[u] * z[base + c];
                if (++c == nb && q + u + 1 < q1) {
                    c = 0;
                    ++s;
                    base = nbr[f * S + s] * nb;
                }
            }
        }
    }
}

// The groups' parts of every row added up through LDS: out[k] for the group-0 threads.
__device__ __forceinline__ void add_groups(const Rows& R, int N, double (&acc)[2], Shared& s) {
    if (R.G == 1) return;                               // N <= BS / 2: one row a thread
    __syncthreads();
    if (R.row < N) s.red[R.grp * R.RW + R.row] = acc[0];
    __syncthreads();
    if (R.grp == 0 && R.row < N) {
        double t = acc[0];
        for (int g = 1; g < R.G; ++g) t += s.red[g * R.RW + R.row];
        acc[0] = t;
    }
}

// s.h[i] = <V_i, w> for i < J, w in LDS
__device__ __forceinline__ void dots(const SmallCycle& a, int J, Shared& s) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int i = wave * 4; i < J; i += NW * 4) {
        double acc[4] = {};
        for (int k0 = lane; k0 < a.N; k0 += 256) {
            double v[4][4];
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    v[c][u] = a.V[(size_t)(i + c < J ? i + c : i) * a.ld + (k0 + 64 * u < a.N ? k0 + 64 * u : k0)];
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (k0 + 64 * u < a.N) acc[c] += v[c][u] * s.w[k0 + 64 * u];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double t = wave_ops::wave_sum_all(acc[c]);
            if (lane == 0 && i + c < J) s.h[i + c] = t;
        }
    }
}

// the group's part of sum_i B_i[k] h[i], i < J
__device__ __forceinline__ void combine(const SmallCycle& a, const Rows& R, const double* __restrict__ B, int J,
                                        const double* h, double (&acc)[2]) {
    const int i0 = R.grp * J / R.G, i1 = (R.grp + 1) * J / R.G;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        acc[p] = 0.0;
        const int k = R.row + p * BS;
        if (k >= a.N) continue;
        for (int i = i0; i < i1; i += 8) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = B[(size_t)(i + u < i1 ? i + u : i) * a.ld + k];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i + u < i1) acc[p] += v[u] * h[i + u];
        }
    }
}

template <class T>
__global__ __launch_bounds__(BS) void k_small_cycle(SmallCycle a) {
    __shared__ Shared s;
    const int tid = threadIdx.x, N = a.N, nb = a.nb, S = a.S;
    Rows R;
    R.G = 1;
    while (R.G * 2 * N <= BS && R.G < 16) R.G *= 2;
    R.RW = BS / R.G;
    R.grp = tid / R.RW;
    R.row = tid - R.grp * R.RW;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int k = R.row + p * BS < N ? R.row + p * BS : 0;
        R.f[p] = k / nb;
        R.r[p] = k - R.f[p] * nb;
    }
    const bool own = R.grp == 0;
    const int* nbr = a.nbr;
    if (a.nf * S <= NBR_LDS) {
        for (int k = tid; k < a.nf * S; k += BS) s.nbr[k] = a.nbr[k];
        nbr = s.nbr;
    }
    // r = b - K x
    for (int k = tid; k < N; k += BS) s.z[k] = a.x[k];
    __syncthreads();
    double acc[2], w[2], ss = 0.0;
    mul_rows<double>(a, R, a.K64, S, false, nbr, s.z, acc);
    add_groups(R, N, acc, s);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int k = R.row + p * BS;
        w[p] = (own && k < N) ? a.b[k] - acc[p] : 0.0;
        ss += w[p] * w[p];
    }
    const double beta = sqrt(block_sum(ss, s));
    int k_done = 0, nonfinite = !isfinite(beta);
    double est = beta;
    if (tid == 0) s.g[0] = beta;
    double scale = beta;
    bool go = !(beta <= a.target || !isfinite(beta) || a.jmax <= 0);
    long long ticks[3] = {0, 0, 0};
    for (int j = 0; go; ++j) {
        const long long t0 = wall_clock64();
        // v_j = w / its norm, z_j = M^{-1} v_j, w = K z_j
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int k = R.row + p * BS;
            if (own && k < N) {
                const double v = w[p] / scale;
                a.V[(size_t)j * a.ld + k] = v;
                s.z[k] = v;
            }
        }
        __syncthreads();
        if (a.Binv) {
            mul_rows<T>(a, R, (const T*)a.Binv, 1, true, nbr, s.z, acc);
            add_groups(R, N, acc, s);
            __syncthreads();
#pragma unroll
            for (int p = 0; p < 2; ++p)
                if (own && R.row + p * BS < N) s.z[R.row + p * BS] = acc[p];
            __syncthreads();
        }
        const long long t1 = wall_clock64();
        mul_rows<T>(a, R, (const T*)a.K, S, false, nbr, s.z, acc);
        add_groups(R, N, acc, s);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int k = R.row + p * BS;
            w[p] = acc[p];
            if (own && k < N) s.w[k] = w[p];
        }
        __syncthreads();
        const long long t2 = wall_clock64();
        // Gram-Schmidt, the coefficients of both passes summed in the Hessenberg column
        double* col = a.H + (size_t)j * a.ldh;
        ss = 0.0;
        for (int pass = 0; pass < a.passes; ++pass) {
            dots(a, j + 1, s);
            __syncthreads();
            for (int i = tid; i <= j; i += BS) col[i] = pass ? col[i] + s.h[i] : s.h[i];
            combine(a, R, a.V, j + 1, s.h, acc);
            add_groups(R, N, acc, s);
            ss = 0.0;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int k = R.row + p * BS;
                if (own && k < N) {
                    w[p] -= acc[p];
                    s.w[k] = w[p];
                    ss += w[p] * w[p];
                }
            }
            __syncthreads();
        }
        const double hn = sqrt(block_sum(ss, s));
        // the earlier rotations on the new column, the new rotation, the residual estimate
        for (int i = tid; i <= j; i += BS) s.h[i] = col[i];
        __syncthreads();
        if (tid == 0) {
            double h = s.h[0];
            for (int i = 0; i < j; ++i) {
                const double nx = s.h[i + 1];
                s.h[i] = s.cs[i] * h + s.sn[i] * nx;
                h = -s.sn[i] * h + s.cs[i] * nx;
            }
            double c = 1.0, sg = 0.0;
            if (hn != 0.0) {
                const double r = hypot(h, hn);
                c = h / r;
                sg = hn / r;
            }
            s.cs[j] = c;
            s.sn[j] = sg;
            s.h[j] = c * h + sg * hn;
            const double gj = s.g[j];
            s.g[j + 1] = -sg * gj;
            s.g[j] = c * gj;
            const double e = fabs(s.g[j + 1]);
            s.scal[0] = e;
            s.scal[1] = s.h[j];
            a.hist[j] = e;
            s.stop = e <= a.target || hn == 0.0 || j + 1 >= a.jmax || !isfinite(e);
        }
        __syncthreads();
        for (int i = tid; i <= j; i += BS) col[i] = s.h[i];
        est = s.scal[0];
        if (!isfinite(est) || !isfinite(s.scal[1])) nonfinite = 1;
        k_done = j + 1;
        scale = hn;
        go = !s.stop;
        __syncthreads();
        const long long t3 = wall_clock64();
        ticks[0] += t1 - t0;
        ticks[1] += t2 - t1;
        ticks[2] += t3 - t2;
    }
    // R y = g by columns (one wave; the next column is loaded while one is applied), then
    // x += M^{-1} V y (the preconditioner is the same in every step)
    if (k_done > 0) {
        if (tid < 64) {
            double nx[4];
            auto load = [&](int c) {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    nx[u] = (c >= 0 && tid + 64 * u <= c) ? a.H[(size_t)c * a.ldh + tid + 64 * u] : 0.0;
            };
            double y[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) y[u] = tid + 64 * u < k_done ? s.g[tid + 64 * u] : 0.0;
            load(k_done - 1);
            for (int c = k_done - 1; c >= 0; --c) {
                double r[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) r[u] = nx[u];
                load(c - 1);
                const int du = c >> 6;
                const double rd = du == 0 ? r[0] : du == 1 ? r[1] : du == 2 ? r[2] : r[3];
                const double gc = du == 0 ? y[0] : du == 1 ? y[1] : du == 2 ? y[2] : y[3];
                const double yc = wave_ops::read_lane(gc, c & 63) / wave_ops::read_lane(rd, c & 63);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (tid + 64 * u < c) y[u] -= r[u] * yc;
                    if (tid + 64 * u == c) y[u] = yc;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (tid + 64 * u < k_done) s.h[tid + 64 * u] = y[u];
        }
        __syncthreads();
        combine(a, R, a.V, k_done, s.h, acc);
        add_groups(R, N, acc, s);
        if (a.Binv) {
            __syncthreads();
#pragma unroll
            for (int p = 0; p < 2; ++p)
                if (own && R.row + p * BS < N) s.z[R.row + p * BS] = acc[p];
            __syncthreads();
            mul_rows<T>(a, R, (const T*)a.Binv, 1, true, nbr, s.z, acc);
            add_groups(R, N, acc, s);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p)
            if (own && R.row + p * BS < N) a.x[R.row + p * BS] += acc[p];
    }
    if (tid == 0) {
        GmresCtl& c = *a.ctl;
        c.done = 1;
        c.k = k_done;
        c.jmax = a.jmax;
        c.nonfinite = nonfinite;
        c.target = a.target;
        c.beta = beta;
        c.est = est;
        for (int i = 0; i < 3; ++i) c.ticks[i] = ticks[i];
    }
}

}  // namespace

hdg_status small_cycle(hdg_ctx ctx, const SmallCycle& a, bool fp32) {
    if (a.N > SMALL_CYCLE_MAX || a.jmax > 200) {
        ctx->err = "small_cycle: size above its limit";
        return HDG_ERR_ARG;
    }
    void* args[] = {(void*)&a};
    const void* k = fp32 ? (const void*)k_small_cycle<float> : (const void*)k_small_cycle<double>;
    HDG_HIP_CHECK(ctx, hipLaunchKernel(k, dim3(1), dim3(BS), args, 0, ctx->stream));
    HDG_LAUNCH_CHECK(ctx);
    return HDG_OK;
}
