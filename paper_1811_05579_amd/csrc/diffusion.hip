// diffusion.hip -- the discrete nonlinear diffusion limit on the GPU (the
// grte_diff_* calls of include/grte.h): the three-stage prediction-
// correction-projection scheme (2.7) of Tang, Wang & Zhang, its sigma/T^3
// form (2.9), and the two-stage scheme (2.8) that the paper gives as the
// counter-example (a compactly supported temperature never spreads).
//
// One step of a slab of N <= 4096 cells is one work-group, up to 1024 threads of one
// to four cells:
//   stage 1   (U* - U^n)/dt = 4 T^3/(4 a T^3 + Cv) (1/dx^2)[F_{j+1}(U*_{j+1} - U*_j) - F_j(U*_j - U*_{j-1})]
//             with face coefficients F = a c K/(3 sigma) (harmonic sigma, mean K = T^m),
//             one tridiagonal solve (tri_wg);
//   stage 2   a (T^4 - U^n)/dt + Cv (T - T^n)/dt = the same flux difference of U*, one
//             scalar Newton per cell (F from K^n, or from (U*)^{3/4} for the printed (2.9));
//   stage 3   U^{n+1} = (T^{n+1})^4 (the state is T).
// The two-stage scheme replaces stages 2-3 by T^{n+1} = max(U*, 0)^{1/4}; the
// limit of the alternative correction (3.14) (the remark closing Section 3)
// replaces stage 2 by the linear update
//   a (U* - U^n)/dt + Cv (T^{n+1} - T^n)/dt = the flux difference of U* (F from K^n).
// Boundaries: zero flux, or ghost temperatures one cell outside the slab with
// the boundary cell's coefficient on the boundary face.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdio>
#include <new>

#include "../../include/grte.h"
#include "solver_common.hpp"

namespace {

struct DiffArgs {
    int N, m, bc, scheme, corrK, maxit;
    double a, at, c, cv, dt;
    double rdx, rcv, rat;             // 1 / dx, 1 / cv, 1 / at
    double gUL, gUR;                  // ghost U = T^4 outside the two ends (Dirichlet)
    const double *T, *sigma0;
    double *Tout, *Ustar;
    int *stat;                        // [0] max Newton iterations, [1] cells at the cap
};

__device__ __forceinline__ double dkpow(double T, int m) { return m == 0 ? 1.0 : T * T * T; }

// a c K/(3 sigma) at interior face i (between cells i-1 and i), sigma = 2 sl sr/(sl + sr)
__device__ __forceinline__ double face_F(const DiffArgs &A, double Kl, double Kr, int i)
{
    const double sl = A.sigma0[i - 1], sr = A.sigma0[i];
    return A.a * A.c * (Kl + Kr) * (sl + sr) / (12.0 * sl * sr);
}

constexpr int DIFF_MAX_N = 4096;      // largest slab: 16 wavefronts, four cells per thread

// One step.  Bound: one chain of dependent operations on one compute unit (loads, two face
// coefficients, the solve, the Newton iterations), hence no division that a product can
// replace and the thread's Newton loops in one.  1000 cells on an MI355X: 8.7 us per step;
// four cells in each of 256 threads, a cyclic reduction through LDS and the cells' Newton
// loops one after the other took 16.6, with clearing the counters as a launch of its own.
template <int NW, int M>
__global__ void __launch_bounds__(64 * NW) diff_kernel(DiffArgs A)
{
    constexpr int NTH = 64 * NW;
    __shared__ double sU[NTH * M];
    __shared__ int sStat[2][NW];
    const int k = threadIdx.x, j0 = k * M;
    const int N = A.N;
    const double rdx = A.rdx, rdx2 = rdx * rdx;
    // stage 1: tridiagonal system for U*
    double lo[M], up[M], b[M], x[M], Tn[M];
    double Fl[M], Fr[M];              // face coefficients from K^n (left/right face of the row)
#pragma unroll
    for (int r = 0; r < M; ++r) {
        const int j = j0 + r;
        Fl[r] = Fr[r] = Tn[r] = 0.0;
        lo[r] = up[r] = 0.0;
        b[r] = 1.0;
        x[r] = 0.0;
        if (j < N) {
            const double Tj = A.T[j];
            Tn[r] = Tj;
            const double Kj = dkpow(Tj, A.m);
            double fl = 0.0, fr = 0.0;
            if (j >= 1) fl = face_F(A, dkpow(A.T[j - 1], A.m), Kj, j);
            else if (A.bc == 1) fl = A.a * A.c * Kj / (3.0 * A.sigma0[0]);
            if (j <= N - 2) fr = face_F(A, Kj, dkpow(A.T[j + 1], A.m), j + 1);
            else if (A.bc == 1) fr = A.a * A.c * Kj / (3.0 * A.sigma0[N - 1]);
            Fl[r] = fl;
            Fr[r] = fr;
            const double T3 = Tj * Tj * Tj;
            const double den = fmin(4.0 * A.at * T3 + A.cv, DBL_MAX);   // (rcp64 of an infinity is NaN)
            const double pref = A.dt * 4.0 * T3 * rcp64(den);
            // interior faces couple to the neighbour; ghost faces move to the right-hand side
            const double wl = (j >= 1) ? fl * rdx2 : 0.0, wr = (j <= N - 2) ? fr * rdx2 : 0.0;
            const double gl = (j == 0 && A.bc == 1) ? fl * rdx2 : 0.0;
            const double gr = (j == N - 1 && A.bc == 1) ? fr * rdx2 : 0.0;
            lo[r] = -pref * wl;
            up[r] = -pref * wr;
            b[r] = 1.0 + pref * (wl + wr + gl + gr);
            x[r] = (Tj * Tj) * (Tj * Tj) + pref * (gl * A.gUL + gr * A.gUR);
        }
    }
    tri_wg<NW, M>(lo, b, up, x);
    // a value per row through LDS, and the two neighbours' back (the row's own beyond an end)
    auto neighbours = [&](const double (&v)[M], double (&vl)[M], double (&vr)[M]) {
#pragma unroll
        for (int r = 0; r < M; ++r) sU[r * NTH + k] = v[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < M; ++r) {
            vl[r] = r > 0 ? v[r > 0 ? r - 1 : 0] : k > 0 ? sU[(M - 1) * NTH + k - 1] : v[0];
            vr[r] = r < M - 1 ? v[r < M - 1 ? r + 1 : 0] : k < NTH - 1 ? sU[k + 1] : v[M - 1];
        }
    };
    double Ul[M], Ur[M], rhs[M], T[M];
    neighbours(x, Ul, Ur);
    if (A.scheme != 1 && A.m == 3 && A.corrK == 1) {
        // the printed (2.9): F from (U*)^{3/4} in stage 2
        double K[M], Kl[M], Kr[M];
#pragma unroll
        for (int r = 0; r < M; ++r) {
            const double q = sqrt(fmax(x[r], 0.0));
            K[r] = q * sqrt(q);
        }
        __syncthreads();
        neighbours(K, Kl, Kr);
#pragma unroll
        for (int r = 0; r < M; ++r) {
            const int j = j0 + r;
            double fl = 0.0, fr = 0.0;
            if (j < N) {
                if (j >= 1) fl = face_F(A, Kl[r], K[r], j);
                else if (A.bc == 1) fl = A.a * A.c * K[r] / (3.0 * A.sigma0[0]);
                if (j <= N - 2) fr = face_F(A, K[r], Kr[r], j + 1);
                else if (A.bc == 1) fr = A.a * A.c * K[r] / (3.0 * A.sigma0[N - 1]);
            }
            Fl[r] = fl;
            Fr[r] = fr;
        }
    }
    int nits = 0, nfail = 0;
    if (A.scheme == 1) {
#pragma unroll
        for (int r = 0; r < M; ++r) T[r] = sqrt(sqrt(fmax(x[r], 0.0)));   // (2.8): projection of U* only
    } else {
        // stage 2: flux difference of U*
        bool newton = false;
#pragma unroll
        for (int r = 0; r < M; ++r) {
            const int j = j0 + r;
            const double us = x[r], Tj = Tn[r], fl = Fl[r], fr = Fr[r];
            double fluxl = 0.0, fluxr = 0.0;                 // +x fluxes through the two faces
            if (j >= 1) fluxl = fl * (us - Ul[r]) * rdx;
            else if (A.bc == 1) fluxl = fl * (us - A.gUL) * rdx;
            if (j <= N - 2) fluxr = fr * (Ur[r] - us) * rdx;
            else if (A.bc == 1) fluxr = fr * (A.gUR - us) * rdx;
            rhs[r] = A.dt * (fluxr - fluxl) * rdx + A.at * (Tj * Tj) * (Tj * Tj) + A.cv * Tj;
            if (A.scheme == 2) {
                // (3.14): no nonlinear solve, U* in the time derivative
                T[r] = Tj + (A.dt * (fluxr - fluxl) * rdx - A.at * (us - (Tj * Tj) * (Tj * Tj))) * A.rcv;
            } else if (A.at == 0.0) {
                T[r] = rhs[r] * A.rcv;
            } else {
                // a_t T^4 + Cv T = rhs: convex and increasing for T >= 0; Newton from a start
                // at or above the root converges monotonically
                T[r] = fmax(fmax(Tj, 0.0), fmax(rhs[r] * A.rcv, sqrt(sqrt(fmax(rhs[r], 0.0) * A.rat))));
                newton = true;
            }
        }
        if (newton) {
            // the thread's cells together: a cell that has converged keeps its value
            bool open[M];
            bool any = false;
#pragma unroll
            for (int r = 0; r < M; ++r) {
                open[r] = j0 + r < N;
                any |= open[r];
            }
            int its = 0;
            while (any && its < A.maxit) {
                any = false;
                ++its;
#pragma unroll
                for (int r = 0; r < M; ++r) {
                    const double T3 = T[r] * T[r] * T[r];
                    const double step = (A.at * T3 * T[r] + A.cv * T[r] - rhs[r]) * rcp64(4.0 * A.at * T3 + A.cv);
                    T[r] = open[r] ? T[r] - step : T[r];
                    open[r] = open[r] && !(fabs(step) <= 0x1p-50 * fmax(fabs(T[r]), 1e-300));
                    any |= open[r];
                }
            }
            nits = its;
#pragma unroll
            for (int r = 0; r < M; ++r) nfail += open[r];
        }
    }
#pragma unroll
    for (int r = 0; r < M; ++r) {
        if (j0 + r < N) {
            A.Ustar[j0 + r] = x[r];
            A.Tout[j0 + r] = T[r];
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        nits = max(nits, __shfl_xor(nits, o, 64));
        nfail += __shfl_xor(nfail, o, 64);
    }
    if ((k & 63) == 0) {
        sStat[0][k >> 6] = nits;
        sStat[1][k >> 6] = nfail;
    }
    __syncthreads();
    if (k == 0) {
        for (int q = 1; q < NW; ++q) {
            nits = max(nits, sStat[0][q]);
            nfail += sStat[1][q];
        }
        A.stat[0] = nits;
        A.stat[1] = nfail;
    }
}

}  // namespace

struct grte_diff {
    int N = 0, m = 0, bc = 0;
    double L = 1, a = 1, c = 1, cv = 1, gTL = 0, gTR = 0;
    hipStream_t stream = nullptr;
    double *T = nullptr, *T2 = nullptr, *sigma0 = nullptr, *Ustar = nullptr;
    int *stat = nullptr;
};

namespace {

grte_status dcopy(grte_diff *dd, void *dst, const void *src, size_t bytes, hipMemcpyKind kind)
{
    if (hipMemcpyAsync(dst, src, bytes, kind, dd->stream) != hipSuccess) return GRTE_E_HIP;
    if (kind != hipMemcpyDeviceToDevice && hipStreamSynchronize(dd->stream) != hipSuccess) return GRTE_E_HIP;
    return GRTE_OK;
}

}  // namespace

extern "C" {

grte_status grte_diff_destroy(grte_diff *dd)
{
    if (!dd) return GRTE_OK;
    void *ps[] = {dd->T, dd->T2, dd->sigma0, dd->Ustar, dd->stat};
    for (void *p : ps)
        if (p) (void)hipFree(p);
    delete dd;
    return GRTE_OK;
}

grte_status grte_diff_create(const grte_diff_problem *pb, grte_diff **out)
{
    if (!out) return GRTE_E_INVAL;
    *out = nullptr;
    if (!pb || pb->nx < 2 || !(pb->length > 0) || !(pb->a > 0) || !(pb->c > 0) || !(pb->cv > 0) ||
        (pb->opacity_law != 0 && pb->opacity_law != 3) || (pb->boundary != 0 && pb->boundary != 1) ||
        !(pb->ghost_left >= 0) || !(pb->ghost_right >= 0))
        return GRTE_E_INVAL;
    if (pb->nx > DIFF_MAX_N) return GRTE_E_UNSUPPORTED;
    grte_diff *dd = new (std::nothrow) grte_diff();
    if (!dd) return GRTE_E_NOMEM;
    dd->N = pb->nx;
    dd->m = pb->opacity_law;
    dd->bc = pb->boundary;
    dd->L = pb->length;
    dd->a = pb->a;
    dd->c = pb->c;
    dd->cv = pb->cv;
    dd->gTL = pb->ghost_left;
    dd->gTR = pb->ghost_right;
    const size_t N = dd->N;
    if (hipMalloc((void **)&dd->T, N * sizeof(double)) != hipSuccess ||
        hipMalloc((void **)&dd->T2, N * sizeof(double)) != hipSuccess ||
        hipMalloc((void **)&dd->sigma0, N * sizeof(double)) != hipSuccess ||
        hipMalloc((void **)&dd->Ustar, N * sizeof(double)) != hipSuccess ||
        hipMalloc((void **)&dd->stat, 2 * sizeof(int)) != hipSuccess) {
        grte_diff_destroy(dd);
        return GRTE_E_NOMEM;
    }
    if (hipMemset(dd->T, 0, N * sizeof(double)) != hipSuccess || hipMemset(dd->Ustar, 0, N * sizeof(double)) != hipSuccess) {
        grte_diff_destroy(dd);
        return GRTE_E_HIP;
    }
    *out = dd;
    return GRTE_OK;
}

grte_status grte_diff_set_stream(grte_diff *dd, void *hip_stream)
{
    if (!dd) return GRTE_E_INVAL;
    dd->stream = (hipStream_t)hip_stream;
    return GRTE_OK;
}

grte_status grte_diff_set_opacity(grte_diff *dd, const double *sigma0, int on_device)
{
    if (!dd || !sigma0) return GRTE_E_INVAL;
    if (!on_device)
        for (int j = 0; j < dd->N; ++j)
            if (!(sigma0[j] > 0) || !std::isfinite(sigma0[j])) return GRTE_E_INVAL;
    return dcopy(dd, dd->sigma0, sigma0, dd->N * sizeof(double),
                 on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice);
}

grte_status grte_diff_set_state(grte_diff *dd, const double *T, int on_device)
{
    if (!dd || !T) return GRTE_E_INVAL;
    if (!on_device)
        for (int j = 0; j < dd->N; ++j)
            if (!(T[j] >= 0) || !std::isfinite(T[j])) return GRTE_E_INVAL;
    return dcopy(dd, dd->T, T, dd->N * sizeof(double), on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice);
}

grte_status grte_diff_get_state(grte_diff *dd, double *T, double *Ustar, int on_device)
{
    if (!dd) return GRTE_E_INVAL;
    const hipMemcpyKind k = on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
    grte_status s = GRTE_OK;
    if (T) s = dcopy(dd, T, dd->T, dd->N * sizeof(double), k);
    if (s == GRTE_OK && Ustar) s = dcopy(dd, Ustar, dd->Ustar, dd->N * sizeof(double), k);
    return s;
}

grte_status grte_diff_step(grte_diff *dd, double dt, int scheme, int corr_K, double a_time, int *newton_its)
{
    if (!dd || !(dt > 0) || !std::isfinite(dt) || scheme < 0 || scheme > 2 || (corr_K != 0 && corr_K != 1) ||
        !std::isfinite(a_time))
        return GRTE_E_INVAL;
    DiffArgs A{};
    A.N = dd->N;
    A.m = dd->m;
    A.bc = dd->bc;
    A.scheme = scheme;
    A.corrK = corr_K;
    A.maxit = 200;
    A.a = dd->a;
    A.at = a_time < 0 ? dd->a : a_time;
    A.c = dd->c;
    A.cv = dd->cv;
    A.dt = dt;
    A.rdx = dd->N / dd->L;
    A.rcv = 1.0 / A.cv;
    A.rat = 1.0 / A.at;
    const double gl2 = dd->gTL * dd->gTL, gr2 = dd->gTR * dd->gTR;
    A.gUL = gl2 * gl2;
    A.gUR = gr2 * gr2;
    A.T = dd->T;
    A.sigma0 = dd->sigma0;
    A.Tout = dd->T2;
    A.Ustar = dd->Ustar;
    A.stat = dd->stat;
    // Two cells per thread from four wavefronts on: each wavefront repeats the merges, each
    // thread's cells its serial part (1000 cells, 50 steps: 503 us with 16 wavefronts of one
    // cell per thread, 435 with 8 of two, 441 with 4 of four); sixteen wavefronts above 2048.
    auto launch = [&](auto nw, auto rows) {
        hipLaunchKernelGGL((diff_kernel<nw.v, rows.v>), dim3(1), dim3(64 * nw.v), 0, dd->stream, A);
    };
    if (dd->N <= 256) launch(Int<4>(), Int<1>());
    else if (dd->N <= 1024) launch(Int<8>(), Int<2>());
    else if (dd->N <= 2048) launch(Int<8>(), Int<4>());
    else launch(Int<16>(), Int<4>());
    if (hipGetLastError() != hipSuccess) return GRTE_E_HIP;
    std::swap(dd->T, dd->T2);
    if (!newton_its) return GRTE_OK;
    int h[2];
    if (hipMemcpyAsync(h, dd->stat, sizeof(h), hipMemcpyDeviceToHost, dd->stream) != hipSuccess ||
        hipStreamSynchronize(dd->stream) != hipSuccess)
        return GRTE_E_HIP;
    *newton_its = h[0];
    return h[1] ? GRTE_E_NOCONV : GRTE_OK;
}

}  // extern "C"
