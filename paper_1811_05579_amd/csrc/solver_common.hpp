// solver_common.hpp -- device building blocks shared by the single-instance
// and the batched AP-step kernels (lane exchanges, tridiagonal factor/solve in
// one work-group, block reductions, grid barrier, node relations).
#pragma once
#include <hip/hip_runtime.h>

namespace {

constexpr int NT = 256;          // threads per work-group of the tridiagonal solvers
constexpr int MAX_M = 16;        // rows per thread -> N <= NT * MAX_M = 4096
constexpr int MAX_N = NT * MAX_M;
constexpr int MAX_P = 64;
constexpr int BAR_STRIDE = 16;   // 64-bit barrier flags, one 128-byte line per work-group

// ---- lane exchanges without LDS: data-parallel moves of the two halves of a double
template <int CTRL, int ROWS = 0xf, int BANKS = 0xf>
__device__ __forceinline__ double dpp_mov(double old, double v)
{
    const long long o = __double_as_longlong(old), x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp((int)o, (int)x, CTRL, ROWS, BANKS, true);
    const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(x >> 32), CTRL, ROWS, BANKS, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double lane_at(double v, int lane)
{
    const long long x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)x, lane), hi = __builtin_amdgcn_readlane((int)(x >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
constexpr int DPP_NEXT = 0x130, DPP_PREV = 0x138;         // lane + 1, lane - 1 over the wavefront (0 past its ends)
constexpr int DPP_MIRROR = 0x140, DPP_HALF_MIRROR = 0x141, DPP_ROW_BCAST = 0x150;   // of 16 lanes; of 8; lane n of every 16 to all of them
constexpr int quad(int a, int b, int c, int d) { return a | b << 2 | c << 4 | d << 6; }

// v + the value of the lane whose number differs in bit 4 (5): a row (half) of the
// wavefront swapped with its own neighbour leaves the lower one's values in one
// result, the upper one's in the other
__device__ __forceinline__ double add_rows(double v)
{
    const long long x = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(x >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) + __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double add_halves(double v)
{
    const long long x = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(x >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) + __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}

// -------------------------------------------------------------------------
// a wavefront's solver with many rows per lane (slab_tile.hpp)
// -------------------------------------------------------------------------

constexpr int LCS_WIN = 4;       // rows of coefficient loads in flight ahead of a recurrence

// 1 / v: v_rcp_f64 refined by two Newton steps, within about an ulp of the quotient
// (the pivots of these diagonally dominant systems are finite, normal, and far from
// zero)
__device__ __forceinline__ double rcp64(double v)
{
    double r = __builtin_amdgcn_rcp(v);
    double e = fma(-v, r, 1.0);
    r = fma(r, e, r);
    e = fma(-v, r, 1.0);
    return fma(r, e, r);
}

// the largest of the wavefront's non-negative values, in every lane
__device__ __forceinline__ double wave_max(double v)
{
    v = fmax(v, dpp_mov<0x111>(v, v));                    // lane - 1, - 2, - 4, - 8 of the row (0 past its end)
    v = fmax(v, dpp_mov<0x112>(v, v));
    v = fmax(v, dpp_mov<0x114>(v, v));
    v = fmax(v, dpp_mov<0x118>(v, v));
    return fmax(fmax(lane_at(v, 15), lane_at(v, 31)), fmax(lane_at(v, 47), lane_at(v, 63)));
}

// The values next to the boundary of the two blocks of 2^L lanes that level L
// merges.  L <= 2: p the other block's, q the own block's; L >= 3: p the lower
// block's last lane's, q the upper block's first lane's.
template <int L>
__device__ __forceinline__ void boundary(double u, double &p, double &q)
{
    if constexpr (L == 0) {
        p = dpp_mov<quad(1, 0, 3, 2)>(u, u);
        q = u;
    } else if constexpr (L == 1) {
        p = dpp_mov<quad(2, 2, 1, 1)>(u, u);
        q = dpp_mov<quad(1, 1, 2, 2)>(u, u);
    } else if constexpr (L == 2) {
        q = dpp_mov<quad(3, 3, 3, 3), 0xf, 0x5>(u, u);
        q = dpp_mov<quad(0, 0, 0, 0), 0xf, 0xa>(q, u);
        p = dpp_mov<DPP_HALF_MIRROR>(q, q);
    } else if constexpr (L == 3) {
        p = dpp_mov<DPP_ROW_BCAST + 7>(u, u);
        q = dpp_mov<DPP_ROW_BCAST + 8>(u, u);
    } else if constexpr (L == 4) {
        double e = dpp_mov<DPP_ROW_BCAST + 15, 0x5>(u, u);
        e = dpp_mov<DPP_ROW_BCAST, 0xa>(e, u);
        // swapping e's odd rows with its own even rows leaves the even rows' value
        // everywhere in one result, the odd rows' in the other
        const long long x = __double_as_longlong(e);
        const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(x >> 32), false, false);
        p = __longlong_as_double(((long long)hi[0] << 32) | lo[0]);
        q = __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
    } else {
        p = lane_at(u, 31);
        q = lane_at(u, 32);
    }
}

// Level L of the separators' factorisation.  A block's values are x = u + w x_left +
// v x_right for the values x_left, x_right next to it.  Merging a lower block (last
// lane: uA, vA, wA) with an upper one (first lane: uB, vB, wB) gives
//   x_A = (uA + vA uB) / (1 - vA wB),  x_B = (uB + wB uA) / (1 - vA wB);
// the lower lanes add v x_B, the upper ones w x_A.
template <int L>
__device__ __forceinline__ void merge_factor(int lane, double &v, double &w, double (&k)[12])
{
    const bool low = ((lane >> L) & 1) == 0;
    double vp, vq, wp, wq;
    boundary<L>(v, vp, vq);
    boundary<L>(w, wp, wq);
    const double vA = L >= 3 ? vp : low ? vq : vp, vB = L >= 3 ? vq : low ? vp : vq;
    const double wA = L >= 3 ? wp : low ? wq : wp, wB = L >= 3 ? wq : low ? wp : wq;
    const double s = (low ? v : w) * rcp64(fma(-vA, wB, 1.0));
    const double cA = low ? s * wB : s, cB = low ? s : s * vA;
    v = low ? cB * vB : fma(cB, vB, v);
    w = low ? fma(cA, wA, w) : cA * wA;
    k[2 * L] = L >= 3 ? cA : low ? cB : cA;
    k[2 * L + 1] = L >= 3 ? cB : low ? cA : cB;
}

template <int L>
__device__ __forceinline__ void merge_solve(double &u, const double (&k)[12])
{
    double p, q;
    boundary<L>(u, p, q);
    u = fma(k[2 * L], p, fma(k[2 * L + 1], q, u));
}

template <int V>
struct Int {
    static constexpr int v = V;
};
// -------------------------------------------------------------------------
// a work-group's tridiagonal solver
// -------------------------------------------------------------------------
// Tridiagonal solve by the work-group: row M k + r is thread k's row r, a, b, c its sub-,
// main and super-diagonal (a = 0 in the first row, c = 0 in the last; padding rows a = c =
// 0, b = 1), x the right-hand side in, the solution out.  The threads' rows but their last
// are eliminated, the last rows of a wavefront merged by blocks of 1, 2, .. 32 lanes
// (merge_factor), and what a wavefront's first and last value answer to its neighbours'
// goes through LDS as lanes 2 w, 2 w + 1 of one more such merge, which every wavefront
// does on its own.  One barrier (two for M > 1).
template <int NW, int M>
__device__ __forceinline__ void tri_wg(const double (&a)[M], const double (&b)[M], const double (&c)[M], double (&x)[M])
{
    static_assert((NW & (NW - 1)) == 0 && NW <= 32, "the wavefronts' ends are the lanes of one wavefront");
    __shared__ double sEnd[3][2 * NW], sFirst[3][NW + 1];
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double inv[M], fl[M], cp = 0.0;
    double W0 = 0.0, A0 = 0.0, C0 = 1.0;               // first row = W0 + A0 z_left + C0 z (M > 1)
#pragma unroll
    for (int i = 0; i < M - 1; ++i) {
        inv[i] = rcp64(i > 0 ? b[i] - a[i] * cp : b[i]);
        x[i] = (i > 0 ? x[i] - a[i] * x[i - 1] : x[i]) * inv[i];
        fl[i] = (i > 0 ? -a[i] * fl[i - 1] : -a[i]) * inv[i];
        W0 = fma(C0, x[i], W0);
        A0 = fma(C0, fl[i], A0);
        cp = c[i] * inv[i];
        C0 = -C0 * cp;
    }
    double B = b[M - 1], A = a[M - 1], C = c[M - 1], D = x[M - 1];
    if constexpr (M > 1) {
        if (l == 0) {
            sFirst[0][w] = W0;
            sFirst[1][w] = A0;
            sFirst[2][w] = C0;
        }
        if (threadIdx.x < 3) sFirst[threadIdx.x][NW] = 0.0;
        __syncthreads();
        double Wn = dpp_mov<DPP_NEXT>(W0, W0), An = dpp_mov<DPP_NEXT>(A0, A0), Cn = dpp_mov<DPP_NEXT>(C0, C0);
        if (l == 63) {
            Wn = sFirst[0][w + 1];
            An = sFirst[1][w + 1];
            Cn = sFirst[2][w + 1];
        }
        D -= A * x[M > 1 ? M - 2 : 0] + C * Wn;
        B += C * An - A * cp;
        A *= fl[M > 1 ? M - 2 : 0];
        C *= Cn;
    }
    const double ib = rcp64(B);
    double u = D * ib, wl = -A * ib, vr = -C * ib, k[12];
    auto merge = [&](auto L) {
        merge_factor<L.v>(l, vr, wl, k);
        merge_solve<L.v>(u, k);
    };
    merge(Int<0>());
    merge(Int<1>());
    merge(Int<2>());
    merge(Int<3>());
    merge(Int<4>());
    merge(Int<5>());
    if (l == 0 || l == 63) {
        const int e = 2 * w + (l > 0);
        sEnd[0][e] = u;
        sEnd[1][e] = vr;
        sEnd[2][e] = wl;
    }
    __syncthreads();
    double xl, xr;                                     // the values next to the wavefront's rows
    {
        const double u0 = u, v0 = vr, w0 = wl;
        u = l < 2 * NW ? sEnd[0][l] : 0.0;
        vr = l < 2 * NW ? sEnd[1][l] : 0.0;
        wl = l < 2 * NW ? sEnd[2][l] : 0.0;
        if constexpr (NW > 1) merge(Int<1>());
        if constexpr (NW > 2) merge(Int<2>());
        if constexpr (NW > 4) merge(Int<3>());
        if constexpr (NW > 8) merge(Int<4>());
        if constexpr (NW > 16) merge(Int<5>());
        xl = w > 0 ? lane_at(u, w > 0 ? 2 * w - 1 : 0) : 0.0;
        xr = w < NW - 1 ? lane_at(u, w < NW - 1 ? 2 * w + 2 : 0) : 0.0;
        u = fma(v0, xr, fma(w0, xl, u0));
    }
    x[M - 1] = u;
    if constexpr (M > 1) {
        double zl = dpp_mov<DPP_PREV>(u, u);
        if (l == 0) zl = xl;
#pragma unroll
        for (int i = M - 2; i >= 0; --i) x[i] = fma(fl[i], zl, x[i]) - c[i] * inv[i] * x[i + 1];
    }
}

// The same solve in two parts, for an operator with many right-hand sides: wg_factor once,
// wg_solve per right-hand side (one barrier).  A wavefront's last row sees the first row of
// the next wavefront, x = W0 + A0 z + C0 z'; its response vr is to W0 + C0 z', so that
// nothing has to pass between the wavefronts before the merges.  The two ends' buffers in
// LDS alternate (ph).
template <int NW>
struct WgLds {
    double a0[NW + 1], c0[NW + 1], ev[2 * NW], ew[2 * NW];
    double u[2][2 * NW], w0[2][NW + 1];
};
constexpr int WG_KEEP = 8;                      // rows per thread up to which a / pivot and c / pivot are kept
template <int M, bool KEEP = M <= WG_KEEP>
struct WgFac {
    static constexpr int NK = KEEP ? M - 1 : 1;
    double inv[M - 1], av[NK], cv[NK];          // interior rows: 1 / pivot, a / pivot, c / pivot
    double as, cs, ib;                          // last row: a, c, 1 / pivot
    double k[12], wl, vr;                       // its merges within the wavefront; responses to the rows next to it
    double kq[12], ve, cx;                      // the wavefronts' ends
};

template <int NW, int M, bool KEEP, class GA, class GC>
__device__ __forceinline__ void wg_factor(GA a, const double (&b)[M], GC c, WgFac<M, KEEP> &F, WgLds<NW> &S)
{
    static_assert(M >= 2 && (NW == 2 || NW == 4 || NW == 8), "rows per thread; levels of the ends' merge below");
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double A0 = 0.0, C0 = 1.0, f = 1.0, cp = 0.0;
#pragma unroll
    for (int i = 0; i < M - 1; ++i) {
        const double ai = a(i);
        F.inv[i] = rcp64(i > 0 ? b[i] - ai * cp : b[i]);
        const double av = ai * F.inv[i];
        cp = c(i) * F.inv[i];
        if constexpr (KEEP) {
            F.av[i] = av;
            F.cv[i] = cp;
        }
        f = -f * av;
        A0 = fma(C0, f, A0);
        C0 = -C0 * cp;
    }
    if (l == 0) {
        S.a0[w] = A0;
        S.c0[w] = C0;
    }
    if (threadIdx.x == 0) S.a0[NW] = S.c0[NW] = S.w0[0][NW] = S.w0[1][NW] = 0.0;
    __syncthreads();
    double An = dpp_mov<DPP_NEXT>(A0, A0), Cn = dpp_mov<DPP_NEXT>(C0, C0);
    if (l == 63) {
        An = S.a0[w + 1];
        Cn = 1.0;
    }
    F.cx = S.c0[w + 1];
    F.as = a(M - 1);
    F.cs = c(M - 1);
    F.ib = rcp64(b[M - 1] - F.as * cp + F.cs * An);
    double wl = -(F.as * f) * F.ib, vr = -(F.cs * Cn) * F.ib;
    merge_factor<0>(l, vr, wl, F.k);
    merge_factor<1>(l, vr, wl, F.k);
    merge_factor<2>(l, vr, wl, F.k);
    merge_factor<3>(l, vr, wl, F.k);
    merge_factor<4>(l, vr, wl, F.k);
    merge_factor<5>(l, vr, wl, F.k);
    F.wl = wl;
    F.vr = vr;
    if (l == 0 || l == 63) {
        S.ev[2 * w + (l > 0)] = vr;
        S.ew[2 * w + (l > 0)] = wl;
    }
    __syncthreads();
    const bool end = l < 2 * NW;
    F.ve = end ? S.ev[l] : 0.0;
    vr = end ? F.ve * S.c0[(l >> 1) + 1] : 0.0;
    wl = end ? S.ew[l] : 0.0;
    merge_factor<1>(l, vr, wl, F.kq);
    if constexpr (NW > 2) merge_factor<2>(l, vr, wl, F.kq);
    if constexpr (NW > 4) merge_factor<3>(l, vr, wl, F.kq);
}

// x: right-hand side in, solution out; a, c as given to wg_factor
template <int NW, int M, bool KEEP, class GA, class GC>
__device__ __forceinline__ void wg_solve(GA a, GC c, const WgFac<M, KEEP> &F, double (&x)[M], WgLds<NW> &S, int &ph)
{
    auto av = [&](int i) {
        if constexpr (KEEP) return F.av[i];
        else return a(i) * F.inv[i];
    };
    auto cv = [&](int i) {
        if constexpr (KEEP) return F.cv[i];
        else return c(i) * F.inv[i];
    };
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double W0 = 0.0, pr = 1.0;
#pragma unroll
    for (int i = 0; i < M - 1; ++i) {
        x[i] = i > 0 ? fma(-av(i), x[i - 1], x[i] * F.inv[i]) : x[0] * F.inv[0];
        W0 = fma(pr, x[i], W0);
        pr = -pr * cv(i);
    }
    double u = (x[M - 1] - F.as * x[M - 2] - F.cs * dpp_mov<DPP_NEXT>(W0, W0)) * F.ib;
    merge_solve<0>(u, F.k);
    merge_solve<1>(u, F.k);
    merge_solve<2>(u, F.k);
    merge_solve<3>(u, F.k);
    merge_solve<4>(u, F.k);
    merge_solve<5>(u, F.k);
    if (l == 0) {
        S.u[ph][2 * w] = u;
        S.w0[ph][w] = W0;
    }
    if (l == 63) S.u[ph][2 * w + 1] = u;
    __syncthreads();
    double e = l < 2 * NW ? fma(F.ve, S.w0[ph][(l >> 1) + 1], S.u[ph][l]) : 0.0;
    merge_solve<1>(e, F.kq);
    if constexpr (NW > 2) merge_solve<2>(e, F.kq);
    if constexpr (NW > 4) merge_solve<3>(e, F.kq);
    const double xl = w > 0 ? lane_at(e, w > 0 ? 2 * w - 1 : 0) : 0.0;
    const double xr = w < NW - 1 ? fma(F.cx, lane_at(e, w < NW - 1 ? 2 * w + 2 : 0), S.w0[ph][w + 1]) : 0.0;
    ph ^= 1;
    u = fma(F.vr, xr, fma(F.wl, xl, u));
    x[M - 1] = u;
    double f = dpp_mov<DPP_PREV>(u, u);
    if (l == 0) f = xl;
#pragma unroll
    for (int i = 0; i < M - 1; ++i) {
        f = -f * av(i);
        x[i] += f;
    }
#pragma unroll
    for (int i = M - 2; i >= 0; --i) x[i] = fma(-cv(i), x[i + 1], x[i]);
}

// the largest over the work-group of two non-negative values each (the same in every
// thread; its barrier also separates the caller's LDS writes from what follows; another
// barrier must lie between two calls)
template <int NW>
__device__ __forceinline__ void wg_max2(double &a, double &b)
{
    __shared__ double m2[2][NW];
    a = wave_max(a);
    b = wave_max(b);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        m2[0][w] = a;
        m2[1][w] = b;
    }
    __syncthreads();
    a = m2[0][0];
    b = m2[1][0];
#pragma unroll
    for (int q = 1; q < NW; ++q) {
        a = fmax(a, m2[0][q]);
        b = fmax(b, m2[1][q]);
    }
}

// -------------------------------------------------------------------------
// exchange and barrier over a set of co-resident work-groups of a cooperative launch
// -------------------------------------------------------------------------
// What the work-groups pass to each other between barriers goes through agent-scope
// accesses of single words: they bypass the caches that the dies do not share, so that
// the barrier needs no write-back and no invalidation of an L2.
__device__ __forceinline__ void agent_put(double *p, double v)
{
    __hip_atomic_store((unsigned long long *)p, (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double agent_get(const double *p)
{
    return __longlong_as_double((long long)__hip_atomic_load((const unsigned long long *)p, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT));
}

// The set is `nblk` work-groups whose member index is `bid` (0..nblk-1), with
// their own flag array.  Every work-group publishes the generation number in
// its own flag (no contended counter); lanes of wave 0 watch one flag each.  Every
// wavefront waits until its own puts have reached the level that all dies share before
// the work-group barrier ahead of the flag, and the gets behind the closing barrier are
// issued after the flags were seen.  Ordinary stores are not made visible.
// The wait is bounded: on a timeout, or when another work-group has already
// reported one, the error flag is raised and false is returned so that every
// work-group leaves the iteration instead of hanging the device.
__device__ __forceinline__ bool grid_barrier(unsigned long long *flags, unsigned long long gen, int *err,
                                             int bid, int nblk)
{
    __shared__ int s_fail;
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        s_fail = 0;
        __hip_atomic_store(&flags[(size_t)bid * BAR_STRIDE], gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (threadIdx.x < 64) {
        bool fail = false;
        for (int b = threadIdx.x; b < nblk; b += 64) {
            unsigned spins = 0;
            while (__hip_atomic_load(&flags[(size_t)b * BAR_STRIDE], __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT) < gen) {
                if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 ||
                    ++spins > (1u << 20)) {
                    fail = true;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        if (fail) {
            atomicOr(err, 1);
            s_fail = 1;
        }
    }
    __syncthreads();
    return s_fail == 0;
}

__device__ __forceinline__ double kpow(double T, int m) { return m == 0 ? 1.0 : T * T * T; }

// O^n may be stored in binary64 or binary32 (OT); arithmetic is binary64
template <class OT>
__device__ __forceinline__ double node_flux(const double *Eall, const OT *O, const double *Aw,
                                            const double *Bc, double mu, int N, int P, int i, int p)
{
    // interior node i (1..N-1): O_i = Aw_i O^n_i - Bc_i mu (E_i - E_{i-1})
    return Aw[i] * (double)O[(size_t)i * P + p] -
           Bc[i] * mu * (Eall[(size_t)i * P + p] - Eall[(size_t)(i - 1) * P + p]);
}

template <class OT>
__device__ __forceinline__ double node_any(const double *Eall, const OT *O, const double *Aw,
                                           const double *Bc, double mu, double bl, double br, double eps,
                                           int N, int P, int i, int p)
{
    if (i >= 1 && i <= N - 1) return node_flux(Eall, O, Aw, Bc, mu, N, P, i, p);
    if (i == 0)   // inflow relation (4.7) at x = 0
        return 2.0 / eps * (bl - Eall[p]) - node_flux(Eall, O, Aw, Bc, mu, N, P, 1, p);
    // i == N, (4.7) at x = L
    return 2.0 / eps * (Eall[(size_t)(N - 1) * P + p] - br) - node_flux(Eall, O, Aw, Bc, mu, N, P, N - 1, p);
}

// -------------------------------------------------------------------------
// prediction iteration: acceleration and stopping test
// -------------------------------------------------------------------------
// Adaptive Chebyshev semi-iteration on top of the preconditioned Richardson
// update z = res + D^-1 (G res).  The iteration matrix I - (I + D^-1 G) S has a
// real spectrum in [0, b] with b < 1 (b ~ 0.1-0.3 on optically thick slabs), so
// the three-term Chebyshev recurrence for that interval needs no inner
// products; it replaces the plain updates by d_k = alpha_k d_{k-1} + beta_k z_k
// once the plain contraction ratio r = |z_k| / |z_{k-1}| (max norms relative
// to max|rho|) has settled: two consecutive ratios within CHEB_STAB of each
// other, r <= CHEB_RMAX (larger ratios belong to the transient of the first
// updates from a poor start, not to the spectrum), and the update norm still
// above CHEB_MARGIN times the tolerance (close to it the norms approach the
// rounding level).  The interval is [0, CHEB_KAPPA r].  The solve falls back to
// plain updates for good if, CHEB_PROG or more recurrence steps in, the update
// norm is above what plain updates at ratio r would have reached, or at any
// point above the norm at which the recurrence began.  The state is a function
// of the reduced norms only, so every thread of a tile, and every work-group of
// a cooperative solve, takes the same decisions.  Convergence is tested on
// max|z| as for the plain iteration.
struct ChebState {
    int nr = 0;                 // plain updates taken
    int on = 0;                 // recurrence running
    int off = 0;                // fell back to plain updates
    int j = 0;                  // recurrence steps taken
    // relative update norms max|z| / max|rho|, newest first (binary32: they
    // only steer the recurrence and the decisions around it)
    float q1 = 0.0f, q2 = 0.0f, q3 = 0.0f;
    float q0 = 0.0f, r0 = 0.0f, rj = 1.0f;   // at the start: norm, ratio; r0^j
    float s1 = 0.0f, rp = 0.0f, de = 1.0f;   // recurrence parameters
};
constexpr int CHEB_K0 = 3, CHEB_PROG = 4;
constexpr float CHEB_KAPPA = 1.2f, CHEB_STAB = 0.15f, CHEB_RMAX = 0.5f, CHEB_BMIN = 0.02f, CHEB_MARGIN = 100.0f;

// coefficients (alpha, beta) of this update
__device__ __forceinline__ void cheb_coeffs(ChebState &C, int accel, double tol, double &alpha, double &beta)
{
    alpha = 0.0;
    beta = 1.0;
    if (!accel || C.off || C.nr < CHEB_K0) return;
    if (!C.on) {
        if (!(C.q1 > CHEB_MARGIN * (float)tol) || !(C.q2 > 0.0f) || !(C.q3 > 0.0f)) return;
        const float r = C.q1 / C.q2, r2 = C.q2 / C.q3;
        if (!(r <= CHEB_RMAX) || !(fabsf(r - r2) <= CHEB_STAB * r)) return;
        const float b = fmaxf(CHEB_BMIN, CHEB_KAPPA * r);
        const float th = 1.0f - 0.5f * b;
        C.de = 0.5f * b;
        C.s1 = th / C.de;
        C.rp = 1.0f / C.s1;
        C.q0 = C.q1;
        C.r0 = r;
        C.rj = 1.0f;
        C.j = 0;
        C.on = 1;
        beta = 1.0 / (double)th;
        return;
    }
    const float rn = 1.0f / (2.0f * C.s1 - C.rp);
    alpha = (double)(rn * C.rp);
    beta = (double)(2.0f * rn / C.de);
    C.rp = rn;
}

// record this update's relative norm q
__device__ __forceinline__ void cheb_record(ChebState &C, float q)
{
    if (C.on) {
        ++C.j;
        C.rj *= C.r0;
        if (q > C.q0 || (C.j >= CHEB_PROG && q > C.q0 * C.rj)) {
            C.on = 0;
            C.off = 1;
        }
    } else {
        ++C.nr;
    }
    C.q3 = C.q2;
    C.q2 = C.q1;
    C.q1 = q;
}

// Stopping test of the prediction iteration for update norm md and iterate
// norm mr, with the relative update norms q = md / mr of this update and
// qprev, qprev2, qprev3 of the three before: 1 if md <= tol mr; 2 (a
// safeguard) when the updates have reached the rounding level of the residual,
// where they only fluctuate and further updates do not improve the iterate:
// either md <= PRED_FLOOR tol mr and the relative update norm has not
// decreased over the last two updates, or md <= PRED_STALL tol mr and it is
// still above 0.9 of what it was three updates earlier (no progress; a
// converging iteration shrinks it by the contraction ratio every update, well
// below 0.9^(1/3) here).  0 otherwise.
constexpr double PRED_FLOOR = 16.0, PRED_STALL = 64.0;
__device__ __forceinline__ int pred_stop(double md, double mr, float q, float qprev, float qprev2, float qprev3,
                                         int it, double tol)
{
    if (md <= tol * mr) return 1;
    if (it > 2 && md <= PRED_FLOOR * tol * mr && q >= qprev && qprev >= qprev2) return 2;
    if (it > 3 && md <= PRED_STALL * tol * mr && q >= 0.9f * qprev3) return 2;
    return 0;
}


// -------------------------------------------------------------------------
// scalar temperature equation (4.13): Newton with an upper bound of the root
// -------------------------------------------------------------------------
// g is convex and increasing for T >= 0, and its root lies below both
// single-term roots (C/q4)^{1/4} and C/lin, C = rhs + lin Tn (each term alone
// is non-negative), and above half the smaller of them; iterates are clamped to
// that bound, so a start far below the root (a cold cell heated by the inflow)
// does not overshoot by orders of magnitude and then creep back by 3/4 per
// step.  The root and the stopping test are those of the plain iteration.
__device__ __forceinline__ double newton_cap(double q4, double lin, double rhs, double Tn)
{
    const double C = rhs + lin * Tn;
    // no positive root, or a linear equation (Newton exact in one step): no bound
    if (!(C > 0.0) || !(q4 > 0.0)) return INFINITY;
    // widened by 2^-50 so that rounding never puts the bound below the root
    return fmin(sqrt(sqrt(C / q4)), C / lin) * (1.0 + 0x1p-50);
}

__device__ __forceinline__ bool newton_quartic(double T0, double Tn, double q4, double lin, double rhs, int maxit,
                                               double &T, int &its)
{
    const double cap = newton_cap(q4, lin, rhs, Tn);
    T = T0;
    for (int k = 0; k < maxit; ++k) {
        const double T2 = T * T;
        const double g = q4 * T2 * T2 + lin * (T - Tn) - rhs;
        const double dg = 4.0 * q4 * T2 * T + lin;
        const double Tp = T;
        T = fmin(T - g / dg, cap);
        const double step = Tp - T;
        ++its;
        if (fabs(step) <= 0x1p-50 * fmax(fabs(T), fabs(Tn))) return true;
    }
    return false;
}

}  // namespace
