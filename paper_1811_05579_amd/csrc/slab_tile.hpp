// slab_tile.hpp -- the prediction solve of one slab by one "tile" of NW
// wavefronts (device code shared by the batched and the single-slab path).
//
// The angular moment rho solves S rho = s (grte.hip, file header) by the update
// z = res + D^{-1}(G res).  T_p and D do not change during the iteration, and
// the residual obeys
//     res_{k+1} = res_k - d_k + sum_p omega_p T_p^{-1} (G d_k),   d_k = rho_{k+1} - rho_k,
// exactly, so the tile factors every T_p (and D) once, forms the true residual of
// the starting iterate in that first pass, and from then on solves all pairs for
// the one right-hand side G d_k held in LDS.  d_k is the difference of the rounded
// iterates, so res stays the residual of the rho that is held.  The rounding of a
// true residual is that of the v_p = T_p^{-1} [r_p - (T_p - G) rho], which shrink to
// the anisotropy E_p - rho as rho converges, and stiff slabs amplify it by up to
// a c beta; the residual is therefore formed anew once, when the updates have fallen
// to TILE_FRESH (the recursion then adds the rounding of updates below that only).
// When the recursion meets the stopping test, the updates go on with true residuals
// until one of those meets it (usually the first), so that the accepted iterate is
// the one that a solve with true residuals throughout ends at, whatever the path.
// The right-hand sides r_p are read four times in most solves, not once per update,
// and no division is left in the iteration.
//
// One wavefront solves one pair on its own (row j = lane M + i, LDS position i 64 +
// lane): the interior rows 0..M-2 of each lane's chunk are eliminated top-down,
// the separators (row M-1) form a 64-row tridiagonal system solved by merging
// blocks of 1, 2, 4, .. 32 lanes.  What does not depend on the right-hand side is
// kept per pair in global memory (fac_doubles, read as 16-byte
// words): the reciprocal pivots of the interior rows, the two merge coefficients
// per level, the separators' reciprocal diagonal.  The pairs are dealt to the
// wavefronts in turn; their angular sums meet in LDS in a fixed order.
//
// Bound: with one slab per compute unit, the LDS reads of the off-diagonals and the
// right-hand side (3 words per row and pair, 5 above KEEP_ROWS) against ~11 binary64
// operations, at two wavefronts per SIMD; with every compute unit busy, the stream of
// the factorisations (M + 12 words per lane and pair and update, ~5.8 TB/s).  Measured
// on an MI355X: one 1023-cell slab of 32 pairs, 15 updates, 178 us; 2048 such slabs
// 2.44 ms.  A tile that factored each pair again in every update and read its r_p
// (four wavefronts) took 1.07 ms per step on an ensemble of 24
// slabs and 5.0 ms on one of 4096; this one 0.44 and 2.8 ms.
#pragma once
#include "solver_common.hpp"

namespace {

// doubles of one pair's factorisation, M rows per lane (M even): the pivots of the
// interior rows, the reciprocal diagonal and two merge coefficients per level
constexpr int fac_doubles(int M) { return (M + 12) * 64; }

// the separator system of one pair, one row per lane
struct LaneRed {
    double k[12], ib;
};
constexpr double TILE_FRESH = 1e-7;       // relative update norm at which the true residual is formed anew

// v through an empty asm: the compiler cannot hoist what is derived from the
// result out of the enclosing loop (keeps per-row addresses out of registers)
__device__ __forceinline__ int opaque(int v)
{
    __asm__ volatile("" : "+v"(v));
    return v;
}

__device__ __forceinline__ double opaque_d(double v)
{
    __asm__ volatile("" : "+v"(v));
    return v;
}

// the value is formed here and no memory access moves across: without it the
// arithmetic of many rows sinks below their loads, which then all stay in registers
__device__ __forceinline__ void pin(double &v) { __asm__ volatile("" : "+v"(v) : : "memory"); }

// Factor the wavefront's system, a(i), b(i), c(i) the sub-, main and super-diagonal of
// the lane's row i (a = 0 in row 0 of the system, c = 0 in its last row)
template <int M, class GA, class GB, class GC>
__device__ __forceinline__ void lane_factor(GA a, GB b, GC c, double (&inv)[M - 1], LaneRed &F)
{
    static_assert(M >= 2, "at least two rows per lane");
    // cp = c / pivot of the last row; f: the rows' response to the left separator,
    // pr = prod(-c / pivot), A0 = sum pr f: the first row's response to it
    double cp = 0.0, f = 0.0, pr = 1.0, A0 = 0.0;
#pragma unroll
    for (int i = 0; i < M - 1; ++i) {
        const double ai = a(i);
        inv[i] = rcp64(i > 0 ? b(i) - ai * cp : b(i));
        f = (i > 0 ? -ai * f : -ai) * inv[i];
        A0 += pr * f;
        cp = c(i) * inv[i];
        pr = -pr * cp;
        if (i % LCS_WIN == LCS_WIN - 1) {
            pin(A0);
            pin(pr);
        }
    }
    // x_0 = .. + A0 z_left + pr z,  x_{M-2} = .. + f z_left - cp z
    const double A0n = dpp_mov<DPP_NEXT>(A0, A0), C0n = dpp_mov<DPP_NEXT>(pr, pr);
    const double as = a(M - 1), cs = c(M - 1);
    F.ib = rcp64(b(M - 1) - as * cp + cs * A0n);
    double w = -(as * f) * F.ib, v = -(cs * C0n) * F.ib;
    const int lane = opaque(threadIdx.x & 63);
    merge_factor<0>(lane, v, w, F.k);
    merge_factor<1>(lane, v, w, F.k);
    merge_factor<2>(lane, v, w, F.k);
    merge_factor<3>(lane, v, w, F.k);
    merge_factor<4>(lane, v, w, F.k);
    merge_factor<5>(lane, v, w, F.k);
}

// Solve with the factorisation: off-diagonals m2 ll(i), m2 lu(i); x: right-hand
// side in, solution out.  Up to KEEP_ROWS rows per lane the products of the
// off-diagonals with the pivots are kept in registers from the forward pass; above
// that they are formed again (the coefficients read twice instead of once), as x,
// the pivots and the caller's sums fill the register file.  next(0) is called once
// the pivots and ib are read for the last time, next(1) once the coefficients k
// are: the caller may load the next factorisation into them.
constexpr int KEEP_ROWS = 16;
template <int M, class GL, class GU, class Next>
__device__ __forceinline__ void lane_solve(double m2, GL ll, GU lu, const double (&inv)[M - 1], const LaneRed &F,
                                           double (&x)[M], Next next)
{
    constexpr bool KEEP = M <= KEEP_ROWS;
    double av[KEEP ? M - 1 : 1], cv[KEEP ? M - 1 : 1];
    // forward; w = the first interior row's value for zero separators
    double y = 0.0, w = 0.0, pr = 1.0;
#pragma unroll
    for (int i = 0; i < M - 1; ++i) {
        const double t = m2 * inv[i], a = ll(i) * t, c = lu(i) * t;
        if constexpr (KEEP) {
            av[i] = a;
            cv[i] = c;
        }
        y = i > 0 ? fma(-a, y, x[i] * inv[i]) : x[0] * inv[0];
        x[i] = y;
        w = fma(pr, y, w);
        pr = -pr * c;
        if (i % LCS_WIN == LCS_WIN - 1) {
            pin(w);
            pin(pr);
        }
    }
    const double ib = F.ib;
    if constexpr (KEEP) next(0);
    double z = (x[M - 1] - m2 * ll(M - 1) * y - m2 * lu(M - 1) * dpp_mov<DPP_NEXT>(w, w)) * ib;
    merge_solve<0>(z, F.k);
    merge_solve<1>(z, F.k);
    merge_solve<2>(z, F.k);
    merge_solve<3>(z, F.k);
    merge_solve<4>(z, F.k);
    merge_solve<5>(z, F.k);
    if constexpr (KEEP) next(1);
    double f = dpp_mov<DPP_PREV>(z, z);
    x[M - 1] = z;
    if constexpr (KEEP) {
#pragma unroll
        for (int i = 0; i < M - 1; ++i) {
            f = -f * av[i];
            x[i] += f;
        }
#pragma unroll
        for (int i = M - 2; i >= 0; --i) x[i] = fma(-cv[i], x[i + 1], x[i]);
    } else {
        // (m2 through an empty asm per pass: the products with the pivots are formed
        // again rather than kept for all rows)
        const double mf = opaque_d(m2);
#pragma unroll
        for (int i = 0; i < M - 1; ++i) {
            f = -f * (ll(i) * (mf * inv[i]));
            x[i] += f;
            if (i % LCS_WIN == LCS_WIN - 1) pin(x[i]);
        }
        const double mb = opaque_d(m2);
#pragma unroll
        for (int i = M - 2; i >= 0; --i) {
            x[i] = fma(-(lu(i) * (mb * inv[i])), x[i + 1], x[i]);
            if (i % LCS_WIN == 0) pin(x[i]);
        }
        next(0);
        next(1);
    }
}

// a factorisation in memory: the pivots and the reciprocal diagonal (M values), then
// the merge coefficients, 16-byte words of consecutive lanes
template <int M>
__device__ __forceinline__ void fac_store(double *fac, int lane, const double (&inv)[M - 1], const LaneRed &F)
{
    double2 *q = reinterpret_cast<double2 *>(fac) + lane;
#pragma unroll
    for (int i = 0; i < M / 2; ++i) q[i * 64] = make_double2(inv[2 * i], 2 * i + 1 < M - 1 ? inv[(2 * i + 1) % (M - 1)] : F.ib);
#pragma unroll
    for (int i = 0; i < 6; ++i) q[(M / 2 + i) * 64] = make_double2(F.k[2 * i], F.k[2 * i + 1]);
}

// part 0: the pivots and the reciprocal diagonal; 1: the merge coefficients
template <int M>
__device__ __forceinline__ void fac_load(const double *fac, int lane, int part, double (&inv)[M - 1], LaneRed &F)
{
    const double2 *q = reinterpret_cast<const double2 *>(fac) + lane;
    if (part == 0) {
#pragma unroll
        for (int i = 0; i < M / 2; ++i) {
            const double2 d = q[i * 64];
            inv[2 * i] = d.x;
            if (2 * i + 1 < M - 1) inv[(2 * i + 1) % (M - 1)] = d.y;
            else F.ib = d.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const double2 d = q[(M / 2 + i) * 64];
            F.k[2 * i] = d.x;
            F.k[2 * i + 1] = d.y;
        }
    }
}

// make the tile's LDS and global writes visible to the whole tile
template <int NW>
__device__ __forceinline__ void tile_sync()
{
    if constexpr (NW > 1) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
}

// LDS of a tile (doubles): the two off-diagonals, the right-hand side G d, the
// wavefronts' angular sums (also rho, Lam, Lam - G of the first and last pass) and
// the maxima.  Eight wavefronts of more than 28 rows per lane share four slots.
template <int NW, int M>
constexpr int tile_slots() { return NW == 8 && M > 28 ? 4 : NW; }
template <int NW, int M>
constexpr int tile_lds()
{
    return (3 + (tile_slots<NW, M>() < 3 ? 3 : tile_slots<NW, M>())) * 64 * M + 2 * NW;
}

// one slab's system, as the tile reads it
struct TileSys {
    int N, P;
    const double *mu, *om;
    const double *Ll, *Lu, *Lam, *LmG;   // per cell
    double bd0, bdN;                     // the inflow terms of the two end cells
    double mu1, mu2, omw;                // sum omega mu, sum omega mu^2, 1 - sum omega
    const double *rhs;                   // r_p at rhs + p rhs_stride, cell order, zero beyond N up to 64 M
    size_t rhs_stride;
    const double *rho0;                  // starting iterate per cell
    double *rho_out;                     // converged rho per cell
    double *fac;                         // (P + 1) x fac_doubles(M): the pairs' factorisations, then D's
    int accel, maxit;
    double tol;
    double *hist;                        // max|z| / max|rho| of the updates (null: not kept)
};

// x[K NW + w] by selects on the wavefront's number (registers have no index; each
// value goes through an empty asm, or the compiler indexes the array in memory)
template <int K, int NW, int M>
__device__ __forceinline__ double own_of(const double (&x)[M], int w)
{
    double v = opaque_d(x[K * NW]);
#pragma unroll
    for (int q = 1; q < NW; ++q) {
        if (K * NW + q < M) {
            const double t = opaque_d(x[K * NW + q]);
            v = w == q ? t : v;
        }
    }
    return v;
}
// f(Int<k>, r) for the rows r = k NW + w < M
template <int NW, int M, int K = 0, class F>
__device__ __forceinline__ void own_rows(int w, F &f)
{
    if constexpr (K * NW < M) {
        if (K * NW + NW <= M || K * NW + w < M) f(Int<K>(), K * NW + w);
        own_rows<NW, M, K + 1>(w, f);
    }
}

// Runs the iteration; store(p, first row, x) takes E*_p of the lane's M rows.
// Returns the updates up to the one that met the stopping test: the cap holds for those.
// The updates that confirm it with true residuals are not counted and have a cap of the
// same size; if they run out of it, all updates are returned.  converged as pred_stop.
template <int NW, int M, class Store>
__device__ __forceinline__ int pred_tile(const TileSys &S, double *sm, int &converged, Store store)
{
    constexpr int NP = 64 * M, NS = tile_slots<NW, M>(), RO = (M + NW - 1) / NW;
    constexpr bool HOLD = M <= 10;       // a wavefront with one pair keeps its factorisation in registers
    double *sll = sm, *slu = sm + NP, *sg = sm + 2 * NP, *slot = sm + 3 * NP;
    double *red = sm + tile_lds<NW, M>() - 2 * NW;
    const int tid = NW == 1 ? (threadIdx.x & 63) : threadIdx.x;
    const int w = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = S.N, P = S.P;
    constexpr int FD = fac_doubles(M);
    auto lpos = [](int j) { return (j % M) * 64 + j / M; };
    // rows r = w (mod NW) of every lane are wavefront w's to update
    auto own = [&](auto f) { own_rows<NW, M>(w, f); };
    for (int j = tid; j < NP; j += 64 * NW) {
        const int t = lpos(j);
        const bool in = j < N;
        sll[t] = in ? S.Ll[j] : 0.0;
        slu[t] = in ? S.Lu[j] : 0.0;
        slot[t] = in ? S.rho0[j] : 0.0;
        slot[NP + t] = in ? S.Lam[j] : 1.0;          // padding rows: T_p = D = 1, no coupling
        slot[2 * NP + t] = in ? S.LmG[j] : 1.0;
    }
    tile_sync<NW>();
    double rho[RO], G[RO], res[RO];
    float dch[RO];                                    // previous update (steers the next one only)
    {
        const int l = opaque(threadIdx.x & 63);
        own([&](auto kc, int r) {
            constexpr int k = kc.v;
            const int t = r * 64 + l;
            rho[k] = slot[t];
            G[k] = slot[NP + t] - slot[2 * NP + t];
            dch[k] = 0.0f;
        });
    }
    double inv[M - 1], x[M], acc[M];
    LaneRed F;
    double invD[HOLD ? M - 1 : 1];
    LaneRed FDif;
    // y = r_p - (Lam - G + mu^2 L + mu B) rho of pair p's rows, L rho by neighbour
    // differences (near convergence they are formed almost exactly)
    auto residual = [&](int p, double m1, double m2) {
        const int l = opaque(threadIdx.x & 63), j0 = l * M, rl1 = N - 1 - j0;
        const double *rh = slot + l, *lg = slot + 2 * NP + l, *ll = sll + l, *lu = slu + l;
        const double *src = S.rhs + (size_t)p * S.rhs_stride + j0;
        const double b0 = l == 0 ? S.bd0 : 0.0;
#pragma unroll
        for (int r = 0; r < M; ++r) x[r] = src[r];
#pragma unroll
        for (int r = 0; r < M; ++r) {
            const double rj = rh[r * 64];
            // an in-bounds dummy where there is no neighbour: its coefficient is 0 there
            const double rl = (r > 0) ? rh[(r - 1) * 64] : (l > 0 ? rh[(M - 1) * 64 - 1] : rj);
            const double rn = (r < M - 1) ? rh[(r + 1) * 64] : (l < 63 ? rh[1] : rj);
            const double q = ll[r * 64] * (rl - rj) + lu[r * 64] * (rn - rj);
            const double bd = (r == 0 ? b0 : 0.0) + (r == rl1 ? S.bdN : 0.0);
            x[r] = x[r] - lg[r * 64] * rj - m2 * q - m1 * bd * rj;
            pin(x[r]);
        }
    };
    // with the factorisation held; while its second half runs, that of pair nx (P: D)
    // is loaded in its place (nx < 0: none)
    auto solve = [&](double m2, double (&iv)[M - 1], LaneRed &f, int nx) {
        const int l = opaque(threadIdx.x & 63);
        const double *ll = sll + l, *lu = slu + l;
        lane_solve<M>(m2, [&](int i) { return ll[i * 64]; }, [&](int i) { return lu[i * 64]; }, iv, f, x, [&](int part) {
            if (nx >= 0) fac_load<M>(S.fac + (size_t)nx * FD, opaque(threadIdx.x & 63), part, iv, f);
        });
    };
    auto fetch = [&](int p, double (&iv)[M - 1], LaneRed &f) {
        const int l = opaque(threadIdx.x & 63);
        fac_load<M>(S.fac + (size_t)p * FD, l, 0, iv, f);
        fac_load<M>(S.fac + (size_t)p * FD, l, 1, iv, f);
    };
    // the factorisation of pair p (p = P: of D)
    auto factor = [&](int p, double m1, double m2, const double *diag) {
        const int l = opaque(threadIdx.x & 63), rl1 = N - 1 - l * M;
        const double *ll = sll + l, *lu = slu + l, *la = diag + l;
        const double b0 = l == 0 ? S.bd0 : 0.0;
        lane_factor<M>([&](int i) { return m2 * ll[i * 64]; },
                       [&](int i) {
                           const double bd = (i == 0 ? b0 : 0.0) + (i == rl1 ? S.bdN : 0.0);
                           return la[i * 64] + m2 * (-(ll[i * 64] + lu[i * 64])) + m1 * bd;
                       },
                       [&](int i) { return m2 * lu[i * 64]; }, inv, F);
        fac_store<M>(S.fac + (size_t)p * FD, l, inv, F);
    };
    // rho and Lam - G of all rows into LDS, for residual
    auto stage = [&]() {
        const int l = opaque(threadIdx.x & 63);
        own([&](auto kc, int r) { slot[r * 64 + l] = rho[kc.v]; });
        for (int j = tid; j < NP; j += 64 * NW) slot[2 * NP + lpos(j)] = j < N ? S.LmG[j] : 1.0;
        tile_sync<NW>();
    };
    auto add = [&](double wp) {
#pragma unroll
        for (int r = 0; r < M; ++r) acc[r] = fma(wp, x[r], acc[r]);
    };
    auto clear = [&]() {
#pragma unroll
        for (int r = 0; r < M; ++r) acc[r] = 0.0;
    };
    // the wavefronts' sums into the slots (fixed order: with fewer slots than
    // wavefronts, w + NS joins w first)
    auto publish = [&]() {
        const int l = opaque(threadIdx.x & 63);
        double *q = slot + (w % NS) * NP + l;
        if constexpr (NS < NW) {
            if (w >= NS) {
#pragma unroll
                for (int r = 0; r < M; ++r) q[r * 64] = acc[r];
            }
            tile_sync<NW>();
            if (w < NS) {
#pragma unroll
                for (int r = 0; r < M; ++r) q[r * 64] = acc[r] + q[r * 64];
            }
        } else {
#pragma unroll
            for (int r = 0; r < M; ++r) q[r * 64] = acc[r];
        }
        tile_sync<NW>();
    };
    auto total = [&](int t) {
        double s = slot[t];
#pragma unroll
        for (int q = 1; q < NS; ++q) s += slot[q * NP + t];
        return s;
    };

    // ---- first pass: factor, true residual of the starting iterate
    clear();
    for (int p = w; p < P; p += NW) {
        const double m1 = S.mu[p], m2 = m1 * m1;
        factor(p, m1, m2, slot + NP);
        residual(p, m1, m2);
        solve(m2, inv, F, -1);
        add(S.om[p]);
    }
    if (w == NW - 1) factor(P, S.mu1, S.mu2, slot + 2 * NP);
    tile_sync<NW>();                                   // the slots read by all: they take the sums now
    publish();
    {
        const int l = opaque(threadIdx.x & 63);
        own([&](auto kc, int r) {
            constexpr int k = kc.v;
            res[k] = total(r * 64 + l) - S.omw * rho[k];
        });
    }
    // ---- updates (HOLD: D's factorisation and that of a wavefront's only pair stay in
    // registers; else each solve loads the next one's)
    if constexpr (HOLD) {
        fetch(P, invD, FDif);
        if (w < P) fetch(w, inv, F);
    } else {
        fetch(P, inv, F);
    }
    const int first = w < P ? w : -1;
    int it = 0, met = 0;
    bool fresh = S.tol >= TILE_FRESH;                  // no residual to form anew (any more)
    ChebState C;
    // D f = G res by every wavefront, into x
    auto diffuse = [&]() {
        const int l = opaque(threadIdx.x & 63);
        own([&](auto kc, int r) { slot[r * 64 + l] = G[kc.v] * res[kc.v]; });
        tile_sync<NW>();
#pragma unroll
        for (int r = 0; r < M; ++r) x[r] = slot[r * 64 + l];
        if constexpr (HOLD) solve(S.mu2, invD, FDif, -1);
        else solve(S.mu2, inv, F, first);
    };
    converged = 0;
    bool exact = true, polish = false;                 // res is a true residual; only those from here on
    while (true) {
        diffuse();
        double alpha, beta, md = 0.0, mr = 0.0;
        cheb_coeffs(C, S.accel, S.tol, alpha, beta);
        {
            const int l = opaque(threadIdx.x & 63);
            own([&](auto kc, int r) {
                constexpr int k = kc.v;
                const double z = res[k] + own_of<k, NW>(x, w);
                const double upd = alpha * (double)dch[k] + beta * z;
                dch[k] = (float)upd;
                const double nw = rho[k] + upd;
                const double d = nw - rho[k];
                rho[k] = nw;
                res[k] -= d;
                sg[r * 64 + l] = G[k] * d;
                md = fmax(md, fabs(z));
                mr = fmax(mr, fabs(nw));
            });
        }
        md = wave_max(md);
        mr = wave_max(mr);
        if constexpr (NW > 1) {
            if ((threadIdx.x & 63) == 0) {
                red[w] = md;
                red[NW + w] = mr;
            }
            tile_sync<NW>();
            md = red[0];
            mr = red[NW];
#pragma unroll
            for (int q = 1; q < NW; ++q) {
                md = fmax(md, red[q]);
                mr = fmax(mr, red[NW + q]);
            }
        } else {
            tile_sync<NW>();
        }
        ++it;
        if (S.hist && tid == 0 && it <= GRTE_HIST_CAP) S.hist[it - 1] = mr > 0.0 ? md / mr : md;
        const float qprev = C.q1, qprev2 = C.q2, qprev3 = C.q3;
        const float q = (float)(mr > 0.0 ? md / mr : md);
        cheb_record(C, q);
        // (the same in every lane of every wavefront: scalar decisions)
        const int stop = __builtin_amdgcn_readfirstlane(pred_stop(md, mr, q, qprev, qprev2, qprev3, it, S.tol));
        if (stop && exact) {
            converged = stop;
            break;
        }
        if (polish ? it - met >= S.maxit : !stop && it >= S.maxit) break;
        if (stop && !polish) {                         // plain updates, and the test's history anew
            polish = true;
            met = it;
            C.on = 0;
            C.off = 1;
            C.q1 = C.q2 = C.q3 = INFINITY;
        }
        const bool anew = polish || __builtin_amdgcn_readfirstlane(!fresh && md <= TILE_FRESH * mr);
        exact = anew;
        if (anew) {
            fresh = true;
            stage();
        }
        clear();
        for (int p = w; p < P; p += NW) {
            const double m1 = S.mu[p], m2 = m1 * m1;
            // HOLD: the next pair, around to the first; else D after the last
            const int nx = p + NW < P ? p + NW : HOLD ? (p == w ? -1 : w) : P;
            if (anew) {
                residual(p, m1, m2);
            } else {
                const int l = opaque(threadIdx.x & 63);
#pragma unroll
                for (int r = 0; r < M; ++r) x[r] = sg[r * 64 + l];
            }
            solve(m2, inv, F, nx);
            add(S.om[p]);
        }
        if (anew) tile_sync<NW>();                     // rho read by all before the slots take the sums
        publish();
        {
            const int l = opaque(threadIdx.x & 63);
            own([&](auto kc, int r) {
                constexpr int k = kc.v;
                const double t = total(r * 64 + l);
                res[k] = anew ? t - S.omw * rho[k] : res[k] + t;
            });
        }
    }
    // ---- last pass: E*_p = rho + T_p^{-1} [r_p - (T_p - G) rho]
    stage();
    for (int p = w; p < P; p += NW) {
        const double m1 = S.mu[p], m2 = m1 * m1;
        residual(p, m1, m2);
        solve(m2, inv, F, p + NW < P ? p + NW : -1);
        const int l = opaque(threadIdx.x & 63);
#pragma unroll
        for (int r = 0; r < M; ++r) x[r] += slot[r * 64 + l];
        store(p, l * M, x);
    }
    for (int j = tid; j < N; j += 64 * NW) S.rho_out[j] = slot[lpos(j)];
    tile_sync<NW>();                                   // the tile's LDS and E* settled
    return polish && converged ? met : it;
}

}  // namespace
