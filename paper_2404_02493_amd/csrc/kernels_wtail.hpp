// The small levels of the wave cycle in one workgroup.
//
// Below a few hundred nodes per side every operation of the cycle is a handful
// of microseconds of work, so separate launches are dominated by their latency.
// k_wave_tail runs the whole coarse part of Algorithm 1 from a given level down
// (Chebyshev pre-smoothing, residual + full weighting, the coarser cycle,
// bilinear prolongation, post-smoothing, and the coarsest level's Chebyshev
// iteration) in one workgroup of 1024 threads.  A thread owns the nodes t, t + 1024, ... of
// a level (at most NPT of the first level, one of the others) and keeps their fields in
// registers; stencils and transfers exchange values through two LDS buffers, one barrier
// each, and what a level needs again on the way up waits in LDS.  The arithmetic is FP64 on
// every level (it issues at the FP32 rate): bound by the chain of barriers and LDS round
// trips, about 0.4 us a Chebyshev step.  Measured with levels 32^2 and 16^2 below 64^2: the
// arrays in global memory 45-50 us, so 9-13 us.
#pragma once

#include "kernels_wave.hpp"

namespace helm {

constexpr int WT_THREADS = 1024;
constexpr int WT_MAXL = 14;
constexpr int WT_NODES = 4 * WT_THREADS;  // at most this many nodes on the first level
constexpr int WT_ROW = 256;               // and on a row or column of it (sides differ by 16 at most)

struct TailWaveLevel {
    Geom G;
    int f64;           // arrays of this level are complex128 / double
    const void* n2;
    void* g;
    void* u;
    const double* la;  // device: la[0] = spectral bound of A^* A, la[1] = Chebyshev alpha
};

struct TailWaveArgs {
    TailWaveLevel lv[WT_MAXL + 1];  // indexed by level
    int l0;                         // first level handled here (>= 3)
    int L;
    int cheb_pre, cheb_post, cheb_coarse;
    int level3_literal;
};

// One level held by the workgroup, NPT nodes a thread.  An LDS buffer keeps node p at
// p + WT_ROW; the row behind the last one and the node after it must be 0 (the open edge;
// column nx is column 0 of the next row, the ring).
template <int NPT>
struct WtLevel {
    c128 kp[NPT];
    bool ok[NPT];
    int nx, N;
    double ih2;
    __device__ __forceinline__ static int p(int k) { return (int)threadIdx.x + k * WT_THREADS; }
    __device__ __forceinline__ void init(const TailWaveLevel& W, size_t o) {
        nx = W.G.nx;
        N = W.G.nx * W.G.ny;
        ih2 = W.G.inv_h2;
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int q = p(k) < N ? p(k) : 0;
            const int sh = __builtin_ctz((unsigned)nx), i = q >> sh, j = q & (nx - 1);
            ok[k] = p(k) < N && i > 0 && j > 0;
            const double n2 = W.f64 ? bsh_one(o, (const double*)W.n2)[q] : double(bsh_one(o, (const float*)W.n2)[q]);
            kp[k] = kappa_at<double>(W.G, n2, i, j);
        }
    }
    __device__ __forceinline__ void load(const TailWaveLevel& W, const void* a, size_t o, c128 (&v)[NPT]) const {
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            v[k] = c128{};
            if (ok[k]) v[k] = W.f64 ? bsh_one(o, (const c128*)a)[p(k)] : ccast<double>(bsh_one(o, (const c64*)a)[p(k)]);
        }
    }
    // v to the buffer s, and the zero row behind it
    __device__ __forceinline__ void put(const c128 (&v)[NPT], c128* s) const {
#pragma unroll
        for (int k = 0; k < NPT; ++k)
            if (p(k) < N) s[WT_ROW + p(k)] = v[k];
        if ((int)threadIdx.x <= nx) s[WT_ROW + N + threadIdx.x] = c128{};
    }
    template <bool CJ>
    __device__ __forceinline__ c128 apply(const c128* s, int k) const {  // A s or A^* s, 0 off the unknowns
        if (!ok[k]) return c128{};
        const c128* a = s + WT_ROW + p(k);
        const c128 nb = ((a[-nx] + a[nx]) + a[-1]) + a[1];
        const c128 kap = CJ ? conjg(kp[k]) : kp[k];
        return ih2 * (4.0 * a[0] - nb) - kap * a[0];
    }
    // m Chebyshev steps for A u = g from u (ZERO: from 0), s0 and s1 free on entry and return
    template <bool ZERO>
    __device__ void cheb(const TailWaveLevel& W, size_t o, int m, const c128 (&g)[NPT], c128 (&u)[NPT], c128* s0,
                         c128* s1) const {
        const double* la = bsh_one(o, W.la);
        const double lam = la[0], a = lam / la[1];
        const double theta = 0.5 * (lam + a), dc = 0.5 * (lam - a);
        c128 r[NPT], d[NPT];
        if constexpr (ZERO) {
            put(g, s1);
        } else {
            put(u, s0);
            __syncthreads();
            c128 t[NPT];
#pragma unroll
            for (int k = 0; k < NPT; ++k) t[k] = g[k] - apply<false>(s0, k);
            put(t, s1);
        }
        __syncthreads();
        const double inv_theta = 1.0 / theta;
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            if constexpr (ZERO) u[k] = c128{};
            r[k] = apply<true>(s1, k);
            d[k] = inv_theta * r[k];
        }
        double rho = dc / theta;
#pragma unroll 1
        for (int step = 1; step < m; ++step) {
            const double den = 2.0 * theta - dc * rho, rho_new = dc / den;
            const double c1 = rho_new * rho, c2 = 2.0 / den;
            rho = rho_new;
            put(d, s0);
            __syncthreads();
            c128 t[NPT];
#pragma unroll
            for (int k = 0; k < NPT; ++k) t[k] = apply<false>(s0, k);
            put(t, s1);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < NPT; ++k) {
                r[k] = r[k] - apply<true>(s1, k);
                u[k] = u[k] + d[k];
                d[k] = c1 * d[k] + c2 * r[k];
            }
        }
#pragma unroll
        for (int k = 0; k < NPT; ++k) u[k] = u[k] + d[k];
        __syncthreads();
    }
    // gc = R (g - A u) at this thread's node of the coarse level (SMOOTH false: u = 0)
    template <bool SMOOTH>
    __device__ c128 restrict_to(const c128 (&g)[NPT], const c128 (&u)[NPT], int ncx, int ncy, c128* s0, c128* s1) const {
        if constexpr (SMOOTH) {
            put(u, s0);
            __syncthreads();
            c128 t[NPT];
#pragma unroll
            for (int k = 0; k < NPT; ++k) t[k] = ok[k] ? g[k] - apply<false>(s0, k) : c128{};
            put(t, s1);
        } else {
            put(g, s1);
        }
        __syncthreads();
        c128 v{};
        const int q = threadIdx.x;
        if (q < ncx * ncy) {
            const int sh = __builtin_ctz((unsigned)ncx), I = q >> sh, J = q & (ncx - 1);
            if (I > 0 && J > 0) {
                const c128* a = s1 + WT_ROW + 2 * I * nx + 2 * J;
                const c128 ud = ((a[-nx] + a[nx]) + a[-1]) + a[1];
                const c128 dg = ((a[-nx - 1] + a[-nx + 1]) + a[nx - 1]) + a[nx + 1];
                v = (1.0 / 16.0) * ((4.0 * a[0] + 2.0 * ud) + dg);
            }
        }
        __syncthreads();
        return v;
    }
    // u += P uc, uc one value a thread of the coarse level C
    __device__ void prolong_from(const WtLevel<1>& Cl, c128 uc, c128 (&u)[NPT], c128* s0) const {
        const c128 v[1] = {uc};
        Cl.put(v, s0);
        __syncthreads();
        const int sh = __builtin_ctz((unsigned)nx), ncx = Cl.nx;
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            if (!ok[k]) continue;
            const int i = p(k) >> sh, j = p(k) & (nx - 1);
            // the next coarse nodes for odd i or j, the same again for even ones
            const c128* a = s0 + WT_ROW + (i >> 1) * ncx + (j >> 1);
            const int dj = j & 1, di = (i & 1) * ncx;
            u[k] = u[k] + 0.25 * ((a[0] + a[di]) + (a[dj] + a[di + dj]));
        }
        __syncthreads();
    }
};

// The cycle on levels l0..L from a zero iterate, as the per-level host recursion runs
// it (no ADR correction here: l0 >= 3).  NPT: nodes of level l0 per thread.
template <int NPT>
__global__ __launch_bounds__(WT_THREADS) void k_wave_tail(TailWaveArgs a, BatchIdx bi) {
    const size_t o = bi.off();  // the level arrays of this problem (shifted where they are read)
    constexpr int LB = NPT * WT_THREADS + 2 * WT_ROW + 2;
    // levels below l0: g and u of their pre-smoothing, at most NPT / 4 * 4/3 * 1024 nodes each
    constexpr int ST = NPT == 1 ? 352 : 1376, SH = WT_THREADS + 2 * WT_ROW + 2;
    constexpr bool INSIDE = LB >= SH + 2 * ST;  // behind the part of s1 that those levels use
    __shared__ c128 s0[LB], s1[LB + (INSIDE ? 0 : 2 * ST)];
    c128* stash = s1 + (INSIDE ? SH : LB);
    const int tid = threadIdx.x;
    auto smooth = [&](int l) { return l != 3; };
    const TailWaveLevel& W0 = a.lv[a.l0];
    WtLevel<NPT> T0;
    T0.init(W0, o);
    c128 g0[NPT], u0[NPT];
    T0.load(W0, W0.g, o, g0);
#pragma unroll
    for (int k = 0; k < NPT; ++k) u0[k] = c128{};
    if (a.l0 == a.L) {
        T0.template cheb<true>(W0, o, a.cheb_coarse, g0, u0, s0, s1);
    } else {
        c128 g[1], u[1];
        const Geom& G1 = a.lv[a.l0 + 1].G;
        if (smooth(a.l0)) {
            T0.template cheb<true>(W0, o, a.cheb_pre, g0, u0, s0, s1);
            g[0] = T0.template restrict_to<true>(g0, u0, G1.nx, G1.ny, s0, s1);
        } else {
            g[0] = T0.template restrict_to<false>(g0, u0, G1.nx, G1.ny, s0, s1);
        }
        WtLevel<1> T;
        int at = 0;
        for (int l = a.l0 + 1; l < a.L; ++l) {  // descend (all of these are smoothed but level 3)
            const TailWaveLevel& W = a.lv[l];
            T.init(W, o);
            const Geom& Gc = a.lv[l + 1].G;
            u[0] = c128{};
            if (smooth(l)) T.template cheb<true>(W, o, a.cheb_pre, g, u, s0, s1);
            if (tid < T.N) {
                stash[at + tid] = g[0];
                stash[ST + at + tid] = u[0];
            }
            at += T.N;
            g[0] = smooth(l) ? T.template restrict_to<true>(g, u, Gc.nx, Gc.ny, s0, s1)
                             : T.template restrict_to<false>(g, u, Gc.nx, Gc.ny, s0, s1);
        }
        WtLevel<1> Cl;
        Cl.init(a.lv[a.L], o);
        Cl.template cheb<true>(a.lv[a.L], o, a.cheb_coarse, g, u, s0, s1);
        for (int l = a.L - 1; l > a.l0; --l) {  // ascend
            const TailWaveLevel& W = a.lv[l];
            const c128 uc = u[0];
            T.init(W, o);
            at -= T.N;
            g[0] = tid < T.N ? stash[at + tid] : c128{};
            u[0] = tid < T.N ? stash[ST + at + tid] : c128{};
            T.prolong_from(Cl, uc, u, s0);
            if (l != 3 || a.level3_literal) T.template cheb<false>(W, o, a.cheb_post, g, u, s0, s1);
            Cl = T;
        }
        T0.prolong_from(Cl, u[0], u0, s0);
        if (a.l0 != 3 || a.level3_literal) T0.template cheb<false>(W0, o, a.cheb_post, g0, u0, s0, s1);
    }
#pragma unroll
    for (int k = 0; k < NPT; ++k)
        if (T0.p(k) < T0.N) {
            if (W0.f64)
                bsh_one(o, (c128*)W0.u)[T0.p(k)] = u0[k];
            else
                bsh_one(o, (c64*)W0.u)[T0.p(k)] = ccast<float>(u0[k]);
        }
}

}  // namespace helm
