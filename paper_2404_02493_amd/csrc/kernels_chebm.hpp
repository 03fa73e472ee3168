// Whole Chebyshev smoothing of a wave level in one pass, with the transfer beside it:
//   k_cheb_down   u = Chebyshev(0, g), rc = R (g - A u)   (pre-smoothing, restriction)
//   k_cheb_up     u = Chebyshev(u_in + P ec, g)           (prolongation, post-smoothing)
// up to CHEBM = 5 steps (the iteration of chebyshev(): r = A^*(g - A u), d = r / theta, then
// u += d, r -= A^* A d, d = c1 d + c2 r).  A block loads g, n^2 (and u, ec) on an FT x FT
// tile and the rings that the steps use up, two nodes a step, keeps u, r, d and
// kappa in registers and exchanges d and A d through two LDS buffers; g is read
// and u written once instead of six arrays a step, and a smoothing is one launch instead
// of five.  As in kernels_adrfuse.hpp nothing carries a condition: off the unknowns the
// stencil's factors are 0, and what the region's border makes of its missing neighbours
// never reaches a value that is used.
// Bound by the issue of vector instructions, LDS accesses and barriers, not by bytes, so the
// threads own only the nodes that the steps need: those that r = A^*(g - A u) alone reads go
// through LDS once.  Measured: 7.1-8 us a smoothing on up to 256^2 (7.6-8.3 with threads on
// those nodes too), 14 us on 512^2, and on 1024^2 in FP32, where 64 x 64 tiles are one wave of
// blocks and the 62 x 62 that fitted before were two, 40 -> 24 us down and 43 -> 26 us up.
#pragma once

#include "kernels_adrfuse.hpp"

namespace helm {

constexpr int CHEBM = 5;  // most steps of one pass

// Threads per block by tile edge: the fewest slots on the fullest SIMD that the region of the
// steps leaves (FT + 19 nodes a side down, FT + 16 up), from eight wavefronts on.  k_cheb_down
// at 16 x 16 with four wavefronts of five nodes a thread took 9.8 us (11 of two: 7.9).
template <int FT>
struct ChebCfg {
    static constexpr int DOWN = FT <= 32 ? 704 : 1024;
    static constexpr int UP = FT == 16 ? 512 : FT == 32 ? 768 : 1024;
};

// A v (CJ: A^* v) at the node that a points to in rows of W; kp: kappa, l: 1/h^2, both 0 off
// the unknowns.
template <bool CJ, int W, typename T>
__device__ __forceinline__ cplx<T> cheb_apply(const cplx<T>* a, T l, cplx<T> kp) {
    const cplx<T> c = a[0];
    const cplx<T> nb = ((a[-W] + a[W]) + a[-1]) + a[1];
    const cplx<T> s4 = mk<T>(fma(T(4), c.re, -nb.re), fma(T(4), c.im, -nb.im));
    const T ki = CJ ? -kp.im : kp.im;
    return mk<T>(fma(l, s4.re, fma(ki, c.im, -(kp.re * c.re))), fma(l, s4.im, -fma(ki, c.re, kp.re * c.im)));
}

// A region of RW x RW nodes (arithmetic type T) of a wave level from node (i0, j0), thread t owning the nodes
// t, t + FB, ...
template <typename T, int RW, int FB>
struct ChebReg {
    static constexpr int N = RW * RW, NPT = (N + FB - 1) / FB;
    static constexpr int S0 = RW + 1, LB = NPT * FB + 2 * S0;  // node 0 in an LDS buffer; its size
    // kappa and 1/h^2, both 0 off the unknowns.  The Laplacian keeps 4 c - sum before it is
    // scaled: folded into one diagonal 4/h^2 - kappa the rounding of that diagonal is a
    // relative error of ten times the precision in kappa, the same at every application.
    cplx<T> kp[NPT];
    T l[NPT];
    bool ok[NPT];
    unsigned p[NPT];
    __device__ __forceinline__ static int q(int k) { return (int)threadIdx.x + k * FB; }
    __device__ __forceinline__ static int row(int k) { return (int)((unsigned)q(k) / (unsigned)RW); }
    __device__ __forceinline__ static int col(int k) { return q(k) - row(k) * RW; }
    __device__ __forceinline__ static bool in(int k, int lo, int hi) {
        return (unsigned)(row(k) - lo) <= (unsigned)(hi - lo) && (unsigned)(col(k) - lo) <= (unsigned)(hi - lo);
    }
    __device__ __forceinline__ void place(const Geom& G, int i0, int j0) {
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int gi = i0 + row(k), gj = j0 + col(k);
            ok[k] = q(k) < N && gi >= 1 && gi < G.ny && gj >= 1 && gj < G.nx;
            p[k] = ok[k] ? (unsigned)(gi * G.nx + gj) : 0u;
        }
    }
    template <typename S>
    __device__ __forceinline__ void load(const cplx<S>* __restrict__ a, cplx<T> (&v)[NPT]) const {
#pragma unroll
        for (int k = 0; k < NPT; ++k) v[k] = ccast<T>(ld_off(a, p[k]));
    }
    template <typename S>
    __device__ __forceinline__ void load(const S* __restrict__ a, T (&v)[NPT]) const {
#pragma unroll
        for (int k = 0; k < NPT; ++k) v[k] = T(ld_off(a, p[k]));
    }
    __device__ __forceinline__ void coefs(const Geom& G, const T (&n2)[NPT], int i0, int j0) {
        const T ih2 = T(G.inv_h2);
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const cplx<T> kap = kappa_at<T>(G, n2[k], i0 + row(k), j0 + col(k));
            l[k] = ok[k] ? ih2 : T(0);
            kp[k] = ok[k] ? kap : cplx<T>{};
        }
    }
    __device__ __forceinline__ static void put(const cplx<T> (&v)[NPT], cplx<T>* s) {
#pragma unroll
        for (int k = 0; k < NPT; ++k) s[S0 + q(k)] = v[k];
    }
    // A s (CJ: A^* s) at node k
    template <bool CJ>
    __device__ __forceinline__ cplx<T> apply(const cplx<T>* s, int k) const {
        return cheb_apply<CJ, RW>(s + S0 + q(k), l[k], kp[k]);
    }
    // A^* s at node k from a buffer that holds D more nodes on every side, node 0 at s
    template <int D>
    __device__ __forceinline__ cplx<T> apply_start(const cplx<T>* s, int k) const {
        constexpr int W = RW + 2 * D;
        return cheb_apply<true, W>(s + (row(k) + D) * W + col(k) + D, l[k], kp[k]);
    }
    // The m Chebyshev steps from r = A^*(g - A u): u, r, d in registers, d and A d through s0
    // and s1 (s0 must be free to write, s1 after one more barrier); on return s0 is free.
    __device__ __forceinline__ void steps(const double* __restrict__ cc, int m, cplx<T> (&u)[NPT], cplx<T> (&r)[NPT],
                                          cplx<T>* s0, cplx<T>* s1) const {
        cplx<T> d[NPT];
        const T inv_theta = T(cc[0]);
#pragma unroll
        for (int k = 0; k < NPT; ++k) d[k] = inv_theta * r[k];
#pragma unroll 1
        for (int step = 1; step < m; ++step) {
            const T c1 = T(cc[3 * step + 1]), c2 = T(cc[3 * step + 2]);
            put(d, s0);
            __syncthreads();
            cplx<T> t[NPT];
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
    }
};

// u = m Chebyshev steps from 0 for A u = g (every node of u written, 0 on the ring) and
// rc = R (g - A u) on the coarse grid; fuse_tiles(G.nx, G.ny, FT) blocks, m <= CHEBM.
template <typename S, typename Tc, int FT, typename T>
__global__ __launch_bounds__(ChebCfg<FT>::DOWN) void k_cheb_down(Geom G, const S* __restrict__ n2,
                                                                 const cplx<S>* __restrict__ g,
                                                                 cplx<S>* __restrict__ uout, cplx<Tc>* __restrict__ rc,
                                                                 const double* __restrict__ cc, int m, BatchIdx bi) {
    bshift(bi.off(), n2, g, uout, rc, cc);
    // u is needed one node before the tile and two behind it (the residual on the tile and one
    // node behind); the steps use up 2 (CHEBM - 1) more, and r = A^* g one more of g
    constexpr int LO = 1 + 2 * (CHEBM - 1), RW = FT + 2 * LO + 1, FB = ChebCfg<FT>::DOWN, TC = FT / 2;
    constexpr int OW = RW + 2, NO = (OW * OW + FB - 1) / FB;
    using R = ChebReg<T, RW, FB>;
    constexpr int GB = OW * OW > R::LB ? OW * OW : R::LB;
    __shared__ cplx<T> buf[R::LB + GB];
    cplx<T>* s0 = buf;
    cplx<T>* s1 = buf + R::LB;
    int ti, tj;
    tile_index(fuse_side(G.nx, FT), ti, tj);
    const int i0 = 1 + ti * FT - LO, j0 = 1 + tj * FT - LO;
    R F;
    F.place(G, i0, j0);
    cplx<T> u[R::NPT], r[R::NPT];
    {
        cplx<T> gv[NO];
        T nv[R::NPT];
#pragma unroll
        for (int k = 0; k < NO; ++k) {
            const int q = (int)threadIdx.x + k * FB;
            const int gi = i0 - 1 + (int)((unsigned)q / (unsigned)OW), gj = j0 - 1 + (int)((unsigned)q % (unsigned)OW);
            const bool in = q < OW * OW && gi >= 1 && gi < G.ny && gj >= 1 && gj < G.nx;
            gv[k] = ccast<T>(ld_off(g, in ? (unsigned)(gi * G.nx + gj) : 0u));
        }
        F.load(n2, nv);
        fuse_ring(uout, G.nx, G.ny, ti, tj, FT);
        fuse_ring(rc, G.nx / 2, G.ny / 2, ti, tj, TC);
#pragma unroll
        for (int k = 0; k < NO; ++k) {
            const int q = (int)threadIdx.x + k * FB;
            if (q < OW * OW) s1[q] = gv[k];
        }
        F.coefs(G, nv, i0, j0);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < R::NPT; ++k) {
        u[k] = cplx<T>{};
        r[k] = R::q(k) < R::N ? F.template apply_start<1>(s1, k) : cplx<T>{};
    }
    F.steps(cc, m, u, r, s0, s1);
    R::put(u, s0);
    cplx<T> gv[R::NPT];
    F.load(g, gv);
#pragma unroll
    for (int k = 0; k < R::NPT; ++k)
        if (R::in(k, LO, LO + FT - 1) && F.ok[k]) st_off(uout, F.p[k], ccast<S>(u[k]));
    __syncthreads();
#pragma unroll
    for (int k = 0; k < R::NPT; ++k) s1[R::S0 + R::q(k)] = gv[k] - F.template apply<false>(s0, k);
    __syncthreads();
    const int ncx = G.nx / 2, ncy = G.ny / 2;
    for (int q = threadIdx.x; q < TC * TC; q += FB) {
        const int ci = q / TC, cj = q - ci * TC;
        const int I = 1 + ti * TC + ci, J = 1 + tj * TC + cj;
        if (I >= ncy || J >= ncx) continue;
        // fine centre (2I, 2J) at region row 2I - i0 = 2 ci + 1 + LO
        const cplx<T>* a = s1 + R::S0 + (2 * ci + 1 + LO) * RW + 2 * cj + 1 + LO;
        const cplx<T> ud = ((a[-RW] + a[RW]) + a[-1]) + a[1];
        const cplx<T> dg = ((a[-RW - 1] + a[-RW + 1]) + a[RW - 1]) + a[RW + 1];
        rc[(size_t)I * ncx + J] = ccast<Tc>(T(1.0 / 16.0) * ((T(4) * a[0] + T(2) * ud) + dg));
    }
}

// uout = m Chebyshev steps from u_in + P ec for A u = g (every node written, 0 on the ring);
// fuse_tiles(G.nx, G.ny, FT) blocks, m <= CHEBM; uout must not overlap uin.
template <typename S, typename Tc, int FT, typename T>
__global__ __launch_bounds__(ChebCfg<FT>::UP) void k_cheb_up(Geom G, const S* __restrict__ n2,
                                                             const cplx<S>* __restrict__ g,
                                                             const cplx<S>* __restrict__ uin,
                                                             const cplx<Tc>* __restrict__ ec, cplx<S>* __restrict__ uout,
                                                             const double* __restrict__ cc, int m, BatchIdx bi) {
    bshift(bi.off(), n2, g, uin, ec, uout, cc);
    // the steps use up 2 (CHEBM - 1) nodes; r = A^* (g - A u) takes two more of u
    constexpr int LO = 2 * (CHEBM - 1), RW = FT + 2 * LO, FB = ChebCfg<FT>::UP;
    constexpr int OW = RW + 4;
    constexpr int RC = OW / 2 + 1;  // coarse nodes under the outer region, from (its origin) / 2
    using R = ChebReg<T, RW, FB>;
    using RO = ChebReg<T, OW, FB>;
    static_assert(FT % 2 == 0 && RC * RC <= RO::LB && R::LB <= RO::LB, "coarse values in one buffer");
    __shared__ cplx<T> buf[2 * RO::LB];
    cplx<T>* s0 = buf;
    cplx<T>* s1 = buf + RO::LB;
    int ti, tj;
    tile_index(fuse_side(G.nx, FT), ti, tj);
    const int i0 = 1 + ti * FT - LO, j0 = 1 + tj * FT - LO;  // odd
    R F;
    F.place(G, i0, j0);
    cplx<T> u[R::NPT], r[R::NPT];
    T ni[R::NPT];
    {
        const int o0 = i0 - 2, q0 = j0 - 2;
        const int I0 = o0 >> 1, J0 = q0 >> 1, ncx = G.nx / 2, ncy = G.ny / 2;
        RO O;
        O.place(G, o0, q0);
        cplx<T> uo[RO::NPT], gv[RO::NPT];
        T nv[RO::NPT];
        O.load(uin, uo);
        O.load(g, gv);
        O.load(n2, nv);
        for (int q = threadIdx.x; q < RC * RC; q += FB) {
            const int I = I0 + q / RC, J = J0 + q % RC;
            const bool in = I >= 1 && J >= 1 && I < ncy && J < ncx;
            s1[q] = ccast<T>(ec[in ? (size_t)I * ncx + J : 0]);
        }
        F.load(n2, ni);
        fuse_ring(uout, G.nx, G.ny, ti, tj, FT);
        O.coefs(G, nv, o0, q0);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < RO::NPT; ++k) {
            // between the coarse nodes (gi / 2, gj / 2) and, for odd gi or gj, the next ones; for
            // even ones the same again, so the mean of four is exact
            const int gi = o0 + RO::row(k), gj = q0 + RO::col(k);
            const int l = O.ok[k] ? ((gi >> 1) - I0) * RC + (gj >> 1) - J0 : 0;
            const int dj = gj & 1, di = (gi & 1) * RC;
            const cplx<T> e = T(0.25) * ((s1[l] + s1[l + di]) + (s1[l + dj] + s1[l + di + dj]));
            uo[k] = O.ok[k] ? uo[k] + e : cplx<T>{};
        }
        RO::put(uo, s0);
        __syncthreads();
        cplx<T> t[RO::NPT];
#pragma unroll
        for (int k = 0; k < RO::NPT; ++k) t[k] = gv[k] - O.template apply<false>(s0, k);
        RO::put(t, s1);
    }
#pragma unroll
    for (int k = 0; k < R::NPT; ++k)
        u[k] = R::q(k) < R::N ? s0[RO::S0 + (R::row(k) + 2) * OW + R::col(k) + 2] : cplx<T>{};
    F.coefs(G, ni, i0, j0);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < R::NPT; ++k)
        r[k] = R::q(k) < R::N ? F.template apply_start<2>(s1 + RO::S0, k) : cplx<T>{};
    F.steps(cc, m, u, r, s0, s1);
#pragma unroll
    for (int k = 0; k < R::NPT; ++k)
        if (R::in(k, LO, LO + FT - 1) && F.ok[k]) st_off(uout, F.p[k], ccast<S>(u[k]));
}

}  // namespace helm
