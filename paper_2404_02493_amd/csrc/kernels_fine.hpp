// Level 1 in two passes: the damped Jacobi sweep with the restriction of its residual, and the
// prolongation with the sweep that follows it.
//   k_fine_down   u1 = u + (w/d)(g - A u), rc = R (g - A u1)
//   k_fine_up     out = v + (w/d)(g - A v), v = u1 + P ec
// d = 4/h^2 - kappa the diagonal of A.  ZERO: the cycle starts from u = 0, where u1 = (w/d) g is
// recomputed by the second pass instead of stored.  A block owns a 32 x 32 tile; u, u1 and
// the residual pass through LDS on the tile and rings of up to three nodes.
// Launch bound on small grids, bound by vector issue on large ones (the rings recompute a
// third).  Measured, the four or (ZERO) two launches they replace -> both passes:
// nonzero start 256^2 20 -> 8.7 us, 1024^2 32 -> 19 us, 4096^2 395 -> 280 us (FP32), 1024^2
// FP64 44 -> 27 us; zero start 512^2 FP64 row marches 33 -> 10 us.  From 2048^2 up the zero
// start stays with the row marches of kernels_jac0.hpp (36 us there for both), which issue a
// third of the instructions once there are enough strips to hide their row-to-row latency.
#pragma once

#include "kernels_chebm.hpp"

namespace helm {

constexpr int FINE_FT = 32;
template <bool ZERO>
constexpr int FINE_DOWN = ZERO ? 640 : 704;
constexpr int FINE_UP = 640;

// (w / d) v at node k, by one reciprocal of |d|^2 (FP32: the hardware's, corrected once): a
// rounding more than by divisions.  Error of the two passes alone against FP64 from a nonzero start
// (512^2, FP32): 5.37e-8, with divisions 5.29e-8 (from zero 5.19e-8, where the row marches have
// 8.4e-8); a whole cycle's is 3e-7 to 6e-7.
template <typename R, typename T>
__device__ __forceinline__ cplx<T> fine_sweep(const R& F, int k, T w, cplx<T> v) {
    const T dr = T(4) * F.l[k] - F.kp[k].re, di = -F.kp[k].im, D = dr * dr + di * di;
    T r;
    if constexpr (sizeof(T) == 4) {
        r = __builtin_amdgcn_rcpf(D);
        r = fma(fma(-D, r, T(1)), r, r);
    } else {
        r = T(1) / D;
    }
    const T s = w * r;
    return mk<T>(s * fma(v.re, dr, v.im * di), s * fma(v.im, dr, -(v.re * di)));
}

// rc on the coarse grid (every node) and, unless ZERO, u1 on the fine one;
// fuse_tiles(G.nx, G.ny, FINE_FT) blocks.
template <typename T, typename Tc, bool ZERO>
__global__ __launch_bounds__(FINE_DOWN<ZERO>) void k_fine_down(Geom G, const T* __restrict__ n2,
                                                               const cplx<T>* __restrict__ g,
                                                               const cplx<T>* __restrict__ uin,
                                                               const double* __restrict__ wp, cplx<T>* __restrict__ u1,
                                                               cplx<Tc>* __restrict__ rc, BatchIdx bi) {
    bshift(bi.off(), n2, g, uin, wp, u1, rc);
    // u1 one node before the tile and two behind it, u one more
    constexpr int LO = ZERO ? 1 : 2, FT = FINE_FT, RW = FT + 2 * LO + 1, FB = FINE_DOWN<ZERO>, TC = FT / 2;
    using R = ChebReg<T, RW, FB>;
    __shared__ cplx<T> buf[2 * R::LB];
    cplx<T>* s0 = buf;
    cplx<T>* s1 = buf + R::LB;
    const T w = T(wp[0]);
    int ti, tj;
    tile_index(fuse_side(G.nx, FT), ti, tj);
    const int i0 = 1 + ti * FT - LO, j0 = 1 + tj * FT - LO;
    R F;
    F.place(G, i0, j0);
    cplx<T> gv[R::NPT], u[R::NPT];
    T nv[R::NPT];
    F.load(g, gv);
    F.load(n2, nv);
    if constexpr (!ZERO) F.load(uin, u);
    fuse_ring(rc, G.nx / 2, G.ny / 2, ti, tj, TC);
    if constexpr (!ZERO) fuse_ring(u1, G.nx, G.ny, ti, tj, FT);
    F.coefs(G, nv, i0, j0);
    if constexpr (!ZERO) {
        R::put(u, s0);
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < R::NPT; ++k) {
        cplx<T> v;
        if constexpr (ZERO)
            v = fine_sweep(F, k, w, gv[k]);
        else
            v = u[k] + fine_sweep(F, k, w, gv[k] - F.template apply<false>(s0, k));
        u[k] = F.ok[k] ? v : cplx<T>{};
        if constexpr (!ZERO)
            if (R::in(k, LO, LO + FT - 1) && F.ok[k]) st_off(u1, F.p[k], v);
    }
    R::put(u, s1);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < R::NPT; ++k) s0[R::S0 + R::q(k)] = gv[k] - F.template apply<false>(s1, k);
    __syncthreads();
    const int ncx = G.nx / 2, ncy = G.ny / 2;
    for (int q = threadIdx.x; q < TC * TC; q += FB) {
        const int ci = q / TC, cj = q - ci * TC;
        const int I = 1 + ti * TC + ci, J = 1 + tj * TC + cj;
        if (I >= ncy || J >= ncx) continue;
        const cplx<T>* a = s0 + R::S0 + (2 * ci + 1 + LO) * RW + 2 * cj + 1 + LO;
        const cplx<T> ud = ((a[-RW] + a[RW]) + a[-1]) + a[1];
        const cplx<T> dg = ((a[-RW - 1] + a[-RW + 1]) + a[RW - 1]) + a[RW + 1];
        rc[(size_t)I * ncx + J] = ccast<Tc>(T(1.0 / 16.0) * ((T(4) * a[0] + T(2) * ud) + dg));
    }
}

// out on every fine node (0 on the ring); out must not overlap g or u1.
// fuse_tiles(G.nx, G.ny, FINE_FT) blocks.
template <typename T, typename Tc, bool ZERO>
__global__ __launch_bounds__(FINE_UP) void k_fine_up(Geom G, const T* __restrict__ n2, const cplx<T>* __restrict__ g,
                                                     const cplx<T>* __restrict__ u1, const cplx<Tc>* __restrict__ ec,
                                                     const double* __restrict__ wp, cplx<T>* __restrict__ out,
                                                     BatchIdx bi) {
    bshift(bi.off(), n2, g, u1, ec, wp, out);
    constexpr int LO = 1, FT = FINE_FT, RW = FT + 2 * LO, FB = FINE_UP;
    constexpr int RC = RW / 2 + 1;  // coarse nodes under the region, from FT ti / 2
    using R = ChebReg<T, RW, FB>;
    __shared__ cplx<T> s0[R::LB];
    __shared__ cplx<Tc> sc[RC * RC];
    const T w = T(wp[0]);
    int ti, tj;
    tile_index(fuse_side(G.nx, FT), ti, tj);
    const int i0 = 1 + ti * FT - LO, j0 = 1 + tj * FT - LO;  // even
    const int I0 = i0 >> 1, J0 = j0 >> 1, ncx = G.nx / 2, ncy = G.ny / 2;
    R F;
    F.place(G, i0, j0);
    cplx<T> gv[R::NPT], u[R::NPT];
    T nv[R::NPT];
    F.load(g, gv);
    F.load(n2, nv);
    if constexpr (!ZERO) F.load(u1, u);
    for (int q = threadIdx.x; q < RC * RC; q += FB) {
        const int I = I0 + q / RC, J = J0 + q % RC;
        const bool in = I >= 1 && J >= 1 && I < ncy && J < ncx;
        sc[q] = ec[in ? (size_t)I * ncx + J : 0];
    }
    fuse_ring(out, G.nx, G.ny, ti, tj, FT);
    F.coefs(G, nv, i0, j0);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < R::NPT; ++k) {
        // between the coarse nodes (gi / 2, gj / 2) and, for odd gi or gj, the next ones; for
        // even ones the same again, so the mean of four is exact
        const int gi = i0 + R::row(k), gj = j0 + R::col(k);
        const int l = F.ok[k] ? ((gi >> 1) - I0) * RC + (gj >> 1) - J0 : 0;
        const int dj = gj & 1, di = (gi & 1) * RC;
        const cplx<T> e = ccast<T>(Tc(0.25) * ((sc[l] + sc[l + di]) + (sc[l + dj] + sc[l + di + dj])));
        if constexpr (ZERO) u[k] = fine_sweep(F, k, w, gv[k]);
        u[k] = F.ok[k] ? u[k] + e : cplx<T>{};
    }
    R::put(u, s0);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < R::NPT; ++k)
        if (R::in(k, LO, LO + FT - 1) && F.ok[k])
            st_off(out, F.p[k], u[k] + fine_sweep(F, k, w, gv[k] - F.template apply<false>(s0, k)));
}

}  // namespace helm
