// Travel-time phase on the device: the factored eikonal equation (Section 3.2.1).
//
// tau = tau0 tau1 with tau0 = |x - x0|, the exact solution for unit slowness
// (eq. eikonal_cons), and tau1 from |tau0 grad tau1 + tau1 grad tau0|^2 = s^2.
// Discretisation: the first-order Godunov upwind form on the fine nodes with grad tau0
// exact.  Per axis the neighbour of smaller tau is upwind; with sgn = +1 for the
// west/south one and -1 for the east/north one the discrete derivative of tau is
// a t - b with a = sgn r/h + g, b = sgn r tau1(q)/h (r = tau0, g = grad tau0,
// t = tau1 at the node).  Candidates: both axes ((a_x t - b_x)^2 + (a_y t - b_y)^2
// = s^2, larger root, kept if upwind on both axes), and each axis alone
// (sgn (a t - b) = s); the smallest one replaces tau1 if it is smaller.  Nodes
// within sqrt(2) h of the source are fixed at the straight-ray mean slowness.
//
// Fast sweeping: Gauss-Seidel passes in the four orders (i up, j up), (i up, j down),
// (i down, j up), (i down, j down).  A pass runs as a wavefront over B x B tiles
// (B = 64, or the shorter side when smaller; B divides both sides): the tiles of one
// anti-diagonal (in the pass's orientation) are independent, one block per tile; inside a
// tile one wavefront walks the node anti-diagonals, lane l holding row l of the tile.  A
// node then sees exactly the values the sequential pass would give it (updated neighbours
// behind it, old ones ahead), so every pass equals the sequential one; the local
// update rounds every operation separately (no contraction; quotients by h = 2^-m
// are the exact products by 1/h), so the result is the same double precision numbers
// as a sequential implementation of the same steps.
// The two passes with the same direction of i run together, the second one Tx + 1 tile
// diagonals behind the first: it then meets only tiles whose neighbours the first has
// finished, and never a neighbour that the first still has to read (2 Tx + Ty launches for
// the pair instead of 2 (Tx + Ty - 1)).
#pragma once

#include "kernels_sstep.hpp"

namespace helm {

struct EikSrc {
    int nx, ny;  // nodes per row / per column of the fine grid, h = 1 / max(nx, ny)
    double h, xs, ys;
    double rfix;  // nodes with r <= rfix are fixed
};

__device__ __forceinline__ double eik_r(const EikSrc& E, int i, int j) {
#pragma clang fp contract(off)
    const double dx = double(j) * E.h - E.xs;
    const double dy = double(i) * E.h - E.ys;
    return sqrt(dx * dx + dy * dy);
}

// New tau1 at a node that is not fixed: rn = tau0 / h there, (gx, gy) = grad tau0, sp = s,
// from the neighbour values tw, te, ts, tn (+inf where missing or not reached yet) and
// their tau0 values rw, re, rs, rm (south, north); +inf when no candidate exists.  The sign
// sgn = +-1 of the chosen neighbour is taken out of the axis's a and b (sgn a = rn + sgn g and
// sgn b = rn t(q)): every product and quotient that they enter holds the sign twice or is
// compared with its sign, and a change of sign rounds nothing.
__device__ __forceinline__ double eik_update(double rn, double gx, double gy, double sp, double tw, double te,
                                             double ts, double tn, double rw, double re, double rs, double rm) {
#pragma clang fp contract(off)
    const double inf = __builtin_huge_val();
    // a missing neighbour (+inf) is never the smaller one; of equal ones west and south
    const bool east = re * te < rw * tw, north = rm * tn < rs * ts;
    const double ux = east ? te : tw, uy = north ? tn : ts;
    const double ax = east ? rn - gx : rn + gx, ay = north ? rn - gy : rn + gy;
    const bool hx = ux < inf, hy = uy < inf;
    const double bx = rn * ux, by = rn * uy;
    const double A = ax * ax + ay * ay, B = ax * bx + ay * by, C = (bx * bx + by * by) - sp * sp;
    const double disc = B * B - A * C;
    const double t2 = (B + sqrt(disc)) / A;  // NaN or unused unless both axes have a neighbour
    const double tx = (bx + sp) / ax, ty = (by + sp) / ay;
    double best = inf;
    if (hx && hy && A > 0.0 && disc >= 0.0 && ax * t2 - bx >= 0.0 && ay * t2 - by >= 0.0 && t2 < best) best = t2;
    if (hx && ax > 0.0 && tx < best) best = tx;
    if (hy && ay > 0.0 && ty < best) best = ty;
    return best;
}

// s = sqrt(n^2) on the fine nodes.
__global__ __launch_bounds__(BLOCK) void k_eik_slowness(size_t N, const double* __restrict__ n2,
                                                        double* __restrict__ s) {
    for (size_t p = blockIdx.x * (size_t)BLOCK + threadIdx.x; p < N; p += (size_t)gridDim.x * BLOCK)
        s[p] = sqrt(n2[p]);
}

// tau1 = (s(node) + s(src node)) / 2 on the fixed nodes, +inf elsewhere.
__global__ __launch_bounds__(BLOCK) void k_eik_init(EikSrc E, const double* __restrict__ s, size_t psrc,
                                                    double* __restrict__ t1) {
    const size_t N = (size_t)E.nx * E.ny;
    const double ssrc = s[psrc];
    for (size_t p = blockIdx.x * (size_t)BLOCK + threadIdx.x; p < N; p += (size_t)gridDim.x * BLOCK) {
        int i, j;
        rowcol(p, E.nx, i, j);
        t1[p] = eik_r(E, i, j) <= E.rfix ? (s[p] + ssrc) / 2.0 : __builtin_huge_val();
    }
}

// One tile of the pass (IUP, JUP): tile (I, J) of the pass's orientation
// (a = IUP ? i : ny-1-i, b = JUP ? j : nx-1-j); EIK_TB threads, B divides nx and ny.
// part[tile] (tile in grid orientation, nx / B tiles per row) keeps the largest single
// decrease of tau1 in the round.
// Bound by the issue of the node chain: 2 B - 1 dependent updates of one wavefront.  So all
// threads first stage tau1 and its geometry (tau0 and grad tau0, two divisions and a square
// root a node) in LDS, and the chain keeps the neighbours behind a node in registers (its own
// last value; the lane before it), reads everything ahead one step early and has no
// barrier.  s is read from global memory PF steps early (with it the LDS would be full).
constexpr int EIK_TB = 256;
template <int B>
struct EikLds {
    static constexpr int R = B + 2;
    double tl[R * R + 8];  // tau1 of the tile and its halo (the margin is read, not used)
    double rl[R * R + 8];  // tau0 there
    double gx[B * B + B], gy[B * B + B];
};
template <int B, bool IUP, bool JUP>
__device__ __forceinline__ void eik_tile(const EikSrc& E, const double* __restrict__ s, double* __restrict__ t1, int I,
                                         int J, double* __restrict__ part, EikLds<B>& L) {
    constexpr int R = EikLds<B>::R, PF = 8;
    const int n = E.nx, ny = E.ny, Tx = n / B, Ty = ny / B;
    const int a0 = I * B, b0 = J * B;
    const double inf = __builtin_huge_val();
    auto gi = [&](int a) { return IUP ? a : ny - 1 - a; };
    auto gj = [&](int b) { return JUP ? b : n - 1 - b; };
    for (int q = threadIdx.x; q < R * R; q += EIK_TB) {
        const int la = q / R - 1, lb = q % R - 1;
        const int a = a0 + la, b = b0 + lb;
        const bool in = a >= 0 && a < ny && b >= 0 && b < n;
        L.tl[q] = in ? t1[(size_t)gi(a) * n + gj(b)] : inf;
        const double r = in ? eik_r(E, gi(a), gj(b)) : 1.0;  // off the grid: 1.0 * inf, never the smaller
        L.rl[q] = r;
        if (la >= 0 && la < B && lb >= 0 && lb < B) {
#pragma clang fp contract(off)
            L.gx[la * B + lb] = (double(gj(b)) * E.h - E.xs) / r;
            L.gy[la * B + lb] = (double(gi(a)) * E.h - E.ys) / r;
        }
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const double nh = double(n > ny ? n : ny);
        const int la = threadIdx.x < B ? (int)threadIdx.x : B - 1;
        const bool row = threadIdx.x < B;
        // at step k this lane is at column k - la; LDS positions of column 0 of its row
        double* tl = L.tl + (la + 1) * R + 1 - la;
        const double* rl = L.rl + (la + 1) * R + 1 - la;
        const double* gxl = L.gx + la * B - la;
        const double* gyl = L.gy + la * B - la;
        const double* srow = s + (size_t)gi(a0 + la) * n;
        auto s_at = [&](int k) {  // s at step k (any column of the row where the lane is not in the tile)
            const int lb = k - la;
            return srow[gj(b0 + (lb < 0 ? 0 : lb >= B ? B - 1 : lb))];
        };
        double sv[PF];
#pragma unroll
        for (int q = 0; q < PF; ++q) sv[q] = s_at(q);
        double tp = tl[-1], tc = tl[0], tx = tl[1];  // tau1 behind (updated), at and ahead of the node
        double rp = rl[-1], rc = rl[0], rx = rl[1];
        double tb = tl[-R], ta = tl[R], rb = rl[-R], ra = rl[R], gx = gxl[0], gy = gyl[0];
        double dmax = 0.0;
        // 2 B - 1 steps, rounded up to PF (no lane is in the tile in the last one)
        for (int k0 = 0; k0 < 2 * B; k0 += PF) {
#pragma unroll
            for (int q = 0; q < PF; ++q) {
                const int k = k0 + q;
                // everything ahead of the next node, none of it written before the next step
                const double txn = tl[k + 2], tbn = tl[k + 1 - R], tan = tl[k + 1 + R];
                const double rxn = rl[k + 2], rbn = rl[k + 1 - R], ran = rl[k + 1 + R];
                const double gxn = gxl[k + 1], gyn = gyl[k + 1];
                const double sp = sv[q];
                sv[q] = s_at(k + PF);
                // behind in the other axis: the last value of the lane before (row -1: the halo)
                const double tprev = lane_prev(tp);
                const double tbr = la == 0 ? tb : tprev;
                const double t = eik_update(rc * nh, gx, gy, sp, JUP ? tp : tx, JUP ? tx : tp, IUP ? tbr : ta,
                                            IUP ? ta : tbr, JUP ? rp : rx, JUP ? rx : rp, IUP ? rb : ra,
                                            IUP ? ra : rb);
                const int lb = k - la;
                const bool on = row && lb >= 0 && lb < B;
                if (on && rc > E.rfix && t < tc) {
                    const double dec = tc - t;  // +inf for a node not reached before
                    dmax = dec > dmax ? dec : dmax;
                    tl[k] = t;
                    tc = t;
                }
                tp = tc;  // off the tile: what lies to the left of the next node
                tc = tx;
                tx = txn;
                rp = rc;
                rc = rx;
                rx = rxn;
                tb = tbn;
                ta = tan;
                rb = rbn;
                ra = ran;
                gx = gxn;
                gy = gyn;
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double o = __shfl_xor(dmax, off, 64);
            dmax = o > dmax ? o : dmax;
        }
        if (threadIdx.x == 0) {
            const int ti = IUP ? I : Ty - 1 - I, tj = JUP ? J : Tx - 1 - J;
            double* pp = part + (size_t)ti * Tx + tj;
            *pp = dmax > *pp ? dmax : *pp;
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < B * B; q += EIK_TB)
        t1[(size_t)gi(a0 + q / B) * n + gj(b0 + q % B)] = L.tl[(q / B + 1) * R + q % B + 1];
}

// Anti-diagonal d1 of the pass (IUP, j up) in the first n1 blocks, d2 of the pass
// (IUP, j down) in the others.
template <int B, bool IUP>
__global__ __launch_bounds__(EIK_TB) void k_eik_pass(EikSrc E, const double* __restrict__ s, double* __restrict__ t1,
                                                     int d1, int n1, int d2, double* __restrict__ part) {
    __shared__ EikLds<B> L;
    const int Tx = E.nx / B;
    const bool first = (int)blockIdx.x < n1;
    const int d = first ? d1 : d2, x = first ? (int)blockIdx.x : (int)blockIdx.x - n1;
    const int I = (d < Tx ? 0 : d - Tx + 1) + x;
    if (first)
        eik_tile<B, IUP, true>(E, s, t1, I, d - I, part, L);
    else
        eik_tile<B, IUP, false>(E, s, t1, I, d - I, part, L);
}

// out[block] = max of the block's share of x[0..N) and of 0 (blocks of 1024 threads; maxima
// are exact in any order).
__global__ __launch_bounds__(1024) void k_eik_max(size_t N, const double* __restrict__ x, double* __restrict__ out) {
    __shared__ double sm[1024];
    double m = 0.0;
    for (size_t p = (size_t)blockIdx.x * 1024 + threadIdx.x; p < N; p += (size_t)gridDim.x * 1024)
        m = x[p] > m ? x[p] : m;
    sm[threadIdx.x] = m;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sm[threadIdx.x] = sm[threadIdx.x + w] > sm[threadIdx.x] ? sm[threadIdx.x + w] : sm[threadIdx.x];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = sm[0];
}

// phi = min(phi, tau0 tau1) (first arrival over the sources).
__global__ __launch_bounds__(BLOCK) void k_eik_phase(EikSrc E, const double* __restrict__ t1,
                                                     double* __restrict__ phi) {
    const size_t N = (size_t)E.nx * E.ny;
    for (size_t p = blockIdx.x * (size_t)BLOCK + threadIdx.x; p < N; p += (size_t)gridDim.x * BLOCK) {
        int i, j;
        rowcol(p, E.nx, i, j);
        const double v = eik_r(E, i, j) * t1[p];
        phi[p] = v < phi[p] ? v : phi[p];
    }
}

}  // namespace helm

namespace helm {

// ADR coefficients of one level from tau1 (fine, FP64) of the source (xs, ys) with the
// product rule of Section 3.2.1: with tau0 = r = |x - x0|, grad tau0 = (x - x0)/r and
// Lap tau0 = 1/r exact and the finite-difference rule applied to tau1,
//   grad phi = r grad tau1 + tau1 grad tau0,
//   Lap phi  = tau1 / r + 2 grad tau0 . grad tau1 + r Lap tau1;
// at nodes closer than one level spacing to the source the rule is applied to
// phi = r tau1 itself.  car (level 2 only, may be null): the carrier of phi.
template <typename T>
__global__ __launch_bounds__(BLOCK) void k_adr_coef_fac(Geom G, const double* __restrict__ n2f,
                                                        const double* __restrict__ tau1, double xs, double ys,
                                                        double k, int sigma, double strength,
                                                        T* __restrict__ px_out, T* __restrict__ py_out,
                                                        cplx<T>* __restrict__ c0_out, cplx<T>* __restrict__ car_out) {
    const int nx = G.nx, ny = G.ny, s = G.s, nfx = G.nfx;
    const size_t N = (size_t)nx * ny;
    const double h = 1.0 / (nx > ny ? nx : ny);
    auto R = [&](int a, int b) -> double {
        const double dx = double(b) * h - xs, dy = double(a) * h - ys;
        return sqrt(dx * dx + dy * dy);
    };
    auto T1 = [&](int a, int b) -> double { return tau1[(size_t)a * s * nfx + (size_t)b * s]; };
    auto PHI = [&](int a, int b) -> double { return R(a, b) * T1(a, b); };
    for (size_t p = blockIdx.x * (size_t)BLOCK + threadIdx.x; p < N; p += (size_t)gridDim.x * BLOCK) {
        int i, j;
        rowcol(p, nx, i, j);
        if (car_out) car_out[p] = adr_carrier<T>(PHI(i, j), k, sigma);
        if (i == 0 || j == 0) {
            px_out[p] = T(0);
            py_out[p] = T(0);
            c0_out[p] = cplx<T>{};
            continue;
        }
        double px, py, lap;
        const double r = R(i, j);
        if (r < h) {
            fd_phase_rule(PHI, i, j, nx, ny, h, px, py, lap);
        } else {
            double t1x, t1y, t1l;
            fd_phase_rule(T1, i, j, nx, ny, h, t1x, t1y, t1l);
            const double gx = (double(j) * h - xs) / r, gy = (double(i) * h - ys) / r;
            const double t1 = T1(i, j);
            px = r * t1x + t1 * gx;
            py = r * t1y + t1 * gy;
            lap = t1 / r + 2.0 * (gx * t1x + gy * t1y) + r * t1l;
        }
        adr_coef_store<T>(G, n2f, i, j, p, px, py, lap, k, sigma, strength, px_out, py_out, c0_out);
    }
}

}  // namespace helm
