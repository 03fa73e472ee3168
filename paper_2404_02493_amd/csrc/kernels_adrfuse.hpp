// ADR V-cycle levels whose passes are joined across a Gram pass: each kernel finishes one
// GMRES(3) smoother (its coefficients from the Gram sums of the kernel before), hands the
// result to the next operation of the V-cycle and forms the Gram sums of the smoother
// that follows, so an ADR step on levels 2..LA takes 2 (LA - 2) + 1 launches:
//   k_fuse_start  level 2: b = (g - A u) e^{-i theta}; Gram sums of the pre-smoother
//   k_fuse_down   level l: x = pre-smoother, b_{l+1} = R (b - M x); Gram sums on l + 1
//   k_fuse_up     level l: x += P x_{l+1}, x_{l+1} the finished smoother of level l + 1;
//                 Gram sums of the post-smoother on l
//   k_fuse_step   level 2: u += x e^{i theta}, x the finished post-smoother, and, unless it is
//                 the last ADR step, k_fuse_start of the next one
// On levels of a few hundred nodes per side a pass is bound by its launch, one memory
// round trip and the issue time of its vector instructions on the CUs that it occupies,
// so recomputing the rings that the next operation needs costs less than the launches
// that it saves.  Measured per kernel (FP32): 6-7 us on a 128^2 level 2, 9.5-12 us on
// 512^2 (one 32 x 32 tile per CU), about 4 us of either being launch and first loads; FP64 on
// 512^2 11-15 us.  A whole cycle, against separate Gram, solve, combination and transfer
// launches (15 a step instead of 5): 744 -> 385 us at 128^2 in FP64, 823 -> 395 us at 256^2,
// 942 -> 645 us at 1024^2 in FP32, 1068 -> 913 us there in FP64 (and 654 -> 550 us when, beside
// later steps elsewhere, the FP64 kernels stopped spilling).
//
// A block owns a tile of FTxFT nodes of the finer level (half of that on the coarser one)
// and builds the Krylov vectors as sstep_tile does, one vector per barrier in two LDS
// buffers, on the tile and the rings that the chain of operations needs.  Loads, LDS
// accesses and stencils carry no conditions: off the unknowns the fields are read at
// index 0 (the zero ring) and the stencil coefficients are 0, and a node at the region's
// border reads whatever lies beside its buffer; what it makes of it never reaches a value
// that is used, one application carrying it one node further into the rings.
#pragma once

#include "kernels_tail.hpp"

namespace helm {

// Up to this many partials every block of the consumer sums the Gram partials and solves
// the normal equations itself (at most 32 KiB of partials per block).
constexpr int FUSE_FOLD = 256;
// Up to this many blocks of all problems of a batch class together (five per CU) the levels
// are joined.  Beyond, the launches that joining saves no longer count and the rings that it
// recomputes do.  Twenty iterations of a class in ms, joined | separate passes, by its problems:
//   512^2 (256 tiles of 16 x 16)    3: 12.5 | 21.2   5: 18.4 | 23.8   8: 26.2 | 26.9   20: 59 | 41
//   1024^2 (256 tiles of 32 x 32)   3: 22.2 | 23.0   5: 34.4 | 31.7   8: 52.2 | 44.6   20: 130 | 100
//   256^2 (64 tiles of 16 x 16)     8: 10.4 | 17.6   20: 18.7 | about 20
// The two edges cross at about eight and between three and four problems; the one line lies
// between, at five of either.
constexpr int FUSE_SHARED = 1280;

__host__ __device__ inline int fuse_side(int m, int ft) { return (m - 2) / ft + 1; }
__host__ __device__ inline int fuse_tiles(int nx, int ny, int ft) { return fuse_side(nx, ft) * fuse_side(ny, ft); }

// Threads per block: as few idle ones as the region's nodes allow, at most 1024.  The vectors of
// DOWN and STEP on 32 x 32 tiles take 120-240 registers: eight wavefronts (two per SIMD, five
// and four nodes a thread) keep them free of spills (FP64 on 512^2: DOWN with 896 threads
// of three nodes spilled 36 registers, 21.3 us against 11.8; STEP with 768 spilled 20, 18.4
// against 15.2; FP32 the same within 0.3 us).
template <int FT>
struct FuseCfg;
template <>
struct FuseCfg<16> {
    static constexpr int DOWN = 640, UP = 576, START = 576, STEP = 960, LAST = 512;
};
template <>
struct FuseCfg<32> {
    static constexpr int DOWN = 512, UP = 832, START = 832, STEP = 512, LAST = 768;
};
template <>
struct FuseCfg<64> {  // k_fuse_up without Gram sums only
    static constexpr int UP = 768;
};

// The coefficients c_1..c_3 of the smoother that the previous kernel's ng Gram partials
// belong to (ng <= FUSE_FOLD): FuseSums adds them up (one wavefront per entry, a
// fixed order), fuse_coef_solve (after a barrier) solves in the last wavefront,
// fuse_coef_get (after another) reads.  sh: FUSE_SH doubles of LDS.
constexpr int FUSE_SH = 22;
// (the loads come first in a kernel, then those of its fields, then the sums: the
// coefficients are the longest chain of a pass)
template <int FB>
struct FuseSums {
    static constexpr int NW = FB / 64, R = (16 + NW - 1) / NW, SB = FUSE_FOLD / 64;
    double t[R][SB];
    __device__ __forceinline__ FuseSums(const double* __restrict__ part, int ng) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int v = wave + r * NW < 16 ? wave + r * NW : 15;
            const double* __restrict__ row = part + (size_t)v * ng;
#pragma unroll
            for (int k = 0; k < SB; ++k) {
                const int b = k * 64 + lane;
                const double x = row[b < ng ? b : 0];
                t[r][k] = b < ng ? x : 0.0;
            }
        }
    }
    __device__ __forceinline__ void sum(double* sh) const {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            double a = t[r][0];
#pragma unroll
            for (int k = 1; k < SB; ++k) a += t[r][k];
            const double s = wave_sum(a);
            if (lane == 0 && wave + r * NW < 16) sh[wave + r * NW] = s;
        }
    }
};
template <int FB>
__device__ __forceinline__ void fuse_coef_solve(double* sh) {
    if (threadIdx.x < FB - 64) return;
    double y[6];
    double beta;
    int cols;
    sstep_small_solve<3>(sh, 1e-12, y, cols, beta);
    if (threadIdx.x == FB - 1) {
#pragma unroll
        for (int q = 0; q < 6; ++q) sh[16 + q] = y[q];
    }
}
template <typename T>
__device__ __forceinline__ void fuse_coef_get(const double* sh, cplx<T> (&c)[3]) {
#pragma unroll
    for (int q = 0; q < 3; ++q) c[q] = mk<T>(T(sh[16 + 2 * q]), T(sh[17 + 2 * q]));
}

// The (RW + 2) x (RW + 2) nodes of a field from (i0 - 1, j0 - 1) for the first application of a
// chain: load() issues the loads, put() stores them in rows of RW + 2.  Its ring then takes no
// slot of the threads in the rest of the chain.
template <typename T, int RW, int FB>
struct FuseOuter {
    static constexpr int W = RW + 2, N = W * W, NPT = (N + FB - 1) / FB;
    cplx<T> v[NPT];
    __device__ __forceinline__ void load(const AdrGeom& A, const cplx<T>* __restrict__ a, int i0, int j0) {
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int q = (int)threadIdx.x + k * FB;
            const int gi = i0 - 1 + (int)((unsigned)q / (unsigned)W), gj = j0 - 1 + (int)((unsigned)q % (unsigned)W);
            const bool in = q < N && gi >= 1 && gi < A.ny && gj >= 1 && gj < A.nx;
            v[k] = ld_off(a, in ? (unsigned)(gi * A.nx + gj) : 0u);
        }
    }
    __device__ __forceinline__ void put(cplx<T>* s) const {
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int q = (int)threadIdx.x + k * FB;
            if (q < N) s[q] = v[k];
        }
    }
};

// A region of RW x RW nodes of a level whose node (0, 0) is (i0, j0), over FB threads: thread
// t owns region nodes t, t + FB, ...  LB: size of an LDS buffer (nodes and margins), S0 the
// index of node 0 in it.
template <typename T, int RW, int FB>
struct FuseReg {
    static constexpr int N = RW * RW, NPT = (N + FB - 1) / FB;
    static constexpr bool SPARE = N + 64 <= NPT * FB;  // whole wavefronts without a node
    static constexpr int S0 = RW + 1, LB = NPT * FB + 2 * S0;
    UpCoef<T> cf[NPT];
    bool ok[NPT];     // an unknown of the level
    unsigned p[NPT];  // its index (0 off the unknowns)
    __device__ __forceinline__ static int q(int k) { return (int)threadIdx.x + k * FB; }
    __device__ __forceinline__ static int row(int k) { return (int)((unsigned)q(k) / (unsigned)RW); }
    __device__ __forceinline__ static int col(int k) { return q(k) - row(k) * RW; }
    __device__ __forceinline__ static bool has(int k) { return !SPARE || q(k) < N; }
    __device__ __forceinline__ static bool in(int k, int lo, int hi) {  // rows and columns lo..hi
        return (unsigned)(row(k) - lo) <= (unsigned)(hi - lo) && (unsigned)(col(k) - lo) <= (unsigned)(hi - lo);
    }
    __device__ __forceinline__ void place(const AdrGeom& A, int i0, int j0) {
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int gi = i0 + row(k), gj = j0 + col(k);
            ok[k] = q(k) < N && gi >= 1 && gi < A.ny && gj >= 1 && gj < A.nx;
            p[k] = ok[k] ? (unsigned)(gi * A.nx + gj) : 0u;
        }
    }
    template <typename V>
    __device__ __forceinline__ void load(const V* __restrict__ a, V (&v)[NPT]) const {
#pragma unroll
        for (int k = 0; k < NPT; ++k) v[k] = ld_off(a, p[k]);
    }
    __device__ __forceinline__ void coefs(const AdrGeom& A, const T (&fx)[NPT], const T (&fy)[NPT],
                                          const cplx<T> (&cc)[NPT]) {
#pragma unroll
        for (int k = 0; k < NPT; ++k) cf[k] = up_coef<T>(A, fx[k], fy[k], cc[k], ok[k]);
    }
    __device__ __forceinline__ static void put(const cplx<T> (&v)[NPT], cplx<T>* s) {
#pragma unroll
        for (int k = 0; k < NPT; ++k)
            if (has(k)) s[S0 + q(k)] = v[k];
    }
    // v = M s from a buffer that holds one more node on every side, node 0 of it at s
    __device__ __forceinline__ void apply_start(const cplx<T>* s, cplx<T> (&v)[NPT], bool sub = false) const {
        constexpr int W = RW + 2;
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            if (!has(k)) continue;
            const cplx<T>* a = s + (row(k) + 1) * W + col(k) + 1;
            const cplx<T> m = up_apply<T>(cf[k], a[0], a[-1], a[1], a[-W], a[W]);
            v[k] = sub ? v[k] - m : m;
        }
    }
    // v = the centre nodes of such a buffer
    __device__ __forceinline__ static void get_start(const cplx<T>* s, cplx<T> (&v)[NPT]) {
        constexpr int W = RW + 2;
#pragma unroll
        for (int k = 0; k < NPT; ++k) v[k] = has(k) ? s[(row(k) + 1) * W + col(k) + 1] : cplx<T>{};
    }
    // v = M s, or v -= M s
    __device__ __forceinline__ void apply(const cplx<T>* s, cplx<T> (&v)[NPT], bool sub = false) const {
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            if (!has(k)) continue;
            const cplx<T>* a = s + S0 + q(k);
            const cplx<T> m = up_apply<T>(cf[k], a[0], a[-1], a[1], a[-RW], a[RW]);
            v[k] = sub ? v[k] - m : m;
        }
    }
    // kv[1..NK] = M kv[0], ... through s0 and s1 in turn (kv[0] into s0), one barrier per
    // vector; s0 must be free to write.  The last application reads s0 for odd NK, else s1.
    template <int NK>
    __device__ __forceinline__ void chain(cplx<T> (&kv)[NK + 1][NPT], cplx<T>* s0, cplx<T>* s1) const {
        static_for<NK>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            cplx<T>* s = (j & 1) ? s1 : s0;
            put(kv[j], s);
            __syncthreads();
            apply(s, kv[j + 1]);
        });
    }
    // Gram sums of kv[0..3] over the unknowns lo..hi to part[v * gridDim.x + blockIdx.x].
    // red: FB / 64 * 16 doubles of LDS.
    __device__ __forceinline__ void gram(const cplx<T> (&kv)[4][NPT], int lo, int hi, double* red,
                                         double* __restrict__ part) const {
        double acc[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.0;
#pragma unroll
        for (int k = 0; k < NPT; ++k)
            if (in(k, lo, hi) && ok[k]) {
                const cplx<T> kk[4] = {kv[0][k], kv[1][k], kv[2][k], kv[3][k]};
                gram_add<T, 3>(acc, kk);
            }
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const double s = wave_sum16(acc);
        if (!(lane & 3)) red[wave * 16 + (lane >> 2)] = s;
        __syncthreads();
        if (threadIdx.x < 16) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < FB / 64; ++w) t += red[w * 16 + threadIdx.x];
            part[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
        }
    }
};

// The zero ring (row 0, column 0) of x over this tile's rows and columns.
template <typename T>
__device__ __forceinline__ void fuse_ring(cplx<T>* __restrict__ x, int nx, int ny, int ti, int tj, int edge) {
    const int t = threadIdx.x;
    if (t >= edge) return;
    const int j = 1 + tj * edge + t, i = 1 + ti * edge + t;
    if (ti == 0 && j < nx) x[j] = cplx<T>{};
    if (tj == 0 && i < ny) x[(size_t)i * nx] = cplx<T>{};
    if (ti == 0 && tj == 0 && t == 0) x[0] = cplx<T>{};
}

// Pre-smoother of level l (x0 = 0) finished on the tile, b_{l+1} = R (b - M x) (the residual
// K_0 - sum_j c_j K_j) on the coarse tile and a ring of 3, K_0..K_3 of the coarse
// smoother there and its Gram sums.  fuse_tiles(A.nx, A.ny, FT) blocks.
template <typename T, int FT>
__global__ __launch_bounds__((FuseCfg<FT>::DOWN)) void k_fuse_down(
    AdrGeom A, AdrGeom Ac, const T* __restrict__ px, const T* __restrict__ py, const cplx<T>* __restrict__ c0,
    const cplx<T>* __restrict__ b, const double* __restrict__ part_in, int ng, cplx<T>* __restrict__ xout,
    const T* __restrict__ pxc, const T* __restrict__ pyc, const cplx<T>* __restrict__ c0c, cplx<T>* __restrict__ bc,
    double* __restrict__ part_out, BatchIdx bi) {
    bshift(bi.off(), px, py, c0, b, part_in, xout, pxc, pyc, c0c, bc, part_out);
    constexpr int FB = FuseCfg<FT>::DOWN, TC = FT / 2;
    constexpr int HC = 3, RC = TC + 2 * HC;          // coarse region
    constexpr int OF = 2 * HC + 2, RW = 2 * RC + 5;  // fine region of K_1.., the tile at OF
    using RO = FuseOuter<T, RW, FB>;                 // and of K_0
    using RF = FuseReg<T, RW, FB>;
    using RG = FuseReg<T, RC, FB>;
    constexpr int LB = RO::N > RF::LB ? RO::N : RF::LB;
    static_assert(2 * RG::LB <= LB, "coarse buffers in one fine buffer");
    static_assert(((RF::NPT * FB - 1) / RW + 3) * RO::W <= 2 * LB, "reads beside the last node");
    __shared__ cplx<T> buf[2 * LB];
    __shared__ double sh[FUSE_SH], red[FB / 64 * 16];
    cplx<T>* s0 = buf;
    cplx<T>* s1 = buf + LB;
    int ti, tj;
    tile_index(fuse_side(A.nx, FT), ti, tj);
    const int i0 = 1 + ti * FT - OF, j0 = 1 + tj * FT - OF;
    const int I0 = 1 + ti * TC - HC, J0 = 1 + tj * TC - HC;  // 2 I0 = i0 + 3
    const FuseSums<FB> cs(part_in, ng);
    RF F;
    RG G;
    F.place(A, i0, j0);
    G.place(Ac, I0, J0);
    cplx<T> kv[4][RF::NPT], cc[RF::NPT], ccc[RG::NPT];
    T fx[RF::NPT], fy[RF::NPT], fxc[RG::NPT], fyc[RG::NPT];
    RO K0;
    K0.load(A, b, i0, j0);
    F.load(px, fx);
    F.load(py, fy);
    F.load(c0, cc);
    G.load(pxc, fxc);
    G.load(pyc, fyc);
    G.load(c0c, ccc);
    cs.sum(sh);
    fuse_ring(xout, A.nx, A.ny, ti, tj, FT);
    fuse_ring(bc, Ac.nx, Ac.ny, ti, tj, TC);
    F.coefs(A, fx, fy, cc);
    K0.put(s0);
    __syncthreads();
    fuse_coef_solve<FB>(sh);
    RF::get_start(s0, kv[0]);
    F.apply_start(s0, kv[1]);
    RF::put(kv[1], s1);
    __syncthreads();
    F.apply(s1, kv[2]);
    RF::put(kv[2], s0);  // s0 was last read before the barrier above
    cplx<T> c[3];
    fuse_coef_get(sh, c);
    // x and the residual K_0 - c_1 K_1 - c_2 K_2 before the last application, which leaves two
    // vectors instead of four beside it
    cplx<T> rv[RF::NPT];
#pragma unroll
    for (int k = 0; k < RF::NPT; ++k) {
        cplx<T> xv{};
        rv[k] = kv[0][k];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            xv = xv + c[q] * kv[q][k];
            if (q < 2) rv[k] = rv[k] - c[q] * kv[q + 1][k];
        }
        if (RF::in(k, OF, OF + FT - 1) && F.ok[k]) st_off(xout, F.p[k], xv);
    }
    __syncthreads();
    F.apply(s0, kv[3]);
#pragma unroll
    for (int k = 0; k < RF::NPT; ++k) s1[RF::S0 + RF::q(k)] = rv[k] - c[2] * kv[3][k];  // exact on 2..RW - 3
    __syncthreads();
    G.coefs(Ac, fxc, fyc, ccc);
    cplx<T> kc[4][RG::NPT];
#pragma unroll
    for (int k = 0; k < RG::NPT; ++k) {
        const cplx<T>* r = s1 + RF::S0 + (G.ok[k] ? (2 * RG::row(k) + 3) * RW + 2 * RG::col(k) + 3 : RW + 1);
        const cplx<T> ud = ((r[-RW] + r[RW]) + r[-1]) + r[1];
        const cplx<T> dg = ((r[-RW - 1] + r[-RW + 1]) + r[RW - 1]) + r[RW + 1];
        const cplx<T> v = T(1.0 / 16.0) * ((T(4) * r[0] + T(2) * ud) + dg);
        if (RG::in(k, HC, HC + TC - 1) && G.ok[k]) st_off(bc, G.p[k], v);
        kc[0][k] = G.ok[k] ? v : cplx<T>{};
    }
    G.template chain<3>(kc, s0, s0 + RG::LB);
    G.gram(kc, HC, HC + TC - 1, red, part_out);
}

// Gram sums of the pre-smoother on the first joined level when that is not level 2.
// fuse_tiles(A.nx, A.ny, FT) blocks.
template <typename T, int FT>
__global__ __launch_bounds__((FuseCfg<FT>::LAST)) void k_fuse_gram(AdrGeom A, const T* __restrict__ px,
                                                                 const T* __restrict__ py,
                                                                 const cplx<T>* __restrict__ c0,
                                                                 const cplx<T>* __restrict__ b,
                                                                 double* __restrict__ part_out, BatchIdx bi) {
    bshift(bi.off(), px, py, c0, b, part_out);
    constexpr int FB = FuseCfg<FT>::LAST, H = 3, RW = FT + 2 * H;
    using RF = FuseReg<T, RW, FB>;
    __shared__ cplx<T> buf[2 * RF::LB];
    __shared__ double red[FB / 64 * 16];
    int ti, tj;
    tile_index(fuse_side(A.nx, FT), ti, tj);
    RF F;
    F.place(A, 1 + ti * FT - H, 1 + tj * FT - H);
    cplx<T> kv[4][RF::NPT], cc[RF::NPT];
    T fx[RF::NPT], fy[RF::NPT];
    F.load(b, kv[0]);
    F.load(px, fx);
    F.load(py, fy);
    F.load(c0, cc);
    F.coefs(A, fx, fy, cc);
    F.template chain<3>(kv, buf, buf + RF::LB);
    F.gram(kv, H, H + FT - 1, red, part_out);
}

// The smoother of the coarser level finished on the coarse nodes around the tile (X0C: the
// post-smoother from x_c; else the coarsest level's from zero), x = x_in + P x_c on the tile
// and, with GRAM, on a ring of 4, and the Gram sums of the post-smoother from x.
// fuse_tiles(A.nx, A.ny, FT) blocks; with GRAM xout must not overlap xin (without, the two
// are one array and xout's ring is left alone).
template <typename T, bool X0C, int FT, bool GRAM>
__global__ __launch_bounds__((FuseCfg<FT>::UP)) void k_fuse_up(
    AdrGeom A, AdrGeom Ac, const T* __restrict__ px, const T* __restrict__ py, const cplx<T>* __restrict__ c0,
    const cplx<T>* __restrict__ b, const cplx<T>* __restrict__ xin, cplx<T>* __restrict__ xout,
    const T* __restrict__ pxc, const T* __restrict__ pyc, const cplx<T>* __restrict__ c0c,
    const cplx<T>* __restrict__ bc, const cplx<T>* __restrict__ xc, const double* __restrict__ part_in, int ng,
    double* __restrict__ part_out, BatchIdx bi) {
    bshift(bi.off(), px, py, c0, b, xin, xout, pxc, pyc, c0c, bc, xc, part_in, part_out);
    constexpr int FB = FuseCfg<FT>::UP, TC = FT / 2;
    constexpr int H = GRAM ? 4 : 0, RW = FT + 2 * H;  // fine region: fine node 1 + FT ti - H + r
    constexpr int HC = X0C ? 3 : 2, RC = TC + H + 1 + 2 * HC;  // coarse node TC ti - H / 2 - HC + r
    using RF = FuseReg<T, RW, FB>;
    using RG = FuseReg<T, RC, FB>;
    constexpr int LB = !GRAM || RG::LB > RF::LB ? RG::LB : RF::LB;
    __shared__ cplx<T> buf[2 * LB];
    __shared__ cplx<T> xs[RG::NPT * FB];
    __shared__ double sh[FUSE_SH], red[FB / 64 * 16];
    cplx<T>* s0 = buf;
    cplx<T>* s1 = buf + LB;
    int ti, tj;
    tile_index(fuse_side(A.nx, FT), ti, tj);
    const int i0 = 1 + ti * FT - H, j0 = 1 + tj * FT - H;
    const int I0 = ti * TC - H / 2 - HC, J0 = tj * TC - H / 2 - HC;
    const FuseSums<FB> cs(part_in, ng);
    RG G;
    RF F;
    G.place(Ac, I0, J0);
    F.place(A, i0, j0);
    cplx<T> kc[3][RG::NPT], x0[RG::NPT], ccc[RG::NPT], kv[4][RF::NPT], x[RF::NPT], cc[RF::NPT];
    T fx[RF::NPT], fy[RF::NPT], fxc[RG::NPT], fyc[RG::NPT];
    G.load(bc, kc[0]);
    if constexpr (X0C) G.load(xc, x0);
    G.load(pxc, fxc);
    G.load(pyc, fyc);
    G.load(c0c, ccc);
    F.load(xin, x);
    if constexpr (GRAM) {
        F.load(b, kv[0]);
        F.load(px, fx);
        F.load(py, fy);
        F.load(c0, cc);
        fuse_ring(xout, A.nx, A.ny, ti, tj, FT);
    }
    cs.sum(sh);
    G.coefs(Ac, fxc, fyc, ccc);
    if constexpr (X0C) {
        RG::put(x0, s1);
        __syncthreads();
        fuse_coef_solve<FB>(sh);
        G.apply(s1, kc[0], true);
        G.template chain<2>(kc, s0, s1);
    } else {
        RG::put(kc[0], s0);
        __syncthreads();
        fuse_coef_solve<FB>(sh);
        G.apply(s0, kc[1]);
        RG::put(kc[1], s1);
        __syncthreads();
        G.apply(s1, kc[2]);
    }
    cplx<T> c[3];
    fuse_coef_get(sh, c);
#pragma unroll
    for (int k = 0; k < RG::NPT; ++k) {
        if (!RG::has(k)) continue;
        cplx<T> v{};
        if constexpr (X0C) v = x0[k];
#pragma unroll
        for (int q = 0; q < 3; ++q) v = v + c[q] * kc[q][k];
        xs[RG::q(k)] = v;  // exact on the nodes HC..RC - 1 - HC
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < RF::NPT; ++k) {
        // fine node (gi, gj) between the coarse nodes (gi / 2, gj / 2) and, for odd gi or gj,
        // the next ones; for even ones the same again, so the mean of four is exact
        const int gi = i0 + RF::row(k), gj = j0 + RF::col(k);
        const int l = F.ok[k] ? ((gi >> 1) - I0) * RC + (gj >> 1) - J0 : 0;
        const int dj = gj & 1, di = (gi & 1) * RC;
        const cplx<T> e = T(0.25) * ((xs[l] + xs[l + di]) + (xs[l + dj] + xs[l + di + dj]));
        const cplx<T> v = x[k] + e;
        x[k] = F.ok[k] ? v : cplx<T>{};
        if (RF::in(k, H, H + FT - 1) && F.ok[k]) st_off(xout, F.p[k], v);
    }
    if constexpr (GRAM) {
        F.coefs(A, fx, fy, cc);
        RF::put(x, s0);  // s0 and s1 were last read before the barrier above
        __syncthreads();
        F.apply(s0, kv[0], true);
        F.template chain<3>(kv, s1, s0);
        F.gram(kv, H, H + FT - 1, red, part_out);
    }
}

// b = (g - A u) e^{-i theta} at the unknowns of the region from u in LDS (0 off the unknowns;
// rows of W, region node (0, 0) at su), 0 elsewhere.
template <int W, typename RF, typename T>
__device__ __forceinline__ void fuse_demod(const RF& R, int i0, int j0, const ModArgs<T>& mod, const cplx<T>* su,
                                           const cplx<T> (&car)[RF::NPT], const cplx<T> (&g)[RF::NPT],
                                           const T (&n2)[RF::NPT], cplx<T> (&b)[RF::NPT]) {
    const T ih2 = T(mod.G.inv_h2);
#pragma unroll
    for (int k = 0; k < RF::NPT; ++k) {
        if (!RF::has(k)) continue;
        const cplx<T>* a = su + RF::row(k) * W + RF::col(k);
        const cplx<T> cu = a[0];
        const cplx<T> nb = ((a[-W] + a[W]) + a[-1]) + a[1];
        const cplx<T> lap = ih2 * (T(4) * cu - nb);
        const cplx<T> kap = kappa_at<T>(mod.G, n2[k], i0 + RF::row(k), j0 + RF::col(k));
        const cplx<T> v = (g[k] - (lap - kap * cu)) * conjg(car[k]);
        b[k] = R.ok[k] ? v : cplx<T>{};
    }
}

// First ADR step of a cycle: the demodulated residual and the Gram sums of the
// pre-smoother on level 2.  mod.u read, mod.bout written.
template <typename T, int FT>
__global__ __launch_bounds__((FuseCfg<FT>::START)) void k_fuse_start(AdrGeom A, const T* __restrict__ px,
                                                                   const T* __restrict__ py,
                                                                   const cplx<T>* __restrict__ c0, ModArgs<T> mod,
                                                                   double* __restrict__ part_out, BatchIdx bi) {
    bshift(bi.off(), px, py, c0, mod, part_out);
    constexpr int FB = FuseCfg<FT>::START, H = 3, RW = FT + 2 * H;
    using RF = FuseReg<T, RW, FB>;
    using RO = FuseOuter<T, RW, FB>;
    constexpr int LB = RO::N > RF::LB ? RO::N : RF::LB;
    static_assert(((RF::NPT * FB - 1) / RW + 3) * RO::W <= 2 * LB, "reads beside the last node");
    __shared__ cplx<T> buf[2 * LB];
    __shared__ double red[FB / 64 * 16];
    int ti, tj;
    tile_index(fuse_side(A.nx, FT), ti, tj);
    const int i0 = 1 + ti * FT - H, j0 = 1 + tj * FT - H;
    RF F;
    RO U;
    F.place(A, i0, j0);
    cplx<T> car[RF::NPT], g[RF::NPT], kv[4][RF::NPT], cc[RF::NPT];
    T n2[RF::NPT], fx[RF::NPT], fy[RF::NPT];
    U.load(A, mod.u, i0, j0);
    F.load(mod.car, car);
    F.load(mod.g, g);
    F.load(mod.n2, n2);
    F.load(px, fx);
    F.load(py, fy);
    F.load(c0, cc);
    fuse_ring(mod.bout, A.nx, A.ny, ti, tj, FT);
    U.put(buf);
    __syncthreads();
    fuse_demod<RO::W, RF, T>(F, i0, j0, mod, buf + RO::W + 1, car, g, n2, kv[0]);
    F.coefs(A, fx, fy, cc);
#pragma unroll
    for (int k = 0; k < RF::NPT; ++k)
        if (RF::in(k, H, H + FT - 1) && F.ok[k]) st_off(mod.bout, F.p[k], kv[0][k]);
    F.template chain<3>(kv, buf + LB, buf);
    F.gram(kv, H, H + FT - 1, red, part_out);
}

// The post-smoother of level 2 finished (x from x0), u_out = u + x e^{i theta}; with NEXT
// also the demodulated residual of the next ADR step and the Gram sums of its
// pre-smoother (x on the tile and a ring of 4, the residual on a ring of 3).
template <typename T, bool NEXT, int FT>
__global__ __launch_bounds__((NEXT ? FuseCfg<FT>::STEP : FuseCfg<FT>::LAST)) void k_fuse_step(
    AdrGeom A, const T* __restrict__ px, const T* __restrict__ py, const cplx<T>* __restrict__ c0,
    const cplx<T>* __restrict__ b, const cplx<T>* __restrict__ x0, const double* __restrict__ part_in, int ng,
    ModArgs<T> mod, double* __restrict__ part_out, BatchIdx bi) {
    bshift(bi.off(), px, py, c0, b, x0, part_in, mod, part_out);
    constexpr int FB = NEXT ? FuseCfg<FT>::STEP : FuseCfg<FT>::LAST;
    constexpr int XH = NEXT ? 4 : 0, H = 2 + XH, RW = FT + 2 * H;  // region of r = b - M x0
    constexpr int HN = 3, RN = FT + 2 * HN;                        // and of the next right-hand side
    using RF = FuseReg<T, RW, FB>;
    using RO = FuseOuter<T, RW, FB>;
    using RS = FuseReg<T, RN, FB>;
    constexpr int LB = RO::N > RF::LB ? RO::N : RF::LB;
    static_assert(((RF::NPT * FB - 1) / RW + 3) * RO::W <= 2 * LB, "reads beside the last node");
    static_assert(!NEXT || (RS::LB <= LB && (RS::NPT * FB - 1) / RN + 3 <= 2 * LB / RW), "next step's vectors");
    __shared__ cplx<T> buf[2 * LB];
    __shared__ double sh[FUSE_SH], red[NEXT ? FB / 64 * 16 : 1];
    cplx<T>* s0 = buf;
    cplx<T>* s1 = buf + LB;
    int ti, tj;
    tile_index(fuse_side(A.nx, FT), ti, tj);
    const int i0 = 1 + ti * FT - H, j0 = 1 + tj * FT - H;
    const FuseSums<FB> cs(part_in, ng);
    RF F;
    RO X;
    F.place(A, i0, j0);
    cplx<T> x[RF::NPT], u[RF::NPT], car[RF::NPT], kk[3][RF::NPT], cc[RF::NPT];
    T fx[RF::NPT], fy[RF::NPT];
    X.load(A, x0, i0, j0);
    F.load(b, kk[0]);
    F.load(px, fx);
    F.load(py, fy);
    F.load(c0, cc);
#pragma unroll
    for (int k = 0; k < RF::NPT; ++k) {
        // u may be the array that the other tiles write (NEXT false): own nodes only
        const unsigned p = NEXT || RF::in(k, H, H + FT - 1) ? F.p[k] : 0u;
        u[k] = ld_off(mod.u, p);
        car[k] = ld_off(mod.car, p);
    }
    cs.sum(sh);
    fuse_ring(mod.uout, A.nx, A.ny, ti, tj, FT);
    F.coefs(A, fx, fy, cc);
    X.put(s0);
    __syncthreads();
    fuse_coef_solve<FB>(sh);
    RF::get_start(s0, x);
    F.apply_start(s0, kk[0], true);
    F.template chain<2>(kk, s1, s0);
    cplx<T> c[3];
    fuse_coef_get(sh, c);
#pragma unroll
    for (int k = 0; k < RF::NPT; ++k) {
        if (!RF::has(k)) continue;
#pragma unroll
        for (int q = 0; q < 3; ++q) x[k] = x[k] + c[q] * kk[q][k];
        u[k] = u[k] + x[k] * car[k];
        if (RF::in(k, H, H + FT - 1) && F.ok[k]) st_off(mod.uout, F.p[k], u[k]);
    }
    if constexpr (NEXT) {
        // on the smaller region, with fewer nodes a thread, from fields read again (L2; loading
        // them with the first ones gained nothing in FP32 and spills in FP64)
        RS S;
        const int n0 = i0 + H - HN, m0 = j0 + H - HN;
        S.place(A, n0, m0);
        cplx<T> g[RS::NPT], cr[RS::NPT], c0s[RS::NPT], kv[4][RS::NPT];
        T n2[RS::NPT], fxs[RS::NPT], fys[RS::NPT];
        S.load(mod.g, g);
        S.load(mod.n2, n2);
        S.load(mod.car, cr);
        S.load(px, fxs);
        S.load(py, fys);
        S.load(c0, c0s);
        fuse_ring(mod.bout, A.nx, A.ny, ti, tj, FT);
#pragma unroll
        for (int k = 0; k < RF::NPT; ++k) u[k] = F.ok[k] ? u[k] : cplx<T>{};
        RF::put(u, s1);  // s1 was last read before the last barrier of the chain
        __syncthreads();
        fuse_demod<RW, RS, T>(S, n0, m0, mod, s1 + RF::S0 + (H - HN) * (RW + 1), cr, g, n2, kv[0]);
        S.coefs(A, fxs, fys, c0s);
#pragma unroll
        for (int k = 0; k < RS::NPT; ++k)
            if (RS::in(k, HN, HN + FT - 1) && S.ok[k]) st_off(mod.bout, S.p[k], kv[0][k]);
        S.template chain<3>(kv, s0, s1);
        S.gram(kv, HN, HN + FT - 1, red, part_out);
    }
}

}  // namespace helm
