// Lane scan of the filter's fold pass at d >= 6: the inclusive scan of a tile's
// 64 lane aggregates as a launch of its own, one workgroup of d / 2 waves per
// tile, the aggregates in LDS by [field][lane]. At each of the six levels every
// lane of every wave forms M = I + C_x J_y and its factors for its lane, and
// wave w the columns w and d - 1 - w of the products (as many entries of the
// symmetric ones for each wave); the last two waves also take b and eta. In the
// fold itself, one lane held two aggregates, the factors and the products: at
// d = 8 (FP32) 304 values, so that a level took 36 us of moves between
// registers, spills and 5600 instructions with one wave on a SIMD. Here a wave
// has about a third of them, operands come from LDS where they are used, and a
// SIMD holds several waves. Same order of operations as agg_combine, but for the
// symmetric form of M^-1 C_x at d = 8 in FP64 (lane_scan_symmetric).
#pragma once
#include "filter_ops.h"

// Whether M^-1 C_x, symmetric in exact arithmetic, enters C as its upper triangle
// on both sides of the diagonal (through zs): for a sum of two components M is
// nearly singular where the series is dense, the two triangles then differ by
// far more than the rounding of either, and the next level multiplies the
// difference. Matern-3/2 + RBF-6, 1 100 steps 1e-3 apart, noise variance 1e-6,
// 64 steps a lane: error of the filtered variance of f 1.8e-10, of f_var 2e-9;
// with the full M^-1 C_x 2.2e-7 and 5e-6.
template <int D, typename T>
constexpr bool lane_scan_symmetric() { return sizeof(T) == 8 && D >= 8; }

// y <- x (x) y, or with MOM, for an x that starts at the series start (A = 0),
// the conditioning of its moments (moments_apply) in FP64; x: lane - o, on:
// whether this lane takes part. All waves of the workgroup call it; s is the
// tile's aggregates, az room for d^2 values of CT per lane, zs (where
// lane_scan_symmetric) for the triangle.
template <int D, typename T, typename CT, bool MOM>
__device__ __forceinline__ void lane_scan_level(T *s, CT *az, CT *zs, int w, int lane, int o, bool on)
{
    constexpr int W = PSSGP_WAVE, NS = AggLayout<D>::NS;
    constexpr int OB = D * D, OC = OB + D, OE = OC + NS, OJ = OE + D;
    const T *sx = s + (on ? lane - o : lane);
    T *sy = s + lane;
    auto X = [&](int f) { return CT(sx[f * W]); };
    auto Y = [&](int f) { return CT(sy[f * W]); };
    // d = 6: the operands of a row are not loaded before the row's turn, which
    // leaves room for two waves on a SIMD (FP64, 3e5 steps: the call 512 -> 470
    // us); at d = 8 there is one anyway, and the loads ahead are worth 8 %
    auto row = [] {
        if constexpr (D < 8) asm volatile("" ::: "memory");
    };
    const int j0 = w, j1 = D - 1 - w;  // this wave's columns, j0 < j1
    CT M[D][D];
    int piv[D];
    {
        T J[NS];
#pragma unroll
        for (int q = 0; q < NS; q++) J[q] = sy[(OJ + q) * W];
#pragma unroll
        for (int i = 0; i < D; i++) {
            row();
            if constexpr (MOM) {
#pragma unroll
                for (int q = 0; q < NS; q++) asm volatile("" : "+v"(J[q]));
            }
            CT c[D];
#pragma unroll
            for (int k = 0; k < D; k++) c[k] = X(OC + sidx<D>(i, k));
#pragma unroll
            for (int j = 0; j < D; j++) {
                CT acc = (i == j) ? CT(1) : CT(0);
#pragma unroll
                for (int k = 0; k < D; k++) acc = fma(c[k], CT(J[sidx<D>(k, j)]), acc);
                M[i][j] = acc;
            }
        }
    }
    lu_factor<D, CT>(M, piv);
    row();
    // b (last wave) or eta (the one before it)
    CT vec[D];
    if (w == D / 2 - 1) {
        CT z[D];
#pragma unroll
        for (int i = 0; i < D; i++) {
            row();
            CT ce = X(OB + i);
#pragma unroll
            for (int k = 0; k < D; k++) ce = fma(X(OC + sidx<D>(i, k)), Y(OE + k), ce);
            z[i] = ce;
        }
        lu_solve<D, CT>(M, piv, z);
#pragma unroll
        for (int i = 0; i < D; i++) {
            row();
            CT bb = Y(OB + i);
#pragma unroll
            for (int k = 0; k < D; k++) bb = fma(Y(i * D + k), z[k], bb);
            vec[i] = bb;
        }
    } else if (!MOM && w == D / 2 - 2) {
        CT u[D], v[D];
#pragma unroll
        for (int i = 0; i < D; i++) {
            row();
            CT acc = Y(OE + i);
#pragma unroll
            for (int k = 0; k < D; k++) acc = fma(-Y(OJ + sidx<D>(i, k)), X(OB + k), acc);
            u[i] = acc;
        }
#pragma unroll
        for (int i = 0; i < D; i++) {
            row();
            CT cu = CT(0);
#pragma unroll
            for (int k = 0; k < D; k++) cu = fma(X(OC + sidx<D>(i, k)), u[k], cu);
            v[i] = cu;
        }
        lu_solve<D, CT>(M, piv, v);
#pragma unroll
        for (int i = 0; i < D; i++) {
            row();
            CT ue = u[i];
#pragma unroll
            for (int k = 0; k < D; k++) ue = fma(-Y(OJ + sidx<D>(i, k)), v[k], ue);
            u[i] = ue;
        }
#pragma unroll
        for (int i = 0; i < D; i++) {
            row();
            CT e = X(OE + i);
#pragma unroll
            for (int k = 0; k < D; k++) e = fma(X(k * D + i), u[k], e);
            vec[i] = e;
        }
    }
    row();
    // columns of A_y M^-1 C_x
    {
        CT c0[D], c1[D];
#pragma unroll
        for (int i = 0; i < D; i++) { c0[i] = X(OC + sidx<D>(i, j0)); c1[i] = X(OC + sidx<D>(i, j1)); }
        lu_solve<D, CT>(M, piv, c0);
        lu_solve<D, CT>(M, piv, c1);
        if constexpr (lane_scan_symmetric<D, T>()) {
#pragma unroll
            for (int i = 0; i < D; i++) {
                if (i <= j0) zs[sidx<D>(i, j0) * W + lane] = c0[i];
                if (i <= j1) zs[sidx<D>(i, j1) * W + lane] = c1[i];
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < D; i++) { c0[i] = zs[sidx<D>(i, j0) * W + lane]; c1[i] = zs[sidx<D>(i, j1) * W + lane]; }
        }
#pragma unroll
        for (int i = 0; i < D; i++) {
            row();
            CT a0 = CT(0), a1 = CT(0);
#pragma unroll
            for (int k = 0; k < D; k++) {
                const CT a = Y(i * D + k);
                a0 = fma(a, c0[k], a0);
                a1 = fma(a, c1[k], a1);
            }
            az[(i * D + j0) * W + lane] = a0;
            az[(i * D + j1) * W + lane] = a1;
        }
    }
    row();
    // columns of A and J
    CT na0[D], na1[D], nj0[D], nj1[D];
    if constexpr (!MOM) {
        CT x0[D], x1[D], z0[D], z1[D];
#pragma unroll
        for (int i = 0; i < D; i++) { x0[i] = X(i * D + j0); x1[i] = X(i * D + j1); }
        lu_solve<D, CT>(M, piv, x0);
        lu_solve<D, CT>(M, piv, x1);
#pragma unroll
        for (int i = 0; i < D; i++) {
            row();
            CT a0 = CT(0), a1 = CT(0), b0 = CT(0), b1 = CT(0);
#pragma unroll
            for (int k = 0; k < D; k++) {
                const CT a = Y(i * D + k), j = Y(OJ + sidx<D>(i, k));
                a0 = fma(a, x0[k], a0);
                a1 = fma(a, x1[k], a1);
                b0 = fma(j, x0[k], b0);
                b1 = fma(j, x1[k], b1);
            }
            na0[i] = a0;
            na1[i] = a1;
            z0[i] = b0;
            z1[i] = b1;
        }
#pragma unroll
        for (int i = 0; i < D; i++) {
            if (i > j1) continue;
            row();
            CT a0 = X(OJ + sidx<D>(i, j0)), a1 = X(OJ + sidx<D>(i, j1));
#pragma unroll
            for (int k = 0; k < D; k++) {
                const CT a = X(k * D + i);
                a0 = fma(a, z0[k], a0);
                a1 = fma(a, z1[k], a1);
            }
            nj0[i] = a0;
            nj1[i] = a1;
        }
    }
    row();
    CT r0[D], r1[D];
#pragma unroll
    for (int k = 0; k < D; k++) { r0[k] = Y(j0 * D + k); r1[k] = Y(j1 * D + k); }
    // every read of the old aggregates is done, but for C_y, whose entries
    // only the wave that writes them reads below
    __syncthreads();
#pragma unroll
    for (int i = 0; i < D; i++) {
        if (i > j1) continue;
        row();
        CT a0 = Y(OC + sidx<D>(i, j0)), a1 = Y(OC + sidx<D>(i, j1));
#pragma unroll
        for (int k = 0; k < D; k++) {
            const CT a = az[(i * D + k) * W + lane];
            a0 = fma(a, r0[k], a0);
            a1 = fma(a, r1[k], a1);
        }
        if (on) {
            if (i <= j0) sy[(OC + sidx<D>(i, j0)) * W] = T(a0);
            sy[(OC + sidx<D>(i, j1)) * W] = T(a1);
        }
    }
    if (on) {
#pragma unroll
        for (int i = 0; i < D; i++) {
            sy[(i * D + j0) * W] = MOM ? T(0) : T(na0[i]);
            sy[(i * D + j1) * W] = MOM ? T(0) : T(na1[i]);
            if (i <= j0) sy[(OJ + sidx<D>(i, j0)) * W] = MOM ? T(0) : T(nj0[i]);
            if (i <= j1) sy[(OJ + sidx<D>(i, j1)) * W] = MOM ? T(0) : T(nj1[i]);
            if (w == D / 2 - 1) sy[(OB + i) * W] = T(vec[i]);
            if (w == D / 2 - 2) sy[(OE + i) * W] = MOM ? T(0) : T(vec[i]);
        }
    }
    __syncthreads();
}

// lanep: the lanes' aggregates from the fold, replaced by the inclusive
// prefixes; aggp: the tile aggregates. In tile 0 the prefixes that reach lane 0
// start at the series start: a pair of filter moments, whose conditioning on a
// later aggregate cancels when that is informative, so in FP64.
template <int D, typename T>
__global__ __launch_bounds__(PSSGP_WAVE *D / 2, 1) void lane_scan_kernel(T *lanep, T *aggp)
{
    constexpr int AGG = AggLayout<D>::SIZE, W = PSSGP_WAVE;
    __shared__ T s[AGG * W];
    __shared__ double az[D * D * W];
    __shared__ T zs[lane_scan_symmetric<D, T>() ? AggLayout<D>::NS * W : 1];
    const int tile = (int)blockIdx.x, lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / W);
    T *rec = lanep + (size_t)tile * (AGG * W);
    for (int i = (int)threadIdx.x; i < AGG * W; i += W * D / 2) s[i] = rec[i];
    __syncthreads();
    for (int o = 1; o < W; o <<= 1) {
        if (sizeof(T) == 8 || tile != 0) {
            lane_scan_level<D, T, T, false>(s, (T *)az, zs, w, lane, o, lane >= o);
        } else {
            // lanes o .. 2 o - 1 take a prefix from the series start, which
            // this level leaves as it is; the lanes above read theirs first
            lane_scan_level<D, T, T, false>(s, (T *)az, zs, w, lane, o, lane >= 2 * o);
            lane_scan_level<D, T, double, true>(s, az, nullptr, w, lane, o, lane >= o && lane < 2 * o);
        }
    }
    for (int i = (int)threadIdx.x; i < AGG * W; i += W * D / 2) rec[i] = s[i];
    for (int i = (int)threadIdx.x; i < AGG; i += W * D / 2) aggp[(size_t)tile * AGG + i] = s[i * W + W - 1];
}
