// Parallel Kalman filter with missing measurements (paper section 3) as a
// three-pass scan, and the discretisation map.
//
// Work decomposition: one wave (64 lanes) per tile, each lane owns `chunk`
// consecutive steps.
//   fold    each lane folds its steps into a chunk aggregate (the element of
//           a step is built from the FP64 discretisation and rounded to the
//           scan type T); wave-level inclusive scan of the 64 chunk
//           aggregates (Kogge-Stone over lane shuffles) with the general
//           operator; every lane stores its inclusive aggregate
//   carry   one workgroup scans the tile aggregates and stores the filter
//           moments entering every tile (tile_scan.h)
//   finish  each lane applies its exclusive lane prefix to the tile's carry,
//           which gives the filter moments just before its chunk, then
//           re-runs its steps as a plain Kalman filter (prediction and
//           conditioning in FP64), writing (m, P), the adjoint's records or
//           the smoother's handover, and summing the log-likelihood terms in
//           FP64 per lane.
// One series: the per-tile log-likelihood partials are summed in a fixed order
// (last_tile, launch_tile_sums). At d >= 6 the fold's lane scan may be a launch
// of its own (split_lane_scan). Batched: the fold and finish grids cover up to
// two groups of series with different state layouts (one carry scan per
// group) and write one log-likelihood partial per series segment of a lane
// (at the segment's first step) that a second kernel sums per series.
#pragma once
#include "device_common.h"
#include "filter_ops.h"
#include "lane_scan.h"
#include "launch.h"
#include "smoother_ops.h"
#include "tile_scan.h"
#include "tile_scan_team.h"

// Finish-pass outputs: filter moments in the [entry][n] layout, per-step
// records for the adjoint (RecLayout, tile layout), or what the smoother of
// the same call needs: its elements step by step (elem_index), or per-step
// predicted P h and h m, the lanes' end moments and smoother elements
// (HandLayout).
enum : int { F_MOMENTS = 1, F_RECS = 2, F_ELEMS = 4, F_LANES = 8 };
template <int D, typename T>
constexpr int fused_mode() { return lane_handover(D, sizeof(T) == 8) ? F_LANES : F_ELEMS; }

template <typename T>
struct FilterParams {
    const double *t;
    const T *y;
    const uint8_t *mask;
    const double *noise_k;
    int64_t n;
    int chunk;
    int ntiles;
    T *m;
    T *P;
    double *loglik;
    T *rec;             // F_RECS: per-step records (RecLayout, tile layout)
    double *ll_terms;  // batched: per-segment log-likelihood partials, at each segment's first step
    const double *cst;  // model constants of the transition
    WsCtl *ctl;
    T *aggp;
    T *inclp;
    T *lanep;
    double *partials;
    T *elem;        // F_ELEMS: smoother element of every step (elem_index)
    double *hand;   // F_LANES: per-step handover to the smoother (HandLayout)
    double *bound;  // F_LANES: end moments of the lanes (HandLayout)
    T *slane;       // F_ELEMS (lane_aggregate_handover), F_LANES: the smoother's lane records
};

// Tile geometry: steps [k_begin, k_end) split into ntiles tiles; workspace
// tile slots start at slot_base.
struct TileRange {
    int64_t k_begin, k_end;
    int ntiles;
    int slot_base;
};

// Transition of a step, Dl = F - I (F = 0 at a series start, so Dl = -I
// there) and Q, rounded to U, with the constants at cst: for FP32 scans (T)
// from the expansion of F, for FP64 scans by the FP64 discretisation.
template <class LY, typename U, typename T = U>
__device__ __forceinline__ void step_transition(const DevModel &mdl, cdouble *cst, const StepScale &sc,
                                                double dt, bool first, U (&Dl)[LY::D][LY::D],
                                                U (&Q)[LY::D][LY::D])
{
    constexpr int D = LY::D;
    if constexpr (sizeof(T) == 8) {
        double F64[D][D], Q64[D][D];
        discretize<LY, true>(mdl, cst, sc, dt, first, F64, Q64);
#pragma unroll
        for (int i = 0; i < D; i++)
#pragma unroll
            for (int j = 0; j < D; j++) {
                Dl[i][j] = U(F64[i][j] - (i == j ? 1.0 : 0.0));
                Q[i][j] = U(Q64[i][j]);
            }
    } else {
        discretize_fast<LY, U>(mdl, cst, sc, dt, first, Dl, Q);
    }
}

// Per-lane view of the step inputs with the next step's values loaded one
// iteration ahead.
template <typename T>
struct StepInputs {
    double tc, tp;
    T yc;
    bool oc;
    __device__ __forceinline__ void start(const double *t, const T *y, const uint8_t *mask, int64_t k0, int64_t k1,
                                          int64_t k_begin)
    {
        tc = tp = 0.0;
        yc = T(0);
        oc = false;
        if (k0 < k1) {
            tc = t[k0];
            tp = (k0 > k_begin) ? t[k0 - 1] : tc;
            yc = y ? y[k0] : T(0);
            oc = mask ? (mask[k0] != 0) : true;
        }
    }
};

// Smoother element of step k (supplement, Proposition 2), built by the
// filter right after predicting step k + 1, from what that prediction
// already holds: the filtered moments (m, P) of step k and, in FP64,
// Y = F P, mp = F m and Pp = F P F^T + Q of step k + 1:
//   Pp = C C^T (Cholesky), Y = C^-1 F P, L = P - Y^T Y,
//   E = (C^-T Y)^T = P F^T Pp^-1, g = m - E mp.
// At the last step of a series the caller passes the prior transition
// (F = 0, Q = Pinf), for which these give exactly the element (0, m, P).
// e receives the element rounded to T, in the smoother's coordinates
// z' = S z, S = I + e_0 e_B^T (smoother_shear_col; B = 0: identity).
// (m, P) come in U (the filter carries them in FP64).
template <int D, int B, typename T, typename U = T>
__device__ __forceinline__ void smoother_element_from_prediction(const U (&m)[D], const U (&P)[D][D],
                                                                 double (&Y)[D][D], const double (&mp)[D],
                                                                 const double (&Pp)[D][D], SAgg<D, T> &e,
                                                                 uint32_t &bad)
{
    // Y holds F P on entry and is overwritten
    double C[D][D];
#pragma unroll
    for (int i = 0; i < D; i++)
#pragma unroll
        for (int j = 0; j <= i; j++) C[i][j] = Pp[i][j];
    double rd[D];  // reciprocals of the Cholesky diagonal
    if (!cholesky<D, double>(C, rd)) bad |= PSSGP_STATUS_CHOLESKY;
#pragma unroll
    for (int j = 0; j < D; j++)
#pragma unroll
        for (int i = 0; i < D; i++) {
            double acc = Y[i][j];
#pragma unroll
            for (int q = 0; q < i; q++) acc = fma(-C[i][q], Y[q][j], acc);
            Y[i][j] = acc * rd[i];
        }
    // L' = S P S^T - (Y S^T)^T (Y S^T); Y S^T is column 0 plus column B
    if constexpr (B > 0) {
#pragma unroll
        for (int q = 0; q < D; q++) Y[q][0] += Y[q][B];
    }
#pragma unroll
    for (int i = 0; i < D; i++)
#pragma unroll
        for (int j = i; j < D; j++) {
            double acc = (double)P[i][j];
            if constexpr (B > 0) {
                if (i == 0) acc += (double)P[B][j] + (j == 0 ? (double)P[0][B] + (double)P[B][B] : 0.0);
            }
#pragma unroll
            for (int q = 0; q < D; q++) acc = fma(-Y[q][i], Y[q][j], acc);
            e.L[i][j] = T(acc);
            e.L[j][i] = e.L[i][j];
        }
#pragma unroll
    for (int j = 0; j < D; j++)
#pragma unroll
        for (int i = D - 1; i >= 0; i--) {
            double acc = Y[i][j];
#pragma unroll
            for (int q = i + 1; q < D; q++) acc = fma(-C[q][i], Y[q][j], acc);
            Y[i][j] = acc * rd[i];
        }
    // Y = (S E)^T: g' = S m - (S E) mp, E' = (S E) S^-1 (column B minus column 0)
#pragma unroll
    for (int i = 0; i < D; i++) {
        double acc = (double)m[i];
        if constexpr (B > 0) {
            if (i == 0) acc += (double)m[B];
        }
#pragma unroll
        for (int q = 0; q < D; q++) acc = fma(-Y[q][i], mp[q], acc);
        e.g[i] = T(acc);
#pragma unroll
        for (int j = 0; j < D; j++) e.E[i][j] = T((B > 0 && j == B) ? Y[B][i] - Y[0][i] : Y[j][i]);
    }
}

// The smoother element of a step is handed over (stored in the tile layout
// with non-temporal stores: it is read back only after the whole filter, and
// with ordinary stores the caches fetched every line before writing it,
// which doubled the pass's HBM traffic) and, where the smoother takes lane
// aggregates from the filter
// (lane_aggregate_handover), also appended to the lane's running smoother
// aggregate: acc <- acc (x) e (acc covers the lane's earlier steps).
template <int D, typename T, bool LANEAGG>
__device__ __forceinline__ void hand_over_element(const SAgg<D, T> &e, T *out, SAgg<D, T> &acc)
{
    sagg_store_nt<D, T>(out, e, PSSGP_WAVE);
    if constexpr (LANEAGG) sagg_combine<D, T>(acc, e, acc);
}

// Smoother element of a lane: the map from the smoothed moments of the lane's
// last step to those of the step before its first one (supplement,
// Proposition 2, for the whole run of steps at once). The finish pass runs,
// next to the filter, the fixed-point smoother of that earlier state: its
// moments (m0, P0) given the lane's observations so far and its
// cross-covariance G with the current state (row: current state), which
// start as the lane's entering moments and P and are updated per step by
// G <- F G, w = G^T h, m0 += w v / S, P0 -= w w^T / S, G -= K w^T. With (m, P)
// the filter moments of the last step and P = C C^T,
//   Z = C^-1 G, L = P0 - Z^T Z, E = (C^-T Z)^T = G^T P^-1, g = m0 - E m.
// This is what composing the steps' elements gives, without forming one per
// step (no Cholesky factor, solves and three matrix products per step).
// All in the smoother's coordinates z' = S z, S = I + e_0 e_B^T
// (smoother_shear_col; B = 0: identity), whose first state is f, and with the
// first row of S P S^T taken as r P h, r = R / S (1 at a missing step), from the
// last conditioning (ph): formed as a difference it keeps no digit of a
// filtered variance of f below 1e-16 of the predicted one, and for a sum of two
// components P is then not positive definite. (h G, which is as small, may be a
// sum of its two rows: the factor's first column, of the size of its root, takes
// their rounding into nothing larger than that.) G comes in the filter's coordinates and is overwritten; m, C and rd
// receive S m, the factor and the reciprocals of its diagonal. In a lane that
// ends the series (end) E = 0, and the factor, which nothing uses, is not
// judged.
template <int D, int B, typename T>
__device__ __forceinline__ void lane_smoother_element(const double (&m0)[D], double (&P0)[D][D], double (&G)[D][D],
                                                      double (&m)[D], const double (&P)[D][D], double fm,
                                                      const double (&ph)[D], double r,
                                                      bool end, double (&C)[D][D], double (&rd)[D], SAgg<D, T> &e,
                                                      uint32_t &bad)
{
    m[0] = fm;
    double hph = ph[0];
    if constexpr (B > 0) hph += ph[B];
#pragma unroll
    for (int i = 0; i < D; i++) {
        C[i][0] = r * (i == 0 ? hph : ph[i]);
#pragma unroll
        for (int j = 1; j <= i; j++) C[i][j] = P[i][j];
    }
    if (!cholesky<D, double>(C, rd) && !end) bad |= PSSGP_STATUS_CHOLESKY;
#pragma unroll
    for (int i = 0; i < D; i++)
#pragma unroll
        for (int j = 0; j < D; j++) G[i][j] = end ? 0.0 : G[i][j];
    if constexpr (B > 0) {
#pragma unroll
        for (int c = 0; c < D; c++) G[0][c] += G[B][c];
#pragma unroll
        for (int q = 0; q < D; q++) G[q][0] += G[q][B];
    }
#pragma unroll
    for (int j = 0; j < D; j++)
#pragma unroll
        for (int i = 0; i < D; i++) {
            double acc = G[i][j];
#pragma unroll
            for (int q = 0; q < i; q++) acc = fma(-C[i][q], G[q][j], acc);
            G[i][j] = acc * rd[i];
        }
    // L = S P0 S^T - Z^T Z
#pragma unroll
    for (int i = 0; i < D; i++)
#pragma unroll
        for (int j = i; j < D; j++) {
            double acc = P0[i][j];
            if constexpr (B > 0) {
                if (i == 0) acc += P0[j < B ? j : B][j < B ? B : j] + (j == 0 ? P0[0][B] + P0[B][B] : 0.0);
            }
#pragma unroll
            for (int q = 0; q < D; q++) acc = fma(-G[q][i], G[q][j], acc);
            e.L[i][j] = T(acc);
            e.L[j][i] = e.L[i][j];
        }
#pragma unroll
    for (int j = 0; j < D; j++)
#pragma unroll
        for (int i = D - 1; i >= 0; i--) {
            double acc = G[i][j];
#pragma unroll
            for (int q = i + 1; q < D; q++) acc = fma(-C[q][i], G[q][j], acc);
            G[i][j] = acc * rd[i];
        }
    // G = E^T: g = S m0 - E S m
#pragma unroll
    for (int i = 0; i < D; i++) {
        double acc = m0[i];
        if constexpr (B > 0) {
            if (i == 0) acc += m0[B];
        }
#pragma unroll
        for (int q = 0; q < D; q++) acc = fma(-G[q][i], m[q], acc);
        e.g[i] = T(acc);
#pragma unroll
        for (int j = 0; j < D; j++) e.E[i][j] = T(G[j][i]);
    }
}

// Predicted moments of one step in FP64 from (m, P) (in T) and the FP64
// transition Dl = F - I, Q: mp = m + Dl m, Y = F P = P + Dl P,
// Pp = Y F^T + Q = Y + Y Dl^T + Q. FP64 keeps Pp consistent with P to
// the precision the smoother element needs (its L is P minus a Gram matrix
// that nearly equals P when Q is small).
template <int D, typename T, class SP>
__device__ __forceinline__ void predict_step(const T (&m)[D], const T (&P)[D][D], const double (&Dl)[D][D],
                                             const double (&Q)[D][D], double (&mp)[D], double (&Y)[D][D],
                                             double (&Pp)[D][D])
{
#pragma unroll
    for (int i = 0; i < D; i++) {
        double acc = (double)m[i];
#pragma unroll
        for (int k2 = 0; k2 < D; k2++)
            if (SP::dl(i, k2)) acc = fma(Dl[i][k2], (double)m[k2], acc);
        mp[i] = acc;
#pragma unroll
        for (int j = 0; j < D; j++) {
            double y = (double)P[i][j];
#pragma unroll
            for (int k2 = 0; k2 < D; k2++)
                if (SP::dl(i, k2)) y = fma(Dl[i][k2], (double)P[k2][j], y);
            Y[i][j] = y;
        }
    }
#pragma unroll
    for (int i = 0; i < D; i++)
#pragma unroll
        for (int j = i; j < D; j++) {
            double acc = SP::dl(i, j) ? Y[i][j] + Q[i][j] : Y[i][j];
#pragma unroll
            for (int k2 = 0; k2 < D; k2++)
                if (SP::dl(j, k2)) acc = fma(Y[i][k2], Dl[j][k2], acc);
            Pp[i][j] = acc;
            Pp[j][i] = acc;
        }
}

// One step of the fixed-point smoother of the state before the lane
// (lane_smoother_element), in two parts so that the transition's operands are
// dead before the conditioning: G <- F G with Dl = F - I, and the update with
// gain K, innovation v, w = 1 / S (0 at a missing step) and r = R / S (1
// there). h (I - K h) = r h: the observed row of G is scaled by r, since
// 1 - h K would lose log10(S / R) digits. P0 is kept in its upper triangle;
// B as in smoother_shear_col.
template <int D, class SP>
__device__ __forceinline__ void fixed_point_predict(const double (&Dl)[D][D], double (&G)[D][D])
{
#pragma unroll
    for (int c = 0; c < D; c++) {
        double g[D];
#pragma unroll
        for (int i = 0; i < D; i++) {
            double acc = G[i][c];
#pragma unroll
            for (int q = 0; q < D; q++)
                if (SP::dl(i, q)) acc = fma(Dl[i][q], G[q][c], acc);
            g[i] = acc;
        }
#pragma unroll
        for (int i = 0; i < D; i++) G[i][c] = g[i];
    }
}

template <int D, int B, class SP>
__device__ __forceinline__ void fixed_point_update(const double (&K)[D], double v, double w, double r,
                                                   double (&m0)[D], double (&P0)[D][D], double (&G)[D][D])
{
    double wh[D];
#pragma unroll
    for (int c = 0; c < D; c++) {
        double acc = 0.0;
#pragma unroll
        for (int i = 0; i < D; i++)
            if (SP::obs(i)) acc += G[i][c];
        wh[c] = acc;
#pragma unroll
        for (int i = 1; i < D; i++) G[i][c] = fma(-K[i], acc, G[i][c]);
        G[0][c] = B > 0 ? fma(r, acc, -G[B][c]) : r * acc;
    }
#pragma unroll
    for (int i = 0; i < D; i++) {
        const double a = wh[i] * w;
        m0[i] = fma(a, v, m0[i]);
#pragma unroll
        for (int j = i; j < D; j++) P0[i][j] = fma(-a, wh[j], P0[i][j]);
    }
}

// Whether the fold leaves the lane scan to lane_scan_kernel: at d >= 6 in FP64
// (filter and smoother: 2 000 steps at d = 6 357 -> 272 us, at d = 8 634 -> 379;
// 131 101 steps at d = 8 890 -> 685 with the chunk chosen for it and the
// symmetric form of the scan); in FP32 at
// d = 8 up to two workgroups a CU (1 000 steps 551 -> 469, 320 000 steps 679 ->
// 618 us; 2^20 steps 778 -> 821 to 900). There, and at d = 6 in FP32 at any size
// (1 000 steps 249 -> 264), the workgroup of tile 0 with its FP64 conditioning
// takes longest, and every wave forming the factors costs more than it saves
// once the SIMDs are full.
template <int D, typename T>
constexpr bool may_split() { return D >= 6 && (sizeof(T) == 8 || D >= 8); }
template <int D, typename T>
__host__ __device__ constexpr bool split_lane_scan(int ntiles)
{
    return may_split<D, T>() && (sizeof(T) == 8 || ntiles <= 512);
}

// Fold pass of one tile: each lane folds its chunk into an aggregate, the
// wave scans the 64 chunk aggregates (inclusive, time order) and stores them
// at lanep; lane 63 then holds the tile aggregate.
template <class LY, typename T, typename CT, bool SPLIT, class SV>
__device__ __forceinline__ void filter_tile_fold(const FilterParams<T> &p, const DevModel &mdl, cdouble *cst,
                                                 SV &sv, const TileRange &tr, int tile)
{
    constexpr int D = LY::D;
    constexpr int AGG = AggLayout<D>::SIZE;
    const int lane = lane_id();
    const int slot = tr.slot_base + tile;
    const int64_t chunk_id = (int64_t)slot * PSSGP_WAVE + lane;
    const int64_t k0 = tr.k_begin + ((int64_t)tile * PSSGP_WAVE + lane) * p.chunk;
    const int64_t k1 = (k0 + p.chunk < tr.k_end) ? k0 + p.chunk : tr.k_end;
    T h[D];
#pragma unroll
    for (int i = 0; i < D; i++) h[i] = T(LY::hobs(i));
    FAgg<D, T> agg;
    agg_identity<D, T>(agg);
    bool from_start = false;  // the aggregate covers a series start, so its A is 0
    StepInputs<T> in;
    in.start(p.t, p.y, p.mask, k0, k1, tr.k_begin);
    const OptInputs opt(p.mask, p.noise_k, p.t);
    for (int64_t k = k0; k < k1; k++) {
        const int64_t kn = (k + 1 < k1) ? k + 1 : k;
        const double tn = p.t[kn];
        const T yn = p.y[kn];
        const bool on = opt.observed(kn);
        const T R = T(opt.noise_var(k));
        if constexpr (reload_constants<D>()) PSSGP_RELOAD_CONSTANTS();
        sv.seek(k);
        const bool first = sv.first(k);
        from_start = from_start || first;
        const double dt = first ? 0.0 : in.tc - in.tp;
        cdouble *c = cst;
        if constexpr (reload_constants<D>()) PSSGP_LAUNDER(c);
        T Dl[D][D], Q[D][D];
        step_transition<LY, T, T>(mdl, c, sv.sc, dt, first, Dl, Q);
        const T yk = in.oc ? in.yc : T(0);
        agg_fold<D, T, Sparsity<LY>>(agg, Dl, Q, h, p.noise_k ? R : T(sv.R), yk, in.oc);
        in.tp = in.tc;
        in.tc = tn;
        in.yc = yn;
        in.oc = on;
    }
    if constexpr (SPLIT) {
        agg_store<D, T>(lane_rec(p.lanep, slot, AGG, lane), agg, PSSGP_WAVE);
        return;
    }
    for (int o = 1; o < PSSGP_WAVE; o <<= 1) {
        FAgg<D, T> other;
        agg_shfl_up<D, T>(agg, other, o);
        const bool other_from_start = __shfl_up((int)from_start, o, PSSGP_WAVE) != 0;
        if (lane >= o) {
            if (other_from_start) {
                // the earlier prefix starts at a series start: it is a pair of
                // filter moments (A = 0; its eta, J are never used again), and
                // the combination is its conditioning on the later aggregate,
                // which cancels when that aggregate is informative: in FP64
                moments_apply<D, T, double>(other.b, other.C, agg, agg.b, agg.C);
#pragma unroll
                for (int i = 0; i < D; i++) {
                    agg.eta[i] = T(0);
#pragma unroll
                    for (int j = 0; j < D; j++) { agg.A[i][j] = T(0); agg.J[i][j] = T(0); }
                }
            } else {
                agg_combine<D, T, CT>(other, agg, agg);
            }
            from_start = from_start || other_from_start;
        }
    }
    agg_store<D, T>(lane_rec(p.lanep, slot, AGG, lane), agg, PSSGP_WAVE);
    if (lane == PSSGP_WAVE - 1) agg_store<D, T>(p.aggp + (size_t)slot * AGG, agg);  // tile aggregate
}

// Finish pass of one tile: each lane takes the moments entering the tile
// (carry pass), applies its exclusive lane prefix (every prefix from a
// series start has A = 0, so only (b, C) are carried) and re-runs its steps
// as a plain Kalman filter, writing (m, P) and summing the log-likelihood
// terms in FP64. ll_out receives this lane's partial.
template <class LY, typename T, typename CT, int MODE, class SV>
__device__ __forceinline__ void filter_tile_finish(const FilterParams<T> &p, const DevModel &mdl,
                                                   cdouble *cst, SV &sv, const TileRange &tr, int tile,
                                                   double &ll_out)
{
    constexpr int D = LY::D;
    constexpr int AGG = AggLayout<D>::SIZE;
    constexpr int INCL = AggLayout<D>::INCL;
    const int lane = lane_id();
    const int slot = tr.slot_base + tile;
    const int64_t chunk_id = (int64_t)slot * PSSGP_WAVE + lane;
    const int64_t k0 = tr.k_begin + ((int64_t)tile * PSSGP_WAVE + lane) * p.chunk;
    const int64_t k1 = (k0 + p.chunk < tr.k_end) ? k0 + p.chunk : tr.k_end;
    using SP = Sparsity<LY>;
    T h[D];
#pragma unroll
    for (int i = 0; i < D; i++) h[i] = T(LY::hobs(i));
    uint32_t bad = 0;

    constexpr bool ELEMS = (MODE & F_ELEMS) != 0, LANES = (MODE & F_LANES) != 0;
    using HL = HandLayout<D>;
    // smoother lane aggregate accumulated from the handed-over elements
    constexpr bool LANEAGG = ELEMS && lane_aggregate_handover<D>();
    SAgg<D, T> sacc;
    if constexpr (LANEAGG || LANES) sagg_identity<D, T>(sacc);

    T m0[D], P0[D][D];
    moments_load<D, T>(p.inclp + (size_t)slot * INCL, m0, P0);
    // the first step's inputs are requested before the lane's entering
    // moments are formed, so that their latency overlaps that arithmetic
    StepInputs<T> in;
    in.start(p.t, p.y, p.mask, k0, k1, tr.k_begin);
    if (lane > 0) {
        FAgg<D, T> excl;
        agg_load<D, T>(lane_rec(p.lanep, slot, AGG, lane - 1), excl, PSSGP_WAVE);
        moments_apply<D, T, CT>(m0, P0, excl, m0, P0);
    }
    // the lane carries its filter moments in FP64 from step to step: the
    // prediction and the conditioning are FP64 anyway, and the moments in T
    // would cost a conversion each way per step
    double m[D], P[D][D];
#pragma unroll
    for (int i = 0; i < D; i++) {
        m[i] = (double)m0[i];
#pragma unroll
        for (int j = 0; j < D; j++) P[i][j] = (double)P0[i][j];
    }
    // fixed-point smoother of the lane's first step (lane_smoother_element),
    // set at the end of that step
    double fm[D], fP[D][D], fG[D][D];
    if constexpr (LANES) {
#pragma unroll
        for (int i = 0; i < D; i++) {
            fm[i] = m[i];
#pragma unroll
            for (int j = 0; j < D; j++) fP[i][j] = fG[i][j] = P[i][j];
        }
    }

    double ll = 0.0;  // FP64 per-lane sum of the log-likelihood terms
    // many series: one FP64 partial sum of the terms per series segment of
    // the lane, stored at the segment's first step (series_loglik_kernel
    // reads the series start and the lane starts inside the series)
    constexpr bool SEG = !std::is_same<SV, OneSeries>::value;
    double seg = 0.0;
    int64_t seg_k = k0;
    // the first step's inputs are waited for before the loop, so that the
    // loop's first use of them carries no wait into later iterations
    asm volatile("" ::"v"(in.tc), "v"(in.tp), "v"(in.yc), "v"((int)in.oc));
    const OptInputs opt(p.mask, p.noise_k, p.t);
    // a series that ends with the lane: the fixed-point smoother has seen all
    // its observations (E = 0), and there is no step after to end the run with
    const bool end = k1 >= tr.k_end;
    static_assert(!LANES || !SEG, "a run over series starts");
    const int64_t ke = (LANES && k1 > k0 && !end) ? k1 + 1 : k1;
    for (int64_t k = k0; k < ke; k++) {
        // (F_ELEMS: the last step of the lane loads the time of the next lane's
        // first step, which its smoother element needs after the loop: no load
        // after the loop waits behind the element stores)
        const int64_t kn = (k + 1 < (ELEMS ? tr.k_end : ke)) ? k + 1 : k;
        const double tn = p.t[kn];
        const T yn = p.y[kn];
        const bool on = opt.observed(kn);
        const T Rk = T(opt.noise_var(k));
        if constexpr (reload_constants<D>()) PSSGP_RELOAD_CONSTANTS();
        sv.seek(k);
        const bool first = sv.first(k);
        const double dt = first ? 0.0 : in.tc - in.tp;
        if (!(dt >= 0.0)) bad |= (dt < 0.0) ? PSSGP_STATUS_UNSORTED : PSSGP_STATUS_NONFINITE;
        cdouble *c = cst;
        if constexpr (reload_constants<D>()) PSSGP_LAUNDER(c);
        double Dl[D][D], Q[D][D];
        step_transition<LY, double, T>(mdl, c, sv.sc, dt, first, Dl, Q);
        const bool obs = in.oc;
        const T yk = obs ? in.yc : T(0);
        const T R = p.noise_k ? Rk : T(sv.R);
        in.tp = in.tc;
        in.tc = tn;
        in.yc = yn;
        in.oc = on;
        // predict in FP64 (mp = F m, Y = F P, Pp = F P F^T + Q)
        double mp[D], Y[D][D], Pp[D][D];
        predict_step<D, double, Sparsity<LY>>(m, P, Dl, Q, mp, Y, Pp);
        // (the fixed-point smoother of the lane's first step is overwritten
        // below; a branch around it costs 5 % of the call at d = 6 and gains 2 %
        // at d = 8)
        if constexpr (LANES) {
            if (D <= 6 || k > k0) fixed_point_predict<D, Sparsity<LY>>(Dl, fG);
        }
        // the loads of this iteration are waited for here, before the
        // handover stores: the wait counter is in order, so a wait after
        // the stores would also wait for all of them
        asm volatile("" ::"v"(tn), "v"(yn), "v"((int)on), "v"(Rk));
        if constexpr (ELEMS) {
            // smoother element of the previous step of this lane
            if (k > k0) {
                SAgg<D, T> e;
                smoother_element_from_prediction<D, smoother_shear_col<LY>(), T, double>(m, P, Y, mp, Pp, e, bad);
                hand_over_element<D, T, LANEAGG>(e, p.elem + elem_index<D>(slot, p.chunk, (int)(k - 1 - k0), lane),
                                                 sacc);
            }
        }
        // conditioning on y_k in FP64 (symmetric form): the subtraction
        // that cancels when the noise is small against the predicted
        // variance is done in FP64
        double Ph[D], S = (double)R, hm = 0.0;
#pragma unroll
        for (int i = 0; i < D; i++) {
            double acc = 0.0;
#pragma unroll
            for (int j = 0; j < D; j++)
                if (SP::obs(j)) acc = fma(Pp[i][j], (double)h[j], acc);
            Ph[i] = acc;
            if (SP::obs(i)) hm = fma((double)h[i], mp[i], hm);
        }
#pragma unroll
        for (int i = 0; i < D; i++)
            if (SP::obs(i)) S = fma((double)h[i], Ph[i], S);
        const double v = (double)yk - hm;
        const double w = obs ? rcp64(S) : 0.0;
        // branch-free: missing steps add an exact zero
        bad |= (obs && (!(S > 0.0) || !isfinite(S))) ? PSSGP_STATUS_BAD_S : 0u;
        bad |= (obs && !isfinite(yk)) ? PSSGP_STATUS_NONFINITE : 0u;
        // log(2 pi S): in FP32 for the FP32 scans (the hardware base-2
        // logarithm, about 1e-7 absolute on a term of size 1, far below the
        // FP32 tolerance of the sum), in FP64 otherwise
        double lg;
        if constexpr (sizeof(T) == 4)
            lg = (double)__builtin_amdgcn_logf((float)(6.283185307179586 * S)) * 0.6931471805599453;
        else
            lg = log(6.283185307179586 * S);
        const double term = (obs && (!LANES || k < k1)) ? -0.5 * (lg + v * v * w) : 0.0;
        if constexpr (SEG) {
            if (first && k > k0) {
                if (p.ll_terms) p.ll_terms[seg_k] = seg;
                seg = 0.0;
                seg_k = k;
            }
            seg += term;
        } else {
            if (p.ll_terms && (!LANES || k < k1)) p.ll_terms[k] = term;
        }
        ll += term;
        double K[D];
#pragma unroll
        for (int i = 0; i < D; i++) K[i] = Ph[i] * w;
        if constexpr (LANES) {
            // non-temporal: read back by the smoother after all of it is written
            double *hp = p.hand + HL::step(slot, p.chunk, (int)(k - k0), lane);
#pragma unroll
            for (int i = 0; i < D; i++) __builtin_nontemporal_store(Ph[i], hp + i * PSSGP_WAVE);
            __builtin_nontemporal_store(hm, hp + D * PSSGP_WAVE);
            __builtin_nontemporal_store(obs ? v : 0.0, hp + (D + 1) * PSSGP_WAVE);
            __builtin_nontemporal_store(__builtin_copysign(dt, obs ? 1.0 : -1.0), hp + (D + 2) * PSSGP_WAVE);
            const double r = obs ? (double)R * w : 1.0;
            fixed_point_update<D, smoother_shear_col<LY>(), Sparsity<LY>>(K, v, w, r, fm, fP, fG);
        }
        if constexpr ((MODE & F_RECS) != 0) {
            constexpr int NS = RecLayout<D>::NS;
            constexpr size_t W = PSSGP_WAVE;
            // non-temporal: the records are read back by the adjoint only
            // after all of them have been written
            T *rp = p.rec + rec_index<D>(slot, p.chunk, (int)(k - k0), lane);
#pragma unroll
            for (int i = 0; i < D; i++) {
                __builtin_nontemporal_store(T(mp[i]), rp + i * W);
                __builtin_nontemporal_store(T(K[i]), rp + (D + NS + i) * W);
            }
#pragma unroll
            for (int i = 0; i < D; i++)
#pragma unroll
                for (int j = i; j < D; j++) __builtin_nontemporal_store(T(Pp[i][j]), rp + (D + sidx<D>(i, j)) * W);
            __builtin_nontemporal_store(T(S), rp + (2 * D + NS) * W);
            __builtin_nontemporal_store(obs ? T(v) : T(0), rp + (2 * D + NS + 1) * W);
        }
#pragma unroll
        for (int i = 0; i < D; i++) m[i] = fma(K[i], v, mp[i]);
#pragma unroll
        for (int i = 0; i < D; i++)
#pragma unroll
            for (int j = i; j < D; j++) {
                const double c = fma(S * K[i], K[j], fma(-Ph[i], K[j], fma(-K[i], Ph[j], Pp[i][j])));
                P[i][j] = c;
                P[j][i] = c;
            }
        if constexpr (LANES) {
            // from here on
            if (k == k0) {
#pragma unroll
                for (int i = 0; i < D; i++) {
                    fm[i] = m[i];
#pragma unroll
                    for (int j = 0; j < D; j++) fP[i][j] = fG[i][j] = P[i][j];
                }
            }
        }
        if constexpr ((MODE & F_MOMENTS) != 0) {
#pragma unroll
            for (int i = 0; i < D; i++) p.m[(size_t)i * p.n + k] = T(m[i]);
#pragma unroll
            for (int i = 0; i < D; i++)
#pragma unroll
                for (int j = i; j < D; j++) p.P[(size_t)sidx<D>(i, j) * p.n + k] = T(P[i][j]);
        }
    }
    if constexpr (ELEMS) {
        // element of the lane's last step: predict the next step (the first of
        // the next lane), or take the prior transition at a series end
        if (k1 > k0) {
            sv.seek(k1 - 1);
            const bool last = end || sv.last(k1 - 1);
            const double dt = last ? 0.0 : in.tc - in.tp;  // t[k1] - t[k1 - 1]
            cdouble *c = cst;
            PSSGP_LAUNDER(c);
            double Dl[D][D], Q[D][D], mp[D], Y[D][D], Pp[D][D];
            step_transition<LY, double, T>(mdl, c, sv.sc, dt, last, Dl, Q);
            predict_step<D, double, Sparsity<LY>>(m, P, Dl, Q, mp, Y, Pp);
            SAgg<D, T> e;
            smoother_element_from_prediction<D, smoother_shear_col<LY>(), T, double>(m, P, Y, mp, Pp, e, bad);
            hand_over_element<D, T, LANEAGG>(e, p.elem + elem_index<D>(slot, p.chunk, (int)(k1 - 1 - k0), lane), sacc);
        }
    }
    if constexpr (LANES) {
        // the lane's smoother element (identity for a lane without steps) and
        // its end moments, the covariance as its Cholesky factor
        if (k1 > k0) {
            // (the last conditioning from the handover: kept in registers over
            // the loop it cost 5 % of the call at d = 8)
            constexpr int B = smoother_shear_col<LY>();
            const double *hp = p.hand + HL::step(slot, p.chunk, (int)(ke - 1 - k0), lane);
            double C[D][D], rd[D], ph[D];
#pragma unroll
            for (int i = 0; i < D; i++) ph[i] = hp[i * PSSGP_WAVE];
            const double hph = B > 0 ? ph[0] + ph[B] : ph[0], R = (double)T(sv.R);
            const bool obs = !__builtin_signbit(hp[(D + 2) * PSSGP_WAVE]);
            const double w = obs ? rcp64(R + hph) : 0.0;
            const double f = fma(hph * w, hp[(D + 1) * PSSGP_WAVE], hp[D * PSSGP_WAVE]);
            lane_smoother_element<D, B, T>(fm, fP, fG, m, P, f, ph, obs ? R * w : 1.0, end, C, rd, sacc, bad);
            double *bp = p.bound + HL::lane(slot, lane);
#pragma unroll
            for (int i = 0; i < D; i++) {
                bp[i * PSSGP_WAVE] = m[i];
#pragma unroll
                for (int j = 0; j <= i; j++)
                    bp[(D + sidx<D>(j, i)) * PSSGP_WAVE] = (i == j) ? rd[i] : C[i][j];
            }
        }
    }
    if constexpr (LANEAGG || LANES) {
        // the smoother's fold pass over this tile, done here: the wave scans
        // the lanes' smoother aggregates (identity for a lane without steps)
        // as suffixes (inclusive, reverse time order) into the lane records
        // at slane, and lane 0 stores the tile aggregate in the scan region
        // the two scans share (the filter's carry has consumed it)
        constexpr int SAGG = SAggLayout<D>::SIZE;
        for (int o = 1; o < PSSGP_WAVE; o <<= 1) {
            SAgg<D, T> other;
            sagg_shfl_down<D, T>(sacc, other, o);
            if (lane + o < PSSGP_WAVE) sagg_combine<D, T>(sacc, other, sacc);
        }
        sagg_store<D, T>(lane_rec(p.slane, slot, SAGG, lane), sacc, PSSGP_WAVE);
        if (lane == 0) sagg_store<D, T>(p.aggp + (size_t)slot * SAGG, sacc);
    }
    if constexpr (SEG) {
        if (p.ll_terms && k1 > k0) p.ll_terms[seg_k] = seg;
    }
    if (bad) status_or(&p.ctl->status, bad);
    ll_out = ll;
}

// CT: arithmetic type of the lane scan's combinations. SPLIT: lane_scan_kernel
// does the lane scan (a template argument: with both in one kernel the fold of
// 2^20 steps at d = 8 took 150 us more)
template <class LY, typename T, typename CT, bool SPLIT>
__global__ __launch_bounds__(PSSGP_WAVE, (fold_waves<LY::D, T>())) void filter_fold_kernel(FilterParams<T> p,
                                                                                        DevModel mdl_arg)
{
    __shared__ DevModel mdl;
    model_to_lds(mdl_arg, mdl);
    OneSeries sv;
    sv.init(mdl, p.n);
    TileRange tr{0, p.n, p.ntiles, 0};
    filter_tile_fold<LY, T, CT, SPLIT, OneSeries>(p, mdl, (cdouble *)p.cst, sv, tr, (int)blockIdx.x);
}

template <class LY, typename T, typename CT, int MODE>
__global__ __launch_bounds__(PSSGP_WAVE, (finish_waves<LY::D, T>())) void filter_finish_kernel(FilterParams<T> p,
                                                                                            DevModel mdl_arg)
{
    __shared__ DevModel mdl;
    const int lane = lane_id();
    const int tile = (int)blockIdx.x;
    model_to_lds(mdl_arg, mdl);
    OneSeries sv;
    sv.init(mdl, p.n);
    TileRange tr{0, p.n, p.ntiles, 0};
    double ll = 0.0;
    filter_tile_finish<LY, T, CT, MODE, OneSeries>(p, mdl, (cdouble *)p.cst, sv, tr, tile, ll);

    // log-likelihood: deterministic wave sum, tile partial; the partials are
    // summed in a fixed order here, by the smoother of the same call or by
    // launch_tile_sums
    const double tot = wave_sum(ll);
    if (lane == 0) p.partials[tile] = tot;
    if constexpr (!(MODE & (F_ELEMS | F_LANES))) {
        if (p.ntiles <= LAST_TILES && last_tile(p.ctl, p.ntiles)) {
            const double s = sum_over_tiles(p.partials, p.ntiles, 1);
            if (lane == 0) *p.loglik = s;
        }
    }
}

// One thread per step: F[k] (row-major d*d) and Q[k] (packed, entry-major).
template <class LY>
__global__ __launch_bounds__(256) void discretize_kernel(DevModel mdl, const double *t, int64_t n,
                                                         double *Fo, double *Qo, WsCtl *ctl)
{
    constexpr int D = LY::D;
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    double F[D][D], Q[D][D];
    const double dt = (k > 0) ? t[k] - t[k - 1] : 0.0;
    if (!(dt >= 0.0)) status_or(&ctl->status, (dt < 0.0) ? PSSGP_STATUS_UNSORTED : PSSGP_STATUS_NONFINITE);
    discretize<LY, false>(mdl, (cdouble *)nullptr, model_scale(mdl), dt, k == 0, F, Q);
#pragma unroll
    for (int i = 0; i < D; i++)
#pragma unroll
        for (int j = 0; j < D; j++) Fo[(size_t)k * D * D + i * D + j] = F[i][j];
#pragma unroll
    for (int i = 0; i < D; i++)
#pragma unroll
        for (int j = i; j < D; j++) Qo[(size_t)sidx<D>(i, j) * n + k] = Q[i][j];
}

template <class LY, typename T>
FilterParams<T> filter_params(const FilterLaunch &a)
{
    FilterParams<T> p;
    p.t = a.t;
    p.y = (const T *)a.y;
    p.mask = a.mask;
    p.noise_k = a.noise_k;
    p.n = a.n;
    p.chunk = a.chunk;
    p.ntiles = a.ntiles;
    p.m = (T *)a.m;
    p.P = (T *)a.P;
    p.loglik = a.loglik;
    p.rec = (T *)a.rec;
    p.ll_terms = nullptr;
    p.cst = a.ws.cst;
    p.ctl = a.ws.ctl;
    p.inclp = (T *)a.ws.inclp;
    p.aggp = (T *)a.ws.aggp;
    p.lanep = (T *)a.ws.lanep;
    p.partials = a.ws.partials;
    p.elem = (T *)a.elem;
    p.hand = a.hand;
    p.bound = a.bound;
    p.slane = (T *)a.slane;
    return p;
}

template <class LY, typename T, typename CT>
int launch_filter_t(const DevModel &mdl, const FilterLaunch &a, hipStream_t s)
{
    FilterParams<T> p = filter_params<LY, T>(a);
    const dim3 grid(a.ntiles), block(PSSGP_WAVE);
    pass_event(a.ev, 0, s);
    launch_consts<LY, T>(mdl, a.ws.cst, s);
    if constexpr (may_split<LY::D, T>()) {
        if (split_lane_scan<LY::D, T>(a.ntiles)) {
            hipLaunchKernelGGL((filter_fold_kernel<LY, T, T, true>), grid, block, 0, s, p, mdl);
            hipLaunchKernelGGL((lane_scan_kernel<LY::D, T>), grid, dim3(PSSGP_WAVE * LY::D / 2), 0, s, p.lanep, p.aggp);
        }
    }
    if constexpr (!split_lane_scan<LY::D, T>(1 << 30)) {
        if (!split_lane_scan<LY::D, T>(a.ntiles))
            hipLaunchKernelGGL((filter_fold_kernel<LY, T, T, false>), grid, block, 0, s, p, mdl);
    }
    int rc = (int)hipGetLastError();
    if (rc) return rc;
    pass_event(a.ev, 1, s);
    if (a.rec) {
        // forward pass of the gradient: the finish writes the per-step
        // records of the adjoint (from its FP64 prediction). (The carry scan in
        // FP64 as well measured no gain in accuracy once the series-start
        // prefixes and lane starts were conditioned in FP64: noise-variance
        // derivative 8.6e-5 vs 7.0e-5 at d = 8, 2^20 steps, at 2.5x the carry
        // time.)
        rc = launch_filter_carry<LY::D, T, CT>(a.ws, 0, a.ntiles, s);
        if (rc) return rc;
        pass_event(a.ev, 2, s);
        hipLaunchKernelGGL((filter_finish_kernel<LY, T, double, F_RECS>), grid, block, 0, s, p, mdl);
    } else {
        rc = launch_filter_carry<LY::D, T, CT>(a.ws, 0, a.ntiles, s);
        if (rc) return rc;
        pass_event(a.ev, 2, s);
        // lane-start moments (the lane's exclusive prefix applied to the
        // tile's carry, once per lane) in FP64
        if (a.fused)
            hipLaunchKernelGGL((filter_finish_kernel<LY, T, double, fused_mode<LY::D, T>()>), grid, block, 0, s, p, mdl);
        else if (a.m)
            hipLaunchKernelGGL((filter_finish_kernel<LY, T, double, F_MOMENTS>), grid, block, 0, s, p, mdl);
        else
            hipLaunchKernelGGL((filter_finish_kernel<LY, T, double, 0>), grid, block, 0, s, p, mdl);
    }
    rc = (int)hipGetLastError();
    if (rc) return rc;
    // (the gradient call sums both its passes after the second)
    if (!a.fused && !a.rec && a.ntiles > LAST_TILES) rc = launch_tile_sums(a.ws.partials, a.loglik, nullptr, nullptr, 0, a.ntiles, s);
    pass_event(a.ev, 3, s);
    return rc;
}

template <int B0, int B1>
int launch_filter_layout(const DevModel &mdl, bool f64, const FilterLaunch &a, hipStream_t s)
{
    return f64 ? launch_filter_t<Layout<B0, B1>, double, double>(mdl, a, s)
               : launch_filter_t<Layout<B0, B1>, float, typename CombineType<float>::type>(mdl, a, s);
}

template <int B0, int B1>
int launch_discretize_layout(const DevModel &mdl, const double *t, int64_t n, double *F, double *Q,
                             WsCtl *ctl, hipStream_t s)
{
    const dim3 grid((unsigned)((n + 255) / 256)), block(256);
    hipLaunchKernelGGL((discretize_kernel<Layout<B0, B1>>), grid, block, 0, s, mdl, t, n, F, Q, ctl);
    return (int)hipGetLastError();
}
