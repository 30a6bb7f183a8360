// Parallel RTS smoother (supplement, eq. smoother and Proposition 2) as a
// reverse scan over the elements (E, g, L).
//
// Element of step k (built in FP64 from the FP64 discretisation of
// dt = t[k+1] - t[k] and the filter moments (m_k, P_k)):
//   E_k = P_k F^T (F P_k F^T + Q)^-1     (Cholesky of the predicted covariance)
//   g_k = m_k - E_k F m_k,   L_k = P_k - E_k F P_k
// and (0, m, P) at the last step. Operator, x earlier than y:
//   (E_x, g_x, L_x) (x) (E_y, g_y, L_y) = (E_x E_y, E_x g_y + g_x, E_x L_y E_x^T + L_x)
// Every suffix that ends at the last step has E = 0 and its (g, L) are the
// smoothed moments.
//
// Three passes in reverse time order (tile_scan.h), one wave per tile and
// `chunk` steps per lane:
//   fold    each lane composes its elements from right to left; wave-level
//           inclusive suffix scan (Kogge-Stone over lane shuffles); each
//           lane stores its inclusive suffix aggregate
//   carry   one workgroup scans the tile aggregates from the end and stores
//           the smoothed moments after every tile
//   finish  each lane applies its exclusive lane suffix to the carry, giving
//           the smoothed moments after its chunk, and runs the RTS recursion
//           backwards over its steps, writing H m^s and H P^s H^T.
#pragma once
#include "device_common.h"
#include "launch.h"
#include "smoother_ops.h"
#include "tile_scan.h"

template <typename T>
struct SmoothParams {
    const double *t;
    const T *m;
    const T *P;
    int64_t n;
    int chunk;
    int ntiles;
    T *f_mean;
    T *f_var;
    T *ms;
    T *Ps;
    WsCtl *ctl;
    T *aggp;
    T *inclp;
    T *lanep;
    const double *cst;  // model constants of the transition
    const double *partials;  // fused call: the filter's log-likelihood by tiles, and its sum
    double *loglik;
    const T *elem;           // fused call, an element per step (elem_index)
    const double *hand;      // fused call, an element per lane (HandLayout) and
    const double *bound;
};

struct STileRange {
    int64_t k_begin, k_end;
    int ntiles;
    int slot_base;
};

// Fold pass of one tile: each lane composes its chunk's elements from the
// right, the wave scans the 64 chunk aggregates as suffixes (inclusive,
// reverse time order) and stores them at lanep; lane 0 then holds the tile
// aggregate.
template <class LY, typename T, bool ELEMS, class SV>
__device__ __forceinline__ void smoother_tile_fold(const SmoothParams<T> &p, const DevModel &mdl,
                                                   cdouble *cst, SV &sv, const STileRange &tr, int tile)
{
    constexpr int D = LY::D;
    constexpr int AGG = SAggLayout<D>::SIZE;
    const int lane = lane_id();
    const int slot = tr.slot_base + tile;
    const int64_t chunk_id = (int64_t)slot * PSSGP_WAVE + lane;
    const int64_t k0 = tr.k_begin + ((int64_t)tile * PSSGP_WAVE + lane) * p.chunk;
    const int64_t k1 = (k0 + p.chunk < tr.k_end) ? k0 + p.chunk : tr.k_end;
    uint32_t bad = 0;  // reported by the finish pass
    SAgg<D, T> agg;
    sagg_identity<D, T>(agg);
    // (a fused call with lane aggregates has its fold pass done by the
    // filter's finish pass and does not launch this one)
    for (int64_t k = k1 - 1; k >= k0; k--) {
        if constexpr (reload_constants<D>()) PSSGP_RELOAD_CONSTANTS();
        sv.seek(k);
        SAgg<D, T> e;
        if constexpr (ELEMS) {
            sagg_load_nt<D, T>(p.elem + elem_index<D>(slot, p.chunk, (int)(k - k0), lane), e, PSSGP_WAVE);
        } else {
            cdouble *c = cst;
            if constexpr (reload_constants<D>()) PSSGP_LAUNDER(c);
            smoother_element<LY, T, SV>(mdl, c, sv, p.t, p.m + k, p.P + k, (size_t)p.n, k, e, bad);
        }
        sagg_combine<D, T>(e, agg, agg);
    }
    if constexpr (smoother_by_rows<D, T>()) {
        // the lane scan runs by rows (rows_lane_scan)
        sagg_store<D, T>(lane_rec(p.lanep, slot, AGG, lane), agg, PSSGP_WAVE);
    } else {
        for (int o = 1; o < PSSGP_WAVE; o <<= 1) {
            SAgg<D, T> other;
            sagg_shfl_down<D, T>(agg, other, o);
            if (lane + o < PSSGP_WAVE) sagg_combine<D, T>(agg, other, agg);
        }
        sagg_store<D, T>(lane_rec(p.lanep, slot, AGG, lane), agg, PSSGP_WAVE);
        if (lane == 0) sagg_store<D, T>(p.aggp + (size_t)slot * AGG, agg);  // tile aggregate
    }
}

// Finish pass of one tile: each lane takes the smoothed moments entering
// the tile from the right (carry pass), applies its exclusive lane suffix
// and runs the backward RTS recursion over its chunk.
// Steps whose handed-over elements it loads ahead of their use, per group
// (small states only: their per-step work is short against a load's latency).
template <int D>
constexpr int smoother_prefetch_group()
{
    return D <= 2 ? 4 : (D == 3 ? 2 : 1);
}

template <class LY, typename T, bool FULL, bool ELEMS, class SV>
__device__ __forceinline__ void smoother_tile_finish(const SmoothParams<T> &p, const DevModel &mdl,
                                                     cdouble *cst, SV &sv, const STileRange &tr, int tile,
                                                     T *s_out)
{
    constexpr int D = LY::D;
    constexpr int AGG = SAggLayout<D>::SIZE;
    constexpr int INCL = SAggLayout<D>::INCL;
    const int lane = lane_id();
    const int slot = tr.slot_base + tile;
    const int64_t chunk_id = (int64_t)slot * PSSGP_WAVE + lane;
    const int64_t k0 = tr.k_begin + ((int64_t)tile * PSSGP_WAVE + lane) * p.chunk;
    const int64_t k1 = (k0 + p.chunk < tr.k_end) ? k0 + p.chunk : tr.k_end;
    uint32_t bad = 0;
    // the elements and moments are in the smoother's coordinates
    constexpr int B = smoother_shear_col<LY>();
    T h[D];
    smoother_obs_row<D, B, T>(mdl, h);
    const int64_t tile_start = tr.k_begin + (int64_t)tile * PSSGP_WAVE * p.chunk;
    const int tile_len = PSSGP_WAVE * p.chunk;

    T ms[D], Ps[D][D];
    gl_load<D, T>(p.inclp + (size_t)slot * INCL, ms, Ps);
    if (lane < PSSGP_WAVE - 1) {
        SAgg<D, T> excl;
        sagg_load<D, T>(lane_rec(p.lanep, slot, AGG, lane + 1), excl, PSSGP_WAVE);
        sagg_apply<D, T>(excl, ms, Ps, ms, Ps);
    }
    // one step of the backward recursion from its element
    auto step_out = [&](const SAgg<D, T> &e, int64_t k) {
        sagg_apply<D, T>(e, ms, Ps, ms, Ps);
        T Ph[D];
        mat_vec<D, T>(Ps, h, Ph);
        // f outputs staged in LDS (index k - tile start) for coalesced stores
        s_out[k - tile_start] = dot<D, T>(h, ms);
        s_out[tile_len + (k - tile_start)] = dot<D, T>(h, Ph);
        if constexpr (FULL) {
            T mo[D], Po[D][D];
            from_smoother_coords<D, B, T>(ms, Ps, mo, Po);
#pragma unroll
            for (int i = 0; i < D; i++) p.ms[(size_t)i * p.n + k] = mo[i];
#pragma unroll
            for (int i = 0; i < D; i++)
#pragma unroll
                for (int j = i; j < D; j++) p.Ps[(size_t)sidx<D>(i, j) * p.n + k] = Po[i][j];
        }
    };
    // (single series only: in the batched form, chunk 16 over series of
    // uneven lengths, the grouping measured 5 % slower)
    constexpr int G = std::is_same<SV, OneSeries>::value ? smoother_prefetch_group<D>() : 1;
    if constexpr (ELEMS && G > 1) {
        // small states: the elements of the next G steps are loaded while
        // the current G are processed (a lane's recursion is otherwise one
        // dependent load per step); indices below k0 are clamped to k0, so
        // every load is in the tile's region and none sits in a branch
        auto load = [&](int64_t k, SAgg<D, T> &e) {
            const int j = k >= k0 ? (int)(k - k0) : 0;
            sagg_load_nt<D, T>(p.elem + elem_index<D>(slot, p.chunk, j, lane), e, PSSGP_WAVE);
        };
        SAgg<D, T> cur[G], nxt[G];
#pragma unroll
        for (int g = 0; g < G; g++) load(k1 - 1 - g, cur[g]);
        for (int64_t kb = k1 - 1; kb >= k0; kb -= G) {
#pragma unroll
            for (int g = 0; g < G; g++) load(kb - G - g, nxt[g]);
#pragma unroll
            for (int g = 0; g < G; g++) {
                const int64_t k = kb - g;
                if (k >= k0) {
                    sv.seek(k);
                    step_out(cur[g], k);
                }
            }
#pragma unroll
            for (int g = 0; g < G; g++) cur[g] = nxt[g];
        }
    } else {
        for (int64_t k = k1 - 1; k >= k0; k--) {
            if constexpr (reload_constants<D>()) PSSGP_RELOAD_CONSTANTS();
            sv.seek(k);
            SAgg<D, T> e;
            if constexpr (ELEMS) {
                sagg_load_nt<D, T>(p.elem + elem_index<D>(slot, p.chunk, (int)(k - k0), lane), e, PSSGP_WAVE);
            } else {
                cdouble *c = cst;
                if constexpr (reload_constants<D>()) PSSGP_LAUNDER(c);
                smoother_element<LY, T, SV>(mdl, c, sv, p.t, p.m + k, p.P + k, (size_t)p.n, k, e, bad);
            }
            step_out(e, k);
        }
    }
    __syncthreads();
    for (int i = lane; i < tile_len; i += PSSGP_WAVE) {
        const int64_t k = tile_start + i;
        if (k < tr.k_end) {
            p.f_mean[k] = s_out[i];
            p.f_var[k] = s_out[tile_len + i];
        }
    }
    if (bad) status_or(&p.ctl->status, bad);
}

// Smoother pass of a fused call with an element per lane: one tile. Up to the lane's last step it is
// the RTS smoother (the smoothed moments there come from the carry and the
// lane's exclusive suffix); inside the lane the same recursion runs in the
// form of Bryson and Frazier, on the pair (lambda, Lambda) with
//   m^s = m + P lambda,   P^s = P - P Lambda P
// for the filter moments (m, P) of the step, in FP64:
//   lambda = P^-1 (m^s - m), Lambda = P^-1 (P - P^s) P^-1   at the lane's end,
//   step k, from the filtered to the predicted moments, with the predicted
//   P h, S = h P h^T + R, K = P h / S:
//     Lambda <- (I - K h)^T Lambda (I - K h) + h^T h / S
//     lambda <- (I - K h)^T lambda + h^T v / S
//   and over the transition before it, Lambda <- F^T Lambda F, lambda <- F^T lambda.
// f needs only P h and h m of the step, so that the filter hands over D + 3
// values per step (HandLayout) instead of the D^2 + D + D (D + 1) / 2 of a smoother element
// and forms no element per step. With r = R / S (1 at a missing step) the
// filtered P h is r times the predicted one, f_var = r h P h^T - r^2 (P h)^T
// Lambda (P h) and f_mean = h m + h P h^T v / S + r (P h)^T lambda.
// f_var is a difference, and Lambda is rounded relative to its largest entry:
// FP64 carries that for the results of an FP32 scan (gaps of 1e-3 to 100
// length-scales, noise variances of 1e-2 to 1e-14, d = 4, 6 and 8: no further
// from extended precision than an element per step in FP32), and for no other
// (lane_handover).
// Handover and elements together: filter finish + smoother of 2^22 steps at
// d = 6 (FP32, chunk 64) 453 + 169 us with an element per step (63 values; a
// Cholesky factor, two solves and a composition), 288 + 164 us in this form,
// which is bound by its instructions (930 per step).
template <class LY, typename T, class SV>
__device__ __forceinline__ void smoother_tile_fused(const SmoothParams<T> &p, const DevModel &mdl, cdouble *cst,
                                                    SV &sv, const STileRange &tr, int tile, T *s_out)
{
    constexpr int D = LY::D;
    constexpr int AGG = SAggLayout<D>::SIZE;
    constexpr int INCL = SAggLayout<D>::INCL;
    constexpr int B = smoother_shear_col<LY>();
    using SP = Sparsity<LY>;
    using HL = HandLayout<D>;
    const int lane = lane_id();
    const int slot = tr.slot_base + tile;
    const int64_t chunk_id = (int64_t)slot * PSSGP_WAVE + lane;
    const int64_t k0 = tr.k_begin + ((int64_t)tile * PSSGP_WAVE + lane) * p.chunk;
    const int64_t k1 = (k0 + p.chunk < tr.k_end) ? k0 + p.chunk : tr.k_end;
    const int64_t tile_start = tr.k_begin + (int64_t)tile * PSSGP_WAVE * p.chunk;
    const int tile_len = PSSGP_WAVE * p.chunk;
    // a lane's outputs in LDS are chunk + 1 apart: with chunk, a multiple of
    // 4 as a rule, a write of the wave would go to a few banks only
    const int row = p.chunk + 1, half = PSSGP_WAVE * row;
    T *so = s_out + lane * row;
    if (k0 < k1) {
            const bool end = k1 >= tr.k_end;
        const int64_t kl = end ? k1 - 1 : k1;  // last step of the lane's run
        // inputs of that step, requested first
        constexpr size_t ST = (size_t)HL::STEP * PSSGP_WAVE;
        const double *hq = p.hand + HL::step(slot, p.chunk, (int)(kl - k0), lane);
        double ph[D], in[3];  // P h; h m, innovation, length and mask of the step
        auto load = [&](const double *q, double (&x)[D], double (&z)[3]) {
#pragma unroll
            for (int i = 0; i < D; i++) x[i] = __builtin_nontemporal_load(q + i * PSSGP_WAVE);
#pragma unroll
            for (int i = 0; i < 3; i++) z[i] = __builtin_nontemporal_load(q + (D + i) * PSSGP_WAVE);
        };
        load(hq, ph, in);
        double lam[D], Lam[D][D];
        {
            T msT[D], PsT[D][D];
            gl_load<D, T>(p.inclp + (size_t)slot * INCL, msT, PsT);
            if (lane < PSSGP_WAVE - 1) {
                SAgg<D, T> excl;
                sagg_load<D, T>(lane_rec(p.lanep, slot, AGG, lane + 1), excl, PSSGP_WAVE);
                sagg_apply<D, T>(excl, msT, PsT, msT, PsT);
            }
            double ms[D], Ps[D][D];
#pragma unroll
            for (int i = 0; i < D; i++) {
                ms[i] = (double)msT[i];
#pragma unroll
                for (int j = 0; j < D; j++) Ps[i][j] = (double)PsT[i][j];
            }
            const double *bp = p.bound + HL::lane(slot, lane);
            double C[D][D], rd[D];
#pragma unroll
            for (int i = 0; i < D; i++) {
                ms[i] -= bp[i * PSSGP_WAVE];
#pragma unroll
                for (int j = 0; j < i; j++) C[i][j] = bp[(D + sidx<D>(j, i)) * PSSGP_WAVE];
                rd[i] = bp[(D + sidx<D>(i, i)) * PSSGP_WAVE];
            }
            // X = C^-1 P^s, then N = I - C^-1 X^T = C^-1 (P - P^s) C^-T
            auto forward = [&](double (&x)[D]) {
#pragma unroll
                for (int i = 0; i < D; i++) {
#pragma unroll
                    for (int q = 0; q < i; q++) x[i] = fma(-C[i][q], x[q], x[i]);
                    x[i] *= rd[i];
                }
            };
            auto backward = [&](double (&x)[D]) {
#pragma unroll
                for (int i = D - 1; i >= 0; i--) {
#pragma unroll
                    for (int q = i + 1; q < D; q++) x[i] = fma(-C[q][i], x[q], x[i]);
                    x[i] *= rd[i];
                }
            };
            // rows of Ps (symmetric) solved as right-hand sides: Lam[j][.] = C^-1 Ps[.][j]
#pragma unroll
            for (int j = 0; j < D; j++) {
#pragma unroll
                for (int i = 0; i < D; i++) Lam[j][i] = Ps[i][j];
                forward(Lam[j]);
            }
#pragma unroll
            for (int j = 0; j < D; j++) {
                double x[D];
#pragma unroll
                for (int i = 0; i < D; i++) x[i] = Lam[i][j];
                forward(x);
#pragma unroll
                for (int i = 0; i < D; i++) Ps[i][j] = (i == j ? 1.0 : 0.0) - x[i];
            }
#pragma unroll
            for (int j = 0; j < D; j++) {
#pragma unroll
                for (int i = 0; i < D; i++) Lam[j][i] = i <= j ? Ps[i][j] : Ps[j][i];
                backward(Lam[j]);
            }
#pragma unroll
            for (int j = 0; j < D; j++) {
                double x[D];
#pragma unroll
                for (int i = 0; i < D; i++) x[i] = Lam[i][j];
                backward(x);
#pragma unroll
                for (int i = 0; i < D; i++) Ps[i][j] = x[i];
            }
            forward(ms);
            backward(ms);
#pragma unroll
            for (int i = 0; i < D; i++) {
                lam[i] = end ? 0.0 : ms[i];
#pragma unroll
                for (int j = i; j < D; j++) {
                    Lam[i][j] = end ? 0.0 : Ps[i][j];
                    Lam[j][i] = Lam[i][j];
                }
            }
        }
        for (int64_t k = kl;; k--) {
            // the next step's inputs, one iteration ahead
            double nph[D], nin[3];
            hq = k > k0 ? hq - ST : hq;
            load(hq, nph, nin);
            PSSGP_RELOAD_CONSTANTS();
            const double R = (double)T(sv.R), hm = in[0], v = in[1], dt = __builtin_fabs(in[2]);
            const bool oc = !__builtin_signbit(in[2]);
            // here lambda and Lambda are in the coordinates z' = S z (identity
            // for one component), where the observation row is the first unit
            // vector: P h is summed into its first entry
            if constexpr (B > 0) ph[0] += ph[B];
            const double hph = ph[0];
            const double S = R + hph;
            const double w = oc ? rcp64(S) : 0.0;
            const double r = oc ? R * w : 1.0;
            // q = Lambda P h and s = Lambda (I - K h) e_0, whose first factor
            // 1 - K_0 is r: formed as a difference it would lose log10(S / R)
            // digits
            double su[D], phl = 0.0, phq = 0.0, ul = 0.0;
#pragma unroll
            for (int i = 0; i < D; i++) {
                double acc = 0.0;
#pragma unroll
                for (int j = 1; j < D; j++) acc = fma(Lam[i][j], ph[j], acc);
                su[i] = fma(-w, acc, r * Lam[i][0]);
                phq = fma(fma(Lam[i][0], hph, acc), ph[i], phq);
                if (i > 0) ul = fma(lam[i], ph[i], ul);
            }
            phl = fma(lam[0], hph, ul);
            // f outputs staged in LDS for coalesced stores (those of a step
            // past the lane go to the row's spare entry)
            so[k - k0] = T(fma(r, phl, fma(hph * w, v, hm)));
            so[half + (k - k0)] = T(r * fma(-r, phq, hph));
            if (k == k0) break;
            {
                double us = 0.0;
#pragma unroll
                for (int i = 1; i < D; i++) {
                    us = fma(ph[i], su[i], us);
                    Lam[0][i] = su[i];
                    Lam[i][0] = su[i];
                }
                Lam[0][0] = fma(-w, us, fma(r, su[0], w));
                lam[0] = fma(w, v - ul, r * lam[0]);
            }
            // in the filter's coordinates, S^T Lambda' S and S^T lambda', over the
            // transition, whose blocks they keep apart
            if constexpr (B > 0) {
                lam[B] += lam[0];
#pragma unroll
                for (int j = 0; j < D; j++) Lam[B][j] += Lam[0][j];
#pragma unroll
                for (int j = 0; j < D; j++) Lam[j][B] = (j == B) ? Lam[B][B] + Lam[B][0] : Lam[B][j];
            }
            // over the transition into step k (past the lane's first step, so
            // never the series' first)
            cdouble *cc = cst;
            PSSGP_LAUNDER(cc);
            double F[D][D];
            transition_plain<LY>(mdl, cc, sv.sc, dt, false, F);
            double X[D][D], nl[D];
#pragma unroll
            for (int i = 0; i < D; i++) {
                double acc = 0.0;
#pragma unroll
                for (int q3 = 0; q3 < D; q3++)
                    if (SP::dl(q3, i)) acc = fma(F[q3][i], lam[q3], acc);
                nl[i] = acc;
#pragma unroll
                for (int j = 0; j < D; j++) {
                    double x = 0.0;
#pragma unroll
                    for (int q3 = 0; q3 < D; q3++)
                        if (SP::dl(q3, j)) x = fma(Lam[i][q3], F[q3][j], x);
                    X[i][j] = x;
                }
            }
#pragma unroll
            for (int i = 0; i < D; i++) {
                lam[i] = nl[i];
#pragma unroll
                for (int j = i; j < D; j++) {
                    double x = 0.0;
#pragma unroll
                    for (int q3 = 0; q3 < D; q3++)
                        if (SP::dl(q3, i)) x = fma(F[q3][i], X[q3][j], x);
                    Lam[i][j] = x;
                    Lam[j][i] = x;
                }
            }
            // back: S^-T Lambda S^-1, S^-T lambda
            if constexpr (B > 0) {
                lam[B] -= lam[0];
#pragma unroll
                for (int j = 0; j < D; j++) Lam[B][j] -= Lam[0][j];
#pragma unroll
                for (int j = 0; j < D; j++) Lam[j][B] = (j == B) ? Lam[B][B] - Lam[B][0] : Lam[B][j];
            }
#pragma unroll
            for (int i = 0; i < D; i++) ph[i] = nph[i];
#pragma unroll
            for (int i = 0; i < 3; i++) in[i] = nin[i];
        }
    }
    __syncthreads();
    // step i of the tile is step j of lane l, i = l chunk + j
    const int dl = PSSGP_WAVE / p.chunk, dj = PSSGP_WAVE % p.chunk;
    int l = lane / p.chunk, j = lane % p.chunk;
    for (int i = lane; i < tile_len; i += PSSGP_WAVE) {
        const int64_t k = tile_start + i;
        if (k < tr.k_end) {
            p.f_mean[k] = s_out[l * row + j];
            p.f_var[k] = s_out[half + l * row + j];
        }
        l += dl;
        j += dj;
        if (j >= p.chunk) {
            j -= p.chunk;
            l++;
        }
    }
}

// ELEMS: the smoother elements come from the filter of the same call instead
// of being built from the filter moments.
template <class LY, typename T, bool ELEMS>
__global__ __launch_bounds__(PSSGP_WAVE, (smoother_waves<LY::D, T>())) void smoother_fold_kernel(SmoothParams<T> p,
                                                                                           DevModel mdl_arg)
{
    __shared__ DevModel mdl;
    model_to_lds(mdl_arg, mdl);
    OneSeries sv;
    sv.init(mdl, p.n);
    STileRange tr{0, p.n, p.ntiles, 0};
    smoother_tile_fold<LY, T, ELEMS, OneSeries>(p, mdl, (cdouble *)p.cst, sv, tr, (int)blockIdx.x);
}

// The last block of a fused call's smoother, one more than there are tiles,
// sums the filter's log-likelihood.
template <typename T>
__device__ __forceinline__ bool loglik_block(const SmoothParams<T> &p)
{
    if ((int)blockIdx.x != p.ntiles) return false;
    const double s = sum_over_tiles(p.partials, p.ntiles, 1);
    if (lane_id() == 0) *p.loglik = s;
    return true;
}

template <class LY, typename T, bool FULL, bool ELEMS>
__global__ __launch_bounds__(PSSGP_WAVE, (smoother_waves<LY::D, T>())) void smoother_finish_kernel(SmoothParams<T> p,
                                                                                             DevModel mdl_arg)
{
    if constexpr (ELEMS) {
        if (loglik_block(p)) return;
    }
    __shared__ DevModel mdl;
    model_to_lds(mdl_arg, mdl);
    OneSeries sv;
    sv.init(mdl, p.n);
    STileRange tr{0, p.n, p.ntiles, 0};
    extern __shared__ __align__(16) unsigned char pssgp_dyn_smem[];
    smoother_tile_finish<LY, T, FULL, ELEMS, OneSeries>(p, mdl, (cdouble *)p.cst, sv, tr, (int)blockIdx.x,
                                                 reinterpret_cast<T *>(pssgp_dyn_smem));
}

template <class LY, typename T>
__global__ __launch_bounds__(PSSGP_WAVE, (fused_waves<LY::D>())) void smoother_fused_kernel(SmoothParams<T> p,
                                                                                          DevModel mdl_arg)
{
    if (loglik_block(p)) return;
    __shared__ DevModel mdl;
    model_to_lds(mdl_arg, mdl);
    OneSeries sv;
    sv.init(mdl, p.n);
    STileRange tr{0, p.n, p.ntiles, 0};
    extern __shared__ __align__(16) unsigned char pssgp_dyn_smem[];
    smoother_tile_fused<LY, T, OneSeries>(p, mdl, (cdouble *)p.cst, sv, tr, (int)blockIdx.x,
                                          reinterpret_cast<T *>(pssgp_dyn_smem));
}

template <class LY, typename T>
int launch_smoother_t(const DevModel &mdl, const SmoothLaunch &a, hipStream_t s)
{
    SmoothParams<T> p;
    p.t = a.t;
    p.m = (const T *)a.m;
    p.P = (const T *)a.P;
    p.n = a.n;
    p.chunk = a.chunk;
    p.ntiles = a.ntiles;
    p.f_mean = (T *)a.f_mean;
    p.f_var = (T *)a.f_var;
    p.ms = (T *)a.ms;
    p.Ps = (T *)a.Ps;
    p.ctl = a.ws.ctl;
    p.inclp = (T *)a.ws.inclp;
    p.aggp = (T *)a.ws.aggp;
    p.lanep = (T *)a.ws.lanep;
    p.cst = a.ws.cst;
    p.partials = a.ws.partials;
    p.loglik = a.loglik;
    p.elem = (const T *)a.elem;
    p.hand = a.hand;
    p.bound = a.bound;
    const dim3 grid(a.ntiles), block(PSSGP_WAVE);
    pass_event(a.ev, 0, s);
    constexpr bool LANES = lane_handover(LY::D, sizeof(T) == 8);
    constexpr bool FOLDED = LANES || lane_aggregate_handover<LY::D>();
    if (a.fused && FOLDED) {
        // the filter's finish pass of the same call did this pass (lane
        // records at slane, tile aggregates at aggp)
        p.lanep = (T *)a.slane;
    } else {
        if (!a.fused) {
            launch_consts<LY, T>(mdl, a.ws.cst, s);
            hipLaunchKernelGGL((smoother_fold_kernel<LY, T, false>), grid, block, 0, s, p, mdl);
        } else if constexpr (!FOLDED) {
            hipLaunchKernelGGL((smoother_fold_kernel<LY, T, true>), grid, block, 0, s, p, mdl);
        }
        if constexpr (smoother_by_rows<LY::D, T>())
            hipLaunchKernelGGL((rows_lane_scan<LY::D, T>), grid, dim3(PSSGP_WAVE * LY::D), 0, s, p.lanep, p.aggp, 0);
    }
    int rc = (int)hipGetLastError();
    if (rc) return rc;
    pass_event(a.ev, 1, s);
    if constexpr (smoother_by_rows<LY::D, T>())
        rc = launch_smoother_rows_carry<LY::D, T>(a.ws.aggp, 0, a.ntiles, a.ws.inclp, a.ws.gagg, a.ws.gcarry, s);
    else
        rc = launch_tile_scan<SmootherScanOps<LY::D, T>>(a.ws.aggp, 0, a.ntiles, true, a.ws.inclp, a.ws.gagg,
                                                         a.ws.gcarry, s);
    if (rc) return rc;
    pass_event(a.ev, 2, s);
    const bool rows = a.fused && LANES;
    const size_t smem = (size_t)2 * PSSGP_WAVE * (rows ? a.chunk + 1 : a.chunk) * sizeof(T);
    const dim3 fgrid(a.ntiles + (a.fused ? 1 : 0));
    if (a.fused) {
        if constexpr (LANES)
            hipLaunchKernelGGL((smoother_fused_kernel<LY, T>), fgrid, block, smem, s, p, mdl);
        else
            hipLaunchKernelGGL((smoother_finish_kernel<LY, T, false, true>), fgrid, block, smem, s, p, mdl);
    } else if (a.ms && a.Ps)
        hipLaunchKernelGGL((smoother_finish_kernel<LY, T, true, false>), grid, block, smem, s, p, mdl);
    else
        hipLaunchKernelGGL((smoother_finish_kernel<LY, T, false, false>), grid, block, smem, s, p, mdl);
    rc = (int)hipGetLastError();
    pass_event(a.ev, 3, s);
    return rc;
}

template <int B0, int B1>
int launch_smoother_layout(const DevModel &mdl, bool f64, const SmoothLaunch &a, hipStream_t s)
{
    return f64 ? launch_smoother_t<Layout<B0, B1>, double>(mdl, a, s)
               : launch_smoother_t<Layout<B0, B1>, float>(mdl, a, s);
}
