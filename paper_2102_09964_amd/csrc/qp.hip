// Large-state path (quasi-periodic models, d = 10..18): filter and smoother
// scans with one 16-lane team per chunk of steps (qp_team.h, qp_ops.h).
//
// Passes of the fused call (pssgp_predict), one chunk of C steps per team,
// four teams per one-wave workgroup:
//   filter fold     each team folds its chunk into a filter aggregate
//                   (section 3, the raw element of every step applied with
//                   its rank-one information)
//   filter scan     inclusive prefix over the chunk aggregates by
//                   Hillis-Steele levels (ceil(log2 G) launches, the general
//                   operator in FP64); every prefix from the first step has
//                   A = 0, so the prefix of chunk g - 1 holds the filter
//                   moments entering chunk g
//   filter finish   each team re-runs its chunk from those moments as a
//                   Kalman filter in FP64 and sums the log-likelihood terms.
//                   FP64: it writes the smoother element of every step. FP32
//                   (qp_sub_handover): next to it runs the fixed-point smoother
//                   of the state that each sub-chunk of steps starts from,
//                   which gives one smoother element per sub-chunk
//                   (qp_sub_element), and P h, h m, the innovation and the
//                   length of every step go to the smoother, which reads no
//                   input. As the lanes of the one-lane scans, the chunks
//                   overlap by a step: a chunk's first sub-chunk starts from
//                   its first step and its last one ends with the next chunk's
//   loglik          one workgroup sums the per-chunk partials in chunk order
//   smoother fold   each team composes its chunk's elements right to left, or
//   smoother join   those of its chunk's sub-chunks
//   smoother scan   suffix scan of the chunks' elements (Hillis-Steele)
//   smoother finish FP64: each team applies the elements of its chunk backwards
//                   (RTS) and writes f_mean, f_var. FP32: each team runs the
//                   recursion of Bryson and Frazier backwards over a sub-chunk,
//                   as the one-lane scans do (smoother_tile_fused)
// What bounds these passes at the default chunk is the chain of steps of one
// team (256 steps at 2^18 are one wave on every fourth SIMD), so the smoother,
// which needs no further filter aggregate for it, works on sub-chunks.
// 262 107 steps at 16 states (FP32, chunk 256, sub-chunks of 64 steps):
// fold 774, ten filter levels of 64, finish 1619, join 19, ten smoother levels
// of 38, smoother finish 183 us, the call 3.63 ms; with a smoother element per
// step, folded and run again over the chunks, the call took 8.12 ms. FP64 with
// an element per step, chunk 128: fold 416, eleven levels of 129, finish 2085,
// smoother fold 773, eleven levels of 169, smoother finish 1025 us, 7.58 ms.
// Every team of a wave runs the same number of iterations (steps past a
// chunk's end are identity steps), so control flow is uniform.
#include <hip/hip_runtime.h>

#include "../../include/pssgp.h"
#include "qp_launch.h"
#include "qp_ops.h"

namespace {

constexpr int TEAMS = 4;  // teams per one-wave workgroup

__device__ __forceinline__ int team_id() { return (int)(blockIdx.x * TEAMS + (threadIdx.x >> 4)); }

__device__ __forceinline__ void qp_status_or(uint32_t *p, uint32_t bits)
{
    if (bits) __hip_atomic_fetch_or(p, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
struct QPArgs {
    const double *t;
    const T *y;
    const uint8_t *mask;
    int64_t n;
    int chunk;
    int G;          // chunks
    T *fagg[2];     // filter chunk aggregates / prefixes (ping-pong)
    T *elem;        // smoother elements of the steps or of the sub-chunks
    T *sagg[2];     // smoother elements of the chunks / suffixes (ping-pong)
    int sub;        // sub-chunks: steps per sub-chunk of the smoother
    int nsub;       // sub-chunks per chunk
    double *hand;   // per step, then per chunk for the step that it shares with the next: P h (D values),
                    //   h m, innovation (0 at a missing step), length (sign bit set at a missing step)
    double *bound;  // per sub-chunk, by rows, in the smoother's coordinates: Cholesky factor of its end
                    //   covariance, its diagonal's reciprocal, end mean
    double *partials;
    double *loglik;
    T *f_mean;
    T *f_var;
    uint32_t *status;
};

// Inputs of consecutive steps of a team's chunk (every lane reading the
// same), the next step's loaded one step ahead so that they are in flight
// while the current step is computed. Reads are clamped into the series and
// never branch on the optional mask (a missing mask reads the times, whose
// bytes are then ignored): a load inside a branch made the compiler wait
// for every outstanding memory operation right after it.
template <typename T>
struct QPInputs {
    const double *t;
    const T *y;
    const uint8_t *mk;
    bool has_mask;
    int64_t n;
    double tp, tc;  // times of steps k - 1 and k
    T yc;
    uint8_t mc;
    __device__ __forceinline__ void start(const QPArgs<T> &a, int64_t k)
    {
        t = a.t;
        y = a.y;
        mk = a.mask ? a.mask : (const uint8_t *)a.t;
        has_mask = a.mask != nullptr;
        n = a.n;
        const int64_t kc = k < n ? k : n - 1;
        tc = t[kc];
        tp = kc > 0 ? t[kc - 1] : tc;
        yc = y[kc];
        mc = mk[kc];
    }
    // loads of step k + 1 (clamped), issued now
    __device__ __forceinline__ void fetch(int64_t k, double &tn, T &yn, uint8_t &mn) const
    {
        const int64_t kn = k + 1 < n ? k + 1 : n - 1;
        tn = t[kn];
        yn = y[kn];
        mn = mk[kn];
    }
    __device__ __forceinline__ void advance(double tn, T yn, uint8_t mn)
    {
        tp = tc;
        tc = tn;
        yc = yn;
        mc = mn;
    }
    // dt of step k (0 at the series start) and whether it is observed
    __device__ __forceinline__ double dt(int64_t k) const { return k > 0 ? tc - tp : 0.0; }
    __device__ __forceinline__ bool observed() const { return !has_mask || mc != 0; }
};

template <class L, typename T>
__global__ __launch_bounds__(64) void qp_filter_fold(QPArgs<T> a, QPDev m)
{
    const int g = team_id();
    const int64_t k0 = (int64_t)g * a.chunk;
    const int64_t k1 = min(k0 + (int64_t)a.chunk, a.n);
    QAgg<L, T> agg;
    qagg_identity<L, T>(agg);
    uint32_t bad = 0;
    QPInputs<T> in;
    in.start(a, k0);
    for (int it = 0; it < a.chunk; it++) {
        const int64_t k = k0 + it;
        const bool real = k < k1;
        double tn;
        T yn;
        uint8_t mn;
        in.fetch(k, tn, yn, mn);
        const double dt = real ? in.dt(k) : 0.0;
        if (real && !(dt >= 0.0)) bad |= (dt < 0.0) ? PSSGP_STATUS_UNSORTED : PSSGP_STATUS_NONFINITE;
        QPStep<L::J> st;
        qp_step<L::J>(m, dt, real && k == 0, !real, st);
        const bool obs = real && in.observed();
        const T y = obs ? in.yc : T(0);
        in.advance(tn, yn, mn);
        qp_fold<L, T>(agg, m, st, y, obs);
    }
    qagg_store<L, T, T>(a.fagg[0] + (size_t)g * L::D * qagg_fields<L>(), agg, g < a.G);
    qp_status_or(a.status, bad);
}

// one Hillis-Steele level of the filter prefix: out[g] = in[g - o] (x) in[g]
template <class L, typename T>
__global__ __launch_bounds__(64) void qp_filter_level(const T *in, T *out, int G, int o, uint32_t *status)
{
    extern __shared__ __align__(16) double qp_lds[];
    constexpr int PER = L::D * L::D + (L::D + 2 * L::D + 1) + L::D * (2 * L::D + 1);
    double *lds = qp_lds + (threadIdx.x >> 4) * PER;
    const int g = team_id();
    constexpr int NF = L::D * qagg_fields<L>();
    QAgg<L, T> x, y, r;
    const bool has_x = g >= o && g < G;
    qagg_load<L, T, T>(in + (size_t)(has_x ? g - o : 0) * NF, x, has_x);
    if (!has_x) qagg_identity<L, T>(x);
    qagg_load<L, T, T>(in + (size_t)(g < G ? g : 0) * NF, y, g < G);
    uint32_t bad = 0;
    qp_combine<L, T>(x, y, r, lds, bad);
    qagg_store<L, T, T>(out + (size_t)g * NF, r, g < G);
    qp_status_or(status, bad & 16u ? PSSGP_STATUS_BAD_S : 0u);
}

// Filter finish: moments entering the chunk from the prefix of chunk g - 1,
// then a Kalman filter in FP64 over the chunk. QP_ELEMS: the smoother element of
// every step (iteration it builds the element of step k - 1 from the prediction
// of step k; one extra iteration predicts past the chunk for the element of its
// last step). QP_SUBS: the fixed-point smoother of the state that every sub-chunk
// starts from (G, m0, P0 as in lane_smoother_element), which is the last step of
// the sub-chunk before it or the chunk's first step, and the handover; one extra
// iteration is the first step of the next chunk.
enum : int { QP_ELEMS = 1, QP_SUBS = 2 };
template <class L, typename T, int MODE>
__global__ __launch_bounds__(64) void qp_filter_finish(QPArgs<T> a, QPDev m, const T *prefix)
{
    extern __shared__ __align__(16) double qp_lds[];
    constexpr int D = L::D, R = L::RPL;
    double *tbuf = qp_lds + (threadIdx.x >> 4) * (D * D);
    const int g = team_id();
    const int64_t k0 = (int64_t)g * a.chunk;
    const int64_t k1 = min(k0 + (int64_t)a.chunk, a.n);
    double mf[R], P[R][D];
    {
        QAgg<L, T> pre;
        const bool has = g > 0 && g < a.G;
        qagg_load<L, T, T>(prefix + (size_t)(has ? g - 1 : 0) * D * qagg_fields<L>(), pre, has);
#pragma unroll
        for (int s = 0; s < R; s++) {
            mf[s] = (double)pre.b[s];
#pragma unroll
            for (int j = 0; j < D; j++) P[s][j] = (double)pre.C[s][j];
        }
    }
    uint32_t bad = 0;
    double ll = 0.0;
    constexpr int NFS = D * qsagg_fields<L>();
    double m0[R], P0[R][D], G[R][D];
    auto restart = [&]() {
#pragma unroll
        for (int s = 0; s < R; s++) {
            m0[s] = mf[s];
#pragma unroll
            for (int j = 0; j < D; j++) P0[s][j] = G[s][j] = P[s][j];
        }
    };
    const double h0 = m.h[0];
    constexpr bool ELEMS = (MODE & QP_ELEMS) != 0, SUBS = (MODE & QP_SUBS) != 0;
    QPInputs<T> in;
    in.start(a, k0);
    if constexpr (SUBS) restart();
    for (int it = 0; it < a.chunk + (MODE != 0 ? 1 : 0); it++) {
        const int64_t k = k0 + it;
        const bool real = k < k1;
        double tn;
        T yn;
        uint8_t mn;
        in.fetch(k, tn, yn, mn);
        const bool next = ELEMS && k == k1 && k1 > k0;  // element of the chunk's last step
        const bool end = next && k1 >= a.n;             // past the series end: prior transition
        const bool over = SUBS && it == a.chunk && g < a.G && k < a.n;  // the step shared with the next chunk
        const bool live = real || over;
        const double dt = (live || (next && !end)) ? in.dt(k) : 0.0;
        if (real && !(dt >= 0.0)) bad |= (dt < 0.0) ? PSSGP_STATUS_UNSORTED : PSSGP_STATUS_NONFINITE;
        const bool obs = live && in.observed();
        const double yk = obs ? (double)in.yc : 0.0;
        in.advance(tn, yn, mn);
        QPStep<L::J> st;
        qp_step<L::J>(m, dt, (real && k == 0) || end, !(live || next), st);
        // prediction in FP64: Y = F P, mp = F m, Pp = F P F^T + Q
        double Y[R][D], mp[R], Pp[R][D];
        qp_left_F<L, double, double>(st, P, Y, true);
        qp_left_F_vec<L, double, double>(st, mf, mp);
        qp_right_Ft_plus_Q<L, double>(st, Y, Pp);
        if constexpr (SUBS) qp_left_F<L, double, double>(st, G, G, true);
        if constexpr (ELEMS) {
            // every team of the wave builds an element (the LDS transposes
            // need uniform control flow); only those of steps k0..k1-1 are
            // kept
            const bool keep = k > k0 && (real || next);
            QSAgg<L, T> e;
            double Cl[R][D], rd[D];
            uint32_t ebad = 0;
            qp_element<L, T>(m, mf, P, Y, mp, Pp, Cl, rd, e, tbuf, ebad);
            // the next step's loads are waited for before the element stores
            // (the wait counter is in order)
            asm volatile("" ::"v"(tn), "v"(yn), "v"((int)mn));
            qsagg_store<L, T, T>(a.elem + (size_t)(keep ? k - 1 : 0) * NFS, e, keep);
            bad |= keep ? ebad : 0u;
        }
        // conditioning on y_k in FP64
        double c[D];
        qp_obs_combo<L, double>(m, Pp, c);
        const double hm = qp_obs_dot<L, double>(m, mp);
        double S = m.R;
        sfor<0, L::NO>([&](auto qc) {
            constexpr int r = L::obs_row(decltype(qc)::value);
            S = fma(m.h[r], c[r], S);
        });
        if (obs && (!(S > 0.0) || !isfinite(S))) bad |= PSSGP_STATUS_BAD_S;
        if (obs && !isfinite(yk)) bad |= PSSGP_STATUS_NONFINITE;
        const double w = obs ? 1.0 / S : 0.0;
        const double v = obs ? yk - hm : 0.0;
        ll += (obs && real) ? -0.5 * (log(6.283185307179586 * S) + v * v * w) : 0.0;
        double K[D];
#pragma unroll
        for (int j = 0; j < D; j++) K[j] = c[j] * w;
        double gh[D];  // row 0 of S G after the conditioning: h G / h_0 = r G^T h / h_0
        if constexpr (SUBS) {
            // the next step's loads are waited for before the stores (the wait
            // counter is in order)
            asm volatile("" ::"v"(tn), "v"(yn), "v"((int)mn));
            double wh[D];
            qp_obs_combo<L, double>(m, G, wh);  // G^T h
            double *hp = a.hand + (size_t)(real ? k : (over ? a.n + g : 0)) * (D + 3);
#pragma unroll
            for (int s = 0; s < R; s++) {
                const int row = team_lane() + QP_TEAM * s;
                const double cr = qp_pick<D>(c, row), Kr = cr * w, whr = qp_pick<D>(wh, row);
                if (live && row < D) hp[row] = cr;
                m0[s] = fma(whr * w, v, m0[s]);
#pragma unroll
                for (int j = 0; j < D; j++) {
                    P0[s][j] = fma(-(whr * w), wh[j], P0[s][j]);
                    G[s][j] = fma(-Kr, wh[j], G[s][j]);
                }
            }
            if (live && team_lane() == 0) {
                hp[D] = hm;
                hp[D + 1] = v;
                hp[D + 2] = __builtin_copysign(dt, obs ? 1.0 : -1.0);
            }
            // row 0 of G from h G = r G^T h, r = R / S: as a difference it
            // would lose log10(S / R) digits
            const double rs = obs ? m.R * w : 1.0;
            double g0[D];
#pragma unroll
            for (int j = 0; j < D; j++) {
                g0[j] = rs * wh[j];
                gh[j] = g0[j] / h0;
            }
            sfor<1, L::NO>([&](auto qc) {
                constexpr int r = L::obs_row(decltype(qc)::value);
                const double hr = m.h[r];
#pragma unroll
                for (int j = 0; j < D; j++) g0[j] = fma(-hr, team_get<r % QP_TEAM>(G[r / QP_TEAM][j]), g0[j]);
            });
#pragma unroll
            for (int j = 0; j < D; j++) G[0][j] = (obs && team_lane() == 0) ? g0[j] / h0 : G[0][j];
        }
        if (live) {
#pragma unroll
            for (int s = 0; s < R; s++) {
                const int row = team_lane() + QP_TEAM * s;
                const double cr = qp_pick<D>(c, row), Kr = cr * w;
                mf[s] = fma(Kr, v, mp[s]);
#pragma unroll
                for (int j = 0; j < D; j++) P[s][j] = fma(S * Kr, K[j], fma(-cr, K[j], fma(-Kr, c[j], Pp[s][j])));
            }
        }
        if constexpr (SUBS) {
            if (it == 0) restart();
            if (it == a.chunk || ((it + 1) % a.sub == 0 && it + 1 < a.chunk)) {
                // the sub-chunk's element (every team of the wave builds one:
                // the LDS transposes need uniform control flow) and end moments
                const int q = it == a.chunk ? a.nsub - 1 : it / a.sub;
                const int64_t s0 = k0 + (int64_t)q * a.sub;
                const bool any = s0 < k1, end = it == a.chunk ? !over : k + 1 >= a.n;
                const size_t es = (size_t)g * a.nsub + q;
                // S P S^T, S m and the first row of S G from the conditioning:
                // r P h / h_0, f / h_0 and r h G / h_0, r = R / S (1 at a missing
                // step). At the chunk's first step G is the filtered P
                const int row = team_lane();
                const double r = obs ? m.R * w : 1.0, rh = r / h0;
                double hph = 0.0;
                sfor<0, L::NO>([&](auto qc) {
                    constexpr int o = L::obs_row(decltype(qc)::value);
                    hph = fma(m.h[o], c[o], hph);
                });
                double Cl[R][D], ms[R], Gs[R][D], rd[D];
#pragma unroll
                for (int j = 0; j < D; j++) {
                    Cl[0][j] = row == 0 ? rh * c[j] : P[0][j];
                    const double g0 = it == 0 ? rh * c[j] : gh[j];
                    Gs[0][j] = end ? 0.0 : (row == 0 ? g0 : G[0][j]);
                }
                Cl[0][0] = rh * (row == 0 ? hph / h0 : qp_pick<D>(c, row));
                if (end) {  // E = 0, and P need not have a factor
#pragma unroll
                    for (int j = 0; j < D; j++) Cl[0][j] = row == j ? 1.0 : 0.0;
                }
                ms[0] = row == 0 ? fma(hph * w, v, hm) / h0 : mf[0];
                QSAgg<L, T> e;
                uint32_t ebad = 0;
                qp_sub_element<L, T>(m, m0, P0, Gs, ms, Cl, rd, e, tbuf, ebad);
                bad |= any ? ebad : 0u;
                if (!any) qsagg_identity<L, T>(e);
                qsagg_store<L, T, T>(a.elem + es * NFS, e, g < a.G);
                double *bp = a.bound + es * (size_t)(D * (D + 2));
                if (any && row < D) {
#pragma unroll
                    for (int j = 0; j < D; j++) bp[row * (D + 2) + j] = Cl[0][j];
                    bp[row * (D + 2) + D] = qp_pick<D>(rd, row);
                    bp[row * (D + 2) + D + 1] = ms[0];
                }
                restart();
            }
        }
    }
    if (team_lane() == 0 && g < a.G) a.partials[g] = ll;
    qp_status_or(a.status, bad);
}

// log-likelihood: the chunk partials summed in chunk order (one workgroup)
__global__ __launch_bounds__(256) void qp_loglik_sum(const double *partials, int G, double *out)
{
    __shared__ double s_part[256];
    double acc = 0.0;
    for (int i = (int)threadIdx.x; i < G; i += 256) acc += partials[i];
    s_part[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int i = 0; i < 256; i++) tot += s_part[i];
        *out = tot;
    }
}

// The smoother element of each chunk from its steps'
template <class L, typename T>
__global__ __launch_bounds__(64) void qp_smoother_fold(QPArgs<T> a)
{
    const int g = team_id();
    const int64_t k0 = (int64_t)g * a.chunk;
    const int64_t k1 = min(k0 + (int64_t)a.chunk, a.n);
    constexpr int NFS = L::D * qsagg_fields<L>();
    QSAgg<L, T> acc;
    qsagg_identity<L, T>(acc);
    for (int it = 0; it < a.chunk; it++) {
        const int64_t k = k0 + a.chunk - 1 - it;
        const bool real = k < k1;
        QSAgg<L, T> e;
        qsagg_load<L, T, T>(a.elem + (size_t)(real ? k : 0) * NFS, e, real);
        qsagg_combine<L, T>(e, acc, acc);
    }
    qsagg_store<L, T, T>(a.sagg[0] + (size_t)g * NFS, acc, g < a.G);
}

// The smoother element of each chunk from its sub-chunks' (the scan's levels
// then run over the chunks: over the sub-chunks they took 100 instead of 41 us
// each at 2^18 steps)
template <class L, typename T>
__global__ __launch_bounds__(64) void qp_smoother_join(QPArgs<T> a)
{
    const int g = team_id();
    constexpr int NFS = L::D * qsagg_fields<L>();
    const bool on = g < a.G;
    const T *base = a.elem + (size_t)(on ? g : 0) * a.nsub * NFS;
    QSAgg<L, T> acc;
    qsagg_load<L, T, T>(base + (size_t)(a.nsub - 1) * NFS, acc, on);
    for (int q = a.nsub - 2; q >= 0; q--) {
        QSAgg<L, T> e;
        qsagg_load<L, T, T>(base + (size_t)q * NFS, e, on);
        qsagg_combine<L, T>(e, acc, acc);
    }
    qsagg_store<L, T, T>(a.sagg[0] + (size_t)g * NFS, acc, on);
}

// one level of the smoother suffix: out[g] = in[g] (x) in[g + o]
template <class L, typename T>
__global__ __launch_bounds__(64) void qp_smoother_level(const T *in, T *out, int G, int o)
{
    const int g = team_id();
    constexpr int NFS = L::D * qsagg_fields<L>();
    QSAgg<L, T> x, y;
    qsagg_load<L, T, T>(in + (size_t)(g < G ? g : 0) * NFS, x, g < G);
    const bool has_y = g + o < G;
    qsagg_load<L, T, T>(in + (size_t)(has_y ? g + o : 0) * NFS, y, has_y);
    qsagg_combine<L, T>(x, y, x);
    qsagg_store<L, T, T>(out + (size_t)g * NFS, x, g < G);
}

// Smoother finish of one chunk from the elements of its steps: smoothed moments
// after the chunk from the suffix of chunk g + 1 (none after the last chunk: the
// last element has E = 0), then the RTS recursion backwards; f = h_0 z'_0 in the
// smoother's coordinates.
template <class L, typename T>
__global__ __launch_bounds__(64) void qp_smoother_steps(QPArgs<T> a, QPDev m, const T *suffix)
{
    constexpr int D = L::D, R = L::RPL;
    const int g = team_id();
    const int64_t k0 = (int64_t)g * a.chunk;
    const int64_t k1 = min(k0 + (int64_t)a.chunk, a.n);
    constexpr int NFS = D * qsagg_fields<L>();
    T ms[R], Ps[R][D];
    {
        QSAgg<L, T> suf;
        const bool has = g + 1 < a.G;
        qsagg_load<L, T, T>(suffix + (size_t)(has ? g + 1 : 0) * NFS, suf, has);
#pragma unroll
        for (int s = 0; s < R; s++) {
            ms[s] = has ? suf.g[s] : T(0);
#pragma unroll
            for (int j = 0; j < D; j++) Ps[s][j] = has ? suf.L_[s][j] : T(0);
        }
    }
    const double h0 = m.h[0];
    for (int it = 0; it < a.chunk; it++) {
        const int64_t k = k0 + a.chunk - 1 - it;
        const bool real = k < k1;
        QSAgg<L, T> e;
        qsagg_load<L, T, T>(a.elem + (size_t)(real ? k : 0) * NFS, e, real);
        qsagg_apply<L, T>(e, ms, Ps);
        if (real && team_lane() == 0) {
            a.f_mean[k] = T(h0 * (double)ms[0]);
            a.f_var[k] = T(h0 * h0 * (double)Ps[0][0]);
        }
    }
}

// Smoother finish of one sub-chunk: the smoothed moments of its last step (a
// chunk's last sub-chunk: of the next chunk's first) from the elements after it
// (none after the series' end), then the recursion of (lambda, Lambda) backwards
// (smoother_tile_fused has the formulas); row i of Lambda on team lane i, in
// FP64. In the coordinates z' = S z the observation row is h_0 times the first
// unit vector.
template <class L, typename T>
__global__ __launch_bounds__(64) void qp_smoother_finish(QPArgs<T> a, QPDev m, const T *suffix)
{
    extern __shared__ __align__(16) double qp_lds[];
    constexpr int D = L::D, R = L::RPL;
    static_assert(R == 1, "one row per lane");
    double *tbuf = qp_lds + (threadIdx.x >> 4) * (D * D);
    const int es = team_id(), ns = a.G * a.nsub;
    const int g = es / a.nsub, q = es - g * a.nsub;
    const int64_t kc = (int64_t)g * a.chunk;
    const int64_t k0 = kc + (int64_t)q * a.sub;
    const int64_t k1 = min(min(k0 + (int64_t)a.sub, kc + (int64_t)a.chunk), a.n);
    const bool any = es < ns && k0 < k1;
    const int row = team_lane();
    constexpr int NFS = D * qsagg_fields<L>();
    const double h0 = m.h[0];
    double u[D], ur = 0.0;  // shear S = I + e_0 u^T (u: observed rows other than 0)
#pragma unroll
    for (int j = 0; j < D; j++) u[j] = 0.0;
    sfor<1, L::NO>([&](auto qc) {
        constexpr int r = L::obs_row(decltype(qc)::value);
        u[r] = m.u[r];
    });
    ur = qp_pick<D>(u, row);
    double lam[R], Lam[R][D];
    {
        const bool has = any && k1 < a.n;
        double ms[R], Ps[R][D];
        {
            // the suffix after the chunk, then the chunk's later sub-chunks
            // (every team of the wave runs the same number of them)
            const bool nxt = any && g + 1 < a.G;
            QSAgg<L, T> suf;
            qsagg_load<L, T, T>(suffix + (size_t)(nxt ? g + 1 : 0) * NFS, suf, nxt);
            T gm[R], Lm[R][D];
            gm[0] = nxt ? suf.g[0] : T(0);
#pragma unroll
            for (int j = 0; j < D; j++) Lm[0][j] = nxt ? suf.L_[0][j] : T(0);
            for (int i = a.nsub - 1; i >= 1; i--) {
                const bool use = any && i > q;
                qsagg_load<L, T, T>(a.elem + (size_t)(use ? g * a.nsub + i : 0) * NFS, suf, use);
                T g2[R], L2[R][D];
                g2[0] = gm[0];
#pragma unroll
                for (int j = 0; j < D; j++) L2[0][j] = Lm[0][j];
                qsagg_apply<L, T>(suf, g2, L2);
                gm[0] = use ? g2[0] : gm[0];
#pragma unroll
                for (int j = 0; j < D; j++) Lm[0][j] = use ? L2[0][j] : Lm[0][j];
            }
            ms[0] = has ? (double)gm[0] : 0.0;
#pragma unroll
            for (int j = 0; j < D; j++) Ps[0][j] = has ? (double)Lm[0][j] : 0.0;
        }
        const double *bp = a.bound + (size_t)(any ? es : 0) * (D * (D + 2));
        double Cl[R][D], Ct[R][D], rdr[R], rd[D];
        const bool ok = any && row < D;
#pragma unroll
        for (int j = 0; j < D; j++) Cl[0][j] = ok ? bp[row * (D + 2) + j] : (row == j ? 1.0 : 0.0);
        rdr[0] = ok ? bp[row * (D + 2) + D] : 1.0;
        ms[0] -= ok ? bp[row * (D + 2) + D + 1] : 0.0;
        qp_gather<L, double, double>(rdr, rd);
        qp_transpose<L, double>(Cl, Ct, tbuf);
        // N = I - C^-1 P^s C^-T, Lambda = C^-T N C^-1, lambda = P^-1 (m^s - m)
        qp_forward<L>(Cl, rd, Ps);
        qp_transpose<L, double>(Ps, Ps, tbuf);
        qp_forward<L>(Cl, rd, Ps);
#pragma unroll
        for (int j = 0; j < D; j++) Ps[0][j] = (row == j ? 1.0 : 0.0) - Ps[0][j];
        qp_backward<L>(Ct, rd, Ps);
        qp_transpose<L, double>(Ps, Ps, tbuf);
        qp_backward<L>(Ct, rd, Ps);
        qp_symmetrize<L, double>(Ps, tbuf);
        sfor<0, D>([&](auto kk) {
            constexpr int k = decltype(kk)::value;
            ms[0] = row == k ? ms[0] * rd[k] : ms[0];
            const double x = team_get<k>(ms[0]);
            ms[0] = fma(-(row > k ? Cl[0][k] : 0.0), x, ms[0]);
        });
        sfor<0, D>([&](auto kk) {
            constexpr int k = D - 1 - decltype(kk)::value;
            ms[0] = row == k ? ms[0] * rd[k] : ms[0];
            const double x = team_get<k>(ms[0]);
            ms[0] = fma(-(row < k ? Ct[0][k] : 0.0), x, ms[0]);
        });
        lam[0] = has && row < D ? ms[0] : 0.0;
#pragma unroll
        for (int j = 0; j < D; j++) Lam[0][j] = has && row < D ? Ps[0][j] : 0.0;
    }
    // what the filter handed over of a step (clamped into the sub-chunk): P h;
    // h m, innovation, length and mask
    struct In {
        double ph[D], hm, v, dt;
    };
    const bool over = any && k1 == kc + a.chunk && k1 < a.n;
    const int64_t kl = over ? k1 : k1 - 1;  // last step of the run
    auto fetch = [&](int64_t k, In &x) {
        const int64_t c = !any ? 0 : (over && k == k1) ? a.n + g : (k > k0 ? k : k0);
        const double *hp = a.hand + (size_t)c * (D + 3);
#pragma unroll
        for (int j = 0; j < D; j++) x.ph[j] = hp[j];
        x.hm = hp[D];
        x.v = hp[D + 1];
        x.dt = hp[D + 2];
    };
    In x, nx;
    fetch(kl, x);
    for (int it = 0; it <= a.sub; it++) {
        const int64_t k = kl - it;
        const bool live = any && k >= k0;
        fetch(k - 1, nx);
        const bool obs = live && !__builtin_signbit(x.dt);
        sfor<1, L::NO>([&](auto qc) {  // P h in z'
            constexpr int r = L::obs_row(decltype(qc)::value);
            x.ph[0] = fma(u[r], x.ph[r], x.ph[0]);
        });
        const double hph = h0 * x.ph[0], S = m.R + hph;
        const double w = obs ? 1.0 / S : 0.0;
        const double v = obs ? x.v : 0.0;
        const double r = obs ? m.R * w : 1.0;
        const double hw = h0 * w;
        double tt = 0.0;
#pragma unroll
        for (int j = 1; j < D; j++) tt = fma(Lam[0][j], x.ph[j], tt);
        const double phr = qp_pick<D>(x.ph, row);  // 0 on the lanes past D
        const double sr = fma(-hw, tt, r * Lam[0][0]);
        const double phq = team_sum(fma(Lam[0][0], x.ph[0], tt) * phr);
        const double rest = row == 0 ? 0.0 : phr;
        const double us = team_sum(rest * sr), ul = team_sum(rest * lam[0]);
        const double lam0 = team_get<0>(lam[0]), s0 = team_get<0>(sr);
        const double phl = fma(x.ph[0], lam0, ul);
        if (live && k < k1 && row == 0) {
            a.f_mean[k] = T(fma(r, phl, fma(hph * w, v, x.hm)));
            a.f_var[k] = T(r * fma(-r, phq, hph));
        }
        // the observation's update (the identity before the sub-chunk's first step)
        {
            const double l00 = fma(-hw, us, fma(r, s0, h0 * hw));
            double col[R], l0[D];
            col[0] = row == 0 ? l00 : sr;
            qp_gather<L, double, double>(col, l0);  // row 0 of Lambda'
#pragma unroll
            for (int j = 0; j < D; j++) Lam[0][j] = row == 0 ? l0[j] : Lam[0][j];
            Lam[0][0] = col[0];
            const double lm0 = fma(hw, v - ul, r * lam0);
            lam[0] = row == 0 ? lm0 : lam[0];
            // Lambda = S^T Lambda' S, lambda = S^T lambda'
            lam[0] = fma(ur, lm0, lam[0]);
#pragma unroll
            for (int j = 0; j < D; j++) Lam[0][j] = fma(ur, l0[j], Lam[0][j]);
            sfor<1, L::NO>([&](auto qc) {
                constexpr int rr = L::obs_row(decltype(qc)::value);
                Lam[0][rr] = fma(u[rr], Lam[0][0], Lam[0][rr]);
            });
        }
        // over the transition into the step
        if (it < a.sub) {
            QPStep<L::J> st;
            qp_step<L::J>(m, live ? __builtin_fabs(x.dt) : 0.0, false, !live, st);
            qp_right_F<L>(st, Lam, Lam);
            qp_left_Ft<L>(st, Lam, lam);
            // back: Lambda' = S^-T Lambda S^-1, lambda' = S^-T lambda
            double l0[D];
            qp_row<L, 0>(Lam, l0);
            const double lm0 = team_get<0>(lam[0]);
            lam[0] = fma(-ur, lm0, lam[0]);
#pragma unroll
            for (int j = 0; j < D; j++) Lam[0][j] = fma(-ur, l0[j], Lam[0][j]);
            sfor<1, L::NO>([&](auto qc) {
                constexpr int r = L::obs_row(decltype(qc)::value);
                Lam[0][r] = fma(-u[r], Lam[0][0], Lam[0][r]);
            });
        }
        x = nx;
    }
}

template <typename T>
QPArgs<T> qp_args(const QPLaunch &q)
{
    QPArgs<T> a;
    a.t = q.t;
    a.y = (const T *)q.y;
    a.mask = q.mask;
    a.n = q.n;
    a.chunk = q.chunk;
    a.G = q.G;
    a.fagg[0] = (T *)q.fagg[0];
    a.fagg[1] = (T *)q.fagg[1];
    a.sub = q.sub;
    a.nsub = q.nsub;
    a.elem = (T *)q.elem;
    a.sagg[0] = (T *)q.sagg[0];
    a.sagg[1] = (T *)q.sagg[1];
    a.hand = q.hand;
    a.bound = q.bound;
    a.partials = q.partials;
    a.loglik = q.loglik;
    a.f_mean = (T *)q.f_mean;
    a.f_var = (T *)q.f_var;
    a.status = q.status;
    return a;
}

template <class L, typename T>
int qp_launch_t(const QPDev &m, const QPLaunch &q, hipStream_t s)
{
    QPArgs<T> a = qp_args<T>(q);
    const dim3 grid((unsigned)((q.G + TEAMS - 1) / TEAMS)), block(64);
    constexpr int D = L::D;
    const size_t lds_level = (size_t)TEAMS * (D * D + (D + 2 * D + 1) + D * (2 * D + 1)) * sizeof(double);
    const size_t lds_finish = (size_t)TEAMS * D * D * sizeof(double);
    if (q.ev && q.ev[0]) (void)hipEventRecord((hipEvent_t)q.ev[0], s);
    hipLaunchKernelGGL((qp_filter_fold<L, T>), grid, block, 0, s, a, m);
    if (q.ev && q.ev[1]) (void)hipEventRecord((hipEvent_t)q.ev[1], s);
    int src = 0;
    for (int o = 1; o < q.G; o <<= 1) {
        hipLaunchKernelGGL((qp_filter_level<L, T>), grid, block, lds_level, s, (const T *)a.fagg[src],
                           a.fagg[src ^ 1], q.G, o, q.status);
        src ^= 1;
    }
    if (q.ev && q.ev[2]) (void)hipEventRecord((hipEvent_t)q.ev[2], s);
    constexpr bool SUBS = qp_sub_handover(sizeof(T) == 8);
    if (q.elem)
        hipLaunchKernelGGL((qp_filter_finish<L, T, SUBS ? QP_SUBS : QP_ELEMS>), grid, block, lds_finish, s, a, m,
                           (const T *)a.fagg[src]);
    else
        hipLaunchKernelGGL((qp_filter_finish<L, T, 0>), grid, block, lds_finish, s, a, m, (const T *)a.fagg[src]);
    hipLaunchKernelGGL(qp_loglik_sum, dim3(1), dim3(256), 0, s, (const double *)a.partials, q.G, q.loglik);
    if (q.ev && q.ev[3]) (void)hipEventRecord((hipEvent_t)q.ev[3], s);
    int rc = (int)hipGetLastError();
    if (rc || !q.elem) return rc;
    if (q.ev && q.ev[4]) (void)hipEventRecord((hipEvent_t)q.ev[4], s);
    if constexpr (SUBS)
        hipLaunchKernelGGL((qp_smoother_join<L, T>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((qp_smoother_fold<L, T>), grid, block, 0, s, a);
    if (q.ev && q.ev[5]) (void)hipEventRecord((hipEvent_t)q.ev[5], s);
    src = 0;
    for (int o = 1; o < q.G; o <<= 1) {
        hipLaunchKernelGGL((qp_smoother_level<L, T>), grid, block, 0, s, (const T *)a.sagg[src], a.sagg[src ^ 1],
                           q.G, o);
        src ^= 1;
    }
    if (q.ev && q.ev[6]) (void)hipEventRecord((hipEvent_t)q.ev[6], s);
    if constexpr (SUBS) {
        const dim3 sgrid((unsigned)(((int64_t)q.G * q.nsub + TEAMS - 1) / TEAMS));
        hipLaunchKernelGGL((qp_smoother_finish<L, T>), sgrid, block, lds_finish, s, a, m, (const T *)a.sagg[src]);
    } else {
        hipLaunchKernelGGL((qp_smoother_steps<L, T>), grid, block, 0, s, a, m, (const T *)a.sagg[src]);
    }
    if (q.ev && q.ev[7]) (void)hipEventRecord((hipEvent_t)q.ev[7], s);
    return (int)hipGetLastError();
}

}  // namespace

int qp_launch(const QPDev &m, bool f64, const QPLaunch &q, hipStream_t s)
{
    switch (m.J) {
    case 1: return f64 ? qp_launch_t<QPL<1>, double>(m, q, s) : qp_launch_t<QPL<1>, float>(m, q, s);
    case 2: return f64 ? qp_launch_t<QPL<2>, double>(m, q, s) : qp_launch_t<QPL<2>, float>(m, q, s);
    case 3: return f64 ? qp_launch_t<QPL<3>, double>(m, q, s) : qp_launch_t<QPL<3>, float>(m, q, s);
    default: return -1;
    }
}
