// Host interface of the large-state path (quasi-periodic models): model
// construction and the launch of the fused filter + smoother.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qp_team.h"

struct pssgp_model;

// What the filter of a fused call hands to its smoother: a smoother element per
// sub-chunk and two products per step (true), or an element per step. As with
// the one-lane scans (lane_handover) the first costs f_var digits that FP64 is
// chosen for: 10 states, gaps of 0.1, noise variance 1e-4, test points between
// the observations 7e-11 against 1e-13; noise 1e-12 and denser, wrong.
constexpr bool qp_sub_handover(bool f64) { return !f64; }

struct QPLaunch {
    void *const *ev;  // nullable: 8 events (filter fold, scan, finish, end; smoother fold, scan, finish, end)
    const double *t;
    const void *y;
    const uint8_t *mask;
    int64_t n;
    int chunk;
    int G;              // chunks of `chunk` steps
    void *fagg[2];      // G filter aggregates each (ping-pong)
    void *elem;         // smoother elements: n of the steps or, with hand, G nsub of the sub-chunks;
                        //   NULL: log-likelihood only
    int sub, nsub;      // hand: steps per sub-chunk of the smoother, sub-chunks per chunk
    void *sagg[2];      // G smoother elements each (ping-pong)
    double *hand;       // nullable (qp_sub_handover): (n + G) (d + 3) values handed to the smoother
    double *bound;      // hand: G nsub d (d + 2), end moments of the sub-chunks
    double *partials;   // G
    double *loglik;     // device double[1]
    void *f_mean;
    void *f_var;
    uint32_t *status;
};

// Whether a model is a quasi-periodic one (first component PSSGP_QUASIPERIODIC).
bool qp_is_model(const pssgp_model *spec);
// Host construction: 0 or a negative pssgp status code (message through
// pssgp_set_error). tdiag (nullable, d entries): x_canonical = diag(tdiag) z.
int qp_build(const pssgp_model *spec, QPDev *out, double *tdiag);
// Generator G (d*d) and observation row H in the library's coordinates.
void qp_matrices(const QPDev &m, double *G, double *Pinf, double *H);
// Launch (stream-ordered); -1: layout not compiled in, else a hipError_t.
int qp_launch(const QPDev &m, bool f64, const QPLaunch &q, hipStream_t s);
