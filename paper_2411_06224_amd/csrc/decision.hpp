// The convergence decision of a PCG iteration, taken by one workgroup.
#pragma once

#include "launch.hpp"

namespace maspcg {

constexpr int kFlagX0 = 1, kFlagMixed = 2, kFlagRrTrue = 4;

// Sums the n_rr partials of ||r_k||^2 (init: and those of ||b||^2) and records rr,
// the iteration count and, when ||r|| <= tol ||b||, the stop for the host
// and every later kernel.  In mixed precision a stop on the recurrence is
// marked for confirmation on the FP64 residual.  mark: the non-zero value of
// the stop flag.  Needs blockDim.x >= 256 and
// buf[256] doubles of shared memory.
__device__ inline void convergence_decision(const SolverView& v, bool init, int k, double tol, int flags,
                                            int n_rr, int mark, double* buf) {
    DevState* st = v.st;
    if (st->done) return;
    const double rr = sum_partials(v.P_rr, n_rr, buf);
    if (init) {
        const double bb = sum_partials(v.P_bb, v.G, buf);
        const double tol2 = tol * tol * bb;
        const bool bad = !finite(bb) || !finite(rr);
        const bool stop = bad || bb == 0.0 || ((flags & kFlagX0) && rr <= tol2);
        if (threadIdx.x == 0) {
            st->bb = bb;
            st->tol2 = tol2;
            st->rr = rr;
            st->iter = 0;
            if (stop) {
                st->status = bad ? -6 : 0;
                st->done = mark;
            }
        }
    } else {
        const bool bad = !finite(rr);
        const bool conv = rr <= st->tol2;
        if (threadIdx.x == 0) {
            st->rr = rr;
            st->iter = k;
            if (bad || conv) {
                st->status = bad ? -6 : (((flags & kFlagMixed) && !(flags & kFlagRrTrue)) ? kStatusConvergedRecurrence : 0);
                st->done = mark;
            }
        }
    }
}

}  // namespace maspcg
