// The drift, and what a denoiser launch does with each epsilon it forms: store
// it, or take the sequential sampler's step with it at once (a launch and a pass
// over x and epsilon less per step).
#pragma once

#include "pd_internal.h"

namespace pd {

__device__ __forceinline__ float drift(float A, float x, float B, float e) {
    // y = A x + B eps, two products and one sum, each rounded (no contraction)
    return __fadd_rn(__fmul_rn(A, x), __fmul_rn(B, e));
}

// What becomes of epsilon of element i (row-major over the launch's rows).
__device__ __forceinline__ void eps_out(const EpsOut& o, int64_t i, float e) {
    switch (o.mode) {
        case EPS_STORE:
            o.y[i] = e;
            return;
        case EPS_STEP_HEUN:              // the mean of the two evaluations, then the step
            e = __fmul_rn(__fadd_rn(o.eps1[i], e), 0.5f);
            [[fallthrough]];
        case EPS_STEP: {                 // x <- x + ((A x + B eps) [+ z])
            const float x = o.x[i];
            float y = drift(o.A, x, o.B, e);
            if (o.z) y = __fadd_rn(y, o.z[i]);
            o.x[i] = __fadd_rn(x, y);
            return;
        }
        case EPS_PREDICT: {              // the Euler prediction of one step
            const float x = o.x[i];
            o.y[i] = e;
            o.xt[i] = __fadd_rn(x, drift(o.A, x, o.B, e));
            return;
        }
        case EPS_STEP_DPM: {             // x <- x + (((A x + B eps) + R xp) + S ep), (xp, ep) <- (x, eps)
            const float x = o.x[i];
            float y = drift(o.A, x, o.B, e);
            if (o.R != 0.f) y = __fadd_rn(__fadd_rn(y, __fmul_rn(o.R, o.xp[i])), __fmul_rn(o.S, o.ep[i]));
            o.x[i] = __fadd_rn(x, y);
            o.xp[i] = x;
            o.ep[i] = e;
            return;
        }
    }
}

}  // namespace pd
