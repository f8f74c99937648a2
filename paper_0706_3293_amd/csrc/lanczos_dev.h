// Scalars of a Lanczos run on the device, and the sums that a kernel of a step
// finishes for itself.
//
// A step is two kernels: the H x pass needs beta of the step before
// (sigma_k = 1 / beta_{k-1}), pass B needs alpha_k.  Both come from FP64
// partial sums, one per workgroup of the kernel before.  Summing them in a
// kernel of one workgroup costs a launch each (4.6 us back to back, more than
// the pass B of a million rows), so on grids of up to kFoldMax workgroups
// every workgroup sums them itself, in the same fixed order, while its first
// loads would be waiting anyway: at 2048 partials 8 loads per thread.  Larger
// grids keep the one-workgroup finishes, whose share is small there.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.h"

namespace hm {

// A run that has broken down has sigma_k = 0 from there on (sigma_0 = 0 for a
// zero start vector): a kernel of step k does nothing then, and the host takes
// the steps done from it.  No kernel reads a scalar that its own launch
// writes, so all of its workgroups decide alike.
struct LzDev {
    int stopped;     // one-workgroup run: steps done at a breakdown, 0 if none
    int bad_start;   // 1 if |v0| == 0
    double tol;
    double norm0;    // |v0|
    double psi_norm;
};

// Partials a kernel sums for itself (workgroups of the kernel before).
constexpr int kFoldMax = 2048;

// What the H x pass of step k takes from the run (sigma null: a plain product,
// sigma = 1 and no previous vector).
struct LzStep {
    const LzDev *lz = nullptr;
    const double *bpart = nullptr;   // |w|^2 partials of step k - 1 (null: finished already)
    int nb = 0, k = 0;
    const double *alpha = nullptr;
    double *beta = nullptr, *sigma = nullptr, *cprev = nullptr, *scale = nullptr;
};

// Sum of n partials in a fixed order, returned to every thread: thread t adds
// partials t, t + blockDim, ... (8 loads in flight), then the wave and
// workgroup sums.
__device__ __forceinline__ double fold_sum(const double *__restrict__ partial, int n,
                                           double *red /* >= 17 */) {
    constexpr int U = 8;
    const int stride = blockDim.x;
    double s = 0.0;
    int t = threadIdx.x;
    for (; t + (U - 1) * stride < n; t += U * stride) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = partial[t + u * stride];
#pragma unroll
        for (int u = 0; u < U; ++u) s += v[u];
    }
    for (; t < n; t += stride) s += partial[t];
    s = block_sum(s, red);
    if (threadIdx.x == 0) red[16] = s;
    __syncthreads();
    s = red[16];
    __syncthreads();
    return s;
}

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ double uniform(double v) {
    const uint64_t b = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// Scalars of step k: beta_{k-1} from |w|^2, the breakdown test (sigma = 0 if
// the run stops), sigma_k and cprev_k.
struct LzScalars {
    double sigma = 1.0, cprev = 0.0, beta = 0.0, scale = 0.0;
};

__device__ __forceinline__ LzScalars lz_advance(const LzDev *lz, int k, double w2,
                                                const double *alpha, const double *sigma,
                                                const double *scale) {
    LzScalars c;
    c.beta = sqrt(w2);
    c.scale = fmax(scale[k - 1], fmax(fabs(alpha[k - 1]), c.beta));
    const bool go = c.beta > lz->tol * c.scale;
    c.sigma = go ? 1.0 / c.beta : 0.0;
    c.cprev = go ? c.beta * sigma[k - 1] : 0.0;
    return c;
}

// LDS an H x pass needs for its scalars: fold_sum's, then beta and scale, kept
// there for its end (registers are what limits the waves of the gather loops).
constexpr int kLzLds = 19;

// Start of an H x pass: its scalars, false if the run has stopped.
__device__ __forceinline__ bool lz_begin(const LzStep &s, double *red /* >= kLzLds */,
                                         double &sigma, double &cprev) {
    sigma = 1.0;
    cprev = 0.0;
    if (!s.sigma) return true;
    if (!s.bpart) {
        sigma = s.sigma[s.k];
        cprev = s.cprev[s.k];
    } else {
        const bool first = blockIdx.x == 0 && threadIdx.x == 0;
        if (s.sigma[s.k - 1] == 0.0) {
            if (first) s.sigma[s.k] = 0.0;
            return false;
        }
        const LzScalars c =
            lz_advance(s.lz, s.k, fold_sum(s.bpart, s.nb, red), s.alpha, s.sigma, s.scale);
        if (first) {
            red[17] = c.beta;
            red[18] = c.scale;
            if (c.sigma == 0.0) {
                s.sigma[s.k] = 0.0;
                s.beta[s.k - 1] = c.beta;
            }
        }
        sigma = c.sigma;
        cprev = c.cprev;
    }
    return sigma != 0.0;
}

// End of the pass: workgroup 0 stores the scalars for the kernels that follow
// (at its end, so that the store cannot alias what the pass reads).
__device__ __forceinline__ void lz_end(const LzStep &s, const double *red, double sigma,
                                       double cprev) {
    if (!s.sigma || !s.bpart || blockIdx.x != 0 || threadIdx.x != 0) return;
    s.beta[s.k - 1] = red[17];
    s.scale[s.k] = red[18];
    s.sigma[s.k] = sigma;
    s.cprev[s.k] = cprev;
}

}  // namespace hm
