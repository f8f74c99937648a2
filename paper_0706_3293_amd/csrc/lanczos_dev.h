// Scalars of a Lanczos run on the device, and the sums that a kernel of a step
// finishes for itself.
//
// A step is two kernels: the H x pass needs beta of the step before
// (sigma_k = 1 / beta_{k-1}), pass B needs alpha_k.  Both come from FP64
// partial sums, one per workgroup of the kernel before.  Summing them in a
// kernel of one workgroup costs a launch each (4.6 us back to back, more than
// the pass B of a million rows), so on grids of up to kFoldMax workgroups
// every workgroup sums them itself, in the same fixed order, while its first
// loads would be waiting anyway: 8 loads per thread.  Larger grids keep the
// one-workgroup finishes, whose share is small there.
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
    int nb = 0, k = 0;               // their number, 0: in groups (fold_groups)
    const double *alpha = nullptr;
    double *beta = nullptr, *sigma = nullptr, *cprev = nullptr, *scale = nullptr;
};

// Sum of n <= kFoldMax partials, returned to every thread, in the order of a
// workgroup of VT threads that adds partials t, t + VT, ... in thread t, then the
// lanes of every wave and the waves in turn: bit for bit the finish kernel of that
// size (fixed_sum in lanczos.hip), so a run's coefficients do not depend on whether
// its sums are folded.  (Runs past convergence amplify one rounding to 1e-8 of
// the ground state.)  The waves that a smaller workgroup does not have are taken
// by its own ones in turn; all 8 loads of a thread are in flight together.
template <int VT>
__device__ __forceinline__ double fold_sum(const double *__restrict__ partial, int n,
                                           double *red /* >= VT / 64 */) {
    constexpr int kWaves = VT / 64, U = kFoldMax / VT, Q = VT / 256;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    for (int w0 = wid; w0 < kWaves; w0 += Q * nw) {
        // loads without branches: one past the end reads partial 0 and adds 0
        double v[Q][U], s[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = (w0 + q * nw) * 64 + lane + u * VT;
                v[q][u] = partial[t < n ? t : 0];
            }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            s[q] = 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) s[q] += (w0 + q * nw) * 64 + lane + u * VT < n ? v[q][u] : 0.0;
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
            for (int q = 0; q < Q; ++q) s[q] += __shfl_xor(s[q], off, 64);
        if (lane == 0)
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (w0 + q * nw < kWaves) red[w0 + q * nw] = s[q];
    }
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) s += red[w];
    __syncthreads();
    return s;
}

// Pass B's sums come in groups already: partial 16 w + a of kGroups is the sum of
// the slices 64 w + a + 16 j + 1024 i (j < 4, i < 2) that fold_sum<1024> would add
// first, the two of a thread and then the lanes 32 and 16 apart.  What is left of
// that order is four exchanges and the waves in turn: one load per thread instead
// of eight (705,432 rows, FP32, H x with 2048 workgroups: 3 us less).
constexpr int kGroups = 256;

__device__ __forceinline__ double fold_groups(const double *__restrict__ partial,
                                              double *red /* >= 16 */) {
    for (int t = threadIdx.x; t < kGroups; t += blockDim.x) {
        double s = partial[t];
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
        if (t % 16 == 0) red[t / 16] = s;
    }
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kGroups / 16; ++w) s += red[w];
    __syncthreads();
    return s;
}

// Threads of the finishes of the steps' sums, and of the sums before and after
// the steps.
constexpr int kFinishBlock = 1024, kEndsBlock = 256;

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
        const double w2 =
            s.nb ? fold_sum<kFinishBlock>(s.bpart, s.nb, red) : fold_groups(s.bpart, red);
        const LzScalars c = lz_advance(s.lz, s.k, w2, s.alpha, s.sigma, s.scale);
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
