// Dot products of many stored vectors with a few new ones: for ncol columns
// V (blocks of P interleaved columns, block j at V + j * dim * P) and the P
// columns of W, C[col][c] = sum_row V[row][col] W[row][c] in FP64, for the
// full reorthogonalization of the scalar (P = 1) and of the block recurrence.
//
// The contraction V^T W runs on the matrix cores (v_mfma_f64_16x16x4: 16
// columns of V, 4 rows, up to 16 columns of W), which also do the sum over
// the rows of a wave, so a thread holds a handful of accumulators and the
// cross-lane reduction that dominated a vector-ALU version (64 accumulators
// of 64 lanes per workgroup, for 2.8 rows per thread at 184,756 rows) is gone.
// What bounds it is reading V.  A wave takes 64 columns, so one load of W
// serves 64 columns, and every lane loads 16 bytes: two neighbouring columns
// of one row (P >= 2), which go to two accumulators, or two consecutive rows
// of one column (P = 1), which go to two products.  Measured on 184,756 rows
// and blocks of 4 (1 to 40 blocks, and W^T W; 640 launches): 40 -> 20 us on
// average, and the sums of the partials 61 -> 4.9 us (they were one serial
// loop per result); a 40-step run 29.7 -> 8.3 ms.
#pragma once

#include "device_common.h"
#include "lanczos_dev.h"

namespace hm {

constexpr int kTallBlock = 256;      // threads per workgroup (4 waves)
constexpr int kTallSplits = 256;     // most row ranges (partials per result)

typedef double v4d __attribute__((ext_vector_type(4)));

// Two consecutive elements at any element-aligned address.
template <typename T>
using Two = T __attribute__((ext_vector_type(2), aligned(sizeof(T))));
template <typename T>
__device__ __forceinline__ Two<T> load2(const T *__restrict__ p) {
    return *reinterpret_cast<const Two<T> *>(p);
}

// Columns of V one workgroup (blockIdx.y) takes.
template <int P> constexpr int tall_cols() { return P == 1 ? 32 : 64; }

// W - alpha_k sigma_k r instead of W itself, rounded to the vectors' type (the
// scalar recurrence's pass B, which then needs no launch of its own): alpha_k
// is summed here from the H x pass's partials.
template <typename T>
struct TallSub {
    const T *r = nullptr;            // nullptr: W as it is
    const double *apart = nullptr;   // alpha partials (nullptr: finished already)
    int n_hx = 0, k = 0;
    double *alpha = nullptr;
    const double *sigma = nullptr;
};

// alpha_k sigma_k of a TallSub; `write`: this workgroup stores alpha_k.
template <typename T>
__device__ __forceinline__ double tall_factor(const TallSub<T> &sub, double *red, bool write) {
    const double al = sub.apart ? fold_sum<kFinishBlock>(sub.apart, sub.n_hx, red) : sub.alpha[sub.k];
    if (write && sub.apart && threadIdx.x == 0) sub.alpha[sub.k] = al;
    return uniform(al * sub.sigma[sub.k]);
}

// partial[split][col][c] over the rows of split blockIdx.x.  The run has
// stopped, and nothing is done, if *stopped != 0 or *live == 0 (null: neither).
// NG = 1 takes at most 16 columns of the scalar recurrence, with twice the rows
// in flight (92,378 rows, up to 8 columns, FP32: 8.8 -> 5.7 us, with pass B and
// alpha 12.4 -> 7.6).
template <typename T, int P, bool SUB = false, int NG = 2>
__global__ __launch_bounds__(kTallBlock) void tall_dots_kernel(
    const T *__restrict__ V, const T *__restrict__ W, int64_t dim, int ncol,
    double *__restrict__ partial, const int *__restrict__ stopped,
    const double *__restrict__ live, const TallSub<T> sub) {
    static_assert((!SUB && NG == 2) || P == 1, "scalar recurrence");
    if ((stopped && *stopped) || (live && *live == 0.0)) return;
    double factor = 0.0;
    if constexpr (SUB) {
        __shared__ double red[17];
        factor = tall_factor(sub, red, blockIdx.x == 0 && blockIdx.y == 0);
    }
    constexpr int NA = P == 1 ? NG : 2 * NG;       // accumulators of 16 columns
    constexpr int kRows = P == 1 ? 8 : 4;          // rows of one load
    constexpr int U = 8 / NG;                      // loads of a column in flight
    __shared__ double stage[4][16 * NA][P];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int i = lane & 15, kk = lane >> 4;
    const int col0 = blockIdx.y * tall_cols<P>();
    const T *vp[NG];
    bool vok[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int c = P == 1 ? col0 + 16 * g + i : col0 + 32 * g + 2 * i;
        vok[g] = c < ncol;
        const int cc = vok[g] ? c : 0;
        vp[g] = V + (size_t)(cc / P) * (size_t)dim * P + cc % P;
    }
    const bool wok = i < P;
    const T *wp = W + (wok ? i : 0);
    v4d acc[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[a] = v4d{0.0, 0.0, 0.0, 0.0};
    // row ranges in whole steps of the workgroup (4 waves x U loads)
    constexpr int kStep = 4 * U * kRows;
    const int64_t nstep = (dim + kStep - 1) / kStep;
    const int64_t s0 = nstep * blockIdx.x / gridDim.x, s1 = nstep * (blockIdx.x + 1) / gridDim.x;
    for (int64_t s = s0; s < s1; ++s) {
        const int64_t base = s * kStep + wid * (U * kRows);
        double a0[U][NG], a1[U][NG], b0[U], b1[U];
        if constexpr (P == 1) {
            // all loads first, rows past the end read from inside: the values
            // are converted and combined, and a branch around a load would wait
            // for it there
            Two<T> va[U][NG], vw[U], vr[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t r = base + u * kRows + 2 * kk;
                const int64_t rr = max(min(r, dim - 2), (int64_t)0);
#pragma unroll
                for (int g = 0; g < NG; ++g) va[u][g] = load2(vp[g] + rr);
                vw[u] = load2(wp + rr);
                if constexpr (SUB) vr[u] = load2(sub.r + rr);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t r = base + u * kRows + 2 * kk;
                const bool two = r + 1 < dim, one = r < dim;
                const bool at = two || dim == 1;   // the pair that was read starts at r
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    a0[u][g] = vok[g] && one ? (double)(at ? va[u][g].x : va[u][g].y) : 0.0;
                    a1[u][g] = vok[g] && two ? (double)va[u][g].y : 0.0;
                }
                b0[u] = (double)(at ? vw[u].x : vw[u].y);
                b1[u] = (double)vw[u].y;
                if constexpr (SUB) {
                    b0[u] = (double)(T)(b0[u] - factor * (double)(at ? vr[u].x : vr[u].y));
                    b1[u] = (double)(T)(b1[u] - factor * (double)vr[u].y);
                }
                b0[u] = wok && one ? b0[u] : 0.0;
                b1[u] = wok && two ? b1[u] : 0.0;
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                b0[u] = 0.0;
                const int64_t r = base + u * kRows + kk;
                const bool ok = r < dim;
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    a0[u][g] = a1[u][g] = 0.0;
                    if (vok[g] && ok) {
                        const Two<T> v = load2(vp[g] + r * P);
                        a0[u][g] = (double)v.x;
                        a1[u][g] = (double)v.y;
                    }
                }
                if (wok && ok) b0[u] = (double)wp[r * P];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if constexpr (P == 1) {
                    acc[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[u][g], b0[u], acc[g], 0, 0, 0);
                    acc[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[u][g], b1[u], acc[g], 0, 0, 0);
                } else {
                    acc[2 * g] =
                        __builtin_amdgcn_mfma_f64_16x16x4f64(a0[u][g], b0[u], acc[2 * g], 0, 0, 0);
                    acc[2 * g + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[u][g], b0[u],
                                                                          acc[2 * g + 1], 0, 0, 0);
                }
            }
    }
    // result element (m, n) of an accumulator: register v of lane l holds
    // m = 4 v + l / 16, n = l % 16
    if (wok) {
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = 4 * v + kk;
                const int c = P == 1 ? 16 * a + m : 32 * (a / 2) + 2 * m + a % 2;
                stage[wid][c][i] = acc[a][v];
            }
    }
    __syncthreads();
    double *__restrict__ out = partial + ((size_t)blockIdx.x * ncol + col0) * P;
    const int mine = min(tall_cols<P>(), ncol - col0) * P;
    for (int t = threadIdx.x; t < mine; t += kTallBlock) {
        const double *q = &stage[0][0][0] + t;
        constexpr int kWave = 16 * NA * P;
        out[t] = ((q[0] + q[kWave]) + q[2 * kWave]) + q[3 * kWave];
    }
}

// One workgroup sums `nout` consecutive results over the splits in a fixed
// order (64 results x 4 slices of the splits, then the slices in order);
// out[o] for o in [first, first + 64).
__device__ __forceinline__ void tall_sum(const double *__restrict__ partial, int splits, int nout,
                                         int first, double *__restrict__ out,
                                         double (*red)[64] /* [4][64] */) {
    const int o = first + (threadIdx.x & 63), sl = threadIdx.x >> 6;
    double s = 0.0;
    if (o < nout) {
        const int a = splits * sl / 4, b = splits * (sl + 1) / 4;
        int t = a;
        for (; t + 8 <= b; t += 8) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = partial[(size_t)(t + u) * nout + o];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; t < b; ++t) s += partial[(size_t)t * nout + o];
    }
    red[sl][threadIdx.x & 63] = s;
    __syncthreads();
    if (sl == 0 && o < nout) {
        const int l = threadIdx.x & 63;
        out[o] = ((red[0][l] + red[1][l]) + red[2][l]) + red[3][l];
    }
    __syncthreads();
}

// Row ranges of a launch: enough workgroups to fill the chip a few times, at
// least two steps of rows each.
template <int P>
inline int tall_splits(int64_t dim, int ncol) {
    const int64_t step = 4 * 4 * (P == 1 ? 8 : 4);
    const int ny = (ncol + tall_cols<P>() - 1) / tall_cols<P>();
    int64_t s = (dim + 2 * step - 1) / (2 * step);
    s = s < 1024 / ny ? s : 1024 / ny;
    s = s < kTallSplits ? s : kTallSplits;
    return (int)(s > 1 ? s : 1);
}

}  // namespace hm
