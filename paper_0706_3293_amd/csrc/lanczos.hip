// Lanczos three-term recurrence on the GPU (Paige's ordering), the
// ground-state recompute pass and the host tridiagonal eigensolver.
//
// Step k (0-based) with v_k = sigma_k r_k kept as a raw vector r_k and a
// device scalar sigma_k:
//   pass A  beta_{k-1} = |w| of step k - 1; breakdown test; sigma_k =
//           1/beta_{k-1}, cprev_k = beta_{k-1} sigma_{k-1}
//           w = sigma_k (H r_k) - cprev_k r_{k-1}      [fused in the H x kernel]
//           alpha partials  <w, v_k>                   [same kernel, FP64]
//   pass B  alpha_k = sum of partials
//           w -= alpha_k v_k,  partials of |w|^2       [FP64 arithmetic]
//           [ground-state pass: psi += c_k v_k]
// or, with full reorthogonalization, twice h = V^T w, w -= V h in place of
// pass B, whose subtraction the first of them takes over.
// The raw buffers rotate (r_{k+1} is w), so the 1/beta normalization never
// costs a vector pass.  All reductions are per-workgroup partials that the next
// kernel sums in a fixed order (lanczos_dev.h; a kernel of one workgroup on
// large grids): two runs with the same inputs give the same bits, which the
// recompute pass relies on.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "device_common.h"
#include "hm_internal.h"
#include "hx_row.h"
#include "tall_dots.h"

namespace hm {

int launch_hx_generic(const Basis *b, const Couplings *c, int dtype, const HxPass &p,
                      hipStream_t st);
int hx_generic_grid(const Basis *b);
int launch_hx_half(const Basis *b, const Couplings *c, int dtype, bool staged, const HxPass &p,
                   hipStream_t st);
int hx_half_grid(const Basis *b);
int hx_half_chain(const Basis *b);
int hx_staged_grid(const Basis *b);
bool half_supported(const Basis *b);
int half_prepare_tables(Basis *b, const Couplings *c, bool staged);
bool half_fits(const Basis *b, const Couplings *c);
bool staged_fits(const Basis *b, const Couplings *c, int dtype);
int half_low_bits(const Basis *b);
int launch_hx_digit(const Basis *b, const Couplings *c, int dtype, const HxPass &p,
                    hipStream_t st);
int hx_digit_grid(const Basis *b);
int digit_prepare_tables(Basis *b, const Couplings *c, int dtype);
bool digit_fits(const Basis *b, const Couplings *c);
int launch_hx_wg(const Basis *b, const Couplings *c, bool items, const HxPass &p,
                 hipStream_t st);
int hx_wg_grid(const Basis *b);
int wg_prepare_tables(Basis *b, const Couplings *c);
bool wg_fits(const Basis *b, const Couplings *c, int dtype);

// 0 = automatic (the block kernel of the spin, where it applies to the basis
// and its tables fit the budget, else the generic digit kernel), 1 = generic,
// 2 = spin-1/2 block kernel (-1 if it does not apply).  Chosen by 0 only:
// kKernelDigit, the block kernel for s >= 1, kKernelWg, the spin-1/2 kernel with
// one workgroup per block, kKernelStaged, the spin-1/2 block kernel in its
// automatic FP64 split, and for a run without reorthogonalization (plain_run)
// kKernelWgItems, kKernelWg with the dots of kernel 2 in a launch of their own.
constexpr int kKernelDigit = 5, kKernelWg = 6, kKernelStaged = 7, kKernelWgItems = 8;

// Past convergence such a run amplifies its roundings (all-to-all model, 20 sites,
// 300 steps: 1e-16 to 4e-9 of dE0/dJ), so its sums keep kernel 2's order.  The
// launch of the dots pays where kernel 2's waves take three items or more in turn,
// or have many bonds to gather (us a FP64 step, kernel 2 / kKernelWgItems): N = 14
// (14 in turn) 51 / 21, N = 15 (6) 29 / 20, N = 16 (3) 22.3 / 19.8, N = 17 (2, 34
// bonds) 19.6 / 19.8; with all bonds N = 17 (136) 36 / 33, N = 20 (190) 48 / 39; N = 12
// and 13 (1, 66 and 78) 17 / 25 and 19 / 27.
constexpr int kItemsChain = 3, kItemsBonds = 128;
static bool wg_items_pay(const Basis *b, const Couplings *c) {
    return hx_half_chain(b) >= kItemsChain || c->nb >= kItemsBonds;
}

int choose_kernel(const Basis *b, const Couplings *c, int requested, int dtype, bool plain_run) {
    if (requested == 1) return 1;
    if (requested == 0 && b->two_s >= 2) return digit_fits(b, c) ? kKernelDigit : 1;
    if (requested == 0 && wg_fits(b, c, dtype)) {
        if (!plain_run) return kKernelWg;
        if (c && wg_items_pay(b, c)) return kKernelWgItems;
    }
    if (requested == 0 && c && staged_fits(b, c, dtype)) return kKernelStaged;
    const bool ok = c ? half_fits(b, c) : half_supported(b);
    if (requested == 2) return ok ? 2 : -1;
    return ok ? 2 : 1;
}

int hx_partial_count(const Basis *b, int kernel) {
    switch (kernel) {
        case 2: return hx_half_grid(b);
        case kKernelDigit: return hx_digit_grid(b);
        case kKernelWg: return hx_wg_grid(b);
        case kKernelWgItems: return hx_half_grid(b);
        case kKernelStaged: return hx_staged_grid(b);
        default: return hx_generic_grid(b);
    }
}

int prepare_kernel(Basis *b, const Couplings *c, int dtype, int kernel) {
    if (kernel == 2 || kernel == kKernelStaged)
        return half_prepare_tables(b, c, kernel == kKernelStaged);
    if (kernel == kKernelDigit) return digit_prepare_tables(b, c, dtype);
    if (kernel == kKernelWg || kernel == kKernelWgItems) return wg_prepare_tables(b, c);
    return HM_OK;
}

int launch_hx(const Basis *b, const Couplings *c, int dtype, int kernel, const HxPass &p,
              hipStream_t st) {
    if (kernel == 2 || kernel == kKernelStaged)
        return launch_hx_half(b, c, dtype, kernel == kKernelStaged, p, st);
    if (kernel == kKernelDigit) return launch_hx_digit(b, c, dtype, p, st);
    if (kernel == kKernelWg || kernel == kKernelWgItems)
        return launch_hx_wg(b, c, kernel == kKernelWgItems, p, st);
    return launch_hx_generic(b, c, dtype, p, st);
}

// One-workgroup runs (below).  With tables up to kTableRows rows; without, when
// asked for explicitly, up to kSmallMaxDim rows.
constexpr int64_t kTableRows = 3072;
constexpr int64_t kSmallMaxDim = 1 << 20;
constexpr int kTableCoefs = 1024;    // most reorthogonalization coefficients (LDS)
// With reorthogonalization: most bytes of matrix elements, and of stored vectors in
// a step, that one compute unit reads faster than a step's launches take.  One workgroup against
// several kernels, us a step: 2,024 rows, 97,152 row-bonds FP64 10.1 / 18.7;
// 1,716 rows, 133,848 row-bonds FP64 19.4 / 19.1, FP32 12.6 / 20.3; 60
// reorthogonalized steps at 924 rows FP64 20 / 31, at 1,716 rows FP64 33 / 34,
// FP32 17 / 38, at 2,024 rows FP64 41 / 38.
constexpr int64_t kTableBytes = 768 * 1024;

// Most ladder moves a row can have: every move lowers a site that is not at 0
// and raises one that is not at 2s.
static int64_t max_moves(const Basis *b) {
    const int64_t down = std::min<int64_t>(b->A, b->N);
    const int64_t up = std::min<int64_t>((int64_t)b->N * b->two_s - b->A, b->N);
    return (std::min(down * up, (int64_t)b->N * (b->N - 1)) + 3) / 4 * 4;
}

struct Layout {
    size_t lz, alpha, beta, sigma, cprev, scale, coef, hcoef, partial, bpart, dots, r0, r1, r2, V,
        states, mtgt, mcf, total;
    int grid_vec, grid_b, nparts;
};

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

static int vec_grid(int64_t n) {
    int64_t g = (n + kBlock - 1) / kBlock;
    g = std::min<int64_t>(g, kMaxGrid);
    g = std::max<int64_t>(g, 1);
    if (g >= kXcds) g -= g % kXcds;
    return (int)g;
}

// Slices (partials) of pass B: about 8 16-byte vectors per thread of 256, so that long
// vectors run on many more workgroups than fit at once and the dispatcher
// keeps every CU busy to the end (601 M FP32 rows: 1.51 ms on 2048
// workgroups, 1.36 ms on 65536); a row or two per thread on shorter ones.
constexpr int64_t kMaxGridB = 65536;
static int pass_b_grid(int64_t n, size_t es) {
    const int64_t per = (int64_t)(16 / es) * kBlock * 8;
    int64_t g = std::min<int64_t>((n + per - 1) / per, kMaxGridB);
    g = std::max<int64_t>(g, vec_grid(n));
    if (g >= kXcds) g -= g % kXcds;
    return (int)g;
}
// Grids (pass B's and the H x pass's) up to which pass B goes by single rows.
constexpr int kRowsMaxGrid = 64;

// Workspace layout; the partial-sum area holds one entry per workgroup of
// whichever H x kernel may run (kMaxGrid, or a block kernel's grid when that is
// larger), so the layout does not depend on the kernel choice.
static Layout layout(const Basis *b, int steps, int prec, int reorth) {
    Layout L{};
    const size_t es = prec == HM_PREC_F64 ? 8 : 4;
    L.grid_vec = vec_grid(b->dim);
    L.grid_b = pass_b_grid(b->dim, es);
    L.nparts = std::max({kMaxGrid, half_supported(b) ? hx_half_grid(b) : 0, hx_staged_grid(b),
                         b->digit.K > 0 ? hx_digit_grid(b) : 0});
    size_t off = 0;
    // state, alpha, beta and sigma side by side: read back in one copy
    L.lz = off; off = align256(off + sizeof(LzDev));
    L.alpha = off; off = align256(off + sizeof(double) * steps);
    L.beta = off; off = align256(off + sizeof(double) * steps);
    L.sigma = off; off = align256(off + sizeof(double) * (steps + 1));
    L.cprev = off; off = align256(off + sizeof(double) * (steps + 1));
    L.scale = off; off = align256(off + sizeof(double) * (steps + 1));
    L.coef = off; off = align256(off + sizeof(double) * steps);
    L.hcoef = off; off = align256(off + sizeof(double) * (steps + 1));
    L.partial = off; off = align256(off + sizeof(double) * (size_t)L.nparts);
    L.bpart = off; off = align256(off + sizeof(double) * (size_t)std::max(kMaxGrid, L.grid_b));
    L.dots = off;
    if (reorth) off = align256(off + sizeof(double) * (size_t)kTallSplits * (size_t)steps);
    L.r0 = off; off = align256(off + es * (size_t)b->dim);
    L.r1 = off; off = align256(off + es * (size_t)b->dim);
    L.r2 = off; off = align256(off + es * (size_t)b->dim);
    L.V = off;
    if (reorth) off = align256(off + es * (size_t)b->dim * (size_t)steps);
    // decoded states of the one-workgroup run (any basis it may take)
    L.states = off;
    if (b->dim <= kSmallMaxDim) off = align256(off + sizeof(uint64_t) * (size_t)b->dim);
    // move tables of the one-workgroup run
    if (b->dim <= kTableRows) {
        L.mtgt = off; off = align256(off + sizeof(uint16_t) * (size_t)(b->dim * max_moves(b)));
        L.mcf = off; off = align256(off + es * (size_t)(b->dim * max_moves(b)));
    }
    L.total = off;
    return L;
}

// ---------------------------------------------------------------------------
// Vector kernels.  Each workgroup owns one contiguous slice of rows (XCD-aware
// order) and writes one FP64 partial.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kBlock) void sumsq_kernel(const T *__restrict__ x, int64_t n,
                                                       double *__restrict__ partial) {
    __shared__ double red[16];
    int64_t first, last;
    block_rows<int64_t>(xcd_logical_block(blockIdx.x, gridDim.x), gridDim.x, n, first, last);
    double s = 0.0;
    for (int64_t i = first + threadIdx.x; i < last; i += blockDim.x) {
        const double v = (double)x[i];
        s += v * v;
    }
    s = block_sum(s, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// Sum of n partials in a fixed order by one workgroup: thread t adds
// partials t, t + blockDim, t + 2 blockDim, ... in that order, then the wave
// and workgroup sums combine the threads in a fixed order.
__device__ double fixed_sum(const double *__restrict__ partial, int n, double *red) {
    // 16 loads in flight per thread before their additions (large grids of
    // the H x pass write up to 2^20 partials; their loads are served from
    // beyond L2, since other XCDs wrote them)
    constexpr int U = 16;
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
    return block_sum(s, red);
}

// r_0 = v0 / |v0| from the partials of |v0|^2, and the run's first scalars.
template <typename T>
__global__ __launch_bounds__(kBlock) void init_write(const double *__restrict__ v0,
                                                     T *__restrict__ r, int64_t n, LzDev *lz,
                                                     const double *__restrict__ partial, int np,
                                                     double *sigma, double *cprev, double *scale,
                                                     double tol) {
    __shared__ double red[17];
    const double s = fold_sum<kEndsBlock>(partial, np, red);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        lz->bad_start = !(s > 0.0);
        lz->stopped = 0;
        lz->tol = tol;
        lz->norm0 = sqrt(s);
        lz->psi_norm = 0.0;
        sigma[0] = s > 0.0 ? 1.0 : 0.0;
        cprev[0] = 0.0;
        scale[0] = 0.0;
    }
    if (!(s > 0.0)) return;
    const double inv = 1.0 / sqrt(s);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        r[i] = (T)(v0[i] * inv);
}

// On grids of more than kFoldMax workgroups the sums have kernels of their own.
__global__ __launch_bounds__(kFinishBlock) void finish_alpha(const double *sigma,
                                                             const double *partial, int n,
                                                             double *alpha, int k) {
    if (sigma[k] == 0.0) return;
    __shared__ double red[16];
    const double s = fixed_sum(partial, n, red);
    if (threadIdx.x == 0) alpha[k] = s;
}

// 16-byte vector type of an element type.
template <typename T> struct VecOf;
template <> struct VecOf<float> { using type = float4; };
template <> struct VecOf<double> { using type = double2; };

// w -= alpha_k sigma_k r_k (FP64 arithmetic, one rounding), partial |w|^2.
// apart: the H x pass's alpha partials (null: alpha_k is finished already).
// PSI: the ground-state pass, psi += c_k v_k = c_k sigma_k r_k in FP64 (the
// first step writes psi); r_k is read anyway, so this saves a launch and a
// read of r_k per step.
//
// The rows are cut into `slices`, each summed like a workgroup of 256 threads
// would: thread t takes vectors t, t + 256, ..., then the lanes of every wave and
// the four waves in turn are added.  Here a wave takes a whole slice, its lanes the
// four threads of that number, so a slice's sum needs no barrier and a workgroup
// folds alpha_k once for several of them.  GROUPED: a workgroup takes the eight
// slices of a group of fold_groups, two per wave, and writes their sum (kGroups
// workgroups); else four slices, each with a partial of its own.
template <typename T, bool PSI, bool GROUPED>
__global__ __launch_bounds__(kBlock) void pass_b(T *__restrict__ w, const T *__restrict__ r,
                                                 int64_t n, int slices,
                                                 const double *__restrict__ apart, int n_hx,
                                                 double *__restrict__ alpha,
                                                 const double *__restrict__ sigma, int k,
                                                 bool vectors, double *__restrict__ partial,
                                                 const double *__restrict__ coef,
                                                 double *__restrict__ psi) {
    if (sigma[k] == 0.0) return;
    __shared__ double red[17];
    constexpr int S = GROUPED ? 2 : 1;            // slices of a wave
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    // slice b lies where workgroup b of as many would have its rows: those of one
    // XCD are consecutive (workgroup b runs on XCD b % 8, here too)
    int b[S];
    if constexpr (GROUPED) {
#pragma unroll
        for (int i = 0; i < S; ++i)
            b[i] = blockIdx.x / 16 * 64 + blockIdx.x % 16 + 16 * wid + 1024 * i;
    } else {
        b[0] = slices % kXcds == 0
                   ? (blockIdx.x / kXcds * 4 + wid) * kXcds + blockIdx.x % kXcds
                   : blockIdx.x * 4 + wid;
    }
    // 16-byte vector loads and stores over the aligned middle of the range
    // (the buffers start on 256-byte boundaries), single elements at its ends
    constexpr int V = 16 / sizeof(T);
    using Vec = typename VecOf<T>::type;
    Vec *wv = reinterpret_cast<Vec *>(w);
    const Vec *rv = reinterpret_cast<const Vec *>(r);
    int64_t i0[S], j0[S], m0[S], m1[S], j1[S], last[S];
    // the first loads are on their way while alpha_k is summed
    Vec wj[S][4], rj[S][4];
    T wi[S][4], ri[S][4];
#pragma unroll
    for (int i = 0; i < S; ++i) {
        int64_t first = 0;
        last[i] = 0;
        if (b[i] < slices)
            block_rows<int64_t>(xcd_logical_block(b[i], slices), slices, n, first, last[i]);
        m0[i] = vectors ? std::min(last[i], (first + V - 1) / V * V) : last[i];
        m1[i] = std::max(m0[i], last[i] / V * V);
        i0[i] = first + lane;
        j0[i] = m0[i] / V + lane;
        j1[i] = m1[i] / V;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (j0[i] + 64 * q < j1[i]) {
                wj[i][q] = wv[j0[i] + 64 * q];
                rj[i][q] = rv[j0[i] + 64 * q];
            }
            if (i0[i] + 64 * q < m0[i]) {
                wi[i][q] = w[i0[i] + 64 * q];
                ri[i][q] = r[i0[i] + 64 * q];
            }
        }
    }
    const double al = apart ? fold_sum<kFinishBlock>(apart, n_hx, red) : alpha[k];
    if (apart && blockIdx.x == 0 && threadIdx.x == 0) alpha[k] = al;
    const double sg = sigma[k], a = al * sg;
    const double cp = PSI ? coef[k] * sg : 0.0;
    double sum = 0.0;
#pragma unroll
    for (int i = 0; i < S; ++i) {
        double s[4] = {0.0, 0.0, 0.0, 0.0};
        auto one = [&](int q, int64_t at, T wo, T ro) {
            const T wn = (T)((double)wo - a * (double)ro);
            w[at] = wn;
            s[q] += (double)wn * (double)wn;
            if constexpr (PSI) psi[at] = (k > 0 ? psi[at] : 0.0) + cp * (double)ro;
        };
        auto vec = [&](int q, int64_t jj, Vec wo, const Vec ro) {
            T *we = reinterpret_cast<T *>(&wo);
            const T *re = reinterpret_cast<const T *>(&ro);
#pragma unroll
            for (int e = 0; e < V; ++e) {
                we[e] = (T)((double)we[e] - a * (double)re[e]);
                s[q] += (double)we[e] * (double)we[e];
            }
            wv[jj] = wo;
            if constexpr (PSI)
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const int64_t at = jj * V + e;
                    psi[at] = (k > 0 ? psi[at] : 0.0) + cp * (double)re[e];
                }
        };
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (i0[i] + 64 * q < m0[i]) one(q, i0[i] + 64 * q, wi[i][q], ri[i][q]);
            for (int64_t at = i0[i] + 64 * q + 256; at < m0[i]; at += 256)
                one(q, at, w[at], r[at]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (j0[i] + 64 * q < j1[i]) vec(q, j0[i] + 64 * q, wj[i][q], rj[i][q]);
        for (int64_t j = j0[i] + 256; j < j1[i]; j += 256) {
            Vec wn[4], rn[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (j + 64 * q < j1[i]) {
                    wn[q] = wv[j + 64 * q];
                    rn[q] = rv[j + 64 * q];
                }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (j + 64 * q < j1[i]) vec(q, j + 64 * q, wn[q], rn[q]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            for (int64_t at = m1[i] + lane + 64 * q; at < last[i]; at += 256)
                one(q, at, w[at], r[at]);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
            for (int q = 0; q < 4; ++q) s[q] += __shfl_xor(s[q], off, 64);
        const double slice = ((s[0] + s[1]) + s[2]) + s[3];
        sum = i == 0 ? slice : sum + slice;
    }
    if constexpr (GROUPED) {
        if (lane == 0) red[wid] = sum;
        __syncthreads();
        if (threadIdx.x == 0) partial[blockIdx.x] = (red[0] + red[2]) + (red[1] + red[3]);
    } else {
        if (lane == 0 && b[0] < slices) partial[b[0]] = sum;
    }
}

// The same for long vectors, alpha_k finished: a workgroup takes a slice, so that its
// loads stay together in memory (601 M FP32 rows: 1.47 ms, with a wave for each slice
// 1.50).
template <typename T, bool PSI>
__global__ __launch_bounds__(kBlock) void pass_b_long(T *__restrict__ w, const T *__restrict__ r,
                                                      int64_t n, const double *__restrict__ alpha,
                                                      const double *__restrict__ sigma, int k,
                                                      double *__restrict__ partial,
                                                      const double *__restrict__ coef,
                                                      double *__restrict__ psi) {
    if (sigma[k] == 0.0) return;
    __shared__ double red[16];
    int64_t first, last;
    block_rows<int64_t>(xcd_logical_block(blockIdx.x, gridDim.x), gridDim.x, n, first, last);
    constexpr int V = 16 / sizeof(T);
    using Vec = typename VecOf<T>::type;
    const int64_t m0 = std::min(last, (first + V - 1) / V * V);
    const int64_t m1 = std::max(m0, last / V * V);
    Vec *wv = reinterpret_cast<Vec *>(w);
    const Vec *rv = reinterpret_cast<const Vec *>(r);
    const double sg = sigma[k], a = alpha[k] * sg;
    const double cp = PSI ? coef[k] * sg : 0.0;
    double s = 0.0;
    auto one = [&](int64_t i) {
        const T ri = r[i], wi = (T)((double)w[i] - a * (double)ri);
        w[i] = wi;
        s += (double)wi * (double)wi;
        if constexpr (PSI) psi[i] = (k > 0 ? psi[i] : 0.0) + cp * (double)ri;
    };
    for (int64_t i = first + threadIdx.x; i < m0; i += blockDim.x) one(i);
#pragma unroll 2
    for (int64_t j = m0 / V + threadIdx.x; j < m1 / V; j += blockDim.x) {
        Vec wj = wv[j];
        const Vec rj = rv[j];
        T *we = reinterpret_cast<T *>(&wj);
        const T *re = reinterpret_cast<const T *>(&rj);
#pragma unroll
        for (int e = 0; e < V; ++e) {
            we[e] = (T)((double)we[e] - a * (double)re[e]);
            s += (double)we[e] * (double)we[e];
        }
        wv[j] = wj;
        if constexpr (PSI)
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const int64_t i = j * V + e;
                psi[i] = (k > 0 ? psi[i] : 0.0) + cp * (double)re[e];
            }
    }
    for (int64_t i = m1 + threadIdx.x; i < last; i += blockDim.x) one(i);
    s = block_sum(s, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// beta_k and the scalars of step k + 1 from the |w|^2 partials.
__global__ __launch_bounds__(kFinishBlock) void finish_beta(const LzDev *lz,
                                                            const double *partial, int n,
                                                            const double *alpha,
                                                            double *beta, double *sigma,
                                                            double *cprev, double *scale, int k) {
    if (sigma[k] == 0.0) {
        if (threadIdx.x == 0) sigma[k + 1] = 0.0;
        return;
    }
    __shared__ double red[16];
    const double s = n ? fixed_sum(partial, n, red) : fold_groups(partial, red);
    if (threadIdx.x == 0) {
        const LzScalars c = lz_advance(lz, k + 1, s, alpha, sigma, scale);
        beta[k] = c.beta;
        scale[k + 1] = c.scale;
        sigma[k + 1] = c.sigma;
        cprev[k + 1] = c.cprev;
    }
}

// Full reorthogonalization, second half of a pass: w -= sum_{j < nv} h_j V_j
// with h_j summed from the dots' partials (splits x nv; h given instead: they
// are finished already).  SUB: w - alpha_k sigma_k r_k is what the dots were
// taken with.  sq: partials of |w|^2 (the second pass).  Each thread keeps 8
// entries of V in flight; the sums take the vectors in order.
constexpr int kReorthFold = 1024;    // most coefficients a workgroup sums itself

template <typename T, bool SUB>
__global__ __launch_bounds__(kBlock) void reorth_update(const T *__restrict__ V,
                                                        T *__restrict__ w, int64_t n, int nv,
                                                        const double *__restrict__ dots, int splits,
                                                        const double *__restrict__ h,
                                                        const double *__restrict__ live,
                                                        double *__restrict__ sq,
                                                        const TallSub<T> sub) {
    if (*live == 0.0) return;
    __shared__ double red[17];
    __shared__ double hs[kReorthFold];
    double factor = 0.0;
    if constexpr (SUB) factor = tall_factor(sub, red, false);
    if (!h) {
        for (int j = threadIdx.x; j < nv; j += blockDim.x) {
            double s = 0.0;
            for (int t = 0; t < splits; ++t) s += dots[(size_t)t * nv + j];
            hs[j] = s;
        }
        __syncthreads();
        h = hs;
    }
    double s = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        double acc = (double)w[i];
        if constexpr (SUB) acc = (double)(T)(acc - factor * (double)sub.r[i]);
        const T *__restrict__ Vi = V + i;
        int j = 0;
        for (; j + 8 <= nv; j += 8) {
            T v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = Vi[(size_t)(j + q) * (size_t)n];
#pragma unroll
            for (int q = 0; q < 8; ++q) acc -= h[j + q] * (double)v[q];
        }
        for (; j < nv; ++j) acc -= h[j] * (double)Vi[(size_t)j * (size_t)n];
        const T wi = (T)acc;
        w[i] = wi;
        s += (double)wi * (double)wi;
    }
    if (sq) {
        s = block_sum(s, red);
        if (threadIdx.x == 0) sq[blockIdx.x] = s;
    }
}

// h_j from the partials of the dots (64 coefficients per workgroup).
__global__ __launch_bounds__(kTallBlock) void reorth_finish(const double *__restrict__ dots,
                                                            int splits, int nv,
                                                            double *__restrict__ h,
                                                            const double *__restrict__ live) {
    if (*live == 0.0) return;
    __shared__ double red[4][64];
    tall_sum(dots, splits, nv, blockIdx.x * 64, h, red);
}

// Ground-state accumulation of the reorthogonalized recurrence, which has no
// pass B to do it (the first step writes psi).
template <typename T>
__global__ __launch_bounds__(kBlock) void psi_axpy(double *__restrict__ psi,
                                                   const T *__restrict__ r, int64_t n,
                                                   const double *__restrict__ coef,
                                                   const double *__restrict__ sigma, int k) {
    if (sigma[k] == 0.0) return;
    const double a = coef[k] * sigma[k];
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        psi[i] = (k > 0 ? psi[i] : 0.0) + a * (double)r[i];
}

// psi /= |psi| from the partials of |psi|^2.
__global__ __launch_bounds__(kBlock) void scale_psi(double *__restrict__ psi, int64_t n, LzDev *lz,
                                                    const double *__restrict__ partial, int np) {
    __shared__ double red[17];
    const double nrm = sqrt(fold_sum<kEndsBlock>(partial, np, red));
    if (blockIdx.x == 0 && threadIdx.x == 0) lz->psi_norm = nrm;
    if (!(nrm > 0.0)) return;
    const double inv = 1.0 / nrm;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        psi[i] *= inv;
}

// ---------------------------------------------------------------------------
// Small problems: the whole run in one workgroup.
//
// For a few thousand rows a step is little work, but its launches cost 5 us
// each (two without, five with full reorthogonalization).  Here one workgroup
// of 1024 threads runs every step in a single launch: thread t owns rows t,
// t + 1024, ..., reductions are fixed trees, and workgroup barriers order the
// passes, so a run is reproducible and the recompute pass repeats it bit for
// bit.  The recurrence is the same (Paige's ordering, the same breakdown
// test).  One compute unit does all the row work.
//
// lanczos_table_kernel (up to kTableRows rows) finds every row's moves and
// matrix elements once at the start of the run and keeps them in the
// workspace, v_k and w in LDS and the thread's rows in registers: at 924 rows
// and 12 bonds a step is 4.6 us in FP64 (two launches: 13.3) and over 20
// reorthogonalized steps 13 us (five launches: 28).  What bounds it is one
// compute unit's reads of the move tables and of the stored vectors from L2.
// lanczos_small_kernel (v_k stored normalized) runs larger subspaces when asked
// for explicitly.
// ---------------------------------------------------------------------------
constexpr int kSmallBlock = 1024;

template <typename T, typename I>
struct SmallArgs {
    const I *prefix;
    const double *ladder;
    const BondDev *bonds;
    int nb, N, A, two_s, steps, reorth;
    I dim;
    double tol;
    const double *v0;
    T *buf[3];
    T *V;                    // [steps][dim] normalized v_j (full reorthogonalization)
    uint64_t *states;        // [dim] decoded states, filled at the start of the run
    double *alpha, *beta, *hc;
    LzDev *lz;
    const double *coef;      // recompute pass: c_k, else nullptr
    double *psi;
};

__device__ __forceinline__ double block_bcast(double v, double *red, double *slot) {
    v = block_sum(v, red);
    if (threadIdx.x == 0) *slot = v;
    __syncthreads();
    const double r = *slot;
    __syncthreads();
    return r;
}

template <typename T, typename I, int B>
__global__ __launch_bounds__(kSmallBlock) void lanczos_small_kernel(const SmallArgs<T, I> a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[16];
    __shared__ double slot;
    const int plen = a.N * (a.A + 1) * (a.two_s + 1);
    I *P = reinterpret_cast<I *>(smem);
    T *F = reinterpret_cast<T *>(smem + ((plen * sizeof(I) + 15) / 16) * 16);
    for (int t = threadIdx.x; t < plen; t += blockDim.x) P[t] = a.prefix[t];
    for (int t = threadIdx.x; t < a.two_s + 2; t += blockDim.x) F[t] = (T)a.ladder[t];
    __syncthreads();
    const Prefix<I> pv{P, a.A + 1, a.two_s + 1};
    const I n = a.dim;
    const I tid = threadIdx.x, nt = blockDim.x;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nwv = blockDim.x >> 6;

    double s = 0.0;
    for (I i = tid; i < n; i += nt) s += a.v0[i] * a.v0[i];
    s = block_bcast(s, red, &slot);
    if (threadIdx.x == 0) {
        a.lz->tol = a.tol;
        a.lz->norm0 = sqrt(s);
        a.lz->bad_start = !(s > 0.0);
        a.lz->stopped = a.lz->bad_start ? -1 : 0;
        a.lz->psi_norm = 0.0;
    }
    if (!(s > 0.0)) return;
    const double inv0 = 1.0 / sqrt(s);
    for (I i = tid; i < n; i += nt) {
        const T v = (T)(a.v0[i] * inv0);
        a.buf[0][i] = v;
        if (a.reorth) a.V[i] = v;
        if (a.psi) a.psi[i] = 0.0;
        a.states[i] = unrank_state<I, B>(i, pv, a.N, a.A, a.two_s);
    }
    __syncthreads();
    double beta_prev = 0.0, scale = 0.0;
    int stopped = 0;
    for (int k = 0; k < a.steps; ++k) {
        const T *__restrict__ vk = a.buf[k % 3];
        const T *__restrict__ vp = a.buf[(k + 2) % 3];
        T *__restrict__ w = a.buf[(k + 1) % 3];
        // w = H v_k - beta_{k-1} v_{k-1};  alpha_k = <w, v_k>
        double dot = 0.0;
        for (I i = tid; i < n; i += nt) {
            const uint64_t st = a.states[i];
            const T xi = vk[i];
            const T hv = row_hx<T, I, B>(st, i, xi, vk, a.bonds, a.nb, a.two_s, pv, F);
            double wi = (double)hv;
            if (k > 0) wi -= beta_prev * (double)vp[i];
            const T wt = (T)wi;
            w[i] = wt;
            dot += (double)wt * (double)xi;
            if (a.psi) a.psi[i] += a.coef[k] * (double)xi;
        }
        const double alpha = block_bcast(dot, red, &slot);
        // w -= alpha_k v_k (rows of this thread only)
        double ss = 0.0;
        for (I i = tid; i < n; i += nt) {
            const T wi = (T)((double)w[i] - alpha * (double)vk[i]);
            w[i] = wi;
            ss += (double)wi * (double)wi;
        }
        if (a.reorth) {
            __syncthreads();
            for (int rep = 0; rep < 2; ++rep) {
                // h_j = <V_j, w>: one wave per j, lanes over rows, fixed tree
                for (int j = wid; j <= k; j += nwv) {
                    const T *__restrict__ Vj = a.V + (size_t)j * (size_t)n;
                    double d = 0.0;
                    for (I i = lane; i < n; i += 64) d += (double)Vj[i] * (double)w[i];
                    d = wave_sum(d);
                    if (lane == 0) a.hc[j] = d;
                }
                __syncthreads();
                for (I i = tid; i < n; i += nt) {
                    double acc = (double)w[i];
                    for (int j = 0; j <= k; ++j) acc -= a.hc[j] * (double)a.V[(size_t)j * n + i];
                    w[i] = (T)acc;
                }
                __syncthreads();
            }
            ss = 0.0;
            for (I i = tid; i < n; i += nt) ss += (double)w[i] * (double)w[i];
        }
        const double beta = sqrt(block_bcast(ss, red, &slot));
        scale = fmax(scale, fmax(fabs(alpha), beta));
        if (threadIdx.x == 0) {
            a.alpha[k] = alpha;
            a.beta[k] = beta;
        }
        if (!(beta > a.tol * scale)) {
            stopped = k + 1;
            break;
        }
        const double binv = 1.0 / beta;
        for (I i = tid; i < n; i += nt) {
            const T v = (T)((double)w[i] * binv);
            w[i] = v;
            if (a.reorth && k + 1 < a.steps) a.V[(size_t)(k + 1) * n + i] = v;
        }
        beta_prev = beta;
        __syncthreads();
    }
    if (threadIdx.x == 0) a.lz->stopped = stopped;
    if (a.psi) {
        __syncthreads();
        double q = 0.0;
        for (I i = tid; i < n; i += nt) q += a.psi[i] * a.psi[i];
        const double nrm = sqrt(block_bcast(q, red, &slot));
        if (threadIdx.x == 0) a.lz->psi_norm = nrm;
        if (nrm > 0.0)
            for (I i = tid; i < n; i += nt) a.psi[i] /= nrm;
    }
}

template <typename T>
struct TableArgs {
    const uint32_t *prefix;
    const double *ladder;
    const BondDev *bonds;
    int nb, N, A, two_s, steps, reorth, n, halfK;   // halfK > 0: the arithmetic of hx_half.hip
    int normed;              // v_k kept normalized (sigma_k = 1), as lanczos_small_kernel does
    double tol, shift;
    const double *v0;
    T *V;                    // [steps][n] normalized v_j (full reorthogonalization)
    T *r, *rprev;            // r_k and r_{k-1} for the kernels that go on, null: none do
    uint16_t *mtgt;          // [move][n] target rows
    T *mcf;                  // [move][n] matrix elements
    double *alpha, *beta, *sigma, *cprev, *scale;
    LzDev *lz;
    const double *coef;      // recompute pass: c_k, else nullptr
    double *psi;
};

// Sum over the workgroup in every thread in block_sum's order, one barrier; the
// caller alternates between two `red`, so that a fast wave cannot overwrite what a
// slow one reads.
__device__ __forceinline__ double all_sum(double v, double *red /* 16 */) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = 0.0;
#pragma unroll
    for (int w = 0; w < kSmallBlock / 64; ++w) v += red[w];
    return v;
}

template <typename T, int B>
__global__ __launch_bounds__(kSmallBlock) void lanczos_table_kernel(const TableArgs<T> a) {
    constexpr int J = (int)(kTableRows / kSmallBlock);   // rows of a thread
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[2][16];
    __shared__ double hs[kTableCoefs];
    const int n = a.n, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int plen = a.N * (a.A + 1) * (a.two_s + 1);
    uint32_t *P = reinterpret_cast<uint32_t *>(smem);
    T *F = reinterpret_cast<T *>(smem + ((plen * sizeof(uint32_t) + 15) / 16) * 16);
    for (int t = tid; t < plen; t += kSmallBlock) P[t] = a.prefix[t];
    for (int t = tid; t < a.two_s + 2; t += kSmallBlock) F[t] = (T)a.ladder[t];
    __syncthreads();
    const Prefix<uint32_t> pv{P, a.A + 1, a.two_s + 1};
    // the rows' moves in the order and with the roundings of the H x kernel
    // that the steps of larger subspaces run: row_hx's, or with halfK the
    // spin-1/2 block kernel's (low word, high word, straddling)
    T diag[J];
    int cnt[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        diag[j] = 0;
        cnt[j] = 0;
        const int i = tid + j * kSmallBlock;
        if (i >= n) continue;
        const uint64_t st = unrank_state<uint32_t, B>((uint32_t)i, pv, a.N, a.A, a.two_s);
        auto put = [&](uint32_t to, T c) {
            a.mtgt[(size_t)cnt[j] * n + i] = (uint16_t)to;
            a.mcf[(size_t)cnt[j] * n + i] = c;
            ++cnt[j];
        };
        for (int pass = 0; pass < (a.halfK ? 3 : 1); ++pass)
            for (int b = 0; b < a.nb; ++b) {
                const int u = a.bonds[b].u, v = a.bonds[b].v;
                if (a.halfK && pass != (v < a.halfK ? 0 : u >= a.halfK ? 1 : 2)) continue;
                const T mJ4 = (T)a.bonds[b].mJ4, mJ2 = (T)a.bonds[b].mJ2;
                const int au = digit_at<B>(st, u), av = digit_at<B>(st, v);
                diag[j] += mJ4 * (T)((a.two_s - 2 * au) * (a.two_s - 2 * av));
                if (au >= 1 && av < a.two_s)
                    put((uint32_t)i + move_delta<uint32_t, B>(st, u, v, -1, pv),
                        mJ2 * F[au] * F[av + 1]);
                if (av >= 1 && au < a.two_s)
                    put((uint32_t)i + move_delta<uint32_t, B>(st, u, v, +1, pv),
                        mJ2 * F[av] * F[au + 1]);
            }
        while (cnt[j] % 4) put((uint32_t)i, (T)0);   // moves are read in fours
        if (a.halfK) diag[j] = (T)a.shift;
    }
    __syncthreads();
    T *vk = reinterpret_cast<T *>(smem), *ws = vk + n;   // over the prefix table
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int i = tid + j * kSmallBlock;
        if (i < n) s += a.v0[i] * a.v0[i];
    }
    s = all_sum(s, red[0]);
    if (tid == 0) {
        a.lz->tol = a.tol;
        a.lz->norm0 = sqrt(s);
        a.lz->bad_start = !(s > 0.0);
        a.lz->stopped = a.lz->bad_start ? -1 : 0;
        a.lz->psi_norm = 0.0;
        a.sigma[0] = s > 0.0 ? 1.0 : 0.0;
        a.sigma[a.steps] = 0.0;
    }
    if (!(s > 0.0)) return;
    const double inv0 = 1.0 / sqrt(s);
    T vp[J], w[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        vp[j] = w[j] = 0;
        const int i = tid + j * kSmallBlock;
        if (i >= n) continue;
        vk[i] = (T)(a.v0[i] * inv0);
    }
    __syncthreads();
    double sigma = 1.0, cprev = 0.0, scale = 0.0;
    int stopped = 0;
    for (int k = 0; k < a.steps; ++k) {
        // w = sigma_k H r_k - cprev_k r_{k-1};  alpha_k = <w, v_k>, v_k = sigma_k r_k
        double dot = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int i = tid + j * kSmallBlock;
            if (i >= n) continue;
            const T xi = vk[i];
            T off = 0;
            for (int t = 0; t < cnt[j]; t += 4) {
                uint32_t to[4];
                T c[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    to[q] = a.mtgt[(size_t)(t + q) * n + i];
                    c[q] = a.mcf[(size_t)(t + q) * n + i];
                }
                if (a.halfK) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) off += c[q] * (vk[to[q]] - xi);
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) off += c[q] * vk[to[q]];
                }
            }
            const T hv = diag[j] * xi + off;
            double wi = sigma * (double)hv;
            if (k > 0) wi -= cprev * (double)vp[j];
            w[j] = (T)wi;
            dot += (double)w[j] * (sigma * (double)xi);
            if (a.reorth) a.V[(size_t)k * n + i] = (T)(sigma * (double)xi);
            if (a.psi)
                a.psi[i] = (k > 0 ? a.psi[i] : 0.0) + a.coef[k] * sigma * (double)xi;
        }
        const double alpha = all_sum(dot, red[0]), as = alpha * sigma;
        double ss = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int i = tid + j * kSmallBlock;
            if (i >= n) continue;
            w[j] = (T)((double)w[j] - as * (double)vk[i]);
            ss += (double)w[j] * (double)w[j];
            if (a.reorth) ws[i] = w[j];
        }
        if (a.reorth) {
            for (int rep = 0; rep < 2; ++rep) {
                __syncthreads();
                // h_c = <V_c, w>: a wave per column, 8 rows per lane in flight
                for (int c = wid; c <= k; c += kSmallBlock / 64) {
                    const T *__restrict__ Vc = a.V + (size_t)c * n;
                    double d = 0.0;
                    int i = lane;
                    for (; i + 7 * 64 < n; i += 8 * 64) {
                        T v[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q) v[q] = Vc[i + 64 * q];
#pragma unroll
                        for (int q = 0; q < 8; ++q) d += (double)v[q] * (double)ws[i + 64 * q];
                    }
                    for (; i < n; i += 64) d += (double)Vc[i] * (double)ws[i];
                    d = wave_sum(d);
                    if (lane == 0) hs[c] = d;
                }
                __syncthreads();
                ss = 0.0;
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const int i = tid + j * kSmallBlock;
                    if (i >= n) continue;
                    double acc = (double)w[j];
                    const T *__restrict__ Vi = a.V + i;
                    int c = 0;
                    for (; c + 8 <= k + 1; c += 8) {
                        T v[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q) v[q] = Vi[(size_t)(c + q) * n];
#pragma unroll
                        for (int q = 0; q < 8; ++q) acc -= hs[c + q] * (double)v[q];
                    }
                    for (; c <= k; ++c) acc -= hs[c] * (double)Vi[(size_t)c * n];
                    w[j] = (T)acc;
                    ws[i] = w[j];
                    ss += (double)w[j] * (double)w[j];
                }
            }
        }
        const double beta = sqrt(all_sum(ss, red[1]));
        scale = fmax(scale, fmax(fabs(alpha), beta));
        if (tid == 0) {
            a.alpha[k] = alpha;
            a.beta[k] = beta;
        }
        if (!(beta > a.tol * scale)) {
            stopped = k + 1;
            if (tid == 0) a.sigma[k + 1] = 0.0;
            break;
        }
        // every wave has read r_k (the barrier of the sum above)
        const double inv = 1.0 / beta;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int i = tid + j * kSmallBlock;
            if (i >= n) continue;
            vp[j] = vk[i];
            vk[i] = a.normed ? (T)((double)w[j] * inv) : w[j];
        }
        cprev = beta * sigma;
        if (!a.normed) sigma = inv;
        if (tid == 0) a.sigma[k + 1] = sigma;
        __syncthreads();
    }
    if (tid == 0) {
        a.lz->stopped = stopped;
        a.cprev[a.steps] = cprev;
        a.scale[a.steps] = scale;
    }
    if (a.r) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int i = tid + j * kSmallBlock;
            if (i >= n) continue;
            a.r[i] = vk[i];
            a.rprev[i] = vp[j];
        }
        return;
    }
    if (a.psi) {
        double q = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int i = tid + j * kSmallBlock;
            if (i < n) q += a.psi[i] * a.psi[i];
        }
        const double nrm = sqrt(all_sum(q, red[0]));
        if (tid == 0) a.lz->psi_norm = nrm;
        if (nrm > 0.0)
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int i = tid + j * kSmallBlock;
                if (i < n) a.psi[i] /= nrm;
            }
    }
}

// ---------------------------------------------------------------------------
// Host driver
// ---------------------------------------------------------------------------
static thread_local bool g_timing = false;
static thread_local double g_hx_ms = 0.0, g_loop_ms = 0.0;
static thread_local int g_hx_launches = 0;

struct Run {
    Basis *b;
    const Couplings *c;
    int steps, prec, reorth, kernel, use_graph, small;
    int table;                 // steps of lanczos_table_kernel before the step loop
    int normed;                // one-workgroup run: v_k kept normalized
    int halfK;                 // one-workgroup run: low sites of the block kernel whose
                               // arithmetic it takes (0: row_hx's)
    double tol;
    Layout L;
    unsigned char *w;
    hipStream_t st;
    const double *v0;
    const double *coef_host;   // ritz pass: c_k (host), else nullptr
    double *psi;               // ritz pass output, else nullptr
};

template <typename T>
static int enqueue_steps(Run &R, int k0, int k1, std::vector<hipEvent_t> *ev) {
    Basis *b = R.b;
    const int64_t n = b->dim;
    LzDev *lz = (LzDev *)(R.w + R.L.lz);
    double *alpha = (double *)(R.w + R.L.alpha), *beta = (double *)(R.w + R.L.beta);
    double *sigma = (double *)(R.w + R.L.sigma), *cprev = (double *)(R.w + R.L.cprev);
    double *scale = (double *)(R.w + R.L.scale);
    double *coef = (double *)(R.w + R.L.coef), *hc = (double *)(R.w + R.L.hcoef);
    double *partial = (double *)(R.w + R.L.partial), *bpart = (double *)(R.w + R.L.bpart);
    double *dots = (double *)(R.w + R.L.dots);
    T *buf[3] = {(T *)(R.w + R.L.r0), (T *)(R.w + R.L.r1), (T *)(R.w + R.L.r2)};
    T *V = (T *)(R.w + R.L.V);
    const int G = R.L.grid_vec, Gb = R.reorth ? G : R.L.grid_b;
    const int Ghx = hx_partial_count(b, R.kernel);
    const int dtype = R.prec == HM_PREC_F64 ? HM_F64 : HM_F32;
    // sums of few enough partials are left to the kernel that needs them
    const bool fold_a = Ghx <= kFoldMax, fold_b = Gb <= kFoldMax;
    const bool vectors = G > kRowsMaxGrid || Ghx > kRowsMaxGrid;
    // (few slices: a group would leave most workgroups without one)
    const bool grouped = fold_b && !R.reorth && Gb > kGroups;
    const int Wb = grouped ? kGroups
                           : Gb % kXcds == 0 ? (Gb / kXcds + 3) / 4 * kXcds : (Gb + 3) / 4;
    for (int k = k0; k < k1; ++k) {
        T *rk = buf[k % 3], *rprev = buf[(k + 2) % 3], *wn = buf[(k + 1) % 3];
        HxPass p;
        p.x = rk;
        p.y = wn;
        p.p = k > 0 ? rprev : nullptr;
        p.step.lz = lz;
        p.step.bpart = fold_b && k > R.table ? bpart : nullptr;
        p.step.nb = grouped ? 0 : Gb;
        p.step.k = k;
        p.step.alpha = alpha;
        p.step.beta = beta;
        p.step.sigma = sigma;
        p.step.cprev = cprev;
        p.step.scale = scale;
        p.partial = partial;
        p.store = R.reorth ? (void *)(V + (size_t)k * (size_t)n) : nullptr;
        if (ev) HM_HIP(hipEventRecord((*ev)[2 * k], R.st));
        HM_TRY(launch_hx(b, R.c, dtype, R.kernel, p, R.st));
        if (ev) HM_HIP(hipEventRecord((*ev)[2 * k + 1], R.st));
        if (!fold_a)
            hipLaunchKernelGGL(finish_alpha, dim3(1), dim3(kFinishBlock), 0, R.st, sigma, partial,
                               Ghx, alpha, k);
        const double *apart = fold_a ? partial : nullptr;
        if (!R.reorth && !apart && !fold_b) {
            const auto pass_b_kernel = R.psi ? pass_b_long<T, true> : pass_b_long<T, false>;
            hipLaunchKernelGGL(pass_b_kernel, dim3(Gb), dim3(kBlock), 0, R.st, wn, rk, n, alpha,
                               sigma, k, bpart, coef, R.psi);
        } else if (!R.reorth) {
            const auto pass_b_kernel = R.psi ? (grouped ? pass_b<T, true, true> : pass_b<T, true, false>)
                                             : (grouped ? pass_b<T, false, true>
                                                        : pass_b<T, false, false>);
            hipLaunchKernelGGL(pass_b_kernel, dim3(Wb), dim3(kBlock), 0, R.st, wn, rk, n, Gb, apart,
                               Ghx, alpha, sigma, k, vectors, bpart, coef, R.psi);
        } else {
            // beta is the norm after the second pass
            const int nv = k + 1, splits = tall_splits<1>(n, nv);
            const dim3 dg(splits, (nv + tall_cols<1>() - 1) / tall_cols<1>());
            const bool fold_h = nv <= kReorthFold && splits <= 16;
            TallSub<T> sub;
            sub.r = rk;
            sub.apart = apart;
            sub.n_hx = Ghx;
            sub.k = k;
            sub.alpha = alpha;
            sub.sigma = sigma;
            if (R.psi)
                hipLaunchKernelGGL(psi_axpy<T>, dim3(G), dim3(kBlock), 0, R.st, R.psi, rk, n, coef,
                                   sigma, k);
            for (int rep = 0; rep < 2; ++rep) {
                const auto dots_kernel =
                    nv <= 16 ? (rep == 0 ? tall_dots_kernel<T, 1, true, 1>
                                         : tall_dots_kernel<T, 1, false, 1>)
                             : (rep == 0 ? tall_dots_kernel<T, 1, true, 2>
                                         : tall_dots_kernel<T, 1, false, 2>);
                hipLaunchKernelGGL(dots_kernel, dg, dim3(kTallBlock), 0, R.st, V, wn, n, nv, dots,
                                   (const int *)nullptr, sigma + k, sub);
                if (!fold_h)
                    hipLaunchKernelGGL(reorth_finish, dim3((nv + 63) / 64), dim3(kTallBlock), 0,
                                       R.st, dots, splits, nv, hc, sigma + k);
                const double *h = fold_h ? nullptr : hc;
                if (rep == 0)
                    hipLaunchKernelGGL((reorth_update<T, true>), dim3(G), dim3(kBlock), 0, R.st, V,
                                       wn, n, nv, dots, splits, h, sigma + k, (double *)nullptr, sub);
                else
                    hipLaunchKernelGGL((reorth_update<T, false>), dim3(G), dim3(kBlock), 0, R.st, V,
                                       wn, n, nv, dots, splits, h, sigma + k, bpart, sub);
            }
        }
        if (!fold_b || k + 1 == R.steps)
            hipLaunchKernelGGL(finish_beta, dim3(1), dim3(kFinishBlock), 0, R.st, lz, bpart,
                               grouped ? 0 : Gb, alpha, beta, sigma, cprev, scale, k);
    }
    HM_HIP(hipGetLastError());
    return HM_OK;
}

// Waits for the run and copies its results to the host.
static int collect(const Run &R, double *alpha_h, double *beta_h, int *steps_done) {
    HM_HIP(hipGetLastError());
    const size_t bytes = R.L.sigma + sizeof(double) * (R.steps + 1) - R.L.lz;
    std::vector<unsigned char> host(bytes);
    HM_HIP(hipMemcpyAsync(host.data(), R.w + R.L.lz, bytes, hipMemcpyDeviceToHost, R.st));
    HM_HIP(hipStreamSynchronize(R.st));
    LzDev hlz;
    std::memcpy(&hlz, host.data(), sizeof hlz);
    if (hlz.bad_start) return fail(HM_EINVAL, "start vector has zero norm");
    int done = R.steps;
    if (R.small) {
        if (hlz.stopped > 0) done = hlz.stopped;
    } else {
        const double *sigma = (const double *)(host.data() + (R.L.sigma - R.L.lz));
        for (int k = 1; k <= R.steps; ++k)
            if (sigma[k] == 0.0) {
                done = k;
                break;
            }
    }
    if (alpha_h)
        std::memcpy(alpha_h, host.data() + (R.L.alpha - R.L.lz), sizeof(double) * done);
    if (beta_h) std::memcpy(beta_h, host.data() + (R.L.beta - R.L.lz), sizeof(double) * done);
    if (alpha_h) std::fill(alpha_h + done, alpha_h + R.steps, 0.0);
    if (beta_h) std::fill(beta_h + done, beta_h + R.steps, 0.0);
    *steps_done = done;
    return HM_OK;
}

template <typename T, typename I, int B>
static void launch_small_b(const Run &R) {
    const Basis *b = R.b;
    SmallArgs<T, I> a{};
    a.prefix = (const I *)b->d_prefix;
    a.ladder = b->d_ladder;
    a.bonds = R.c->dev;
    a.nb = R.c->nb;
    a.N = b->N;
    a.A = b->A;
    a.two_s = b->two_s;
    a.steps = R.steps;
    a.reorth = R.reorth;
    a.dim = (I)b->dim;
    a.tol = R.tol;
    a.v0 = R.v0;
    a.buf[0] = (T *)(R.w + R.L.r0);
    a.buf[1] = (T *)(R.w + R.L.r1);
    a.buf[2] = (T *)(R.w + R.L.r2);
    a.V = (T *)(R.w + R.L.V);
    a.states = (uint64_t *)(R.w + R.L.states);
    a.alpha = (double *)(R.w + R.L.alpha);
    a.beta = (double *)(R.w + R.L.beta);
    a.hc = (double *)(R.w + R.L.hcoef);
    a.lz = (LzDev *)(R.w + R.L.lz);
    a.coef = R.psi ? (const double *)(R.w + R.L.coef) : nullptr;
    a.psi = R.psi;
    const size_t lds = ((prefix_bytes(b) + 15) / 16) * 16 + (b->two_s + 2) * sizeof(double);
    hipLaunchKernelGGL((lanczos_small_kernel<T, I, B>), dim3(1), dim3(kSmallBlock), lds, R.st,
                       a);
}

template <typename T, int B>
static void launch_table_b(const Run &R, int steps) {
    const Basis *b = R.b;
    TableArgs<T> a{};
    a.prefix = (const uint32_t *)b->d_prefix;
    a.ladder = b->d_ladder;
    a.bonds = R.c->dev;
    a.nb = R.c->nb;
    a.N = b->N;
    a.A = b->A;
    a.two_s = b->two_s;
    a.steps = steps;
    a.reorth = R.reorth;
    a.n = (int)b->dim;
    a.halfK = R.halfK;
    a.normed = R.normed;
    a.tol = R.tol;
    a.shift = R.c->diag_shift;
    a.v0 = R.v0;
    a.V = (T *)(R.w + R.L.V);
    a.mtgt = (uint16_t *)(R.w + R.L.mtgt);
    a.mcf = (T *)(R.w + R.L.mcf);
    if (steps < R.steps) {
        T *buf[3] = {(T *)(R.w + R.L.r0), (T *)(R.w + R.L.r1), (T *)(R.w + R.L.r2)};
        a.r = buf[steps % 3];
        a.rprev = buf[(steps + 2) % 3];
    }
    a.alpha = (double *)(R.w + R.L.alpha);
    a.beta = (double *)(R.w + R.L.beta);
    a.sigma = (double *)(R.w + R.L.sigma);
    a.cprev = (double *)(R.w + R.L.cprev);
    a.scale = (double *)(R.w + R.L.scale);
    a.lz = (LzDev *)(R.w + R.L.lz);
    a.coef = R.psi ? (const double *)(R.w + R.L.coef) : nullptr;
    a.psi = R.psi;
    const size_t pre = ((prefix_bytes(b) + 15) / 16) * 16 + (b->two_s + 2) * sizeof(double);
    const size_t lds = std::max(pre, 2 * sizeof(T) * (size_t)b->dim);
    hipLaunchKernelGGL((lanczos_table_kernel<T, B>), dim3(1), dim3(kSmallBlock), lds, R.st, a);
}

// Bases that lanczos_table_kernel takes: the prefix table, the vectors and the
// coefficients fit the 64 KB of LDS that a launch has without asking for more.
static bool table_fits(const Basis *b) {
    return b->dim <= kTableRows && b->idx32 && prefix_bytes(b) <= 48 * 1024;
}

// The first `steps` steps of a run.
template <typename T>
static int launch_table(const Run &R, int steps) {
    switch (R.b->bits) {
        case 1: launch_table_b<T, 1>(R, steps); break;
        case 2: launch_table_b<T, 2>(R, steps); break;
        case 3: launch_table_b<T, 3>(R, steps); break;
        case 4: launch_table_b<T, 4>(R, steps); break;
        case 5: launch_table_b<T, 5>(R, steps); break;
        case 6: launch_table_b<T, 6>(R, steps); break;
        case 7: launch_table_b<T, 7>(R, steps); break;
        case 8: launch_table_b<T, 8>(R, steps); break;
        default: return fail(HM_ERANGE, "bits per digit %d unsupported", R.b->bits);
    }
    HM_HIP(hipGetLastError());
    return HM_OK;
}

template <typename T>
static int launch_small(const Run &R) {
    HM_TRY(check_lds(R.b));
    if (table_fits(R.b) && (!R.reorth || R.steps <= kTableCoefs))
        return launch_table<T>(R, R.steps);
    if (!R.b->idx32) return fail(HM_ERANGE, "the one-workgroup run needs 32-bit prefix tables");
    switch (R.b->bits) {
        case 1: launch_small_b<T, uint32_t, 1>(R); break;
        case 2: launch_small_b<T, uint32_t, 2>(R); break;
        case 3: launch_small_b<T, uint32_t, 3>(R); break;
        case 4: launch_small_b<T, uint32_t, 4>(R); break;
        case 5: launch_small_b<T, uint32_t, 5>(R); break;
        case 6: launch_small_b<T, uint32_t, 6>(R); break;
        case 7: launch_small_b<T, uint32_t, 7>(R); break;
        case 8: launch_small_b<T, uint32_t, 8>(R); break;
        default: return fail(HM_ERANGE, "bits per digit %d unsupported", R.b->bits);
    }
    HM_HIP(hipGetLastError());
    return HM_OK;
}

// The instantiated graph of the whole step loop for this run.  A capture
// bakes in the kernels and every argument of the step loop: the coupling list
// (by its serial number), the workspace address, the number of steps, the
// precision, reorthogonalization, the H x kernel and the ground-state output
// (the recompute pass), and through the basis handle its schedule and tables.
// The start vector, the breakdown tolerance and the recompute coefficients
// are not part of it: the initialization runs before the graph and leaves
// them in the workspace.  A handle keeps kGraphCacheEntries graphs, least
// recently used first out.
template <typename T>
static int step_graph(Run &R, hipGraphExec_t *out) {
    Basis *b = R.b;
    const std::vector<uint64_t> key = {R.c->serial, (uint64_t)(uintptr_t)R.w,
                                       (uint64_t)R.steps, (uint64_t)R.prec, (uint64_t)R.reorth,
                                       (uint64_t)R.kernel, (uint64_t)(uintptr_t)R.psi,
                                       (uint64_t)R.table, (uint64_t)sizeof(T)};
    {
        std::lock_guard<std::mutex> lock(b->mu);
        for (auto it = b->graphs.begin(); it != b->graphs.end(); ++it)
            if (it->key == key) {
                b->graphs.splice(b->graphs.begin(), b->graphs, it);
                *out = b->graphs.front().exec;
                return HM_OK;
            }
    }
    hipGraph_t graph = nullptr;
    HM_HIP(hipStreamBeginCapture(R.st, hipStreamCaptureModeThreadLocal));
    const int rc = enqueue_steps<T>(R, R.table, R.steps, nullptr);
    hipError_t e = hipStreamEndCapture(R.st, &graph);
    if (rc != HM_OK) {
        if (graph) (void)hipGraphDestroy(graph);
        return rc;
    }
    if (e != hipSuccess) return fail(HM_EDEVICE, "graph capture: %s", hipGetErrorString(e));
    hipGraphExec_t exec = nullptr;
    e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) return fail(HM_EDEVICE, "graph instantiation: %s", hipGetErrorString(e));
    std::lock_guard<std::mutex> lock(b->mu);
    while (b->graphs.size() >= kGraphCacheEntries) {
        // no launch of it can be pending when it is dropped: the run that
        // used it synchronized its stream before returning
        if (b->graphs.back().exec) (void)hipGraphExecDestroy(b->graphs.back().exec);
        b->graphs.pop_back();
    }
    b->graphs.push_front(Basis::Graph{key, exec});
    *out = exec;
    return HM_OK;
}

template <typename T>
static int run_lanczos(Run &R, double *alpha_h, double *beta_h, int *steps_done) {
    Basis *b = R.b;
    const int64_t n = b->dim;
    LzDev *lz = (LzDev *)(R.w + R.L.lz);
    double *partial = (double *)(R.w + R.L.partial);
    double *sigma = (double *)(R.w + R.L.sigma), *cprev = (double *)(R.w + R.L.cprev);
    T *r0 = (T *)(R.w + R.L.r0);
    const int G = R.L.grid_vec;
    if (R.psi) {
        HM_HIP(hipMemcpyAsync(R.w + R.L.coef, R.coef_host, sizeof(double) * R.steps,
                              hipMemcpyHostToDevice, R.st));
    }
    if (R.small) {
        HM_TRY(launch_small<T>(R));
        return collect(R, alpha_h, beta_h, steps_done);
    }
    if (R.table) {
        HM_TRY(launch_table<T>(R, R.table));
    } else {
        hipLaunchKernelGGL(sumsq_kernel<double>, dim3(G), dim3(kBlock), 0, R.st, R.v0, n, partial);
        hipLaunchKernelGGL(init_write<T>, dim3(G), dim3(kBlock), 0, R.st, R.v0, r0, n, lz, partial,
                           G, sigma, cprev, (double *)(R.w + R.L.scale), R.tol);
        HM_HIP(hipGetLastError());
    }

    const bool timing = g_timing;
    // timing events, destroyed on every return path
    struct Events {
        std::vector<hipEvent_t> e;
        ~Events() {
            for (hipEvent_t x : e)
                if (x) (void)hipEventDestroy(x);
        }
    } evs;
    std::vector<hipEvent_t> ev;
    hipEvent_t lo = nullptr, hi = nullptr;
    if (timing) {
        evs.e.assign(2 * (size_t)R.steps + 2, nullptr);
        for (auto &e : evs.e) HM_HIP(hipEventCreate(&e));
        ev.assign(evs.e.begin(), evs.e.begin() + 2 * (size_t)R.steps);
        lo = evs.e[2 * (size_t)R.steps];
        hi = evs.e[2 * (size_t)R.steps + 1];
        HM_HIP(hipEventRecord(lo, R.st));
    }
    int rc = HM_OK;
    if (R.use_graph && !timing) {
        // the step loop as one graph, captured and instantiated on the first
        // call with this key and replayed by later calls
        hipGraphExec_t exec = nullptr;
        HM_TRY(step_graph<T>(R, &exec));
        HM_HIP(hipGraphLaunch(exec, R.st));
    } else {
        rc = enqueue_steps<T>(R, R.table, R.steps, timing ? &ev : nullptr);
        if (rc != HM_OK) return rc;
    }
    if (R.psi) {
        hipLaunchKernelGGL(sumsq_kernel<double>, dim3(G), dim3(kBlock), 0, R.st, R.psi, n,
                           partial);
        hipLaunchKernelGGL(scale_psi, dim3(G), dim3(kBlock), 0, R.st, R.psi, n, lz, partial, G);
    }
    if (timing) HM_HIP(hipEventRecord(hi, R.st));
    HM_TRY(collect(R, alpha_h, beta_h, steps_done));
    const int done = *steps_done;
    if (timing) {
        double hx = 0.0;
        for (int k = 0; k < done; ++k) {
            float ms = 0.f;
            HM_HIP(hipEventElapsedTime(&ms, ev[2 * k], ev[2 * k + 1]));
            hx += ms;
        }
        float loop = 0.f;
        HM_HIP(hipEventElapsedTime(&loop, lo, hi));
        g_hx_ms = hx;
        g_hx_launches = done;
        g_loop_ms = loop;
    }
    return HM_OK;
}

static int check_opts(const Basis *b, const hm_lanczos_opts *o) {
    if (!o) return fail(HM_EINVAL, "opts is null");
    if (o->precision != HM_PREC_F64 && o->precision != HM_PREC_F32_MIXED)
        return fail(HM_EINVAL, "unknown precision %d", o->precision);
    if (o->kernel < 0 || o->kernel > 3) return fail(HM_EINVAL, "unknown kernel %d", o->kernel);
    if (o->kernel == 3 && b->dim > kSmallMaxDim)
        return fail(HM_ERANGE, "the one-workgroup run takes at most %lld rows",
                    (long long)kSmallMaxDim);
    if (o->kernel != 3 && choose_kernel(b, nullptr, o->kernel, HM_F64, false) < 0)
        return fail(HM_EINVAL, "spin-1/2 block kernel not applicable to this basis");
    return HM_OK;
}

// Steps that the automatic choice gives to lanczos_table_kernel: a number that
// does not depend on the length of the run, so that the recompute pass of a run
// that stopped early takes the same kernels.  Without reorthogonalization only
// the smallest runs: beyond convergence such a run amplifies its roundings (1e-16
// to 1e-8 of the ground state in 200 steps), so from kSmallWork row-bonds on its
// sums keep the order of the multi-kernel step (924 rows, FP64: 14 us a step with
// 24 bonds; with 12 bonds, in one workgroup, 4.6).
constexpr int64_t kSmallWork = 16384;
static int table_steps(const Basis *b, int64_t work, const hm_lanczos_opts *o) {
    const int64_t es = o->precision == HM_PREC_F64 ? 8 : 4;
    if (!table_fits(b)) return 0;
    if (!o->full_reorth) return work <= kSmallWork ? INT32_MAX : 0;
    if (work * es > kTableBytes) return 0;
    return (int)std::min<int64_t>(kTableCoefs, kTableBytes / (b->dim * es));
}

static int run_common(hm_basis h, const double *J, const double *d_v0, int32_t steps,
                      const hm_lanczos_opts *o, void *d_work, size_t work_bytes,
                      const double *coef, double *d_psi, double *alpha, double *beta,
                      int32_t *steps_done, void *stream) {
    if (!h || !d_v0 || !d_work || !steps_done) return fail(HM_EINVAL, "null argument");
    if (steps < 1) return fail(HM_EINVAL, "steps must be >= 1");
    Basis *b = &h->impl;
    HM_TRY(check_opts(b, o));
    CouplingsRef cref;
    HM_TRY(get_couplings(b, J, &cref));
    const Couplings *c = cref.get();
    const int64_t work = b->dim * (int64_t)std::max(c->nb, 1);
    const int table = o->kernel == 0 && !g_timing ? table_steps(b, work, o) : 0;
    const bool small = o->kernel == 3 || table >= steps;
    const int dtype = o->precision == HM_PREC_F64 ? HM_F64 : HM_F32;
    int kernel = small ? 1 : choose_kernel(b, c, o->kernel, dtype, !o->full_reorth);
    if (kernel < 0) return fail(HM_ERANGE, "block kernel tables too large for these couplings");
    int prc = prepare_kernel(b, c, dtype, kernel);
    if (prc == HM_ENOMEM &&
        (kernel == kKernelStaged || kernel == kKernelWg || kernel == kKernelWgItems)) {
        kernel = 2;                   // the handle's split, the same tables asked for by number
        clear_error();
        (void)hipGetLastError();
        prc = prepare_kernel(b, c, dtype, kernel);
    }
    if (prc == HM_ENOMEM && kernel != 2) {
        kernel = 1;                   // the kernel without tables
        clear_error();
        (void)hipGetLastError();
    } else {
        HM_TRY(prc);
    }
    Run R{};
    R.small = small ? 1 : 0;
    R.table = small ? 0 : table;
    // the roundings of the run asked for by number; with reorthogonalization those
    // of the step that the run goes on with
    R.normed = o->kernel == 3 || !o->full_reorth;
    if (table > 0 && o->full_reorth && half_supported(b)) {
        std::lock_guard<std::mutex> lock(b->mu);
        b->table_used = true;
        R.halfK = half_low_bits(b);
    }
    R.b = b;
    R.c = c;
    R.steps = steps;
    R.prec = o->precision;
    R.reorth = o->full_reorth ? 1 : 0;
    R.kernel = kernel;
    R.use_graph = o->use_graph ? 1 : 0;
    R.tol = o->breakdown_tol > 0 ? o->breakdown_tol
                                 : (R.prec == HM_PREC_F64 ? 1e-12 : 1e-6);
    R.L = layout(b, steps, R.prec, R.reorth);
    if (work_bytes < R.L.total)
        return fail(HM_EWORKSPACE, "workspace %zu bytes < required %zu", work_bytes, R.L.total);
    R.w = (unsigned char *)d_work;
    R.v0 = d_v0;
    R.coef_host = coef;
    R.psi = d_psi;
    hipStream_t st = (hipStream_t)stream;
    hipStream_t own = nullptr;
    if (R.use_graph && st == nullptr) {
        // the null stream cannot be captured; a blocking stream orders
        // itself after earlier null-stream work
        HM_HIP(hipStreamCreate(&own));
        st = own;
    }
    R.st = st;
    int done = 0;
    int rc = R.prec == HM_PREC_F64 ? run_lanczos<double>(R, alpha, beta, &done)
                                   : run_lanczos<float>(R, alpha, beta, &done);
    if (own) (void)hipStreamDestroy(own);
    if (rc != HM_OK) return rc;
    *steps_done = done;
    return HM_OK;
}

// Lowest eigenvalue of the symmetric tridiagonal T by bisection on the Sturm
// count, then its eigenvector by inverse iteration.
static int sturm_count(int k, const double *a, const double *b, double x) {
    int neg = 0;
    double q = 1.0;
    for (int i = 0; i < k; ++i) {
        const double bb = i > 0 ? b[i - 1] * b[i - 1] : 0.0;
        q = (a[i] - x) - (i > 0 ? bb / q : 0.0);
        if (q == 0.0) q = -1e-300;
        if (q < 0.0) ++neg;
    }
    return neg;
}

static double lowest_eigenvalue(int k, const double *a, const double *b) {
    double lo = 1e300, hi = -1e300;
    for (int i = 0; i < k; ++i) {
        const double r = (i > 0 ? std::fabs(b[i - 1]) : 0.0) + (i + 1 < k ? std::fabs(b[i]) : 0.0);
        lo = std::min(lo, a[i] - r);
        hi = std::max(hi, a[i] + r);
    }
    const double span = std::max(std::fabs(lo), std::fabs(hi));
    lo -= 1e-12 * span + 1e-300;
    hi += 1e-12 * span + 1e-300;
    for (int it = 0; it < 2000; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (mid <= lo || mid >= hi) break;
        if (sturm_count(k, a, b, mid) >= 1) hi = mid;
        else lo = mid;
    }
    return 0.5 * (lo + hi);
}

static void inverse_iteration(int k, const double *a, const double *b, double lam,
                              double *x) {
    // LU of (T - lam I) with partial pivoting for a tridiagonal matrix.
    double norm = 0.0;
    for (int i = 0; i < k; ++i)
        norm = std::max(norm, std::fabs(a[i]) + (i > 0 ? std::fabs(b[i - 1]) : 0.0) +
                                  (i + 1 < k ? std::fabs(b[i]) : 0.0));
    const double tiny = std::max(norm, 1e-300) * 1e-15;
    std::vector<double> d(k), du(k), du2(k), dl(k);
    std::vector<int> piv(k);
    for (int i = 0; i < k; ++i) {
        d[i] = a[i] - lam;
        du[i] = i + 1 < k ? b[i] : 0.0;
        dl[i] = i + 1 < k ? b[i] : 0.0;
        du2[i] = 0.0;
    }
    for (int i = 0; i + 1 < k; ++i) {
        if (std::fabs(d[i]) >= std::fabs(dl[i])) {
            piv[i] = 0;
            if (d[i] == 0.0) d[i] = tiny;
            const double f = dl[i] / d[i];
            dl[i] = f;
            d[i + 1] -= f * du[i];
        } else {
            piv[i] = 1;
            const double f = d[i] / dl[i];
            d[i] = dl[i];
            dl[i] = f;
            const double t = du[i];
            du[i] = d[i + 1];
            d[i + 1] = t - f * d[i + 1];
            if (i + 2 < k) {
                du2[i] = du[i + 1];
                du[i + 1] = -f * du[i + 1];
            }
        }
    }
    for (int i = 0; i < k; ++i)
        if (std::fabs(d[i]) < tiny) d[i] = d[i] < 0 ? -tiny : tiny;
    for (int i = 0; i < k; ++i) x[i] = 1.0 / std::sqrt((double)k) * (1.0 + 0.01 * ((i * 7919) % 13));
    for (int rep = 0; rep < 3; ++rep) {
        // forward: apply L^{-1} with the recorded row swaps
        for (int i = 0; i + 1 < k; ++i) {
            if (piv[i] == 0) {
                x[i + 1] -= dl[i] * x[i];
            } else {
                const double t = x[i];
                x[i] = x[i + 1];
                x[i + 1] = t - dl[i] * x[i + 1];
            }
        }
        // backward: U x = y
        for (int i = k - 1; i >= 0; --i) {
            double s = x[i];
            if (i + 1 < k) s -= du[i] * x[i + 1];
            if (i + 2 < k) s -= du2[i] * x[i + 2];
            x[i] = s / d[i];
        }
        double nrm = 0.0;
        for (int i = 0; i < k; ++i) nrm += x[i] * x[i];
        nrm = std::sqrt(nrm);
        for (int i = 0; i < k; ++i) x[i] /= nrm;
    }
    int first = 0;
    while (first < k && std::fabs(x[first]) < 1e-300) ++first;
    if (first < k && x[first] < 0)
        for (int i = 0; i < k; ++i) x[i] = -x[i];
}

}  // namespace hm

using hm::fail;

extern "C" {

int hm_tridiag_lowest(int32_t k, const double *alpha, const double *beta, double *eval,
                      double *evec) {
    hm::clear_error();
    if (k < 1 || !alpha || !eval || (k > 1 && !beta)) return fail(HM_EINVAL, "bad arguments");
    for (int i = 0; i < k; ++i)
        if (!std::isfinite(alpha[i]) || (i + 1 < k && !std::isfinite(beta[i])))
            return fail(HM_EINVAL, "non-finite tridiagonal entry");
    const double lam = hm::lowest_eigenvalue(k, alpha, beta);
    *eval = lam;
    if (evec) {
        if (k == 1) evec[0] = 1.0;
        else hm::inverse_iteration(k, alpha, beta, lam, evec);
    }
    return HM_OK;
}

int hm_lanczos_workspace(hm_basis h, int32_t steps, const hm_lanczos_opts *o, size_t *bytes) {
    hm::clear_error();
    if (!h || !bytes) return fail(HM_EINVAL, "null argument");
    if (steps < 1) return fail(HM_EINVAL, "steps must be >= 1");
    HM_TRY(hm::check_opts(&h->impl, o));
    *bytes = hm::layout(&h->impl, steps, o->precision, o->full_reorth ? 1 : 0).total;
    return HM_OK;
}

int hm_lanczos(hm_basis h, const double *J, const double *d_v0, int32_t steps,
               const hm_lanczos_opts *o, void *d_work, size_t work_bytes, double *alpha,
               double *beta, double *E0, int32_t *steps_done, void *stream) {
    hm::clear_error();
    if (!alpha || !beta || !E0) return fail(HM_EINVAL, "null output");
    int done = 0;
    HM_TRY(hm::run_common(h, J, d_v0, steps, o, d_work, work_bytes, nullptr, nullptr, alpha,
                          beta, &done, stream));
    *steps_done = done;
    return hm_tridiag_lowest(done, alpha, beta, E0, nullptr);
}

int hm_lanczos_ritz(hm_basis h, const double *J, const double *d_v0, int32_t steps_done,
                    const double *c, const hm_lanczos_opts *o, void *d_work,
                    size_t work_bytes, double *d_psi, double *alpha_out, double *beta_out,
                    void *stream) {
    hm::clear_error();
    if (!c || !d_psi) return fail(HM_EINVAL, "null argument");
    int done = 0;
    HM_TRY(hm::run_common(h, J, d_v0, steps_done, o, d_work, work_bytes, c, d_psi, alpha_out,
                          beta_out, &done, stream));
    if (done != steps_done)
        return fail(HM_EINVAL, "recompute stopped after %d of %d steps", done, steps_done);
    return HM_OK;
}

int hm_set_timing(int32_t enable) {
    hm::g_timing = enable != 0;
    return HM_OK;
}

int hm_last_timing(double *hx_ms, int32_t *hx_launches, double *loop_ms) {
    if (hx_ms) *hx_ms = hm::g_hx_ms;
    if (hx_launches) *hx_launches = hm::g_hx_launches;
    if (loop_ms) *loop_ms = hm::g_loop_ms;
    return HM_OK;
}

}  // extern "C"
