// Block Lanczos on H(M): several lowest eigenpairs at once, degenerate ones
// included, from p start vectors (the multi-vector product H X the batched
// path uses, here in FP64 on one instance).
//
// The paper's recurrence is the single-vector Lanczos method (Secs. 1, 4); its
// block form replaces the scalars alpha_k, beta_k by p x p blocks:
//   V_0 R_0 = X0                      (QR of the start block)
//   W = H V_k - V_{k-1} B_{k-1}^T;   A_k = V_k^T W
//   twice:  W -= sum_{j<=k} V_j (V_j^T W)      (full reorthogonalization; the
//                                               first pass subtracts V_k A_k)
//   V_{k+1} B_k = W                   (QR; B_k upper triangular)
// and the eigenvalues of the block tridiagonal matrix with diagonal blocks
// A_k and sub-diagonal blocks B_k approximate the lowest eigenvalues of H.
//
// Blocks are stored row-interleaved, [dim][p] FP64, so one decode of a basis
// state serves all p columns and a gathered row is p contiguous doubles.  The
// QR is Cholesky QR applied twice (the second pass restores orthogonality to
// rounding level).  Block dot products V^T W run on the matrix cores
// (tall_dots.h) as per-workgroup partials summed in a fixed order, so a run is
// reproducible.  The p x p factorizations, the breakdown test and the blocks
// A_k, B_k stay on the device: a step is 13 launches that the host enqueues
// ahead, where reading each set of dots back cost 5 round trips a step.
#include <algorithm>
#include <cstring>
#include <vector>

#include "device_common.h"
#include "hm_internal.h"
#include "hx_row.h"
#include "tall_dots.h"

namespace hm {

// Device state of one run: nothing is read back before the end, so the host
// only enqueues.
struct BlockDev {
    int stopped;      // steps done when the block Krylov space was exhausted,
                      // -1 if the start block is rank deficient, 0 while running
    double scale;     // running max |entry| of the A and B blocks
};

template <int P>
__device__ __forceinline__ void load_drow(const double *__restrict__ p, double (&v)[P]) {
    if constexpr (P % 2 == 0) {
#pragma unroll
        for (int q = 0; q < P / 2; ++q) {
            const double2 t = reinterpret_cast<const double2 *>(p)[q];
            v[2 * q] = t.x;
            v[2 * q + 1] = t.y;
        }
    } else {
        v[0] = p[0];
    }
}

template <int P>
__device__ __forceinline__ void store_drow(double *__restrict__ p, const double (&v)[P]) {
    if constexpr (P % 2 == 0) {
#pragma unroll
        for (int q = 0; q < P / 2; ++q)
            reinterpret_cast<double2 *>(p)[q] = make_double2(v[2 * q], v[2 * q + 1]);
    } else {
        p[0] = v[0];
    }
}

// Moves whose gathers are in flight together in one row of H X: as many as
// the registers hold rows of P doubles.
template <int P> constexpr int block_moves() { return P <= 4 ? 8 : 16 / P * 2; }

// W = H X - Xprev B^T for [dim][P] blocks (generic digits, any s; Xprev may be
// null).  The moves of a row go in batches: the targets and gathers of a
// batch are issued before its products are added, in bond order.  With s = 1/2
// a bond has at most one move.  Folding the previous block's update in saves a
// launch and two passes over W.
template <typename I, int B, int P>
__global__ __launch_bounds__(kBlock) void block_hx_kernel(
    const I *__restrict__ gprefix, const double *__restrict__ gladder,
    const BondDev *__restrict__ bonds, int nb, int N, int A, int two_s, I dim,
    const double *__restrict__ X, const double *__restrict__ Xprev,
    const double *__restrict__ Bm, double *__restrict__ Y, const BlockDev *__restrict__ dev) {
    if (dev->stopped) return;
    extern __shared__ __align__(16) unsigned char smem[];
    const int plen = N * (A + 1) * (two_s + 1);
    I *Pt = reinterpret_cast<I *>(smem);
    double *F = reinterpret_cast<double *>(smem + ((plen * sizeof(I) + 15) / 16) * 16);
    for (int t = threadIdx.x; t < plen; t += blockDim.x) Pt[t] = gprefix[t];
    for (int t = threadIdx.x; t < two_s + 2; t += blockDim.x) F[t] = gladder[t];
    __syncthreads();
    const Prefix<I> pv{Pt, A + 1, two_s + 1};
    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    I first, last;
    block_rows<I>(lb, gridDim.x, dim, first, last);
    constexpr int kPer = B == 1 ? 1 : 2;                  // moves of one bond
    constexpr int kBatch = block_moves<P>() / kPer;       // bonds of a batch
    for (I row = first + threadIdx.x; row < last; row += blockDim.x) {
        const uint64_t st = unrank_state<I, B>(row, pv, N, A, two_s);
        double xi[P], acc[P];
        load_drow<P>(X + (size_t)row * P, xi);
        double diag = 0.0;
#pragma unroll
        for (int q = 0; q < P; ++q) acc[q] = 0.0;
        for (int b0 = 0; b0 < nb; b0 += kBatch) {
            double xj[kBatch * kPer][P], cf[kBatch * kPer];
            bool on[kBatch * kPer];
#pragma unroll
            for (int t = 0; t < kBatch; ++t) {
#pragma unroll
                for (int m = 0; m < kPer; ++m) on[kPer * t + m] = false;
                const int b = b0 + t;
                if (b >= nb) continue;
                const int u = bonds[b].u, v = bonds[b].v;
                const double mJ2 = bonds[b].mJ2;
                const int au = digit_at<B>(st, u), av = digit_at<B>(st, v);
                diag += bonds[b].mJ4 * (double)((two_s - 2 * au) * (two_s - 2 * av));
                if constexpr (B == 1) {
                    if (au != av) {                       // s = 1/2: F[1] = 1
                        const I j = row + move_delta<I, B>(st, u, v, au ? -1 : +1, pv);
                        cf[t] = mJ2;
                        load_drow<P>(X + (size_t)j * P, xj[t]);
                        on[t] = true;
                    }
                } else {
                    if (au >= 1 && av < two_s) {
                        const I j = row + move_delta<I, B>(st, u, v, -1, pv);
                        cf[2 * t] = mJ2 * F[au] * F[av + 1];
                        load_drow<P>(X + (size_t)j * P, xj[2 * t]);
                        on[2 * t] = true;
                    }
                    if (av >= 1 && au < two_s) {
                        const I j = row + move_delta<I, B>(st, u, v, +1, pv);
                        cf[2 * t + 1] = mJ2 * F[av] * F[au + 1];
                        load_drow<P>(X + (size_t)j * P, xj[2 * t + 1]);
                        on[2 * t + 1] = true;
                    }
                }
            }
#pragma unroll
            for (int m = 0; m < kBatch * kPer; ++m)
                if (on[m])
#pragma unroll
                    for (int q = 0; q < P; ++q) acc[q] += cf[m] * xj[m][q];
        }
#pragma unroll
        for (int q = 0; q < P; ++q) acc[q] += diag * xi[q];
        if (Xprev) {
            load_drow<P>(Xprev + (size_t)row * P, xi);
#pragma unroll
            for (int r = 0; r < P; ++r)
#pragma unroll
                for (int c = 0; c < P; ++c) acc[c] -= xi[r] * Bm[c * P + r];
        }
        store_drow<P>(Y + (size_t)row * P, acc);
    }
}

// out[o] = sum over the row ranges of partial[.][o].
__global__ __launch_bounds__(kTallBlock) void block_dots_finish(
    const double *__restrict__ partial, int splits, int nout, double *__restrict__ out,
    const BlockDev *__restrict__ dev) {
    if (dev->stopped) return;
    __shared__ double red[4][64];
    tall_sum(partial, splits, nout, blockIdx.x * 64, out, red);
}

// W[row][c] -= sum_{j < nblk} sum_r X_j[row][r] M_j[r][c].  In the first pass
// of the reorthogonalization (Aout given) the last block of M is V_k^T W: its
// symmetric part is A_k, which one workgroup writes.
template <int P>
__global__ __launch_bounds__(kBlock) void block_update_kernel(
    const double *__restrict__ X, const double *__restrict__ M, int nblk, int64_t dim,
    double *__restrict__ W, double *__restrict__ Aout, BlockDev *__restrict__ dev) {
    if (dev->stopped) return;
    for (int64_t row = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; row < dim;
         row += (int64_t)gridDim.x * blockDim.x) {
        double w[P];
        load_drow<P>(W + row * P, w);
        for (int j = 0; j < nblk; ++j) {
            double x[P];
            load_drow<P>(X + ((size_t)j * dim + row) * P, x);
            const double *__restrict__ Mj = M + (size_t)j * P * P;
#pragma unroll
            for (int r = 0; r < P; ++r)
#pragma unroll
                for (int c = 0; c < P; ++c) w[c] -= x[r] * Mj[r * P + c];
        }
        store_drow<P>(W + row * P, w);
    }
    if (Aout && blockIdx.x == 0) {
        const double *__restrict__ A = M + (size_t)(nblk - 1) * P * P;
        for (int t = threadIdx.x; t < P * P; t += blockDim.x)
            Aout[t] = 0.5 * (A[t] + A[(t % P) * P + t / P]);
        if (threadIdx.x == 0) {
            double sc = dev->scale;
            for (int t = 0; t < P * P; ++t)
                sc = fmax(sc, fabs(0.5 * (A[t] + A[(t % P) * P + t / P])));
            dev->scale = sc;
        }
    }
}

// One workgroup: G = W^T W from its partials, symmetrized, and its upper
// Cholesky factor R (G = R^T R) in LDS, P rows of eliminations by P x P
// threads.  pass 0 stops the run when W is at rounding level of the
// recurrence's scale or numerically rank deficient (a pivot not above tol
// times the largest diagonal entry); pass 1 also writes R2 R1 to Rout.  k < 0:
// the start block, where stopping is the caller's error.
template <int P>
__global__ __launch_bounds__(kTallBlock) void block_cholesky_kernel(
    const double *__restrict__ partial, int splits, double *__restrict__ G,
    double *__restrict__ R, const double *__restrict__ R1, int pass, int k,
    double *__restrict__ Rout, BlockDev *__restrict__ dev) {
    if (dev->stopped) return;
    constexpr int PP = P * P;
    __shared__ double red[4][64];
    __shared__ double a[PP], r[PP];
    __shared__ int bad;
    for (int f = 0; f < PP; f += 64) tall_sum(partial, splits, PP, f, G, red);
    __syncthreads();
    const int t = threadIdx.x, ti = t / P, tj = t % P;
    if (t < PP) {
        a[t] = ti == tj ? G[t] : 0.5 * (G[t] + G[tj * P + ti]);
        r[t] = 0.0;
    }
    if (t == 0) bad = 0;
    __syncthreads();
    double dmax = 0.0;
    for (int i = 0; i < P; ++i) dmax = fmax(dmax, a[i * P + i]);
    const double floor1 = k < 0 ? 0.0 : 1e-12 * dev->scale;
    const double tol = pass == 0 ? 1e-12 : 1e-14;
    if (t == 0 && (!(dmax > 0.0) || (pass == 0 && !(dmax > floor1 * floor1)))) bad = 1;
    for (int i = 0; i < P; ++i) {
        __syncthreads();
        const double d = a[i * P + i];
        if (t == 0 && !(d > tol * dmax)) bad = 1;
        const double rii = sqrt(d);
        if (t < PP && ti == i && tj >= i) r[t] = tj == i ? rii : a[t] / rii;
        __syncthreads();
        if (t < PP && ti > i && tj >= ti) a[t] -= r[i * P + ti] * r[i * P + tj];
    }
    __syncthreads();
    if (bad) {
        if (t == 0) dev->stopped = k + 1 > 0 ? k + 1 : -1;
        return;
    }
    if (t < PP) R[t] = r[t];
    if (pass == 1 && Rout) {
        double s = 0.0;
        if (t < PP) {
            for (int q = 0; q < P; ++q) s += r[ti * P + q] * R1[q * P + tj];
            Rout[t] = s;
            a[t] = fabs(s);
        }
        __syncthreads();
        if (t == 0) {
            double sc = dev->scale;
            for (int q = 0; q < PP; ++q) sc = fmax(sc, a[q]);
            dev->scale = sc;
        }
    }
}

// W[row] <- W[row] R^{-1} for the upper triangular R (row-vector solve)
template <int P>
__global__ __launch_bounds__(kBlock) void block_trsm_kernel(const double *__restrict__ R,
                                                            int64_t dim, double *__restrict__ W,
                                                            const BlockDev *__restrict__ dev) {
    if (dev->stopped) return;
    for (int64_t row = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; row < dim;
         row += (int64_t)gridDim.x * blockDim.x) {
        double w[P];
        load_drow<P>(W + row * P, w);
#pragma unroll
        for (int c = 0; c < P; ++c) {
            double v = w[c];
#pragma unroll
            for (int r = 0; r < c; ++r) v -= w[r] * R[r * P + c];
            w[c] = v / R[c * P + c];
        }
        store_drow<P>(W + row * P, w);
    }
}

__global__ void block_init(BlockDev *dev) {
    dev->stopped = 0;
    dev->scale = 0.0;
}

struct BlockLayout {
    size_t V, partial, dots, R1, R2, dev, A, B, total;
};

static size_t al256b(size_t x) { return (x + 255) & ~(size_t)255; }

static int block_layout(const Basis *b, int p, int steps, BlockLayout *L) {
    if (p != 1 && p != 2 && p != 4 && p != 8 && p != 16)
        return fail(HM_EINVAL, "block size p must be 1, 2, 4, 8 or 16");
    if (steps < 1) return fail(HM_EINVAL, "steps must be >= 1");
    const size_t blk = (size_t)b->dim * p * sizeof(double), pp = (size_t)p * p;
    size_t off = 0;
    L->V = off; off = al256b(off + blk * (size_t)(steps + 1));
    L->partial = off; off = al256b(off + sizeof(double) * (size_t)(steps + 1) * kTallSplits * pp);
    L->dots = off; off = al256b(off + sizeof(double) * (size_t)(steps + 1) * pp);
    L->R1 = off; off = al256b(off + sizeof(double) * pp);
    L->R2 = off; off = al256b(off + sizeof(double) * pp);
    // the results, read back in one copy
    L->dev = off; off = al256b(off + sizeof(BlockDev));
    L->A = off; off += sizeof(double) * (size_t)steps * pp;
    L->B = off; off += sizeof(double) * (size_t)steps * pp;
    L->total = al256b(off);
    return HM_OK;
}

namespace {

constexpr int kStopCheck = 16;   // steps between two looks at the stop flag

struct BlockRun {
    const Basis *b;
    const Couplings *c;
    int p, steps;
    unsigned char *w;
    BlockLayout L;
    hipStream_t st;
    double *V(int k) const { return (double *)(w + L.V) + (size_t)k * b->dim * p; }
    double *partial() const { return (double *)(w + L.partial); }
    double *dots() const { return (double *)(w + L.dots); }
    double *R(int pass) const { return (double *)(w + (pass == 0 ? L.R1 : L.R2)); }
    BlockDev *dev() const { return (BlockDev *)(w + L.dev); }
    double *A(int k) const { return (double *)(w + L.A) + (size_t)k * p * p; }
    double *B(int k) const { return (double *)(w + L.B) + (size_t)k * p * p; }
};

// Partials of X^T W for nblk blocks of X; returns the number of row ranges.
template <int P>
int dots(const BlockRun &R, const double *X, int nblk, const double *W) {
    const int ncol = nblk * P, splits = tall_splits<P>(R.b->dim, ncol);
    hipLaunchKernelGGL((tall_dots_kernel<double, P>),
                       dim3(splits, (ncol + tall_cols<P>() - 1) / tall_cols<P>()),
                       dim3(kTallBlock), 0, R.st, X, W, (int64_t)R.b->dim, ncol, R.partial(),
                       &R.dev()->stopped, (const double *)nullptr, TallSub<double>{});
    return splits;
}

// Cholesky QR applied twice to W in place (W = Q Rout).
template <int P>
void cholqr2(const BlockRun &R, double *W, int k, double *Rout) {
    for (int pass = 0; pass < 2; ++pass) {
        const int splits = dots<P>(R, W, 1, W);
        hipLaunchKernelGGL((block_cholesky_kernel<P>), dim3(1), dim3(kTallBlock), 0, R.st,
                           R.partial(), splits, R.dots(), R.R(pass), R.R(0), pass, k,
                           pass == 1 ? Rout : nullptr, R.dev());
        hipLaunchKernelGGL((block_trsm_kernel<P>), dim3(generic_grid(R.b->dim)), dim3(kBlock), 0,
                           R.st, R.R(pass), (int64_t)R.b->dim, W, R.dev());
    }
}

template <typename I, int Bb, int P>
int run_block(BlockRun &R, const double *X0, double *Aout, double *Bout, int *done) {
    const Basis *b = R.b;
    const size_t blk = (size_t)b->dim * P * sizeof(double), pp = (size_t)P * P;
    const size_t lds = ((prefix_bytes(b) + 15) / 16) * 16 + (b->two_s + 2) * sizeof(double);
    const int grid = generic_grid(b->dim);
    // V_0 R_0 = X0
    HM_HIP(hipMemcpyAsync(R.V(0), X0, blk, hipMemcpyDeviceToDevice, R.st));
    hipLaunchKernelGGL(block_init, dim3(1), dim3(1), 0, R.st, R.dev());
    cholqr2<P>(R, R.V(0), -1, nullptr);
    for (int k = 0; k < R.steps; ++k) {
        double *W = R.V(k + 1);
        hipLaunchKernelGGL((block_hx_kernel<I, Bb, P>), dim3(grid), dim3(kBlock), lds, R.st,
                           (const I *)b->d_prefix, b->d_ladder, R.c->dev, R.c->nb, b->N, b->A,
                           b->two_s, (I)b->dim, R.V(k), k > 0 ? R.V(k - 1) : (double *)nullptr,
                           k > 0 ? R.B(k - 1) : (double *)nullptr, W, R.dev());
        // twice W -= sum_j V_j (V_j^T W); the first pass's V_k^T W is A_k
        for (int pass = 0; pass < 2; ++pass) {
            const int nout = (k + 1) * P * P, splits = dots<P>(R, R.V(0), k + 1, W);
            hipLaunchKernelGGL(block_dots_finish, dim3((nout + 63) / 64), dim3(kTallBlock), 0,
                               R.st, R.partial(), splits, nout, R.dots(), R.dev());
            hipLaunchKernelGGL((block_update_kernel<P>), dim3(grid), dim3(kBlock), 0, R.st,
                               R.V(0), R.dots(), k + 1, (int64_t)b->dim, W,
                               pass == 0 ? R.A(k) : (double *)nullptr, R.dev());
        }
        if (k + 1 < R.steps) cholqr2<P>(R, W, k, R.B(k));
        HM_HIP(hipGetLastError());
        // a run that has stopped only launches empty kernels: look now and then
        if (k % kStopCheck == kStopCheck - 1 && k + 1 < R.steps) {
            int stopped = 0;
            HM_HIP(hipMemcpyAsync(&stopped, &R.dev()->stopped, sizeof stopped,
                                  hipMemcpyDeviceToHost, R.st));
            HM_HIP(hipStreamSynchronize(R.st));
            if (stopped) break;
        }
    }
    // the state and the blocks in one copy
    const size_t head = R.L.A - R.L.dev;
    std::vector<unsigned char> host(head + 2 * sizeof(double) * R.steps * pp);
    HM_HIP(hipMemcpyAsync(host.data(), R.w + R.L.dev, host.size(), hipMemcpyDeviceToHost, R.st));
    HM_HIP(hipStreamSynchronize(R.st));
    BlockDev dev;
    std::memcpy(&dev, host.data(), sizeof dev);
    if (dev.stopped < 0) return fail(HM_EINVAL, "start block is rank deficient");
    const int n = *done = dev.stopped > 0 ? dev.stopped : R.steps;
    const double *A = (const double *)(host.data() + head), *B = A + (size_t)R.steps * pp;
    std::copy(A, A + n * pp, Aout);
    std::copy(B, B + (n - 1) * pp, Bout);
    return HM_OK;
}

template <typename I, int Bb>
int dispatch_p(BlockRun &R, const double *X0, double *A, double *B, int *done) {
    switch (R.p) {
        case 1: return run_block<I, Bb, 1>(R, X0, A, B, done);
        case 2: return run_block<I, Bb, 2>(R, X0, A, B, done);
        case 4: return run_block<I, Bb, 4>(R, X0, A, B, done);
        case 8: return run_block<I, Bb, 8>(R, X0, A, B, done);
        default: return run_block<I, Bb, 16>(R, X0, A, B, done);
    }
}

template <typename I>
int dispatch_bits(BlockRun &R, const double *X0, double *A, double *B, int *done) {
    switch (R.b->bits) {
        case 1: return dispatch_p<I, 1>(R, X0, A, B, done);
        case 2: return dispatch_p<I, 2>(R, X0, A, B, done);
        case 3: return dispatch_p<I, 3>(R, X0, A, B, done);
        case 4: return dispatch_p<I, 4>(R, X0, A, B, done);
        default: return fail(HM_ERANGE, "block Lanczos supports up to 4 bits per digit");
    }
}

}  // namespace
}  // namespace hm

using hm::fail;

extern "C" {

int hm_block_lanczos_workspace(hm_basis h, int32_t p, int32_t steps, size_t *bytes) {
    hm::clear_error();
    if (!h || !bytes) return fail(HM_EINVAL, "null argument");
    hm::BlockLayout L;
    HM_TRY(hm::block_layout(&h->impl, p, steps, &L));
    *bytes = L.total;
    return HM_OK;
}

int hm_block_lanczos(hm_basis h, const double *J, const double *d_X0, int32_t p, int32_t steps,
                     void *d_work, size_t work_bytes, double *A, double *B, int32_t *steps_done,
                     void *stream) {
    hm::clear_error();
    if (!h || !J || !d_X0 || !d_work || !A || !B || !steps_done)
        return fail(HM_EINVAL, "null argument");
    hm::Basis *b = &h->impl;
    hm::BlockLayout L;
    HM_TRY(hm::block_layout(b, p, steps, &L));
    if (work_bytes < L.total)
        return fail(HM_EWORKSPACE, "workspace %zu bytes < required %zu", work_bytes, L.total);
    if (b->dim < p) return fail(HM_EINVAL, "block size p=%d exceeds the dimension", p);
    HM_TRY(hm::check_lds(b));
    hm::CouplingsRef cref;
    HM_TRY(hm::get_couplings(b, J, &cref));
    const hm::Couplings *c = cref.get();
    std::fill(A, A + (size_t)steps * p * p, 0.0);
    std::fill(B, B + (size_t)steps * p * p, 0.0);
    hm::BlockRun R{b, c, p, steps, (unsigned char *)d_work, L, (hipStream_t)stream};
    int done = 0;
    const int rc = b->idx32 ? hm::dispatch_bits<uint32_t>(R, d_X0, A, B, &done)
                            : hm::dispatch_bits<uint64_t>(R, d_X0, A, B, &done);
    *steps_done = done;
    return rc;
}

}  // extern "C"
