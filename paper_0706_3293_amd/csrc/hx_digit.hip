// Block kernel for the row-gather H x with s >= 1 (Sec. 4, Eq. (E-4-b)).
//
// The generic kernel decodes every row by an N-step digit walk and encodes
// every target by another, so it is bound by vector instructions and the LDS
// latency of the walks (5.2 M rows of the 16-site spin-1 ring, FP32: 250 us,
// 3 % of the copy rate).  Here a state is split into its low K digits L and
// its high N - K digits h.  The basis order is that of the numbers
// sum_u a_u (2s+1)^u, so the rows with one h form a contiguous block, ordered
// like the low words of their digit sum: index = Off(h) + rankL(L).
//   * a bond inside the low word moves within the block: the ranks its two
//     moves lead to are tabulated per low word, the targets are read from the
//     block's copy in LDS;
//   * a bond inside the high word moves all rows of a block to the same rows
//     of another block, so the gathers are coalesced; the target blocks and
//     matrix elements of the moves a high word allows are tabulated per
//     (basis, couplings) in bond order;
//   * a straddling bond takes the target block from one table and the rank
//     from the other.
// A wave takes R blocks of one digit-sum class (the low-word work is done once
// for R rows), copies them to its LDS slice, interleaved, so that one LDS read
// serves the R rows, and goes over them 64 rows at a time.  Every row adds its
// bonds in list order, as row_hx (hx_row.h) does.  In FP32 the diagonal element is
// summed bond by bond with the roundings of row_hx, so that the rows are the
// generic kernel's bit for bit: with equal couplings those roundings are the same
// for many rows and do not average out (coefficients of FP32-mixed runs 1e-8
// apart).  So it is in FP64 with one lane per row up to 2^20 rows; up to 2^19 a run's
// dots are the generic kernel's too, and coefficients past convergence then do not
// depend on the kernel.  In larger FP64 subspaces it is the sum of a low-word part, a high-word
// part (both tabulated) and the straddling bonds (16 sites, s = 1, couplings of
// 1.03: 95 us, bond by bond 140).  Where the type holds all of these sums exactly,
// the tabulated parts give the same.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <vector>

#include "device_common.h"
#include "hm_internal.h"

namespace hm {

int launch_hx_generic(const Basis *b, const Couplings *c, int dtype, const HxPass &p,
                      hipStream_t st);

constexpr int kDigitMaxWords = 16384;        // low words
constexpr size_t kDigitMaxLds = 64 * 1024;   // dynamic; kLzLds scalars more, of the CU's 160 KiB
// Most bytes of tables of one coupling list: a GiB, or what four FP64 vectors take, up
// to 8 GiB.  Sectors far from M = 0 have blocks of a few rows and would hold up to 600
// times the vector (31 sites, s = 1, A = 5, all bonds: 1.1 GB for 2.5 MB) for a product
// that is at most twice as fast (ring of 24 sites, A = 8, 0.44 GB for 45 MB: 224 and 387
// us); four lists of two types may be cached.
constexpr size_t kDigitMaxTables = (size_t)8 << 30, kDigitFreeTables = (size_t)1 << 30;
constexpr int64_t kDigitMaxGrid = 16384;     // workgroups of one launch
constexpr uint32_t kNoBlock = 0xFFFFFFFFu;   // padding slot of a group of blocks

// Up to four bonds with their first site in the low word, consecutive in the
// bond list and all of one kind.
template <typename T>
struct DigitOp {
    int32_t n;           // bonds in use: 1, 2 or 4 (straddling: 1)
    int32_t straddle;    // -1: both sites in the low word, else its slot in the block table
    int32_t first;       // index of the first bond (its table and matrix elements)
    int32_t sv;          // straddling: bit position of the digit in the high word
    T mJ4[4];            // -J/4
};

// Entry of the low-word table for one bond: the ranks of the two moves
// (kRankBits bits each) and an index of the digits.
//   low:         moves a_u - 1, a_v + 1 and the other (the slice's zero entry
//                where the digits do not allow one), index a_u (2s+1) + a_v
//   straddling:  moves a_u - 1 and a_u + 1 (the own rank where the low digit
//                does not allow one), index a_u
constexpr int kRankBits = 12;
constexpr int kDigitMaxSize = (1 << kRankBits) - 1;

// Four moves of a block's high word.
template <typename T, typename I>
struct DigitMoves {
    I off[4];            // first rows of the target blocks
    T cf[4];             // matrix elements
};

// One block: its packed high digits, its first row, the start and size of its
// digit-sum class among the low words, and its number among the blocks of that class.
template <typename I>
struct DigitBlock {
    uint64_t hword;
    I off;
    int32_t cs, size, rank;
};

// Tables of the split that depend on the basis only.
struct DigitTables {
    int K = 0, R = 1, nclass = 0, smax = 0, words = 0;
    int64_t n_blocks = 0, n_groups = 0;
    std::vector<uint16_t> rank;      // low word's rank in its class, by number
    std::vector<uint16_t> word;      // low-word numbers by class start + rank
    std::vector<int32_t> cls;        // [class][2]: start in `word`, size
    void *blocks = nullptr;          // DigitBlock<I> in memory order
    uint32_t *groups = nullptr;      // [n_groups][R] blocks of one class
    uint32_t *rowblk = nullptr;      // block of every row (one lane per row)
    uint16_t *d_rank = nullptr, *d_word = nullptr;   // device copies of rank and word
    void *mem = nullptr;             // the allocation that holds them
};

static void free_digit(void *p) {
    auto *t = (DigitTables *)p;
    if (!t) return;
    if (t->mem) (void)hipFree(t->mem);
    delete t;
}

// Tables of one coupling list in one element type.
struct DigitBonds {
    void *ops = nullptr;             // DigitOp<T>, n_ops of them
    void *cf = nullptr;              // [nF][(2s+1)^2][2] matrix elements of the two moves
    uint32_t *low = nullptr;         // [nF][words] low-word table (class start + rank)
    void *dlow = nullptr;            // [words] diagonal part of the low-word bonds
    void *moves = nullptr;           // [block][mw / 4] DigitMoves<T, I>
    uint32_t *mcnt = nullptr;        // [block] moves the block's high word allows
    void *dhigh = nullptr;           // [block] diagonal part of the high-word bonds
    void *kdiag = nullptr;           // [block][nH] (2 m_u)(2 m_v) of the high-word bonds and
    void *hJ4 = nullptr;             // [nH] their -J/4, where the diagonal goes bond by bond
                                     // (nH padded to fours with zeros)
    void *strad = nullptr;           // [block][nS][2] target blocks of the straddling moves
    int n_ops = 0, nF = 0, nS = 0, nH = 0, mw = 0;   // mw: moves of a row, padded to fours
    void *mem = nullptr;                             // the allocation that holds them
};
struct DigitBondSet {
    DigitBonds by_type[2];
    bool have[2] = {false, false};
    bool seen[2] = {false, false};    // the generic kernel has had the first product
};
static void free_digit_bonds(void *p) {
    auto *s = (DigitBondSet *)p;
    if (!s) return;
    for (auto &b : s->by_type)
        if (b.mem) (void)hipFree(b.mem);
    delete s;
}

template <typename T, typename I>
struct DigitArgs {
    const DigitBlock<I> *blocks;
    const uint32_t *groups;
    const uint32_t *rowblk;          // block of every row (one lane per row)
    const DigitOp<T> *ops;
    const T *cf;
    const uint32_t *low;
    const T *dlow;
    const DigitMoves<T, I> *moves;
    const uint32_t *mcnt;
    const T *dhigh;
    const T *kdiag;
    const T *hJ4;
    const I *strad;
    uint32_t n_groups, run;          // run: consecutive groups of one XCD
    int n_ops, nF, nS, nH, mq, words, smax, two_s, mask;   // mq: move pieces of a row
};

// R consecutive elements of LDS (16-byte reads where they fit).
template <typename T, int R>
__device__ __forceinline__ void lds_row(const T *p, T (&v)[R]) {
    typedef T VR __attribute__((ext_vector_type(R)));
    const VR t = *reinterpret_cast<const VR *>(p);
#pragma unroll
    for (int m = 0; m < R; ++m) v[m] = t[m];
}
template <>
__device__ __forceinline__ void lds_row<float, 1>(const float *p, float (&v)[1]) { v[0] = *p; }
template <>
__device__ __forceinline__ void lds_row<double, 1>(const double *p, double (&v)[1]) { v[0] = *p; }

// (2 m_u)(2 m_v) by the index of the two digits.
template <typename T>
__device__ __forceinline__ void stage_products(T *kt, int two_s) {
    for (int t = threadIdx.x; t < (two_s + 1) * (two_s + 1); t += blockDim.x)
        kt[t] = (T)((two_s - 2 * (t / (two_s + 1))) * (two_s - 2 * (t % (two_s + 1))));
}

// W low-word bonds at once: the table entries, then the R rows' reads and
// products in bond order.  A move that the digits do not allow reads the
// slice's zero entry (its matrix element is zero as well).
template <int W, typename T, int R>
__device__ __forceinline__ void low_bonds(const uint32_t *__restrict__ low, int words, const T *cf,
                                          const T *kt, int WW, const T *xs,
                                          const Const<DigitOp<T>> &op, int q0, bool chain,
                                          T (&diag)[R], T (&off)[R]) {
    constexpr uint32_t kMask = (1u << kRankBits) - 1u;
    uint32_t e[W];
    T x1[W][R], x2[W][R], c[W][2];
#pragma unroll
    for (int q = 0; q < W; ++q) e[q] = low[(size_t)q * words];
#pragma unroll
    for (int q = 0; q < W; ++q) {
        lds_row<T, R>(xs + (e[q] & kMask) * R, x1[q]);
        lds_row<T, R>(xs + ((e[q] >> kRankBits) & kMask) * R, x2[q]);
        lds_row<T, 2>(cf + (q * WW * WW + (int)(e[q] >> (2 * kRankBits))) * 2, c[q]);
    }
#pragma unroll
    for (int q = 0; q < W; ++q)
#pragma unroll
        for (int m = 0; m < R; ++m) {
            off[m] += c[q][0] * x1[q][m];
            off[m] += c[q][1] * x2[q][m];
        }
    if (sizeof(T) == 4 && chain)
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const T k = kt[e[q] >> (2 * kRankBits)];
#pragma unroll
            for (int m = 0; m < R; ++m) diag[m] += op.mJ4[q0 + q] * k;
        }
}

template <typename T, typename I, int R, bool DOT, bool STORE>
__global__ __launch_bounds__(kBlock) void hx_digit_kernel(
    const DigitArgs<T, I> g, const T *__restrict__ x, T *__restrict__ y,
    const T *__restrict__ prev, const LzStep step, double *__restrict__ partial,
    T *__restrict__ store) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[kLzLds];
    double sigma_v, cprev_v;
    if (!lz_begin(step, red, sigma_v, cprev_v)) return;
    const double sigma = uniform(sigma_v), cprev = uniform(cprev_v);   // scalar registers
    const int WW = g.two_s + 1;
    const int ncf = g.nF * WW * WW * 2;
    T *cf = reinterpret_cast<T *>(smem), *kt = cf + ncf;
    T *xs = reinterpret_cast<T *>(smem + ((size_t)(ncf + WW * WW) * sizeof(T) + 31) / 32 * 32) +
            (size_t)(threadIdx.x >> 6) * R * (g.smax + 1);
    for (int t = threadIdx.x; t < ncf; t += blockDim.x) cf[t] = g.cf[t];
    if constexpr (sizeof(T) == 4) stage_products(kt, g.two_s);
    __syncthreads();
    const Const<T> *kdiag = as_const(g.kdiag), *hJ4 = as_const(g.hJ4);
    const bool chain = sizeof(T) == 4 && g.kdiag;
    const int nHc = chain ? g.nH : 0;

    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int two_s = g.two_s;
    // XCDs (workgroup b runs on XCD b % 8) take turns on runs of g.run groups
    uint32_t stride = gridDim.x * nw, wl = blockIdx.x * nw + (threadIdx.x >> 6), x8 = 0;
    const bool by_xcd = gridDim.x % kXcds == 0;
    if (by_xcd) {
        x8 = blockIdx.x % kXcds;
        stride = (gridDim.x / kXcds) * nw;
        wl = (blockIdx.x / kXcds) * nw + (threadIdx.x >> 6);
    }
    wl = __builtin_amdgcn_readfirstlane(wl);
    x8 = __builtin_amdgcn_readfirstlane(x8);
    stride = __builtin_amdgcn_readfirstlane(stride);
    // the tables are read-only for the whole launch: through the constant
    // address space the wave-uniform reads are scalar loads
    const Const<uint32_t> *groups = as_const(g.groups);
    const Const<DigitBlock<I>> *blocks = as_const(g.blocks);
    const Const<DigitOp<T>> *ops = as_const(g.ops);
    const Const<uint32_t> *mcnt = as_const(g.mcnt);
    const Const<DigitMoves<T, I>> *moves = as_const(g.moves);
    const Const<I> *strad = as_const(g.strad);
    const Const<T> *dhigh = as_const(g.dhigh);
    if (lane < R) xs[g.smax * R + lane] = 0;
    double dot = 0.0;
    for (uint32_t l = wl;; l += stride) {
        const uint32_t it = __builtin_amdgcn_readfirstlane(
            by_xcd ? (l / g.run) * (kXcds * g.run) + x8 * g.run + l % g.run : l);
        if (it >= g.n_groups) break;
        uint32_t hb[R];
        bool valid[R];
        I off0[R];
        uint64_t hw[R];
#pragma unroll
        for (int m = 0; m < R; ++m) hb[m] = groups[(size_t)it * R + m];
#pragma unroll
        for (int m = 0; m < R; ++m) {
            valid[m] = hb[m] != kNoBlock;
            if (!valid[m]) hb[m] = hb[0];            // padding slots shadow slot 0
            off0[m] = blocks[hb[m]].off;
            hw[m] = blocks[hb[m]].hword;
        }
        const int cs = blocks[hb[0]].cs, S = blocks[hb[0]].size;
        int nmin = 1 << 30, nmax = 0, nm[R];
        T dh[R];
        const Const<DigitMoves<T, I>> *mrow[R];
#pragma unroll
        for (int m = 0; m < R; ++m) {
            nm[m] = (int)mcnt[hb[m]];
            nmax = max(nmax, nm[m]);
            nmin = min(nmin, nm[m]);
            dh[m] = dhigh[hb[m]];
            mrow[m] = moves + (size_t)hb[m] * g.mq;
        }
        // copy the blocks to LDS.  The slice is private to the wave and a
        // wave's LDS accesses complete in program order; the wave barriers
        // keep the compiler from moving accesses across.
        __builtin_amdgcn_wave_barrier();
        for (int r = lane; r < S; r += 64) {
            T v[R];
#pragma unroll
            for (int m = 0; m < R; ++m) v[m] = load_at(x, off0[m] + (I)r);
#pragma unroll
            for (int m = 0; m < R; ++m) xs[r * R + m] = v[m];
        }
        __builtin_amdgcn_wave_barrier();
        for (int r1 = 0; r1 < S; r1 += 64) {
            const bool live = r1 + lane < S;
            const int r = live ? r1 + lane : 0;       // dead lanes shadow row 0
            const uint32_t *__restrict__ low = g.low + cs + r;
            const T dl = chain ? (T)0 : g.dlow[cs + r];
            T xi[R], diag[R], off[R];
            lds_row<T, R>(xs + r * R, xi);
#pragma unroll
            for (int m = 0; m < R; ++m) {
                diag[m] = chain ? (T)0 : dl + dh[m];
                off[m] = 0;
            }
            // bonds with their first site in the low word, in list order
            for (int o = 0; o < g.n_ops; ++o) {
                const Const<DigitOp<T>> &op = ops[o];
                const T *cfb = cf + op.first * (WW * WW * 2);
                const uint32_t *__restrict__ lo = low + (size_t)op.first * g.words;
                if (op.straddle < 0) {
                    // four bonds at once where the R rows' reads fit the registers
                    if constexpr (R * sizeof(T) <= 16) {
                        if (op.n == 4) {
                            low_bonds<4, T, R>(lo, g.words, cfb, kt, WW, xs, op, 0, chain, diag, off);
                            continue;
                        }
                    } else if (op.n == 4) {
                        low_bonds<2, T, R>(lo, g.words, cfb, kt, WW, xs, op, 0, chain, diag, off);
                        low_bonds<2, T, R>(lo + 2 * (size_t)g.words, g.words,
                                           cfb + 2 * WW * WW * 2, kt, WW, xs, op, 2, chain, diag, off);
                        continue;
                    }
                    if (op.n == 2) low_bonds<2, T, R>(lo, g.words, cfb, kt, WW, xs, op, 0, chain, diag, off);
                    else low_bonds<1, T, R>(lo, g.words, cfb, kt, WW, xs, op, 0, chain, diag, off);
                    continue;
                }
                const uint32_t e = lo[0], rk1 = e & ((1u << kRankBits) - 1u);
                const uint32_t rk2 = (e >> kRankBits) & ((1u << kRankBits) - 1u);
                const int au = (int)(e >> (2 * kRankBits));
                const T sJ = op.mJ4[0] * (T)(two_s - 2 * au);
                T g1[R], g2[R], c[R][2];
#pragma unroll
                for (int m = 0; m < R; ++m) {
                    // the high digit is wave-uniform, the low one per lane
                    const int av = (int)((hw[m] >> op.sv) & g.mask);
                    const Const<I> *so = strad + ((size_t)hb[m] * g.nS + op.straddle) * 2;
                    const bool a1 = au >= 1 && av < two_s, a2 = av >= 1 && au < two_s;
                    const T v1 = load_at(x, a1 ? so[0] + (I)rk1 : off0[m] + (I)r);
                    const T v2 = load_at(x, a2 ? so[1] + (I)rk2 : off0[m] + (I)r);
                    lds_row<T, 2>(cfb + (au * WW + av) * 2, c[m]);
                    if constexpr (sizeof(T) == 8) diag[m] += sJ * (T)(two_s - 2 * av);
                    else diag[m] += op.mJ4[0] * (T)((two_s - 2 * au) * (two_s - 2 * av));
                    g1[m] = a1 ? v1 : (T)0;
                    g2[m] = a2 ? v2 : (T)0;
                }
#pragma unroll
                for (int m = 0; m < R; ++m) {
                    off[m] += c[m][0] * g1[m];
                    off[m] += c[m][1] * g2[m];
                }
            }
            // bonds inside the high word: the moves the blocks allow,
            // coalesced, four of each of the R blocks at once; past the
            // shortest list, finished ones go on with their own block and add
            // nothing
            // (the diagonal's chain takes its four bonds while the gathers are
            // on their way)
            auto add_diag = [&](int b) {
#pragma unroll
                for (int m = 0; m < R; ++m) {
                    const Const<T> *kd = kdiag + (size_t)hb[m] * g.nH + b;
#pragma unroll
                    for (int q = 0; q < 4; ++q) diag[m] += hJ4[b + q] * kd[q];
                }
            };
            int q0 = 0;
            for (; q0 + 4 <= nmin; q0 += 4) {
                T xj[R][4];
#pragma unroll
                for (int m = 0; m < R; ++m)
#pragma unroll
                    for (int q = 0; q < 4; ++q) xj[m][q] = load_at(x, mrow[m][q0 / 4].off[q] + (I)r);
                if (q0 < nHc) add_diag(q0);
#pragma unroll
                for (int m = 0; m < R; ++m)
#pragma unroll
                    for (int q = 0; q < 4; ++q) off[m] += mrow[m][q0 / 4].cf[q] * xj[m][q];
            }
            for (; q0 < nmax; q0 += 4) {
                T xj[R][4];
#pragma unroll
                for (int m = 0; m < R; ++m)
#pragma unroll
                    for (int q = 0; q < 4; ++q) xj[m][q] = load_at(x, mrow[m][q0 / 4].off[q] + (I)r);
                if (q0 < nHc) add_diag(q0);
#pragma unroll
                for (int m = 0; m < R; ++m)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        off[m] += mrow[m][q0 / 4].cf[q] * (q0 + q < nm[m] ? xj[m][q] : (T)0);
            }
            for (; q0 < nHc; q0 += 4) add_diag(q0);
#pragma unroll
            for (int m = 0; m < R; ++m) {
                if (live && valid[m]) {
                    const I row = off0[m] + (I)r;
                    const T hv = diag[m] * xi[m] + off[m];
                    double w = sigma * (double)hv;
                    if (prev) w -= cprev * (double)prev[row];
                    const T wt = (T)w;
                    y[row] = wt;
                    if constexpr (DOT) dot += (double)wt * (sigma * (double)xi[m]);
                    if constexpr (STORE) store[row] = (T)(sigma * (double)xi[m]);
                }
            }
        }
    }
    if constexpr (DOT) {
        const double s = block_sum(dot, red);
        if (threadIdx.x == 0) partial[blockIdx.x] = s;
    }
    lz_end(step, red, sigma, cprev);
}

// The same rows where blocks are short (sectors far from M = 0 have blocks of a
// few rows, which would leave most lanes of a wave per block idle): one lane
// per row, whatever its block.  The block of a row comes from a table, and the
// block's own tables are read per lane, broadcast among the lanes of one
// block; low-word targets are gathered from memory instead of LDS.
template <int W, typename T, typename I>
__device__ __forceinline__ void flat_low_bonds(const uint32_t *__restrict__ low, int words,
                                               const T *cf, const T *kt, int WW, uint32_t zero,
                                               const T *__restrict__ x, I off0, I row,
                                               const Const<DigitOp<T>> &op, int q0, bool chain,
                                               T &diag, T &off) {
    constexpr uint32_t kMask = (1u << kRankBits) - 1u;
    uint32_t e[W];
    T x1[W], x2[W], c[W][2];
#pragma unroll
    for (int q = 0; q < W; ++q) e[q] = low[(size_t)q * words];
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const uint32_t i1 = e[q] & kMask, i2 = (e[q] >> kRankBits) & kMask;
        const T v1 = load_at(x, i1 != zero ? off0 + (I)i1 : row);
        const T v2 = load_at(x, i2 != zero ? off0 + (I)i2 : row);
        lds_row<T, 2>(cf + (q * WW * WW + (int)(e[q] >> (2 * kRankBits))) * 2, c[q]);
        x1[q] = i1 != zero ? v1 : (T)0;
        x2[q] = i2 != zero ? v2 : (T)0;
    }
#pragma unroll
    for (int q = 0; q < W; ++q) {
        off += c[q][0] * x1[q];
        off += c[q][1] * x2[q];
        if (chain) diag += op.mJ4[q0 + q] * kt[e[q] >> (2 * kRankBits)];
    }
}

template <typename T, typename I, bool DOT, bool STORE>
__global__ __launch_bounds__(kBlock) void hx_digit_flat_kernel(
    const DigitArgs<T, I> g, I dim, const T *__restrict__ x, T *__restrict__ y,
    const T *__restrict__ prev, const LzStep step, double *__restrict__ partial,
    T *__restrict__ store) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[kLzLds];
    double sigma_v, cprev_v;
    if (!lz_begin(step, red, sigma_v, cprev_v)) return;
    const double sigma = uniform(sigma_v), cprev = uniform(cprev_v);   // scalar registers
    const int WW = g.two_s + 1, two_s = g.two_s;
    T *cf = reinterpret_cast<T *>(smem), *kt = cf + g.nF * WW * WW * 2;
    for (int t = threadIdx.x; t < g.nF * WW * WW * 2; t += blockDim.x) cf[t] = g.cf[t];
    stage_products(kt, two_s);
    __syncthreads();
    const Const<T> *hJ4 = as_const(g.hJ4);
    const bool chain = g.kdiag != nullptr;
    const Const<DigitOp<T>> *ops = as_const(g.ops);
    I first, last;
    block_rows<I>(xcd_logical_block(blockIdx.x, gridDim.x), gridDim.x, dim, first, last);
    double dot = 0.0;
    for (I row = first + threadIdx.x; row < last; row += blockDim.x) {
        const uint32_t hb = g.rowblk[row];
        const DigitBlock<I> blk = g.blocks[hb];
        const uint32_t r = (uint32_t)(row - blk.off);
        const uint32_t *__restrict__ low = g.low + blk.cs + r;
        const T xi = x[row];
        T diag = 0, off = 0;
        if (!chain) diag = g.dlow[blk.cs + r] + g.dhigh[hb];
        for (int o = 0; o < g.n_ops; ++o) {
            const Const<DigitOp<T>> &op = ops[o];
            const T *cfb = cf + op.first * (WW * WW * 2);
            const uint32_t *__restrict__ lo = low + (size_t)op.first * g.words;
            if (op.straddle < 0) {
                if (op.n == 4)
                    flat_low_bonds<4, T, I>(lo, g.words, cfb, kt, WW, g.smax, x, blk.off, row,
                                            op, 0, chain, diag, off);
                else if (op.n == 2)
                    flat_low_bonds<2, T, I>(lo, g.words, cfb, kt, WW, g.smax, x, blk.off, row,
                                            op, 0, chain, diag, off);
                else
                    flat_low_bonds<1, T, I>(lo, g.words, cfb, kt, WW, g.smax, x, blk.off, row,
                                            op, 0, chain, diag, off);
                continue;
            }
            const uint32_t e = lo[0], rk1 = e & ((1u << kRankBits) - 1u);
            const uint32_t rk2 = (e >> kRankBits) & ((1u << kRankBits) - 1u);
            const int au = (int)(e >> (2 * kRankBits));
            const int av = (int)((blk.hword >> op.sv) & g.mask);
            const I *__restrict__ so = g.strad + ((size_t)hb * g.nS + op.straddle) * 2;
            const bool a1 = au >= 1 && av < two_s, a2 = av >= 1 && au < two_s;
            const I o1 = so[0], o2 = so[1];
            const T v1 = load_at(x, a1 ? o1 + (I)rk1 : row), v2 = load_at(x, a2 ? o2 + (I)rk2 : row);
            T c[2];
            lds_row<T, 2>(cfb + (au * WW + av) * 2, c);
            diag += op.mJ4[0] * (T)((two_s - 2 * au) * (two_s - 2 * av));
            off += c[0] * (a1 ? v1 : (T)0);
            off += c[1] * (a2 ? v2 : (T)0);
        }
        const DigitMoves<T, I> *__restrict__ mv = g.moves + (size_t)hb * g.mq;
        const int n = (int)g.mcnt[hb];
        for (int q0 = 0; q0 < n; q0 += 4) {
            const DigitMoves<T, I> m = mv[q0 / 4];
            T xj[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) xj[q] = load_at(x, m.off[q] + (I)r);
#pragma unroll
            for (int q = 0; q < 4; ++q) off += m.cf[q] * (q0 + q < n ? xj[q] : (T)0);
        }
        if (chain) {
            typedef T V4 __attribute__((ext_vector_type(4)));
            const V4 *__restrict__ kd = reinterpret_cast<const V4 *>(g.kdiag + (size_t)hb * g.nH);
            for (int b = 0; b < g.nH; b += 4) {
                const V4 k4 = kd[b / 4];
#pragma unroll
                for (int q = 0; q < 4; ++q) diag += hJ4[b + q] * k4[q];
            }
        }
        const T hv = diag * xi + off;
        double w = sigma * (double)hv;
        if (prev) w -= cprev * (double)prev[row];
        const T wt = (T)w;
        y[row] = wt;
        if constexpr (DOT) dot += (double)wt * (sigma * (double)xi);
        if constexpr (STORE) store[row] = (T)(sigma * (double)xi);
    }
    if constexpr (DOT) {
        const double s = block_sum(dot, red);
        if (threadIdx.x == 0) partial[blockIdx.x] = s;
    }
    lz_end(step, red, sigma, cprev);
}

// ---------------------------------------------------------------------------
// Tables (built on the device; the host enumerates the blocks)
// ---------------------------------------------------------------------------
// First row of the block of high word hw: the high sites' terms of the
// encoding sum (PI: type of the prefix table).
template <typename I, typename PI>
__device__ __forceinline__ I block_offset(const PI *__restrict__ P, uint64_t hw, int N, int K,
                                          int A, int two_s, int bits, uint32_t mask) {
    const int W = two_s + 1, site = (A + 1) * W;
    I o = 0;
    int at = (N - 1) * site + A * W;              // entry of digit 0 at the next site
    for (int sh = (N - 1 - K) * bits; sh >= 0; sh -= bits) {
        const int a = (int)((hw >> sh) & mask);
        o += (I)P[at + a];
        at -= site + a * W;
    }
    return o;
}

// The blocks in memory order, one thread per block.  count[n][u]: strings of n digits
// that bring a digit sum u of the sites above into hmin..hmax, so a block's number
// decodes to its high word as a row's does to its state.  With groups of R > 1 blocks
// of one class (digit sum of the low word): the number of blocks of a class before
// this one is a sum over the prefix table, which counts the words of fewer sites;
// a group takes its place by its first block, after those of every class that start
// earlier, so the sweep follows memory order.
// Enumerated on the host, these tables were 0.2 ms of the first product at 484,500
// rows and 3 ms at 5.6 M rows in blocks of 8.5.
template <typename I, typename PI>
__global__ __launch_bounds__(kBlock) void digit_blocks(
    const PI *__restrict__ P, const uint32_t *__restrict__ count, const int *__restrict__ cls,
    const uint32_t *__restrict__ base, int64_t n, int N, int K, int A, int two_s, int bits,
    int hmin, int hmax, int R, DigitBlock<I> *__restrict__ blocks, uint32_t *__restrict__ groups,
    uint32_t *__restrict__ place) {
    const uint32_t mask = (1u << bits) - 1u;
    const int nh = N - K, W = two_s + 1, site = (A + 1) * W;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        uint32_t r = (uint32_t)i;
        int sum = 0;
        uint64_t hw = 0;
        for (int k = nh - 1; k >= 0; --k) {
            const uint32_t *__restrict__ row = count + (size_t)k * (hmax + 1);
            int a = 0;
            for (; sum + a <= hmax && r >= row[sum + a]; ++a) r -= row[sum + a];
            hw |= (uint64_t)a << (k * bits);
            sum += a;
        }
        DigitBlock<I> blk;
        blk.hword = hw;
        blk.off = block_offset<I, PI>(P, hw, N, K, A, two_s, bits, mask);
        blk.cs = cls[2 * (A - sum)];
        blk.size = cls[2 * (A - sum) + 1];
        blk.rank = 0;
        if (groups && R == 1) groups[i] = (uint32_t)i;
        if (groups && R > 1) {
            auto before = [&](int s) {       // high words of digit sum s below hw
                uint32_t c = 0;
                int at = (nh - 1) * site + s * W;
                for (int sh = (nh - 1) * bits; sh >= 0 && s >= 0; sh -= bits) {
                    const int a = (int)((hw >> sh) & mask);
                    c += (uint32_t)P[at + a];
                    at -= site + a * W;
                    s -= a;
                }
                return c;
            };
            const uint32_t q = before(sum);
            blk.rank = (int32_t)q;
            if (q % R == 0) {
                uint32_t g = 0;
                for (int s = hmin; s <= hmax; ++s) g += (before(s) + R - 1) / R;
                groups[(size_t)g * R] = (uint32_t)i;
                for (int m = 1; m < R; ++m) groups[(size_t)g * R + m] = kNoBlock;
                place[base[sum - hmin] + q / R] = g;
            }
        }
        blocks[i] = blk;
    }
}

// The other blocks of every group.
template <typename I>
__global__ __launch_bounds__(kBlock) void digit_group_rest(
    const DigitBlock<I> *__restrict__ blocks, int64_t n, int nh, int bits, int hmin, int R,
    const uint32_t *__restrict__ base, const uint32_t *__restrict__ place,
    uint32_t *__restrict__ groups) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t q = (uint32_t)blocks[i].rank;
        if (q % R == 0) continue;
        int sum = 0;
        for (int k = 0; k < nh; ++k)
            sum += (int)((blocks[i].hword >> (k * bits)) & ((1u << bits) - 1u));
        groups[(size_t)place[base[sum - hmin] + q / R] * R + q % R] = (uint32_t)i;
    }
}

// Block of every row: one wave per block.
template <typename I>
__global__ __launch_bounds__(kBlock) void digit_row_blocks(const DigitBlock<I> *__restrict__ blocks,
                                                           int64_t n, uint32_t *__restrict__ rowblk) {
    const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t i = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6; i < n; i += nw)
        for (int r = threadIdx.x & 63; r < blocks[i].size; r += 64)
            rowblk[(size_t)blocks[i].off + r] = (uint32_t)i;
}

// Rows of the block tables: the allowed high-word moves in bond order (first
// a_u - 1, a_v + 1, then the other; padded with the own block and 0), the
// diagonal part, and the target blocks of the straddling bonds' two moves (the
// own block where the high digit does not allow one).  The matrix elements
// have the roundings of row_hx.  2^log_parts threads share a block, each with a range of
// its bonds, since a thread waits for the walks of its targets one after the other
// (484,500 rows, 47,672 blocks, J1-J2 ring: 108 us with a thread per block, 20 with
// 8); the places of a range's moves are counted from the digits alone.
template <typename T, typename I, typename PI>
__global__ __launch_bounds__(kBlock) void digit_rows(
    const PI *__restrict__ P, const DigitBlock<I> *__restrict__ blocks, int64_t n, int log_parts,
    bool lane_per_row, int N, int K, int A, int two_s, int bits, uint32_t mask,
    const BondDev *__restrict__ bonds, int nb, int nF, const double *__restrict__ ladder, int nS, int mw, DigitMoves<T, I> *__restrict__ moves,
    uint32_t *__restrict__ mcnt, T *__restrict__ dhigh, int nH, T *__restrict__ kdiag,
    T *__restrict__ hJ4, I *__restrict__ strad) {
    const int parts = 1 << log_parts;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n << log_parts;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = t >> log_parts;
        const int part = (int)t & (parts - 1);
        const int b0 = (nb * part) >> log_parts, b1 = (nb * (part + 1)) >> log_parts;
        const uint64_t hw = blocks[i].hword;
        const I own = blocks[i].off;
        auto digit = [&](int site) { return (int)((hw >> ((site - K) * bits)) & mask); };
        auto target = [&](uint64_t to) {
            return block_offset<I, PI>(P, to, N, K, A, two_s, bits, mask);
        };
        DigitMoves<T, I> *row = moves + (size_t)i * (mw / 4);
        auto put = [&](int c, I o, T f) {
            row[c / 4].off[c % 4] = o;
            row[c / 4].cf[c % 4] = f;
        };
        int c = 0, s = 0;                 // moves and straddling bonds before b0
        for (int b = 0; b < b0; ++b) {
            const int u = bonds[b].u, v = bonds[b].v;
            if (v < K) continue;
            if (u < K) {
                ++s;
                continue;
            }
            const int au = digit(u), av = digit(v);
            c += (au >= 1 && av < two_s) + (av >= 1 && au < two_s);
        }
        for (int b = b0; b < b1; ++b) {
            const int u = bonds[b].u, v = bonds[b].v;
            if (v < K) continue;
            const int av = digit(v);
            const uint64_t ev = 1ull << ((v - K) * bits);
            if (u < K) {
                I *o = strad + ((size_t)i * nS + s++) * 2;
                o[0] = av < two_s ? target(hw + ev) : own;
                o[1] = av >= 1 ? target(hw - ev) : own;
                continue;
            }
            const int au = digit(u);
            const uint64_t eu = 1ull << ((u - K) * bits);
            const T mJ2 = (T)bonds[b].mJ2;
            if (au >= 1 && av < two_s)
                put(c++, target(hw - eu + ev), mJ2 * (T)ladder[au] * (T)ladder[av + 1]);
            if (av >= 1 && au < two_s)
                put(c++, target(hw + eu - ev), mJ2 * (T)ladder[av] * (T)ladder[au + 1]);
            if (kdiag) {
                kdiag[(size_t)i * nH + b - nF] = (T)((two_s - 2 * au) * (two_s - 2 * av));
                if (i == 0) hJ4[b - nF] = (T)bonds[b].mJ4;
            }
        }
        if (part + 1 < parts) continue;
        double d = 0.0;
        for (int b = nF; b < nb; ++b)
            d += (double)(T)bonds[b].mJ4 *
                 (double)((two_s - 2 * digit(bonds[b].u)) * (two_s - 2 * digit(bonds[b].v)));
        for (int h = nb - nF; kdiag && h < nH; ++h) {
            kdiag[(size_t)i * nH + h] = 0;
            if (i == 0) hJ4[h] = 0;
        }
        mcnt[i] = (uint32_t)c;
        dhigh[i] = (T)d;
        // (one lane per row reads its own list only, a wave of R blocks the longest)
        const int end = lane_per_row ? (c + 3) / 4 * 4 : mw;
        for (; c < end; ++c) put(c, own, (T)0);
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
namespace {

// Whether a vector of doubles stays below 4 GiB: 32-bit indices and byte offsets.
bool small_index(const Basis *b) { return b->dim < ((int64_t)1 << 29); }

int64_t ipow(int64_t b, int e) {
    int64_t r = 1;
    for (int i = 0; i < e; ++i) r *= b;
    return r;
}

// Blocks of a split at K low sites: by digit sum of the low word, the number
// of rows of a block and of blocks.
void split_counts(const Basis *b, int K, std::vector<int64_t> &size, std::vector<int64_t> &blocks) {
    const int nh = b->N - K;
    size.assign((size_t)K * b->two_s + 1, 0);
    blocks.assign(size.size(), 0);
    for (int a = 0; a <= K * b->two_s; ++a) {
        size[a] = b->count(K, a);
        const int ah = b->A - a;
        blocks[a] = ah < 0 || ah > nh * b->two_s ? 0 : b->count(nh, ah);
    }
}

// LDS of a workgroup: matrix elements of the front bonds, R blocks per wave.
size_t digit_lds(const Basis *b, int R, int smax, int nF, size_t es) {
    const size_t W = (size_t)b->two_s + 1;
    return ((2 * (size_t)nF + 1) * W * W * es + 31) / 32 * 32 +
           (size_t)(kBlock / 64) * R * (smax + 1) * es;
}

// Device arrays of one table set in one allocation: those with host contents
// first, then those that kernels fill.
struct Arena {
    struct Part { size_t at, bytes; const void *src; };
    std::vector<Part> parts;         // their vectors live until the upload
    size_t total = 0, filled = 0;    // filled: end of the last part
    template <typename V> size_t add(const std::vector<V> &v) {
        const size_t at = reserve(v.size() * sizeof(V));
        if (!v.empty()) parts.push_back({at, v.size() * sizeof(V), v.data()});
        filled = total;
        return at;
    }
    size_t reserve(size_t bytes) {
        const size_t at = total;
        total = (total + bytes + 255) / 256 * 256;
        return at;
    }
    hipError_t upload(void **mem) const {
        hipError_t e = hipMalloc(mem, total + 256);
        std::vector<unsigned char> host(filled);
        for (const Part &p : parts) std::memcpy(host.data() + p.at, p.src, p.bytes);
        if (e == hipSuccess && filled)
            e = hipMemcpy(*mem, host.data(), filled, hipMemcpyHostToDevice);
        return e;
    }
};

void count_bonds(const Couplings *c, int K, int *nF, int *nH, int *nS) {
    *nF = *nH = *nS = 0;
    for (const BondDev &d : c->host) {
        if (d.u >= K) ++*nH;
        else {
            ++*nF;
            if (d.v >= K) ++*nS;
        }
    }
}

size_t digit_table_bytes(const Basis *b, const DigitSplit &s, const Couplings *c, size_t es) {
    int nF, nH, nS;
    count_bonds(c, s.K, &nF, &nH, &nS);
    const size_t is = small_index(b) ? 4 : 8, bs = 32;
    return (size_t)s.n_blocks *
               ((2 * (size_t)nH + 3) * (is + es) + 4 + (nH + 4) * es + 2 * (size_t)nS * is + bs) +
           (s.flat ? (size_t)b->dim * sizeof(uint32_t) : 0);
}

}  // namespace

// How the rows are split.  A wave per R blocks pays once a wave's lanes are
// mostly in use and there are enough blocks to fill the chip; below that one
// lane per row is faster.  Measured (us per H x of nearest-neighbour rings,
// FP64 / FP32; wave per blocks, lane per row, generic kernel):
//   s = 1,   16 sites, M = 0,  5,196,627 rows:   95 / 60,  121 / 100,  261 / 250
//   s = 1,   18 sites, M = 3, 30,759,120 rows:  590 / 387, 824 / 604, 1662 / 1590
//   s = 3/2, 12 sites, M = 0,  1,703,636 rows:   37 / 27,   43 / 34,    79 / 75
//   s = 1,   16 sites, M = 5,  1,665,456 rows:   53 / 35,   44 / 37,    95 / 91
//   s = 1,   20 sites, M = 13,   484,500 rows:   62 / 34,   21 / 16,    48 / 46
//   s = 1,   14 sites, M = 0,    616,227 rows:   25 / 13,   18 / 12,    39 / 38
// so one lane per row below kFlatRows rows and where fewer than kFlatUse of a
// wave's lanes would have a row.
constexpr int64_t kFlatRows = (int64_t)1 << 20;
constexpr double kFlatUse = 0.6;
constexpr int kFlatWords = 4096;     // most low words with one lane per row

DigitSplit choose_digit_split(const Basis *b) {
    // waves of a launch go in rounds of kSlots (4 per SIMD); a wave's time is
    // that of its group (tables, copy to LDS) plus that of its 64-row chunks,
    // which grows with the rows per lane
    constexpr double kSlots = 4096.0;
    DigitSplit best, flat;
    if (b->two_s < 2 || b->two_s > 15) return best;
    double best_t = 0.0, best_use = 0.0;
    std::vector<int64_t> size, blocks;
    for (int K = 1; K < b->N && ipow(b->two_s + 1, K) <= kDigitMaxWords; ++K) {
        split_counts(b, K, size, blocks);
        for (int R : {1, 2, 4}) {
            DigitSplit s;
            s.K = K;
            s.R = R;
            double work = 0.0, longest = 0.0, lanes = 0.0;
            for (size_t a = 0; a < size.size(); ++a) {
                if (!blocks[a]) continue;
                s.smax = (int)std::min<int64_t>(std::max<int64_t>(s.smax, size[a]), kDigitMaxSize);
                const int64_t n = (blocks[a] + R - 1) / R, chunks = (size[a] + 63) / 64;
                const double t = 1.0 + (double)chunks * (0.5 + 0.25 * R);
                s.n_blocks += blocks[a];
                s.n_groups += n;
                work += (double)n * t;
                lanes += (double)blocks[a] * (double)chunks * 64.0;
                longest = std::max(longest, t);
            }
            if (s.smax >= kDigitMaxSize || s.n_blocks >= ((int64_t)1 << 31)) continue;
            if (R == 1 && ipow(b->two_s + 1, K) <= kFlatWords) {
                flat = s;
                flat.flat = true;
            }
            if ((size_t)(kBlock / 64) * R * (s.smax + 1) * 8 > 36 * 1024) continue;
            const double t = std::max(longest, work / kSlots);
            if (best.K == 0 || t < best_t) {
                best = s;
                best_t = t;
                best_use = (double)b->dim / lanes;
            }
        }
    }
    if (flat.K && (b->dim < kFlatRows || best.K == 0 || best_use < kFlatUse)) return flat;
    return best;
}

// Whether the block kernel for s >= 1 runs these couplings (c null: whether it
// can run on this basis at all): its LDS and its tables fit the budgets.
bool digit_fits(const Basis *b, const Couplings *c) {
    const DigitSplit &s = b->digit;
    if (s.K == 0) return false;
    if (!c) return true;
    int nF, nH, nS;
    count_bonds(c, s.K, &nF, &nH, &nS);
    return digit_lds(b, s.flat ? 0 : s.R, s.smax, nF, 8) <= kDigitMaxLds &&
           digit_table_bytes(b, s, c, 8) <=
               std::min(kDigitMaxTables,
                        std::max(kDigitFreeTables, 4 * sizeof(double) * (size_t)b->dim));
}

// Workgroups for n_groups waves of work: one group per wave up to a grid far
// beyond the resident workgroups, so that the dispatcher evens out groups of
// unequal size (18 sites, s = 1, M = 3, 30.8 M rows, FP32: 483 us on 2048
// workgroups, 417 on 4096, 391 on 16384 and 392 on 65536).
static int grid_of(int64_t n_groups) {
    int64_t g = std::min<int64_t>((n_groups + kBlock / 64 - 1) / (kBlock / 64), kDigitMaxGrid);
    if (g >= kXcds) g -= g % kXcds;
    return (int)std::max<int64_t>(g, 1);
}

// One lane per row: up to 2048 workgroups of 256 rows this is the generic kernel's
// grid, so a run has that kernel's partial sums too.
int hx_digit_grid(const Basis *b) {
    return b->digit.flat ? grid_of((b->dim + 63) / 64) : grid_of(b->digit.n_groups);
}

// The blocks and groups, on the device.
template <typename I, typename PI>
static int put_blocks(const Basis *b, DigitTables *t) {
    const int nh = b->N - t->K, two_s = b->two_s, A = b->A, R = t->R;
    const int hmin = std::max(0, A - t->K * two_s), hmax = std::min(A, nh * two_s);
    std::vector<uint32_t> count((size_t)(nh + 1) * (hmax + 1), 0);
    for (int u = hmin; u <= hmax; ++u) count[u] = 1;
    for (int n = 1; n <= nh; ++n)
        for (int u = 0; u <= hmax; ++u)
            for (int a = 0; a <= two_s && u + a <= hmax; ++a)
                count[(size_t)n * (hmax + 1) + u] += count[(size_t)(n - 1) * (hmax + 1) + u + a];
    const uint32_t blocks = count[(size_t)nh * (hmax + 1)];
    std::vector<uint32_t> base;                 // first group of every digit sum
    uint32_t groups = 0;
    for (int s = hmin; s <= hmax; ++s) {
        base.push_back(groups);
        groups += (uint32_t)((b->count(nh, s) + R - 1) / R);
    }
    if ((int64_t)blocks != t->n_blocks || (int64_t)groups != t->n_groups)
        return fail(HM_EINVAL, "internal: %u blocks in %u groups, expected %lld in %lld", blocks,
                    groups, (long long)t->n_blocks, (long long)t->n_groups);
    const bool flat = b->digit.flat;
    Arena arena;
    const size_t o_count = arena.add(count), o_base = arena.add(base), o_cls = arena.add(t->cls);
    const size_t o_rank = arena.add(t->rank), o_word = arena.add(t->word);
    const size_t o_blocks = arena.reserve((size_t)t->n_blocks * sizeof(DigitBlock<I>));
    const size_t o_groups = arena.reserve(flat ? 0 : (size_t)groups * R * sizeof(uint32_t));
    const size_t o_place = arena.reserve(flat || R == 1 ? 0 : (size_t)groups * sizeof(uint32_t));
    const size_t o_rows = arena.reserve(flat ? (size_t)b->dim * sizeof(uint32_t) : 0);
    const hipError_t e = arena.upload(&t->mem);
    if (e != hipSuccess)
        return fail(e == hipErrorOutOfMemory ? HM_ENOMEM : HM_EDEVICE, "block kernel tables: %s",
                    hipGetErrorString(e));
    unsigned char *m = (unsigned char *)t->mem;
    t->blocks = m + o_blocks;
    t->groups = (uint32_t *)(m + o_groups);
    t->rowblk = (uint32_t *)(m + o_rows);
    t->d_rank = (uint16_t *)(m + o_rank);
    t->d_word = (uint16_t *)(m + o_word);
    auto *blk = (DigitBlock<I> *)t->blocks;
    const uint32_t *d_base = (const uint32_t *)(m + o_base);
    uint32_t *place = (uint32_t *)(m + o_place);
    const dim3 grid((unsigned)std::min<int64_t>((t->n_blocks + kBlock - 1) / kBlock, kMaxGrid));
    hipLaunchKernelGGL((digit_blocks<I, PI>), grid, dim3(kBlock), 0, nullptr,
                       (const PI *)b->d_prefix, (const uint32_t *)(m + o_count),
                       (const int *)(m + o_cls), d_base, t->n_blocks, b->N, t->K, A, two_s, b->bits,
                       hmin, hmax, R, blk, flat ? nullptr : t->groups, place);
    if (!flat && R > 1)
        hipLaunchKernelGGL(digit_group_rest<I>, grid, dim3(kBlock), 0, nullptr, blk, t->n_blocks,
                           nh, b->bits, hmin, R, d_base, place, t->groups);
    if (flat)
        hipLaunchKernelGGL(digit_row_blocks<I>, dim3(kMaxGrid), dim3(kBlock), 0, nullptr, blk,
                           t->n_blocks, t->rowblk);
    HM_HIP(hipGetLastError());
    return HM_OK;
}

static int digit_prepare(Basis *b, DigitTables **out) {
    if (b->digit_tables) {
        *out = (DigitTables *)b->digit_tables;
        return HM_OK;
    }
    const DigitSplit &sp = b->digit;
    const int K = sp.K, W = b->two_s + 1, words = (int)ipow(W, K);
    auto *t = new DigitTables;
    t->K = K;
    t->R = sp.R;
    t->words = words;
    t->smax = sp.smax;
    t->n_blocks = sp.n_blocks;
    t->n_groups = sp.n_groups;
    t->nclass = K * b->two_s + 1;
    // low words, ascending within every digit sum
    t->cls.resize(2 * (size_t)t->nclass);
    for (int a = 0, s = 0; a < t->nclass; ++a) {
        t->cls[2 * a] = s;
        t->cls[2 * a + 1] = (int)b->count(K, a);
        s += t->cls[2 * a + 1];
    }
    t->rank.resize(words);
    t->word.resize(words);
    std::vector<int> fill(t->nclass, 0);
    std::vector<uint8_t> digits(words, 0);             // digit sums
    for (int n = 0; n < words; ++n) {
        const int a = digits[n] = (uint8_t)(digits[n / W] + n % W);
        t->rank[n] = (uint16_t)fill[a];
        t->word[t->cls[2 * a] + fill[a]] = (uint16_t)n;
        ++fill[a];
    }
    const int rc = small_index(b) ? put_blocks<uint32_t, uint32_t>(b, t)
                   : b->idx32     ? put_blocks<uint64_t, uint32_t>(b, t)
                                  : put_blocks<uint64_t, uint64_t>(b, t);
    if (rc != HM_OK) {
        free_digit(t);
        return rc;
    }
    b->digit_tables = t;
    b->digit_tables_free = free_digit;
    *out = t;
    return HM_OK;
}

// Whether the rows are the generic kernel's in FP64 too.  Up to 2^19 rows a run has
// that kernel's partial sums as well (one lane per row, a workgroup for every 256
// rows), so that equal rows make its coefficients equal; up to kFlatRows the first
// product may come from either kernel (digit_put_off).  The sums bond by bond cost 0
// to 4 % there, in short blocks of larger subspaces 15 to 36 % (24 sites, s = 1,
// A = 8, 5.6 M rows: 241 and 278 us).
static bool generic_bits(const Basis *b) { return b->digit.flat && b->dim <= kFlatRows; }

// Whether T holds every sum of diagonal terms of these couplings exactly
// (multiples of one power of two, the largest below 2^24 or 2^53 of it; couplings
// of 1 or 0.25, say): then no order of summation rounds.
template <typename T>
static bool exact_diagonal(const Basis *b, const Couplings *c) {
    constexpr int kBits = std::numeric_limits<T>::digits;
    double sum = 0.0;
    int low = 0;                          // smallest bit set in any -J/4
    bool any = false;
    for (const BondDev &bd : c->host) {
        const T f = (T)bd.mJ4;
        if (f == (T)0) continue;
        if (!std::isfinite(f)) return false;
        int e;
        const double m = std::frexp((double)f, &e);
        const int bit = e - kBits + __builtin_ctzll((uint64_t)std::fabs(std::ldexp(m, kBits)));
        low = any ? std::min(low, bit) : bit;
        any = true;
        sum += std::fabs((double)f) * b->two_s * b->two_s;
    }
    return !any || sum < std::ldexp(1.0, kBits + low);
}

// The low-word table: per bond of a low site (the first nF of the list, which is
// sorted by u; blockIdx.y) and low word, the ranks that its two moves lead to (smax
// where a move is not allowed; with the other site in the high word, the rank with u
// alone changed) and the entry of its matrix elements.  The last blockIdx.y: per low
// word the diagonal part of the bonds inside it.
template <typename T>
__global__ __launch_bounds__(kBlock) void digit_low(const BondDev *__restrict__ bonds, int nF, int K,
                                                    int two_s, int words, int smax,
                                                    const uint16_t *__restrict__ rank,
                                                    const uint16_t *__restrict__ word,
                                                    uint32_t *__restrict__ low,
                                                    T *__restrict__ dlow) {
    const int i = blockIdx.x * kBlock + threadIdx.x, f = blockIdx.y;
    if (i >= words) return;
    const int W = two_s + 1, n = word[i];
    constexpr uint32_t kMask = (1u << kRankBits) - 1u;
    auto power = [&](int q) {
        int w = 1;
        while (q-- > 0) w *= W;
        return w;
    };
    if (f == nF) {
        double sum = 0.0;
        for (int b = 0; b < nF; ++b) {
            if (bonds[b].v >= K) continue;
            const int au = n / power(bonds[b].u) % W, av = n / power(bonds[b].v) % W;
            sum += (double)(T)bonds[b].mJ4 * (double)((two_s - 2 * au) * (two_s - 2 * av));
        }
        dlow[i] = (T)sum;
        return;
    }
    const int v = bonds[f].v, wu = power(bonds[f].u), au = n / wu % W;
    uint32_t r1, r2, e;
    if (v < K) {
        const int wv = power(v), av = n / wv % W;
        r1 = au >= 1 && av < two_s ? rank[n - wu + wv] : smax;
        r2 = av >= 1 && au < two_s ? rank[n + wu - wv] : smax;
        e = (uint32_t)(au * W + av);
    } else {
        r1 = au >= 1 ? rank[n - wu] : rank[n];
        r2 = au < two_s ? rank[n + wu] : rank[n];
        e = (uint32_t)au;
    }
    // (a class without blocks may be larger than the field, and is not used)
    low[(size_t)f * words + i] = (r1 & kMask) | (r2 & kMask) << kRankBits | e << (2 * kRankBits);
}

template <typename T, typename I, typename PI>
static hipError_t build_bonds(const Basis *b, const Couplings *c, const DigitTables *t,
                              DigitBonds *d) {
    const int K = t->K, W = b->two_s + 1, words = t->words, two_s = b->two_s;
    int nH = 0;
    count_bonds(c, K, &d->nF, &nH, &d->nS);
    d->mw = (2 * nH + 3) / 4 * 4;
    // runs of low-word bonds in fours, twos and ones
    std::vector<DigitOp<T>> ops;
    std::vector<T> cf;
    std::vector<const BondDev *> front;
    for (const BondDev &bd : c->host)
        if (bd.u < K) front.push_back(&bd);
    int ns = 0;
    for (size_t i = 0; i < front.size();) {
        DigitOp<T> op{};
        op.first = (int)i;
        size_t n = 1;
        if (front[i]->v >= K) {
            op.straddle = ns++;
            op.sv = (front[i]->v - K) * b->bits;
        } else {
            op.straddle = -1;
            while (n < 4 && i + n < front.size() && front[i + n]->v < K) ++n;
            if (n == 3) n = 2;
        }
        op.n = (int)n;
        for (size_t q = 0; q < n; ++q) op.mJ4[q] = (T)front[i + q]->mJ4;
        ops.push_back(op);
        i += n;
    }
    d->n_ops = (int)ops.size();
    // per front bond the matrix elements, with the roundings of row_hx
    for (const BondDev *bd : front) {
        const T mJ2 = (T)bd->mJ2;
        for (int au = 0; au < W; ++au)
            for (int av = 0; av < W; ++av) {
                // (0 where the digits do not allow the move, also for an infinite mJ2)
                const T one = mJ2 * (T)b->ladder[au], two = mJ2 * (T)b->ladder[av];
                cf.push_back(au >= 1 && av < two_s ? one * (T)b->ladder[av + 1] : (T)0);
                cf.push_back(av >= 1 && au < two_s ? two * (T)b->ladder[au + 1] : (T)0);
            }
    }
    Arena arena;
    const size_t o_ops = arena.add(ops), o_cf = arena.add(cf);
    const size_t o_low = arena.reserve(front.size() * words * sizeof(uint32_t));
    const size_t o_dlow = arena.reserve((size_t)words * sizeof(T));
    const size_t nblk = (size_t)t->n_blocks;
    const size_t o_moves = arena.reserve(nblk * (d->mw / 4) * sizeof(DigitMoves<T, I>));
    const size_t o_mcnt = arena.reserve(nblk * sizeof(uint32_t));
    const size_t o_dhigh = arena.reserve(nblk * sizeof(T));
    const bool chain = (sizeof(T) == 4 || generic_bits(b)) && !exact_diagonal<T>(b, c);
    d->nH = chain ? (nH + 3) / 4 * 4 : 0;
    const size_t o_kdiag = arena.reserve(nblk * d->nH * sizeof(T));
    const size_t o_hJ4 = arena.reserve(d->nH * sizeof(T));
    const size_t o_strad = arena.reserve(nblk * d->nS * 2 * sizeof(I));
    hipError_t e = arena.upload(&d->mem);
    if (e != hipSuccess) return e;
    unsigned char *m = (unsigned char *)d->mem;
    d->ops = m + o_ops;
    d->cf = m + o_cf;
    d->low = (uint32_t *)(m + o_low);
    d->dlow = m + o_dlow;
    d->moves = m + o_moves;
    d->mcnt = (uint32_t *)(m + o_mcnt);
    d->dhigh = m + o_dhigh;
    d->kdiag = chain ? m + o_kdiag : nullptr;
    d->hJ4 = m + o_hJ4;
    d->strad = m + o_strad;
    hipLaunchKernelGGL(digit_low<T>, dim3((words + kBlock - 1) / kBlock, d->nF + 1), dim3(kBlock), 0,
                       nullptr, c->dev, d->nF, K, two_s, words, t->smax, t->d_rank, t->d_word, d->low,
                       (T *)d->dlow);
    // threads for the whole chip, at most one for two bonds
    int log_parts = 0;
    while (log_parts < 5 && (t->n_blocks << log_parts) < kMaxGrid * kBlock &&
           4 << log_parts <= c->nb)
        ++log_parts;
    const int grid = (int)std::min<int64_t>(((t->n_blocks << log_parts) + kBlock - 1) / kBlock,
                                            4 * kMaxGrid);
    hipLaunchKernelGGL((digit_rows<T, I, PI>), dim3(grid), dim3(kBlock), 0, nullptr,
                       (const PI *)b->d_prefix, (const DigitBlock<I> *)t->blocks, t->n_blocks, log_parts,
                       b->digit.flat, b->N, K, b->A, two_s, b->bits, (1u << b->bits) - 1u, c->dev, c->nb, d->nF,
                       b->d_ladder, d->nS, d->mw, (DigitMoves<T, I> *)d->moves, d->mcnt, (T *)d->dhigh,
                       d->nH, (T *)d->kdiag, (T *)d->hJ4, (I *)d->strad);
    e = hipGetLastError();
    // other streams may use the tables from now on
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    return e;
}

template <typename T>
static hipError_t build_bonds_t(const Basis *b, const Couplings *c, const DigitTables *t,
                                DigitBonds *d) {
    if (small_index(b)) return build_bonds<T, uint32_t, uint32_t>(b, c, t, d);
    if (b->idx32) return build_bonds<T, uint64_t, uint32_t>(b, c, t, d);
    return build_bonds<T, uint64_t, uint64_t>(b, c, t, d);
}

// The tables of these couplings in this element type, built on first use.
static DigitBondSet *bond_set(const Couplings *c) {
    auto *cc = const_cast<Couplings *>(c);
    if (!cc->half) {
        cc->half = new DigitBondSet;
        cc->half_free = free_digit_bonds;
    }
    return (DigitBondSet *)cc->half;
}

static int digit_get(Basis *b, const Couplings *c, int dtype, hipStream_t st, DigitTables **tout,
                     const DigitBonds **bout) {
    std::lock_guard<std::mutex> lock(b->mu);
    HM_TRY(device_prepare(b));
    DigitBondSet *set = bond_set(c);
    const int k = dtype == HM_F64 ? 0 : 1;
    if (!set->have[k] && is_capturing(st)) return HM_ENOMEM;
    DigitTables *t = nullptr;
    HM_TRY(digit_prepare(b, &t));
    if (!set->have[k]) {
        DigitBonds d;
        hipError_t e;
        if (dtype == HM_F64) e = build_bonds_t<double>(b, c, t, &d);
        else e = build_bonds_t<float>(b, c, t, &d);
        if (e != hipSuccess) {
            if (d.mem) (void)hipFree(d.mem);
            return fail(e == hipErrorOutOfMemory ? HM_ENOMEM : HM_EDEVICE,
                        "block kernel bonds: %s", hipGetErrorString(e));
        }
        set->by_type[k] = d;
        set->have[k] = true;
    }
    *tout = t;
    *bout = &set->by_type[k];
    return HM_OK;
}

// Builds the tables ahead of a run.
int digit_prepare_tables(Basis *b, const Couplings *c, int dtype) {
    DigitTables *t = nullptr;
    const DigitBonds *d = nullptr;
    return digit_get(b, c, dtype, nullptr, &t, &d);
}

template <typename T, typename I, int R>
static void launch_digit_r(const DigitTables *t, const DigitArgs<T, I> &g, size_t lds,
                           const HxPass &p, hipStream_t st) {
    const int grid = grid_of(t->n_groups);
    const T *x = (const T *)p.x, *pr = (const T *)p.p;
    T *y = (T *)p.y, *store = (T *)p.store;
#define HM_LAUNCH(D, S)                                                                        \
    hipLaunchKernelGGL((hx_digit_kernel<T, I, R, D, S>), dim3(grid), dim3(kBlock), lds, st, g, \
                       x, y, pr, p.step, p.partial, store)
    const bool dot = p.partial != nullptr, sto = store != nullptr;
    if (!dot && !sto) HM_LAUNCH(false, false);
    else if (dot && !sto) HM_LAUNCH(true, false);
    else if (!dot && sto) HM_LAUNCH(false, true);
    else HM_LAUNCH(true, true);
#undef HM_LAUNCH
}

template <typename T, typename I>
static void launch_digit_t(const Basis *b, const DigitTables *t, const DigitBonds *d,
                           const HxPass &p, hipStream_t st) {
    DigitArgs<T, I> g{};
    g.blocks = (const DigitBlock<I> *)t->blocks;
    g.groups = t->groups;
    g.ops = (const DigitOp<T> *)d->ops;
    g.cf = (const T *)d->cf;
    g.low = d->low;
    g.dlow = (const T *)d->dlow;
    g.moves = (const DigitMoves<T, I> *)d->moves;
    g.mcnt = d->mcnt;
    g.dhigh = (const T *)d->dhigh;
    g.kdiag = (const T *)d->kdiag;
    g.hJ4 = (const T *)d->hJ4;
    g.strad = (const I *)d->strad;
    g.n_ops = d->n_ops;
    g.n_groups = (uint32_t)t->n_groups;
    // runs of 64 groups once every XCD gets many of them, else of one
    // workgroup's four, so that few groups still spread over the XCDs
    g.run = t->n_groups >= 8192 ? 64 : kBlock / 64;
    g.nF = d->nF;
    g.nS = d->nS;
    g.nH = d->nH;
    g.mq = d->mw / 4;
    g.words = t->words;
    g.smax = t->smax;
    g.two_s = b->two_s;
    g.mask = (1 << b->bits) - 1;
    g.rowblk = t->rowblk;
    if (b->digit.flat) {
        const size_t W = (size_t)b->two_s + 1, cf = (2 * (size_t)d->nF + 1) * W * W * sizeof(T);
        const int grid = hx_digit_grid(b);
        const T *x = (const T *)p.x, *pr = (const T *)p.p;
        T *y = (T *)p.y, *store = (T *)p.store;
#define HM_LAUNCH(D, S)                                                                          \
    hipLaunchKernelGGL((hx_digit_flat_kernel<T, I, D, S>), dim3(grid), dim3(kBlock), cf, st, g,  \
                       (I)b->dim, x, y, pr, p.step, p.partial, store)
        const bool dot = p.partial != nullptr, sto = store != nullptr;
        if (!dot && !sto) HM_LAUNCH(false, false);
        else if (dot && !sto) HM_LAUNCH(true, false);
        else if (!dot && sto) HM_LAUNCH(false, true);
        else HM_LAUNCH(true, true);
#undef HM_LAUNCH
        return;
    }
    const size_t lds = digit_lds(b, t->R, t->smax, d->nF, sizeof(T));
    if (t->R == 1) launch_digit_r<T, I, 1>(t, g, lds, p, st);
    else if (t->R == 2) launch_digit_r<T, I, 2>(t, g, lds, p, st);
    else launch_digit_r<T, I, 4>(t, g, lds, p, st);
}

// Whether a coupling list's first plain product goes to the generic kernel, whose
// rows are the same bit for bit: where that product costs less than this kernel's
// tables, which a list used once never pays back.  That is below some kFirstWork
// row-bonds, and in blocks of a few rows, whose tables take as long as the rows.
// Measured (us of a first product with new couplings on a used basis, generic kernel
// / tables and product; FP32, J1-J2 rings unless said):
//   s = 1,   12 sites, M = 0,     73,789 rows,   24 bonds:   61 / 90,  later  50 / 30
//   s = 1,   14 sites, M = 0,    616,227 rows,   28 bonds:   97 / 104, later  85 / 38
//   s = 3/2, 12 sites, M = 0,  1,703,636 rows,   12 bonds:  103 / 116, later  91 / 48
//   s = 1,   15 sites, M = 0,  1,787,607 rows,   15 bonds:  120 / 121, later 109 / 48
//   s = 1,   14 sites, M = 0,    616,227 rows,   91 bonds:  308 / 200, later 290 / 86
//   s = 1,   20 sites, M = 13,   484,500 rows,   40 bonds:  112 / 188, later 101 / 54
//   s = 1,   24 sites, M = 16, 5,612,805 rows,   48 bonds:  762 / 1048, later 748 / 406
constexpr int64_t kFirstWork = (int64_t)1 << 25, kFirstRows = 16;

static bool digit_put_off(Basis *b, const Couplings *c, int dtype) {
    if (dtype == HM_F64 && !generic_bits(b)) return false;
    if (b->dim * c->nb >= kFirstWork && b->dim >= kFirstRows * b->digit.n_blocks) return false;
    std::lock_guard<std::mutex> lock(b->mu);
    DigitBondSet *set = bond_set(c);
    const int k = dtype == HM_F64 ? 0 : 1;
    if (set->have[k] || set->seen[k]) return false;
    set->seen[k] = true;
    return true;
}

int launch_hx_digit(const Basis *cb, const Couplings *c, int dtype, const HxPass &p,
                    hipStream_t st) {
    Basis *b = const_cast<Basis *>(cb);
    if (!p.step.sigma && digit_put_off(b, c, dtype)) {
        const int rc = launch_hx_generic(b, c, dtype, p, st);
        if (rc != HM_ERANGE) return rc;
        clear_error();                 // a prefix table beyond that kernel's LDS
    }
    DigitTables *t = nullptr;
    const DigitBonds *d = nullptr;
    const int rc = digit_get(b, c, dtype, st, &t, &d);
    if (rc == HM_ENOMEM && !p.step.sigma) {
        // no memory for the tables, or a product captured before its first
        // use: the generic kernel's rows are the same bit for bit, in larger FP64
        // subspaces within rounding
        clear_error();
        (void)hipGetLastError();
        return launch_hx_generic(b, c, dtype, p, st);
    }
    HM_TRY(rc);
    if (dtype == HM_F64) {
        if (small_index(b)) launch_digit_t<double, uint32_t>(b, t, d, p, st);
        else launch_digit_t<double, uint64_t>(b, t, d, p, st);
    } else {
        if (small_index(b)) launch_digit_t<float, uint32_t>(b, t, d, p, st);
        else launch_digit_t<float, uint64_t>(b, t, d, p, st);
    }
    HM_HIP(hipGetLastError());
    return HM_OK;
}

}  // namespace hm
