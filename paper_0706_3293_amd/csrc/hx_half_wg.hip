// Spin-1/2 block kernel with one workgroup per block (Sec. 4, Eq. (E-4-b)).
//
// The split is that of hx_half.hip: the rows with one high word h are a
// contiguous block of C(K, A - popcount(h)) rows, ordered like the low words.
// The kernels there give a wave its own rows and let it walk the bonds with
// one round of gathers after another.  For a few thousand blocks that is a
// chain of eight or more memory round trips on a chip with a wave or two per
// SIMD (12,870 rows: 12.8 us; 184,756 rows with all 190 bonds: 41 us), and the
// straddling bonds gather per lane.  Here a workgroup takes one block, a row
// per thread, and loads everything in one round: its own block, the blocks
// that its straddling bonds reach (one per distinct high site, whatever the
// number of bonds), all coalesced, into LDS, and the first rows of the
// high-word targets into registers; what follows reads LDS.  Tables are laid
// out per block, so the wave-uniform reads are one round of scalar loads too.
// The sums take the bonds in the order of hx_half_kernel in its own split at K0 low
// sites (bonds below K0 in list order, bonds above, straddling ones), whatever the
// split here, so the rows are equal bit for bit.  With K < K0 low sites a bond of
// any kind here may belong to any of the three there: first low and straddling
// bonds mixed (v < K0), then two lists of high-word bonds around the straddling
// ones with v >= K0.
//
// A Lanczos run without reorthogonalization takes its dots from wg_dots_kernel,
// item by item as hx_half_kernel's waves add them: past convergence such a run
// amplifies its roundings (all-to-all model, 20 sites, 300 steps: to 4e-9 of
// dE0/dJ), so rows and dots keep one order.
#include <algorithm>
#include <cstring>
#include <vector>

#include "device_common.h"
#include "hm_internal.h"

namespace hm {

int half_low_bits(const Basis *b);
int hx_half_grid(const Basis *b);
int hx_half_chain(const Basis *b);

constexpr int kWgMaxK = 12;
constexpr int kWgMaxHighBits = 20;
constexpr size_t kWgMaxLds = 64 * 1024;
constexpr size_t kWgMaxTables = (size_t)4 << 30;
constexpr int kWgPiece = 8;          // high-word targets of a piece

// Up to eight bonds of one kind, consecutive in the bond list, read with two or
// three wide scalar loads.  Low: m holds the two bits of every bond.
// Straddling: the bonds share their low site (m[0] its bit), slot holds the
// slot of every high site.
struct WgOp {
    int32_t n;           // bonds in use: 8, 4, 2 or 1
    uint32_t slot[2];    // a byte each
    int32_t straddle;    // 0: both sites in the low word
    uint32_t m[8];
    double c[8];         // -J/2
};

struct WgTables {
    int K = 0, threads = 256, smax = 0;
    int64_t n_blocks = 0;
    std::vector<uint16_t> rankL, unrankL;
    std::vector<uint32_t> off;       // by high word
    std::vector<uint32_t> blocks;    // high words with rows, in memory order
    int start[kWgMaxK + 2] = {0}, size[kWgMaxK + 2] = {0};
    void *mem = nullptr;
    uint16_t *d_rankL = nullptr, *d_unrankL = nullptr;
    uint32_t *d_off = nullptr, *d_blocks = nullptr;
    uint2 *d_items = nullptr;        // hx_half_kernel's items: first row, rows
    int n_items = 0;
};

static void free_wg(void *p) {
    auto *t = (WgTables *)p;
    if (!t) return;
    if (t->mem) (void)hipFree(t->mem);
    delete t;
}

struct WgBonds {
    void *mem = nullptr;
    WgOp *front = nullptr, *strad = nullptr; // below K0, straddling K0
    uint32_t *vbit = nullptr;                // bit of every straddling high site
    uint32_t *hdr = nullptr;                 // [block][hw]: off, size | start << 16, flips, bits of
                                             // the straddling high sites by slot, then per slot:
                                             // off, size (flips: of the two lists, 16 bits each)
    uint32_t *hoff = nullptr;                // [block][mh] target blocks of the high-word bonds,
    double *hcf = nullptr;                   // [block][mh] their -J/2: mh1 of the first list
    int nfront = 0, nstrad = 0, nslot = 0, mh1 = 0, mh = 0, hw = 0;
};
static void free_wg_bonds(void *p) {
    auto *d = (WgBonds *)p;
    if (!d) return;
    if (d->mem) (void)hipFree(d->mem);
    delete d;
}

struct WgArgs {
    const uint16_t *rankL, *unrankL;
    const WgOp *front, *strad;
    const uint32_t *hdr, *hoff;
    const double *hcf;
    uint32_t n_blocks;
    int K, nfront, nstrad, nslot, mh1, mh, hw, stride;
    double shift;
};

// W low-word bonds from LDS.
template <int W>
__device__ __forceinline__ void wg_low(const Const<WgOp> &op, uint32_t L, uint32_t r,
                                       const uint16_t *rankL, const double *xs, double xi,
                                       double &acc) {
    uint32_t idx[W];
    double xj[W];
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const uint32_t m = op.m[q], t = rankL[L ^ m];
        idx[q] = __popc(L & m) == 1 ? t : r;
    }
#pragma unroll
    for (int q = 0; q < W; ++q) xj[q] = xs[idx[q]];
#pragma unroll
    for (int q = 0; q < W; ++q) acc += op.c[q] * (xj[q] - xi);
}

// W straddling bonds of one low site: they flip where the low bit differs from
// the bond's high bit, which is the same for the whole block.
template <int W>
__device__ __forceinline__ void wg_straddle(const Const<WgOp> &op, uint32_t hmask, bool set,
                                            uint32_t rk, uint32_t r, int stride,
                                            const double *xs, double xi, double &acc) {
    double xj[W];
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const uint32_t slot = (op.slot[q / 4] >> (8 * (q % 4))) & 0xffu;
        const bool hset = (hmask >> slot) & 1u;
        xj[q] = xs[set != hset ? (slot + 1) * stride + rk : r];
    }
#pragma unroll
    for (int q = 0; q < W; ++q) acc += op.c[q] * (xj[q] - xi);
}

template <bool DOT, bool STORE>
__global__ __launch_bounds__(256) void hx_half_wg_kernel(
    const WgArgs g, const double *__restrict__ x, double *__restrict__ y,
    const double *__restrict__ prev, const LzStep step, double *__restrict__ partial,
    double *__restrict__ store) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[kLzLds];
    double *xs = reinterpret_cast<double *>(smem);
    uint16_t *rankL = reinterpret_cast<uint16_t *>(
        smem + ((size_t)(1 + g.nslot) * g.stride * sizeof(double) + 15) / 16 * 16);
    {
        const uint4 *s4 = reinterpret_cast<const uint4 *>(g.rankL);
        uint4 *d4 = reinterpret_cast<uint4 *>(rankL);
        for (int t = threadIdx.x; t < (1 << g.K) / 8; t += blockDim.x) d4[t] = s4[t];
    }
    double sigma = 1.0, cprev = 0.0;
    const double shift = g.shift;
    const Const<uint32_t> *hdrs = as_const(g.hdr), *hoffs = as_const(g.hoff);
    const Const<double> *hcfs = as_const(g.hcf);
    const Const<WgOp> *front = as_const(g.front), *strad = as_const(g.strad);
    double dot = 0.0;
    for (uint32_t it = blockIdx.x;; it += gridDim.x) {
        const bool any = it < g.n_blocks;
        if (!any && it != blockIdx.x) break;
        const Const<uint32_t> *hdr = hdrs + (size_t)(any ? it : 0) * g.hw;
        const uint32_t off = hdr[0], hmask = hdr[3];
        const int S = any ? (int)(hdr[1] & 0xffffu) : 0, cs = (int)(hdr[1] >> 16);
        const int nf = (int)(hdr[2] & 0xffffu), nc = (int)(hdr[2] >> 16);
        // one round of coalesced loads: this block and those its straddling
        // bonds reach
        for (int r = threadIdx.x; any && r < g.stride; r += blockDim.x) {
            double v = 0;
            if (r < S) v = load_at(x, off + (uint32_t)r);
            for (int s0 = 0; s0 < g.nslot; s0 += 4) {
                double t[4];
                bool in[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    in[s] = s0 + s < g.nslot && r < (int)hdr[5 + 2 * (s0 + s)];
                    if (in[s]) t[s] = load_at(x, hdr[4 + 2 * (s0 + s)] + (uint32_t)r);
                }
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    if (in[s]) xs[(1 + s0 + s) * g.stride + r] = t[s];
            }
            if (r < S) xs[r] = v;
        }
        // the step's scalars while the first round is on its way
        if (it == blockIdx.x) {
            double sg, cp;
            if (!lz_begin(step, red, sg, cp)) return;
            sigma = uniform(sg);
            cprev = uniform(cp);
            if (!any) break;
        }
        __syncthreads();
        const Const<uint32_t> *hoff = hoffs + (size_t)it * g.mh;
        const Const<double> *hcf = hcfs + (size_t)it * g.mh;
        for (int r0 = 0; r0 < S; r0 += blockDim.x) {
            const uint32_t r = (uint32_t)r0 + threadIdx.x;
            if ((int)r >= S) break;
            const uint32_t L = g.unrankL[cs + r];
            // the first pieces of high-word targets are on their way meanwhile
            double xh[kWgPiece], xc[kWgPiece];
#pragma unroll
            for (int q = 0; q < kWgPiece; ++q) xh[q] = q < g.mh1 ? load_at(x, hoff[q] + r) : 0.0;
#pragma unroll
            for (int q = 0; q < kWgPiece; ++q)
                xc[q] = g.mh1 + q < g.mh ? load_at(x, hoff[g.mh1 + q] + r) : 0.0;
            double pv = 0;
            if (prev) pv = load_at(prev, off + r);
            const double xi = xs[r];
            double acc = 0;
            auto straddle = [&](const Const<WgOp> &op) {
                const uint32_t m1 = op.m[0], rk = rankL[L ^ m1];
                const bool set = (L & m1) != 0;
                if (op.n == 8) wg_straddle<8>(op, hmask, set, rk, r, g.stride, xs, xi, acc);
                else if (op.n == 4) wg_straddle<4>(op, hmask, set, rk, r, g.stride, xs, xi, acc);
                else if (op.n == 2) wg_straddle<2>(op, hmask, set, rk, r, g.stride, xs, xi, acc);
                else wg_straddle<1>(op, hmask, set, rk, r, g.stride, xs, xi, acc);
            };
            // high-word bonds that flip for h, n of them from place `at` of the
            // block's list (padded with the own block and coefficient 0); the first
            // piece is loaded
            auto high = [&](int at, int n, double (&xj)[kWgPiece]) {
                for (int q0 = 0; q0 < n; q0 += kWgPiece) {
                    if (q0 > 0)
#pragma unroll
                        for (int q = 0; q < kWgPiece; ++q) xj[q] = load_at(x, hoff[at + q0 + q] + r);
#pragma unroll
                    for (int q = 0; q < kWgPiece; ++q) acc += hcf[at + q0 + q] * (xj[q] - xi);
                }
            };
            for (int o = 0; o < g.nfront; ++o) {
                const Const<WgOp> &op = front[o];
                if (op.straddle) straddle(op);
                else if (op.n == 8) wg_low<8>(op, L, r, rankL, xs, xi, acc);
                else if (op.n == 4) wg_low<4>(op, L, r, rankL, xs, xi, acc);
                else if (op.n == 2) wg_low<2>(op, L, r, rankL, xs, xi, acc);
                else wg_low<1>(op, L, r, rankL, xs, xi, acc);
            }
            high(0, nf, xh);
            for (int o = 0; o < g.nstrad; ++o) straddle(strad[o]);
            high(g.mh1, nc, xc);
            const double hv = shift * xi + acc;
            double w = sigma * hv;
            if (prev) w -= cprev * pv;
            y[off + r] = w;
            if constexpr (DOT) dot += w * (sigma * xi);
            if constexpr (STORE) store[off + r] = sigma * xi;
        }
        __syncthreads();       // the next block overwrites the slices
    }
    if constexpr (DOT) {
        const double s = block_sum(dot, red);
        if (threadIdx.x == 0) partial[blockIdx.x] = s;
    }
    lz_end(step, red, sigma, cprev);
}

// <w, v_k> as hx_half_kernel adds it: a wave's lanes go through its items in turn,
// a row each.  Needs the pass that wrote w and the step's scalars to be over.  A
// launch of 4 us, for what the rows' kernel saves (20 sites, 190 bonds: H x 41 ->
// 25 us).
__global__ __launch_bounds__(kBlock) void wg_dots_kernel(const uint2 *__restrict__ items,
                                                         uint32_t n_items,
                                                         const double *__restrict__ w,
                                                         const double *__restrict__ x,
                                                         const double *__restrict__ sigma_k,
                                                         double *__restrict__ partial) {
    const double sigma = *sigma_k;
    if (sigma == 0.0) return;
    __shared__ double red[16];
    const bool by_xcd = gridDim.x % kXcds == 0;
    const uint32_t x8 = by_xcd ? blockIdx.x % kXcds : 0, nw = kBlock / 64;
    const uint32_t wl = __builtin_amdgcn_readfirstlane(
        (by_xcd ? blockIdx.x / kXcds : blockIdx.x) * nw + (threadIdx.x >> 6));
    const uint32_t stride = (by_xcd ? gridDim.x / kXcds : gridDim.x) * nw;
    const uint32_t lane = threadIdx.x & 63;
    const Const<uint2> *it = as_const(items);
    double dot = 0.0;
    constexpr int U = 4;                          // items in flight
    for (uint32_t l = wl;; l += U * stride) {
        if ((by_xcd ? sweep_item(l, x8) : l) >= n_items) break;
        double a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t lu = l + u * stride, i = by_xcd ? sweep_item(lu, x8) : lu;
            const uint32_t row0 = i < n_items ? it[i].x : 0, rows = i < n_items ? it[i].y : 0;
            const uint32_t row = lane < rows ? row0 + lane : 0;
            const double wr = w[row], xr = x[row];
            a[u] = lane < rows ? wr : 0.0;
            b[u] = lane < rows ? sigma * xr : 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) dot = __builtin_fma(a[u], b[u], dot);
    }
    const double s = block_sum(dot, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// Rows of the block tables, one thread per block.
__global__ __launch_bounds__(kBlock) void wg_rows(const uint32_t *__restrict__ blocks, int64_t n,
                                                  const uint32_t *__restrict__ off, int K, int K0,
                                                  int A,
                                                  const int *__restrict__ cls,
                                                  const BondDev *__restrict__ bonds, int nb,
                                                  const uint32_t *__restrict__ vbit, int nslot,
                                                  int mh1, int mh, int hw,
                                                  uint32_t *__restrict__ hdr,
                                                  uint32_t *__restrict__ hoff,
                                                  double *__restrict__ hcf) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t h = blocks[i], own = off[h];
        const int aL = A - __popc(h);
        uint32_t *row = hdr + (size_t)i * hw;
        row[0] = own;
        row[1] = (uint32_t)cls[2 * aL + 1] | (uint32_t)cls[2 * aL] << 16;
        uint32_t hmask = 0;
        for (int s = 0; s < nslot; ++s) {
            const uint32_t t = h ^ vbit[s];
            const int a = A - __popc(t);
            const bool ok = a >= 0 && a <= K;
            row[4 + 2 * s] = ok ? off[t] : own;
            row[5 + 2 * s] = ok ? (uint32_t)cls[2 * a + 1] : 0u;
            hmask |= (h & vbit[s]) ? 1u << s : 0u;
        }
        row[3] = hmask;
        // the bonds that straddle K0 in the second list
        int c[2] = {0, 0};
        for (int b = 0; b < nb; ++b) {
            if (bonds[b].u < K) continue;
            const uint32_t m = 1u << (bonds[b].u - K) | 1u << (bonds[b].v - K);
            if (__popc(h & m) != 1) continue;
            const int list = bonds[b].u < K0 && bonds[b].v >= K0;
            const size_t at = (size_t)i * mh + (list ? mh1 + c[1]++ : c[0]++);
            hoff[at] = off[h ^ m];
            hcf[at] = bonds[b].mJ2;
        }
        row[2] = (uint32_t)c[0] | (uint32_t)c[1] << 16;
        for (int list = 0; list < 2; ++list)
            for (int q = (list ? mh1 : 0) + c[list]; q < (list ? mh : mh1); ++q) {
                hoff[(size_t)i * mh + q] = own;
                hcf[(size_t)i * mh + q] = 0;
            }
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
static int64_t choose2(int n, int k) {
    if (k < 0 || k > n) return 0;
    int64_t r = 1;
    for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
    return r;
}

// Low sites: blocks of at most 252 rows, a row per thread, and about as many
// blocks as rows of one for small N.  Measured (us per FP64 Lanczos step with the
// dots taken in this kernel, J1-J2 rings unless said, K = 8 / 9 / 10 / 11): N = 16 15.9 / 15.7 / 16.1 / 18.4;
// N = 18 20.1 / 16.8 / 16.4 / 19.7; N = 20 27.0 / 23.7 / 22.9 / 24.5; N = 20 with
// all bonds 47.8 / 41.0 / 36.3 / 43.5.
static int wg_low_bits(const Basis *b) { return std::min(10, (b->N + 2) / 2); }

static int64_t wg_blocks(const Basis *b) {
    const int K = wg_low_bits(b), nh = b->N - K;
    int64_t n = 0;
    for (int p = 0; p <= nh; ++p)
        if (b->A - p >= 0 && b->A - p <= K) n += choose2(nh, p);
    return n;
}

static int wg_threads(int K) {
    const int s = (int)choose2(K, K / 2);
    return s <= 64 ? 64 : s <= 128 ? 128 : 256;
}

int hx_wg_grid(const Basis *b) {
    int64_t g = std::min<int64_t>(wg_blocks(b), kMaxGrid);
    if (g >= kXcds) g -= g % kXcds;
    return (int)std::max<int64_t>(g, 1);
}

static void wg_counts(const Couplings *c, int K, int *nL, int *nH, int *nS, int *nslot,
                      uint32_t *vmask) {
    *nL = *nH = *nS = *nslot = 0;
    *vmask = 0;
    for (const BondDev &d : c->host) {
        if (d.u >= K) ++*nH;
        else if (d.v < K) ++*nL;
        else {
            ++*nS;
            *vmask |= 1u << (d.v - K);
        }
    }
    *nslot = __builtin_popcount(*vmask);
}

static size_t wg_lds(int K, int nslot) {
    return ((size_t)(1 + nslot) * choose2(K, K / 2) * sizeof(double) + 15) / 16 * 16 +
           ((size_t)2 << K);
}

// Where it is the automatic choice: FP64, up to kWgRows rows, blocks of
// kWgRowsPerBlock rows on average, no schedule asked for (that is one of
// hx_half.hip's kernels), and two items or more in turn for a wave of hx_half_kernel.
// Measured against hx_half_kernel (us per FP64 Lanczos step, the dots taken in either
// kernel): N = 16 15.7 / 20.7, N = 18 16.4 / 19.8, N = 20 22.9 / 24.7, N = 20 with all
// 190 bonds 36.3 / 51.7; N = 21 28 / 28, N = 22 42 / 37, N = 24 118 / 108, where the
// wave's own rows keep enough gathers in flight; N = 28, M = 10 (5 rows per block)
// 33 / 23.  One H x with its call, where a wave has one item: N = 8 with all bonds
// 25 / 20, N = 12 24 / 20 (all bonds 29 / 23), N = 13 24 / 22 (31 / 25), 16 sites and
// A = 3 24 / 22 (34 / 29); where it has more: N = 14 24 / 53, 16 sites and A = 4
// 27 / 47.  A run whose dots have a launch of their own chooses again among these
// (wg_items_pay in lanczos.hip).
constexpr int64_t kWgRows = (int64_t)1 << 18;
constexpr int64_t kWgRowsPerBlock = 48;
constexpr int kWgChain = 2;

bool wg_fits(const Basis *b, const Couplings *c, int dtype) {
    if (b->two_s != 1 || dtype != HM_F64 || b->N < 4 || b->dim > kWgRows) return false;
    if (b->half_K || b->half_block || b->half_R || b->half_staging || b->half_ipw) return false;
    const int K = wg_low_bits(b);
    if (b->N - K > kWgMaxHighBits) return false;
    const int64_t n = wg_blocks(b);
    // (small N: a block holds what there is)
    if (b->N > 16 && b->dim < kWgRowsPerBlock * n) return false;
    if (hx_half_chain(b) < kWgChain) return false;
    if (!c) return true;
    int nL, nH, nS, nslot;
    uint32_t vm;
    wg_counts(c, K, &nL, &nH, &nS, &nslot, &vm);
    return wg_lds(K, nslot) <= kWgMaxLds &&
           (size_t)n * ((nH + 16) * 12 + 64 + 8 * nslot) <= kWgMaxTables;
}

static int wg_prepare(Basis *b, WgTables **out) {
    if (b->wg_tables) {
        *out = (WgTables *)b->wg_tables;
        return HM_OK;
    }
    auto *t = new WgTables;
    const int K = t->K = wg_low_bits(b), nh = b->N - K, nlow = 1 << K;
    t->threads = wg_threads(K);
    t->rankL.resize(nlow);
    t->unrankL.resize(nlow);
    std::vector<int> fill(K + 1, 0);
    for (int a = 0, s = 0; a <= K; ++a) {
        t->start[a] = s;
        t->size[a] = (int)choose2(K, a);
        s += t->size[a];
    }
    for (int L = 0; L < nlow; ++L) {
        const int a = __builtin_popcount((unsigned)L);
        t->rankL[L] = (uint16_t)fill[a];
        t->unrankL[t->start[a] + fill[a]++] = (uint16_t)L;
    }
    t->smax = (int)choose2(K, K / 2);
    t->off.assign((size_t)1 << nh, 0);
    uint64_t o = 0;
    for (uint32_t h = 0; h < (uint32_t)t->off.size(); ++h) {
        const int a = b->A - __builtin_popcount(h);
        if (a < 0 || a > K) continue;
        t->off[h] = (uint32_t)o;
        t->blocks.push_back(h);
        o += (uint64_t)t->size[a];
    }
    if ((int64_t)o != b->dim) {
        delete t;
        return fail(HM_EINVAL, "internal: block sizes sum to %llu, dim %lld",
                    (unsigned long long)o, (long long)b->dim);
    }
    t->n_blocks = (int64_t)t->blocks.size();
    // the items of hx_half_kernel: 64 rows of a block of its split
    const int K0 = half_low_bits(b);
    std::vector<uint2> items;
    uint32_t row = 0;
    for (uint32_t h = 0; h < 1u << (b->N - K0); ++h) {
        const int S = (int)choose2(K0, b->A - __builtin_popcount(h));
        for (int c = 0; c < S; c += 64) items.push_back(uint2{row + c, (uint32_t)std::min(64, S - c)});
        row += S;
    }
    t->n_items = (int)items.size();
    auto al = [](size_t v) { return (v + 255) / 256 * 256; };
    const size_t o_un = al(nlow * 2), o_off = o_un + al(nlow * 2),
                 o_blk = o_off + al(t->off.size() * 4), o_it = o_blk + al(t->blocks.size() * 4),
                 total = o_it + al(items.size() * sizeof(uint2));
    std::vector<unsigned char> host(total);
    std::memcpy(host.data(), t->rankL.data(), nlow * 2);
    std::memcpy(host.data() + o_un, t->unrankL.data(), nlow * 2);
    std::memcpy(host.data() + o_off, t->off.data(), t->off.size() * 4);
    std::memcpy(host.data() + o_blk, t->blocks.data(), t->blocks.size() * 4);
    std::memcpy(host.data() + o_it, items.data(), items.size() * sizeof(uint2));
    hipError_t e = hipMalloc(&t->mem, total);
    if (e == hipSuccess) e = hipMemcpy(t->mem, host.data(), total, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        free_wg(t);
        return fail(e == hipErrorOutOfMemory ? HM_ENOMEM : HM_EDEVICE, "block kernel tables: %s",
                    hipGetErrorString(e));
    }
    unsigned char *m = (unsigned char *)t->mem;
    t->d_rankL = (uint16_t *)m;
    t->d_unrankL = (uint16_t *)(m + o_un);
    t->d_off = (uint32_t *)(m + o_off);
    t->d_blocks = (uint32_t *)(m + o_blk);
    t->d_items = (uint2 *)(m + o_it);
    b->wg_tables = t;
    b->wg_tables_free = free_wg;
    *out = t;
    return HM_OK;
}

static hipError_t wg_build(const Basis *b, const Couplings *c, const WgTables *t, WgBonds *d) {
    const int K = t->K;
    int nH;
    uint32_t vmask;
    int nL, nS;
    wg_counts(c, K, &nL, &nH, &nS, &d->nslot, &vmask);
    std::vector<uint32_t> vbit;
    for (int v = 0; v < 32; ++v)
        if (vmask >> v & 1) vbit.push_back(1u << v);
    // runs of low-word bonds, and of the straddling bonds of one low site, in
    // eights, fours, twos and ones
    const int K0 = half_low_bits(b);
    std::vector<const BondDev *> below, across;      // first site low; second below K0, or not
    int nH2 = 0;
    for (const BondDev &bd : c->host) {
        if (bd.u < K) (bd.v < K0 ? below : across).push_back(&bd);
        else if (bd.u < K0 && bd.v >= K0) ++nH2;
    }
    auto pieces = [&](const std::vector<const BondDev *> &v) {
        std::vector<WgOp> ops;
        for (size_t i = 0; i < v.size();) {
            const bool straddle = v[i]->v >= K;
            size_t n = 1;
            while (i + n < v.size() && (v[i + n]->v >= K) == straddle &&
                   (!straddle || v[i + n]->u == v[i]->u))
                ++n;
            WgOp op{};
            op.n = n >= 8 ? 8 : n >= 4 ? 4 : n >= 2 ? 2 : 1;
            op.straddle = straddle;
            if (straddle) op.m[0] = 1u << v[i]->u;
            for (int q = 0; q < op.n; ++q, ++i) {
                op.c[q] = v[i]->mJ2;
                if (!straddle) {
                    op.m[q] = 1u << v[i]->u | 1u << v[i]->v;
                    continue;
                }
                const int slot = __builtin_popcount(vmask & ((1u << (v[i]->v - K)) - 1u));
                op.slot[q / 4] |= (uint32_t)slot << (8 * (q % 4));
            }
            ops.push_back(op);
        }
        return ops;
    };
    const std::vector<WgOp> front = pieces(below), strad = pieces(across);
    d->nfront = (int)front.size();
    d->nstrad = (int)strad.size();
    auto padded = [](int n) { return (n + kWgPiece - 1) / kWgPiece * kWgPiece; };
    d->mh1 = padded(nH - nH2);
    d->mh = d->mh1 + padded(nH2);
    d->hw = (4 + 2 * d->nslot + 3 + 8) / 4 * 4;       // slot reads go in fours
    std::vector<int> cls(2 * (K + 1));
    for (int a = 0; a <= K; ++a) {
        cls[2 * a] = t->start[a];
        cls[2 * a + 1] = t->size[a];
    }
    auto al = [](size_t v) { return (v + 255) / 256 * 256; };
    size_t total = 0;
    auto add = [&](size_t bytes) {
        const size_t at = total;
        total += al(bytes + 64);
        return at;
    };
    const size_t nblk = (size_t)t->n_blocks;
    const size_t o_front = add(front.size() * sizeof(WgOp)),
                 o_str = add(strad.size() * sizeof(WgOp)), o_vb = add(vbit.size() * 4),
                 o_cls = add(cls.size() * 4), hostlen = total;
    const size_t o_hdr = add(nblk * d->hw * 4), o_hoff = add(nblk * d->mh * 4),
                 o_hcf = add(nblk * d->mh * sizeof(double));
    std::vector<unsigned char> host(hostlen);
    auto put = [&](size_t at, const void *p, size_t bytes) {
        if (bytes) std::memcpy(host.data() + at, p, bytes);
    };
    put(o_front, front.data(), front.size() * sizeof(WgOp));
    put(o_str, strad.data(), strad.size() * sizeof(WgOp));
    put(o_vb, vbit.data(), vbit.size() * 4);
    put(o_cls, cls.data(), cls.size() * 4);
    hipError_t e = hipMalloc(&d->mem, total);
    if (e == hipSuccess) e = hipMemcpy(d->mem, host.data(), hostlen, hipMemcpyHostToDevice);
    if (e != hipSuccess) return e;
    unsigned char *m = (unsigned char *)d->mem;
    d->front = (WgOp *)(m + o_front);
    d->strad = (WgOp *)(m + o_str);
    d->vbit = (uint32_t *)(m + o_vb);
    d->hdr = (uint32_t *)(m + o_hdr);
    d->hoff = (uint32_t *)(m + o_hoff);
    d->hcf = (double *)(m + o_hcf);
    const int grid = (int)std::min<int64_t>((t->n_blocks + kBlock - 1) / kBlock, kMaxGrid);
    hipLaunchKernelGGL(wg_rows, dim3(grid), dim3(kBlock), 0, nullptr, t->d_blocks, t->n_blocks,
                       t->d_off, K, K0, b->A, (const int *)(m + o_cls), c->dev, c->nb, d->vbit,
                       d->nslot, d->mh1, d->mh, d->hw, d->hdr, d->hoff, d->hcf);
    e = hipGetLastError();
    // other streams may use the tables from now on
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    return e;
}

static int wg_get(Basis *b, const Couplings *c, hipStream_t st, WgTables **tout,
                  const WgBonds **bout) {
    std::lock_guard<std::mutex> lock(b->mu);
    HM_TRY(device_prepare(b));
    auto *cc = const_cast<Couplings *>(c);
    if (!cc->wg && is_capturing(st)) return HM_ENOMEM;
    HM_TRY(wg_prepare(b, tout));
    if (!cc->wg) {
        auto *d = new WgBonds;
        const hipError_t e = wg_build(b, c, *tout, d);
        if (e != hipSuccess) {
            free_wg_bonds(d);
            return fail(e == hipErrorOutOfMemory ? HM_ENOMEM : HM_EDEVICE, "block kernel bonds: %s",
                        hipGetErrorString(e));
        }
        cc->wg = d;
        cc->wg_free = free_wg_bonds;
    }
    *bout = (const WgBonds *)cc->wg;
    return HM_OK;
}

int wg_prepare_tables(Basis *b, const Couplings *c) {
    WgTables *t = nullptr;
    const WgBonds *d = nullptr;
    return wg_get(b, c, nullptr, &t, &d);
}

static void launch_rows(const Basis *b, const Couplings *c, const WgTables *t, const WgBonds *d,
                        const HxPass &p, hipStream_t st) {
    WgArgs g{};
    g.rankL = t->d_rankL;
    g.unrankL = t->d_unrankL;
    g.front = d->front;
    g.strad = d->strad;
    g.hdr = d->hdr;
    g.hoff = d->hoff;
    g.hcf = d->hcf;
    g.n_blocks = (uint32_t)t->n_blocks;
    g.K = t->K;
    g.nfront = d->nfront;
    g.nstrad = d->nstrad;
    g.nslot = d->nslot;
    g.mh1 = d->mh1;
    g.mh = d->mh;
    g.hw = d->hw;
    g.stride = t->smax;
    g.shift = c->diag_shift;
    const int grid = hx_wg_grid(b);
    const size_t lds = wg_lds(t->K, d->nslot);
    const double *x = (const double *)p.x, *pr = (const double *)p.p;
    double *y = (double *)p.y, *store = (double *)p.store;
#define HM_LAUNCH(D, S)                                                                      \
    hipLaunchKernelGGL((hx_half_wg_kernel<D, S>), dim3(grid), dim3(t->threads), lds, st, g,  \
                       x, y, pr, p.step, p.partial, store)
    const bool dot = p.partial != nullptr, sto = store != nullptr;
    if (!dot && !sto) HM_LAUNCH(false, false);
    else if (dot && !sto) HM_LAUNCH(true, false);
    else if (!dot && sto) HM_LAUNCH(false, true);
    else HM_LAUNCH(true, true);
#undef HM_LAUNCH
}

// items: the dots of hx_half_kernel, in a launch of their own.
int launch_hx_wg(const Basis *cb, const Couplings *c, bool items, const HxPass &p,
                 hipStream_t st) {
    Basis *b = const_cast<Basis *>(cb);
    WgTables *t = nullptr;
    const WgBonds *d = nullptr;
    const int rc = wg_get(b, c, st, &t, &d);
    if (rc == HM_ENOMEM && !p.step.sigma) {
        // no memory for the tables, or a product captured before its first use
        clear_error();
        (void)hipGetLastError();
        return launch_hx_built(b, c, HM_F64, p, st);
    }
    HM_TRY(rc);
    HxPass rows = p;
    if (items) rows.partial = nullptr;
    launch_rows(b, c, t, d, rows, st);
    if (items && p.partial)
        hipLaunchKernelGGL(wg_dots_kernel, dim3(hx_half_grid(b)), dim3(kBlock), 0, st, t->d_items,
                           (uint32_t)t->n_items, (const double *)p.y, (const double *)p.x,
                           p.step.sigma + p.step.k, p.partial);
    HM_HIP(hipGetLastError());
    return HM_OK;
}

}  // namespace hm
