// Batched Lanczos: many independent problems (basis, couplings) with up to 16
// start vectors each, every step one set of launches for all of them.
//
// Vectors are stored in FP32 as [dim][NV] rows (NV = 1, 2, 4, 8 or 16), so the
// multi-vector product H X decodes each basis state and encodes each target
// once (Sec. 3.1, 3.2) and gathers the NV entries of a target row with
// contiguous 16-byte loads; with 8 or 16 vectors a row is spread over 2 or 4
// lanes.  Dots and norms are FP64.  Each (instance, vector) pair runs its own
// recurrence (Paige's ordering, as hm_lanczos):
//
//   init  norms of the start vectors, r_0 = v0 / |v0|              (3 launches)
//   step  A:  w = sigma H r - cprev r_prev, alpha partials
//         A': alpha per pair
//         B:  w -= alpha sigma r, |w|^2 partials
//         B': beta, breakdown test, sigma and cprev of the next step
// Work items are 256-row tiles of one instance; a workgroup takes chunks of
// consecutive items and reduces once per run of items of one instance, so every
// sum has a fixed order for a given chunk.  Launches order the passes: a launch
// of a few microseconds costs less than a barrier over the whole grid (8, 15 and
// 28 us on 256, 512 and 1024 workgroups), and the grid need not be resident.
#include <algorithm>
#include <cmath>
#include <vector>

#include "device_common.h"
#include "hm_internal.h"

namespace hm {

constexpr int kBatchBlock = 256;
constexpr int kBatchMaxVec = 16;
constexpr size_t kBatchPrefixLds = 24 * 1024;

struct InstDesc {
    int N, A, two_s, nb;
    uint32_t dim;
    uint32_t vec_off;          // first row of this instance in the stacked vectors
    uint32_t item_first, item_count;
    const uint32_t *prefix;    // 32-bit prefix table of the basis
    const double *ladder;
    const BondDev *bonds;
    const double *v0;          // [dim][nvec] FP64 start vectors
};

struct Item {
    uint32_t inst, row0;
};

constexpr int kStageWaves = kBatchBlock / 64;

// Items a workgroup takes at a time by default: one while the batch has few (the
// workgroups balance better), two later (half the reductions).  us for 8 steps
// with chunk 1 / 2 / 4: 2,700 items 900 / 963 / 1004; 4,600 items 617 / 619 / 716;
// 16,600 items 2171 / 1964 / 2045; 43,800 items 13131 / 12903 / 13001.
constexpr int kFewItems = 8192;
static int default_chunk(int n_items) { return n_items <= kFewItems ? 1 : 2; }

struct BatchArgs {
    const InstDesc *inst;
    const Item *items;
    int ninst, n_items, nvec, steps;
    double tol;
    float *r[3];
    double *partial;           // [n_items][NV], the first item of a segment holds its sum
    double *alpha, *beta;      // [npairs][steps]
    double *E0;                // [npairs]
    double *sigma, *cprev;     // [npairs][steps + 1]
    double *scale, *norm0;     // [npairs]
    int *stopped;              // [npairs]: steps done at breakdown, 0 while running
    int max_prefix;            // entries of the largest prefix table
    int chunk;                 // items a workgroup takes at a time
};

template <int NV>
__device__ __forceinline__ void load_row(const float *__restrict__ p, float (&v)[NV]) {
    if constexpr (NV % 4 == 0) {
#pragma unroll
        for (int q = 0; q < NV / 4; ++q) {
            const float4 t = reinterpret_cast<const float4 *>(p)[q];
            v[4 * q] = t.x;
            v[4 * q + 1] = t.y;
            v[4 * q + 2] = t.z;
            v[4 * q + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = p[q];
    }
}

template <int NV>
__device__ __forceinline__ void store_row(float *__restrict__ p, const float (&v)[NV]) {
    if constexpr (NV % 4 == 0) {
#pragma unroll
        for (int q = 0; q < NV / 4; ++q)
            reinterpret_cast<float4 *>(p)[q] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2],
                                                           v[4 * q + 3]);
    } else {
#pragma unroll
        for (int q = 0; q < NV; ++q) p[q] = v[q];
    }
}

// Lanes per row in the two row passes: with 8 or 16 vectors a row is split
// over NV/4 lanes of 4 vectors (16 bytes) each, so the lanes of a wave read
// whole 64-byte rows together (a 64-lane load touches 16 lines, not 64).
template <int NV>
constexpr int lanes_per_row() { return NV >= 8 ? NV / 4 : 1; }

// FP64 partials of NV columns when G lanes share a row: lane l holds the
// V = NV / G columns starting at (l % G) V.  A fixed butterfly over the lanes of
// one column group (offsets 32 down to G), then thread q < NV adds the wave sums
// of column q in wave order.
template <int NV, int G>
__device__ __forceinline__ void item_partials_g(double (&v)[NV / G], double *stage,
                                                double *out) {
    constexpr int V = NV / G;
#pragma unroll
    for (int off = 32; off >= G; off >>= 1) {
#pragma unroll
        for (int q = 0; q < V; ++q) v[q] += __shfl_xor(v[q], off, 64);
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane < G) {
#pragma unroll
        for (int q = 0; q < V; ++q) stage[wid * NV + lane * V + q] = v[q];
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        double s = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += stage[w * NV + threadIdx.x];
        out[threadIdx.x] = s;
    }
    __syncthreads();
}

// Row differences of the two ladder moves of bond (u, v) in one walk over the
// prefix table: dn = 1 lowers u and raises v, up = 1 raises u and lowers v; with
// 0 (a move that is not allowed) the difference is 0 and every read is the row's
// own entry.
template <int B>
__device__ __forceinline__ void pair_deltas(uint64_t st, int u, int v, int dn, int up,
                                            const Prefix<uint32_t> &P, uint32_t &d_dn,
                                            uint32_t &d_up) {
    int Ap = digit_sum_upto<B>(st, u);
    const int au = digit_at<B>(st, u);
    uint32_t base = P.at(u + 1, Ap, au);
    d_dn = P.at(u + 1, Ap - dn, au - dn) - base;
    d_up = P.at(u + 1, Ap + up, au + up) - base;
    for (int p = u + 1; p < v; ++p) {
        const int ap = digit_at<B>(st, p);
        Ap += ap;
        base = P.at(p + 1, Ap, ap);
        d_dn += P.at(p + 1, Ap - dn, ap) - base;
        d_up += P.at(p + 1, Ap + up, ap) - base;
    }
    const int av = digit_at<B>(st, v);
    Ap += av;
    base = P.at(v + 1, Ap, av);
    d_dn += P.at(v + 1, Ap, av + dn) - base;
    d_up += P.at(v + 1, Ap, av - up) - base;
}

// Chunks of a.chunk consecutive items.  Within a chunk, consecutive items of one
// instance form a segment: threads add their rows' FP64 contributions over the
// segment and the workgroup reduces once per segment, into the slot of the
// segment's first item.
__device__ __forceinline__ int chunk_count(const BatchArgs &a) {
    return (a.n_items + a.chunk - 1) / a.chunk;
}

// Chunk of position t: workgroups t, t + 8, ... run on one XCD, which so sweeps a
// range of consecutive chunks and finds most gathered rows in its own L2.
__device__ __forceinline__ int chunk_at(int t, int n) {
    const int q = n / kXcds, rem = n % kXcds, x = t % kXcds;
    return x * q + min(x, rem) + t / kXcds;
}

// item -> (instance, first row): the instance is the last one that starts at or
// before the item.
__global__ __launch_bounds__(kBatchBlock) void batch_items_kernel(BatchArgs a, Item *items) {
    const uint32_t it = blockIdx.x * kBatchBlock + threadIdx.x;
    if (it >= (uint32_t)a.n_items) return;
    int lo = 0, hi = a.ninst;
    while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (a.inst[mid].item_first <= it) lo = mid;
        else hi = mid;
    }
    items[it] = Item{(uint32_t)lo, (it - a.inst[lo].item_first) * kBatchBlock};
}

// |v0|^2 partials per segment.  Thread t takes column t % NV of the rows
// t / NV, t / NV + 256 / NV, ..., so that a wave reads consecutive entries.
template <int NV>
__global__ __launch_bounds__(kBatchBlock) void batch_norm_kernel(BatchArgs a) {
    __shared__ double stage[kStageWaves * NV];
    const int n_chunks = chunk_count(a), q = threadIdx.x % NV;
    const uint32_t r0 = threadIdx.x / NV;
    double s[1] = {0.0};
    for (int t = blockIdx.x; t < n_chunks; t += gridDim.x) {
        const int c = chunk_at(t, n_chunks), i0 = c * a.chunk, i1 = min(i0 + a.chunk, a.n_items);
        int seg = i0;
        for (int it = i0; it < i1; ++it) {
            const Const<InstDesc> &d = as_const(a.inst)[as_const(a.items)[it].inst];
            const uint32_t i = as_const(a.items)[it].row0 + r0, dim = d.dim;
            const double *v0 = d.v0;
            double v[NV];
#pragma unroll
            for (int t = 0; t < NV; ++t) {
                const uint32_t row = i + t * (kBatchBlock / NV);
                v[t] = row < dim && q < a.nvec ? v0[(size_t)row * a.nvec + q] : 0.0;
            }
#pragma unroll
            for (int t = 0; t < NV; ++t) s[0] += v[t] * v[t];
            if (it + 1 == i1 || (uint32_t)(it + 1) == d.item_first + d.item_count) {
                item_partials_g<NV, NV>(s, stage, a.partial + (size_t)seg * NV);
                s[0] = 0.0;
                seg = it + 1;
            }
        }
    }
}

// r_0 = v0 / |v0|, threads as above.
template <int NV>
__global__ __launch_bounds__(kBatchBlock) void batch_start_kernel(BatchArgs a) {
    const int q = threadIdx.x % NV;
    const uint32_t r0 = threadIdx.x / NV;
    for (int it = blockIdx.x; it < a.n_items; it += gridDim.x) {
        const int inst = as_const(a.items)[it].inst;
        const Const<InstDesc> &d = as_const(a.inst)[inst];
        const uint32_t i = as_const(a.items)[it].row0 + r0, dim = d.dim;
        const double *v0 = d.v0;
        float *out = a.r[0] + (size_t)d.vec_off * NV + q;
        const bool live = q < a.nvec && a.stopped[inst * NV + q] == 0;
        const double norm = a.norm0[inst * NV + q];
        double v[NV];
#pragma unroll
        for (int t = 0; t < NV; ++t) {
            const uint32_t row = i + t * (kBatchBlock / NV);
            v[t] = live && row < dim ? v0[(size_t)row * a.nvec + q] : 0.0;
        }
#pragma unroll
        for (int t = 0; t < NV; ++t) {
            const uint32_t row = i + t * (kBatchBlock / NV);
            if (row < dim) out[(size_t)row * NV] = live ? (float)(v[t] / norm) : 0.0f;
        }
    }
}

// The sums of one instance's segments, and what follows from them for its NV
// pairs: the start norms (kInit), alpha_k (kAlpha), or beta_k, the breakdown test
// and the scalars of step k + 1 (kBeta).  One workgroup per instance: thread t
// adds the slots t / NV, t / NV + 1024 / NV, ... of column t % NV, 8 loads in
// flight; then a fixed tree.
enum { kInit, kAlpha, kBeta };
constexpr int kPairBlock = 1024;

template <int NV, int MODE>
__global__ __launch_bounds__(kPairBlock) void batch_pairs_kernel(BatchArgs a, int k) {
    __shared__ double stage[kPairBlock / 64 * NV];
    const int inst = blockIdx.x;
    const int first = (int)a.inst[inst].item_first, count = (int)a.inst[inst].item_count;
    const int c0 = first / a.chunk, slots = (first + count - 1) / a.chunk - c0 + 1;
    const int q = threadIdx.x % NV;
    auto slot = [&](int s) {
        return a.partial[(size_t)(s == 0 ? first : (c0 + s) * a.chunk) * NV + q];
    };
    constexpr int U = 8, S = kPairBlock / NV;
    double sum = 0.0;
    int s = threadIdx.x / NV;
    for (; s + (U - 1) * S < slots; s += U * S) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = slot(s + u * S);
#pragma unroll
        for (int u = 0; u < U; ++u) sum += v[u];
    }
    for (; s < slots; s += S) sum += slot(s);
#pragma unroll
    for (int off = 32; off >= NV; off >>= 1) sum += __shfl_xor(sum, off, 64);
    if ((threadIdx.x & 63) < NV) stage[threadIdx.x / 64 * NV + q] = sum;
    __syncthreads();
    if (threadIdx.x >= NV) return;
    sum = 0.0;
    for (int w = 0; w < kPairBlock / 64; ++w) sum += stage[w * NV + q];
    const int p = inst * NV + q;
    const size_t o = (size_t)p * (a.steps + 1);
    if (MODE == kInit) {
        const bool live = q < a.nvec && sum > 0.0;
        a.norm0[p] = sqrt(sum);
        a.scale[p] = 0.0;
        a.stopped[p] = live ? 0 : -1;
        a.sigma[o] = live ? 1.0 : 0.0;
        a.cprev[o] = 0.0;
    } else if (MODE == kAlpha) {
        a.alpha[(size_t)p * a.steps + k] = sum;
    } else {
        double b = sqrt(sum), sigma = 0.0, cprev = 0.0;
        if (a.stopped[p] != 0) {
            b = 0.0;
        } else {
            const double sc = fmax(a.scale[p], fmax(fabs(a.alpha[(size_t)p * a.steps + k]), b));
            a.scale[p] = sc;
            if (!(b > a.tol * sc)) {
                a.stopped[p] = k + 1;
            } else {
                sigma = 1.0 / b;
                cprev = b * a.sigma[o + k];
            }
        }
        a.beta[(size_t)p * a.steps + k] = b;
        a.sigma[o + k + 1] = sigma;
        a.cprev[o + k + 1] = cprev;
    }
}

// Pass A.  A wave takes 64 rows of an item in two phases.  First every lane
// decodes a row and walks the bonds, writing the moves that are allowed into the
// row's list in LDS (kList moves; a bond that may not fit any more empties the
// lists first).  Then the G lanes of a row read its list and gather the target
// rows, 8 in flight.  Only allowed moves are gathered (spin 1, 14 sites: 12 of
// 26).  Bound by decoding and encoding: 2,100 vector instructions per 64 rows,
// 60 % of what the units can issue, with 4 waves per SIMD (lists and registers).
// 64 spin-1 chains of 8 to 14 sites, 11.2 M rows of 16 vectors: 1.09 ms (2.0 TB/s
// of the 2.15 GB that have to move), a step 1.54 ms; with every move gathered
// (coefficient 0 for the others) and one barrier per pass a step took 2.3 ms.
constexpr int kList = 16;

template <int NV, int B>
__global__ __launch_bounds__(kBatchBlock) void batch_hx_kernel(BatchArgs a, int k) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double sc_sigma[NV], sc_c[NV];
    // the lists of a wave's rows: move m of row r at [m * 64 + r]
    __shared__ uint2 lists[kBatchBlock / 64][kList * 64];
    __shared__ double stage[kStageWaves * NV];
    uint32_t *P = reinterpret_cast<uint32_t *>(smem);
    double *F = reinterpret_cast<double *>(smem + ((a.max_prefix * 4 + 15) / 16) * 16);
    // G lanes per row, this lane's V columns start at gq
    constexpr int G = lanes_per_row<NV>(), V = NV / G;
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int gq = lane % G * V;
    uint2 *L = lists[wid];
    const float *__restrict__ rk = a.r[k % 3];
    const float *__restrict__ rp = a.r[(k + 2) % 3];
    float *__restrict__ w = a.r[(k + 1) % 3];
    double dacc[V];
#pragma unroll
    for (int q = 0; q < V; ++q) dacc[q] = 0.0;
    int loaded = -1;   // instance whose tables are in LDS
    const int n_chunks = chunk_count(a);
    for (int t = blockIdx.x; t < n_chunks; t += gridDim.x) {
        const int c = chunk_at(t, n_chunks), i0 = c * a.chunk, i1 = min(i0 + a.chunk, a.n_items);
        int seg = i0;
        for (int it = i0; it < i1; ++it) {
            const int inst = as_const(a.items)[it].inst;
            const Const<InstDesc> &d = as_const(a.inst)[inst];
            const int iN = d.N, iA = d.A, two_s = d.two_s, nb = d.nb;
            const uint32_t dim = d.dim, vec_off = d.vec_off;
            // a new instance starts a segment; the previous segment ended with
            // a workgroup barrier, so nobody still reads what is replaced here
            if (inst != loaded) {
                const uint32_t *prefix = d.prefix;
                const double *ladder = d.ladder;
                const int plen = iN * (iA + 1) * (two_s + 1);
                for (int t = threadIdx.x; t < plen; t += kBatchBlock) P[t] = prefix[t];
                for (int t = threadIdx.x; t < two_s + 2; t += kBatchBlock) F[t] = ladder[t];
                if (threadIdx.x < NV) {
                    const int p = inst * NV + threadIdx.x;
                    sc_sigma[threadIdx.x] = a.sigma[(size_t)p * (a.steps + 1) + k];
                    sc_c[threadIdx.x] = a.cprev[(size_t)p * (a.steps + 1) + k];
                }
                loaded = inst;
                __syncthreads();
            }
            const Const<BondDev> *bonds = as_const((const BondDev *)d.bonds);
            const Prefix<uint32_t> pv{P, iA + 1, two_s + 1};
            const float *__restrict__ xr = rk + (size_t)vec_off * NV;
            const uint32_t base = as_const(a.items)[it].row0 + wid * 64;
            if (base < dim) {
                const uint32_t i = base + lane;
                const bool live = i < dim;
                const uint64_t st = live ? unrank_state<uint32_t, B>(i, pv, iN, iA, two_s) : 0;
                // the diagonal in G partial sums, bond b in number (b % 4) G / 4
                float dg[G];
#pragma unroll
                for (int g = 0; g < G; ++g) dg[g] = 0.0f;
                float acc[G][V];
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int q = 0; q < V; ++q) acc[g][q] = 0.0f;
                int cnt = 0;
                // gathers the listed moves of sub-row g (row g * 64 / G + lane / G
                // of the wave), in list order
                auto gather = [&](int g) {
                    const int r = g * (64 / G) + lane / G;
                    const int n = G == 1 ? cnt : __shfl(cnt, r, 64);
                    for (int m = 0; m < n; m += 8) {
                        uint2 e[8];
                        float xj[8][V];
                        const bool more = m + 4 < n;
#pragma unroll
                        for (int t = 0; t < 8; ++t) e[t] = L[(m + t) % kList * 64 + r];
#pragma unroll
                        for (int t = 0; t < 4; ++t)
                            load_row<V>(xr + (size_t)e[t].x * NV + gq, xj[t]);
                        if (more)
#pragma unroll
                            for (int t = 4; t < 8; ++t)
                                load_row<V>(xr + (size_t)e[t].x * NV + gq, xj[t]);
#pragma unroll
                        for (int t = 0; t < 4; ++t)
#pragma unroll
                            for (int q = 0; q < V; ++q)
                                acc[g][q] += __uint_as_float(e[t].y) * xj[t][q];
                        if (more)
#pragma unroll
                            for (int t = 4; t < 8; ++t)
#pragma unroll
                                for (int q = 0; q < V; ++q)
                                    acc[g][q] += __uint_as_float(e[t].y) * xj[t][q];
                    }
                };
                // lists filled up to a multiple of 4 and seen by the whole wave
                auto close = [&]() {
                    while (cnt & 3) L[cnt++ * 64 + lane] = make_uint2(i, 0u);
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                };
                for (int b = 0; b < nb; ++b) {
                    if (__any(cnt > kList - 2)) {
                        close();
#pragma unroll
                        for (int g = 0; g < G; ++g) gather(g);
                        __builtin_amdgcn_wave_barrier();
                        cnt = 0;
                    }
                    const int u = bonds[b].u, v = bonds[b].v;
                    const double mJ2 = bonds[b].mJ2;
                    const float mJ4 = (float)bonds[b].mJ4;
                    const int au = digit_at<B>(st, u), av = digit_at<B>(st, v);
                    const float z = (float)((two_s - 2 * au) * (two_s - 2 * av));
#pragma unroll
                    for (int g = 0; g < G; ++g)
                        if ((b & 3) * G / 4 == g) dg[g] += mJ4 * z;
                    const int dn = live && au >= 1 && av < two_s;
                    const int up = live && av >= 1 && au < two_s;
                    uint32_t d_dn, d_up;
                    pair_deltas<B>(st, u, v, dn, up, pv, d_dn, d_up);
                    if (dn)
                        L[cnt++ * 64 + lane] = make_uint2(
                            i + d_dn, __float_as_uint((float)(mJ2 * F[au] * F[av + 1])));
                    if (up)
                        L[cnt++ * 64 + lane] = make_uint2(
                            i + d_up, __float_as_uint((float)(mJ2 * F[av] * F[au + 1])));
                }
                close();
                float diag = 0.0f;
                if constexpr (G == 1) {
                    diag = dg[0];
                } else {
#pragma unroll
                    for (int g = 0; g < G; ++g) diag += dg[g];
                }
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int r = g * (64 / G) + lane / G;
                    const float dr = G == 1 ? diag : __shfl(diag, r, 64);
                    const uint32_t ir = base + r;
                    const bool rl = ir < dim;
                    float xi[V], prv[V];
                    const size_t row = ((size_t)vec_off + ir) * NV + gq;
                    if (rl) {
                        load_row<V>(rk + row, xi);
                        if (k > 0) load_row<V>(rp + row, prv);
                    }
                    gather(g);
                    if (rl) {
                        float out[V];
#pragma unroll
                        for (int q = 0; q < V; ++q) {
                            const double hv = (double)(dr * xi[q] + acc[g][q]);
                            double wq = sc_sigma[gq + q] * hv;
                            if (k > 0) wq -= sc_c[gq + q] * (double)prv[q];
                            out[q] = (float)wq;
                            dacc[q] += (double)out[q] * (sc_sigma[gq + q] * (double)xi[q]);
                        }
                        store_row<V>(w + row, out);
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
            if (it + 1 == i1 || (uint32_t)(it + 1) == d.item_first + d.item_count) {
                item_partials_g<NV, G>(dacc, stage, a.partial + (size_t)seg * NV);
#pragma unroll
                for (int q = 0; q < V; ++q) dacc[q] = 0.0;
                seg = it + 1;
            }
        }
    }
}

// Pass B: w -= alpha sigma r_k; |w|^2 partials.  Bound by memory.
template <int NV>
__global__ __launch_bounds__(kBatchBlock) void batch_update_kernel(BatchArgs a, int k) {
    constexpr int G = lanes_per_row<NV>(), V = NV / G;
    __shared__ double sc_a[NV];
    __shared__ double stage[kStageWaves * NV];
    const int gq = (int)(threadIdx.x % G) * V;
    const float *__restrict__ rk = a.r[k % 3];
    float *__restrict__ w = a.r[(k + 1) % 3];
    double ss[V];
#pragma unroll
    for (int q = 0; q < V; ++q) ss[q] = 0.0;
    int loaded = -1;
    const int n_chunks = chunk_count(a);
    for (int t = blockIdx.x; t < n_chunks; t += gridDim.x) {
        const int c = chunk_at(t, n_chunks), i0 = c * a.chunk, i1 = min(i0 + a.chunk, a.n_items);
        int seg = i0;
        for (int it = i0; it < i1; ++it) {
            const int inst = as_const(a.items)[it].inst;
            const uint32_t row0 = as_const(a.items)[it].row0;
            const Const<InstDesc> &d = as_const(a.inst)[inst];
            const uint32_t dim = d.dim, vec_off = d.vec_off;
            if (inst != loaded) {
                if (threadIdx.x < NV) {
                    const int p = inst * NV + threadIdx.x;
                    sc_a[threadIdx.x] = a.alpha[(size_t)p * a.steps + k] *
                                        a.sigma[(size_t)p * (a.steps + 1) + k];
                }
                loaded = inst;
                __syncthreads();
            }
            float wv[G][V], rv[G][V];
#pragma unroll
            for (int sub = 0; sub < G; ++sub) {
                const uint32_t i = row0 + sub * (kBatchBlock / G) + threadIdx.x / G;
                if (i >= dim) continue;
                const size_t row = ((size_t)vec_off + i) * NV + gq;
                load_row<V>(w + row, wv[sub]);
                load_row<V>(rk + row, rv[sub]);
            }
#pragma unroll
            for (int sub = 0; sub < G; ++sub) {
                const uint32_t i = row0 + sub * (kBatchBlock / G) + threadIdx.x / G;
                if (i >= dim) continue;
#pragma unroll
                for (int q = 0; q < V; ++q) {
                    wv[sub][q] = (float)((double)wv[sub][q] - sc_a[gq + q] * (double)rv[sub][q]);
                    ss[q] += (double)wv[sub][q] * (double)wv[sub][q];
                }
                store_row<V>(w + ((size_t)vec_off + i) * NV + gq, wv[sub]);
            }
            if (it + 1 == i1 || (uint32_t)(it + 1) == d.item_first + d.item_count) {
                item_partials_g<NV, G>(ss, stage, a.partial + (size_t)seg * NV);
#pragma unroll
                for (int q = 0; q < V; ++q) ss[q] = 0.0;
                seg = it + 1;
            }
        }
    }
}

// E0 of every pair: the lowest eigenvalue of its tridiagonal matrix by Sturm
// counts, one wave per pair.  The lanes count at 64 points inside the bracket, so
// a round narrows it 65 times (bisection one pair after the other on the host
// took 2.6 us a pair at 8 steps); rounds go on until no number lies between the
// ends.
__global__ __launch_bounds__(kBatchBlock) void batch_ground_kernel(BatchArgs a, int npairs) {
    const int p = __builtin_amdgcn_readfirstlane(
        blockIdx.x * (kBatchBlock / 64) + (threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    if (p >= npairs) return;
    const double *al = a.alpha + (size_t)p * a.steps, *be = a.beta + (size_t)p * a.steps;
    const int stop = a.stopped[p], n = stop > 0 ? stop : stop < 0 ? 0 : a.steps;
    double lo = 1e300, hi = -1e300;
    for (int i = lane; i < n; i += 64) {
        const double d = (i > 0 ? fabs(be[i - 1]) : 0.0) + (i + 1 < n ? fabs(be[i]) : 0.0);
        lo = fmin(lo, al[i] - d);
        hi = fmax(hi, al[i] + d);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, off, 64));
        hi = fmax(hi, __shfl_xor(hi, off, 64));
    }
    const double span = fmax(fabs(lo), fabs(hi));
    lo -= 1e-12 * span + 1e-300;
    hi += 1e-12 * span + 1e-300;
    for (int round = 0; round < 2000 && n > 0; ++round) {
        const double mid = 0.5 * (lo + hi);
        if (!(mid > lo && mid < hi)) break;
        const double x = fmin(fmax(lo + (hi - lo) * ((lane + 1) / 65.0), lo), hi);
        bool below = false;   // an eigenvalue below x
        double q = 1.0, bb = 0.0;
        for (int i = 0; i < n; ++i) {
            q = (al[i] - x) - bb / q;
            if (q == 0.0) q = -1e-300;
            below |= q < 0.0;
            bb = be[i] * be[i];
        }
        const uint64_t m = __ballot(below);
        const int f = m ? __ffsll((unsigned long long)m) - 1 : 64;   // first point above E0
        const double below_f = __shfl(x, f > 0 ? f - 1 : 0, 64), at_f = __shfl(x, f & 63, 64);
        const double lo1 = f > 0 ? below_f : lo, hi1 = f < 64 ? at_f : hi;
        if (lo1 == lo && hi1 == hi) {   // the points rounded to the ends
            break;
        }
        lo = lo1;
        hi = hi1;
    }
    if (lane == 0) a.E0[p] = 0.5 * (lo + hi);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
struct BatchLayout {
    size_t desc, bonds, items, E0, stopped, alpha, beta, sigma, cprev, scale, norm0, partial, r0,
        r1, r2, total;
    int n_items, NV, bits;
    uint64_t rows;
};

static size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

static int vec_width(int nvec) {
    int NV = 1;
    while (NV < nvec) NV <<= 1;
    return NV;
}

static int batch_layout(int ninst, const hm_basis *bases, int nvec, int steps, BatchLayout *L) {
    if (ninst < 1) return fail(HM_EINVAL, "ninst must be >= 1");
    if (!bases) return fail(HM_EINVAL, "bases is null");
    if (nvec < 1 || nvec > kBatchMaxVec) return fail(HM_EINVAL, "nvec must be 1..16");
    if (steps < 1) return fail(HM_EINVAL, "steps must be >= 1");
    L->NV = vec_width(nvec);
    L->n_items = 0;
    L->rows = 0;
    // states of every instance are packed with the digit width of the
    // largest spin in the batch
    L->bits = 0;
    for (int k = 0; k < ninst; ++k) {
        if (!bases[k]) return fail(HM_EINVAL, "basis %d is null", k);
        L->bits = std::max(L->bits, bases[k]->impl.bits);
    }
    for (int k = 0; k < ninst; ++k) {
        const Basis &b = bases[k]->impl;
        if (b.N * L->bits > 64)
            return fail(HM_ERANGE,
                        "basis %d: %d sites at %d bits per digit (the batch's widest spin) "
                        "exceed 64 bits", k, b.N, L->bits);
        if (!b.idx32) return fail(HM_ERANGE, "basis %d: dimension too large for the batch", k);
        if (b.prefix_len() * 4 > kBatchPrefixLds)
            return fail(HM_ERANGE, "basis %d: prefix table exceeds the batch LDS budget", k);
        L->n_items += (int)((b.dim + kBatchBlock - 1) / kBatchBlock);
        L->rows += (uint64_t)b.dim;
    }
    if (L->rows >= ((uint64_t)1 << 32)) return fail(HM_ERANGE, "too many rows in the batch");
    const size_t npairs = (size_t)ninst * L->NV;
    size_t off = 0, nb = 0;
    for (int k = 0; k < ninst; ++k) nb += (size_t)bases[k]->impl.N * (bases[k]->impl.N - 1) / 2;
    // descriptors and bonds side by side (one copy to the device), and E0,
    // stopped, alpha and beta (one copy back)
    L->desc = off; off += sizeof(InstDesc) * ninst;
    L->bonds = off; off = al256(off + sizeof(BondDev) * nb);
    L->items = off; off = al256(off + sizeof(Item) * L->n_items);
    L->E0 = off; off += sizeof(double) * npairs;
    L->stopped = off; off = al256(off + sizeof(int) * npairs);
    L->alpha = off; off += sizeof(double) * npairs * steps;
    L->beta = off; off = al256(off + sizeof(double) * npairs * steps);
    L->sigma = off; off = al256(off + sizeof(double) * npairs * (steps + 1));
    L->cprev = off; off = al256(off + sizeof(double) * npairs * (steps + 1));
    L->scale = off; off = al256(off + sizeof(double) * npairs);
    L->norm0 = off; off = al256(off + sizeof(double) * npairs);
    L->partial = off; off = al256(off + sizeof(double) * (size_t)L->n_items * L->NV);
    const size_t vb = sizeof(float) * (size_t)L->rows * L->NV;
    L->r0 = off; off = al256(off + vb);
    L->r1 = off; off = al256(off + vb);
    L->r2 = off; off = al256(off + vb);
    L->total = off;
    return HM_OK;
}

// Every launch of a run.  The grid holds wg_per_cu workgroups per compute unit
// (0: as many workgroups as there are chunks, left to the dispatcher).
template <int NV, int B>
static int launch_batched(const BatchArgs &a, size_t lds, int wg_per_cu, hipStream_t st) {
    const int chunks = (a.n_items + a.chunk - 1) / a.chunk;
    int grid = chunks;
    if (wg_per_cu > 0) {
        int dev = 0, cus = 0;
        HM_HIP(hipGetDevice(&dev));
        HM_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        grid = std::min(grid, wg_per_cu * cus);
    }
    const dim3 g(grid), t(kBatchBlock), gp(a.ninst), tp(kPairBlock);
    const int npairs = a.ninst * NV, gw = (npairs + kBatchBlock / 64 - 1) / (kBatchBlock / 64);
    hipLaunchKernelGGL(batch_items_kernel, dim3((a.n_items + kBatchBlock - 1) / kBatchBlock), t, 0,
                       st, a, const_cast<Item *>(a.items));
    hipLaunchKernelGGL(batch_norm_kernel<NV>, g, t, 0, st, a);
    hipLaunchKernelGGL((batch_pairs_kernel<NV, kInit>), gp, tp, 0, st, a, 0);
    hipLaunchKernelGGL(batch_start_kernel<NV>, dim3(std::min(a.n_items, 1 << 16)), t, 0, st, a);
    for (int k = 0; k < a.steps; ++k) {
        hipLaunchKernelGGL((batch_hx_kernel<NV, B>), g, t, lds, st, a, k);
        hipLaunchKernelGGL((batch_pairs_kernel<NV, kAlpha>), gp, tp, 0, st, a, k);
        hipLaunchKernelGGL(batch_update_kernel<NV>, g, t, 0, st, a, k);
        hipLaunchKernelGGL((batch_pairs_kernel<NV, kBeta>), gp, tp, 0, st, a, k);
    }
    hipLaunchKernelGGL(batch_ground_kernel, dim3(gw), t, 0, st, a, npairs);
    HM_HIP(hipGetLastError());
    return HM_OK;
}

template <int NV>
static int dispatch_bits(int bits, const BatchArgs &args, size_t lds, int wg, hipStream_t st) {
    switch (bits) {
        case 1: return launch_batched<NV, 1>(args, lds, wg, st);
        case 2: return launch_batched<NV, 2>(args, lds, wg, st);
        case 3: return launch_batched<NV, 3>(args, lds, wg, st);
        case 4: return launch_batched<NV, 4>(args, lds, wg, st);
        default: return fail(HM_ERANGE, "batched kernel supports up to 4 bits per digit");
    }
}

}  // namespace hm

using hm::fail;

extern "C" {

int hm_lanczos_batched_workspace(int32_t ninst, const hm_basis *bases, int32_t nvec,
                                 int32_t steps, size_t *bytes) {
    hm::clear_error();
    if (!bytes) return fail(HM_EINVAL, "bytes is null");
    hm::BatchLayout L;
    HM_TRY(hm::batch_layout(ninst, bases, nvec, steps, &L));
    *bytes = L.total;
    return HM_OK;
}

int hm_lanczos_batched(int32_t ninst, const hm_basis *bases, const double *const *J,
                       const double *const *d_v0, int32_t nvec, int32_t steps,
                       double breakdown_tol, int32_t chunk, int32_t wg_per_cu, void *d_work,
                       size_t work_bytes, double *alpha, double *beta, double *E0,
                       int32_t *steps_done, void *stream) {
    hm::clear_error();
    if (!J || !d_v0 || !d_work || !alpha || !beta || !E0 || !steps_done)
        return fail(HM_EINVAL, "null argument");
    if (chunk < 0 || chunk > 64) return fail(HM_EINVAL, "chunk %d outside 0..64", chunk);
    if (wg_per_cu < 0 || wg_per_cu > 8)
        return fail(HM_EINVAL, "workgroups per compute unit %d outside 0..8", wg_per_cu);
    hm::BatchLayout L;
    HM_TRY(hm::batch_layout(ninst, bases, nvec, steps, &L));
    if (work_bytes < L.total)
        return fail(HM_EWORKSPACE, "workspace %zu bytes < required %zu", work_bytes, L.total);
    unsigned char *w = (unsigned char *)d_work;
    hipStream_t st = (hipStream_t)stream;
    // descriptors and bond lists, built here and not in the handles' caches, which
    // hold fewer lists than a batch may bring
    std::vector<unsigned char> up(L.items - L.desc);
    hm::InstDesc *desc = (hm::InstDesc *)up.data();
    hm::BondDev *bonds = (hm::BondDev *)(up.data() + (L.bonds - L.desc));
    const hm::BondDev *d_bonds = (const hm::BondDev *)(w + L.bonds);
    uint32_t vec_off = 0, item_first = 0;
    int max_prefix = 0;
    for (int k = 0; k < ninst; ++k) {
        hm::Basis *b = &bases[k]->impl;
        if (!d_v0[k]) return fail(HM_EINVAL, "start vectors of instance %d are null", k);
        HM_TRY(hm::validate_J(b, J[k]));
        {
            std::lock_guard<std::mutex> lock(b->mu);
            HM_TRY(hm::device_prepare(b));
        }
        const int nb = hm::list_bonds(b, J[k], bonds);
        hm::InstDesc &d = desc[k];
        d.N = b->N;
        d.A = b->A;
        d.two_s = b->two_s;
        d.nb = nb;
        d.dim = (uint32_t)b->dim;
        d.vec_off = vec_off;
        d.item_first = item_first;
        d.item_count = (d.dim + hm::kBatchBlock - 1) / hm::kBatchBlock;
        d.prefix = (const uint32_t *)b->d_prefix;
        d.ladder = b->d_ladder;
        d.bonds = d_bonds;
        d.v0 = d_v0[k];
        vec_off += d.dim;
        item_first += d.item_count;
        bonds += nb;
        d_bonds += nb;
        max_prefix = std::max(max_prefix, (int)b->prefix_len());
    }
    HM_HIP(hipMemcpyAsync(w + L.desc, up.data(), (unsigned char *)bonds - up.data(),
                          hipMemcpyHostToDevice, st));
    hm::BatchArgs a{};
    a.inst = (const hm::InstDesc *)(w + L.desc);
    a.items = (const hm::Item *)(w + L.items);
    a.ninst = ninst;
    a.n_items = L.n_items;
    a.nvec = nvec;
    a.steps = steps;
    a.tol = breakdown_tol > 0 ? breakdown_tol : 1e-6;   // FP32 vectors: FP32 noise floor
    a.r[0] = (float *)(w + L.r0);
    a.r[1] = (float *)(w + L.r1);
    a.r[2] = (float *)(w + L.r2);
    a.partial = (double *)(w + L.partial);
    a.alpha = (double *)(w + L.alpha);
    a.beta = (double *)(w + L.beta);
    a.E0 = (double *)(w + L.E0);
    a.sigma = (double *)(w + L.sigma);
    a.cprev = (double *)(w + L.cprev);
    a.scale = (double *)(w + L.scale);
    a.norm0 = (double *)(w + L.norm0);
    a.stopped = (int *)(w + L.stopped);
    a.max_prefix = max_prefix;
    a.chunk = chunk > 0 ? chunk : hm::default_chunk(L.n_items);
    const size_t lds = ((size_t)(max_prefix * 4 + 15) / 16) * 16 + 32 * sizeof(double);
    const int bits = L.bits;
    int rc;
    switch (L.NV) {
        case 1: rc = hm::dispatch_bits<1>(bits, a, lds, wg_per_cu, st); break;
        case 2: rc = hm::dispatch_bits<2>(bits, a, lds, wg_per_cu, st); break;
        case 4: rc = hm::dispatch_bits<4>(bits, a, lds, wg_per_cu, st); break;
        case 8: rc = hm::dispatch_bits<8>(bits, a, lds, wg_per_cu, st); break;
        default: rc = hm::dispatch_bits<16>(bits, a, lds, wg_per_cu, st); break;
    }
    if (rc != HM_OK) return rc;
    std::vector<unsigned char> down(L.sigma - L.E0);
    HM_HIP(hipMemcpyAsync(down.data(), w + L.E0, down.size(), hipMemcpyDeviceToHost, st));
    HM_HIP(hipStreamSynchronize(st));
    const double *e0 = (const double *)down.data();
    const int *stop = (const int *)(down.data() + (L.stopped - L.E0));
    const double *al = (const double *)(down.data() + (L.alpha - L.E0));
    const double *be = (const double *)(down.data() + (L.beta - L.E0));
    for (int k = 0; k < ninst; ++k)
        for (int q = 0; q < nvec; ++q) {
            const size_t p = (size_t)k * L.NV + q, o = ((size_t)k * nvec + q) * steps;
            if (stop[p] < 0) return fail(HM_EINVAL, "start vector %d of instance %d is zero", q, k);
            const int done = stop[p] > 0 ? stop[p] : steps;
            for (int s = 0; s < steps; ++s) {
                alpha[o + s] = s < done ? al[p * steps + s] : 0.0;
                beta[o + s] = s < done ? be[p * steps + s] : 0.0;
            }
            steps_done[k * nvec + q] = done;
            // an infinite start entry, couplings beyond FP32: no energy (the search
            // of batch_ground_kernel passes over NaN)
            for (int s = 0; s < done; ++s)
                if (!std::isfinite(alpha[o + s]) || (s + 1 < done && !std::isfinite(beta[o + s])))
                    return fail(HM_EINVAL, "vector %d of instance %d: non-finite tridiagonal entry",
                                q, k);
            E0[k * nvec + q] = e0[p];
        }
    return HM_OK;
}

}  // extern "C"
