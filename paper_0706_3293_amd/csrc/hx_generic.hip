// Row-gather H x for any spin s (Sec. 4, Eq. (E-4-b)), and the device
// encoding/decoding entry points (Sec. 3.1, 3.2).
//
// One GPU lane owns one output row i: it decodes |i>, adds the diagonal
// element, and for every bond whose ladder term does not annihilate |i> it
// computes the target index j from the change of the encoding sum and
// gathers x_j.  Only y_i is written, so there are no write conflicts and no
// atomics.  The prefix table and the ladder factors are staged in LDS; the
// bond list is read with wave-uniform (scalar) loads.
#include "device_common.h"
#include "hm_internal.h"
#include "hx_row.h"

namespace hm {

template <typename T, typename I, int B, bool DOT, bool STORE, bool TAB>
__global__ __launch_bounds__(kBlock) void hx_generic_kernel(
    const I *__restrict__ gprefix, const double *__restrict__ gladder,
    const BondDev *__restrict__ bonds, int nb, int N, int A, int two_s, I dim,
    const T *__restrict__ x, T *__restrict__ y, const T *__restrict__ prev,
    const LzStep step, double *__restrict__ partial, T *__restrict__ store) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[kLzLds];
    double sigma_v, cprev_v;
    if (!lz_begin(step, red, sigma_v, cprev_v)) return;
    const double sigma = uniform(sigma_v), cprev = uniform(cprev_v);   // scalar registers
    const int plen = N * (A + 1) * (two_s + 1);
    I *P = reinterpret_cast<I *>(smem);
    const size_t pbytes = ((plen * sizeof(I) + 15) / 16) * 16;
    T *F = reinterpret_cast<T *>(smem + pbytes);
    // TAB: this lane's column of the per-site term positions (row_hx_tab)
    const size_t fbytes = (((size_t)two_s + 2) * sizeof(double) + 15) / 16 * 16;
    uint16_t *sb = reinterpret_cast<uint16_t *>(smem + pbytes + fbytes) + threadIdx.x;
    for (int t = threadIdx.x; t < plen; t += blockDim.x) P[t] = gprefix[t];
    for (int t = threadIdx.x; t < two_s + 2; t += blockDim.x) F[t] = (T)gladder[t];
    __syncthreads();
    const Prefix<I> pv{P, A + 1, two_s + 1};

    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    I first, last;
    block_rows<I>(lb, gridDim.x, dim, first, last);
    double dot = 0.0;
    for (I row = first + threadIdx.x; row < last; row += blockDim.x) {
        const uint64_t st = unrank_state<I, B>(row, pv, N, A, two_s);
        const T xi = x[row];
        T hv;
        if constexpr (TAB)
            hv = row_hx_tab<T, I, B>(st, row, xi, x, bonds, nb, N, two_s, pv, F, sb, blockDim.x);
        else
            hv = row_hx<T, I, B>(st, row, xi, x, bonds, nb, two_s, pv, F);
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

template <typename I, int B>
__global__ __launch_bounds__(kBlock) void unrank_kernel(const I *__restrict__ gprefix, int N,
                                                        int A, int two_s, int64_t dim,
                                                        const int64_t *__restrict__ idx,
                                                        int64_t n, uint64_t *__restrict__ out) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int plen = N * (A + 1) * (two_s + 1);
    I *P = reinterpret_cast<I *>(smem);
    for (int t = threadIdx.x; t < plen; t += blockDim.x) P[t] = gprefix[t];
    __syncthreads();
    const Prefix<I> pv{P, A + 1, two_s + 1};
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = idx[t];
        out[t] = (i < 0 || i >= dim) ? ~0ull : unrank_state<I, B>((I)i, pv, N, A, two_s);
    }
}

template <typename I, int B>
__global__ __launch_bounds__(kBlock) void rank_kernel(const I *__restrict__ gprefix, int N,
                                                      int A, int two_s,
                                                      const uint64_t *__restrict__ states,
                                                      int64_t n, int64_t *__restrict__ out) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int plen = N * (A + 1) * (two_s + 1);
    I *P = reinterpret_cast<I *>(smem);
    for (int t = threadIdx.x; t < plen; t += blockDim.x) P[t] = gprefix[t];
    __syncthreads();
    const Prefix<I> pv{P, A + 1, two_s + 1};
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t st = states[t];
        bool ok = N * B == 64 || (st >> (N * B)) == 0;
        int sum = 0;
        for (int u = 0; u < N; ++u) {
            const int a = digit_at<B>(st, u);
            ok = ok && a <= two_s;
            sum += a;
        }
        ok = ok && sum == A;
        out[t] = ok ? (int64_t)rank_state<I, B>(st, pv, N, A) : (int64_t)-1;
    }
}

// Codec of spins 1/2.  The walk over all sites (unrank_kernel, rank_kernel) is
// bound by its vector instructions, 8 a site.  Decoding walks the sites above the
// low 12 only, with one table entry a site, and looks the low word up: words with
// a set bits lie in ascending order from word_start[a].  Encoding visits the set
// bits only, A of them in every valid state, so the lanes stay together.
// 4 M states of 28 sites: decoding 35 -> 21 us, encoding 46 -> 18 us (floor: 12.5
// each); up to 0.2 M states either way a launch, 8.7 us.
constexpr int kWordBits = 12, kWords = 1 << kWordBits;
struct WordTable {
    uint16_t start[kWordBits + 2];
    alignas(16) uint16_t word[kWords];
};
constexpr WordTable make_word_table() {
    WordTable t{};
    int n = 0;
    for (int a = 0; a <= kWordBits; ++a) {
        t.start[a] = (uint16_t)n;
        for (int w = 0; w < kWords; ++w) {
            int c = 0;
            for (int x = w; x; x &= x - 1) ++c;
            if (c == a) t.word[n++] = (uint16_t)w;
        }
    }
    return t;
}
__device__ const WordTable kWordTable = make_word_table();

// T[k][Ak] = P[k][Ak][1]: states whose site k is empty, of those with Ak bits left.
template <typename I>
__device__ __forceinline__ void load_steps(const I *__restrict__ gprefix, int first, int n, I *T) {
    for (int t = threadIdx.x; t < n; t += blockDim.x) T[t] = gprefix[2 * (first + t) + 1];
}

template <typename I>
__global__ __launch_bounds__(kBlock) void unrank_half_kernel(const I *__restrict__ gprefix, int N,
                                                             int A, int64_t dim,
                                                             const int64_t *__restrict__ idx,
                                                             int64_t n,
                                                             uint64_t *__restrict__ out) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint16_t start[kWordBits + 2];
    __shared__ __align__(16) uint16_t word[kWords];
    I *T = reinterpret_cast<I *>(smem);           // sites 13 .. N
    const int A1 = A + 1, nh = N - kWordBits;
    load_steps(gprefix, kWordBits * A1, nh * A1, T);
    if (threadIdx.x < kWordBits + 1) start[threadIdx.x] = kWordTable.start[threadIdx.x];
    for (int t = threadIdx.x; t < kWords / 8; t += blockDim.x)
        reinterpret_cast<uint4 *>(word)[t] = reinterpret_cast<const uint4 *>(kWordTable.word)[t];
    __syncthreads();
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = idx[t];
        const bool ok = i >= 0 && i < dim;
        I r = ok ? (I)i : (I)0;
        uint32_t hi = 0;
        int e = (nh - 1) * A1 + A;                 // entry of the next site
        for (int k = nh; k >= 1; --k) {
            const I s = T[e];
            const bool set = s <= r;
            r -= set ? s : (I)0;
            hi = 2 * hi + (set ? 1 : 0);
            e -= A1 + (set ? 1 : 0);
        }
        const int Ak = e + A1;                     // bits left for the low word
        const uint32_t lo = word[start[Ak] + (uint32_t)r];
        out[t] = ok ? (uint64_t)hi << kWordBits | lo : ~0ull;
    }
}

__device__ __forceinline__ int top_bit(uint32_t w) { return 31 - __clz((int)w); }
__device__ __forceinline__ int top_bit(uint64_t w) { return 63 - __clzll((long long)w); }

template <typename I, typename Word>
__global__ __launch_bounds__(kBlock) void rank_half_kernel(const I *__restrict__ gprefix, int N,
                                                           int A,
                                                           const uint64_t *__restrict__ states,
                                                           int64_t n, int64_t *__restrict__ out) {
    extern __shared__ __align__(16) unsigned char smem[];
    I *T = reinterpret_cast<I *>(smem);
    const int A1 = A + 1;
    load_steps(gprefix, 0, N * A1, T);
    __syncthreads();
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t st = states[t];
        const bool ok = (N == 64 || st >> N == 0) && __popcll((unsigned long long)st) == A;
        // any A bits in place of a state that is not one of the subspace
        Word w = ok ? (Word)st : A < (int)(8 * sizeof(Word)) ? ((Word)1 << A) - 1 : ~(Word)0;
        I idx = 0;
        for (int a = A; a >= 1; --a) {
            const int p = top_bit(w);
            idx += T[p * A1 + a];
            w ^= (Word)1 << p;
        }
        out[t] = ok ? (int64_t)idx : (int64_t)-1;
    }
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
size_t prefix_bytes(const Basis *b) {
    return b->prefix_len() * (b->idx32 ? sizeof(uint32_t) : sizeof(uint64_t));
}

int check_lds(const Basis *b) {
    if (prefix_bytes(b) + 16 + (b->two_s + 2) * sizeof(double) > kMaxPrefixLds)
        return fail(HM_ERANGE, "prefix table (%zu bytes) exceeds the LDS budget",
                    prefix_bytes(b));
    return HM_OK;
}

int generic_grid(int64_t rows) {
    int64_t g = (rows + kBlock - 1) / kBlock;
    if (g > kMaxGrid) g = kMaxGrid;
    if (g < 1) g = 1;
    if (g >= kXcds) g -= g % kXcds;   // a multiple of 8 enables the XCD mapping
    return (int)g;
}

int hx_generic_grid(const Basis *b) { return generic_grid(b->dim); }

// LDS a workgroup of the generic kernel may take with the term positions.
constexpr size_t kMaxGenericLds = 64 * 1024;

template <typename T, typename I, int B>
static void launch_hx_t(const Basis *b, const Couplings *c, const HxPass &p, int grid,
                        size_t lds, hipStream_t st) {
    const I *pref = (const I *)b->d_prefix;
    const T *x = (const T *)p.x;
    T *y = (T *)p.y;
    const T *pr = (const T *)p.p;
    T *store = (T *)p.store;
    const bool dot = p.partial != nullptr, sto = store != nullptr;
    // tabulated term positions (row_hx_tab) for s >= 1: N x 256 x 2 bytes of
    // LDS beside the prefix table, and positions that fit 16 bits.  Measured
    // (one FP32 H x): s = 1, N = 16 ring 0.284 -> 0.268 ms; s = 2, N = 12
    // ring 0.924 -> 0.826 ms; for s = 1/2 it was slower (N = 28 J1-J2 ring
    // 4.56 -> 5.04 ms), where the digit walks are single popcounts.
    const size_t lds_tab = lds + (size_t)b->N * kBlock * sizeof(uint16_t);
    const bool tab = b->two_s >= 2 && lds_tab <= kMaxGenericLds && b->prefix_len() <= 65535;
#define HM_LAUNCH(D, S, TB)                                                                 \
    hipLaunchKernelGGL((hx_generic_kernel<T, I, B, D, S, TB>), dim3(grid), dim3(kBlock),    \
                       TB ? lds_tab : lds, st, pref, b->d_ladder, c->dev, c->nb, b->N, b->A, \
                       b->two_s, (I)b->dim, x, y, pr, p.step, p.partial, store)
    if (tab) {
        if (!dot && !sto) HM_LAUNCH(false, false, true);
        else if (dot && !sto) HM_LAUNCH(true, false, true);
        else if (!dot && sto) HM_LAUNCH(false, true, true);
        else HM_LAUNCH(true, true, true);
    } else {
        if (!dot && !sto) HM_LAUNCH(false, false, false);
        else if (dot && !sto) HM_LAUNCH(true, false, false);
        else if (!dot && sto) HM_LAUNCH(false, true, false);
        else HM_LAUNCH(true, true, false);
    }
#undef HM_LAUNCH
}

template <typename T, typename I>
static int dispatch_bits(const Basis *b, const Couplings *c, const HxPass &p, int grid,
                         size_t lds, hipStream_t st) {
    switch (b->bits) {
        case 1: launch_hx_t<T, I, 1>(b, c, p, grid, lds, st); break;
        case 2: launch_hx_t<T, I, 2>(b, c, p, grid, lds, st); break;
        case 3: launch_hx_t<T, I, 3>(b, c, p, grid, lds, st); break;
        case 4: launch_hx_t<T, I, 4>(b, c, p, grid, lds, st); break;
        case 5: launch_hx_t<T, I, 5>(b, c, p, grid, lds, st); break;
        case 6: launch_hx_t<T, I, 6>(b, c, p, grid, lds, st); break;
        case 7: launch_hx_t<T, I, 7>(b, c, p, grid, lds, st); break;
        case 8: launch_hx_t<T, I, 8>(b, c, p, grid, lds, st); break;
        default: return fail(HM_ERANGE, "bits per digit %d unsupported", b->bits);
    }
    return HM_OK;
}

int launch_hx_generic(const Basis *b, const Couplings *c, int dtype, const HxPass &p,
                      hipStream_t st) {
    HM_TRY(check_lds(b));
    const int grid = generic_grid(b->dim);
    // prefix table, then the 2s + 2 ladder factors (room for doubles)
    const size_t lds = ((prefix_bytes(b) + 15) / 16) * 16 +
                       (((size_t)b->two_s + 2) * sizeof(double) + 15) / 16 * 16;
    int rc;
    if (dtype == HM_F64)
        rc = b->idx32 ? dispatch_bits<double, uint32_t>(b, c, p, grid, lds, st)
                      : dispatch_bits<double, uint64_t>(b, c, p, grid, lds, st);
    else
        rc = b->idx32 ? dispatch_bits<float, uint32_t>(b, c, p, grid, lds, st)
                      : dispatch_bits<float, uint64_t>(b, c, p, grid, lds, st);
    HM_TRY(rc);
    HM_HIP(hipGetLastError());
    return HM_OK;
}

template <typename I, int B>
static void launch_codec(const Basis *b, bool un, const int64_t *d_idx, const uint64_t *d_st,
                         int64_t n, uint64_t *o_st, int64_t *o_idx, hipStream_t st) {
    int64_t g = (n + kBlock - 1) / kBlock;
    if (g > 4096) g = 4096;
    const size_t lds = prefix_bytes(b);
    if (un)
        hipLaunchKernelGGL((unrank_kernel<I, B>), dim3((int)g), dim3(kBlock), lds, st,
                           (const I *)b->d_prefix, b->N, b->A, b->two_s, b->dim, d_idx, n,
                           o_st);
    else if constexpr (B > 1)                 // spins 1/2 have their own
        hipLaunchKernelGGL((rank_kernel<I, B>), dim3((int)g), dim3(kBlock), lds, st,
                           (const I *)b->d_prefix, b->N, b->A, b->two_s, d_st, n, o_idx);
}

// The spin-1/2 codec where it applies: every state to encode; to decode, 13 to 44
// sites (a high word of 1 to 32).
template <typename I>
static bool launch_codec_half(const Basis *b, bool un, const int64_t *d_idx, const uint64_t *d_st,
                              int64_t n, uint64_t *o_st, int64_t *o_idx, hipStream_t st) {
    const int nh = b->N - kWordBits;
    if (b->two_s != 1 || (un && (nh < 1 || nh > 32))) return false;
    const int64_t g = std::min<int64_t>((n + kBlock - 1) / kBlock, 2048);
    const I *prefix = (const I *)b->d_prefix;
    if (un) {
        hipLaunchKernelGGL(unrank_half_kernel<I>, dim3((int)g), dim3(kBlock),
                           (size_t)nh * (b->A + 1) * sizeof(I), st, prefix, b->N, b->A, b->dim,
                           d_idx, n, o_st);
        return true;
    }
    const size_t lds = (size_t)b->N * (b->A + 1) * sizeof(I);
    if (b->N <= 32)
        hipLaunchKernelGGL((rank_half_kernel<I, uint32_t>), dim3((int)g), dim3(kBlock), lds, st,
                           prefix, b->N, b->A, d_st, n, o_idx);
    else
        hipLaunchKernelGGL((rank_half_kernel<I, uint64_t>), dim3((int)g), dim3(kBlock), lds, st,
                           prefix, b->N, b->A, d_st, n, o_idx);
    return true;
}

template <typename I>
static int codec_bits(const Basis *b, bool un, const int64_t *d_idx, const uint64_t *d_st,
                      int64_t n, uint64_t *o_st, int64_t *o_idx, hipStream_t st) {
    if (launch_codec_half<I>(b, un, d_idx, d_st, n, o_st, o_idx, st)) return HM_OK;
    switch (b->bits) {
        case 1: launch_codec<I, 1>(b, un, d_idx, d_st, n, o_st, o_idx, st); break;
        case 2: launch_codec<I, 2>(b, un, d_idx, d_st, n, o_st, o_idx, st); break;
        case 3: launch_codec<I, 3>(b, un, d_idx, d_st, n, o_st, o_idx, st); break;
        case 4: launch_codec<I, 4>(b, un, d_idx, d_st, n, o_st, o_idx, st); break;
        case 5: launch_codec<I, 5>(b, un, d_idx, d_st, n, o_st, o_idx, st); break;
        case 6: launch_codec<I, 6>(b, un, d_idx, d_st, n, o_st, o_idx, st); break;
        case 7: launch_codec<I, 7>(b, un, d_idx, d_st, n, o_st, o_idx, st); break;
        case 8: launch_codec<I, 8>(b, un, d_idx, d_st, n, o_st, o_idx, st); break;
        default: return fail(HM_ERANGE, "bits per digit %d unsupported", b->bits);
    }
    return HM_OK;
}

int launch_unrank(const Basis *b, const int64_t *d_idx, int64_t n, uint64_t *d_state,
                  hipStream_t st) {
    HM_TRY(check_lds(b));
    HM_TRY(b->idx32 ? codec_bits<uint32_t>(b, true, d_idx, nullptr, n, d_state, nullptr, st)
                    : codec_bits<uint64_t>(b, true, d_idx, nullptr, n, d_state, nullptr, st));
    HM_HIP(hipGetLastError());
    return HM_OK;
}

int launch_rank(const Basis *b, const uint64_t *d_state, int64_t n, int64_t *d_idx,
                hipStream_t st) {
    HM_TRY(check_lds(b));
    HM_TRY(b->idx32 ? codec_bits<uint32_t>(b, false, nullptr, d_state, n, nullptr, d_idx, st)
                    : codec_bits<uint64_t>(b, false, nullptr, d_state, n, nullptr, d_idx, st));
    HM_HIP(hipGetLastError());
    return HM_OK;
}

}  // namespace hm
