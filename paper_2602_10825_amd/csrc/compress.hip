// KV-cache compression at a chunk commit (Sec. 3.3, Eq. (10)-(12); App. C.1, C.2).
//
// Kernels, all stream-ordered, float64 arithmetic, no floating-point atomics:
//   key_stats      pass 1 over K: per token 1/max(||k||,1e-12); per block the partial sum of
//                  normalised keys
//   mean_sim       s = sum_i k^_i from the block partials (fixed order), then pass 2 over K:
//                  the token's norm again (same operations, same bits: cheaper than a side
//                  stream of 16 bytes per token written by pass 1 and read here), then
//                  r_j = (k^_j . s - k^_j . k^_j) / L, the linear-time form of the
//                  diagonal-zeroed column mean of Eq. (11); writes e_j = exp(r_j) and block
//                  partial sums of e.  (The softmax of Eq. (11) is shift-invariant and
//                  |r_j| <= 1 + 1/L, so no max is subtracted.)
//   score_keys     Red_j = e_j / sum e (Eq. (11)), max-pooled importance (Eq. (10)), score
//                  (Eq. (12)) -> order-preserving 64-bit keys; and a histogram of the keys whose
//                  bins are spread over a bracket of the wanted key that a sample of the head's
//                  keys gives
//   select         per head: the bin that holds the budget-th largest key; a few blocks gather its
//                  keys in parallel, the last one to finish ends the select on them in LDS
//   write_kept     ordered compaction of the kept positions (ties: lower position wins;
//                  output ascending); blocks exchange their counts through one word each
//   select_small   the three above in one launch of one block per head, for heads whose keys fit in LDS
//   compact_rows   move the kept K and V rows to positions [0, budget) IN PLACE, one pass of
//                  tiles drawn from a ticket counter; a tile stores only after the
//                  lower tiles that read from its rows have loaded them
// A 16-lane group owns one token row in the two passes over K (16-byte loads, a full
// row per group), so a token's values never depend on where it sits in the launch.
#include <type_traits>

#include "fc_common.hpp"
#include "select_bins.hpp"

#pragma clang fp contract(off)

namespace {

constexpr int kThreads = 256;
constexpr int kGroups = kThreads / 16;
constexpr int kSelThreads = 1024;
constexpr int kItems = 8;
constexpr int kTokBlk = kThreads * kItems;   // tokens per block in the per-token kernels
constexpr int kDigitBits = 11;
constexpr int kBins = 1 << kDigitBits;
constexpr int kCand = 4096;   // candidates resolved in LDS
constexpr int kRank = 256;    // candidates resolved by comparing each with each
constexpr int kScoreThreads = 512, kScoreItems = 4;                 // of score_keys
constexpr int kScoreBlk = kScoreThreads * kScoreItems;
constexpr int kHalo = 192;    // importance beside a block's tokens that score_keys can keep in LDS
constexpr int kSmallL = kSelThreads * 4;   // heads up to this length are selected by one block
constexpr int kUnroll = 8;    // independent loads in flight per thread in the selection scans

// ---- bookkeeping of the in-place compaction (kernels further down) ----------------------
// Rows per tile of the compaction: 16 KB or more of each cache.  (128-byte rows in tiles of 64 were bound
// by what each tile costs: 24 heads of 84000 -> 40000 rows 187 us, in tiles of 128 108.)
__host__ __device__ constexpr int tile_rows(int row_bytes) { return row_bytes <= 128 ? 128 : 64; }
constexpr uint32_t kSpinLimit = 1u << 24;

// Words of the sync area (uint32), all reset earlier in the call:
//   [0]                                  status word (non-zero: a bounded wait ran out)
//   [64 * (h + 1)]                       ticket counter of head h (one per 256-byte line:
//                                        atomics on one line serialise)
//   [64 * (H + 1) + h * ntile + t]       "tile t of head h has been read"
//   [64 * (H + 1) + (H + h) * ntile + t] source row of the last destination row of tile t
__host__ __device__ inline size_t sync_words(int H, int ntile) { return (size_t)2 * H * ntile + 64 * ((size_t)H + 1); }
__device__ __forceinline__ uint32_t* sync_flags(uint32_t* sync, int H, int ntile, int h) {
    return sync + 64 * (H + 1) + (int64_t)h * ntile;
}
__device__ __forceinline__ int32_t* sync_tile_last(uint32_t* sync, int H, int ntile, int h) {
    return reinterpret_cast<int32_t*>(sync + 64 * (H + 1) + (int64_t)(H + h) * ntile);
}


// ---- per-lane slice of one token row: raw bits held in registers, widened exactly ------
template <typename T, int D>
struct Slice {
    static constexpr int EL = D / 16;                       // elements per lane
    static constexpr int NW = EL * (int)sizeof(T) / 4;      // 32-bit words per lane
    typedef uint32_t raw_t __attribute__((ext_vector_type(NW)));
    static __device__ __forceinline__ raw_t load(const T* row, int u) {
        return *reinterpret_cast<const raw_t*>(row + u * EL);
    }
    static __device__ __forceinline__ void widen(const raw_t& r, double (&x)[EL]) {
        if constexpr (sizeof(T) == 8) {
#pragma unroll
            for (int e = 0; e < EL; ++e) x[e] = __hiloint2double((int)r[2 * e + 1], (int)r[2 * e]);
        } else if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                x[2 * w] = (double)bf16lo_to_f32(r[w]);
                x[2 * w + 1] = (double)bf16hi_to_f32(r[w]);
            }
        } else {
#pragma unroll
            for (int w = 0; w < NW; ++w) x[w] = (double)__uint_as_float(r[w]);
        }
    }
};

// Sixteen sums over the 16 lanes of a group, one wanted per lane (lane u wants the sum of
// v[u]): in the step for lane bit b a lane keeps the half of its values whose index has bit b
// like its own, hands the other half to its partner and adds what it receives -- 15 exchanges
// instead of the 64 of sixteen all-reduces.  Every sum is added up along the same tree over
// the lanes (bit 1, 2, 4, 8), so its bits do not depend on which token it belongs to.
__device__ __forceinline__ double group_sum_scatter(double (&v)[16], int u) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {    // lane bit 1 <-> value index bit 1: pairs (2i, 2i+1)
        const bool up = u & 1;
        const double keep = up ? v[2 * i + 1] : v[2 * i], give = up ? v[2 * i] : v[2 * i + 1];
        v[i] = keep + __shfl_xor(give, 1, 16);          // v[i] now belongs to index 2i + (u&1)
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {    // bit 2: indices 4i + (u&1) and 4i + 2 + (u&1)
        const bool up = u & 2;
        const double keep = up ? v[2 * i + 1] : v[2 * i], give = up ? v[2 * i] : v[2 * i + 1];
        v[i] = keep + __shfl_xor(give, 2, 16);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {    // bit 4
        const bool up = u & 4;
        const double keep = up ? v[2 * i + 1] : v[2 * i], give = up ? v[2 * i] : v[2 * i + 1];
        v[i] = keep + __shfl_xor(give, 4, 16);
    }
    {                                // bit 8
        const bool up = u & 8;
        const double keep = up ? v[1] : v[0], give = up ? v[0] : v[1];
        return keep + __shfl_xor(give, 8, 16);
    }
}

// Eight sums over the 16 lanes of a group: lanes u and u + 8 both end with the sum of v[u % 8]
// (three halving steps as above, then one exchange between the two halves of the group).
__device__ __forceinline__ double group_sum_scatter8(double (&v)[8], int u) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool up = u & 1;
        const double keep = up ? v[2 * i + 1] : v[2 * i], give = up ? v[2 * i] : v[2 * i + 1];
        v[i] = keep + __shfl_xor(give, 1, 16);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const bool up = u & 2;
        const double keep = up ? v[2 * i + 1] : v[2 * i], give = up ? v[2 * i] : v[2 * i + 1];
        v[i] = keep + __shfl_xor(give, 2, 16);
    }
    const bool up = u & 4;
    const double keep = up ? v[1] : v[0], give = up ? v[0] : v[1];
    const double half = keep + __shfl_xor(give, 4, 16);
    // the lower lane's term first on both sides, so both lanes get the same bits
    const double other = __shfl_xor(half, 8, 16);
    return (u & 8) ? other + half : half + other;
}

// The two passes over K.  A group of 16 lanes takes R consecutive tokens per round (R = 16 or
// 8): all R row slices are requested first, the per-token sums are reduced over the group so
// that lane u ends with token u's, and lane u finishes token u (square root, reciprocal,
// exponential) -- one token per lane instead of every lane repeating the same float64 work.
// With R = 8 the widened rows of pass 1 stay in registers for their second use.  Rows past the
// end of the head re-read its last row (branch-free loads) and are given weight zero.
template <typename T, int D, int R>
__device__ __forceinline__ void load_round(typename Slice<T, D>::raw_t (&raw)[R], const T* base,
                                           int64_t tok_stride, int j0, int L, int u) {
    const int jb = j0 < L ? j0 : L - 1;         // a round wholly past the end re-reads the last row
    const int room = L - 1 - jb;                // rows of this round that exist beyond the first
    const T* rb = base + (int64_t)jb * tok_stride;
#pragma unroll
    for (int i = 0; i < R; ++i)
        raw[i] = Slice<T, D>::load(rb + (int64_t)(i < room ? i : room) * tok_stride, u);
}

template <int R>
__device__ __forceinline__ double scatter_sum(double (&v)[R], int u) {
    if constexpr (R == 16) return group_sum_scatter(v, u);
    else return group_sum_scatter8(v, u);
}

template <typename T, int D, int R>
__global__ __launch_bounds__(kThreads) void key_stats_kernel(
    const T* __restrict__ k_cache, int64_t head_stride, int64_t tok_stride, int L,
    double* __restrict__ psum) {
    typedef Slice<T, D> S;
    constexpr int EL = S::EL;
    constexpr bool KEEP = (R == 8);   // the widened rows stay in registers between the two uses
    const int h = blockIdx.y;
    const int g = threadIdx.x / 16, u = threadIdx.x % 16;
    const T* base = k_cache + (int64_t)h * head_stride;
    double acc[EL];
#pragma unroll
    for (int e = 0; e < EL; ++e) acc[e] = 0.0;
    const int stride = gridDim.x * kGroups * R;
    auto round = [&](typename S::raw_t (&raw)[R], int j0) {
        double xs[KEEP ? R : 1][EL];
        double part[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            double x[EL];
            S::widen(raw[i], x);
            double n2 = 0.0;
#pragma unroll
            for (int e = 0; e < EL; ++e) n2 = fma(x[e], x[e], n2);
            part[i] = n2;
            if constexpr (KEEP) {
#pragma unroll
                for (int e = 0; e < EL; ++e) xs[i][e] = x[e];
            }
        }
        const double mine = scatter_sum<R>(part, u);
        const double inv_mine = 1.0 / fmax(sqrt(mine), 1e-12);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            double inv = __shfl(inv_mine, i, 16);
            inv = (j0 + i < L) ? inv : 0.0;   // rows past the end were re-reads of the last row
            if constexpr (KEEP) {
#pragma unroll
                for (int e = 0; e < EL; ++e) acc[e] = fma(xs[i][e], inv, acc[e]);
            } else {
                double x[EL];
                asm volatile("" : "+v"(raw[i]));   // widen again here rather than keep R rows of doubles live
                S::widen(raw[i], x);
#pragma unroll
                for (int e = 0; e < EL; ++e) acc[e] = fma(x[e], inv, acc[e]);
            }
        }
    };
    // the rows of the next round are requested before the current round is worked on: with the
    // two or three wavefronts per SIMD that the registers allow, nothing else hides their latency
    // (rounds of 16 rows of wider storage would need more registers than a wavefront has)
    if constexpr (R == 8) {
        typename S::raw_t ra[R], rb[R];
        int j0 = (blockIdx.x * kGroups + g) * R;
        if (j0 < L) load_round<T, D, R>(ra, base, tok_stride, j0, L, u);
        for (; j0 < L; j0 += 2 * stride) {
            if (j0 + stride < L) load_round<T, D, R>(rb, base, tok_stride, j0 + stride, L, u);
            __builtin_amdgcn_sched_barrier(0);
            round(ra, j0);
            if (j0 + stride < L) {
                if (j0 + 2 * stride < L) load_round<T, D, R>(ra, base, tok_stride, j0 + 2 * stride, L, u);
                __builtin_amdgcn_sched_barrier(0);
                round(rb, j0 + stride);
            }
        }
    } else {
        for (int j0 = (blockIdx.x * kGroups + g) * R; j0 < L; j0 += stride) {
            typename S::raw_t raw[R];
            load_round<T, D, R>(raw, base, tok_stride, j0, L, u);
            round(raw, j0);
        }
    }
    __shared__ double sh[kGroups][D];
#pragma unroll
    for (int e = 0; e < EL; ++e) sh[g][u * EL + e] = acc[e];
    __syncthreads();
    if (threadIdx.x < D) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < kGroups; ++k) t += sh[k][threadIdx.x];
        psum[((int64_t)h * gridDim.x + blockIdx.x) * D + threadIdx.x] = t;
    }
}

// Pass 2: r_j = (k^_j . s - k^_j . k^_j) / L for every token, e_j = exp(r_j) and the block's
// partial sum of e.  Every block first adds up the head's few block partials of pass 1 itself,
// in block order (s = sum_i k^_i; the same bits in every block), which saves a launch.
template <typename T, int D, int R>
__global__ __launch_bounds__(kThreads) void mean_sim_kernel(
    const T* __restrict__ k_cache, int64_t head_stride, int64_t tok_stride, int L,
    const double* __restrict__ psum, int npart,
    double* __restrict__ e_out, double* __restrict__ pz, uint32_t* __restrict__ hist_all) {
    typedef Slice<T, D> S;
    constexpr int EL = S::EL;
    const int h = gridDim.y - 1 - blockIdx.y;   // pass 1 read the last heads last: they may still be cached
    const int g = threadIdx.x / 16, u = threadIdx.x % 16;
    const T* base = k_cache + (int64_t)h * head_stride;
    if (hist_all && blockIdx.x == 0)   // the first-digit histogram that score_keys adds to
        for (int i = threadIdx.x; i < kFirstBins; i += kThreads) hist_all[(int64_t)h * kFirstBins + i] = 0u;
    __shared__ double sh_s[D];
    if (threadIdx.x < D) {
        const double* p = psum + (int64_t)h * npart * D + threadIdx.x;
        double t = 0.0;
        int b = 0;
        for (; b + 8 <= npart; b += 8) {      // eight loads in flight, added in block order
            double v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = p[(int64_t)(b + q) * D];
#pragma unroll
            for (int q = 0; q < 8; ++q) t += v[q];
        }
        for (; b < npart; ++b) t += p[(int64_t)b * D];
        sh_s[threadIdx.x] = t;
    }
    __syncthreads();
    double s[EL];
#pragma unroll
    for (int e = 0; e < EL; ++e) s[e] = sh_s[u * EL + e];
    const double dL = (double)L;
    double zsum = 0.0;
    const int stride = gridDim.x * kGroups * R;
    for (int j0 = (blockIdx.x * kGroups + g) * R; j0 < L; j0 += stride) {
        typename S::raw_t raw[R];
        load_round<T, D, R>(raw, base, tok_stride, j0, L, u);
        const bool have = u < R && j0 + u < L;
        double part[R], part2[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            double x[EL];
            S::widen(raw[i], x);
            double dot = 0.0, n2 = 0.0;
#pragma unroll
            for (int e = 0; e < EL; ++e) dot = fma(x[e], s[e], dot);
#pragma unroll
            for (int e = 0; e < EL; ++e) n2 = fma(x[e], x[e], n2);   // as in pass 1, bit for bit
            part[i] = dot;
            part2[i] = n2;
        }
        const double mine = scatter_sum<R>(part, u);
        const double n2 = scatter_sum<R>(part2, u);
        if (have) {
            const double inv = 1.0 / fmax(sqrt(n2), 1e-12);
            const double2 ti = make_double2(inv, (n2 * inv) * inv);
            const double ej = exp((mine * ti.x - ti.y) / dL);
            e_out[(int64_t)h * L + j0 + u] = ej;
            zsum += ej;
        }
    }
    __shared__ double shz[kThreads];
    shz[threadIdx.x] = zsum;
    __syncthreads();
    if (threadIdx.x < 64) {   // fixed order: four strided terms per lane, then the lanes in order
        double z = (shz[threadIdx.x] + shz[threadIdx.x + 64]) + (shz[threadIdx.x + 128] + shz[threadIdx.x + 192]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) z += __shfl_down(z, o, FC_WAVE);
        if (threadIdx.x == 0) pz[(int64_t)h * gridDim.x + blockIdx.x] = z;
    }
}

// Sum over the first kThreads threads of a block, along a fixed tree (distances 128, 64, ..., 1): the same
// bits in every block that runs it.  A block of more threads passes anything in the others.
__device__ __forceinline__ double block_sum_fixed(double v, double* sh) {   // sh: kThreads + 1
    static_assert(kThreads == 256, "four terms per lane");
    const int t = threadIdx.x;
    if (t < kThreads) sh[t] = v;
    __syncthreads();
    if (t < FC_WAVE) {
        double z = (sh[t] + sh[t + 128]) + (sh[t + 64] + sh[t + 192]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) z += __shfl_down(z, o, FC_WAVE);
        if (t == 0) sh[kThreads] = z;
    }
    __syncthreads();
    return sh[kThreads];
}

// Histogram increment that survives skew: the digits most lanes of a wavefront share are
// counted once per wavefront (up to four rounds of leader election); the rest go one by one.
__device__ __forceinline__ void hist_add(uint32_t* hist, bool in, uint32_t dgt) {
    uint64_t act = __ballot(in);
#pragma unroll 1
    for (int round = 0; round < 4 && act; ++round) {
        const int leader = __ffsll((long long)act) - 1;
        const uint32_t d0 = __shfl(dgt, leader, FC_WAVE);
        const uint64_t same = __ballot(in && dgt == d0);
        if ((int)(threadIdx.x & 63) == leader) atomicAdd(&hist[d0], (uint32_t)__popcll(same));
        in = in && (dgt != d0);
        act &= ~same;
    }
    if (in) atomicAdd(&hist[dgt], 1u);
}

__device__ __forceinline__ uint64_t score_key(double score) {
    if (score == 0.0) score = 0.0;  // -0 -> +0
    const uint64_t b = (uint64_t)__double_as_longlong(score);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__device__ __forceinline__ double key_score(uint64_t key) {   // the score of a key
    return __longlong_as_double((long long)((key >> 63) ? key & 0x7fffffffffffffffull : ~key));
}

// Eq. (11) and (12) of one token: e = exp(r), the pooled importance, z = sum of e over the head
__device__ __forceinline__ uint64_t token_key(double e, double pooled, double z, double lambda) {
    const double red = e / z;
    const double a = lambda * pooled;
    const double b = (1.0 - lambda) * red;
    return score_key(a - b);
}

// fc_first_digit's choice of bins: the same in every wavefront that looks at the same edges
__device__ __forceinline__ int first_digit_shift(const uint64_t* edge, int n) {
    const int sh = __builtin_amdgcn_readfirstlane(fc_even_shift(edge, n));
    return __any(fc_crowded(edge, n, sh, threadIdx.x & (FC_WAVE - 1))) ? -1 : sh;
}

// ---- keys: Eq. (10)-(12) per token, fully parallel ------------------------------------
// Where the first digit's bins lie decides how many keys the select has to look at again: every block
// takes the same 128 keys of the head and lays the bins between those some ranks above and below the
// wanted one (select_bins.hpp).  A wanted key outside (5 deviations) costs time only.
// Every block compares the sampled keys with each other, 16384 comparisons, which more threads share and larger blocks
// make rarer (scoring and selection, us; threads x tokens each 256 x 8 / 512 x 4 in turn on one card: 12 heads of 51000 keys
// 90.7 / 88.9, 8 of 20000 52.9 / 50.3, 4 of 5000 35.1 / 32.7, 24 of 74880 214.5 / 214.8; on another 1024 x 4 and 1024 x 8 are
// slower than 512 x 4 for the short ones, 33.3 / 34.8 / 36.2 for 4 of 5000).
template <typename MT>   // importance as given (float) or pooled over a key group (double)
__global__ __launch_bounds__(kScoreThreads) void score_keys_kernel(
    const double* __restrict__ e_all, const MT* __restrict__ mass_all,
    const double* __restrict__ pz_all, int nblkz, int L, int budget, int pool_k,
    double lambda, uint64_t* __restrict__ keys_all, uint64_t* __restrict__ edge_all,
    uint32_t* __restrict__ hist_all, uint32_t* __restrict__ sync, int ntile, uint32_t* __restrict__ selsync,
    uint64_t* __restrict__ agg_all, int n_agg) {
    constexpr int TPS = kScoreThreads / kSample;   // threads per sampled token
    const int h = blockIdx.y, tid = threadIdx.x;
    const double* e = e_all + (int64_t)h * L;
    const MT* mass = mass_all + (int64_t)h * L;
    uint64_t* keys = keys_all + (int64_t)h * L;
    __shared__ double shd[kThreads + 1];
    __shared__ MT ms[kScoreBlk + 2 * kHalo];
    __shared__ uint64_t sample[kSample];
    __shared__ uint64_t edge[kEdges];
    __shared__ uint32_t hist[kFirstBins];
    const int half = pool_k / 2;
    const FcBracket br = fc_bracket(budget, L);
    const int n_int = br.bottom - br.top;
    // The sample: one token of each 128th of the head (L >= kSample), not always the same one of it.
    // TPS neighbouring threads take token q, every TPS-th distance of its importance window each; everything
    // is requested before the sums that z needs.
    const int sq = tid / TPS, slen = L / kSample;
    const int sj = (int)((int64_t)sq * L / kSample) + (int)(((uint32_t)sq * 2654435761u >> 12) % (uint32_t)slen);
    const double se = e[sj];
    MT simp = mass[sj];
    auto window = [&](auto n, int d0) {           // every TPS-th distance from d0 on, n of them in flight together
        constexpr int N = decltype(n)::value;
        MT lo[N], hi[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int d = d0 + TPS * i < half ? d0 + TPS * i : half;
            lo[i] = mass[sj - d >= 0 ? sj - d : 0];
            hi[i] = mass[sj + d < L ? sj + d : L - 1];
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const MT nb = lo[i] > hi[i] ? lo[i] : hi[i];
            simp = simp > nb ? simp : nb;
        }
    };
    int d0 = 1 + tid % TPS;
    for (; d0 + 12 * TPS <= half; d0 += 16 * TPS) window(std::integral_constant<int, 16>(), d0);
    for (; d0 <= half; d0 += 2 * TPS) window(std::integral_constant<int, 2>(), d0);
#pragma unroll
    for (int o = 1; o < TPS; o <<= 1) {
        const MT nb = __shfl_xor(simp, o, FC_WAVE);
        simp = simp > nb ? simp : nb;
    }
    if (blockIdx.x == 0) {   // state later kernels of this call start from: tile flags, tickets
        uint32_t* flags = sync_flags(sync, gridDim.y, ntile, h);
        for (int i = tid; i < ntile; i += kScoreThreads) flags[i] = 0u;
        if (tid == 0) sync[64 * (h + 1)] = 0u;
        if (h == 0 && tid == 0) sync[0] = 0u;
        if (tid < 3) selsync[h * 64 + tid] = 0u;
        for (int i = tid; i < n_agg; i += kScoreThreads) agg_all[(int64_t)h * n_agg + i] = 0ull;
    }
    for (int i = tid; i < kFirstBins; i += kScoreThreads) hist[i] = 0u;
    if (tid < kEdges) edge[tid] = ~0ull;
    const int j0 = blockIdx.x * kScoreBlk;
    double ev[kScoreItems];
    MT imp[kScoreItems];
#pragma unroll
    for (int i = 0; i < kScoreItems; ++i) {
        const int j = j0 + i * kScoreThreads + tid;
        ev[i] = (j < L) ? e[j] : 0.0;
        imp[i] = (j < L) ? mass[j] : (MT)0;
    }
    const bool staged = half <= kHalo;            // the window comes from LDS
    if (staged) {
        auto beside = [&](int i) {                // i < 2 half: the tokens to the left, then those to the right
            const int j = i < half ? j0 - 1 - i : j0 + kScoreBlk + i - half;
            return mass[j < 0 ? 0 : (j < L ? j : L - 1)];
        };
        auto slot = [&](int i) { return i < half ? kHalo - 1 - i : kHalo + kScoreBlk + i - half; };
        const MT first = tid < 2 * half ? beside(tid) : (MT)0;
#pragma unroll
        for (int i = 0; i < kScoreItems; ++i) ms[kHalo + i * kScoreThreads + tid] = imp[i];
        if (tid < 2 * half) ms[slot(tid)] = first;
        for (int i = tid + kScoreThreads; i < 2 * half; i += kScoreThreads) ms[slot(i)] = beside(i);
    }
    // Z = sum_j e_j: the block partials of the pass that wrote e, in a fixed order
    double z = 0.0;
    if (tid < kThreads)
        for (int i = tid; i < nblkz; i += kThreads) z += pz_all[(int64_t)h * nblkz + i];
    z = block_sum_fixed(z, shd);   // its barriers publish ms too
    const uint64_t sk = token_key(se, (double)simp, z, lambda);
    if (tid % TPS == 0) sample[sq] = sk;
    __syncthreads();
    {   // rank of each sampled key from the top (ties by index); its threads count a part each
        uint32_t above = 0;
        const int c0 = tid % TPS * (kSample / TPS);
#pragma unroll 8
        for (int i = c0; i < c0 + kSample / TPS; ++i) {
            const uint64_t o = sample[i];
            above += (o > sk || (o == sk && i < sq)) ? 1u : 0u;
        }
#pragma unroll
        for (int o = 1; o < TPS; o <<= 1) above += __shfl_xor(above, o, FC_WAVE);
        if (tid % TPS == 0 && (int)above >= br.top && (int)above <= br.bottom) edge[br.bottom - (int)above] = sk;
    }
    __syncthreads();
    if (blockIdx.x == 0 && tid < kEdges) edge_all[(int64_t)h * kEdges + tid] = edge[tid];
    const int even_sh = first_digit_shift(edge, n_int);

    auto pool = [&](auto at) {   // Eq. (10): window max, -inf outside [0, L)
        for (int d = 1; d <= half; ++d) {
#pragma unroll
            for (int i = 0; i < kScoreItems; ++i) {
                const int j = j0 + i * kScoreThreads + tid;
                if (j < L) {
                    const MT lo = (j - d >= 0) ? at(j - d) : imp[i];
                    const MT hi = (j + d < L) ? at(j + d) : imp[i];
                    const MT nb = lo > hi ? lo : hi;
                    imp[i] = imp[i] > nb ? imp[i] : nb;
                }
            }
        }
    };
    if (staged) pool([&](int j) { return ms[j - j0 + kHalo]; });
    else pool([&](int j) { return mass[j]; });
    uint64_t kv[kScoreItems];
#pragma unroll
    for (int i = 0; i < kScoreItems; ++i) {
        const int j = j0 + i * kScoreThreads + tid;
        kv[i] = 0ull;
        if (j < L) {
            kv[i] = token_key(ev[i], (double)imp[i], z, lambda);
            keys[j] = kv[i];
        }
    }
    // the two outer bins hold most of the keys: counted by the wavefront; the others are spread
    uint32_t below = 0, above = 0;
#pragma unroll
    for (int i = 0; i < kScoreItems; ++i) {
        const bool in = j0 + i * kScoreThreads + tid < L;
        const uint32_t dgt = fc_first_digit(kv[i], edge, n_int, even_sh);
        below += __popcll(__ballot(in && dgt == 0u));
        above += __popcll(__ballot(in && dgt == (uint32_t)(kFirstBins - 1)));
        if (in && dgt != 0u && dgt != (uint32_t)(kFirstBins - 1)) atomicAdd(&hist[dgt], 1u);
    }
    if ((tid & 63) == 0) {
        atomicAdd(&hist[0], below);
        atomicAdd(&hist[kFirstBins - 1], above);
    }
    __syncthreads();
    for (int i = tid; i < kFirstBins; i += kScoreThreads)
        if (hist[i]) atomicAdd(&hist_all[(int64_t)h * kFirstBins + i], hist[i]);
}

// From a histogram of `nb` <= 2048 bins (counts of the current candidates by digit), find the
// bin that holds the `need`-th largest candidate and the number of candidates in higher
// bins.  All 1024 threads take part: thread t owns the two bins nb-1-2t and nb-2-2t, a block
// scan in descending bin order gives the count above each, and the one thread whose bin
// straddles `need` publishes the answer.  (A single thread walking the bins would pay one
// LDS round trip per bin.)
__device__ __forceinline__ void pick_bin_parallel(const uint32_t* hist, int nb, uint32_t need,
                                                  uint32_t* wsum, uint64_t prefix, int shift,
                                                  uint64_t* out_prefix, uint32_t* out_need,
                                                  uint32_t* out_count) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid / FC_WAVE;
    const int b0 = nb - 1 - 2 * tid, b1 = nb - 2 - 2 * tid;
    const uint32_t h0 = (b0 >= 0) ? hist[b0] : 0u;
    const uint32_t h1 = (b1 >= 0) ? hist[b1] : 0u;
    uint32_t inc = h0 + h1;   // inclusive scan over threads (= descending bins)
#pragma unroll
    for (int o = 1; o < FC_WAVE; o <<= 1) {
        const uint32_t t = __shfl_up(inc, o, FC_WAVE);
        if (lane >= o) inc += t;
    }
    __syncthreads();
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint32_t above = inc - (h0 + h1);
    for (int w = 0; w < wave; ++w) above += wsum[w];
    if (b0 >= 0 && above < need && need <= above + h0) {
        *out_prefix = prefix | ((uint64_t)b0 << shift);
        *out_need = need - above;
        *out_count = h0;
    } else if (b1 >= 0 && above + h0 < need && need <= above + h0 + h1) {
        *out_prefix = prefix | ((uint64_t)b1 << shift);
        *out_need = need - above - h0;
        *out_count = h1;
    }
}

// Append `k` to an LDS list from the lanes with `take`; one counter update per wavefront.
__device__ __forceinline__ void list_append(uint64_t* list, uint32_t* counter, bool take, uint64_t k) {
    const uint64_t m = __ballot(take);
    if (m == 0) return;
    const int lane = threadIdx.x & 63;
    const int leader = __ffsll((long long)m) - 1;
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(counter, (uint32_t)__popcll(m));
    base = __shfl(base, leader, FC_WAVE);
    if (take) list[base + __popcll(m & ((1ull << lane) - 1ull))] = k;
}

// The `need`-th largest of n <= kRank keys: every key is compared with every other one.
__device__ __forceinline__ void rank_select(const uint64_t* cand, uint32_t n, uint32_t need, uint64_t* out_key,
                                            uint32_t* out_need) {
    if (threadIdx.x < n) {
        const uint64_t k = cand[threadIdx.x];
        uint32_t gt = 0, eq = 0;
        for (uint32_t i = 0; i < n; ++i) {
            const uint64_t o = cand[i];
            gt += o > k ? 1u : 0u;
            eq += o == k ? 1u : 0u;
        }
        if (gt < need && need <= gt + eq) { *out_key = k; *out_need = need - gt; }   // equal keys write the same
    }
}

// ---- per head: finish the select -> threshold key and the number of its copies kept.
// A few blocks per head.  Every block reads the first-digit histogram and picks the same bin.
// If that bin holds at most kCand keys (the usual case), the blocks scan the head's keys in
// parallel and append the bin's keys to a list in global memory; the block that finishes last
// (an integer count, nobody waits) pulls the list into LDS and finishes the select there.
// Otherwise -- many equal or nearly equal scores, or a wanted key outside the bracket -- block 0 goes
// on alone with further histogram passes over global memory.  The list is written and read with
// agent-scope accesses: its writers may sit on other XCDs, whose L2 this block does not see.
// A candidate is a key k with k - base <= limit, and k - base is what the further digits are of.
// selsync[h * 64 + 0] = length of the list, [+1] = blocks done, [+2] = ticket of write_kept.
__global__ __launch_bounds__(kSelThreads) void select_kernel(
    const uint64_t* __restrict__ keys_all, const uint64_t* __restrict__ edge_all,
    const uint32_t* __restrict__ hist_all, int L, int budget, uint64_t* __restrict__ sel,
    uint64_t* __restrict__ cand_all, uint32_t* __restrict__ selsync) {
    const int h = blockIdx.y, part = blockIdx.x, nparts = gridDim.x;
    const int tid = threadIdx.x;
    const uint64_t* keys = keys_all + (int64_t)h * L;
    __shared__ uint32_t hist[kBins];
    __shared__ uint64_t cand[kCand];
    __shared__ uint64_t few[kRank];
    __shared__ uint32_t wtot[kSelThreads / FC_WAVE];
    __shared__ uint64_t sh_prefix;
    __shared__ uint32_t sh_need, sh_count, sh_ncand, sh_nfew;   // lengths of cand and few: a counter each,
                                                                // zeroed barriers before anyone adds to it
    __shared__ int sh_last;

    __shared__ uint64_t edge[kEdges];
    const FcBracket br = fc_bracket(budget, L);
    if (tid < kEdges) edge[tid] = edge_all[(int64_t)h * kEdges + tid];
    if (tid == 0) sh_ncand = sh_nfew = 0u;
    if (tid < kFirstBins) hist[tid] = hist_all[(int64_t)h * kFirstBins + tid];
    __syncthreads();
    pick_bin_parallel(hist, kFirstBins, (uint32_t)budget, wtot, 0ull, 0, &sh_prefix, &sh_need, &sh_count);
    __syncthreads();
    uint32_t need = sh_need;
    uint32_t count = sh_count;        // keys in the bin chosen last
    uint64_t base, limit;
    fc_bin_keys((uint32_t)sh_prefix, edge, br.bottom - br.top, first_digit_shift(edge, br.bottom - br.top), &base, &limit);
    int rem = limit ? 64 - __clzll((long long)limit) : 0;      // undecided low bits
    uint64_t prefix = 0ull;
    if (rem == 0) {
        if (part == 0 && tid == 0) { sel[2 * h] = base; sel[2 * h + 1] = need; }
        return;
    }
    bool in_lds = false;
    uint32_t ncand = 0;
    __syncthreads();
    if (count <= (uint32_t)kCand) {
        uint64_t* cand_g = cand_all + (int64_t)h * kCand;
        uint32_t* cnt = &selsync[h * 64];
        const int lane = tid & 63;
        for (int b0 = part * kSelThreads * kUnroll; b0 < L; b0 += nparts * kSelThreads * kUnroll) {
            uint64_t kv[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int j = b0 + u * kSelThreads + tid;
                kv[u] = keys[j < L ? j : L - 1] - base;
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const bool take = kv[u] <= limit && b0 + u * kSelThreads + tid < L;
                const uint64_t m = __ballot(take);
                if (m == 0) continue;
                const int leader = __ffsll((long long)m) - 1;
                uint32_t at = 0;
                if (lane == leader)
                    at = __hip_atomic_fetch_add(cnt, (uint32_t)__popcll(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                at = __shfl(at, leader, FC_WAVE);
                if (take) {
                    const uint32_t pos = at + __popcll(m & ((1ull << lane) - 1ull));
                    if (pos < (uint32_t)kCand)   // cannot be more than the histogram counted
                        __hip_atomic_store(&cand_g[pos], kv[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this block's part of the list is out
        __syncthreads();
        if (tid == 0)
            sh_last = __hip_atomic_fetch_add(&selsync[h * 64 + 1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                      (uint32_t)(nparts - 1);
        __syncthreads();
        if (!sh_last) return;
        ncand = __hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (ncand > (uint32_t)kCand) ncand = kCand;
        for (uint32_t i = tid; i < ncand; i += kSelThreads)
            cand[i] = __hip_atomic_load(&cand_g[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        in_lds = true;
    } else if (part != 0) {
        return;       // too many candidates: block 0 goes on alone
    }
    for (;;) {
        const uint64_t himask = (rem >= 64) ? 0ull : (~0ull << rem);
        // few candidates left and still in global memory: pull them into LDS and finish there
        if (!in_lds && count <= (uint32_t)kCand) {
            for (int b0 = 0; b0 < L; b0 += kSelThreads * kUnroll) {
                uint64_t kv[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    const int j = b0 + u * kSelThreads + tid;
                    kv[u] = keys[j < L ? j : L - 1] - base;
                }
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    list_append(cand, &sh_ncand,
                                kv[u] <= limit && (kv[u] & himask) == prefix && b0 + u * kSelThreads + tid < L, kv[u]);
            }
            __syncthreads();
            ncand = sh_ncand;
            in_lds = true;
        }
        if (in_lds && count <= (uint32_t)kRank) {   // very few: no more digits
            for (uint32_t i0 = 0; i0 < ncand; i0 += kSelThreads) {
                const uint64_t k = (i0 + tid < ncand) ? cand[i0 + tid] : 0ull;
                list_append(few, &sh_nfew, i0 + tid < ncand && (k & himask) == prefix, k);
            }
            __syncthreads();
            rank_select(few, sh_nfew, need, &sh_prefix, &sh_need);
            __syncthreads();
            prefix = sh_prefix;
            need = sh_need;
            break;
        }
        const int w = in_lds ? (rem < 8 ? rem : 8) : (rem < kDigitBits ? rem : kDigitBits);
        const int shift = rem - w;
        const int nb = 1 << w;
        for (int i = tid; i < nb; i += kSelThreads) hist[i] = 0;
        __syncthreads();
        if (in_lds) {
            for (uint32_t i0 = 0; i0 < ncand; i0 += kSelThreads) {
                const uint32_t i = i0 + tid;
                const uint64_t k = (i < ncand) ? cand[i] : 0ull;
                hist_add(hist, i < ncand && (k & himask) == prefix, (uint32_t)(k >> shift) & (nb - 1));
            }
        } else {
            for (int b0 = 0; b0 < L; b0 += kSelThreads * kUnroll) {
                uint64_t kv[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    const int j = b0 + u * kSelThreads + tid;
                    kv[u] = keys[j < L ? j : L - 1] - base;
                }
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    hist_add(hist, kv[u] <= limit && (kv[u] & himask) == prefix && b0 + u * kSelThreads + tid < L,
                             (uint32_t)(kv[u] >> shift) & (nb - 1));
            }
        }
        __syncthreads();
        pick_bin_parallel(hist, nb, need, wtot, prefix, shift, &sh_prefix, &sh_need, &sh_count);
        __syncthreads();
        prefix = sh_prefix;
        need = sh_need;
        count = sh_count;
        rem = shift;
        if (rem == 0) break;
    }
    if (tid == 0) {
        sel[2 * h] = base + prefix;
        sel[2 * h + 1] = need;
    }
}

// ---- ordered compaction of the kept positions: position = #greater before + min(#equal
//      before, need).  A block (2048 tokens, drawn from the head's ticket counter so that lower
//      blocks are always already running) publishes how many of its keys lie above and at the
//      threshold, in one 64-bit word with a valid bit, and then adds up the words of the blocks
//      below it -- they publish before they look at anyone else's, so every wait ends.
__global__ __launch_bounds__(kThreads) void write_kept_kernel(const uint64_t* __restrict__ keys_all,
                                                              const uint64_t* __restrict__ sel, int L,
                                                              int budget, int32_t* __restrict__ kept_all,
                                                              uint32_t* __restrict__ sync, int ntile,
                                                              int trows, uint32_t* __restrict__ selsync,
                                                              uint64_t* __restrict__ agg_all) {
    const int h = blockIdx.y, tid = threadIdx.x;
    const int wave = tid / FC_WAVE, lane = tid & 63;
    const uint64_t* keys = keys_all + (int64_t)h * L;
    int32_t* kept = kept_all + (int64_t)h * budget;
    int32_t* tile_last = sync_tile_last(sync, gridDim.y, ntile, h);   // for the compaction that follows
    uint64_t* agg = agg_all + (int64_t)h * gridDim.x;
    const uint64_t thr = sel[2 * h];
    const uint32_t need = (uint32_t)sel[2 * h + 1];
    __shared__ uint32_t wtot[2][kThreads / FC_WAVE];
    __shared__ int sh_blk;
    if (tid == 0)
        sh_blk = (int)__hip_atomic_fetch_add(&selsync[h * 64 + 2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int blk = sh_blk;
    const int first = blk * kTokBlk;

    const int j0 = first + tid * kItems;   // contiguous items per thread: order = position
    uint32_t fgt = 0, feq = 0;
    uint64_t kv[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) kv[i] = (j0 + i < L) ? keys[j0 + i] : 0ull;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        if (j0 + i < L) {
            fgt |= (kv[i] > thr) ? (1u << i) : 0u;
            feq |= (kv[i] == thr) ? (1u << i) : 0u;
        }
    }
    const uint32_t cg = __popc(fgt), ce = __popc(feq);
    uint32_t sg = cg, se = ce;   // inclusive wave scans
#pragma unroll
    for (int o = 1; o < FC_WAVE; o <<= 1) {
        const uint32_t tg = __shfl_up(sg, o, FC_WAVE);
        const uint32_t te = __shfl_up(se, o, FC_WAVE);
        if (lane >= o) { sg += tg; se += te; }
    }
    if (lane == 63) { wtot[0][wave] = sg; wtot[1][wave] = se; }
    __syncthreads();
    uint32_t gt_before = sg - cg, eq_before = se - ce;
    uint32_t tot_g = 0, tot_e = 0;
#pragma unroll
    for (int w = 0; w < kThreads / FC_WAVE; ++w) {
        if (w < wave) { gt_before += wtot[0][w]; eq_before += wtot[1][w]; }
        tot_g += wtot[0][w];
        tot_e += wtot[1][w];
    }
    if (tid == 0)
        __hip_atomic_store(&agg[blk], (1ull << 63) | ((uint64_t)tot_g << 32) | (uint64_t)tot_e, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    // what lies below this block
    uint32_t ng = 0, ne = 0;
    bool ok = true;
    for (int b = tid; b < blk; b += kThreads) {
        uint64_t v = __hip_atomic_load(&agg[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint32_t spins = 0;
        while (!(v >> 63)) {
            if (++spins > kSpinLimit) { ok = false; break; }
            __builtin_amdgcn_s_sleep(2);
            v = __hip_atomic_load(&agg[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        ng += (uint32_t)(v >> 32) & 0x7fffffffu;
        ne += (uint32_t)v;
    }
    if (!ok) atomicOr(&sync[0], 2u);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { ng += __shfl_xor(ng, o, FC_WAVE); ne += __shfl_xor(ne, o, FC_WAVE); }
    __syncthreads();
    if (lane == 0) { wtot[0][wave] = ng; wtot[1][wave] = ne; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kThreads / FC_WAVE; ++w) { gt_before += wtot[0][w]; eq_before += wtot[1][w]; }
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const bool g = (fgt >> i) & 1u, e = (feq >> i) & 1u;
        if (g || (e && eq_before < need)) {
            const uint32_t pos = gt_before + (eq_before < need ? eq_before : need);
            kept[pos] = j0 + i;
            if ((pos + 1) % (uint32_t)trows == 0 || (int)pos == budget - 1) tile_last[pos / (uint32_t)trows] = j0 + i;
        }
        gt_before += g ? 1u : 0u;
        eq_before += e ? 1u : 0u;
    }
}

// ---- a head of at most kSmallL keys: scores, select and kept positions by one block.  Such a call is
// bound by its launches, each a chain of dependent round trips (4 heads of 1312 keys: the three
// kernels above 25 us of the call's 44, this one 11).  Same operations per token, same order of the
// sum of e, so the same keys.
template <typename MT>
__global__ __launch_bounds__(kSelThreads) void select_small_kernel(
    const double* __restrict__ e_all, const MT* __restrict__ mass_all, const double* __restrict__ pz_all, int nblkz,
    int L, int budget, int pool_k, double lambda, int32_t* __restrict__ kept_all, uint32_t* __restrict__ sync, int ntile,
    int trows) {
    constexpr int PER = kSmallL / kSelThreads;
    const int h = blockIdx.x, tid = threadIdx.x, wave = tid / FC_WAVE, lane = tid & 63;
    const double* e = e_all + (int64_t)h * L;
    const MT* mass = mass_all + (int64_t)h * L;
    int32_t* kept = kept_all + (int64_t)h * budget;
    int32_t* tile_last = sync_tile_last(sync, gridDim.x, ntile, h);
    __shared__ MT ms[kSmallL];
    __shared__ uint64_t keys[kSmallL];
    __shared__ double shd[kThreads + 1];
    __shared__ uint32_t hist[kBins];
    __shared__ uint64_t few[kRank];
    __shared__ uint64_t red[2][kSelThreads / FC_WAVE];
    __shared__ uint32_t wtot[2][kSelThreads / FC_WAVE];
    __shared__ uint64_t sh_prefix;
    __shared__ uint32_t sh_need, sh_count, sh_n;

    double ev[PER];
    MT imp[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int j = i * kSelThreads + tid;
        ev[i] = e[j < L ? j : L - 1];
        imp[i] = mass[j < L ? j : L - 1];
    }
    double z = 0.0;   // the order of score_keys
    if (tid < kThreads)
        for (int i = tid; i < nblkz; i += kThreads) z += pz_all[(int64_t)h * nblkz + i];
    {   // what the compaction starts from
        uint32_t* flags = sync_flags(sync, gridDim.x, ntile, h);
        for (int i = tid; i < ntile; i += kSelThreads) flags[i] = 0u;
        if (tid == 0) sync[64 * (h + 1)] = 0u;
        if (h == 0 && tid == 0) sync[0] = 0u;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) ms[i * kSelThreads + tid] = imp[i];
    if (tid == 0) sh_n = 0u;
    z = block_sum_fixed(z, shd);   // its barriers publish ms too
    const int half = pool_k / 2;
    for (int d = 1; d <= half; ++d) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int j = i * kSelThreads + tid;
            if (j < L) {
                const MT lo = (j - d >= 0) ? ms[j - d] : imp[i];
                const MT hi = (j + d < L) ? ms[j + d] : imp[i];
                const MT nb = lo > hi ? lo : hi;
                imp[i] = imp[i] > nb ? imp[i] : nb;
            }
        }
    }
    uint64_t kv[PER], kmin = ~0ull, kmax = 0ull;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int j = i * kSelThreads + tid;
        kv[i] = 0ull;
        if (j < L) {
            kv[i] = token_key(ev[i], (double)imp[i], z, lambda);
            kmin = kv[i] < kmin ? kv[i] : kmin;
            kmax = kv[i] > kmax ? kv[i] : kmax;
            keys[j] = kv[i];
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint64_t a = (uint64_t)__shfl_xor((long long)kmin, o, FC_WAVE), b = (uint64_t)__shfl_xor((long long)kmax, o, FC_WAVE);
        kmin = a < kmin ? a : kmin;
        kmax = b > kmax ? b : kmax;
    }
    if (lane == 0) { red[0][wave] = kmin; red[1][wave] = kmax; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSelThreads / FC_WAVE; ++w) {
        kmin = red[0][w] < kmin ? red[0][w] : kmin;
        kmax = red[1][w] > kmax ? red[1][w] : kmax;
    }
    // The first cut in bins of equal width in the score: with scores of both signs the keys' leading digits are their
    // exponents, and most of a head shares two or three of those.  The bin number never falls as the score
    // rises, so the bin that holds the wanted key is a range of keys.  Scoring and selection of 4 heads of 1312 keys
    // 24.5 -> 21.7 us, 12 of 4096 29.3 -> 23.8, 24 of 3000 33.2 -> 28.3: one histogram instead of two or three.
    uint32_t need = (uint32_t)budget, count = (uint32_t)L;
    uint64_t prefix = 0ull;
    int rem = kmax > kmin ? 64 - __clzll((long long)(kmax - kmin)) : 0;
    const double smin = key_score(kmin), width = key_score(kmax) - smin;
    if (count > (uint32_t)kRank && width > 0.0 && width < 1.0e300) {
        const double per = (double)kBins / width;
        uint32_t bin[PER];
        for (int i = tid; i < kBins; i += kSelThreads) hist[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const bool in = i * kSelThreads + tid < L;
            const double at = (key_score(kv[i]) - smin) * per;
            bin[i] = in ? (uint32_t)(at < (double)(kBins - 1) ? at : (double)(kBins - 1)) : ~0u;
            if (in) atomicAdd(&hist[bin[i]], 1u);
        }
        __syncthreads();
        pick_bin_parallel(hist, kBins, need, wtot[0], 0ull, 0, &sh_prefix, &sh_need, &sh_count);
        __syncthreads();
        if (sh_count <= (uint32_t)kRank) {
            const uint32_t want = (uint32_t)sh_prefix, left = sh_need;
#pragma unroll
            for (int i = 0; i < PER; ++i) list_append(few, &sh_n, bin[i] == want, kv[i] - kmin);
            __syncthreads();
            rank_select(few, sh_n, left, &sh_prefix, &sh_need);
            __syncthreads();
            prefix = sh_prefix;
            need = sh_need;
            rem = 0;
        }
    }
    // digits of the distance from the smallest key, until few candidates are left
    while (rem > 0) {
        const uint64_t himask = (rem >= 64) ? 0ull : (~0ull << rem);
        if (count <= (uint32_t)kRank) {
#pragma unroll
            for (int i = 0; i < PER; ++i)
                list_append(few, &sh_n, i * kSelThreads + tid < L && ((kv[i] - kmin) & himask) == prefix, kv[i] - kmin);
            __syncthreads();
            rank_select(few, sh_n, need, &sh_prefix, &sh_need);
            __syncthreads();
            prefix = sh_prefix;
            need = sh_need;
            break;
        }
        const int w = rem < kDigitBits ? rem : kDigitBits, shift = rem - w, nb = 1 << w;
        for (int i = tid; i < nb; i += kSelThreads) hist[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i)
            hist_add(hist, i * kSelThreads + tid < L && ((kv[i] - kmin) & himask) == prefix,
                     (uint32_t)((kv[i] - kmin) >> shift) & (uint32_t)(nb - 1));
        __syncthreads();
        pick_bin_parallel(hist, nb, need, wtot[0], prefix, shift, &sh_prefix, &sh_need, &sh_count);
        __syncthreads();
        prefix = sh_prefix;
        need = sh_need;
        count = sh_count;
        rem = shift;
    }
    const uint64_t thr = kmin + prefix;
    // kept positions in order: #greater before + min(#equal before, need)
    const int j0 = tid * PER;
    uint32_t fgt = 0, feq = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (j0 + i < L) {
            fgt |= (keys[j0 + i] > thr) ? (1u << i) : 0u;
            feq |= (keys[j0 + i] == thr) ? (1u << i) : 0u;
        }
    }
    const uint32_t cg = __popc(fgt), ce = __popc(feq);
    uint32_t sg = cg, se = ce;
#pragma unroll
    for (int o = 1; o < FC_WAVE; o <<= 1) {
        const uint32_t tg = __shfl_up(sg, o, FC_WAVE), te = __shfl_up(se, o, FC_WAVE);
        if (lane >= o) { sg += tg; se += te; }
    }
    __syncthreads();
    if (lane == 63) { wtot[0][wave] = sg; wtot[1][wave] = se; }
    __syncthreads();
    uint32_t gt_before = sg - cg, eq_before = se - ce;
    for (int w = 0; w < wave; ++w) { gt_before += wtot[0][w]; eq_before += wtot[1][w]; }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const bool g = (fgt >> i) & 1u, q = (feq >> i) & 1u;
        if (g || (q && eq_before < need)) {
            const uint32_t pos = gt_before + (eq_before < need ? eq_before : need);
            kept[pos] = j0 + i;
            if ((pos + 1) % (uint32_t)trows == 0 || (int)pos == budget - 1) tile_last[pos / (uint32_t)trows] = j0 + i;
        }
        gt_before += g ? 1u : 0u;
        eq_before += q ? 1u : 0u;
    }
}

__global__ void iota_kernel(int32_t* kept, int H, int n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < (int64_t)H * n) kept[i] = (int32_t)(i % n);
}

// ---- in-place compaction ---------------------------------------------------------------
// Rows are VPR 16-byte vectors; a tile is tile_rows() destination rows of one head.  The launch is a
// fixed number of blocks that draw tiles from ONE ticket counter until it runs out: ticket g is
// tile g / H of head g % H, so a head's tiles are drawn in ascending order while consecutive
// tickets -- the tiles in flight at any moment -- are spread over all heads and seldom depend
// on one another.  Tile t may overwrite rows that a lower tile of its head still has to read
// (sources never lie below their destination): it stores only after every lower tile whose
// last source row reaches into its rows has published "read".
// A block works on its tiles in a two-stage pipeline: before it waits for the current tile's predecessors
// and stores it, it requests the next tile's row indices, what it needs to know about the tile's
// predecessors (their last source row, their flag) and, in launches of many tiles per block or per head,
// the rows themselves.
// (Rows loaded early are safe: no tile is stored before the lower tiles that read from it say so, and
// higher ones never do.  They pay where a block has many tiles or heads are long: with the rows requested only after
// the stores, a block that waited had nothing in flight: 12 heads of 51000 -> 40800 rows, 15 tiles per block, 126
// us, now 112; of 20000 -> 18000, 7, 65 and 60; 4 of 46900 -> 37353 float rows, 5 and 584 tiles per head, the call
// 108 and 104; 24 of 74880 -> 37440, where few tiles wait, 190 and 192.  Elsewhere the stores, behind the wait
// for the row indices, come too late: 12 of 4494 -> 4036, 1.5 tiles per block and 64 per head, 24.1, early 26.1; 24
// of 6761 -> 5804, 4.3 and 91, 40.4 and 43.6.)  Every wait ends: a tile waits only for tiles of lower
// tickets; such a tile is held by a running block either as its current tile (published as soon
// as its rows have arrived, before that block waits for anything) or as its next tile, which
// becomes current once that block's current tile -- drawn earlier still -- is done; following
// the waits leads strictly back in drawing order, so there is no cycle.
template <int VPR>
__global__ __launch_bounds__(kThreads) void compact_rows_kernel(
    uint4* __restrict__ k_cache, uint4* __restrict__ v_cache, int64_t head_stride_v,
    int64_t tok_stride_v, int H, int L, int budget, int ntile, const int32_t* __restrict__ kept_all,
    uint32_t* __restrict__ sync) {
    constexpr int kTileRows = tile_rows(VPR * 16);
    constexpr int LDN = kTileRows * VPR / kThreads;   // vectors per thread per matrix
    constexpr int RPP = kThreads / VPR;               // rows per pass
    // (the first ticket has a word of its own: no barrier lies between its reads and the store of the second)
    __shared__ uint32_t sh_first, sh_ticket;
    const int tid = threadIdx.x;
    const int lrow = tid / VPR, lcol = tid % VPR;
    const uint32_t total = (uint32_t)ntile * (uint32_t)H;
    const bool early = total >= 5u * gridDim.x || ntile >= 160;   // the next tile's rows before this one waits, see above
    uint32_t* ticket = &sync[64];

    // what a tile needs before its rows can be requested
    struct Tile {
        int h, tile;
        int src[LDN];
        int t_first, last_first;      // the nearest lower tile this thread looks at, its last source row
        uint32_t flag_first;          // and its "read" flag as seen when the indices were requested
    };
    auto request = [&](uint32_t g, Tile& T) {
        T.h = (int)(g % (uint32_t)H);
        T.tile = (int)(g / (uint32_t)H);
        const int32_t* kept = kept_all + (int64_t)T.h * budget;
#pragma unroll
        for (int p = 0; p < LDN; ++p) {
            const int s = T.tile * kTileRows + p * RPP + lrow;
            T.src[p] = (s < budget) ? kept[s] : -1;
        }
        T.t_first = T.tile - 1 - tid;
        T.last_first = -1;
        T.flag_first = 1u;
        if (T.t_first >= 0) {
            T.last_first = sync_tile_last(sync, H, ntile, T.h)[T.t_first];
            T.flag_first = __hip_atomic_load(&sync_flags(sync, H, ntile, T.h)[T.t_first], __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        }
    };

    struct Rows { u32x4_native k[LDN], v[LDN]; };   // native vectors: the arrays stay in registers
    auto load_rows = [&](Tile& T, Rows& R) {
        const uint4* kh = k_cache + T.h * head_stride_v;
        const uint4* vh = v_cache + T.h * head_stride_v;
#pragma unroll
        for (int p = 0; p < LDN; ++p) {
            const int s = T.tile * kTileRows + p * RPP + lrow;
            if (T.src[p] >= L) T.src[p] = -1;   // never read outside the compressed range
            if (T.src[p] == s) T.src[p] = -1;   // already in place
            // branch-free: a row that is not moved loads row 0 instead (in range, value unused),
            // so that all loads of the tile are in flight together
            const int64_t a = (int64_t)(T.src[p] >= 0 ? T.src[p] : 0) * tok_stride_v + lcol;
            R.k[p] = *reinterpret_cast<const u32x4_native*>(kh + a);
            R.v[p] = *reinterpret_cast<const u32x4_native*>(vh + a);
        }
    };

    if (tid == 0) sh_first = atomicAdd(ticket, 1u);
    __syncthreads();
    uint32_t g = sh_first;
    if (g >= total) return;
    Tile cur;
    Rows rows;
    request(g, cur);
    load_rows(cur, rows);
    uint32_t g_next = 0;
    if (tid == 0) g_next = atomicAdd(ticket, 1u);               // travels with the rows
    for (;;) {
        const int row0 = cur.tile * kTileRows;
        uint4* kh = k_cache + cur.h * head_stride_v;
        uint4* vh = v_cache + cur.h * head_stride_v;
        uint32_t* flags = sync_flags(sync, H, ntile, cur.h);
        const int32_t* tile_last = sync_tile_last(sync, H, ntile, cur.h);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // the rows are in registers
        if (tid == 0) sh_ticket = g_next;
        __syncthreads();
        // No fence: nothing this block wrote has to become visible -- only the ORDER "rows
        // loaded, then flag" matters, and the loads have returned.  (A release fence here would
        // write back the whole L2 of this XCD, once per tile.)
        if (tid == 0) __hip_atomic_fetch_or(&flags[cur.tile], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        g = sh_ticket;
        const bool more = g < total;
        Tile nxt;
        Rows nrows;
        auto next_rows = [&]() {
            load_rows(nxt, nrows);
            if (tid == 0) g_next = atomicAdd(ticket, 1u);
        };
        if (more) request(g, nxt);            // on its way while this tile waits and stores
        if (more && early) next_rows();
        // Lower tiles whose last (= largest) source row is >= row0 read from this tile's rows.
        // The last source rows ascend with the tile, so each thread walks down from its nearest
        // tile and stops at the first one that ends below row0.
        bool ok = true;
        int t = cur.t_first, last = cur.last_first;
        uint32_t flag = cur.flag_first;
        while (t >= 0 && last >= row0) {
            uint32_t spins = 0;
            while (flag == 0u) {
                if (++spins > kSpinLimit) { ok = false; break; }
                __builtin_amdgcn_s_sleep(2);
                flag = __hip_atomic_load(&flags[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            t -= kThreads;
            if (t >= 0) {
                last = tile_last[t];
                flag = __hip_atomic_load(&flags[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (!ok) atomicOr(&sync[0], 1u);
        __syncthreads();
#pragma unroll
        for (int p = 0; p < LDN; ++p) {
            const int s = row0 + p * RPP + lrow;
            if (cur.src[p] >= 0) {
                const int64_t a = (int64_t)s * tok_stride_v + lcol;
                // streaming stores: written the ordinary way, up to a cache's worth of these rows
                // stays behind as dirty lines and is written back during whichever kernel runs
                // next (a following pass over 460 MB of cold keys: 118 us instead of 90)
                __builtin_nontemporal_store(rows.k[p], reinterpret_cast<u32x4_native*>(kh + a));
                __builtin_nontemporal_store(rows.v[p], reinterpret_cast<u32x4_native*>(vh + a));
            }
        }
        if (!more) break;
        if (!early) next_rows();
        cur = nxt;
        rows = nrows;
    }
}

// What compact_rows starts from, for the calls that bring their own kept list: zeroed tickets,
// flags and status word, and every tile's last source row.  grid = (blocks, H).
__global__ __launch_bounds__(kThreads) void prep_compact_kernel(uint32_t* __restrict__ sync, int H, int ntile,
                                                                const int32_t* __restrict__ kept_all,
                                                                int budget, int trows) {
    const int h = blockIdx.y;
    uint32_t* flags = sync_flags(sync, H, ntile, h);
    int32_t* tile_last = sync_tile_last(sync, H, ntile, h);
    for (int t = blockIdx.x * kThreads + threadIdx.x; t < ntile; t += gridDim.x * kThreads) {
        flags[t] = 0u;
        const int e = ((t + 1) * trows < budget ? (t + 1) * trows : budget) - 1;
        tile_last[t] = kept_all[(int64_t)h * budget + e];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sync[64 * (h + 1)] = 0u;
        if (h == 0) sync[0] = 0u;
    }
}

// Blocks of the compaction: two per compute unit, never more than there are tiles.  Measured (12 heads
// of 51000 -> 40800 rows of 256 bytes / 24 of 74880 -> 37440): 256 blocks 119 / 215 us, 384 116 / 201, 512 112
// / 193, 640 116 / 195 -- more streams in flight keep less of each open DRAM page in use.
unsigned compact_grid(int ntile, int H) {
    const int64_t tiles = (int64_t)ntile * H;
    return (unsigned)(tiles < 512 ? tiles : 512);
}

struct WsLayout {
    size_t e, keys, psum, pz, edge, hist, sel, cand, selsync, agg, sync, total;
    int nblk, nb2, ntile;
};

WsLayout layout(int H, int L, int d, int budget, fc_dtype dtype) {
    WsLayout w;
    int nblk = (L + kGroups * 16 - 1) / (kGroups * 16);   // one round of 16 tokens per group
    // three blocks per compute unit over all heads: the passes run at what the memory system
    // gives for one large read stream with small per-token side streams, whatever the launch
    // shape (512 to 4096 blocks were within 3 % of each other), so the partials stay few
    const int cap = 768 / (H > 0 ? H : 1) > 0 ? 768 / (H > 0 ? H : 1) : 1;
    if (nblk > cap) nblk = cap;
    if (nblk < 1) nblk = 1;
    w.nblk = nblk;
    w.nb2 = (L + kTokBlk - 1) / kTokBlk;
    const size_t esz = (dtype == FC_BF16) ? 2 : 4;
    size_t off = 0;
    w.e = off;       off += fc_align_up((size_t)H * L * 8);
    w.keys = off;    off += fc_align_up((size_t)H * L * 8);
    w.psum = off;    off += fc_align_up((size_t)H * nblk * d * 8);
    w.pz = off;      off += fc_align_up((size_t)H * nblk * 8);
    w.edge = off;    off += fc_align_up((size_t)H * kEdges * 8);
    w.hist = off;    off += fc_align_up((size_t)H * kFirstBins * 4);
    w.sel = off;     off += fc_align_up((size_t)H * 16);
    w.cand = off;    off += fc_align_up((size_t)H * kCand * 8);
    w.selsync = off; off += fc_align_up((size_t)H * 64 * 4);
    w.agg = off;     off += fc_align_up((size_t)H * w.nb2 * 8);
    const int trows = tile_rows(d * (int)esz);
    w.ntile = (((budget < L) ? budget : L) + trows - 1) / trows;
    w.sync = off;    off += fc_align_up(sync_words(H, w.ntile) * 4);
    w.total = off;
    return w;
}

template <typename T, int D, typename MT>
int launch_typed(const FcCompressArgs& a, const MT* mass, hipStream_t s, bool compact = true) {
    const WsLayout w = layout(a.H_k, a.L_k, a.d, a.budget, a.dtype);
    // (the float64 instantiation moves no rows: its layout has the tiles of four-byte rows)
    constexpr int TR = tile_rows(D * (int)(sizeof(T) == 8 ? 4 : sizeof(T)));
    if constexpr (sizeof(T) <= 4) {   // (the float64 instantiation scores pooled keys: no rows to move)
        if (a.phase == 2) {           // rows only: the kept list is the caller's
            uint32_t* sync2 = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(a.ws) + w.sync);
            prep_compact_kernel<<<dim3((w.ntile + kThreads - 1) / kThreads, a.H_k), kThreads, 0, s>>>(
                sync2, a.H_k, w.ntile, a.kept, a.budget, TR);
            FC_LAUNCH_CHECK();
            constexpr int VPR2 = D * (int)sizeof(T) / 16;
            const int64_t hs2 = a.head_stride * (int64_t)sizeof(T) / 16, ts2 = a.tok_stride * (int64_t)sizeof(T) / 16;
            compact_rows_kernel<VPR2><<<dim3(compact_grid(w.ntile, a.H_k)), kThreads, 0, s>>>(
                (uint4*)a.k_cache, (uint4*)a.v_cache, hs2, ts2, a.H_k, a.L_k, a.budget, w.ntile, a.kept, sync2);
            FC_LAUNCH_CHECK();
            return FC_OK;
        }
    }
    char* ws = reinterpret_cast<char*>(a.ws);
    double* e = reinterpret_cast<double*>(ws + w.e);
    uint64_t* keys = reinterpret_cast<uint64_t*>(ws + w.keys);
    double* psum = reinterpret_cast<double*>(ws + w.psum);
    double* pz = reinterpret_cast<double*>(ws + w.pz);
    uint64_t* edge = reinterpret_cast<uint64_t*>(ws + w.edge);
    uint32_t* hist = reinterpret_cast<uint32_t*>(ws + w.hist);
    uint64_t* sel = reinterpret_cast<uint64_t*>(ws + w.sel);
    uint64_t* cand = reinterpret_cast<uint64_t*>(ws + w.cand);
    uint32_t* selsync = reinterpret_cast<uint32_t*>(ws + w.selsync);
    uint64_t* agg = reinterpret_cast<uint64_t*>(ws + w.agg);
    uint32_t* sync = reinterpret_cast<uint32_t*>(ws + w.sync);
    const T* kc = reinterpret_cast<const T*>(a.k_cache);

    // rounds of 8 tokens for two-byte storage (the widened rows stay in registers), of 16 otherwise
    constexpr int R = sizeof(T) == 2 ? 8 : 16;
    key_stats_kernel<T, D, R><<<dim3(w.nblk, a.H_k), kThreads, 0, s>>>(kc, a.head_stride, a.tok_stride,
                                                                      a.L_k, psum);
    FC_LAUNCH_CHECK();
    const bool small = a.L_k <= kSmallL;
    mean_sim_kernel<T, D, R><<<dim3(w.nblk, a.H_k), kThreads, 0, s>>>(
        kc, a.head_stride, a.tok_stride, a.L_k, psum, w.nblk, e, pz, small ? nullptr : hist);
    FC_LAUNCH_CHECK();
    if (small) {
        select_small_kernel<MT><<<a.H_k, kSelThreads, 0, s>>>(e, mass, pz, w.nblk, a.L_k, a.budget, a.pool_k, a.lambda,
                                                              a.kept, sync, w.ntile, TR);
        FC_LAUNCH_CHECK();
    } else {
        score_keys_kernel<MT><<<dim3((a.L_k + kScoreBlk - 1) / kScoreBlk, a.H_k), kScoreThreads, 0, s>>>(e, mass, pz, w.nblk, a.L_k, a.budget, a.pool_k,
                                                                  a.lambda, keys, edge, hist, sync, w.ntile,
                                                                  selsync, agg, w.nb2);
        FC_LAUNCH_CHECK();
        // blocks per head that scan for the candidates: one batch of loads each, up to 131072 keys
        constexpr int kBatch = kSelThreads * kUnroll;
        const int nparts = a.L_k <= 16 * kBatch ? (a.L_k + kBatch - 1) / kBatch : 16;
        select_kernel<<<dim3(nparts, a.H_k), kSelThreads, 0, s>>>(keys, edge, hist, a.L_k, a.budget, sel, cand,
                                                                 selsync);
        FC_LAUNCH_CHECK();
        write_kept_kernel<<<dim3(w.nb2, a.H_k), kThreads, 0, s>>>(keys, sel, a.L_k, a.budget, a.kept, sync, w.ntile, TR,
                                                                  selsync, agg);
        FC_LAUNCH_CHECK();
    }
    if (!compact || a.phase == 1) return FC_OK;   // scoring and selection only
    if constexpr (sizeof(T) <= 4) {
        constexpr int VPR = D * (int)sizeof(T) / 16;
        const int64_t hs = a.head_stride * (int64_t)sizeof(T) / 16, ts = a.tok_stride * (int64_t)sizeof(T) / 16;
        compact_rows_kernel<VPR><<<dim3(compact_grid(w.ntile, a.H_k)), kThreads, 0, s>>>(
            (uint4*)a.k_cache, (uint4*)a.v_cache, hs, ts, a.H_k, a.L_k, a.budget, w.ntile, a.kept, sync);
        FC_LAUNCH_CHECK();
    }
    return FC_OK;
}

// ---- key granularity above the token (frame- or chunk-level keys, App. D.2.1) ------------
// Group g = tokens [g*group, (g+1)*group): its key is the mean key, its importance the mean
// mass, both float64 sums in a fixed order divided by the group size and kept as float64.
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void group_pool_kernel(
    const T* __restrict__ k_cache, int64_t head_stride, int64_t tok_stride, int group, int G,
    const float* __restrict__ mass, int L, double* __restrict__ k_pooled,
    double* __restrict__ mass_pooled) {
    typedef Slice<T, D> S;
    constexpr int EL = S::EL;
    const int g = blockIdx.x, h = blockIdx.y;
    const int r0 = threadIdx.x / 16, u = threadIdx.x % 16;
    const T* base = k_cache + (int64_t)h * head_stride + (int64_t)g * group * tok_stride;
    double acc[EL];
#pragma unroll
    for (int e = 0; e < EL; ++e) acc[e] = 0.0;
    for (int r = r0; r < group; r += kGroups) {
        double x[EL];
        S::widen(S::load(base + (int64_t)r * tok_stride, u), x);
#pragma unroll
        for (int e = 0; e < EL; ++e) acc[e] += x[e];
    }
    __shared__ double sh[kGroups][D];
    __shared__ double shm[kThreads + 1];
#pragma unroll
    for (int e = 0; e < EL; ++e) sh[r0][u * EL + e] = acc[e];
    double m = 0.0;
    for (int r = threadIdx.x; r < group; r += kThreads) m += (double)mass[(int64_t)h * L + (int64_t)g * group + r];
    m = block_sum_fixed(m, shm);   // includes the barrier that publishes sh
    if (threadIdx.x < D) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < kGroups; ++k) t += sh[k][threadIdx.x];
        k_pooled[((int64_t)h * G + g) * D + threadIdx.x] = t / (double)group;
    }
    if (threadIdx.x == 0) mass_pooled[(int64_t)h * G + g] = m / (double)group;
}

// kept groups -> kept token positions
__global__ __launch_bounds__(kThreads) void expand_groups_kernel(
    const int32_t* __restrict__ kept_groups, int n_groups, int group, int32_t* __restrict__ kept) {
    const int h = blockIdx.y;
    const int64_t n = (int64_t)n_groups * group;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads)
        kept[(int64_t)h * n + i] = kept_groups[(int64_t)h * n_groups + i / group] * group + (int32_t)(i % group);
}

struct GroupedLayout {
    size_t k_pooled, mass_pooled, kept_groups, inner, sync, total;
    int G, Bg, ntile;      // (64-row tiles; longer ones need less of the sync area)
};

GroupedLayout grouped_layout(int H, int L, int d, int budget, int group) {
    GroupedLayout w;
    w.G = L / group;
    w.Bg = budget / group;
    w.ntile = (budget + 63) / 64;
    size_t off = 0;
    w.k_pooled = off;    off += fc_align_up((size_t)H * w.G * d * 8);
    w.mass_pooled = off; off += fc_align_up((size_t)H * w.G * 8);
    w.kept_groups = off; off += fc_align_up((size_t)H * (w.Bg > 0 ? w.Bg : 1) * 4);
    w.inner = off;       off += layout(H, w.G, d, w.Bg > 0 ? w.Bg : 1, FC_F32).total;
    w.sync = off;        off += fc_align_up(sync_words(H, w.ntile) * 4);
    w.total = off;
    return w;
}

template <typename T, int D>
int launch_grouped(const FcCompressArgs& a, hipStream_t s) {
    const GroupedLayout w = grouped_layout(a.H_k, a.L_k, a.d, a.budget, a.group);
    char* ws = reinterpret_cast<char*>(a.ws);
    double* k_pooled = reinterpret_cast<double*>(ws + w.k_pooled);
    double* mass_pooled = reinterpret_cast<double*>(ws + w.mass_pooled);
    int32_t* kept_groups = reinterpret_cast<int32_t*>(ws + w.kept_groups);
    uint32_t* sync = reinterpret_cast<uint32_t*>(ws + w.sync);
    group_pool_kernel<T, D><<<dim3(w.G, a.H_k), kThreads, 0, s>>>(
        (const T*)a.k_cache, a.head_stride, a.tok_stride, a.group, w.G, a.mass, a.L_k, k_pooled,
        mass_pooled);
    FC_LAUNCH_CHECK();
    // the token-level scoring and selection, run on the groups
    FcCompressArgs b = a;
    b.k_cache = k_pooled; b.v_cache = k_pooled;
    b.head_stride = (int64_t)w.G * D; b.tok_stride = D; b.dtype = FC_F32;
    b.L_k = w.G; b.budget = w.Bg; b.mass = nullptr; b.kept = kept_groups; b.ws = ws + w.inner;
    b.group = 1;
    const int st = launch_typed<double, D, double>(b, mass_pooled, s, false);
    if (st != FC_OK) return st;
    int gx = (int)(((int64_t)w.Bg * a.group + kThreads * 4 - 1) / (kThreads * 4));
    gx = gx < 1 ? 1 : (gx > 256 ? 256 : gx);
    expand_groups_kernel<<<dim3(gx, a.H_k), kThreads, 0, s>>>(kept_groups, w.Bg, a.group, a.kept);
    FC_LAUNCH_CHECK();
    constexpr int VPR = D * (int)sizeof(T) / 16, TR = tile_rows(VPR * 16);
    const int ntile = (a.budget + TR - 1) / TR;
    prep_compact_kernel<<<dim3((ntile + kThreads - 1) / kThreads, a.H_k), kThreads, 0, s>>>(
        sync, a.H_k, ntile, a.kept, a.budget, TR);
    FC_LAUNCH_CHECK();
    const int64_t hs = a.head_stride * (int64_t)sizeof(T) / 16, ts = a.tok_stride * (int64_t)sizeof(T) / 16;
    compact_rows_kernel<VPR><<<dim3(compact_grid(ntile, a.H_k)), kThreads, 0, s>>>(
        (uint4*)a.k_cache, (uint4*)a.v_cache, hs, ts, a.H_k, a.L_k, a.budget, ntile, a.kept, sync);
    FC_LAUNCH_CHECK();
    return FC_OK;
}

}  // namespace

size_t fc_compress_grouped_workspace(int H_k, int L_k, int d, int budget, int group) {
    return grouped_layout(H_k, L_k, d, budget, group).total;
}

size_t fc_compress_status_offset(int H_k, int L_k, int d, int budget, int group, fc_dtype dtype) {
    if (group > 1) return grouped_layout(H_k, L_k, d, budget, group).sync;
    return layout(H_k, L_k, d, budget, dtype).sync;
}

size_t fc_compress_workspace(int H_k, int L_k, int d, int budget, fc_dtype dtype) {
    return layout(H_k, L_k, d, budget, dtype).total;
}

int fc_launch_compress(const FcCompressArgs& a, hipStream_t s) {
    if (a.budget >= a.L_k) {  // cache-filling phase: nothing to drop
        if (a.phase == 2) return FC_OK;   // every row is already in place
        const int64_t n = (int64_t)a.H_k * a.L_k;
        iota_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(a.kept, a.H_k, a.L_k);
        FC_LAUNCH_CHECK();
        return FC_OK;
    }
    if (a.group > 1) {
        if (a.dtype == FC_BF16) {
            if (a.d == 128) return launch_grouped<bf16_t, 128>(a, s);
            if (a.d == 64) return launch_grouped<bf16_t, 64>(a, s);
        } else {
            if (a.d == 128) return launch_grouped<float, 128>(a, s);
            if (a.d == 64) return launch_grouped<float, 64>(a, s);
        }
        return FC_UNSUPPORTED;
    }
    if (a.dtype == FC_BF16) {
        if (a.d == 128) return launch_typed<bf16_t, 128, float>(a, a.mass, s);
        if (a.d == 64) return launch_typed<bf16_t, 64, float>(a, a.mass, s);
    } else {
        if (a.d == 128) return launch_typed<float, 128, float>(a, a.mass, s);
        if (a.d == 64) return launch_typed<float, 64, float>(a, a.mass, s);
    }
    return FC_UNSUPPORTED;
}
