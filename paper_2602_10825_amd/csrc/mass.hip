// Per-key attention mass (importance), Sec. 3.3 Eq. (9), over an observation window of
// query rows (App. C.2: the last 50 tokens of the last denoising chunk).
//
//   mass[h_k, j] = 1/(W*G) * sum over rows w and the G query heads of key head h_k of
//                  softmax_j(q_w . k_j * scale), the softmax running over j < mass_len only.
//
// Two passes over the keys (the softmax normaliser of a row is known only after all keys):
//   stats  per-row (reference point, sum of exp2 above it) per range of keys -> partials
//   lse    (between them) per row: the partials merged, fixed order     -> log2-sum-exp
//   cols   per key: sum over rows of exp2(s - lse), fixed order         -> mass
// Both passes run on the matrix cores.  bf16 with one group of 64 rows: 128-key tiles staged through
// LDS by coalesced 16-byte loads (the passes are bound by the two reads of K), each in the
// orientation that makes its reduction in-lane: stats forms S^T = K Q^T (one row per lane,
// its keys in registers: the row's max and sum need no exchange, 8 partials per row are
// merged once per block); cols forms S = Q K^T (one key per lane, the 64 padded rows in
// registers: the key's sum over rows is in-lane).  bf16 with more rows, and fp32, are bound by
// arithmetic and have kernels of their own.  Every sum has a fixed order: the result is
// deterministic.  No atomics.
#include "f32_split.hpp"

namespace {

constexpr int kRowGroup = 64;
constexpr int kNT = 256;
constexpr float kPosBig = 1.0e30f;
constexpr float kNegBig = -1.0e30f;
constexpr float kLog2e = 1.4426950408889634f;

// First observation row; handles the "tail of the last compact block" addressing when n_rec is given.
__device__ __forceinline__ bool resolve_rows(const FcMassArgs& a, int64_t& row0) {
    if (a.n_rec) {
        const int R = *a.n_rec;
        if (R <= 0 || R > a.A || a.rec_idx[R - 1] != a.A - 1) return false;
        row0 = (int64_t)R * a.L_c - a.W;
    } else {
        row0 = 0;
    }
    return true;
}

// ---- fp32: on the bf16 matrix cores ---------------------------------------------------
// Both operands in three bf16 parts (f32_split.hpp), read straight into registers in the products' own layout:
// lane (half, n) holds elements 16 st + 8 half .. + 8 of row n.
// Both passes form S^T = K Q^T, one observation row per lane.  A wavefront keeps 32 rows (pass 1) or 32 keys
// (pass 2), split once, and passes over the others, whose next step is split between the products of this
// one, while the rows after those are loaded over them.  Pass 1's rows are split once for the block, in LDS: with them in
// registers head dimension 128 took 256 of those, and 12 heads, 50 rows on 4000 keys 65 us.  Bound by the vector ALU and the
// lines that a load touches in large calls and by latency in small ones.
// Whole call, us, fp32 matrix cores / now: four query heads on one x 64, 50 rows on 512 keys 19.5 / 15.3; 12 x 128, 50 rows on
// 4000 keys 54 / 44, on 51000 358 / 263; 12 x 64, 969 rows on 10647 keys 398 / 271; 8 heads on 2 x 128, 1671 rows on 1892 keys
// 289 / 185.  Error against float64 of 17 shapes 0.45 to 1.0 of that of the fp32 matrix cores, nowhere larger.
constexpr int kF32Waves = 8;

// Columns 16 st + 8 half .. + 8 for st < N of a row, given from column 8 half on.
template <int N>
__device__ __forceinline__ void load_row_f32(const float* row, f32x4_t (&f)[2 * N]) {
#pragma unroll
    for (int st = 0; st < N; ++st) {
        f[2 * st] = *reinterpret_cast<const f32x4_t*>(row + 16 * st);
        f[2 * st + 1] = *reinterpret_cast<const f32x4_t*>(row + 16 * st + 4);
    }
}
// S^T of the operand that stays, `stay(st)`, and the rows that pass: `f` holds the first N steps of `row`, and of `next` when
// this returns.  STAY_K: keys stay (and Q passes).  `stay_row`, `row`, `next`: this lane's row of each in memory, from column
// 8 half on.  Once more with fp32 products where an entry has no parts, or loses some (`odd`: of the operand that stays).
// Times c2, rounded: unrounded in one instruction with the maximum's subtraction, the largest score would not cancel, and from
// 2^31 on its exponential is infinite.
template <int D, bool STAY_K, int N, typename F>
__device__ __forceinline__ f32x16_t scores_f32(F stay, bool odd, const float* stay_row, f32x4_t (&f)[2 * N],
                                               const float* row, const float* next, float c2) {
    constexpr int KS = D / 16;
    static_assert(KS % N == 0, "a step's place in f is the same in every row");
    f32x16_t c, c1;                                            // the largest products, and the others
#pragma unroll
    for (int i = 0; i < 16; ++i) c[i] = c1[i] = 0.f;
    Split8 cur, nxt;
    auto split = [&](Split8& x, int st, int p) __attribute__((always_inline)) {
        const f32x4_t& v = f[2 * (st % N) + (p >> 1)];
        split_pair(x, p, v[2 * (p & 1)], v[2 * (p & 1) + 1]);
    };
#pragma unroll
    for (int p = 0; p < 4; ++p) split(cur, 0, p);
#pragma unroll
    for (int st = 0; st < KS; ++st) {
        const Split8 x = stay(st);
        const Split8 &k = STAY_K ? x : cur, &q = STAY_K ? cur : x;
        const bool more = st + 1 < KS;
        const float* from = st + N < KS ? row + 16 * (st + N) : next + 16 * (st + N - KS);
        f[2 * (st % N)] = *reinterpret_cast<const f32x4_t*>(from);
        f[2 * (st % N) + 1] = *reinterpret_cast<const f32x4_t*>(from + 4);
        split_mfma(k.l, q.h, c1); if (more) split(nxt, st + 1, 0); __builtin_amdgcn_sched_barrier(0);
        split_mfma(k.h, q.l, c1); __builtin_amdgcn_sched_barrier(0);
        split_mfma(k.m, q.m, c1); if (more) split(nxt, st + 1, 1); __builtin_amdgcn_sched_barrier(0);
        split_mfma(k.m, q.h, c1); if (more) split(nxt, st + 1, 2); __builtin_amdgcn_sched_barrier(0);
        split_mfma(k.h, q.m, c1); __builtin_amdgcn_sched_barrier(0);
        split_mfma(k.h, q.h, c); if (more) split(nxt, st + 1, 3); __builtin_amdgcn_sched_barrier(0);
        cur = nxt;
    }
    c += c1;
#pragma unroll
    for (int i = 0; i < 16; ++i) odd = odd || !__builtin_isfinite(c[i]);
    if (__any(odd)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) c[i] = 0.f;
#pragma unroll 1
        for (int st = 0; st < KS; ++st)
#pragma unroll
            for (int j = 0; j < 2; ++j) {                      // contracts over elements that lie 8 apart
                const f32x4_t x = *reinterpret_cast<const f32x4_t*>((STAY_K ? stay_row : row) + 16 * st + 4 * j);
                const f32x4_t y = *reinterpret_cast<const f32x4_t*>((STAY_K ? row : stay_row) + 16 * st + 4 * j);
#pragma unroll
                for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i], y[i], c, 0, 0, 0);
            }
    }
    {
#pragma clang fp contract(off)
        return c * c2;
    }
}

// log2-sum-exp from the largest exponent and the sum above it.  log2(sum) = e + log2(f), 1/2 <= f < 1, so that
// the logarithm's own error (one of its last place) stays below the one rounding of the total: mx + e in two
// terms.  (mx + log2(sum) as it stands made every entry of the importance wrong by up to 3e-7, now 1e-7.)
__device__ __forceinline__ float log2_sum(float mx, float sum) {
    const float e = (float)__builtin_amdgcn_frexp_expf(sum), f = __builtin_amdgcn_frexp_mantf(sum);
    const float hi = mx + e, b = hi - mx;
    const float lo = (mx - (hi - b)) + (e - b);
    return hi + (lo + __builtin_amdgcn_logf(f));
}
// A row with at most kFewPartials of them is merged by whoever needs it; the launch between the passes is left out
// (four heads on one x 64, 50 rows on 512 keys: 3.0 of 22 us).  With more, each block of pass 2 would read and merge
// them all, and on a full cache that took longer than the launch; and with many tiles of rows each wavefront of
// pass 2 merges again for every tile (12 x 64, 969 rows on 10647 keys 248 -> 281 us).
constexpr int kFewPartials = 4, kFewTiles = 8;
__device__ __forceinline__ float lse_of_few(const float* __restrict__ m, const float* __restrict__ l, int np) {
    float mi[kFewPartials], li[kFewPartials], mx = kNegBig, sum = 0.f;
#pragma unroll
    for (int i = 0; i < kFewPartials; ++i) {
        mi[i] = i < np ? m[i] : kNegBig;
        li[i] = i < np ? l[i] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < kFewPartials; ++i) mx = fmaxf(mx, mi[i]);
#pragma unroll
    for (int i = 0; i < kFewPartials; ++i) sum = fmaf(li[i], __builtin_amdgcn_exp2f(mi[i] - mx), sum);
    return log2_sum(mx, sum);
}

// A tile of rows is 32 of the W * G that use one key head: with a tile of its own for every query head,
// 24 x 128 with four heads on one, two rows each, took 367 us on 16384 keys (one tile for the eight: 135).
struct F32Row { int h, w; bool ok; };
__device__ __forceinline__ F32Row f32_row(const FcMassArgs& a, int hk, int r) {
    const int G = a.H_q / a.H_k;
    const bool ok = r < a.W * G;
    const int g = ok ? r / a.W : 0;
    return F32Row{hk * G + g, ok ? r - g * a.W : 0, ok};
}

// Pass 1: a block is 32 rows of one key head and one of S key ranges; its wavefronts take every eighth
// 32-key tile and are merged through LDS.
template <int D>
__global__ __launch_bounds__(kF32Waves * 64, 2) void mass_stats_f32_kernel(FcMassArgs a, int nrg, int S, float* __restrict__ pm,
                                                                          float* __restrict__ pl) {
    int64_t row0;
    if (!resolve_rows(a, row0)) return;
    const int s = blockIdx.x % S, rt = blockIdx.x / S, hk = blockIdx.y;   // (only grid.x takes any number of rows)
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n = lane & 31, half = lane >> 5;
    const float* kh = (const float*)a.k_cache + (int64_t)hk * a.head_stride;
    const float c2 = a.scale * kLog2e;
    const int T = (a.mass_len + 31) / 32;
    const int t_end = (int)((int64_t)T * (s + 1) / S);
    const F32Row row = f32_row(a, hk, rt * 32 + n);               // padding rows: computed, not used
    const float* q_row = (const float*)a.q_base + ((row0 + row.w) * a.H_q + row.h) * D + 8 * half;
    f32x4_t k[D / 8];
    auto k_row = [&](int t) {
        const int j = t * 32 + n < a.mass_len ? t * 32 + n : a.mass_len - 1;
        return kh + (int64_t)j * a.tok_stride + 8 * half;
    };
    int t = (int)((int64_t)T * s / S) + wave;
    if (t < t_end) load_row_f32<D / 16>(k_row(t), k);
    // Q's parts, once for the block
    constexpr int QROW = D + 8;
    __shared__ __attribute__((aligned(16))) bf16_t qs[3][32 * QROW];
    bool odd = false;
    if (tid < 32 * (D / 8)) {
        const int e = tid % (D / 8);
        const F32Row r = f32_row(a, hk, rt * 32 + tid / (D / 8));
        const float* p = (const float*)a.q_base + ((row0 + r.w) * a.H_q + r.h) * D + 8 * e;
        f32x4_t v[2] = {*reinterpret_cast<const f32x4_t*>(p), *reinterpret_cast<const f32x4_t*>(p + 4)};
        Split8 x;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            odd = odd || odd_magnitude(v[0][i]) || odd_magnitude(v[1][i]);
            split_pair(x, i, v[i >> 1][2 * (i & 1)], v[i >> 1][2 * (i & 1) + 1]);
        }
        bf16_t* at = &qs[0][tid / (D / 8) * QROW + 8 * e];
        *reinterpret_cast<u32x4_native*>(at) = x.h;
        *reinterpret_cast<u32x4_native*>(at + 32 * QROW) = x.m;
        *reinterpret_cast<u32x4_native*>(at + 64 * QROW) = x.l;
    }
    __shared__ __attribute__((aligned(16))) uint32_t odd_s[kF32Waves];   // by the wavefront that split the rows
    odd = __any(odd);
    if (lane == 0) odd_s[wave] = odd;
    __syncthreads();
    const u32x4_native odd0 = *reinterpret_cast<const u32x4_native*>(odd_s), odd1 = *reinterpret_cast<const u32x4_native*>(odd_s + 4);
    odd = (odd0[0] | odd0[1] | odd0[2] | odd0[3] | odd1[0] | odd1[1] | odd1[2] | odd1[3]) != 0u;
    auto q = [&](int st) __attribute__((always_inline)) {
        const bf16_t* at = &qs[0][n * QROW + 8 * half + 16 * st];
        return Split8{*reinterpret_cast<const u32x4_native*>(at), *reinterpret_cast<const u32x4_native*>(at + 32 * QROW),
                      *reinterpret_cast<const u32x4_native*>(at + 64 * QROW)};
    };
    float m = kNegBig, l = 0.f;
    for (; t < t_end; t += kF32Waves) {
        const f32x16_t st = scores_f32<D, false, D / 16>(q, odd, q_row, k, k_row(t), k_row(t + kF32Waves < t_end ? t + kF32Waves : t), c2);
        const int key0 = t * 32 + half * 4;
        const bool full = t * 32 + 32 <= a.mass_len;
        float tm = kNegBig;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (full || key0 + (r >> 2) * 8 + (r & 3) < a.mass_len) tm = fmaxf(tm, st[r]);
        const float mn = fmaxf(m, tm);
        float acc = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (full || key0 + (r >> 2) * 8 + (r & 3) < a.mass_len) acc += __builtin_amdgcn_exp2f(st[r] - mn);
        // no real key yet (m and mn both at the floor): keep l = 0
        l = (mn > kNegBig) ? fmaf(l, __builtin_amdgcn_exp2f(m - mn), acc) : 0.f;
        m = mn;
    }
    __shared__ float merge[2][2 * kF32Waves][32];
    merge[0][wave * 2 + half][n] = m;
    merge[1][wave * 2 + half][n] = l;
    __syncthreads();
    if (tid < 32 && row.ok) {                                     // (lane n of the first wavefront: its own row)
        float mx = kNegBig, sum = 0.f;
#pragma unroll
        for (int i = 0; i < 2 * kF32Waves; ++i) mx = fmaxf(mx, merge[0][i][tid]);
#pragma unroll
        for (int i = 0; i < 2 * kF32Waves; ++i) sum = fmaf(merge[1][i][tid], __builtin_amdgcn_exp2f(merge[0][i][tid] - mx), sum);
        const int64_t at = ((int64_t)row.h * nrg * kRowGroup + row.w) * S + s;
        pm[at] = mx;
        pl[at] = sum;
    }
}

// Sums over the 32 lanes n of 16 values each: in the step for lane bit k a lane keeps the half of
// its values whose index has bit k like its own; lane n ends with the sum of value n % 16.
__device__ __forceinline__ float lanes_sum_scatter(float (&v)[16], int n) {
#pragma unroll
    for (int k = 1; k < 16; k <<= 1) {
        const bool up = n & k;
#pragma unroll
        for (int i = 0; i < 8 / k; ++i) {
            const float keep = up ? v[2 * i + 1] : v[2 * i], give = up ? v[2 * i] : v[2 * i + 1];
            v[i] = keep + __shfl_xor(give, k, FC_WAVE);
        }
    }
    return v[0] + __shfl_xor(v[0], 16, FC_WAVE);
}

// Pass 2: a wavefront keeps 32 keys; `parts` wavefronts of a block share the 32-row tiles of the key head
// (every parts-th each) and are added up in order.  NW wavefronts per block: with few tiles of rows four, of which the
// registers of head dimension 64 let three blocks run at once where one of eight would (50 rows, 4 heads on one x 64, 512
// keys 17.7 -> 15.3 us for the call; 12 x 128, 4000 keys 47 -> 43.7; 2 x 64, 32 rows on 39849 keys 32.3 -> 29.5); with many the eight
// wavefronts share their rows in the L1 (12 x 64, 969 rows on 10647 keys 271, in blocks of four 292).
template <int D, int NW>
__global__ __launch_bounds__(NW * 64, D == 64 && NW < kF32Waves ? 3 : 2) void mass_cols_f32_kernel(FcMassArgs a, int nrg, int parts,
                                                                         const float* __restrict__ lse2, const float* __restrict__ pm,
                                                                         const float* __restrict__ pl, int np) {
    const int hk = blockIdx.y, kb = NW / parts;             // key blocks of 32 per block
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n = lane & 31, half = lane >> 5;
    const int jb = blockIdx.x * kb * 32;
    int64_t row0;
    if (!resolve_rows(a, row0)) {
        if (tid < kb * 32 && jb + tid < a.mass_len) a.mass[(int64_t)hk * a.mass_len + jb + tid] = __uint_as_float(0x7fc00000u);
        return;
    }
    __shared__ float merge[NW][32];
    const int G = a.H_q / a.H_k;
    const int part = wave / kb, key0 = jb + (wave % kb) * 32;
    const float c2 = a.scale * kLog2e;
    const int nt = (int)(((int64_t)a.W * G + 31) / 32);            // tiles of 32 rows
    float sums[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) sums[r] = 0.f;
    const float* k_row = (const float*)a.k_cache + (int64_t)hk * a.head_stride + (int64_t)(key0 + n < a.mass_len ? key0 + n : a.mass_len - 1) * a.tok_stride + 8 * half;
    constexpr int N = 4;                                           // steps of the passing rows in flight: they come from the caches
    Split8 kp[D / 16];
    f32x4_t q[2 * N];
    bool odd = false;
    float ls = 0.f;
    const float *q_row = nullptr, *q_next = nullptr;
    auto next_q = [&](int t) {                                     // rows and normalisers of tile t
        const F32Row row = f32_row(a, hk, t * 32 + n);
        q_next = (const float*)a.q_base + ((row0 + row.w) * a.H_q + row.h) * D + 8 * half;
        const int64_t at = (int64_t)row.h * nrg * kRowGroup + row.w;
        const float v = lse2 ? lse2[at] : lse_of_few(pm + at * np, pl + at * np, np);
        ls = row.ok ? v : __builtin_inff();                        // padding rows: their terms vanish
    };
    if (part < nt) {
        next_q(part);
        load_row_f32<N>(q_next, q);
    }
    {
        f32x4_t f[D / 8];
        load_row_f32<D / 16>(k_row, f);
#pragma unroll
        for (int j = 0; j < D / 4; ++j) {
            const float x = f[j >> 1][2 * (j & 1)], y = f[j >> 1][2 * (j & 1) + 1];
            odd = odd || odd_magnitude(x) || odd_magnitude(y);
            split_pair(kp[j >> 2], j & 3, x, y);
        }
    }
    auto k = [&](int st) __attribute__((always_inline)) { return kp[st]; };
    for (int t = part; t < nt; t += parts) {
        const float neg = -ls;
        q_row = q_next;
        if (t + parts < nt) next_q(t + parts);
        const f32x16_t st = scores_f32<D, true, N>(k, odd, k_row, q, q_row, q_next, c2);
#pragma unroll
        for (int r = 0; r < 16; ++r) sums[r] += __builtin_amdgcn_exp2f(st[r] + neg);
    }
    const float v = lanes_sum_scatter(sums, n);
    if (n < 16) merge[wave][(n >> 2) * 8 + half * 4 + (n & 3)] = v;
    __syncthreads();
    if (tid < kb * 32 && jb + tid < a.mass_len) {
        float tot = 0.f;
        for (int p = 0; p < parts; ++p) tot += merge[p * kb + (tid >> 5)][tid & 31];
        a.mass[(int64_t)hk * a.mass_len + jb + tid] = tot / (float)(a.W * G);
    }
}

// Few rows per key head, W * G <= kFewRows: one thread per key, its key in registers, the rows broadcast
// from LDS.  Bound by the two reads of K.
constexpr int kFewRows = 8;

template <int D>
__device__ __forceinline__ void load_key_f32(const FcMassArgs& a, int hk, int j, f32x4_t (&k)[D / 4]) {
    const float* p = (const float*)a.k_cache + (int64_t)hk * a.head_stride + (int64_t)(j < a.mass_len ? j : a.mass_len - 1) * a.tok_stride;
#pragma unroll
    for (int e = 0; e < D / 4; ++e) k[e] = *reinterpret_cast<const f32x4_t*>(p + 4 * e);
}
template <int D>
__device__ __forceinline__ float dot_f32(const f32x4_t (&k)[D / 4], const float* q) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < D; ++e) s = fmaf(k[e / 4][e % 4], q[e], s);
    return s;
}
__device__ __forceinline__ void stage_rows_f32(const FcMassArgs& a, int64_t row0, int hk, int rows, int D, float* qs) {
    for (int i = threadIdx.x; i < rows * D; i += kNT) {
        const F32Row row = f32_row(a, hk, i / D);
        qs[i] = ((const float*)a.q_base)[((row0 + row.w) * a.H_q + row.h) * D + i % D];
    }
}

template <int D>
__global__ __launch_bounds__(kNT) void mass_stats_f32_few_kernel(FcMassArgs a, int np, float* __restrict__ pm,
                                                                float* __restrict__ pl) {
    int64_t row0;
    if (!resolve_rows(a, row0)) return;
    const int hk = blockIdx.y, tid = threadIdx.x, rows = a.W * (a.H_q / a.H_k);
    const int j = blockIdx.x * kNT + tid;
    __shared__ __attribute__((aligned(16))) float qs[kFewRows * D];
    stage_rows_f32(a, row0, hk, rows, D, qs);
    f32x4_t k[D / 4];
    load_key_f32<D>(a, hk, j, k);
    __syncthreads();
    const float c2 = a.scale * kLog2e;
    const int slot = blockIdx.x * (kNT / FC_WAVE) + tid / FC_WAVE;
    int at = hk * (a.H_q / a.H_k) * kRowGroup;        // of the row's partials; the head's rows are a.W of kRowGroup
    for (int r = 0, w = 0; r < rows; ++r) {
        const float s = j < a.mass_len ? dot_f32<D>(k, qs + r * D) * c2 : kNegBig;
        const float mx = wave_max_all(s);
        const float sum = wave_sum_all(__builtin_amdgcn_exp2f(s - mx));
        if (tid % FC_WAVE == 0) {
            pm[(int64_t)(at + w) * np + slot] = mx;
            pl[(int64_t)(at + w) * np + slot] = sum;
        }
        if (++w == a.W) { w = 0; at += kRowGroup; }
    }
}

template <int D>
__global__ __launch_bounds__(kNT) void mass_cols_f32_few_kernel(FcMassArgs a, const float* __restrict__ lse2) {
    const int hk = blockIdx.y, tid = threadIdx.x;
    const int j = blockIdx.x * kNT + tid;
    int64_t row0;
    if (!resolve_rows(a, row0)) {
        if (j < a.mass_len) a.mass[(int64_t)hk * a.mass_len + j] = __uint_as_float(0x7fc00000u);
        return;
    }
    const int rows = a.W * (a.H_q / a.H_k);
    __shared__ __attribute__((aligned(16))) float qs[kFewRows * D];
    stage_rows_f32(a, row0, hk, rows, D, qs);
    f32x4_t k[D / 4];
    load_key_f32<D>(a, hk, j, k);
    __syncthreads();
    const float c2 = a.scale * kLog2e;
    float acc = 0.f;
    const float* ls = lse2 + hk * (a.H_q / a.H_k) * kRowGroup;
    for (int r = 0, w = 0; r < rows; ++r) {
        acc += __builtin_amdgcn_exp2f(dot_f32<D>(k, qs + r * D) * c2 - ls[w]);
        if (++w == a.W) { w = 0; ls += kRowGroup; }
    }
    if (j < a.mass_len) a.mass[(int64_t)hk * a.mass_len + j] = acc / (float)rows;
}

// Between the passes: log2-sum-exp of every observation row over all keys, from the blocks'
// partials.  One block per (row group, query head); four lanes per row take every fourth
// partial (loads batched four deep) and merge in a fixed order.  Padding rows get a huge
// normaliser: their terms vanish.
__global__ __launch_bounds__(kNT) void mass_lse_kernel(const float* __restrict__ pm,
                                                            const float* __restrict__ pl, int nrg, int np,
                                                            int W, float* __restrict__ lse2) {
    const int rg = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
    const int w0 = rg * kRowGroup;
    const int nw = (W - w0 < kRowGroup) ? W - w0 : kRowGroup;
    const int row = tid >> 2, part = tid & 3;
    const float* m = pm + (((int64_t)h * nrg + rg) * kRowGroup + row) * np;
    const float* l = pl + (((int64_t)h * nrg + rg) * kRowGroup + row) * np;
    float mx = kNegBig, sum = 0.f;
    for (int i0 = part; i0 < np; i0 += 16) {
        float mi[4], li[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + 4 * u;
            mi[u] = i < np ? m[i] : kNegBig;
            li[u] = i < np ? l[i] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float mn = fmaxf(mx, mi[u]);
            sum = sum * __builtin_amdgcn_exp2f(mx - mn) + li[u] * __builtin_amdgcn_exp2f(mi[u] - mn);
            mx = mn;
        }
    }
#pragma unroll
    for (int o = 1; o < 4; o <<= 1) {
        const float mo = __shfl_xor(mx, o, FC_WAVE), so = __shfl_xor(sum, o, FC_WAVE);
        const float mn = fmaxf(mx, mo);
        // the lower lane's term first on both sides, so partners agree bit for bit
        const float lo = (part & o) ? so * __builtin_amdgcn_exp2f(mo - mn) : sum * __builtin_amdgcn_exp2f(mx - mn);
        const float hi = (part & o) ? sum * __builtin_amdgcn_exp2f(mx - mn) : so * __builtin_amdgcn_exp2f(mo - mn);
        sum = lo + hi;
        mx = mn;
    }
    if (part == 0) {
        lse2[((int64_t)h * nrg + rg) * kRowGroup + row] = row < nw ? log2_sum(mx, sum) : kPosBig;
    }
}

// ---- bf16: matrix-core passes -------------------------------------------------------

constexpr int kTile = 128;            // keys per tile: 4 wavefronts x 32 keys
constexpr int kTilesPerBlock = 8;      // at most
constexpr int kMinTilesPerBlock = 4;
constexpr int kSpan = kTile * kTilesPerBlock;

template <int D>
struct __attribute__((aligned(16))) MassSmem {
    // rows padded by 16 bytes: the 16-byte fragment reads of 32 consecutive rows then fall
    // on distinct LDS banks.  The 16-byte alignment is what lets them be single ds_read_b128.
    __attribute__((aligned(16))) bf16_t q[kRowGroup][D + 8];
    union __attribute__((aligned(16))) {
        __attribute__((aligned(16))) bf16_t k[kTile][D + 8];
        float merge[2][32][17];          // (max, sum) partials of the rows, after the tile loop
    };
    float lse[kRowGroup];
    float acc[kSpan];
};

template <int D>
__device__ __forceinline__ void stage_q_bf16(const FcMassArgs& a, int64_t row0, int h,
                                             bf16_t (*qs)[D + 8]) {
    constexpr int PR = D / 8;   // 16-byte pieces per row
    for (int i = threadIdx.x; i < kRowGroup * PR; i += kNT) {
        const int w = i / PR, c = i % PR;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (w < a.W)
            v = *reinterpret_cast<const uint4*>((const bf16_t*)a.q_base +
                                                ((row0 + w) * a.H_q + h) * D + c * 8);
        *reinterpret_cast<uint4*>(&qs[w][c * 8]) = v;
    }
}

// 128-key tile -> registers (coalesced: consecutive threads take consecutive 16-byte pieces);
// rows past mass_len re-read the last valid row and are masked by the callers.
template <int D>
__device__ __forceinline__ void fetch_ktile(const FcMassArgs& a, const bf16_t* kh, int j0,
                                            u32x4_native (&kr)[D / 16]) {
    constexpr int PR = D / 8;
#pragma unroll
    for (int i = 0; i < D / 16; ++i) {
        const int p = threadIdx.x + kNT * i;
        int j = j0 + p / PR;
        j = j < a.mass_len ? j : a.mass_len - 1;
        kr[i] = *reinterpret_cast<const u32x4_native*>(kh + (int64_t)j * a.tok_stride + (p % PR) * 8);
    }
}
template <int D>
__device__ __forceinline__ void store_ktile(bf16_t (*ks)[D + 8], const u32x4_native (&kr)[D / 16]) {
    constexpr int PR = D / 8;
#pragma unroll
    for (int i = 0; i < D / 16; ++i) {
        const int p = threadIdx.x + kNT * i;
        *reinterpret_cast<u32x4_native*>(&ks[p / PR][(p % PR) * 8]) = kr[i];
    }
}

// S[row][key] for the 64 staged rows and this wavefront's 32 keys of the tile:
// s[rb][r] = row rb*32 + (r/4)*8 + (lane/32)*4 + r%4, key = wave*32 + lane%32.
template <int D>
__device__ __forceinline__ void tile_scores(const MassSmem<D>& sm, int wave, int lane,
                                            f32x16_t (&s)[2]) {
    const int n = lane & 31, half = lane >> 5;
    bf16x8_t kf[D / 16];
#pragma unroll
    for (int kb = 0; kb < D / 16; ++kb)
        kf[kb] = *reinterpret_cast<const bf16x8_t*>(&sm.k[wave * 32 + n][kb * 16 + half * 8]);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        f32x16_t c = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int kb = 0; kb < D / 16; ++kb) {
            const bf16x8_t qf =
                *reinterpret_cast<const bf16x8_t*>(&sm.q[rb * 32 + n][kb * 16 + half * 8]);
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf, kf[kb], c, 0, 0, 0);
        }
        s[rb] = c;
    }
}

// S^T[key][row] for this wavefront's 32 keys of the tile and the 64 staged rows (the operands
// of tile_scores swapped): st[rb][r] = key wave*32 + (r/4)*8 + (lane/32)*4 + r%4,
// row rb*32 + lane%32 -- one observation row per lane, so its max and sum are in-lane.
template <int D>
__device__ __forceinline__ void tile_scores_t(const MassSmem<D>& sm, int wave, int lane,
                                              f32x16_t (&st)[2]) {
    const int n = lane & 31, half = lane >> 5;
    bf16x8_t kf[D / 16];
#pragma unroll
    for (int kb = 0; kb < D / 16; ++kb)
        kf[kb] = *reinterpret_cast<const bf16x8_t*>(&sm.k[wave * 32 + n][kb * 16 + half * 8]);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        f32x16_t c = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int kb = 0; kb < D / 16; ++kb) {
            const bf16x8_t qf =
                *reinterpret_cast<const bf16x8_t*>(&sm.q[rb * 32 + n][kb * 16 + half * 8]);
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb], qf, c, 0, 0, 0);
        }
        st[rb] = c;
    }
}

// Pass 1: per observation row, max and sum of exp2 over this block's span of keys.
template <int D>
__global__ __launch_bounds__(kNT, 2) void mass_stats_bf16_kernel(FcMassArgs a, int np, int tpb,
                                                              float* __restrict__ pm,
                                                              float* __restrict__ pl) {
    int64_t row0;
    if (!resolve_rows(a, row0)) return;
    __shared__ __attribute__((aligned(16))) MassSmem<D> sm;
    const int h = blockIdx.y;
    const int hk = h / (a.H_q / a.H_k);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int n = lane & 31, half = lane >> 5;
    const bf16_t* kh = (const bf16_t*)a.k_cache + (int64_t)hk * a.head_stride;
    const int span = tpb * kTile;
    const int jb = blockIdx.x * span;
    const int left = a.mass_len - jb;
    const int nt = left >= span ? tpb : (left + kTile - 1) / kTile;
    const float c2 = a.scale * kLog2e;
    u32x4_native kr[D / 16];
    fetch_ktile<D>(a, kh, jb, kr);             // on its way while the rows are staged
    stage_q_bf16<D>(a, row0, h, sm.q);
    float m[2] = {kNegBig, kNegBig}, l[2] = {0.f, 0.f};   // of row rb*32 + n over this lane's keys
    for (int t = 0; t < nt; ++t) {
        __syncthreads();
        store_ktile<D>(sm.k, kr);
        __syncthreads();
        if (t + 1 < nt) fetch_ktile<D>(a, kh, jb + (t + 1) * kTile, kr);   // never another block's tile
        f32x16_t st[2];
        tile_scores_t<D>(sm, wave, lane, st);
        const int key0 = jb + t * kTile + wave * 32 + half * 4;   // + (r/4)*8 + r%4
        if (key0 - half * 4 + 32 <= a.mass_len) {     // all 32 keys of this wavefront are real
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) {
                float tm = st[rb][0];
#pragma unroll
                for (int r = 1; r < 16; ++r) tm = fmaxf(tm, st[rb][r]);
                const float mn = fmaxf(m[rb], tm * c2);
                float acc = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc += __builtin_amdgcn_exp2f(fmaf(st[rb][r], c2, -mn));
                l[rb] = fmaf(l[rb], __builtin_amdgcn_exp2f(m[rb] - mn), acc);
                m[rb] = mn;
            }
        } else {                                      // the ragged end of the scored range
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) {
                float tm = kNegBig;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (key0 + (r >> 2) * 8 + (r & 3) < a.mass_len) tm = fmaxf(tm, st[rb][r] * c2);
                const float mn = fmaxf(m[rb], tm);
                float acc = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (key0 + (r >> 2) * 8 + (r & 3) < a.mass_len)
                        acc += __builtin_amdgcn_exp2f(fmaf(st[rb][r], c2, -mn));
                // no real key yet (m and mn both at the floor): keep l = 0
                l[rb] = (mn > kNegBig) ? fmaf(l[rb], __builtin_amdgcn_exp2f(m[rb] - mn), acc) : 0.f;
                m[rb] = mn;
            }
        }
    }
    // merge the 8 partials of every row (4 wavefronts x 2 lane halves), in a fixed order
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        sm.merge[0][rb * 16 + (n >> 1)][(n & 1) * 8 + wave * 2 + half] = m[rb];
        sm.merge[1][rb * 16 + (n >> 1)][(n & 1) * 8 + wave * 2 + half] = l[rb];
    }
    __syncthreads();
    if (tid < kRowGroup) {
        const int q = tid;   // rb*32 + n
        const float* mp = &sm.merge[0][(q >> 5) * 16 + ((q & 31) >> 1)][(q & 1) * 8];
        const float* lp = &sm.merge[1][(q >> 5) * 16 + ((q & 31) >> 1)][(q & 1) * 8];
        float mx = kNegBig;
#pragma unroll
        for (int i = 0; i < 8; ++i) mx = fmaxf(mx, mp[i]);
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) sum += lp[i] * __builtin_amdgcn_exp2f(mp[i] - mx);
        pm[((int64_t)h * kRowGroup + q) * np + blockIdx.x] = mx;
        pl[((int64_t)h * kRowGroup + q) * np + blockIdx.x] = sum;
    }
}

template <int D>
__global__ __launch_bounds__(kNT, 2) void mass_cols_bf16_kernel(FcMassArgs a, int tpb,
                                                             const float* __restrict__ lse2, const float* __restrict__ pm,
                                                             const float* __restrict__ pl, int np) {
    const int hk = gridDim.y - 1 - blockIdx.y;   // the first pass read the last heads last: they may still be cached
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int span = tpb * kTile;
    const int jb = blockIdx.x * span;
    const int left = a.mass_len - jb;
    const int nkeys = left >= span ? span : left;
    int64_t row0;
    if (!resolve_rows(a, row0)) {
        for (int i = tid; i < nkeys; i += kNT)
            a.mass[(int64_t)hk * a.mass_len + jb + i] = __uint_as_float(0x7fc00000u);
        return;
    }
    __shared__ __attribute__((aligned(16))) MassSmem<D> sm;
    const int G = a.H_q / a.H_k;
    const bf16_t* kh = (const bf16_t*)a.k_cache + (int64_t)hk * a.head_stride;
    const int nt = (nkeys + kTile - 1) / kTile;
    const float c2 = a.scale * kLog2e;
    for (int i = tid; i < kSpan; i += kNT) sm.acc[i] = 0.f;
    for (int g = 0; g < G; ++g) {
        const int h = hk * G + g;
        __syncthreads();
        u32x4_native kr[D / 16];
        fetch_ktile<D>(a, kh, jb, kr);         // on its way while the rows are staged
        stage_q_bf16<D>(a, row0, h, sm.q);
        if (tid < kRowGroup) {
            const int64_t at = (int64_t)h * kRowGroup + tid;
            sm.lse[tid] = lse2 ? lse2[at] : tid < a.W ? lse_of_few(pm + at * np, pl + at * np, np) : kPosBig;
        }
        __syncthreads();
        float lr[2][16];
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                lr[rb][r] = sm.lse[rb * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3)];
        for (int t = 0; t < nt; ++t) {
            __syncthreads();
            store_ktile<D>(sm.k, kr);
            __syncthreads();
            if (t + 1 < nt) fetch_ktile<D>(a, kh, jb + (t + 1) * kTile, kr);   // never another block's tile
            f32x16_t s[2];
            tile_scores<D>(sm, wave, lane, s);
            float v = 0.f;
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                for (int r = 0; r < 16; ++r) v += __builtin_amdgcn_exp2f(s[rb][r] * c2 - lr[rb][r]);
            v += __shfl_xor(v, 32, FC_WAVE);
            if (lane < 32) sm.acc[t * kTile + wave * 32 + lane] += v;   // one owner per key
        }
    }
    __syncthreads();
    const float inv = 1.0f / (float)(a.W * G);
    for (int i = tid; i < nkeys; i += kNT) {
        a.mass[(int64_t)hk * a.mass_len + jb + i] = sm.acc[i] * inv;
    }
}

// ---- bf16, more than one group of 64 observation rows (frame-level queries, App. D.2.1) ------
// With many row groups the product S^T = K Q^T is real matrix work.  One operand stays in a
// wavefront's registers for the whole kernel (64 rows x D), the other passes through LDS in tiles
// of 64 rows that all wavefronts of the block read:
//   stats  64 observation rows stay, a range of keys passes: per lane one row's running sum
//   cols   64 keys stay, the rows of all the head's groups pass: per lane 32 keys' running sums
// Bound: vector ALU and matrix cores alike, 16 cycles each per 64 scores and pass (fma 4, exp2 8, add 4), at the
// 1.8 to 1.95 GHz that the chip runs under both: 0.9 ms for 24 heads, 1872 rows, 74880 keys.  (Counters: matrix cores busy in
// 0.53 of the cycles, the vector ALU in 0.65, both at once in 0.35, neither in 0.17.)  So each score costs nothing but those
// three instructions -- no running maximum: the reference point m of a lane is raised only when a
// sum of 16 terms exceeds 2^40 -- and the products of a 32-row step are issued between the
// exponentials of the step before, one set of accumulators filled while the other is read.  Each
// fragment read from LDS serves two products.  (Key tiles staged once per four row groups, the
// queries double-buffered in LDS with a barrier per tile and group, a running maximum in pass 1, the
// products and the vector work of a tile one after the other, before / this, whole call, us: 24 x 128,
// 1872 rows on 74880 keys 2833 / 1681 (passes 880 and 935); 2 heads on 1, 700 rows on 60000 keys 180
// / 87; 4 x 128, 2040 rows on 700 keys 459 / 72; 24 x 64, 130 rows on 84240 keys 235 / 210.)  The loads of the
// passing tiles take a scalar base and a 32-bit offset per lane (a 64-bit product per row, lane and tile was a tenth
// of the vector work), padding rows are not cleared (their normaliser makes the terms vanish), and a sum is not added
// right behind its own exponential: 1715 -> 1630 on one card; 4 x 128, 2040 rows on 700 keys 72 -> 62; 8 heads on 2
// x 128, 97 rows on 5000 keys 33.2 -> 29.4; 24 x 64, 130 rows on 84240 keys 210 and 212.  (Exponent, exponential and
// sum of an element beside three products in turn, no vector instruction behind one that it needs: the same.)
constexpr int kStream = 64;             // rows of a tile that passes
constexpr int kRing = 3;                // tiles in LDS: read, complete, being written
constexpr float kTooBig = 1.0995116e12f;   // 2^40

template <int D>
struct __attribute__((aligned(16))) MassWideSmem {
    // padded like MassSmem::k
    __attribute__((aligned(16))) bf16_t x[kRing][kStream][D + 8];
    float lse[kRing][kStream];          // cols: the rows' normalisers
};

// One step: nxt = products of the 32 rows whose fragments start at `cur`, sums += exponentials of
// `prev`.  `frag` holds the first kAhead fragments of the step on entry and of the next one (at `after`)
// on exit.  At raised priority, so that the other wavefront of the SIMD fills the step's gaps and stores and loads
// its tiles in them (in turn on one card, medians): 24 x 64, 1872 rows on 74880 keys 1149 -> 1100 us, 130 rows on 84240 keys
// 212 -> 202; 24 x 128, 1872 rows 1616 -> 1605, which is within the spread.  COLS: the resident operand is K and sums[b][r] one key each; else it is Q and sums[b][0..1]
// are two halves of the sum of row b.  neg[b]: what the exponents are lowered by.
constexpr int kAhead = 4;
template <int D, bool COLS, int NS>
__device__ __forceinline__ void mass_step(f32x16_t (&nxt)[2], const f32x16_t (&prev)[2], const bf16x8_t (&stay)[2][D / 16],
                                          bf16x8_t (&frag)[kAhead], const bf16_t* cur, const bf16_t* after, float c2,
                                          const float (&neg)[2], float (&sums)[2][NS]) {
    constexpr int KS = D / 16, E = 32 / (2 * KS);   // exponentials beside each product
    __builtin_amdgcn_s_setprio(1);
    f32x16_t zero;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero[i] = 0.f;
#pragma unroll
    for (int kb = 0; kb < KS; ++kb) {
        const bf16x8_t fr = frag[kb % kAhead];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            if constexpr (COLS)
                nxt[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(stay[b][kb], fr, kb ? nxt[b] : zero, 0, 0, 0);
            else
                nxt[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr, stay[b][kb], kb ? nxt[b] : zero, 0, 0, 0);
            if (b == 1)
                frag[kb % kAhead] = *reinterpret_cast<const bf16x8_t*>(
                    kb + kAhead < KS ? cur + (kb + kAhead) * 16 : after + (kb + kAhead - KS) * 16);
            // the exponentials first: a sum right behind its own waits for it
            float w[E];
#pragma unroll
            for (int i = 0; i < E; ++i) {
                const int e = (2 * kb + b) * E + i;
                w[i] = __builtin_amdgcn_exp2f(fmaf(prev[e >> 4][e & 15], c2, neg[e >> 4]));
                asm volatile("" : "+v"(w[i]));      // computed here, next to the matrix products
            }
#pragma unroll
            for (int i = 0; i < E; ++i) {
                const int e = (2 * kb + b) * E + i, q = e >> 4, r = e & 15;
                float& sum = sums[q][COLS ? r : r & 1];
                sum += w[i];
                asm volatile("" : "+v"(sum));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __builtin_amdgcn_s_setprio(0);
}

// The sums of step `prev` (32 keys from `key0` on, of which those below `end` count) once more, from a
// reference point that fits them: taken for the first keys, ragged ends and sums that became too big.
__device__ __forceinline__ void stats_raise(const f32x16_t (&prev)[2], int key0, int end, float c2, float (&m)[2],
                                            float (&l)[2]) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        float tm = kNegBig;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (key0 + (r >> 2) * 8 + (r & 3) < end) tm = fmaxf(tm, prev[b][r] * c2);
        const float mn = fmaxf(m[b], tm);
        float acc = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (key0 + (r >> 2) * 8 + (r & 3) < end) acc += __builtin_amdgcn_exp2f(fmaf(prev[b][r], c2, -mn));
        // no real key yet (m and mn both at the floor): keep l = 0
        l[b] = (mn > kNegBig) ? fmaf(l[b], __builtin_amdgcn_exp2f(m[b] - mn), acc) : 0.f;
        m[b] = mn;
    }
}

// Pass 1.  A block has NW wavefronts of 64 rows and one of S ranges of the keys; consecutive blocks
// of an XCD share the range (its L2 serves all but the first).
template <int D, int NW>
__global__ __launch_bounds__(NW * 64, 2) void mass_stats_wide_kernel(FcMassArgs a, int nrg, int S, float* __restrict__ pm,
                                                                    float* __restrict__ pl) {
    constexpr int KS = D / 16, PR = D / 8, NT = NW * 64, LD = kStream * PR / NT;
    int64_t row0;
    if (!resolve_rows(a, row0)) return;
    __shared__ __attribute__((aligned(16))) MassWideSmem<D> sm;
    const int RB = (nrg + NW - 1) / NW;
    const int n_items = a.H_q * S * RB, per = (n_items + 7) / 8;
    const int item = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || item >= n_items) return;
    const int s = (item / RB) % S, h = item / RB / S;
    const int hk = h / (a.H_q / a.H_k);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n = lane & 31, half = lane >> 5;
    const int rg = (item % RB) * NW + wave;
    const bool active = rg < nrg;                 // a wavefront without rows only helps to load
    const bf16_t* kh = (const bf16_t*)a.k_cache + (int64_t)hk * a.head_stride;
    const int T = (a.mass_len + kStream - 1) / kStream;
    const int t_lo = (int)((int64_t)T * s / S), nt = (int)((int64_t)T * (s + 1) / S) - t_lo;
    const float c2 = a.scale * kLog2e;

    bf16x8_t stay[2][KS];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int w = rg * kRowGroup + b * 32 + n;
        const bf16_t* qp = (const bf16_t*)a.q_base + ((row0 + (w < a.W ? w : 0)) * a.H_q + h) * D + half * 8;
#pragma unroll
        for (int kb = 0; kb < KS; ++kb) {
            u32x4_native v = *reinterpret_cast<const u32x4_native*>(qp + kb * 16);
            if (w >= a.W) v = u32x4_native{0u, 0u, 0u, 0u};
            stay[b][kb] = __builtin_bit_cast(bf16x8_t, v);
        }
    }
    u32x4_native kr[LD];
    const uint32_t row_b = (uint32_t)a.tok_stride * 2u, col_b = (uint32_t)(tid % PR) * 16u;   // (NT is a multiple of PR)
    const uint32_t off0 = (uint32_t)(tid / PR) * row_b + col_b, step = (uint32_t)(NT / PR) * row_b;
    auto fetch = [&](int t) {                     // rows past the end re-read the last one and are masked
        const int j0 = (t_lo + (t < nt ? t : nt - 1)) * kStream;
        const char* base = reinterpret_cast<const char*>(kh + (int64_t)j0 * a.tok_stride);
        const int left = a.mass_len - j0 - 1;
        const uint32_t last = (uint32_t)(left < kStream - 1 ? left : kStream - 1) * row_b + col_b;
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const uint32_t off = off0 + (uint32_t)i * step;
            kr[i] = *reinterpret_cast<const u32x4_native*>(base + (off < last ? off : last));
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const int p = tid + NT * i;
            *reinterpret_cast<u32x4_native*>(&sm.x[buf][p / PR][(p % PR) * 8]) = kr[i];
        }
    };
    fetch(0);
    store(0);
    fetch(1);
    __syncthreads();
    bf16x8_t frag[kAhead];
#pragma unroll
    for (int f = 0; f < kAhead; ++f) frag[f] = *reinterpret_cast<const bf16x8_t*>(&sm.x[0][n][f * 16 + half * 8]);
    f32x16_t sa[2], sb[2];
    float m[2] = {kNegBig, kNegBig}, l[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 16; ++i) sb[0][i] = sb[1][i] = 0.f;
    // after a step: its sums, of the 32 keys of subtile u (counted from the start of the range)
    auto take = [&](const f32x16_t (&prev)[2], const float (&sums)[2][2], int u) {
        const float s0 = sums[0][0] + sums[0][1], s1 = sums[1][0] + sums[1][1];
        const int first = t_lo * kStream + u * 32;
        if (first + 32 > a.mass_len || __any(!(s0 <= kTooBig) || !(s1 <= kTooBig)))
            stats_raise(prev, first + half * 4, a.mass_len, c2, m, l);
        else {
            l[0] += s0;
            l[1] += s1;
        }
    };
    int buf = 0;
    for (int t = 0; t < nt; ++t) {
        const int nbuf = buf + 1 == kRing ? 0 : buf + 1;
        // Tile t + 1 goes where tile t - 2 was: the barrier in the middle of t - 1 is behind every
        // wavefront's last read of that one.  Visible past this tile's barrier, read after it.
        store(nbuf);
        fetch(t + 2);
        const bf16_t* x0 = &sm.x[buf][n][half * 8];
        const bf16_t* x1 = &sm.x[buf][32 + n][half * 8];
        if (active) {
            float sums[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
            const float neg[2] = {-m[0], -m[1]};
            mass_step<D, false, 2>(sa, sb, stay, frag, x0, x1, c2, neg, sums);
            if (t > 0) take(sb, sums, 2 * t - 1);
        }
        lds_barrier();
        if (active) {
            float sums[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
            const float neg[2] = {-m[0], -m[1]};
            mass_step<D, false, 2>(sb, sa, stay, frag, x1, &sm.x[nbuf][n][half * 8], c2, neg, sums);
            take(sa, sums, 2 * t);
        }
        buf = nbuf;
    }
    if (!active) return;
    stats_raise(sb, (t_lo + nt) * kStream - 32 + half * 4, a.mass_len, c2, m, l);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        // the two lane halves saw different keys of the same rows
        const float mo = __shfl_xor(m[b], 32, FC_WAVE), lo = __shfl_xor(l[b], 32, FC_WAVE);
        const float mx = fmaxf(m[b], mo);
        const float sum = fmaf(lo, __builtin_amdgcn_exp2f(mo - mx), l[b] * __builtin_amdgcn_exp2f(m[b] - mx));
        if (half == 0) {
            const int64_t at = (((int64_t)h * nrg + rg) * kRowGroup + b * 32 + n) * S + s;
            pm[at] = mx;
            pl[at] = sum;
        }
    }
}

// Pass 2.  A block has NW wavefronts of 64 keys of one key head.
template <int D, int NW>
__global__ __launch_bounds__(NW * 64, 2) void mass_cols_wide_kernel(FcMassArgs a, int nrg, const float* __restrict__ lse2) {
    constexpr int KS = D / 16, PR = D / 8, NT = NW * 64, LD = kStream * PR / NT;
    const int hk = gridDim.y - 1 - blockIdx.y;   // the first pass read the last heads last
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n = lane & 31, half = lane >> 5;
    const int jb = blockIdx.x * NT;
    int64_t row0;
    if (!resolve_rows(a, row0)) {
        if (jb + tid < a.mass_len) a.mass[(int64_t)hk * a.mass_len + jb + tid] = __uint_as_float(0x7fc00000u);
        return;
    }
    __shared__ __attribute__((aligned(16))) MassWideSmem<D> sm;
    const int G = a.H_q / a.H_k;
    const bf16_t* kh = (const bf16_t*)a.k_cache + (int64_t)hk * a.head_stride;
    const float c2 = a.scale * kLog2e;
    const int key0 = jb + wave * 64;
    const bool active = key0 < a.mass_len;

    const int nt = G * nrg;                       // tiles of 64 rows: query head g = t / nrg, group t % nrg
    int ft = 0, fg = 0, frg = 0;                  // the tile that is fetched next
    u32x4_native qr[LD];
    float lr = 0.f;
    const uint32_t row_b = (uint32_t)a.H_q * D * 2u, col_b = (uint32_t)(tid % PR) * 16u;   // (NT is a multiple of PR)
    const uint32_t off0 = (uint32_t)(tid / PR) * row_b + col_b, step = (uint32_t)(NT / PR) * row_b;
    auto fetch = [&]() {                          // padding rows: the last one again; their normaliser makes the terms vanish
        const int h = hk * G + fg, left = a.W - frg * kRowGroup - 1;
        const char* base = reinterpret_cast<const char*>((const bf16_t*)a.q_base + ((row0 + frg * kRowGroup) * a.H_q + h) * D);
        const uint32_t last = (uint32_t)(left < kRowGroup - 1 ? left : kRowGroup - 1) * row_b + col_b;
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const uint32_t off = off0 + (uint32_t)i * step;
            qr[i] = *reinterpret_cast<const u32x4_native*>(base + (off < last ? off : last));
        }
        if (tid < kRowGroup) lr = lse2[((int64_t)h * nrg + frg) * kRowGroup + tid];
        if (++ft < nt && ++frg == nrg) { frg = 0; ++fg; }      // past the last tile: that one again
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const int p = tid + NT * i;
            *reinterpret_cast<u32x4_native*>(&sm.x[buf][p / PR][(p % PR) * 8]) = qr[i];
        }
        if (tid < kRowGroup) sm.lse[buf][tid] = lr;
    };
    fetch();                                      // before the keys: it is needed first
    bf16x8_t stay[2][KS];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int j = key0 + b * 32 + n < a.mass_len ? key0 + b * 32 + n : a.mass_len - 1;
#pragma unroll
        for (int kb = 0; kb < KS; ++kb)
            stay[b][kb] = *reinterpret_cast<const bf16x8_t*>(kh + (int64_t)j * a.tok_stride + kb * 16 + half * 8);
    }
    store(0);
    fetch();
    __syncthreads();
    bf16x8_t frag[kAhead];
#pragma unroll
    for (int f = 0; f < kAhead; ++f) frag[f] = *reinterpret_cast<const bf16x8_t*>(&sm.x[0][n][f * 16 + half * 8]);
    f32x16_t sa[2], sb[2];
    float sums[2][16];
#pragma unroll
    for (int i = 0; i < 16; ++i) { sb[0][i] = sb[1][i] = 0.f; sums[0][i] = sums[1][i] = 0.f; }
    float neg_b = -kPosBig;                       // of the rows in sb: none yet, their terms vanish
    int buf = 0;
    for (int t = 0; t < nt; ++t) {
        const int nbuf = buf + 1 == kRing ? 0 : buf + 1;
        store(nbuf);                              // as in pass 1
        fetch();
        const bf16_t* x0 = &sm.x[buf][n][half * 8];
        const bf16_t* x1 = &sm.x[buf][32 + n][half * 8];
        const float neg_a = -sm.lse[buf][n], neg_next = -sm.lse[buf][32 + n];   // padding rows: huge
        if (active) {
            const float neg[2] = {neg_b, neg_b};
            mass_step<D, true, 16>(sa, sb, stay, frag, x0, x1, c2, neg, sums);
        }
        lds_barrier();
        if (active) {
            const float neg[2] = {neg_a, neg_a};
            mass_step<D, true, 16>(sb, sa, stay, frag, x1, &sm.x[nbuf][n][half * 8], c2, neg, sums);
        }
        neg_b = neg_next;
        buf = nbuf;
    }
    if (!active) return;
    const float inv = 1.0f / (float)(a.W * G);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        float v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = sums[b][r] + __builtin_amdgcn_exp2f(fmaf(sb[b][r], c2, neg_b));
        const float tot = lanes_sum_scatter(v, n);
        const int r = n & 15, j = key0 + b * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
        if (n < 16 && j < a.mass_len) a.mass[(int64_t)hk * a.mass_len + j] = tot * inv;
    }
}

// Wavefronts per block of the two passes and key ranges of the first.  Pass 1: as many wavefronts
// as there are row groups (a block of 8 fills a compute unit's registers, of two of 2 its LDS holds
// three), then the number of ranges whose last round of blocks is fullest, a block's prologue and
// the merge of its partial counted as 8 tiles.  A range has at least 8 tiles: the partials fit the
// workspace, which has room for one per 512 keys.  Pass 2: the widest block that still leaves two
// per compute unit.
struct MassWidePlan { int nw1, S, nw2; };
inline MassWidePlan mass_wide_plan(int H_q, int H_k, int nrg, int mass_len) {
    MassWidePlan p;
    p.nw1 = nrg > 4 ? 8 : (nrg > 2 ? 4 : 2);
    const int64_t slots = 256 * (p.nw1 == 8 ? 1 : (p.nw1 == 4 ? 2 : 3));
    const int64_t units = (int64_t)H_q * ((nrg + p.nw1 - 1) / p.nw1);
    const int T = (mass_len + kStream - 1) / kStream;
    p.S = 1;
    double best = 0.0;
    for (int S = 1; S == 1 || (S <= 128 && T >= 8 * S); ++S) {
        const double cost = (double)((units * S + slots - 1) / slots) * ((double)((T + S - 1) / S) + 8.0);
        if (S == 1 || cost < 0.99 * best) { best = cost; p.S = S; }
    }
    p.nw2 = 8;
    while (p.nw2 > 2 && (int64_t)H_k * ((mass_len + p.nw2 * 64 - 1) / (p.nw2 * 64)) < 512) p.nw2 /= 2;
    return p;
}

template <int D, int NW>
int launch_stats_wide(const FcMassArgs& a, int nrg, int S, float* pm, float* pl, hipStream_t s) {
    const int64_t items = (int64_t)a.H_q * S * ((nrg + NW - 1) / NW);
    mass_stats_wide_kernel<D, NW><<<(unsigned)((items + 7) / 8 * 8), NW * 64, 0, s>>>(a, nrg, S, pm, pl);
    FC_LAUNCH_CHECK();
    return FC_OK;
}
template <int D, int NW>
int launch_cols_wide(const FcMassArgs& a, int nrg, const float* lse2, hipStream_t s) {
    mass_cols_wide_kernel<D, NW><<<dim3((a.mass_len + NW * 64 - 1) / (NW * 64), a.H_k), NW * 64, 0, s>>>(a, nrg, lse2);
    FC_LAUNCH_CHECK();
    return FC_OK;
}
template <int D>
int launch_wide(const FcMassArgs& a, hipStream_t s) {
    const int nrg = (a.W + kRowGroup - 1) / kRowGroup;
    const MassWidePlan p = mass_wide_plan(a.H_q, a.H_k, nrg, a.mass_len);
    float* pm = reinterpret_cast<float*>(a.ws);
    float* pl = pm + (size_t)a.H_q * nrg * kRowGroup * p.S;
    float* lse2 = pl + (size_t)a.H_q * nrg * kRowGroup * p.S;
    int st = p.nw1 == 8   ? launch_stats_wide<D, 8>(a, nrg, p.S, pm, pl, s)
             : p.nw1 == 4 ? launch_stats_wide<D, 4>(a, nrg, p.S, pm, pl, s)
                          : launch_stats_wide<D, 2>(a, nrg, p.S, pm, pl, s);
    if (st != FC_OK) return st;
    mass_lse_kernel<<<dim3(nrg, a.H_q), kNT, 0, s>>>(pm, pl, nrg, p.S, a.W, lse2);
    FC_LAUNCH_CHECK();
    return p.nw2 == 8   ? launch_cols_wide<D, 8>(a, nrg, lse2, s)
           : p.nw2 == 4 ? launch_cols_wide<D, 4>(a, nrg, lse2, s)
                        : launch_cols_wide<D, 2>(a, nrg, lse2, s);
}

// Tiles per block, 4 to 8: blocks of one launch take about the same time, so they run in rounds
// of as many blocks as the chip holds (two per compute unit); the span is chosen so that the
// last round is as full as possible (the MAGI-1-like layer: 3528 blocks of 4 tiles fill 6.9
// rounds of 512, where 1776 blocks of 8 tiles left the fourth round half empty).
inline int mass_tiles_per_block(int mass_len, int heads) {
    const int64_t slots = 512;
    int best = kTilesPerBlock;
    double best_eff = -1.0;
    for (int tpb = kTilesPerBlock; tpb >= kMinTilesPerBlock; --tpb) {
        const int64_t blocks = (int64_t)heads * ((mass_len + tpb * kTile - 1) / (tpb * kTile));
        const int64_t rounds = (blocks + slots - 1) / slots;
        const double eff = (double)blocks / (double)(rounds * slots);
        if (eff > best_eff + 0.02) { best_eff = eff; best = tpb; }   // longer spans unless clearly fuller
    }
    return best;
}

template <int D>
int launch_bf16(const FcMassArgs& a, hipStream_t s) {
    if (a.W > kRowGroup) return launch_wide<D>(a, s);
    const int tpb = mass_tiles_per_block(a.mass_len, a.H_q);
    const int np = (a.mass_len + tpb * kTile - 1) / (tpb * kTile);
    float* pm = reinterpret_cast<float*>(a.ws);
    float* pl = pm + (size_t)a.H_q * kRowGroup * np;
    float* lse2 = pl + (size_t)a.H_q * kRowGroup * np;
    mass_stats_bf16_kernel<D><<<dim3(np, a.H_q), kNT, 0, s>>>(a, np, tpb, pm, pl);
    FC_LAUNCH_CHECK();
    if (np > kFewPartials) {
        mass_lse_kernel<<<dim3(1, a.H_q), kNT, 0, s>>>(pm, pl, 1, np, a.W, lse2);
        FC_LAUNCH_CHECK();
    } else {
        lse2 = nullptr;
    }
    mass_cols_bf16_kernel<D><<<dim3(np, a.H_k), kNT, 0, s>>>(a, tpb, lse2, pm, pl, np);
    FC_LAUNCH_CHECK();
    return FC_OK;
}

// With few rows the matrix cores work on padding, and one thread per key is faster (heads x keys: head dimension
// 64 / 128; one thread per key against matrix cores, us): one row, 24 x 16384 45 against 63 / 74 against 113, 12 x 4096
// 13.5 : 18 / 17 : 26, 4 x 20000 24 : 25 / 33 : 43, 8 x 60000 75 : 65 / 119 : 120, 2 x 38000 33 : 27 / 41 : 45, 1 x 20000 18 : 17 / 21.5 :
// 24, 1 x 38000 25 : 21 / 34 : 29; four, 24 x 4096 20 : 24 / 31 : 42, 12 x 4096 16 : 18 / 22 : 26, 8 x 20000 34 : 33 / 50 : 55, 4 x
// 20000 28 : 25 / 38 : 42, 2 x 20000 22 : 20 / 30 : 27, 1 x 4096 16 : 15.5 / 21 : 21; eight, 24 x 4096 25 : 24 / 39.5 : 42, 12 x
// 12000 33 : 35 / 53.5 : 60, 12 x 4096 20.5 : 18 / 30 : 26, 8 x 20000 39 : 33 / 58 : 55.  Few long heads leave most threads'
// chains of loads uncovered.
inline bool f32_one_thread_per_key(int64_t rows, int H_k, int mass_len, int d) {
    if (rows <= 2) return H_k >= 12 || mass_len < (d == 128 && H_k > 1 ? 49152 : 24576);
    if (rows <= 4) return H_k >= 12 || (d == 128 && H_k >= 4 && mass_len < 49152);
    return rows <= kFewRows && H_k >= 12 && (int64_t)H_k * mass_len >= 24 * 4096;
}
template <int D>
int launch_f32_few(const FcMassArgs& a, hipStream_t s) {
    const int nkb = (a.mass_len + kNT - 1) / kNT, np = nkb * (kNT / FC_WAVE);
    float* pm = reinterpret_cast<float*>(a.ws);
    float* pl = pm + (size_t)a.H_q * kRowGroup * np;
    float* lse2 = pl + (size_t)a.H_q * kRowGroup * np;
    mass_stats_f32_few_kernel<D><<<dim3(nkb, a.H_k), kNT, 0, s>>>(a, np, pm, pl);
    FC_LAUNCH_CHECK();
    mass_lse_kernel<<<dim3(1, a.H_q), kNT, 0, s>>>(pm, pl, 1, np, a.W, lse2);
    FC_LAUNCH_CHECK();
    mass_cols_f32_few_kernel<D><<<dim3(nkb, a.H_k), kNT, 0, s>>>(a, lse2);
    FC_LAUNCH_CHECK();
    return FC_OK;
}

// Key ranges of pass 1: enough for two blocks per compute unit, a range at least one 32-key tile per
// wavefront, and no more partials than the workspace holds (per row group one per 512 keys; one
// group alone has room for one per 64).  Pass 2: as few wavefronts on the same keys as still give two
// blocks per compute unit, never more than there are row tiles.
template <int D>
int launch_f32(const FcMassArgs& a, hipStream_t s) {
    const int64_t rows = (int64_t)a.W * (a.H_q / a.H_k);
    if (f32_one_thread_per_key(rows, a.H_k, a.mass_len, D)) return launch_f32_few<D>(a, s);
    const int nrg = (a.W + kRowGroup - 1) / kRowGroup, rt = (int)((rows + 31) / 32);
    const int most = nrg == 1 ? a.mass_len / 256 : a.mass_len / 512;
    const int64_t units = (int64_t)a.H_k * rt;
    int S = (int)((511 + units) / units);
    S = S < most ? S : most;
    S = S < 1 ? 1 : S;
    float* pm = reinterpret_cast<float*>(a.ws);
    float* pl = pm + (size_t)a.H_q * nrg * kRowGroup * S;
    float* lse2 = pl + (size_t)a.H_q * nrg * kRowGroup * S;
    mass_stats_f32_kernel<D><<<dim3(S * rt, a.H_k), kF32Waves * 64, 0, s>>>(a, nrg, S, pm, pl);
    FC_LAUNCH_CHECK();
    if (S > kFewPartials || rt > kFewTiles) {
        mass_lse_kernel<<<dim3(nrg, a.H_q), kNT, 0, s>>>(pm, pl, nrg, S, a.W, lse2);
        FC_LAUNCH_CHECK();
    } else {
        lse2 = nullptr;
    }
    auto blocks = [&](int parts, int waves) { const int keys = waves / parts * 32; return (a.mass_len + keys - 1) / keys; };
    int parts = 1;
    while (parts < kF32Waves && 2 * parts <= rt && (int64_t)a.H_k * blocks(parts, kF32Waves) < 512) parts *= 2;
    if (parts <= kF32Waves / 2 && rt <= kFewTiles)
        mass_cols_f32_kernel<D, kF32Waves / 2><<<dim3(blocks(parts, kF32Waves / 2), a.H_k), kF32Waves * 32, 0, s>>>(a, nrg, parts, lse2, pm, pl, S);
    else
        mass_cols_f32_kernel<D, kF32Waves><<<dim3(blocks(parts, kF32Waves), a.H_k), kF32Waves * 64, 0, s>>>(a, nrg, parts, lse2, pm, pl, S);
    FC_LAUNCH_CHECK();
    return FC_OK;
}

}  // namespace

size_t fc_mass_workspace(int W, int H_q, int mass_len) {
    // one row group: a partial per 64 keys and row
    const size_t np = ((size_t)mass_len + 255) / 256 * 4;
    const size_t one = ((size_t)2 * H_q * kRowGroup * np + (size_t)H_q * kRowGroup) * sizeof(float);
    // more: all of them in one launch, a partial per 512 keys and row
    const size_t nrg = ((size_t)(W > 0 ? W : 1) + kRowGroup - 1) / kRowGroup;
    const size_t nps = ((size_t)mass_len + kMinTilesPerBlock * kTile - 1) / (kMinTilesPerBlock * kTile);
    const size_t many = ((size_t)2 * H_q * nrg * kRowGroup * nps + (size_t)H_q * nrg * kRowGroup) * sizeof(float);
    return fc_align_up(one > many ? one : many);
}

int fc_launch_mass(const FcMassArgs& a, hipStream_t s) {
    if (a.dtype == FC_BF16) {
        if (a.d == 128) return launch_bf16<128>(a, s);
        if (a.d == 64) return launch_bf16<64>(a, s);
    } else {
        if (a.d == 128) return launch_f32<128>(a, s);
        if (a.d == 64) return launch_f32<64>(a, s);
    }
    return FC_UNSUPPORTED;
}
