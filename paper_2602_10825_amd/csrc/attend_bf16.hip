// bf16 chunk-causal flash attention on the CDNA4 matrix cores (Sec. 3.3:
// softmax(q K^T d^-1/2) V, clean KV cache + active chunks 0..c visible to chunk c).
//
// One workgroup = 256 query rows of one head of one recompute chunk: 8 wavefronts of 32 rows,
// two per SIMD with 256 registers each.  Per 64-key tile:
//   S^T = K Q^T   v_mfma_f32_32x32x16_bf16, A = K fragment from LDS, B = Q fragment held
//                 in registers.  Computing the transpose puts one query per lane
//                 (column = lane % 32) and 16 keys of each 32-key block in that lane's
//                 accumulator registers, so the row max / row sum are in-lane reductions
//                 plus one exchange with lane ^ 32.
//   P   = exp2(S^T * scale*log2(e) - m)  fp32, cast to bf16: the accumulator layout already
//                 is the B-operand layout of the next product (contraction index = key, with
//                 a fixed permutation of the keys inside each 16-key group that V's LDS layout
//                 mirrors).  The row sums are taken over the ROUNDED weights
//                 (v_dot2c_f32_bf16 with a vector of ones), i.e. over exactly the weights V is
//                 multiplied with.
//   O^T += V^T P^T  A = V^T fragment read from the row-major V tile with the transposing
//                 LDS load ds_read_b64_tr_b16 (each 16-lane group turns 4 keys x 16 dv into
//                 16 lanes x 4 keys), two loads per 8-key fragment.
// The reference point m of the exponent is NOT the running row max: it is raised (and O, l
// rescaled) only when some row sum of a tile exceeds 2^40, which the sums reveal for free.
// exp2(S c2 - m) then stays far inside the fp32 / bf16 exponent range, the final O / l is
// unchanged, and the steady state carries no row-max reduction and no rescale at all.
// The first tile always takes the raise path once (m starts at -1e30).
//
// Order of the work.  Step j multiplies O += V P(j-1), then S(j+1) = K Q^T, 32 products in one
// chain of even spacing, with the weights of tile j -- 4 to 5 vector instructions a product --
// between them: matrix cores and vector ALU are both fed all the time, whatever the other
// wavefront of the SIMD does.  S needs one set of registers only: a key block's scores are all
// weighted before its accumulators start on the next tile.  Fragments are read from LDS four
// products ahead.  K sits in a ring of four tiles and V in two: tile j+2 of K and j of V are
// stored early in step j and become visible at the step's one barrier, which stands in the
// middle of the products, so that the first fragments of the next step are read before this one
// ends and no wavefront waits for LDS behind the barrier.  (A product's operands first, then
// its vector work, in two separate phases per tile: 24 x 128, 4 chunks of 9360 rows on 74880 clean
// keys 38.2 ms / 1183 TFLOP/s against 37.2 ms / 1216; constant operands, which the power limit
// lets run at full clock, 1495 against 1620; head dimension 64 590 against 575 us.)
// Work-groups are mapped so that the 32 compute units of one XCD work on the same head
// and chunk at the same time and share the K/V stream through that XCD's L2.
//
// Launches that do not fill the chip.  Where the units of 256 rows are fewer than the compute
// units, their keys are split over several blocks; where they are more, those of the last, partly
// filled round are (the plan and the merge of the partials: attend_split.hpp).  Where 256-row units
// would be mostly padding or still too few, a second body takes 32 rows per block and divides the
// keys over the block's wavefronts.  attend alone, us before / now: 8 heads on 2, 328 rows on 1984
// keys 53 / 18; 12 x 128, 600 rows on 5200 keys 126 / 40, 1500 rows on 51689 keys 1141 / 433, 256
// rows on 49201 keys 1076 / 106; 2 x 64, 278 rows on 60724 keys 982 / 36; 24 x 64, 2 chunks of 2040
// rows on 18360 keys (1.5 rounds of units) 550 / 451.
#include <utility>

#include "attend_split.hpp"

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int BQ = kWideRows;   // query rows per workgroup
constexpr int BK = 64;       // keys per tile

constexpr int NT = 64 * (BQ / 32);   // 8 wavefronts of 32 query rows, two per SIMD

// f(0), ..., f(N - 1) with the argument a compile-time constant: every choice made on it is made when
// the loop is written out
template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>()), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl<N>(f, std::make_integer_sequence<int, N>());
}

template <int D>
struct WideSmem {
    static constexpr int KROW = D + 8;        // padded K row (bf16): 16-byte fragment reads of 16
                                              // consecutive keys fall in distinct banks
    static constexpr int VROW = D + 32;       // padded V row: the 4 key rows of one transposing
                                              // load fall in disjoint bank quarters
    __attribute__((aligned(16))) bf16_t K[4][BK * KROW];
    __attribute__((aligned(16))) bf16_t V[2][BK * VROW];
    int seg_start[FC_MAX_ACTIVE + 2], seg_len[FC_MAX_ACTIVE + 2];
    int seg_first, off_first, n_tiles;
};

template <int D>
__device__ __forceinline__ void attend_wide(const FcAttendArgs& a, const FcAttendPlan& p, uint32_t valid,
                                            WideSmem<D>& sm, float* parts) {
    constexpr int KS = D / 16;        // contraction steps of Q K^T
    constexpr int DVB = D / 32;       // 32-wide blocks of the value dimension
    constexpr int KROW = WideSmem<D>::KROW, VROW = WideSmem<D>::VROW;
    constexpr int VPR = D / 8;        // 16-byte vectors per K/V row
    constexpr int LD = BK * VPR / NT; // global loads per thread per tile (K, and again V)
    constexpr float kTooBig = 1.0995116e12f;  // 2^40: a row sum above this triggers a raise of m
    constexpr int NPV = 4 * DVB, NQK = 2 * KS, N = NPV + NQK;   // matrix products of a step: P V, Q K^T
    constexpr int PF = 4;             // fragments are read this many products ahead

    const WideItem wi = wide_item<false>(a, p, valid, blockIdx.x);
    if (!wi.ok) return;
    const int r = wi.r, h = wi.h, tile = wi.tile;
    const int c = a.rec_idx[r];
    const int hk = h / (a.H_q / a.H_k);

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;   // wave: scalar
    const int l32 = lane & 31, hh = lane >> 5;

    // ---- Q fragments (B operand of S^T = K Q^T): lane holds Q[q = l32][16*step + 8*hh ..+8)
    bf16x8_t qf[KS];
    const int row_in_chunk = tile * BQ + wave * 32 + l32;
    {
        const int rc = row_in_chunk > a.L_c - 1 ? a.L_c - 1 : row_in_chunk;
        const bf16_t* qp = (const bf16_t*)a.q + (((int64_t)r * a.L_c + rc) * a.H_q + h) * D + 8 * hh;
#pragma unroll
        for (int st = 0; st < KS; ++st) qf[st] = *reinterpret_cast<const bf16x8_t*>(qp + 16 * st);
    }
    const float c2 = a.scale * 1.4426950408889634f;
    const bf16_t* kbase = (const bf16_t*)a.k_cache + (int64_t)hk * a.head_stride;
    const bf16_t* vbase = (const bf16_t*)a.v_cache + (int64_t)hk * a.head_stride;

    // ---- visible key segments (clean region, then active chunks 0..c; adjacent ones merged) and
    //      this block's range of their 64-key tiles
    if (tid == 0) {
        int n = 0, sgi = -1, nt = 0;
        while (sgi <= c) {
            int start = (sgi < 0) ? 0 : a.active_off[sgi];
            int len = (sgi < 0) ? a.L_clean : a.L_c;
            ++sgi;
            while (sgi <= c && a.active_off[sgi] == start + len) { len += a.L_c; ++sgi; }
            if (len > 0) { sm.seg_start[n] = start; sm.seg_len[n] = len; ++n; nt += (len + BK - 1) / BK; }
        }
        const int lo = (int)((int64_t)nt * wi.s / wi.S);
        int skip = lo, sg = 0;
        while (sg < n - 1 && skip >= (sm.seg_len[sg] + BK - 1) / BK) { skip -= (sm.seg_len[sg] + BK - 1) / BK; ++sg; }
        sm.seg_first = sg;
        sm.off_first = skip * BK < sm.seg_len[sg] ? skip * BK : 0;
        sm.n_tiles = (int)((int64_t)nt * (wi.s + 1) / wi.S) - lo;
    }
    __syncthreads();
    const int nt = __builtin_amdgcn_readfirstlane(sm.n_tiles);
    int seg = __builtin_amdgcn_readfirstlane(sm.seg_first);
    int start = __builtin_amdgcn_readfirstlane(sm.seg_start[seg]);
    int len = __builtin_amdgcn_readfirstlane(sm.seg_len[seg]);
    int t0 = __builtin_amdgcn_readfirstlane(sm.off_first);
    int to_step = nt - 1;             // tiles after the one (start, len, t0) point at

    u32x4_native kreg[LD], vreg[LD];
    const int ld_row = tid / VPR, ld_col = tid % VPR;
    constexpr int RPP = NT / VPR;     // rows per pass of the block's loads
    const uint32_t ts = (uint32_t)a.tok_stride;

    // tile (pos, valid) -> registers: wavefront-uniform base plus a 32-bit byte offset per lane; rows
    // past the end of a segment re-read its last one.  K runs two tiles ahead of V.
    int64_t pos_k, pos_v, pos_q0 = 0, pos_q1 = 0;      // element offsets of the tiles' first rows
    int nv_k, nv_v, nv_q0 = BK, nv_q1 = BK;
    auto step_tile = [&]() {          // K's next tile; V's is the one K had two calls before
        pos_v = pos_q1; nv_v = nv_q1;
        pos_q1 = pos_q0; nv_q1 = nv_q0;
        pos_k = (int64_t)(start + t0) * a.tok_stride;
        nv_k = len - t0 < BK ? len - t0 : BK;
        pos_q0 = pos_k; nv_q0 = nv_k;
        if (to_step > 0) {
            --to_step;
            t0 += BK;
            if (t0 >= len) {
                ++seg;
                start = __builtin_amdgcn_readfirstlane(sm.seg_start[seg]);
                len = __builtin_amdgcn_readfirstlane(sm.seg_len[seg]);
                t0 = 0;
            }
        }
    };
    uint32_t voff[LD];
#pragma unroll
    for (int i = 0; i < LD; ++i) voff[i] = ((uint32_t)(i * RPP + ld_row) * ts + (uint32_t)ld_col * 8u) * 2u;
    const uint32_t voff_row = ts * 2u;
    auto load_rows = [&](u32x4_native& dst, const bf16_t* base, int64_t pos, int nv, int i) {
        const char* b = reinterpret_cast<const char*>(base + pos);
        uint32_t off = voff[i];
        if (nv < BK) {
            const int over = i * RPP + ld_row - (nv - 1);
            off -= over > 0 ? (uint32_t)over * voff_row : 0u;
        }
        dst = *reinterpret_cast<const u32x4_native*>(b + off);
    };
    const int st_k = ld_row * KROW + ld_col * 8, st_v = ld_row * VROW + ld_col * 8;
    // per-lane offsets of the fragment reads.  Transposing V read: lane s of a 16-lane group addresses
    // key (s/4), dv 4*(s%4) of the group's 4-key x 16-dv patch; groups 0/1 cover dv 0-15 / 16-31,
    // lane half = key half
    const int l16 = lane & 15;
    const int k_frag = l32 * KROW + 8 * hh;
    const int v_frag = (hh * 4 + (l16 >> 2)) * VROW + ((lane >> 4) & 1) * 16 + (l16 & 3) * 4;

    f32x16_t o[DVB], s[2];
#pragma unroll
    for (int dv = 0; dv < DVB; ++dv)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[dv][i] = 0.f;
    float m = kNegBig, lsum = 0.f;
    u32x4_native P[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) P[t] = u32x4_native{0u, 0u, 0u, 0u};
    const bf16x2_t ones = {(__bf16)1.0f, (__bf16)1.0f};

    auto read_k = [&](const bf16_t* Kb, int f) {      // product f: key block f / KS, contraction step f % KS
        return *reinterpret_cast<const bf16x8_t*>(&Kb[(f / KS) * 32 * KROW + 16 * (f % KS)]);
    };
    auto read_v = [&](const bf16_t* Vb, int f) {      // product f: 16-key step f / DVB, value block f % DVB
        const bf16_t* vp = Vb + (f / DVB) * 16 * VROW + (f % DVB) * 32;
        const s16x4_t lo = lds_read_tr(vp), hi = lds_read_tr(vp + 8 * VROW);
        return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto mask_tail = [&](f32x16_t (&x)[2], int nv) {   // ragged end of a segment: keys past it
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (kb * 32 + (i >> 2) * 8 + hh * 4 + (i & 3) >= nv) x[kb][i] = kNegBig;
    };
    auto qk = [&](const bf16_t* Kb, f32x16_t (&x)[2]) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int i = 0; i < 16; ++i) x[kb][i] = 0.f;
#pragma unroll
            for (int st = 0; st < KS; ++st)
            {
                x[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_k(Kb, kb * KS + st), qf[st], x[kb], 0, 0, 0);
                if (st & 1) __builtin_amdgcn_sched_barrier(0);   // (few fragments in registers at a time)
            }
        }
    };
    float ps0, ps1;
    auto pack4 = [&](float x0, float x1, float x2, float x3, int q) {  // four weights: rounded to bf16, added to the row sum
        const bf16x2_t lo = {(__bf16)x0, (__bf16)x1}, hi = {(__bf16)x2, (__bf16)x3};
        uint32_t w0 = __builtin_bit_cast(uint32_t, lo), w1 = __builtin_bit_cast(uint32_t, hi);
        asm volatile("" : "+v"(w0), "+v"(w1));
        // the sums run over the ROUNDED weights, the ones V is multiplied with
        ps0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w0), ones, ps0, false);
        ps1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w1), ones, ps1, false);
        asm volatile("" : "+v"(ps0), "+v"(ps1));
        P[q >> 1][(q & 1) * 2] = w0;
        P[q >> 1][(q & 1) * 2 + 1] = w1;
    };

    if (nt > 0) {
        // ---- K(0), K(1) into the ring, K(2) and V(0) on their way, S(0); "V(-1)" finite (its P is zero)
        int nv_prev = BK, nv_cur, nv_next;   // valid keys of the tile before S's, of S's and of the next one
        {
            step_tile();
            nv_cur = nv_k;
#pragma unroll
            for (int i = 0; i < LD; ++i) load_rows(kreg[i], kbase, pos_k, nv_k, i);
            step_tile();
            nv_next = nv_k;
#pragma unroll
            for (int i = 0; i < LD; ++i) load_rows(vreg[i], kbase, pos_k, nv_k, i);
#pragma unroll
            for (int i = 0; i < LD; ++i) {
                *reinterpret_cast<u32x4_native*>(&sm.K[0][st_k + i * RPP * KROW]) = kreg[i];
                *reinterpret_cast<u32x4_native*>(&sm.K[1][st_k + i * RPP * KROW]) = vreg[i];
            }
            for (int i = tid; i < BK * VROW / 8; i += NT) reinterpret_cast<uint4*>(sm.V[1])[i] = make_uint4(0, 0, 0, 0);
            step_tile();
#pragma unroll
            for (int i = 0; i < LD; ++i) {
                load_rows(kreg[i], kbase, pos_k, nv_k, i);
                load_rows(vreg[i], vbase, pos_v, nv_v, i);
            }
        }
        __syncthreads();
        qk(&sm.K[0][k_frag], s);
        if (nv_cur < BK) mask_tail(s, nv_cur);
        bf16x8_t frag[PF];
#pragma unroll
        for (int f = 0; f < PF; ++f) frag[f] = read_v(&sm.V[1][v_frag], f);
        float psum = 0.f;
        int j = 0;
        // Inner loop = steady state.  It is left when a row sum shows that m must be raised; the outer
        // loop does that and re-enters.
        for (;;) {
        bool finished = false, raise;
        do {
            lsum += psum;
            if (j == nt) { finished = true; break; }
            const bf16_t* Kn = &sm.K[(j + 1) & 3][k_frag];
            const bf16_t* Vp = &sm.V[(j + 1) & 1][v_frag];
            const bf16_t* Vn = &sm.V[j & 1][v_frag];
            bf16_t* Kw = &sm.K[(j + 2) & 3][st_k];
            bf16_t* Vw = &sm.V[j & 1][st_v];
            const float mneg = -m;
            float wt[8];                               // weights on their way into P
            ps0 = ps1 = 0.f;
            constexpr int NEXP = NPV + KS - 1;         // products over which the exponentials are spread
            constexpr int BAR = NPV + KS / 2;
            // the chain before the other wavefront's masks and address steps (in turn on one card, medians: 24 x 64, 2 chunks
            // of 2040 rows on 18360 keys 452 -> 448 us; 12 x 128, 10200 rows on 61200 3195 -> 3182; 24 x 128, 4 x 9360 rows on
            // 74880 clean keys 37.59 -> 37.36 ms)
            __builtin_amdgcn_s_setprio(1);
            static_for<N>([&](auto F) __attribute__((always_inline)) {
                constexpr int f = F;
                // matrix cores: O += V P(j-1), then S(j+1) = K Q^T
                const bf16x8_t fr = frag[f % PF];
                if constexpr (f < NPV) {
                    o[f % DVB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr, __builtin_bit_cast(bf16x8_t, P[f / DVB]), o[f % DVB], 0, 0, 0);
                } else {
                    constexpr int g = f - NPV;
                    if constexpr (g % KS == 0) {
                        f32x16_t z;
#pragma unroll
                        for (int i = 0; i < 16; ++i) z[i] = 0.f;
                        s[g / KS] = z;
                    }
                    s[g / KS] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr, qf[g % KS], s[g / KS], 0, 0, 0);
                }
                // LDS: the fragment of product f + PF
                if constexpr (f + PF < NPV) frag[f % PF] = read_v(Vp, f + PF);
                else if constexpr (f + PF < N) frag[f % PF] = read_k(Kn, f + PF - NPV);
                else frag[f % PF] = read_v(Vn, f + PF - N);
                // vector ALU: weights of tile j
                constexpr int e0 = f < NEXP ? 32 * f / NEXP : 32, e1 = f < NEXP ? 32 * (f + 1) / NEXP : 32;
                static_for<e1 - e0>([&](auto E) __attribute__((always_inline)) {
                    constexpr int e = e0 + E;
                    float w = __builtin_amdgcn_exp2f(fmaf(s[e >> 4][e & 15], c2, mneg));
                    asm volatile("" : "+v"(w));       // computed here, next to the matrix products
                    wt[e & 7] = w;
                });
                static_for<8>([&](auto Q) __attribute__((always_inline)) {
                    // weights q are ready, and the products with the P register they replace are issued
                    constexpr int q = Q, fe = ((q + 1) * 4 * NEXP + 31) / 32 - 1, fp = (q / 2 + 1) * DVB;
                    if constexpr (f == (fe > fp ? fe : fp))
                        pack4(wt[(4 * q) & 7], wt[(4 * q + 1) & 7], wt[(4 * q + 2) & 7], wt[(4 * q + 3) & 7], q);
                });
                // staging: K(j+2), V(j) to LDS, then the loads of K(j+3), V(j+1)
                if constexpr (f >= 2 && f < 2 + LD)
                    *reinterpret_cast<u32x4_native*>(Kw + (f - 2) * RPP * KROW) = kreg[f - 2];
                if constexpr (f >= 2 + LD && f < 2 + 2 * LD)
                    *reinterpret_cast<u32x4_native*>(Vw + (f - 2 - LD) * RPP * VROW) = vreg[f - 2 - LD];
                if constexpr (f == 2 + 2 * LD) step_tile();
                if constexpr (f >= 2 + 2 * LD && f < 2 + 3 * LD) {
                    load_rows(kreg[f - 2 - 2 * LD], kbase, pos_k, nv_k, f - 2 - 2 * LD);
                    load_rows(vreg[f - 2 - 2 * LD], vbase, pos_v, nv_v, f - 2 - 2 * LD);
                }
                if constexpr (f == BAR) {
                    // K(j+2), V(j) are visible past this point: this wavefront's stores are done (seven
                    // or more later LDS accesses are behind them, LDS serves them in order), and every
                    // other one's too
                    __builtin_amdgcn_sched_barrier(0);
                    __builtin_amdgcn_s_waitcnt(0xC67F);      // lgkmcnt(6)
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            psum = ps0 + ps1;
            __builtin_amdgcn_s_setprio(0);
            if (nv_next < BK) mask_tail(s, nv_next);
            nv_prev = nv_cur;
            nv_cur = nv_next;
            nv_next = nv_q1;          // of tile j + 2
            ++j;
            raise = __any(psum > kTooBig);
        } while (!raise);
        if (finished) break;
        {
            // S of the tile just weighted again, its true row maximum, O and l to the new scale (the
            // products so far are in the old one), its weights anew
            f32x16_t x[2];
            qk(&sm.K[(j - 1) & 3][k_frag], x);
            if (nv_prev < BK) mask_tail(x, nv_prev);
            float v = fmaxf(x[0][0], x[1][0]);
#pragma unroll
            for (int i = 1; i < 16; ++i) v = fmaxf(v, fmaxf(x[0][i], x[1][i]));
            v = fmaxf(v, __shfl_xor(v, 32, FC_WAVE));
            const float mnew = fmaxf(m, v * c2);
            const float alpha = __builtin_amdgcn_exp2f(m - mnew);
            m = mnew;
            lsum *= alpha;
#pragma unroll
            for (int dv = 0; dv < DVB; ++dv) o[dv] *= alpha;
            ps0 = ps1 = 0.f;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int kb = q >> 2, i = (q & 3) * 4;
                pack4(__builtin_amdgcn_exp2f(fmaf(x[kb][i], c2, -m)), __builtin_amdgcn_exp2f(fmaf(x[kb][i + 1], c2, -m)),
                      __builtin_amdgcn_exp2f(fmaf(x[kb][i + 2], c2, -m)), __builtin_amdgcn_exp2f(fmaf(x[kb][i + 3], c2, -m)), q);
            }
            psum = ps0 + ps1;
        }
        }
        // ---- drain: O += V P of the last tile
        const bf16_t* Vl = &sm.V[(nt - 1) & 1][v_frag];
#pragma unroll
        for (int f = 0; f < NPV; ++f)
            o[f % DVB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f < PF ? frag[f] : read_v(Vl, f), __builtin_bit_cast(bf16x8_t, P[f / DVB]), o[f % DVB], 0, 0, 0);
    }

    // ---- epilogue: normalise, store O (bf16) and the row log-sum-exp; or leave the partial
    {
        const float ltot = lsum + __shfl_xor(lsum, 32, FC_WAVE);
        if (wi.S > 1) {
            const int64_t part = (wi.unit * (BQ / kUnitRows) + wave) * wi.S + wi.s;   // 32 rows each
            float* po = parts + (part * kUnitRows + l32) * D;
#pragma unroll
            for (int dv = 0; dv < DVB; ++dv)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    store_out(po + dv * 32 + g * 8 + hh * 4, o[dv][4 * g], o[dv][4 * g + 1], o[dv][4 * g + 2],
                              o[dv][4 * g + 3]);
            if (hh == 0) {
                float* ml = parts + (int64_t)p.parts * kUnitRows * D + part * 2 * kUnitRows;
                ml[l32] = m;
                ml[kUnitRows + l32] = ltot;
            }
            return;
        }
        const float inv = 1.0f / ltot;
        if (row_in_chunk < a.L_c) {
            const int64_t row = (int64_t)r * a.L_c + row_in_chunk;
            bf16_t* op = (bf16_t*)a.out + (row * a.H_q + h) * D;
#pragma unroll
            for (int dv = 0; dv < DVB; ++dv)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int e0 = dv * 32 + g * 8 + hh * 4;
                    store_out(op + e0, o[dv][4 * g] * inv, o[dv][4 * g + 1] * inv, o[dv][4 * g + 2] * inv,
                              o[dv][4 * g + 3] * inv);
                }
            if (a.lse && hh == 0)
                a.lse[(int64_t)h * a.A * a.L_c + row] =
                    (m + __builtin_amdgcn_logf(ltot)) * 0.6931471805599453f;
        }
    }
}

// ---- few query rows ---------------------------------------------------------------------
// 32 query rows per block; its 8 wavefronts take every 8th 32-key tile of the range and never meet
// before the end, where their partials are merged through LDS.  Each stages its own tile in LDS
// (coalesced loads one tile ahead; K read straight into registers in the operand's layout, 32
// bytes of 32 rows per load, took twice as long) and follows the row maximum at a distance of
// 2^8.  A tile costs a wavefront about 1.9 us, most of it the 16 KB that nothing shares with the
// other wavefronts; that is why launches with enough rows take the 256-row body, where 8
// wavefronts share every tile.
template <int D>
struct NarrowSmem {
    static constexpr int KROW = D + 8, VROW = D + 32, OROW = D + 4;   // padded rows, as in WideSmem
    __attribute__((aligned(16))) union {
        struct { bf16_t k[kSplitWaves][32 * KROW], v[kSplitWaves][32 * VROW]; } t;   // one tile per wavefront
        float o[kSplitWaves * kUnitRows * OROW];        // partial O at the end
    };
    float m_s[kSplitWaves * kUnitRows], l_s[kSplitWaves * kUnitRows];
    Segments sg;
};

template <int D>
__device__ __forceinline__ void attend_narrow(const FcAttendArgs& a, const FcAttendPlan& p, uint32_t valid,
                                              NarrowSmem<D>& sm, float* parts) {
    constexpr int KS = D / 16;           // contraction steps of Q K^T
    constexpr int DVB = D / 32;          // 32-wide blocks of the value dimension
    constexpr int KROW = NarrowSmem<D>::KROW, VROW = NarrowSmem<D>::VROW, OROW = NarrowSmem<D>::OROW;
    constexpr int VPR = D / 8;           // 16-byte vectors per row
    constexpr int LD = 32 * VPR / FC_WAVE;
    constexpr float kSlack = 8.0f;       // the exponents' reference follows the row maximum at this distance (log2)
    Segments& sg = sm.sg;
    float *m_s = sm.m_s, *l_s = sm.l_s;

    const SplitItem it = split_item(a, p, valid, blockIdx.x);
    if (!it.ok) return;
    const int hk = it.h / (a.H_q / a.H_k);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l32 = lane & 31, hh = lane >> 5;
    const float c2 = a.scale * 1.4426950408889634f;
    if (tid == 0) list_segments(a, it.c, sg);

    // B operand of S^T = K Q^T: lane holds Q[q = l32][16 step + 8 hh .. + 8)
    bf16x8_t qf[KS];
    {
        int rc = it.tile * kUnitRows + l32;
        if (rc > a.L_c - 1) rc = a.L_c - 1;
        const bf16_t* qp = (const bf16_t*)a.q + (((int64_t)it.r * a.L_c + rc) * a.H_q + it.h) * D + 8 * hh;
#pragma unroll
        for (int st = 0; st < KS; ++st) qf[st] = *reinterpret_cast<const bf16x8_t*>(qp + 16 * st);
    }
    __syncthreads();
    const bf16_t* kbase = (const bf16_t*)a.k_cache + (int64_t)hk * a.head_stride;
    const bf16_t* vbase = (const bf16_t*)a.v_cache + (int64_t)hk * a.head_stride;
    const uint32_t ts = (uint32_t)a.tok_stride;
    const int nt = __builtin_amdgcn_readfirstlane(sg.tile0[sg.n]);
    const int t_end = (int)((int64_t)nt * (it.s + 1) / it.S);
    int t = (int)((int64_t)nt * it.s / it.S) + wave;

    f32x16_t o[DVB];
#pragma unroll
    for (int b = 0; b < DVB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[b][i] = 0.f;
    float m = kNegBig, l = 0.f;

    u32x4_native kr[LD], vr[LD];
    int seg = 0, nvalid = 0;
    const int ld_row = lane / VPR, ld_col = lane % VPR;
    // tile tt -> registers, by rows; a row past the end of its segment re-reads the last one
    auto fetch = [&](int tt) {
        while (tt >= __builtin_amdgcn_readfirstlane(sg.tile0[seg + 1])) ++seg;
        const int off = (tt - __builtin_amdgcn_readfirstlane(sg.tile0[seg])) * 32;
        const int left = __builtin_amdgcn_readfirstlane(sg.len[seg]) - off;
        const int64_t pos = (int64_t)(__builtin_amdgcn_readfirstlane(sg.start[seg]) + off) * a.tok_stride;
        nvalid = left < 32 ? left : 32;
        const char* kt = reinterpret_cast<const char*>(kbase + pos);
        const char* vt = reinterpret_cast<const char*>(vbase + pos);
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            int row = i * (FC_WAVE / VPR) + ld_row;
            row = row < nvalid ? row : nvalid - 1;
            const uint32_t at = ((uint32_t)row * ts + 8u * (uint32_t)ld_col) * 2u;
            kr[i] = *reinterpret_cast<const u32x4_native*>(kt + at);
            vr[i] = *reinterpret_cast<const u32x4_native*>(vt + at);
        }
    };
    const int l16 = lane & 15;
    bf16_t *kw = sm.t.k[wave], *vw = sm.t.v[wave];
    const bf16_t* v_frag = vw + (hh * 4 + (l16 >> 2)) * VROW + ((lane >> 4) & 1) * 16 + (l16 & 3) * 4;
    if (t < t_end) fetch(t);
    while (t < t_end) {
        // the wavefront's own tile: its LDS accesses are served in order, no barrier is needed
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const int row = i * (FC_WAVE / VPR) + ld_row;
            *reinterpret_cast<u32x4_native*>(&kw[row * KROW + ld_col * 8]) = kr[i];
            *reinterpret_cast<u32x4_native*>(&vw[row * VROW + ld_col * 8]) = vr[i];
        }
        const int nv = nvalid;
        t += kSplitWaves;
        if (t < t_end) fetch(t);                        // the next tile, behind all of this one
        f32x16_t s;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            const bf16x8_t kf = *reinterpret_cast<const bf16x8_t*>(&kw[l32 * KROW + 16 * st + 8 * hh]);
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[st], s, 0, 0, 0);
        }
        if (nv < 32) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if ((i >> 2) * 8 + hh * 4 + (i & 3) >= nv) s[i] = kNegBig;
        }
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, FC_WAVE)) * c2;
        if (__any(mx > m + kSlack)) {
            const float mn = fmaxf(m, mx);
            const float alpha = __builtin_amdgcn_exp2f(m - mn);
            m = mn;
            l *= alpha;
#pragma unroll
            for (int b = 0; b < DVB; ++b) o[b] *= alpha;
        }
        const float mneg = -m;
        const bf16x2_t ones = {(__bf16)1.0f, (__bf16)1.0f};
        bf16x8_t pf[2];
        float l0 = 0.f, l1 = 0.f;
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(s[i], c2, mneg));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(s[i + 1], c2, mneg));
            const float p2 = __builtin_amdgcn_exp2f(fmaf(s[i + 2], c2, mneg));
            const float p3 = __builtin_amdgcn_exp2f(fmaf(s[i + 3], c2, mneg));
            const bf16x2_t lo = {(__bf16)p0, (__bf16)p1}, hi = {(__bf16)p2, (__bf16)p3};
            // the sums run over the rounded weights, the ones V is multiplied with
            l0 = __builtin_amdgcn_fdot2_f32_bf16(lo, ones, l0, false);
            l1 = __builtin_amdgcn_fdot2_f32_bf16(hi, ones, l1, false);
            pf[i >> 3][i & 7] = lo[0];
            pf[i >> 3][(i & 7) + 1] = lo[1];
            pf[i >> 3][(i & 7) + 2] = hi[0];
            pf[i >> 3][(i & 7) + 3] = hi[1];
        }
        l += l0 + l1;
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int b = 0; b < DVB; ++b) {
                const bf16_t* vp = v_frag + tt * 16 * VROW + b * 32;
                const s16x4_t lo = lds_read_tr(vp), hi = lds_read_tr(vp + 8 * VROW);
                const bf16x8_t vf = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[tt], o[b], 0, 0, 0);
            }
    }
    l += __shfl_xor(l, 32, FC_WAVE);
    __syncthreads();                                    // every wavefront is done with its V tile
    if (hh == 0) { m_s[wave * kUnitRows + l32] = m; l_s[wave * kUnitRows + l32] = l; }
#pragma unroll
    for (int b = 0; b < DVB; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<f32x4_t*>(&sm.o[(wave * kUnitRows + l32) * OROW + b * 32 + g * 8 + hh * 4]) =
                f32x4_t{o[b][4 * g], o[b][4 * g + 1], o[b][4 * g + 2], o[b][4 * g + 3]};
    __syncthreads();
    finish_unit<bf16_t, D, OROW>(a, p, it, sm.o, m_s, l_s, parts);
}

// WIDE and NARROW say which of the two bodies some recompute count of this launch asks for.
template <int D, bool WIDE, bool NARROW>
__global__ __launch_bounds__(NT) void attend_bf16_kernel(FcAttendArgs a, FcAttendPlan p, float* parts) {
    static_assert(NT == kSplitThreads, "both bodies run on the same block");
    const uint32_t valid = valid_blocks(a);
    const int R = __popc(valid);
    if (R == 0) return;
    union Smem {
        WideSmem<WIDE ? D : 64> w;
        NarrowSmem<NARROW ? D : 64> n;
    };
    __shared__ __attribute__((aligned(16))) char raw[WIDE && NARROW ? sizeof(Smem) : WIDE ? sizeof(WideSmem<D>) : sizeof(NarrowSmem<D>)];
    if (WIDE && (!NARROW || !p.narrow[R - 1]))
        attend_wide<D>(a, p, valid, *reinterpret_cast<WideSmem<D>*>(raw), parts);
    else if (NARROW)
        attend_narrow<D>(a, p, valid, *reinterpret_cast<NarrowSmem<D>*>(raw), parts);
}

template <int D>
int launch_bf16(const FcAttendArgs& a, hipStream_t s) {
    FcAttendPlan p = fc_attend_plan_bf16(a.A, a.L_c, a.L_clean, a.H_q, D, true);
    if (!fc_room_for_partials(a.ws, a.ws_bytes, p.parts, D))
        p = fc_attend_plan_bf16(a.A, a.L_c, a.L_clean, a.H_q, D, false);
    bool wide = false, narrow = false;
    for (int R = 0; R < a.A; ++R) (p.narrow[R] ? narrow : wide) = true;
    if (!narrow)
        attend_bf16_kernel<D, true, false><<<p.grid, NT, 0, s>>>(a, p, (float*)a.ws);
    else if (!wide)
        attend_bf16_kernel<D, false, true><<<p.grid, NT, 0, s>>>(a, p, (float*)a.ws);
    else
        attend_bf16_kernel<D, true, true><<<p.grid, NT, 0, s>>>(a, p, (float*)a.ws);
    FC_LAUNCH_CHECK();
    if (p.merge_grid > 0) {
        attend_merge_kernel<bf16_t, D><<<p.merge_grid, 256, 0, s>>>(a, p, (const float*)a.ws);
        FC_LAUNCH_CHECK();
    }
    return FC_OK;
}

}  // namespace

int fc_launch_attend_bf16(const FcAttendArgs& a, hipStream_t s) {
    if (a.d == 128) return launch_bf16<128>(a, s);
    if (a.d == 64) return launch_bf16<64>(a, s);
    return FC_UNSUPPORTED;
}
