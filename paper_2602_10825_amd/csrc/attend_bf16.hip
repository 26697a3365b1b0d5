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
#include <utility>

#include "fc_common.hpp"

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int BQ = 256;      // query rows per workgroup
constexpr int BK = 64;       // keys per tile
constexpr int NXCD = 8;
constexpr float kNegBig = -1.0e30f;

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));

// Transposing LDS load: within each group of 16 lanes, lane s passes the address of 4
// consecutive bf16; lane i receives element (i % 4) of the data addressed by lanes
// i/4, i/4 + 4, i/4 + 8, i/4 + 12.
__device__ __forceinline__ s16x4_t lds_read_tr(const bf16_t* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (s16x4_t __attribute__((address_space(3)))*)(p));
}

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
    int n_tiles;
};

template <int D>
__global__ __launch_bounds__(NT) void attend_bf16_kernel(FcAttendArgs a, int tiles, int per) {
    __shared__ WideSmem<D> sm;
    constexpr int KS = D / 16;        // contraction steps of Q K^T
    constexpr int DVB = D / 32;       // 32-wide blocks of the value dimension
    constexpr int KROW = WideSmem<D>::KROW, VROW = WideSmem<D>::VROW;
    constexpr int VPR = D / 8;        // 16-byte vectors per K/V row
    constexpr int LD = BK * VPR / NT; // global loads per thread per tile (K, and again V)
    constexpr float kTooBig = 1.0995116e12f;  // 2^40: a row sum above this triggers a raise of m
    constexpr int NPV = 4 * DVB, NQK = 2 * KS, N = NPV + NQK;   // matrix products of a step: P V, Q K^T
    constexpr int PF = 4;             // fragments are read this many products ahead

    const int bid = blockIdx.x;
    const int xcd = bid % NXCD, slot = bid / NXCD;
    const int rank = slot / per;
    const int item = xcd * per + slot % per;
    if (item >= a.H_q * tiles) return;
    const int R = min(*a.n_rec, a.A);         // a count or an entry outside the valid range
    if (rank >= R) return;                    // (a caller's mistake) is skipped, never followed
    const int r = R - 1 - rank;               // heaviest (latest) chunk first
    const int c = a.rec_idx[r];
    if ((unsigned)c >= (unsigned)a.A) return;
    const int h = item / tiles, tile = item % tiles;
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

    // ---- visible key segments (clean region, then active chunks 0..c; adjacent ones merged)
    if (tid == 0) {
        int n = 0, sgi = -1, nt = 0;
        while (sgi <= c) {
            int start = (sgi < 0) ? 0 : a.active_off[sgi];
            int len = (sgi < 0) ? a.L_clean : a.L_c;
            ++sgi;
            while (sgi <= c && a.active_off[sgi] == start + len) { len += a.L_c; ++sgi; }
            if (len > 0) { sm.seg_start[n] = start; sm.seg_len[n] = len; ++n; nt += (len + BK - 1) / BK; }
        }
        sm.n_tiles = nt;
    }
    __syncthreads();
    const int nt = __builtin_amdgcn_readfirstlane(sm.n_tiles);
    int seg = 0, t0 = 0;
    int start = __builtin_amdgcn_readfirstlane(sm.seg_start[0]);
    int len = __builtin_amdgcn_readfirstlane(sm.seg_len[0]);
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

    // ---- epilogue: normalise, store O (bf16) and the row log-sum-exp
    {
        const float ltot = lsum + __shfl_xor(lsum, 32, FC_WAVE);
        const float inv = 1.0f / ltot;
        if (row_in_chunk < a.L_c) {
            const int64_t row = (int64_t)r * a.L_c + row_in_chunk;
            bf16_t* op = (bf16_t*)a.out + (row * a.H_q + h) * D;
#pragma unroll
            for (int dv = 0; dv < DVB; ++dv)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int e0 = dv * 32 + g * 8 + hh * 4;
                    uint2 pk;
                    pk.x = (uint32_t)f32_to_bf16(o[dv][4 * g] * inv) |
                           ((uint32_t)f32_to_bf16(o[dv][4 * g + 1] * inv) << 16);
                    pk.y = (uint32_t)f32_to_bf16(o[dv][4 * g + 2] * inv) |
                           ((uint32_t)f32_to_bf16(o[dv][4 * g + 3] * inv) << 16);
                    *reinterpret_cast<uint2*>(op + e0) = pk;
                }
            if (a.lse && hh == 0)
                a.lse[(int64_t)h * a.A * a.L_c + row] =
                    (m + __builtin_amdgcn_logf(ltot)) * 0.6931471805599453f;
        }
    }
}

}  // namespace

int fc_launch_attend_bf16(const FcAttendArgs& a, hipStream_t s) {
    const int tiles = (a.L_c + BQ - 1) / BQ;
    const int items = a.H_q * tiles;
    const int per = (items + NXCD - 1) / NXCD;
    const dim3 grid((unsigned)(NXCD * per * a.A));
    if (a.d == 128)
        attend_bf16_kernel<128><<<grid, NT, 0, s>>>(a, tiles, per);
    else if (a.d == 64)
        attend_bf16_kernel<64><<<grid, NT, 0, s>>>(a, tiles, per);
    else
        return FC_UNSUPPORTED;
    FC_LAUNCH_CHECK();
    return FC_OK;
}
