// K/V scatter of the recompute chunks into their cache slots, and the fp32 chunk-causal
// attention kernel (Sec. 3.3; softmax(q K^T d^-1/2) V with a chunk-granular causal mask).
//
#include "attend_split.hpp"
#include "f32_split.hpp"

namespace {

// ------------------------------------------------------------------ K/V scatter
// new [rows, H_k, d] token-major  ->  cache[h][slot + t][0..d)
__global__ __launch_bounds__(256) void scatter_kv_kernel(
    const uint4* __restrict__ k_new, const uint4* __restrict__ v_new, uint4* __restrict__ k_cache,
    uint4* __restrict__ v_cache, int64_t head_stride_v, int64_t tok_stride_v, int H_k, int vpr,
    int L_c, FcScatterArgs args) {
    const int r = blockIdx.y;
    if (r >= *args.n_rec) return;
    const int c = args.rec_idx[r];
    if ((unsigned)c >= (unsigned)args.A) return;   // not a chunk: skipped, never followed
    const int64_t slot = args.active_off[c];
    const int64_t per_chunk = (int64_t)L_c * H_k * vpr;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < per_chunk; i += stride) {
        const int v = (int)(i % vpr);
        const int h = (int)((i / vpr) % H_k);
        const int64_t t = i / ((int64_t)vpr * H_k);
        const int64_t dst = h * head_stride_v + (slot + t) * tok_stride_v + v;
        k_cache[dst] = k_new[(int64_t)r * per_chunk + i];
        v_cache[dst] = v_new[(int64_t)r * per_chunk + i];
    }
}

// ------------------------------------------------------------------ fp32 attention
// On the f16 matrix cores, every operand in two f16 parts (f32_split.hpp).  A block is 32 query rows; its 8
// wavefronts take every 8th 32-key tile and never meet before the end, where their partials are merged
// through LDS; a launch of few rows still occupies eight wavefronts per 32 rows.  Bound by the vector
// ALU: about 600 instructions a tile and wavefront, two thirds of them splitting K and V, against 48
// products of 32 cycles.
//   S^T = K Q^T  puts one query per lane, so maximum and sum are in-lane but for one exchange,
//   and the accumulators of S^T already are the B operand of  O^T += V^T P^T.
//   Q is split once, a scale per row; K a scale per key, read as rows and turned to the operand's layout
//   in LDS (read straight into that layout, 32 bytes of 32 rows a load: 357 -> 379 us below); V one scale
//   that follows the largest finite entry the wavefront has seen; the weights none, their range is the choice
//   of the reference.
// 12 heads x 128, 2 chunks of 1021 rows on 4083 clean keys: 650 us on the fp32 matrix cores (69 % busy, no
// vector instruction beside them), now 357; 24 x 128, 460 rows on 4890 keys 237 / 130; 12 x 64, 2 x 174 rows on
// 18580 keys 246 / 163; 4 query heads on 1 x 64, 2 x 128 rows on 512: 19 / 14.  Relative error against float64
// 3.4e-7 .. 6.3e-7 before, 2.9e-7 .. 4.2e-7 now; at twice the logits 8e-7 .. 16e-7 and 5e-7 .. 7e-7.
// The two chains of products run at raised priority (the other wavefront of the SIMD fills their gaps): 8 heads on 2 x 128,
// 2 x 200 rows on 3000 keys 43.0 -> 41.4, 12 x 64, 300 rows on 3000 27.8 -> 27.0.  (The body with shared tiles below: 24 x 64
// 133.6 -> 131.0, but 24 x 128, 460 rows on 3350 keys 107.7 -> 109.4: not taken.)
template <int N> struct VecF;
template <> struct VecF<4> { typedef float type __attribute__((ext_vector_type(4))); };
template <> struct VecF<2> { typedef float type __attribute__((ext_vector_type(2))); };

template <int D>
__global__ __launch_bounds__(kSplitThreads) void attend_f32_kernel(FcAttendArgs a, FcAttendPlan p, float* parts) {
    constexpr int KS = D / 16;           // contraction steps of Q K^T
    constexpr int NB = D / 32;           // 32-wide blocks of the value dimension
    constexpr int ROW = D + 4;           // padded rows of K tiles and of the partial O (floats),
    constexpr int QROW = D + 8;          // and of Q's parts (f16): 16-byte reads of 32 rows spread over the banks
    // The exponents' reference follows the row maximum at a distance: weights are at most 2^15, and those
    // above 2^-13 of the largest so far (2^-2) are split without loss.
    constexpr float kTop = 15.0f, kStart = 12.0f;
    typedef typename VecF<NB>::type vrow_t;
    __shared__ __attribute__((aligned(16))) float buf[kSplitWaves * kUnitRows * ROW];   // a K tile per wavefront, partial O at the end
    __shared__ __attribute__((aligned(16))) bf16_t q_s[2 * kUnitRows * QROW];            // Q's two parts
    __shared__ float m_s[kSplitWaves * kUnitRows], l_s[kSplitWaves * kUnitRows];
    __shared__ __attribute__((aligned(16))) float k_scale[kSplitWaves][32];
    __shared__ float q_scale[kUnitRows];
    __shared__ Segments sg;

    const SplitItem it = split_item(a, p, valid_blocks(a), blockIdx.x);
    if (!it.ok) return;
    const int hk = it.h / (a.H_q / a.H_k);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l32 = lane & 31, hh = lane >> 5;
    const float c2 = a.scale * 1.4426950408889634f;   // fold log2(e): exp(x) = exp2(x*log2 e)

    if (tid == 0) list_segments(a, it.c, sg);
    if (tid < kUnitRows * (D / 8)) {
        const int row = tid / (D / 8), e = tid % (D / 8);
        int rc = it.tile * kUnitRows + row;
        if (rc > a.L_c - 1) rc = a.L_c - 1;
        const float* qp = (const float*)a.q + (((int64_t)it.r * a.L_c + rc) * a.H_q + it.h) * D + 8 * e;
        const f32x4_t v0 = *reinterpret_cast<const f32x4_t*>(qp) * c2, v1 = *reinterpret_cast<const f32x4_t*>(qp + 4) * c2;
        float most = max_abs4(max_abs4(0.f, v0), v1);
#pragma unroll
        for (int x = 1; x < D / 8; x <<= 1) most = fmaxf(most, __shfl_xor(most, x, FC_WAVE));
        float inv;
        const float sc = split_scale(most, inv);
        if (e == 0) q_scale[row] = inv;
        Split8 s;
        split_pair(s, 0, v0[0], v0[1], sc); split_pair(s, 1, v0[2], v0[3], sc);
        split_pair(s, 2, v1[0], v1[1], sc); split_pair(s, 3, v1[2], v1[3], sc);
        *reinterpret_cast<u32x4_native*>(q_s + row * QROW + 8 * e) = s.h;
        *reinterpret_cast<u32x4_native*>(q_s + (kUnitRows + row) * QROW + 8 * e) = s.l;
    }
    __syncthreads();

    const float* kbase = (const float*)a.k_cache + (int64_t)hk * a.head_stride;
    const float* vbase = (const float*)a.v_cache + (int64_t)hk * a.head_stride;
    const int nt = __builtin_amdgcn_readfirstlane(sg.tile0[sg.n]);
    const int t_end = (int)((int64_t)nt * (it.s + 1) / it.S);
    int t = (int)((int64_t)nt * it.s / it.S) + wave;

    f32x16_t o[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[b][i] = 0.f;
    float m = kNegBig, l = 0.f;
    const float qs = q_scale[l32];
    float v_most = 0.f, v_sc = 1.f, v_inv = 1.f;      // V's scale, the wavefront's: it fits entries of up to v_most
    const uint32_t ts = (uint32_t)a.tok_stride;

    f32x4_t kf[2 * KS];
    vrow_t vf[16];
    int seg = 0, pos = 0, nvalid = 0;
    auto locate = [&](int tt) {
        while (tt >= __builtin_amdgcn_readfirstlane(sg.tile0[seg + 1])) ++seg;
        const int off = (tt - __builtin_amdgcn_readfirstlane(sg.tile0[seg])) * 32;
        const int left = __builtin_amdgcn_readfirstlane(sg.len[seg]) - off;
        pos = __builtin_amdgcn_readfirstlane(sg.start[seg]) + off;
        nvalid = left < 32 ? left : 32;
    };
    // Whole rows at a time; A operand of S^T = K Q^T: lane (hh, l32) holds K[l32][16 st + 8 hh .. + 8)
    constexpr int LPR = D / 4, RPL = FC_WAVE / LPR;     // lanes per row, rows per load
    const int ld_row = lane / LPR, ld_col = 4 * (lane % LPR);
    const uint32_t k_off = ((uint32_t)ld_row * ts + (uint32_t)ld_col) * 4u, v_off = ((uint32_t)hh * 4u * ts + (uint32_t)(NB * l32)) * 4u;
    float* const k_tile = buf + wave * 32 * ROW;
    auto load_k = [&]() {
        const char* kt = reinterpret_cast<const char*>(kbase + (int64_t)pos * a.tok_stride);   // scalar
        const uint32_t last = (uint32_t)(nvalid - 1) * ts * 4u + (uint32_t)ld_col * 4u;   // rows past the end: the last one again
        uint32_t off = k_off;
        asm volatile("" : "+v"(off));                  // (computed here each time: sixteen offsets kept in registers spill)
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j) {
            kf[j] = *reinterpret_cast<const f32x4_t*>(kt + (off < last ? off : last));
            off += (uint32_t)RPL * ts * 4u;
        }
    };
    auto turn_k = [&]() {                // the wavefront's own tile: LDS serves its accesses in order, no barrier is needed
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j) *reinterpret_cast<f32x4_t*>(k_tile + (j * RPL + ld_row) * ROW + ld_col) = kf[j];
        asm volatile("" ::: "memory");
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j) kf[j] = *reinterpret_cast<const f32x4_t*>(k_tile + l32 * ROW + 16 * (j >> 1) + 8 * hh + 4 * (j & 1));
    };
    // A operand of O^T += V^T P^T: row l32 of block b is value column NB * l32 + b, so one wide load
    // per key serves all blocks; step tt contracts over the 16 keys of accumulators 8 tt .. 8 tt + 7
    // of both lane halves
    auto load_v = [&](int tt, int vpos, int nv) {
        const char* vt = reinterpret_cast<const char*>(vbase + (int64_t)vpos * a.tok_stride);   // scalar
        const uint32_t last = ((uint32_t)(nv - 1) * ts + (uint32_t)(NB * l32)) * 4u;
        uint32_t off0 = v_off + (uint32_t)tt * 16u * ts * 4u;
        asm volatile("" : "+v"(off0));
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int i = 8 * tt + e;
            const uint32_t off = off0 + (uint32_t)((e >> 2) * 8 + (e & 3)) * ts * 4u;
            vf[i] = *reinterpret_cast<const vrow_t*>(vt + (off < last ? off : last));
        }
    };
    const bf16_t* q_frag = q_s + l32 * QROW + 8 * hh;
    auto read_q = [&](int st) {
        return Split8{*reinterpret_cast<const u32x4_native*>(q_frag + 16 * st),
                      *reinterpret_cast<const u32x4_native*>(q_frag + kUnitRows * QROW + 16 * st)};
    };

    if (t < t_end) { locate(t); load_k(); }
    while (t < t_end) {
        const int nv = nvalid, vpos = pos;
        turn_k();
        // each key's own scale; the accumulators need those of 16 other keys
        float most = 0.f, k_sc;
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j) most = max_abs4(most, kf[j]);
        most = fmaxf(most, __shfl_xor(most, 32, FC_WAVE));
        {
            float inv;
            k_sc = split_scale(most, inv);
            k_scale[wave][l32] = inv;
        }
        auto split_k = [&](Split8& x, int st, int p) __attribute__((always_inline)) {
            split_pair(x, p, kf[2 * st + (p >> 1)][2 * (p & 1)], kf[2 * st + (p >> 1)][2 * (p & 1) + 1], k_sc);
        };
        f32x16_t s, s1;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = s1[i] = 0.f;
        Split8 cur, nxt, qc = read_q(0), qn;
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int p = 0; p < 4; ++p) split_k(cur, 0, p);
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            if (st + 1 < KS) qn = read_q(st + 1);
            split_mfma(cur.l, qc.h, s1);
            if (st + 1 < KS) { split_k(nxt, st + 1, 0); split_k(nxt, st + 1, 1); }
            __builtin_amdgcn_sched_barrier(0);
            split_mfma(cur.h, qc.h, s);
            if (st + 1 < KS) { split_k(nxt, st + 1, 2); split_k(nxt, st + 1, 3); }
            __builtin_amdgcn_sched_barrier(0);
            split_mfma(cur.h, qc.l, s1);
            if (st == KS / 2 - 1) load_v(0, vpos, nv);     // K's first half is used up: its registers are free
            __builtin_amdgcn_sched_barrier(0);
            cur = nxt;
            qc = qn;
        }
        __builtin_amdgcn_s_setprio(0);
        load_v(1, vpos, nv);
        t += kSplitWaves;
        if (t < t_end) { locate(t); load_k(); }        // the next tile's keys, behind the softmax and P V
        __builtin_amdgcn_sched_barrier(0);
        s += s1;
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
            const f32x4_t ks = *reinterpret_cast<const f32x4_t*>(&k_scale[wave][2 * i + 4 * hh]);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[i + e] = s[i + e] * ks[e] * qs;
        }
        if (nv < 32) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if ((i >> 2) * 8 + hh * 4 + (i & 3) >= nv) s[i] = kNegBig;
        }
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
        if (__any(mx > m + kTop)) {
            const float mn = fmaxf(m, fmaxf(mx, __shfl_xor(mx, 32, FC_WAVE)) - kStart);
            const float alpha = __builtin_amdgcn_exp2f(m - mn);
            m = mn;
            l *= alpha;
#pragma unroll
            for (int b = 0; b < NB; ++b) o[b] *= alpha;
        }
        float p0 = 0.f, p1 = 0.f;
        Split8 ps[2];
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            const float x0 = __builtin_amdgcn_exp2f(s[i] - m), x1 = __builtin_amdgcn_exp2f(s[i + 1] - m);
            p0 += x0;
            p1 += x1;
            split_pair(ps[i >> 3], (i & 7) >> 1, x0, x1, 1.0f);
        }
        l += p0 + p1;
        // V's scale leaves a factor of four before it has to follow a larger entry
        float vm = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int b = 0; b < NB; ++b) vm = fmaxf(vm, fabsf(vf[i][b]));
        if (__any(vm > v_most)) {
            vm = v_most;                                  // an infinity spoils its own column only
#pragma unroll
            for (int i = 0; i < 16; ++i)
#pragma unroll
                for (int b = 0; b < NB; ++b) vm = max_finite(vm, vf[i][b]);
        }
        if (__any(vm > v_most)) {
            float inv;
            const float sc = split_scale(wave_max_all(vm), inv, 2);
            const float down = sc * v_inv;                // old scale to new; O is zero while there is no old one
            v_sc = sc; v_inv = inv; v_most = 32768.0f * inv;
#pragma unroll
            for (int b = 0; b < NB; ++b) o[b] *= down;
        }
        auto split_v = [&](Split8& x, int g, int p) __attribute__((always_inline)) {
            split_pair(x, p, vf[8 * (g / NB) + 2 * p][g % NB], vf[8 * (g / NB) + 2 * p + 1][g % NB], v_sc);
        };
        // two blocks of O at a time
        Split8 va, vb, na, nb;
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int p = 0; p < 4; ++p) { split_v(va, 0, p); split_v(vb, 1, p); }
#pragma unroll
        for (int g = 0; g < 2 * NB; g += 2) {
            f32x16_t &oa = o[g % NB], &ob = o[g % NB + 1];
            const Split8& pc = ps[g / NB];
            const bool more = g + 2 < 2 * NB;
            split_mfma(va.l, pc.h, oa); if (more) split_v(na, g + 2, 0); if (more) split_v(na, g + 2, 1); __builtin_amdgcn_sched_barrier(0);
            split_mfma(vb.l, pc.h, ob); if (more) split_v(na, g + 2, 2); if (more) split_v(na, g + 2, 3); __builtin_amdgcn_sched_barrier(0);
            split_mfma(va.h, pc.l, oa); if (more) split_v(nb, g + 3, 0); __builtin_amdgcn_sched_barrier(0);
            split_mfma(vb.h, pc.l, ob); if (more) split_v(nb, g + 3, 1); __builtin_amdgcn_sched_barrier(0);
            split_mfma(va.h, pc.h, oa); if (more) split_v(nb, g + 3, 2); __builtin_amdgcn_sched_barrier(0);
            split_mfma(vb.h, pc.h, ob); if (more) split_v(nb, g + 3, 3); __builtin_amdgcn_sched_barrier(0);
            va = na;
            vb = nb;
        }
        __builtin_amdgcn_s_setprio(0);
    }

    l += __shfl_xor(l, 32, FC_WAVE);
    __syncthreads();                                   // Q is no longer read
    if (hh == 0) { m_s[wave * kUnitRows + l32] = m; l_s[wave * kUnitRows + l32] = l; }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        vrow_t v;
#pragma unroll
        for (int b = 0; b < NB; ++b) v[b] = o[b][i] * v_inv;
        *reinterpret_cast<vrow_t*>(&buf[(wave * kUnitRows + l32) * ROW + NB * ((i >> 2) * 8 + hh * 4 + (i & 3))]) = v;
    }
    __syncthreads();
    finish_unit<float, D, ROW>(a, p, it, buf, m_s, l_s, parts);
}

// ---- many query rows ----------------------------------------------------------------------------
// 128 query rows per block, 32 per wavefront, two blocks per compute unit.  The four wavefronts share every
// 32-key tile: it is read once, split into its f16 parts once (an eighth of the vector work of the body
// above) and double-buffered in LDS.  Step t: tile t's products and softmax, with the splitting of tile t + 1
// between the products of Q K^T, the loads of tile t + 2 behind them, and one barrier at the end.  V's scale
// is the block's; it is fixed a step before the tile is split, when the wavefronts have exchanged the
// largest entries that it does not fit yet.  The plan takes this body where it is cheaper over the recompute
// counts (attend_split.hpp).  us on the fp32 matrix cores / in 32-row blocks / here: 12 x 128, 2 chunks of 1021 rows on
// 4083 clean keys 650 / 357 / 277; 24 x 128, 460 rows on 3350 keys 237 / 130 / 114, 4 chunks of 460 617 / - / 311; 4 x 128, 4 of
// 1500 on 2000 815 / - / 292; 24 x 64, 2 of 500 on 4000 292 / - / 148.  Matrix cores 30 % busy: a wavefront issues for 2300
// of the 5400 cycles that a tile takes it and waits for LDS, memory and the barrier in the rest; half an XCD's blocks
// more would help, registers (256) and LDS (76 KB a block) allow two per compute unit.
template <int CTRL>
__device__ __forceinline__ float max_dpp(float v) {
    return fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true)));
}
// the maximum over each group of N consecutive lanes (8 or 16)
template <int N>
__device__ __forceinline__ float max_lanes(float v) {
    v = max_dpp<0xB1>(v);                   // quad_perm: neighbours
    v = max_dpp<0x4E>(v);                   // quad_perm: pairs
    v = max_dpp<0x141>(v);                  // row_half_mirror: the other four of eight
    return N == 16 ? max_dpp<0x140>(v) : v; // row_mirror: the other eight of sixteen
}

constexpr int kSharedThreads = 2 * kSharedRows;

template <int D>
__global__ __launch_bounds__(kSharedThreads, 2) void attend_f32_shared_kernel(FcAttendArgs a, FcAttendPlan p, float* parts) {
    constexpr int KS = D / 16;           // contraction steps of Q K^T
    constexpr int NB = D / 32;           // 32-wide blocks of the value dimension
    constexpr int KROW = D + 8, VROW = D + 32;       // padded rows, as in the bf16 kernel
    constexpr int LPR = D / 8;           // threads per row of a tile, eight entries each
    constexpr int RPP = kSharedThreads / LPR, NP = 32 / RPP;   // rows per pass, passes per tile
    constexpr float kTop = 15.0f, kStart = 12.0f;    // as above
    __shared__ __attribute__((aligned(16))) bf16_t K_s[2][2][32 * KROW], V_s[2][2][32 * VROW];   // [buffer][part]
    __shared__ __attribute__((aligned(16))) float k_scale[2][32], v_over[2][4];
    __shared__ Segments sg;

    const uint32_t valid = valid_blocks(a);
    if (valid == 0) return;
    const WideItem wi = wide_item<kSharedRows, false>(a, p, valid, blockIdx.x);
    if (!wi.ok) return;
    const int hk = wi.h / (a.H_q / a.H_k);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l32 = lane & 31, hh = lane >> 5, l16 = lane & 15;
    const float c2 = a.scale * 1.4426950408889634f;
    if (tid == 0) list_segments(a, a.rec_idx[wi.r], sg);

    // B operand of S^T = K Q^T: lane holds Q[q = l32][16 st + 8 hh .. + 8), scaled per row
    const int row_in_chunk = wi.tile * kSharedRows + wave * 32 + l32;
    Split8 qf[KS];
    float qs;
    {
        const int rc = row_in_chunk > a.L_c - 1 ? a.L_c - 1 : row_in_chunk;
        const float* qp = (const float*)a.q + (((int64_t)wi.r * a.L_c + rc) * a.H_q + wi.h) * D + 8 * hh;
        f32x4_t x[2 * KS];
        float most = 0.f;
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j) {
            x[j] = *reinterpret_cast<const f32x4_t*>(qp + 16 * (j >> 1) + 4 * (j & 1)) * c2;
            most = max_abs4(most, x[j]);
        }
        most = fmaxf(most, __shfl_xor(most, 32, FC_WAVE));
        const float sc = split_scale(most, qs);
#pragma unroll
        for (int st = 0; st < KS; ++st)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                split_pair(qf[st], e, x[2 * st + (e >> 1)][2 * (e & 1)], x[2 * st + (e >> 1)][2 * (e & 1) + 1], sc);
    }
    __syncthreads();

    const float* kbase = (const float*)a.k_cache + (int64_t)hk * a.head_stride;
    const float* vbase = (const float*)a.v_cache + (int64_t)hk * a.head_stride;
    const uint32_t ts = (uint32_t)a.tok_stride;
    const int nt_all = __builtin_amdgcn_readfirstlane(sg.tile0[sg.n]);
    const int t_lo = (int)((int64_t)nt_all * wi.s / wi.S), nt = (int)((int64_t)nt_all * (wi.s + 1) / wi.S) - t_lo;

    f32x16_t o[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[b][i] = 0.f;
    float m = kNegBig, l = 0.f;
    float v_most = 0.f, v_sc = 1.f, v_inv = 1.f;      // V's scale of the next tile to be split

    // tile t of the range -> registers, eight entries of a row per thread; rows past the end: the last one again
    f32x4_t kr[2 * NP], vr[2 * NP];
    int seg = 0, nv_load = 32;                        // valid keys of the tile loaded last
    const int ld_row = tid / LPR, ld_col = 8 * (tid % LPR);
    const uint32_t ld_off = ((uint32_t)ld_row * ts + (uint32_t)ld_col) * 4u;
    auto load = [&](int t) {
        const int tt = t_lo + (t < nt ? t : nt - 1);
        while (tt >= __builtin_amdgcn_readfirstlane(sg.tile0[seg + 1])) ++seg;
        const int off = (tt - __builtin_amdgcn_readfirstlane(sg.tile0[seg])) * 32;
        const int left = __builtin_amdgcn_readfirstlane(sg.len[seg]) - off;
        const int64_t pos = (int64_t)(__builtin_amdgcn_readfirstlane(sg.start[seg]) + off) * a.tok_stride;
        nv_load = left < 32 ? left : 32;
        const char* kt = reinterpret_cast<const char*>(kbase + pos);
        const char* vt = reinterpret_cast<const char*>(vbase + pos);
        const uint32_t last = ((uint32_t)(nv_load - 1) * ts + (uint32_t)ld_col) * 4u;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            uint32_t at = ld_off + (uint32_t)(j * RPP) * ts * 4u;
            at = at < last ? at : last;
            kr[2 * j] = *reinterpret_cast<const f32x4_t*>(kt + at);
            kr[2 * j + 1] = *reinterpret_cast<const f32x4_t*>(kt + at + 16);
            vr[2 * j] = *reinterpret_cast<const f32x4_t*>(vt + at);
            vr[2 * j + 1] = *reinterpret_cast<const f32x4_t*>(vt + at + 16);
        }
    };
    // what of the loaded V tile the scale does not fit: its largest entry per wavefront, or 0
    auto report_v = [&](int buf) {
        float vm = 0.f;
#pragma unroll
        for (int j = 0; j < 2 * NP; ++j) vm = max_abs4(vm, vr[j]);
        float over = 0.f;
        if (__any(vm > v_most)) {                         // an infinity spoils its own column only
            vm = 0.f;
#pragma unroll
            for (int j = 0; j < 2 * NP; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) vm = max_finite(vm, vr[j][e]);
            over = wave_max_all(vm);
        }
        if (lane == 0) v_over[buf][wave] = over;
    };
    // the scale for the tile reported in `buf`; returns what O is to be multiplied with before that tile is added
    auto follow_v = [&](int buf) {
        const f32x4_t x = *reinterpret_cast<const f32x4_t*>(v_over[buf]);
        const float over = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
        if (!(over > v_most)) return 1.0f;
        float inv;
        const float sc = split_scale(over, inv, 2);       // room for entries four times as large
        const float down = sc * v_inv;
        v_sc = sc; v_inv = inv; v_most = 32768.0f * inv;
        return down;
    };
    const int st_k = ld_row * KROW + ld_col, st_v = ld_row * VROW + ld_col;
    // The loaded tile into buffer `buf`, in pieces: piece i < 4 NP is a pair of K (i even) or V entries, the last of a
    // row's part stores it.
    Split8 ksp, vsp;
    float k_sc = 1.f;
    auto stage = [&](int buf, int j, int e) __attribute__((always_inline)) {
        if (e == 0) {
            const float most = max_lanes<LPR>(max_abs4(max_abs4(0.f, kr[2 * j]), kr[2 * j + 1]));
            float inv;
            k_sc = split_scale(most, inv);
            if (tid % LPR == 0) k_scale[buf][j * RPP + ld_row] = inv;
        }
        split_pair(ksp, e, kr[2 * j + (e >> 1)][2 * (e & 1)], kr[2 * j + (e >> 1)][2 * (e & 1) + 1], k_sc);
        split_pair(vsp, e, vr[2 * j + (e >> 1)][2 * (e & 1)], vr[2 * j + (e >> 1)][2 * (e & 1) + 1], v_sc);
        if (e == 3) {
            *reinterpret_cast<u32x4_native*>(&K_s[buf][0][st_k + j * RPP * KROW]) = ksp.h;
            *reinterpret_cast<u32x4_native*>(&K_s[buf][1][st_k + j * RPP * KROW]) = ksp.l;
            *reinterpret_cast<u32x4_native*>(&V_s[buf][0][st_v + j * RPP * VROW]) = vsp.h;
            *reinterpret_cast<u32x4_native*>(&V_s[buf][1][st_v + j * RPP * VROW]) = vsp.l;
        }
    };
    const int k_frag = l32 * KROW + 8 * hh;
    const int v_frag = (hh * 4 + (l16 >> 2)) * VROW + ((lane >> 4) & 1) * 16 + (l16 & 3) * 4;
    auto read_k = [&](int buf, int st) __attribute__((always_inline)) {
        return Split8{*reinterpret_cast<const u32x4_native*>(&K_s[buf][0][k_frag + 16 * st]),
                      *reinterpret_cast<const u32x4_native*>(&K_s[buf][1][k_frag + 16 * st])};
    };
    auto read_v1 = [&](const bf16_t* vp) __attribute__((always_inline)) {
        const s16x4_t lo = lds_read_tr(vp), hi = lds_read_tr(vp + 8 * VROW);
        return __builtin_bit_cast(u32x4_native, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto read_v = [&](int buf, int g) __attribute__((always_inline)) {    // g: 16-key step g / NB, value block g % NB
        const int at = v_frag + (g / NB) * 16 * VROW + (g % NB) * 32;
        return Split8{read_v1(&V_s[buf][0][at]), read_v1(&V_s[buf][1][at])};
    };

    if (nt > 0) {
        load(0);
        int nv = nv_load;
        report_v(0);
        __syncthreads();
        follow_v(0);                                  // (O is zero)
#pragma unroll
        for (int j = 0; j < NP; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) stage(0, j, e);
        load(1);
        report_v(1);
        __syncthreads();
        for (int t = 0; t < nt; ++t) {
            const int buf = t & 1;
            const float down = follow_v(buf ^ 1);
            const int nv_next = nv_load;
            f32x16_t s, s1;
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = s1[i] = 0.f;
            Split8 f0 = read_k(buf, 0), f1 = read_k(buf, 1), f2;
#pragma unroll
            for (int st = 0; st < KS; ++st) {
                if (st + 2 < KS) f2 = read_k(buf, st + 2);
                f32x16_t &c0 = st & 1 ? s : s1, &c1 = st & 1 ? s1 : s;   // no product waits for the one before it
                split_mfma(f0.l, qf[st].h, c0);
                __builtin_amdgcn_sched_barrier(0);
                split_mfma(f0.h, qf[st].h, c1);
                // tile t + 1: NP * 4 pieces over the steps
                if (st < 4 * NP) stage(buf ^ 1, st / 4, st % 4);
                __builtin_amdgcn_sched_barrier(0);
                split_mfma(f0.h, qf[st].l, c0);
                __builtin_amdgcn_sched_barrier(0);
                f0 = f1;
                f1 = f2;
            }
            load(t + 2);
            __builtin_amdgcn_sched_barrier(0);
            s += s1;
#pragma unroll
            for (int i = 0; i < 16; i += 4) {
                const f32x4_t ks = *reinterpret_cast<const f32x4_t*>(&k_scale[buf][2 * i + 4 * hh]);
#pragma unroll
                for (int e = 0; e < 4; ++e) s[i + e] = s[i + e] * ks[e] * qs;
            }
            if (nv < 32) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if ((i >> 2) * 8 + hh * 4 + (i & 3) >= nv) s[i] = kNegBig;
            }
            nv = nv_next;
            float mx = s[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
            if (__any(mx > m + kTop)) {
                const float mn = fmaxf(m, fmaxf(mx, __shfl_xor(mx, 32, FC_WAVE)) - kStart);
                const float alpha = __builtin_amdgcn_exp2f(m - mn);
                m = mn;
                l *= alpha;
#pragma unroll
                for (int b = 0; b < NB; ++b) o[b] *= alpha;
            }
            Split8 va = read_v(buf, 0), vb = read_v(buf, 1), na, nb;
            float p0 = 0.f, p1 = 0.f;
            Split8 ps[2];
#pragma unroll
            for (int i = 0; i < 16; i += 2) {
                const float x0 = __builtin_amdgcn_exp2f(s[i] - m), x1 = __builtin_amdgcn_exp2f(s[i + 1] - m);
                p0 += x0;
                p1 += x1;
                split_pair(ps[i >> 3], (i & 7) >> 1, x0, x1, 1.0f);
            }
            l += p0 + p1;
            // two blocks of O at a time
#pragma unroll
            for (int g = 0; g < 2 * NB; g += 2) {
                f32x16_t &oa = o[g % NB], &ob = o[g % NB + 1];
                const Split8& pc = ps[g / NB];
                if (g + 2 < 2 * NB) { na = read_v(buf, g + 2); nb = read_v(buf, g + 3); }
                split_mfma(va.l, pc.h, oa);
                split_mfma(vb.l, pc.h, ob);
                split_mfma(va.h, pc.l, oa);
                split_mfma(vb.h, pc.l, ob);
                split_mfma(va.h, pc.h, oa);
                split_mfma(vb.h, pc.h, ob);
                va = na;
                vb = nb;
                __builtin_amdgcn_sched_barrier(0);
            }
            if (down != 1.0f) {
#pragma unroll
                for (int b = 0; b < NB; ++b) o[b] *= down;
            }
            report_v(buf);
            __syncthreads();
        }
    }

    const float ltot = l + __shfl_xor(l, 32, FC_WAVE);
    if (wi.S > 1) {
        const int64_t part = (wi.unit * (kSharedRows / kUnitRows) + wave) * wi.S + wi.s;   // 32 rows each
        float* po = parts + (part * kUnitRows + l32) * D;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                store_out(po + b * 32 + g * 8 + hh * 4, o[b][4 * g] * v_inv, o[b][4 * g + 1] * v_inv, o[b][4 * g + 2] * v_inv,
                          o[b][4 * g + 3] * v_inv);
        if (hh == 0) {
            float* ml = parts + (int64_t)p.parts * kUnitRows * D + part * 2 * kUnitRows;
            ml[l32] = m;
            ml[kUnitRows + l32] = ltot;
        }
        return;
    }
    if (row_in_chunk >= a.L_c) return;
    const float inv = 1.0f / ltot;
    const int64_t row = (int64_t)wi.r * a.L_c + row_in_chunk;
    float* op = (float*)a.out + (row * a.H_q + wi.h) * D;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            store_out(op + b * 32 + g * 8 + hh * 4, o[b][4 * g] * v_inv * inv, o[b][4 * g + 1] * v_inv * inv,
                      o[b][4 * g + 2] * v_inv * inv, o[b][4 * g + 3] * v_inv * inv);
    if (a.lse && hh == 0)
        a.lse[(int64_t)wi.h * a.A * a.L_c + row] = (m + __builtin_amdgcn_logf(ltot)) * 0.6931471805599453f;
}

template <int D>
int launch_f32(const FcAttendArgs& a, hipStream_t s) {
    FcAttendPlan p = fc_attend_plan_f32(a.A, a.L_c, a.L_clean, a.H_q, true);
    if (!fc_room_for_partials(a.ws, a.ws_bytes, p.parts, D))    // (those of 32-row blocks are a third or less)
        p = fc_attend_plan_f32(a.A, a.L_c, a.L_clean, a.H_q, true, false);
    if (!fc_room_for_partials(a.ws, a.ws_bytes, p.parts, D))
        p = fc_attend_plan_f32(a.A, a.L_c, a.L_clean, a.H_q, false);
    if (p.narrow[0])                                   // one form for every recompute count
        attend_f32_kernel<D><<<p.grid, kSplitThreads, 0, s>>>(a, p, (float*)a.ws);
    else
        attend_f32_shared_kernel<D><<<p.grid, kSharedThreads, 0, s>>>(a, p, (float*)a.ws);
    FC_LAUNCH_CHECK();
    if (p.merge_grid > 0) {
        attend_merge_kernel<float, D, kSharedRows, false><<<p.merge_grid, 256, 0, s>>>(a, p, (const float*)a.ws);
        FC_LAUNCH_CHECK();
    }
    return FC_OK;
}

}  // namespace

int fc_launch_scatter_kv(const FcScatterArgs& a, hipStream_t s) {
    const int esz = (a.dtype == FC_BF16) ? 2 : 4;
    const int vpr = a.d * esz / 16;                       // 16-byte vectors per row
    const int64_t hs = a.head_stride * esz / 16, ts = a.tok_stride * esz / 16;
    const int64_t per_chunk = (int64_t)a.L_c * a.H_k * vpr;
    int gx = (int)((per_chunk + 256 * 4 - 1) / (256 * 4));
    gx = gx < 1 ? 1 : (gx > 2048 ? 2048 : gx);
    scatter_kv_kernel<<<dim3(gx, a.A), 256, 0, s>>>((const uint4*)a.k_new, (const uint4*)a.v_new,
                                                     (uint4*)a.k_cache, (uint4*)a.v_cache, hs, ts,
                                                     a.H_k, vpr, a.L_c, a);
    FC_LAUNCH_CHECK();
    return FC_OK;
}

int fc_launch_attend_f32(const FcAttendArgs& a, hipStream_t s) {
    if (a.d == 64) return launch_f32<64>(a, s);
    if (a.d == 128) return launch_f32<128>(a, s);
    return FC_UNSUPPORTED;
}

size_t fc_attend_split_workspace(int A, int L_c, int H_q, int d) {
    return fc_align_up((size_t)fc_split_parts_bound(A, L_c, H_q) * fc_split_part_bytes(d));
}
