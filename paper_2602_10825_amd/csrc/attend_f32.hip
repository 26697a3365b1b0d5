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
// On the bf16 matrix cores, every operand in three bf16 parts (f32_split.hpp); two bodies, as in bf16 (attend_bf16.hip), and
// the launch plan's costs say which (attend_split.hpp).
//   S^T = K Q^T  puts one query per lane, so maximum and sum are in-lane but for one exchange,
//   and the accumulators of S^T already are the B operand of  O^T += V^T P^T.
constexpr int BQ = kWideRows;        // query rows per block of the wide body
constexpr int BK = 32;               // keys per tile
constexpr int NT = kSplitThreads;
// The exponents' reference is raised this far beyond the row maximum when that passes it (log2): weights are at most 1.
constexpr float kAhead = 4.0f;

// The 32 rows of a wavefront over its tiles t, t + step, ... < t_end once more, with fp32 products: for inputs of which a
// part or a sum was not finite.  `q` is the lane's own row from column 4 hh on; value column col0 + b col_step of the lane
// is row l32 of block b.  Slow: every wavefront reads its operands from memory.
template <int D>
__device__ __forceinline__ void rows_in_fp32(const float* q, const float* kbase, const float* vbase, uint32_t ts, const Segments& sg,
                                             int t, int t_end, int step, float c2, int col0, int col_step,
                                             f32x16_t (&o)[D / 32], float& m, float& l) {
    constexpr int NB = D / 32;
    const int lane = threadIdx.x & 63, l32 = lane & 31, hh = lane >> 5;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[b][i] = 0.f;
    m = kNegBig;
    l = 0.f;
    int seg = 0;
#pragma unroll 1
    for (; t < t_end; t += step) {
        while (t >= __builtin_amdgcn_readfirstlane(sg.tile0[seg + 1])) ++seg;
        const int off = (t - __builtin_amdgcn_readfirstlane(sg.tile0[seg])) * BK;
        const int left = __builtin_amdgcn_readfirstlane(sg.len[seg]) - off, nv = left < BK ? left : BK;
        const int64_t pos = (int64_t)(__builtin_amdgcn_readfirstlane(sg.start[seg]) + off) * ts;
        const float *kt = kbase + pos, *vt = vbase + pos;
        const float* kr = kt + (uint32_t)(l32 < nv ? l32 : nv - 1) * ts + 4 * hh;
        f32x16_t s;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll 2
        for (int j = 0; j < D / 8; ++j) {        // the product of step (j, i) contracts over elements 8 j + i and 8 j + 4 + i
            const f32x4_t kf = *reinterpret_cast<const f32x4_t*>(kr + 8 * j), qf = *reinterpret_cast<const f32x4_t*>(q + 8 * j) * c2;
#pragma unroll
            for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[i], qf[i], s, 0, 0, 0);
        }
        if (nv < BK) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if ((i >> 2) * 8 + hh * 4 + (i & 3) >= nv) s[i] = kNegBig;
        }
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
        const float mn = fmaxf(m, fmaxf(mx, __shfl_xor(mx, 32, FC_WAVE))), alpha = __builtin_amdgcn_exp2f(m - mn);
        m = mn;
        float ps = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) { s[i] = __builtin_amdgcn_exp2f(s[i] - mn); ps += s[i]; }
        l = fmaf(l, alpha, ps);
#pragma unroll
        for (int b = 0; b < NB; ++b) o[b] *= alpha;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int key = (i >> 2) * 8 + hh * 4 + (i & 3);
            const float* vr = vt + (uint32_t)(key < nv ? key : nv - 1) * ts + col0;
#pragma unroll
            for (int b = 0; b < NB; ++b) o[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[b * col_step], s[i], o[b], 0, 0, 0);
        }
    }
}
template <int NB>
__device__ __forceinline__ bool to_do_in_fp32(bool odd, const f32x16_t (&o)[NB], float l) {
    uint64_t lanes = __ballot(odd) | odd_sum(l);
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) lanes |= odd_sum(o[b][i]);
    return lanes != 0;
}

// ---- few query rows -----------------------------------------------------------------------------
// A block is 32 query rows; its 8 wavefronts take every 8th 32-key tile and never meet before the end, where their
// partials are merged through LDS; a launch of few rows still occupies eight wavefronts per 32 rows.  Bound by the vector
// ALU: about 950 instructions a tile and wavefront, three quarters of them splitting K and V, against 96 products of 32 cycles.
// Q's parts are in LDS; K is read as rows and turned to the operand's layout there.  us on the fp32 matrix cores / here: 12 x 128,
// 6 chunks of 87 rows on 4399 clean keys 208 / 136; 2 x 128, 700 rows on 10400 keys 106 / 69; 8 x 64, 86 rows on 16100 54 / 42; 4
// query heads on 1 x 64, 2 x 128 rows on 512 clean keys 22 / 16.5.  (Each tile's sum by itself, as in the body below: 60
// registers too many at head dimension 128, 136 -> 200.)  The two chains of products run at raised priority (in turn on one
// card: 123 -> 121 and 15.8 -> 15.0 for the first and the last of these).
template <int N> struct VecF;
template <> struct VecF<4> { typedef float type __attribute__((ext_vector_type(4))); };
template <> struct VecF<2> { typedef float type __attribute__((ext_vector_type(2))); };

template <int D>
struct NarrowSmem {
    static constexpr int ROW = D + 4;    // padded rows of K tiles and of the partial O (floats),
    static constexpr int QROW = D + 8;   // and of Q's parts (bf16): 16-byte reads of 32 rows spread over the banks
    __attribute__((aligned(16))) bf16_t q[3][kUnitRows * QROW];              // (first: 16-bit offsets reach all of it)
    __attribute__((aligned(16))) float buf[kSplitWaves * kUnitRows * ROW];   // a K tile per wavefront, partial O at the end
    float m_s[kSplitWaves * kUnitRows], l_s[kSplitWaves * kUnitRows];
    __attribute__((aligned(16))) uint32_t odd[kSplitWaves];   // rows of Q that need fp32 products, by the wavefront that split them
    Segments sg;
};

template <int D>
__device__ __forceinline__ void attend_narrow(const FcAttendArgs& a, const FcAttendPlan& p, uint32_t valid,
                                              NarrowSmem<D>& sm, float* parts) {
    constexpr int KS = D / 16;           // contraction steps of Q K^T
    constexpr int NB = D / 32;           // 32-wide blocks of the value dimension
    constexpr int ROW = NarrowSmem<D>::ROW, QROW = NarrowSmem<D>::QROW;
    typedef typename VecF<NB>::type vrow_t;
    Segments& sg = sm.sg;

    const SplitItem it = split_item(a, p, valid, blockIdx.x);
    if (!it.ok) return;
    const int hk = it.h / (a.H_q / a.H_k);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l32 = lane & 31, hh = lane >> 5;
    const float c2 = a.scale * 1.4426950408889634f;   // fold log2(e): exp(x) = exp2(x*log2 e)
    auto q_row = [&](int row) {
        int rc = it.tile * kUnitRows + row;
        if (rc > a.L_c - 1) rc = a.L_c - 1;
        return (const float*)a.q + (((int64_t)it.r * a.L_c + rc) * a.H_q + it.h) * D;
    };

    if (tid == 0) list_segments(a, it.c, sg);
    bool odd = false;
    if (tid < kUnitRows * (D / 8)) {
        const int row = tid / (D / 8), e = tid % (D / 8);
        const float* qp = q_row(row) + 8 * e;
        const f32x4_t v0 = *reinterpret_cast<const f32x4_t*>(qp) * c2, v1 = *reinterpret_cast<const f32x4_t*>(qp + 4) * c2;
#pragma unroll
        for (int i = 0; i < 4; ++i) odd = odd || odd_magnitude(v0[i]) || odd_magnitude(v1[i]);
        Split8 s;
        split_pair(s, 0, v0[0], v0[1]); split_pair(s, 1, v0[2], v0[3]);
        split_pair(s, 2, v1[0], v1[1]); split_pair(s, 3, v1[2], v1[3]);
        *reinterpret_cast<u32x4_native*>(sm.q[0] + row * QROW + 8 * e) = s.h;
        *reinterpret_cast<u32x4_native*>(sm.q[1] + row * QROW + 8 * e) = s.m;
        *reinterpret_cast<u32x4_native*>(sm.q[2] + row * QROW + 8 * e) = s.l;
    }
    odd = __any(odd);
    if (lane == 0) sm.odd[wave] = odd;
    __syncthreads();

    const float* kbase = (const float*)a.k_cache + (int64_t)hk * a.head_stride;
    const float* vbase = (const float*)a.v_cache + (int64_t)hk * a.head_stride;
    const int nt = __builtin_amdgcn_readfirstlane(sg.tile0[sg.n]);
    const int t_end = (int)((int64_t)nt * (it.s + 1) / it.S);
    const int t_first = (int)((int64_t)nt * it.s / it.S) + wave;
    int t = t_first;

    f32x16_t o[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[b][i] = 0.f;
    float m = kNegBig, l = 0.f;
    const uint32_t ts = (uint32_t)a.tok_stride;

    f32x4_t kf[2 * KS];
    vrow_t vf[16];
    int seg = 0, pos = 0, nvalid = 0;
    auto locate = [&](int tt) {
        while (tt >= __builtin_amdgcn_readfirstlane(sg.tile0[seg + 1])) ++seg;
        const int off = (tt - __builtin_amdgcn_readfirstlane(sg.tile0[seg])) * BK;
        const int left = __builtin_amdgcn_readfirstlane(sg.len[seg]) - off;
        pos = __builtin_amdgcn_readfirstlane(sg.start[seg]) + off;
        nvalid = left < BK ? left : BK;
    };
    // Whole rows at a time; A operand of S^T = K Q^T: lane (hh, l32) holds K[l32][16 st + 8 hh .. + 8)
    constexpr int LPR = D / 4, RPL = FC_WAVE / LPR;     // lanes per row, rows per load
    const int ld_row = lane / LPR, ld_col = 4 * (lane % LPR);
    const uint32_t k_off = ((uint32_t)ld_row * ts + (uint32_t)ld_col) * 4u, v_off = ((uint32_t)hh * 4u * ts + (uint32_t)(NB * l32)) * 4u;
    float* const k_tile = sm.buf + wave * 32 * ROW;
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
    const int q_frag = l32 * QROW + 8 * hh;
    auto read_q = [&](int st) {
        return Split8{*reinterpret_cast<const u32x4_native*>(&sm.q[0][q_frag + 16 * st]),
                      *reinterpret_cast<const u32x4_native*>(&sm.q[1][q_frag + 16 * st]),
                      *reinterpret_cast<const u32x4_native*>(&sm.q[2][q_frag + 16 * st])};
    };

    if (t < t_end) { locate(t); load_k(); }
    while (t < t_end) {
        const int nv = nvalid, vpos = pos;
        turn_k();
        auto split_k = [&](Split8& x, int st, int p) __attribute__((always_inline)) {
            split_pair(x, p, kf[2 * st + (p >> 1)][2 * (p & 1)], kf[2 * st + (p >> 1)][2 * (p & 1) + 1]);
        };
        f32x16_t s, s1;                                // the largest products, and the others
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = s1[i] = 0.f;
        Split8 cur, nxt, qc;
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int p = 0; p < 4; ++p) split_k(cur, 0, p);
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            const bool more = st + 1 < KS;
            qc = read_q(st);
            split_mfma(cur.l, qc.h, s1); if (more) split_k(nxt, st + 1, 0); __builtin_amdgcn_sched_barrier(0);
            split_mfma(cur.h, qc.l, s1); __builtin_amdgcn_sched_barrier(0);
            split_mfma(cur.m, qc.m, s1); if (more) split_k(nxt, st + 1, 1); __builtin_amdgcn_sched_barrier(0);
            split_mfma(cur.m, qc.h, s1); if (more) split_k(nxt, st + 1, 2); __builtin_amdgcn_sched_barrier(0);
            split_mfma(cur.h, qc.m, s1); __builtin_amdgcn_sched_barrier(0);
            split_mfma(cur.h, qc.h, s); if (more) split_k(nxt, st + 1, 3);
            if (st == KS / 2 - 1) load_v(0, vpos, nv);     // K's first half is used up: its registers are free
            __builtin_amdgcn_sched_barrier(0);
            cur = nxt;
        }
        __builtin_amdgcn_s_setprio(0);
        load_v(1, vpos, nv);
        __builtin_amdgcn_sched_barrier(0);
        s += s1;
        if (nv < BK) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if ((i >> 2) * 8 + hh * 4 + (i & 3) >= nv) s[i] = kNegBig;
        }
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
        if (__any(mx > m)) {
            const float top = fmaxf(mx, __shfl_xor(mx, 32, FC_WAVE)), mn = top > m ? top + kAhead : m;
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
            split_pair(ps[i >> 3], (i & 7) >> 1, x0, x1);
        }
        l += p0 + p1;
        auto split_v = [&](Split8& x, int g, int p) __attribute__((always_inline)) {
            split_pair(x, p, vf[8 * (g / NB) + 2 * p][g % NB], vf[8 * (g / NB) + 2 * p + 1][g % NB]);
        };
        t += kSplitWaves;
        Split8 va, na;
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int p = 0; p < 4; ++p) split_v(va, 0, p);
#pragma unroll
        for (int g = 0; g < 2 * NB; ++g) {
            f32x16_t& oa = o[g % NB];
            const Split8& pc = ps[g / NB];
            const bool more = g + 1 < 2 * NB;
            split_mfma(va.l, pc.h, oa); if (more) split_v(na, g + 1, 0); __builtin_amdgcn_sched_barrier(0);
            split_mfma(va.h, pc.l, oa); __builtin_amdgcn_sched_barrier(0);
            split_mfma(va.m, pc.m, oa); if (more) split_v(na, g + 1, 1); __builtin_amdgcn_sched_barrier(0);
            split_mfma(va.m, pc.h, oa); if (more) split_v(na, g + 1, 2); __builtin_amdgcn_sched_barrier(0);
            split_mfma(va.h, pc.m, oa); __builtin_amdgcn_sched_barrier(0);
            split_mfma(va.h, pc.h, oa); if (more) split_v(na, g + 1, 3); __builtin_amdgcn_sched_barrier(0);
            va = na;
            if (g == NB - 1 && t < t_end) { locate(t); load_k(); }   // V's first half is used up: the next tile's keys
        }
        __builtin_amdgcn_s_setprio(0);
    }
    const u32x4_native odd0 = *reinterpret_cast<const u32x4_native*>(sm.odd), odd1 = *reinterpret_cast<const u32x4_native*>(sm.odd + 4);
    odd = (odd0[0] | odd0[1] | odd0[2] | odd0[3] | odd1[0] | odd1[1] | odd1[2] | odd1[3]) != 0u;
    if (to_do_in_fp32<NB>(odd, o, l))
        rows_in_fp32<D>(q_row(l32) + 4 * hh, kbase, vbase, ts, sg, t_first, t_end, kSplitWaves, c2, NB * l32, 1, o, m, l);

    l += __shfl_xor(l, 32, FC_WAVE);
    __syncthreads();                                   // every wavefront is done with its K tile
    if (hh == 0) { sm.m_s[wave * kUnitRows + l32] = m; sm.l_s[wave * kUnitRows + l32] = l; }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        vrow_t v;
#pragma unroll
        for (int b = 0; b < NB; ++b) v[b] = o[b][i];
        *reinterpret_cast<vrow_t*>(&sm.buf[(wave * kUnitRows + l32) * ROW + NB * ((i >> 2) * 8 + hh * 4 + (i & 3))]) = v;
    }
    __syncthreads();
    finish_unit<float, D, ROW>(a, p, it, sm.buf, sm.m_s, sm.l_s, parts);
}

// ---- many query rows ----------------------------------------------------------------------------
// 256 query rows per block, 32 per wavefront, whose Q stays in registers (some of its last parts in LDS).  The eight
// wavefronts share every 32-key tile: it is read once, split into its parts once (an eighth of the vector work of the body
// above) and double-buffered in LDS.  Step t: tile t's products and softmax, with the splitting of tile t + 1 between the
// products of Q K^T, the loads of tile t + 2 among those of P V, and one barrier at the end.  A tile's contribution to O is summed up by itself and then added, which
// costs nothing, as that is one instruction with the rescaling of O, and rounds O once per 32 keys instead of 12 times.  The
// smaller products of Q K^T come first for the same reason.  us on the fp32 matrix cores / here: 12 x 128, 2 chunks of 1021
// rows on 4083 clean keys 690 / 398; 24 x 128, 460 rows on 3350 keys 239 / 132; 24 x 64, 1024 rows on 61024 3110 / 1890; 12 x 64, 2 of
// 1021 on 4083 349 / 212.  Q K^T runs at raised priority, so that the wavefronts of a SIMD part (in turn: 408 -> 398, 217 -> 212;
// over P V instead 401, 221).  Relative error against float64, 22 shapes: 3.4e-7 .. 16e-7 and, with the body above, 2.0e-7 ..
// 5.4e-7, nowhere larger.  Matrix cores 62 % busy while a block runs (1.86 GHz): no product covers the weights of a tile's first
// half.  (A half-tile shift between the two wavefronts of a SIMD, with a third V buffer: 442 -> 464.)  All of Q's parts in
// registers are 24 too many: five were read back from memory in each tile, 435 -> 411.
template <int D>
struct WideSmem {
    static constexpr int KROW = D + 8, VROW = D + 32;       // padded rows, as in the bf16 kernel
    __attribute__((aligned(16))) bf16_t K[2][3][BK * KROW], V[2][3][BK * VROW];   // [buffer][part]
    static constexpr int QL = D == 128 ? 6 : 0;      // steps of which Q's last part is kept here, every wavefront's own
    u32x4_native ql[QL > 0 ? QL : 1][kSplitWaves][FC_WAVE];
    Segments sg;
};

template <int D>
__device__ __forceinline__ void attend_wide(const FcAttendArgs& a, const FcAttendPlan& p, uint32_t valid,
                                            WideSmem<D>& sm, float* parts) {
    constexpr int KS = D / 16;           // contraction steps of Q K^T
    constexpr int NB = D / 32;           // 32-wide blocks of the value dimension
    constexpr int KROW = WideSmem<D>::KROW, VROW = WideSmem<D>::VROW;
    constexpr int QL = WideSmem<D>::QL;
    constexpr int EPT = BK * D / NT;     // entries of K, and of V, per thread and tile: all of one row
    constexpr int LPR = D / EPT;         // threads per row
    typedef uint32_t word_t __attribute__((ext_vector_type(EPT / 2)));
    static_assert(NT / LPR == BK && EPT % 4 == 0, "one pass per tile");
    Segments& sg = sm.sg;

    const WideItem wi = wide_item<true>(a, p, valid, blockIdx.x);
    if (!wi.ok) return;
    const int hk = wi.h / (a.H_q / a.H_k);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l32 = lane & 31, hh = lane >> 5, l16 = lane & 15;
    const float c2 = a.scale * 1.4426950408889634f;
    if (tid == 0) list_segments(a, a.rec_idx[wi.r], sg);

    // B operand of S^T = K Q^T: lane holds Q[q = l32][16 st + 8 hh .. + 8)
    const int row_in_chunk = wi.tile * BQ + wave * 32 + l32;
    const float* q_row = (const float*)a.q + (((int64_t)wi.r * a.L_c + (row_in_chunk > a.L_c - 1 ? a.L_c - 1 : row_in_chunk)) * a.H_q + wi.h) * D;
    Split8 qf[KS];
    bool odd = false;
#pragma unroll
    for (int st = 0; st < KS; ++st) {
        const f32x4_t x0 = *reinterpret_cast<const f32x4_t*>(q_row + 16 * st + 8 * hh) * c2;
        const f32x4_t x1 = *reinterpret_cast<const f32x4_t*>(q_row + 16 * st + 8 * hh + 4) * c2;
#pragma unroll
        for (int i = 0; i < 4; ++i) odd = odd || odd_magnitude(x0[i]) || odd_magnitude(x1[i]);
        split_pair(qf[st], 0, x0[0], x0[1]); split_pair(qf[st], 1, x0[2], x0[3]);
        split_pair(qf[st], 2, x1[0], x1[1]); split_pair(qf[st], 3, x1[2], x1[3]);
        if (st < QL) sm.ql[st][wave][lane] = qf[st].l;
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

    // tile t of the range -> registers, entries of one row per thread; rows past the end: the last one again
    f32x4_t kr[EPT / 4], vr[EPT / 4];
    int seg = 0, nv_load = BK;                        // valid keys of the tile loaded last
    const int ld_row = tid / LPR, ld_col = EPT * (tid % LPR);
    const uint32_t ld_off = ((uint32_t)ld_row * ts + (uint32_t)ld_col) * 4u;
    auto load = [&](int t) {
        const int tt = t_lo + (t < nt ? t : nt - 1);
        while (tt >= __builtin_amdgcn_readfirstlane(sg.tile0[seg + 1])) ++seg;
        const int off = (tt - __builtin_amdgcn_readfirstlane(sg.tile0[seg])) * BK;
        const int left = __builtin_amdgcn_readfirstlane(sg.len[seg]) - off;
        const int64_t pos = (int64_t)(__builtin_amdgcn_readfirstlane(sg.start[seg]) + off) * a.tok_stride;
        nv_load = left < BK ? left : BK;
        const char* kt = reinterpret_cast<const char*>(kbase + pos);
        const char* vt = reinterpret_cast<const char*>(vbase + pos);
        const uint32_t last = ((uint32_t)(nv_load - 1) * ts + (uint32_t)ld_col) * 4u;
        const uint32_t at = ld_off < last ? ld_off : last;
#pragma unroll
        for (int j = 0; j < EPT / 4; ++j) {
            kr[j] = *reinterpret_cast<const f32x4_t*>(kt + at + 16 * j);
            vr[j] = *reinterpret_cast<const f32x4_t*>(vt + at + 16 * j);
        }
    };
    const int st_k = ld_row * KROW + ld_col, st_v = ld_row * VROW + ld_col;
    // The loaded tile into buffer `buf`, a pair of K's and V's entries at a time; the last pair stores.
    Split8 ksp, vsp;
    auto store_part = [&](bf16_t* at, const u32x4_native& x) __attribute__((always_inline)) {
        word_t w;
#pragma unroll
        for (int i = 0; i < EPT / 2; ++i) w[i] = x[i];
        *reinterpret_cast<word_t*>(at) = w;
    };
    auto stage_k = [&](int buf, int e) __attribute__((always_inline)) {
        split_pair(ksp, e, kr[e >> 1][2 * (e & 1)], kr[e >> 1][2 * (e & 1) + 1]);
        if (e < EPT / 2 - 1) return;
        store_part(&sm.K[buf][0][st_k], ksp.h); store_part(&sm.K[buf][1][st_k], ksp.m); store_part(&sm.K[buf][2][st_k], ksp.l);
    };
    auto stage_v = [&](int buf, int e) __attribute__((always_inline)) {
        split_pair(vsp, e, vr[e >> 1][2 * (e & 1)], vr[e >> 1][2 * (e & 1) + 1]);
        if (e < EPT / 2 - 1) return;
        store_part(&sm.V[buf][0][st_v], vsp.h); store_part(&sm.V[buf][1][st_v], vsp.m); store_part(&sm.V[buf][2][st_v], vsp.l);
    };
    const int k_frag = l32 * KROW + 8 * hh;
    const int v_frag = (hh * 4 + (l16 >> 2)) * VROW + ((lane >> 4) & 1) * 16 + (l16 & 3) * 4;
    auto read_k = [&](int buf, int st) __attribute__((always_inline)) {
        return Split8{*reinterpret_cast<const u32x4_native*>(&sm.K[buf][0][k_frag + 16 * st]),
                      *reinterpret_cast<const u32x4_native*>(&sm.K[buf][1][k_frag + 16 * st]),
                      *reinterpret_cast<const u32x4_native*>(&sm.K[buf][2][k_frag + 16 * st])};
    };
    auto read_kh = [&](int buf, int st) __attribute__((always_inline)) {
        return *reinterpret_cast<const u32x4_native*>(&sm.K[buf][0][k_frag + 16 * st]);
    };
    auto read_v1 = [&](const bf16_t* vp) __attribute__((always_inline)) {
        const s16x4_t lo = lds_read_tr(vp), hi = lds_read_tr(vp + 8 * VROW);
        return __builtin_bit_cast(u32x4_native, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto read_v = [&](int buf, int g) __attribute__((always_inline)) {    // g: value block g / 2, 16-key step g % 2
        const int at = v_frag + (g % 2) * 16 * VROW + (g / 2) * 32;
        return Split8{read_v1(&sm.V[buf][0][at]), read_v1(&sm.V[buf][1][at]), read_v1(&sm.V[buf][2][at])};
    };

    if (nt > 0) {
        load(0);
        int nv = nv_load;
#pragma unroll
        for (int e = 0; e < EPT / 2; ++e) { stage_k(0, e); stage_v(0, e); }
        load(1);
        lds_barrier();
#pragma unroll 1
        for (int t = 0; t < nt; ++t) {
            const int buf = t & 1;
            f32x16_t s;
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = 0.f;
            // the smaller products first: then only the largest ones, K's first parts read once more, round the scores' bits
            Split8 f0 = read_k(buf, 0), f1;
            __builtin_amdgcn_s_setprio(1);
            u32x4_native h0, h1, h2;
#pragma unroll
            for (int st = 0; st < KS; ++st) {
                if (st + 1 < KS) f1 = read_k(buf, st + 1);
                else { h0 = read_kh(buf, 0); h1 = read_kh(buf, 1); }
                const u32x4_native ql = st < QL ? sm.ql[st][wave][lane] : qf[st].l;
                split_mfma(f0.l, qf[st].h, s);
                split_mfma(f0.m, qf[st].m, s);
                __builtin_amdgcn_sched_barrier(0);
                if (st < EPT / 2) stage_k(buf ^ 1, st);    // tile t + 1
                else stage_v(buf ^ 1, st - EPT / 2);
                split_mfma(f0.m, qf[st].h, s);
                split_mfma(f0.h, ql, s);
                split_mfma(f0.h, qf[st].m, s);
                __builtin_amdgcn_sched_barrier(0);
                f0 = f1;
            }
#pragma unroll
            for (int st = 0; st < KS; ++st) {
                if (st + 2 < KS) h2 = read_kh(buf, st + 2);
                split_mfma(h0, qf[st].h, s);
                __builtin_amdgcn_sched_barrier(0);
                h0 = h1;
                h1 = h2;
            }
            __builtin_amdgcn_s_setprio(0);
            Split8 va = read_v(buf, 0), na;
            if (nv < BK) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if ((i >> 2) * 8 + hh * 4 + (i & 3) >= nv) s[i] = kNegBig;
            }
            nv = nv_load;                                  // of tile t + 1
            float mx = s[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
            float alpha = 1.0f;
            if (__any(mx > m)) {
                const float top = fmaxf(mx, __shfl_xor(mx, 32, FC_WAVE)), mn = top > m ? top + kAhead : m;
                alpha = __builtin_amdgcn_exp2f(m - mn);
                m = mn;
                l *= alpha;
            }
            float p0 = 0.f, p1 = 0.f;
            Split8 ps[2];
            auto weights = [&](int i) __attribute__((always_inline)) {      // of accumulators i and i + 1
                const float x0 = __builtin_amdgcn_exp2f(s[i] - m), x1 = __builtin_amdgcn_exp2f(s[i + 1] - m);
                p0 += x0;
                p1 += x1;
                split_pair(ps[i >> 3], (i & 7) >> 1, x0, x1);
            };
#pragma unroll
            for (int i = 0; i < 8; i += 2) weights(i);
            f32x16_t x;
#pragma unroll
            for (int g = 0; g < 2 * NB; ++g) {                 // value block g / 2, 16-key step g % 2
                const int b = g / 2;
                if (g % 2 == 0) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) x[i] = 0.f;
                }
                if (g + 1 < 2 * NB) na = read_v(buf, g + 1);
                const Split8& pc = ps[g % 2];
                split_mfma(va.l, pc.h, x); if (g == 0) weights(8); __builtin_amdgcn_sched_barrier(0);
                split_mfma(va.h, pc.l, x); if (g == 0) weights(10); __builtin_amdgcn_sched_barrier(0);
                split_mfma(va.m, pc.m, x); if (g == 0) weights(12); __builtin_amdgcn_sched_barrier(0);
                split_mfma(va.m, pc.h, x); if (g == 0) weights(14); __builtin_amdgcn_sched_barrier(0);
                split_mfma(va.h, pc.m, x); __builtin_amdgcn_sched_barrier(0);
                split_mfma(va.h, pc.h, x);
                va = na;
                if (g % 2 == 1) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) o[b][i] = fmaf(o[b][i], alpha, x[i]);
                }
                if (g == 1) load(t + 2);                   // (the scores' registers are free)
            }
            l += p0 + p1;
            lds_barrier();
        }
    }
    if (to_do_in_fp32<NB>(odd, o, l))
        rows_in_fp32<D>(q_row + 4 * hh, kbase, vbase, ts, sg, t_lo, t_lo + nt, 1, c2, l32, 32, o, m, l);

    const float ltot = l + __shfl_xor(l, 32, FC_WAVE);
    if (wi.S > 1) {
        const int64_t part = (wi.unit * (BQ / kUnitRows) + wave) * wi.S + wi.s;   // 32 rows each
        float* po = parts + (part * kUnitRows + l32) * D;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                store_out(po + b * 32 + g * 8 + hh * 4, o[b][4 * g], o[b][4 * g + 1], o[b][4 * g + 2], o[b][4 * g + 3]);
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
            store_out(op + b * 32 + g * 8 + hh * 4, o[b][4 * g] * inv, o[b][4 * g + 1] * inv, o[b][4 * g + 2] * inv, o[b][4 * g + 3] * inv);
    if (a.lse && hh == 0)
        a.lse[(int64_t)wi.h * a.A * a.L_c + row] = (m + __builtin_amdgcn_logf(ltot)) * 0.6931471805599453f;
}

// WIDE and NARROW say which of the two bodies some recompute count of this launch asks for.
template <int D, bool WIDE, bool NARROW>
__global__ __launch_bounds__(NT) void attend_f32_kernel(FcAttendArgs a, FcAttendPlan p, float* parts) {
    const uint32_t valid = valid_blocks(a);
    const int R = __popc(valid);
    if (R == 0) return;
    constexpr size_t w = WIDE ? sizeof(WideSmem<D>) : 0, n = NARROW ? sizeof(NarrowSmem<D>) : 0;
    __shared__ __attribute__((aligned(16))) char raw[w > n ? w : n];
    if (WIDE && (!NARROW || !p.narrow[R - 1]))
        attend_wide<D>(a, p, valid, *reinterpret_cast<WideSmem<D>*>(raw), parts);
    else if (NARROW)
        attend_narrow<D>(a, p, valid, *reinterpret_cast<NarrowSmem<D>*>(raw), parts);
}

template <int D>
int launch_f32(const FcAttendArgs& a, hipStream_t s) {
    FcAttendPlan p = fc_attend_plan_f32(a.A, a.L_c, a.L_clean, a.H_q, true, D);
    if (!fc_room_for_partials(a.ws, a.ws_bytes, p.parts, D))
        p = fc_attend_plan_f32(a.A, a.L_c, a.L_clean, a.H_q, false, D);
    bool wide = false, narrow = false;
    for (int R = 0; R < a.A; ++R) (p.narrow[R] ? narrow : wide) = true;
    if (!narrow)
        attend_f32_kernel<D, true, false><<<p.grid, NT, 0, s>>>(a, p, (float*)a.ws);
    else if (!wide)
        attend_f32_kernel<D, false, true><<<p.grid, NT, 0, s>>>(a, p, (float*)a.ws);
    else
        attend_f32_kernel<D, true, true><<<p.grid, NT, 0, s>>>(a, p, (float*)a.ws);
    FC_LAUNCH_CHECK();
    if (p.merge_grid > 0) {
        attend_merge_kernel<float, D><<<p.merge_grid, 256, 0, s>>>(a, p, (const float*)a.ws);
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
