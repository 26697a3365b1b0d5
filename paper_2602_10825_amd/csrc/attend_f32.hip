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
//   that follows the largest entry the wavefront has seen; the weights none, their range is the choice
//   of the reference.
// 12 heads x 128, 2 chunks of 1021 rows on 4083 clean keys: 650 us on the fp32 matrix cores (69 % busy, no
// vector instruction beside them), now 357; 24 x 128, 460 rows on 4890 keys 237 / 130; 12 x 64, 2 x 174 rows on
// 18580 keys 246 / 163; 4 query heads on 1 x 64, 2 x 128 rows on 512: 19 / 14.  Relative error against float64
// 3.4e-7 .. 6.3e-7 before, 2.9e-7 .. 4.2e-7 now; at twice the logits 8e-7 .. 16e-7 and 5e-7 .. 7e-7.
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
        load_v(1, vpos, nv);
        t += kSplitWaves;
        if (t < t_end) { locate(t); load_k(); }        // the next tile's keys, behind the softmax and P V
        __builtin_amdgcn_sched_barrier(0);
        s += s1;
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
            const f32x4_t ks = *reinterpret_cast<const f32x4_t*>(&k_scale[wave][2 * i + 4 * hh]);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[i + e] *= ks[e] * qs;
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
            float inv;
            const float sc = split_scale(4.0f * wave_max_all(vm), inv);
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

template <int D>
int launch_f32(const FcAttendArgs& a, hipStream_t s) {
    FcAttendPlan p = fc_attend_plan_f32(a.A, a.L_c, a.L_clean, a.H_q, true);
    if (!fc_room_for_partials(a.ws, a.ws_bytes, p.parts, D))
        p = fc_attend_plan_f32(a.A, a.L_c, a.L_clean, a.H_q, false);
    attend_f32_kernel<D><<<p.grid, kSplitThreads, 0, s>>>(a, p, (float*)a.ws);
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
