// K/V scatter of the recompute chunks into their cache slots, and the fp32 chunk-causal
// attention kernel (Sec. 3.3; softmax(q K^T d^-1/2) V with a chunk-granular causal mask).
//
#include "attend_split.hpp"

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
// Bound by the fp32 matrix cores (v_mfma_f32_32x32x2_f32, 157 TFLOP/s; a library product of two
// 8192 matrices reaches 153).  A block is 32 query rows; its 8 wavefronts take every 8th 32-key
// tile, read K and V straight into registers in the operands' own layout and never meet before
// the end, where their partials are merged through LDS: at 64 matrix-core cycles per product
// there is time for the uncoalesced K reads, nothing has to be shared through LDS except Q, and a
// launch of few rows still occupies eight wavefronts per 32 rows.
//   S^T = K Q^T  puts one query per lane, so maximum and sum are in-lane but for one exchange,
//   and the accumulators of S^T already are the B operand of  O^T += V^T P^T.
// 12 heads x 128, 2 chunks of 1021 rows on 4083 clean keys: 642 us, 110 TFLOP/s (one row per
// thread on the vector ALU: 18.8 ms, 3.7); 4 query heads on 1 x 64, 2 x 128 rows on 512: 19 us
// (1136 us).  Splitting over blocks as well (us without / with): 8 heads x 128, 448 rows on 33682
// keys 1217 / 592; 1 head, 68 rows on 30068 keys 1066 / 72; 12 heads, 1021 rows on 6125: 451 / 365.
typedef float f32x16_t __attribute__((ext_vector_type(16)));

template <int N> struct VecF;
template <> struct VecF<4> { typedef float type __attribute__((ext_vector_type(4))); };
template <> struct VecF<2> { typedef float type __attribute__((ext_vector_type(2))); };

template <int D>
__global__ __launch_bounds__(kSplitThreads) void attend_f32_kernel(FcAttendArgs a, FcAttendPlan p, float* parts) {
    constexpr int NB = D / 32;           // 32-wide blocks of the value dimension
    constexpr int ROW = D + 4;           // padded LDS rows (floats): 16-byte reads of 32 rows spread over the banks
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    typedef typename VecF<NB>::type vrow_t;
    __shared__ __attribute__((aligned(16))) float buf[kSplitWaves * kUnitRows * ROW];   // Q first, partial O at the end
    __shared__ float m_s[kSplitWaves * kUnitRows], l_s[kSplitWaves * kUnitRows];
    __shared__ Segments sg;

    const SplitItem it = split_item(a, p, valid_blocks(a), blockIdx.x);
    if (!it.ok) return;
    const int hk = it.h / (a.H_q / a.H_k);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l32 = lane & 31, hh = lane >> 5;
    const float c2 = a.scale * 1.4426950408889634f;   // fold log2(e): exp(x) = exp2(x*log2 e)

    if (tid == 0) list_segments(a, it.c, sg);
    for (int i = tid; i < kUnitRows * (D / 4); i += kSplitThreads) {
        const int row = i / (D / 4), e = i % (D / 4);
        int rc = it.tile * kUnitRows + row;
        if (rc > a.L_c - 1) rc = a.L_c - 1;
        f32x4_t v = *reinterpret_cast<const f32x4_t*>(
            (const float*)a.q + (((int64_t)it.r * a.L_c + rc) * a.H_q + it.h) * D + 4 * e);
        *reinterpret_cast<f32x4_t*>(&buf[row * ROW + 4 * e]) = v * c2;
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
    const uint32_t ts = (uint32_t)a.tok_stride;

    f32x4_t kf[D / 8];
    vrow_t vf[16];
    int seg = 0, pos = 0, nvalid = 0;
    auto locate = [&](int tt) {
        while (tt >= __builtin_amdgcn_readfirstlane(sg.tile0[seg + 1])) ++seg;
        const int off = (tt - __builtin_amdgcn_readfirstlane(sg.tile0[seg])) * 32;
        const int left = __builtin_amdgcn_readfirstlane(sg.len[seg]) - off;
        pos = __builtin_amdgcn_readfirstlane(sg.start[seg]) + off;
        nvalid = left < 32 ? left : 32;
    };
    // A operand of S^T = K Q^T: lane (hh, l32) holds K[l32][8 j + 4 hh .. + 4); the MFMA of step
    // (j, i) contracts over the two elements 8 j + i and 8 j + 4 + i
    auto load_k = [&]() {
        const int kr = l32 < nvalid ? l32 : nvalid - 1;
        const char* kt = reinterpret_cast<const char*>(kbase + (int64_t)pos * a.tok_stride);   // scalar
        const uint32_t off = ((uint32_t)kr * ts + 4u * (uint32_t)hh) * 4u;
#pragma unroll
        for (int j = 0; j < D / 8; ++j) kf[j] = *reinterpret_cast<const f32x4_t*>(kt + off + 32 * j);
    };
    if (t < t_end) { locate(t); load_k(); }
    while (t < t_end) {
        // A operand of O^T += V^T P^T: row l32 of block b is value column NB * l32 + b, so one
        // wide load per key serves all blocks; step i contracts over the two keys of accumulator i
        const int nv = nvalid;
        const char* vt = reinterpret_cast<const char*>(vbase + (int64_t)pos * a.tok_stride);   // scalar
        if (nv == 32) {
            const uint32_t off = ((uint32_t)hh * 4u * ts + (uint32_t)(NB * l32)) * 4u;
#pragma unroll
            for (int i = 0; i < 16; ++i)
                vf[i] = *reinterpret_cast<const vrow_t*>(vt + (uint64_t)(((i >> 2) * 8 + (i & 3)) * ts) * 4u + off);
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                int key = (i >> 2) * 8 + hh * 4 + (i & 3);
                key = key < nv ? key : nv - 1;
                vf[i] = *reinterpret_cast<const vrow_t*>(vt + ((uint32_t)key * ts + (uint32_t)(NB * l32)) * 4u);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x16_t s;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int j = 0; j < D / 8; ++j) {
            const f32x4_t qf = *reinterpret_cast<const f32x4_t*>(&buf[l32 * ROW + 8 * j + 4 * hh]);
#pragma unroll
            for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j][i], qf[i], s, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        t += kSplitWaves;
        if (t < t_end) { locate(t); load_k(); }        // the next tile's keys, behind the softmax and P V
        if (nv < 32) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if ((i >> 2) * 8 + hh * 4 + (i & 3) >= nv) s[i] = kNegBig;
        }
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, FC_WAVE));
        const float mn = fmaxf(m, mx);
        const float alpha = __builtin_amdgcn_exp2f(m - mn);
        m = mn;
        float ps = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) { s[i] = __builtin_amdgcn_exp2f(s[i] - mn); ps += s[i]; }
        l = fmaf(l, alpha, ps);
#pragma unroll
        for (int b = 0; b < NB; ++b) o[b] *= alpha;
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int b = 0; b < NB; ++b) o[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[i][b], s[i], o[b], 0, 0, 0);
    }

    l += __shfl_xor(l, 32, FC_WAVE);
    __syncthreads();                                   // Q is no longer read
    if (hh == 0) { m_s[wave * kUnitRows + l32] = m; l_s[wave * kUnitRows + l32] = l; }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        vrow_t v;
#pragma unroll
        for (int b = 0; b < NB; ++b) v[b] = o[b][i];
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
