// What the attention kernels that split the keys share: the plan (how many key ranges), the
// list of visible key segments, and the merge of the ranges' partial results.
//
// A work unit is 32 query rows of one head of one recompute chunk.  Its keys are divided over
// the 8 wavefronts of a block (merged through LDS), and, where the launch has fewer units than
// the chip has compute units, over S blocks besides: each of those leaves an unnormalised
// partial (O, row reference m, row sum l) in the workspace and attend_merge_kernel puts the S
// partials together.  S depends on the number of recompute chunks R, which only the device
// knows, so the host prepares the answer for every R.
#pragma once

#include "fc_common.hpp"

constexpr int kUnitRows = 32;
constexpr int kSplitWaves = 8;
constexpr int kSplitThreads = kSplitWaves * FC_WAVE;
constexpr int kMaxSplits = 32;
constexpr int kCus = 256;
constexpr float kNegBig = -1.0e30f;

struct FcSplitPlan {
    int tiles;                           // 32-row tiles per chunk
    int grid;                            // blocks of the attention launch
    int merge_grid;                      // blocks of the merge launch (0: never needed)
    int parts;                           // partials the workspace has to hold
    uint8_t splits[FC_MAX_ACTIVE];       // S for R = 1 .. A
};

// S minimises rounds of one block per compute unit, times the key tiles of a round.  A block also
// costs `block_cost` key tiles of prologue and merging, and the merge launch twice that; a range
// has at least `block_cost` tiles, and no launch is split into more than four blocks per compute
// unit (so the partials stay within 18 MB).
inline int fc_choose_splits(int64_t units, int key_tiles, int block_cost) {
    int cap = key_tiles / block_cost;
    cap = cap < 1 ? 1 : (cap > kMaxSplits ? kMaxSplits : cap);
    int best = 1;
    double best_cost = 0.0;
    for (int s = 1; s <= cap; ++s) {
        if (s > 1 && units * s > 4 * kCus) break;
        const double rounds = (double)((units * s + kCus - 1) / kCus);
        const double cost = rounds * ((double)key_tiles / s + block_cost) + (s > 1 ? 2 * block_cost : 0);
        if (s == 1 || cost < 0.97 * best_cost) { best = s; best_cost = cost; }
    }
    return best;
}

inline FcSplitPlan fc_split_plan(int A, int L_c, int L_clean, int H_q, int block_cost, bool may_split) {
    FcSplitPlan p{};
    p.tiles = (L_c + kUnitRows - 1) / kUnitRows;
    const int key_tiles = (int)(((int64_t)L_clean + (int64_t)A * L_c + 31) / 32);
    for (int R = 1; R <= A; ++R) {
        const int64_t units = (int64_t)R * H_q * p.tiles;
        const int S = may_split ? fc_choose_splits(units, key_tiles, block_cost) : 1;
        p.splits[R - 1] = (uint8_t)S;
        const int n = (int)((units * S + 7) / 8 * 8);
        if (n > p.grid) p.grid = n;
        if (S > 1) {
            if (units > p.merge_grid) p.merge_grid = (int)units;
            if (units * S > p.parts) p.parts = (int)(units * S);
        }
    }
    return p;
}
// Most partials a launch with these shapes can need, whatever the number of keys.
inline int fc_split_parts_bound(int A, int L_c, int H_q) {
    const int64_t tiles = (L_c + kUnitRows - 1) / kUnitRows;
    int64_t most = 0;
    for (int R = 1; R <= A; ++R) {
        const int64_t units = (int64_t)R * H_q * tiles;
        int64_t s = 4 * kCus / units;
        if (s > kMaxSplits) s = kMaxSplits;
        if (s > 1 && units * s > most) most = units * s;
    }
    return (int)most;
}
// bytes per partial: O [32][d], then m [32] and l [32]
inline size_t fc_split_part_bytes(int d) { return (size_t)kUnitRows * (d + 2) * sizeof(float); }

// ---- device side ---------------------------------------------------------------------------
// The recompute list is the device's: a count above A is cut to A and an entry outside [0, A) is
// skipped (nothing is read or written for it).  Bit r of the mask = row block r holds a chunk; R =
// the number of such blocks, so that a malformed list is planned like the well-formed one.
__device__ __forceinline__ uint32_t valid_blocks(const FcAttendArgs& a) {
    const int lane = threadIdx.x & (FC_WAVE - 1);
    const int c = a.rec_idx[lane < a.A ? lane : 0];
    const uint32_t mask = (uint32_t)__ballot(lane < min(*a.n_rec, a.A) && (unsigned)c < (unsigned)a.A);
    return mask;
}
// the row block with `rank` valid ones above it: latest (heaviest) chunk first
__device__ __forceinline__ int block_of_rank(uint32_t mask, int rank) {
    for (int i = 0; i < rank; ++i) mask &= ~(0x80000000u >> __clz((int)mask));
    return 31 - __clz((int)mask);
}

struct SplitItem { int R, S, r, c, h, tile, s; int64_t part; bool ok; };

// Block -> (head, chunk, key range, row tile).  Consecutive blocks go round the 8 XCDs, so item
// numbers are dealt to them in contiguous runs: the row tiles that read the same keys run on
// one XCD and share its L2.
__device__ __forceinline__ SplitItem split_item(const FcAttendArgs& a, const FcSplitPlan& p, int bid) {
    SplitItem it;
    it.ok = false;
    const uint32_t valid = valid_blocks(a);
    it.R = __popc(valid);
    if (it.R == 0) return it;
    it.S = p.splits[it.R - 1];
    const int n = it.R * a.H_q * p.tiles * it.S;
    const int per = (n + 7) / 8;
    const int slot = bid >> 3;
    const int item = (bid & 7) * per + slot;
    if (slot >= per || item >= n) return it;
    it.tile = item % p.tiles;
    int rest = item / p.tiles;
    it.s = rest % it.S;
    rest /= it.S;
    const int rank = rest % it.R;
    it.h = rest / it.R;
    it.part = (int64_t)((it.h * it.R + rank) * p.tiles + it.tile) * it.S + it.s;
    it.r = block_of_rank(valid, rank);
    it.c = a.rec_idx[it.r];
    it.ok = true;
    return it;
}

// Visible key segments of chunk c (clean region, then active chunks 0..c; adjacent ones merged)
// with the number of 32-key tiles before each.  Filled by one thread.
struct Segments {
    int n;
    int start[FC_MAX_ACTIVE + 1], len[FC_MAX_ACTIVE + 1], tile0[FC_MAX_ACTIVE + 2];
};
__device__ __forceinline__ void list_segments(const FcAttendArgs& a, int c, Segments& sg) {
    int n = 0, sgi = -1, t = 0;
    while (sgi <= c) {
        const int start = (sgi < 0) ? 0 : a.active_off[sgi];
        int len = (sgi < 0) ? a.L_clean : a.L_c;
        ++sgi;
        while (sgi <= c && a.active_off[sgi] == start + len) { len += a.L_c; ++sgi; }
        if (len > 0) {
            sg.start[n] = start; sg.len[n] = len; sg.tile0[n] = t;
            t += (len + 31) / 32;
            ++n;
        }
    }
    sg.tile0[n] = t;
    sg.n = n;
}

__device__ __forceinline__ void store_out(float* p, float v0, float v1, float v2, float v3) {
    *reinterpret_cast<float4*>(p) = make_float4(v0, v1, v2, v3);
}
__device__ __forceinline__ void store_out(bf16_t* p, float v0, float v1, float v2, float v3) {
    uint2 pk;
    pk.x = (uint32_t)f32_to_bf16(v0) | ((uint32_t)f32_to_bf16(v1) << 16);
    pk.y = (uint32_t)f32_to_bf16(v2) | ((uint32_t)f32_to_bf16(v3) << 16);
    *reinterpret_cast<uint2*>(p) = pk;
}

// End of a block: the 8 wavefronts' partials (O in LDS, rows of OROW floats; m and l per row)
// are put together; one thread per 16th of a row.  Writes the result (S = 1) or the partial.
template <typename T, int D, int OROW>
__device__ __forceinline__ void finish_unit(const FcAttendArgs& a, const FcSplitPlan& p, const SplitItem& it,
                                            const float* o_s, const float* m_s, const float* l_s,
                                            float* parts) {
    constexpr int PER = D / 16;
    const int row = threadIdx.x >> 4, c0 = (threadIdx.x & 15) * PER;
    float mt = kNegBig;
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) mt = fmaxf(mt, m_s[w * kUnitRows + row]);
    float acc[PER], l = 0.f;
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] = 0.f;
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) {
        const float f = __builtin_amdgcn_exp2f(m_s[w * kUnitRows + row] - mt);
        l = fmaf(l_s[w * kUnitRows + row], f, l);
        const float* src = o_s + (w * kUnitRows + row) * OROW + c0;
#pragma unroll
        for (int e = 0; e < PER; ++e) acc[e] = fmaf(src[e], f, acc[e]);
    }
    const int row_in_chunk = it.tile * kUnitRows + row;
    if (it.S > 1) {
        float* po = parts + (it.part * kUnitRows + row) * D + c0;
#pragma unroll
        for (int e = 0; e < PER; e += 4) store_out(po + e, acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
        if (c0 == 0) {
            float* ml = parts + (int64_t)p.parts * kUnitRows * D + it.part * 2 * kUnitRows;
            ml[row] = mt;
            ml[kUnitRows + row] = l;
        }
        return;
    }
    if (row_in_chunk >= a.L_c) return;
    const float inv = 1.0f / l;
    const int64_t grow = (int64_t)it.r * a.L_c + row_in_chunk;
    T* op = (T*)a.out + (grow * a.H_q + it.h) * D + c0;
#pragma unroll
    for (int e = 0; e < PER; e += 4) store_out(op + e, acc[e] * inv, acc[e + 1] * inv, acc[e + 2] * inv, acc[e + 3] * inv);
    if (a.lse && c0 == 0)
        a.lse[(int64_t)it.h * a.A * a.L_c + grow] = (mt + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
}

// The S partials of every unit -> out and lse.  One block per unit, 8 threads per row.
template <typename T, int D>
__global__ __launch_bounds__(256) void attend_merge_kernel(FcAttendArgs a, FcSplitPlan p, const float* parts) {
    constexpr int PER = D / 8;
    const uint32_t valid = valid_blocks(a);
    const int R = __popc(valid);
    if (R == 0) return;
    const int S = p.splits[R - 1];
    const int unit = blockIdx.x;
    if (S == 1 || unit >= R * a.H_q * p.tiles) return;
    const int tile = unit % p.tiles;
    const int r = block_of_rank(valid, (unit / p.tiles) % R), h = unit / (p.tiles * R);
    const int row = threadIdx.x >> 3, c0 = (threadIdx.x & 7) * PER;
    const int row_in_chunk = tile * kUnitRows + row;
    if (row_in_chunk >= a.L_c) return;
    const float* ml = parts + (int64_t)p.parts * kUnitRows * D + (int64_t)unit * S * 2 * kUnitRows;
    float mt = kNegBig;
    for (int s = 0; s < S; ++s) mt = fmaxf(mt, ml[s * 2 * kUnitRows + row]);
    float acc[PER], l = 0.f;
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] = 0.f;
    for (int s = 0; s < S; ++s) {
        const float f = __builtin_amdgcn_exp2f(ml[s * 2 * kUnitRows + row] - mt);
        l = fmaf(ml[(s * 2 + 1) * kUnitRows + row], f, l);
        const float4* src = reinterpret_cast<const float4*>(parts + (((int64_t)unit * S + s) * kUnitRows + row) * D + c0);
#pragma unroll
        for (int e = 0; e < PER / 4; ++e) {
            const float4 v = src[e];
            acc[4 * e] = fmaf(v.x, f, acc[4 * e]);
            acc[4 * e + 1] = fmaf(v.y, f, acc[4 * e + 1]);
            acc[4 * e + 2] = fmaf(v.z, f, acc[4 * e + 2]);
            acc[4 * e + 3] = fmaf(v.w, f, acc[4 * e + 3]);
        }
    }
    const float inv = 1.0f / l;
    const int64_t grow = (int64_t)r * a.L_c + row_in_chunk;
    T* op = (T*)a.out + (grow * a.H_q + h) * D + c0;
#pragma unroll
    for (int e = 0; e < PER; e += 4) store_out(op + e, acc[e] * inv, acc[e + 1] * inv, acc[e + 2] * inv, acc[e + 3] * inv);
    if (a.lse && c0 == 0)
        a.lse[(int64_t)h * a.A * a.L_c + grow] = (mt + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
}
