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

constexpr int kWideRows = 256;        // query rows per block of the wide bodies

struct FcAttendPlan {
    int tiles;                           // 32-row tiles per chunk
    int grid;                            // blocks of the attention launch
    int merge_grid;                      // blocks of the merge launch (0: never needed)
    int parts;                           // 32-row partials the workspace has to hold
    uint8_t narrow[FC_MAX_ACTIVE];       // for R = 1 .. A: 32-row blocks (else 256-row blocks)
    uint8_t splits[FC_MAX_ACTIVE];       // and the number of key ranges S
};

// Cost of a launch of 32-row blocks, one per compute unit at a time, in the time of one key tile
// (32 keys, one of the block's 8 wavefronts): rounds of blocks times the tiles of a range.  A
// block also costs `block_cost` tiles of prologue and merging, and the merge launch twice that; a
// range has at least 8 tiles, and no launch is split into more than four blocks per compute unit.
// The partials of such a launch are at most 17 MB, those of split 256-row blocks (two per compute
// unit, eight partials each) at most 68.
inline double fc_narrow_cost(int64_t units, int key_tiles, int block_cost, bool may_split, int* splits) {
    int cap = may_split ? key_tiles / kSplitWaves : 1;
    cap = cap < 1 ? 1 : (cap > kMaxSplits ? kMaxSplits : cap);
    double best_cost = 0.0;
    for (int s = 1; s <= cap; ++s) {
        if (s > 1 && units * s > 4 * kCus) break;
        const double rounds = (double)((units * s + kCus - 1) / kCus);
        const int per_wave = ((key_tiles + s - 1) / s + kSplitWaves - 1) / kSplitWaves;
        const double cost = rounds * (per_wave * kSplitWaves + block_cost) + (s > 1 ? 2 * block_cost : 0);
        if (s == 1 || cost < 0.97 * best_cost) { *splits = s; best_cost = cost; }
    }
    return best_cost;
}

inline void fc_plan_add(FcAttendPlan& p, int R, int64_t blocks, int64_t merge_units, int S) {
    p.splits[R - 1] = (uint8_t)S;
    const int n = (int)((blocks + 7) / 8 * 8);
    if (n > p.grid) p.grid = n;
    if (S > 1) {
        if (merge_units > p.merge_grid) p.merge_grid = (int)merge_units;
        if (merge_units * S > p.parts) p.parts = (int)(merge_units * S);
    }
}

// Wide launch: U = R * H_q * ceil(L_c / 256) units.  With fewer units than compute units all of them
// are split S ways; otherwise only those of the last, partly filled round (per XCD: the units
// past the last multiple of 32).
struct FcWideShape { int per, n, full, rem; };   // per XCD: units of one chunk, of all, unsplit, split
__host__ __device__ inline FcWideShape fc_wide_shape(int R, int items, int S) {
    FcWideShape w;
    w.per = (items + 7) / 8;
    w.n = R * w.per;
    w.full = S > 1 ? w.n / (kCus / 8) * (kCus / 8) : w.n;
    w.rem = w.n - w.full;
    return w;
}

// Microseconds, from times of both forms with forced S: a wide block's 64 keys, its fixed cost, the merge launch, a split
// block's further cost (short pipeline, writing and merging its partial) and what the merge takes per range; an eighth of
// the time in which a narrow block's 8 wavefronts take one 32-key tile each, and its fixed cost in those.
struct FcAttendCosts { double w_tile, w_block, w_merge, w_parts, w_range, n_tile; int n_block; bool by_chunk; };

inline FcAttendPlan fc_attend_plan(int A, int L_c, int L_clean, int H_q, bool may_split, const FcAttendCosts& c) {
    FcAttendPlan p{};
    p.tiles = (L_c + kUnitRows - 1) / kUnitRows;
    const int64_t keys = (int64_t)L_clean + (int64_t)A * L_c;
    const int items = H_q * ((L_c + kWideRows - 1) / kWideRows);
    for (int R = 1; R <= A; ++R) {
        int Sn = 1, Sw = 1;
        const int64_t units = (int64_t)R * H_q * p.tiles;
        const double narrow = c.n_tile * fc_narrow_cost(units, (int)((keys + 31) / 32), c.n_block, may_split, &Sn);
        // Rounds of 256-row units run heaviest chunk first; the chunk of rank r sees at most this many tiles.
        // (With the newest chunk's keys counted for all, 24 x 64 with 6 chunks of 386 rows and no context split
        // a last round that sees a sixth of them: 51 us against 44.)
        auto seen = [&](int rank) { return (double)(((int64_t)L_clean + (int64_t)(A - rank) * L_c + 63) / 64); };
        const FcWideShape u = fc_wide_shape(R, items, 1);
        const int full_rounds = u.n / (kCus / 8), left = u.n % (kCus / 8);
        double before = 0.0;                      // the full rounds
        for (int rank = 0, q = 0; rank < R; ++rank) {
            int end = ((rank + 1) * u.per + kCus / 8 - 1) / (kCus / 8);
            if (end > full_rounds) end = full_rounds;
            before += (end - q) * (seen(rank) * c.w_tile + c.w_block);
            q = end;
        }
        const double T = left ? seen(full_rounds * (kCus / 8) / u.per) : 0.0;   // of the last, partly filled one
        double last = left ? T * c.w_tile + c.w_block : 0.0;
        for (int S = 2; S <= kMaxSplits && left && may_split && T >= 2 * S; ++S) {
            const int64_t split = full_rounds == 0 ? (int64_t)R * items * S : (int64_t)8 * left * S;   // blocks of split units
            if (split > 2 * kCus) break;
            const double rounds = (double)((split + kCus - 1) / kCus);
            const double cost = rounds * (T / S * c.w_tile + c.w_block + c.w_parts) + c.w_merge + S * c.w_range;
            // (behind full rounds the last one's start overlaps their end)
            if (cost < (full_rounds ? last - c.w_block : 0.97 * last)) { last = cost; Sw = S; }
        }
        if (narrow < before + last) {
            p.narrow[R - 1] = 1;
            fc_plan_add(p, R, units * Sn, units, Sn);
        } else {
            const FcWideShape w = fc_wide_shape(R, items, Sw);
            const bool flat = Sw > 1 && w.full == 0;
            const int64_t split_units = Sw == 1 ? 0 : flat ? (int64_t)R * items : (int64_t)8 * w.rem;
            const int64_t share = ((c.by_chunk ? 1 : R) * (int64_t)items * Sw + 7) / 8;      // of an XCD
            fc_plan_add(p, R, flat ? (int64_t)8 * (c.by_chunk ? R : 1) * share : (int64_t)8 * w.full + split_units * Sw,
                        split_units * (kWideRows / kUnitRows), Sw);
        }
    }
    return p;
}
// bf16, 12 x 128: 600 rows on 5200 keys narrow 40 / wide 50 with S = 4; 1200 rows 91 / 57; 1500 rows on 51689 keys 1040 / 470.
inline FcAttendPlan fc_attend_plan_bf16(int A, int L_c, int L_clean, int H_q, int d, bool may_split) {
    return fc_attend_plan(A, L_c, L_clean, H_q, may_split, d == 128 ? FcAttendCosts{1.75, 5.0, 5.0, 14.0, 0.0, 0.235, 11, false}
                                                                    : FcAttendCosts{1.15, 5.0, 5.0, 8.0, 0.0, 0.17, 11, false});
}
// fp32, best S of each: 12 x 128, 2 chunks of 1021 rows on 4083 clean keys narrow 481 / wide 381; 6 of 87 on 4399 122 / 226; 24 x 128,
// 460 rows on 3350 156 / 127; 2 x 128, 700 rows on 10400 66 / 87; 12 x 64, 2 of 174 on 18406 175 / 162; 4 x 64, 2 of 500 on 3000 40 / 46.
inline FcAttendPlan fc_attend_plan_f32(int A, int L_c, int L_clean, int H_q, bool may_split, int d = 128) {
    return fc_attend_plan(A, L_c, L_clean, H_q, may_split, d == 128 ? FcAttendCosts{8.2, 8.0, 5.0, 16.0, 0.5, 0.74, 8, true}
                                                                    : FcAttendCosts{4.5, 6.0, 5.0, 8.0, 0.5, 0.42, 8, true});
}

// Most 32-row partials a launch with these shapes can need, whatever the number of keys.  The wide
// plan takes S only where the last round costs less than with every smaller S'.  Both costs are a + b T
// in the number of tiles T and a never falls with S (more rounds of blocks, a merge), so b, the rounds of
// split blocks over S, has to be smaller.
inline int64_t fc_split_parts_bound(int A, int L_c, int H_q) {
    const int64_t tiles = (L_c + kUnitRows - 1) / kUnitRows;
    const int64_t items = (int64_t)H_q * ((L_c + kWideRows - 1) / kWideRows);
    int64_t most = 0;
    for (int R = 1; R <= A; ++R) {
        const int64_t units = (int64_t)R * H_q * tiles;
        int64_t s = 4 * kCus / units;
        if (s > kMaxSplits) s = kMaxSplits;
        if (s > 1 && units * s > most) most = units * s;
        double least = (double)((fc_wide_shape(R, (int)items, 1).full + kCus / 8 - 1) / (kCus / 8));
        for (int S = 2; S <= kMaxSplits; ++S) {
            const FcWideShape w = fc_wide_shape(R, (int)items, S);
            const int64_t split = w.full == 0 ? (int64_t)R * items * S : (int64_t)8 * w.rem * S;
            if (split == 0 || split > 2 * kCus) break;
            const double b = (double)(w.full / (kCus / 8)) + (double)((split + kCus - 1) / kCus) / S;
            if (b >= least) continue;
            least = b;
            if (split * (kWideRows / kUnitRows) > most) most = split * (kWideRows / kUnitRows);
        }
    }
    return most;
}
// bytes per partial: O [32][d], then m [32] and l [32]
inline size_t fc_split_part_bytes(int d) { return (size_t)kUnitRows * (d + 2) * sizeof(float); }

// Room for the plan's partials?  They are written and read 16 bytes at a time; a pointer that does not
// allow that is no room.
inline bool fc_room_for_partials(const void* ws, size_t ws_bytes, int parts, int d) {
    return parts == 0 || (ws && ((uintptr_t)ws & 15u) == 0 && ws_bytes >= (size_t)parts * fc_split_part_bytes(d));
}

// ---- device side ---------------------------------------------------------------------------
// The recompute list is the device's: a count above A is cut to A and an entry outside [0, A) is
// skipped (nothing is read or written for it).  The list may end after *n_rec entries: what lies
// beyond is not read.  The chunk of row block i, or -1:
__host__ __device__ inline int fc_listed_chunk(const int32_t* rec_idx, int n_rec, int A, int i) {
    if (i >= n_rec || i >= A) return -1;
    const int c = rec_idx[i];
    return (unsigned)c < (unsigned)A ? c : -1;
}
// Bit r of the mask = row block r holds a chunk; R = the number of such blocks, so that a malformed
// list is planned like the well-formed one.
__device__ __forceinline__ uint32_t valid_blocks(const FcAttendArgs& a) {
    return (uint32_t)__ballot(fc_listed_chunk(a.rec_idx, *a.n_rec, a.A, threadIdx.x & (FC_WAVE - 1)) >= 0);
}
// the row block with `rank` valid ones above it: latest (heaviest) chunk first
__device__ __forceinline__ int block_of_rank(uint32_t mask, int rank) {
    for (int i = 0; i < rank; ++i) mask &= ~(0x80000000u >> __clz((int)mask));
    return 31 - __clz((int)mask);
}

struct SplitItem { int R, S, r, c, h, tile, s; int64_t part; bool ok; };

// Block -> (head, chunk, key range, row tile) of a launch of 32-row blocks.  Consecutive blocks go
// round the 8 XCDs, so item numbers are dealt to them in contiguous runs: the row tiles that read
// the same keys run on one XCD and share its L2.
__device__ __forceinline__ SplitItem split_item(const FcAttendArgs& a, const FcAttendPlan& p, uint32_t valid, int bid) {
    SplitItem it;
    const int R = __popc(valid);
    it.ok = false;
    if (R == 0) return it;
    it.R = R;
    it.S = p.splits[R - 1];
    const int n = R * a.H_q * p.tiles * it.S;
    const int per = (n + 7) / 8;
    const int slot = bid >> 3;
    const int item = (bid & 7) * per + slot;
    if (slot >= per || item >= n) return it;
    it.tile = item % p.tiles;
    int rest = item / p.tiles;
    it.s = rest % it.S;
    rest /= it.S;
    const int rank = rest % R;
    it.h = rest / R;
    it.part = (int64_t)((it.h * R + rank) * p.tiles + it.tile) * it.S + it.s;
    it.r = block_of_rank(valid, rank);
    it.c = a.rec_idx[it.r];
    it.ok = true;
    return it;
}

// The same for 256-row blocks.  The 32 compute units of an XCD work on the same head and chunk at
// the same time and share the K/V stream through its L2; heaviest chunk first.  `unit` numbers the
// split units.
struct WideItem { int r, h, tile, s, S; int64_t unit; bool ok; };
__device__ __forceinline__ WideItem wide_unit(const FcAttendArgs& a, uint32_t valid, int items, int rank, int item) {
    WideItem wi;
    const int tiles = (a.L_c + kWideRows - 1) / kWideRows;
    wi.ok = item < items;
    wi.r = block_of_rank(valid, rank);
    wi.h = item / tiles;
    wi.tile = item % tiles;
    return wi;
}
// BY_CHUNK: where all units are split, every XCD has its share of each chunk's blocks, heaviest first (fp32, 12 x 128, 2 chunks of
// 1021 rows on 4083 clean keys 432 -> 404 us, 12 x 64 240 -> 228, 4 chunks of 385 rows 178 -> 167, 8 x 128, 3 of 500 160 -> 162.5;
// bf16 gains or loses, 2 x 128, 6 of 2000 rows 189 -> 170, 12 x 128, 2 of 1000 on 53000 keys 625 -> 643, and keeps the other order).
template <bool BY_CHUNK>
__device__ __forceinline__ WideItem wide_item(const FcAttendArgs& a, const FcAttendPlan& p, uint32_t valid, int bid) {
    WideItem wi;
    const int R = __popc(valid);
    wi.ok = false;
    const int items = a.H_q * ((a.L_c + kWideRows - 1) / kWideRows);
    const int S = p.splits[R - 1];
    const FcWideShape w = fc_wide_shape(R, items, S);
    const int xcd = bid & 7, slot = bid >> 3;
    if (S > 1 && w.full == 0) {
        if (BY_CHUNK) {
            const int n = items * S, per = (n + 7) / 8, rank = slot / per, e = xcd * per + slot % per;
            if (rank >= R || e >= n) return wi;
            wi = wide_unit(a, valid, items, rank, e % items);
            wi.s = e / items; wi.S = S; wi.unit = (int64_t)rank * items + e % items;
            return wi;
        }
        // all units split: range-major, so that the row tiles of a head that read one range are neighbours
        const int U = R * items, n = U * S, per = (n + 7) / 8;
        const int e = xcd * per + slot;
        if (slot >= per || e >= n) return wi;
        const int u = e % U;
        wi = wide_unit(a, valid, items, u / items, u % items);
        wi.s = e / U; wi.S = S; wi.unit = u;
        return wi;
    }
    int j = slot;
    if (slot >= w.full) {
        const int b = slot - w.full;
        if (S == 1 || b >= w.rem * S) return wi;
        j = w.full + b % w.rem;
        wi = wide_unit(a, valid, items, j / w.per, xcd * w.per + j % w.per);
        wi.s = b / w.rem; wi.S = S; wi.unit = xcd * w.rem + b % w.rem;
        return wi;
    }
    wi = wide_unit(a, valid, items, j / w.per, xcd * w.per + j % w.per);
    wi.s = 0; wi.S = 1; wi.unit = 0;
    return wi;
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

typedef short s16x4_t __attribute__((ext_vector_type(4)));

// Transposing LDS load: within each group of 16 lanes, lane s passes the address of 4
// consecutive bf16; lane i receives element (i % 4) of the data addressed by lanes
// i/4, i/4 + 4, i/4 + 8, i/4 + 12.
__device__ __forceinline__ s16x4_t lds_read_tr(const bf16_t* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (s16x4_t __attribute__((address_space(3)))*)(p));
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
__device__ __forceinline__ void finish_unit(const FcAttendArgs& a, const FcAttendPlan& p, const SplitItem& it,
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
__global__ __launch_bounds__(256) void attend_merge_kernel(FcAttendArgs a, FcAttendPlan p, const float* parts) {
    constexpr int PER = D / 8;
    const uint32_t valid = valid_blocks(a);
    const int R = __popc(valid);
    if (R == 0) return;
    const int S = p.splits[R - 1];
    if (S == 1) return;
    const int unit = blockIdx.x;
    int tile, r, h;
    if (p.narrow[R - 1]) {
        if (unit >= R * a.H_q * p.tiles) return;
        tile = unit % p.tiles;
        r = block_of_rank(valid, (unit / p.tiles) % R);
        h = unit / (p.tiles * R);
    } else {
        constexpr int SUB = kWideRows / kUnitRows;
        const int items = a.H_q * ((a.L_c + kWideRows - 1) / kWideRows);
        const FcWideShape w = fc_wide_shape(R, items, S);
        const int u = unit / SUB;
        WideItem wi;
        if (w.full == 0) {
            if (u >= R * items) return;
            wi = wide_unit(a, valid, items, u / items, u % items);
        } else {
            if (u >= 8 * w.rem) return;
            const int j = w.full + u % w.rem;
            wi = wide_unit(a, valid, items, j / w.per, (u / w.rem) * w.per + j % w.per);
        }
        if (!wi.ok) return;
        tile = wi.tile * SUB + unit % SUB;
        r = wi.r;
        h = wi.h;
    }
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
