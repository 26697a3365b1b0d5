// First digit of the top-B selection: where its bins lie.
//
// A key is the order-preserving 64-bit image of a score.  Some keys of the head are sampled, and those
// some ranks above and below the wanted one bound a bracket; one bin holds everything below it and one
// everything above.  Inside, the bins have equal widths in the key (510 of them) where that spreads the
// sampled keys.  It does not where zero lies inside: a key is nearly the logarithm of its score, all
// exponents lie between the bounds, and a fifth to a half of the head falls into one bin (24 heads of 39904
// keys, importance weighted 0.3: selection call 143 us).  There, and wherever five neighbouring sampled keys
// share a bin, the bins follow the sample: 8 of equal width between each two neighbours (118 us).  Such a
// digit takes a search, 4 us more in score_keys of 12 heads of 51000 keys, so it is not taken always.
// Either way a bin holds about a thousandth of the head, seldom more than six 128ths.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

constexpr int kSample = 128;      // sampled keys per head
constexpr int kSampleWide = 28;   // the bracket's half width in ranks of the sample: five deviations
constexpr int kEdges = 64;        // room for the bracket's sampled keys (57 at most), the rest all ones
constexpr int kSubBits = 3;
// every block of a head adds to the bins in global memory: more of them cost score_keys what they save
// the select (24 heads of 74880 keys, the two together with 256, 512 and 2048 bins: 42, 43 and 44 us)
constexpr int kFirstBits = 9;
constexpr int kFirstBins = 1 << kFirstBits;

// Ranks (from the top) of the sampled keys that bound the bracket; the intervals between them are the
// ranks' difference, 28 to 56.
struct FcBracket { int top, bottom; };
__host__ __device__ inline FcBracket fc_bracket(int budget, int L) {
    const int want = (int)((int64_t)budget * kSample / L);
    FcBracket b;
    b.top = want > kSampleWide ? want - kSampleWide : 0;
    b.bottom = want + kSampleWide < kSample - 1 ? want + kSampleWide : kSample - 1;
    return b;
}

// In what follows edge[0 .. n] are the bracket's sampled keys, ascending.

// Equal widths: the shift that makes 256 to 510 bins of the bracket
__host__ __device__ inline int fc_even_shift(const uint64_t* edge, int n) {
    const uint64_t w = edge[n] - edge[0];
    const int bits = w ? 64 - __builtin_clzll(w) : 0;
    int sh = bits > kFirstBits - 1 ? bits - (kFirstBits - 1) : 0;
    if (sh > 0 && (w >> (sh - 1)) <= (uint64_t)(kFirstBins - 3)) --sh;
    return sh;
}
// Do five sampled keys, i to i + 4, share a bin of that width?  Then equal widths are not taken.  (Of 57 evenly
// spread ones five do in one head of a thousand, three in every third.)
__host__ __device__ inline bool fc_crowded(const uint64_t* edge, int n, int sh, int i) {
    return i + 4 <= n && (edge[i] - edge[0]) >> sh == (edge[i + 4] - edge[0]) >> sh;
}

// Bins that follow the sample: interval i is [edge[i], edge[i + 1]), the last one with its upper end; the width
// of its bins as a shift
__host__ __device__ inline int fc_sub_shift(uint64_t width) {
    const int bits = width ? 64 - __builtin_clzll(width) : 0;
    return bits > kSubBits ? bits - kSubBits : 0;
}

// even_sh: the shift of equal widths, or -1
__host__ __device__ inline uint32_t fc_first_digit(uint64_t k, const uint64_t* edge, int n, int even_sh) {
    uint32_t in;
    if (even_sh >= 0) {
        in = 1u + (uint32_t)((k - edge[0]) >> even_sh);
    } else {
        int i = 0;
#pragma unroll
        for (int step = kEdges / 2; step > 0; step >>= 1) i += edge[i + step] <= k ? step : 0;
        i = i < n ? i : n - 1;
        in = 1u + ((uint32_t)i << kSubBits) + (uint32_t)((k - edge[i]) >> fc_sub_shift(edge[i + 1] - edge[i]));
    }
    return k < edge[0] ? 0u : (k > edge[n] ? (uint32_t)(kFirstBins - 1) : in);
}

// The keys of a bin that is not empty: those with k - base <= limit.
__host__ __device__ inline void fc_bin_keys(uint32_t bin, const uint64_t* edge, int n, int even_sh, uint64_t* base,
                                            uint64_t* limit) {
    if (bin == 0u) {
        *base = 0ull;
        *limit = edge[0] - 1ull;
    } else if (bin == (uint32_t)(kFirstBins - 1)) {
        *base = edge[n] + 1ull;
        *limit = ~0ull - *base;
    } else {
        uint64_t lo = edge[0], end = edge[n];
        uint32_t sub = bin - 1u;
        int sh = even_sh;
        if (sh < 0) {
            const int i = (int)(sub >> kSubBits);
            lo = edge[i];
            end = i + 1 < n ? edge[i + 1] - 1ull : edge[n];
            sub &= (1u << kSubBits) - 1u;
            sh = fc_sub_shift(edge[i + 1] - lo);
        }
        *base = lo + ((uint64_t)sub << sh);
        const uint64_t width = (1ull << sh) - 1ull;
        *limit = end - *base < width ? end - *base : width;
    }
}
