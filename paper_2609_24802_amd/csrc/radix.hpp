// Stable LSD radix sort of int32 keys that carries the input position of every key: the CSR transpose,
// the radius cell directory and the kNN curve order.
//
// A pass is a histogram per tile and a scatter; digits are equally wide over the passes.  Small inputs
// spend their time on launches and dependent latencies, not on bytes, hence:
//   - up to kDirectTiles tiles the scatter sums the preceding tiles' counts itself (a 1,024-digit row
//     per tile, coalesced, all loads in flight) instead of waiting for scan launches; larger inputs
//     take one scan launch per pass;
//   - digits of up to kMaxBits bits up to kWideKeys keys (2 passes for the cells of 1M points instead
//     of 3); above that 8 bits, whose longer runs of equal digits suit the memory-bound scatter;
//   - the first histogram is taken where the keys are formed (key_tile), the last scatter can write
//     the caller's records (Out::rec).
// Scatter: a wavefront owns a contiguous piece of the tile and ranks it round by round with ballots and
// its own LDS counters (no block barrier between rounds), so ranks follow the input order; one scan over
// the digits places the tile in LDS grouped by digit, and runs leave with consecutive lanes on
// consecutive addresses.  Measured, cell directory of 131,072 points (18 bits): 3 passes of
// histogram + 3-launch scan + scatter took 75 us, 2 passes of histogram + scatter
// 27 us (the first histogram inside the key kernel); 1M points (20 bits): 105 and 60 us.
#pragma once

#include "common.hpp"

namespace tiga {
namespace radix {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / kWave;
constexpr int kMaxBits = 10;
constexpr int kMaxDigits = 1 << kMaxBits;
constexpr int64_t kDirectTiles = 64;
constexpr int64_t kWideKeys = int64_t{1} << 21;

// Shape of a sort: `items` keys per thread (tiles of items * kThreads keys), `passes` of `rb` bits.
struct Shape {
    int64_t n, tiles;
    int items, passes, rb;
    bool direct;
};

inline Shape shape_for(int64_t n, int64_t key_limit) {
    Shape s;
    s.n = n;
    int bits = 1;
    while (bits < 31 && (int64_t{1} << bits) < key_limit) ++bits;
    const int most = n <= kWideKeys ? kMaxBits : 8;
    s.passes = (bits + most - 1) / most;
    s.rb = (bits + s.passes - 1) / s.passes;
    // the smallest tile that keeps the direct form: more blocks in flight
    s.items = 2;
    while (s.items < 8 && n > kDirectTiles * s.items * kThreads) s.items *= 2;
    s.tiles = ceil_div(n > 0 ? n : 1, s.items * kThreads);
    s.direct = s.tiles <= kDirectTiles;
    return s;
}

struct Ws {
    int32_t *k[2], *a[2];
    uint32_t *counts;   // [tiles][digits] keys per tile and digit (after the scan launch: in earlier tiles)
    uint32_t *totals;   // [digits], scan launch only
};

inline Ws carve(Carve &c, int64_t n) {
    Ws w;
    for (int i = 0; i < 2; ++i) {
        w.k[i] = c.take<int32_t>(n);
        w.a[i] = c.take<int32_t>(n);
    }
    // tiles * digits: at most kDirectTiles + n / tile rows of kMaxDigits, or of 256 above kWideKeys, where it is
    // kept at no less than at kWideKeys, so that a workspace for n keys holds every smaller sort
    constexpr int64_t tile = 8 * kThreads;
    const int64_t big = ceil_div(n > 0 ? n : 1, tile);
    const int64_t rows = big > kDirectTiles ? big : kDirectTiles;
    const int64_t wide = kWideKeys / tile * kMaxDigits;
    w.counts = c.take<uint32_t>(n <= kWideKeys ? rows * kMaxDigits : (rows * 256 > wide ? rows * 256 : wide));
    w.totals = c.take<uint32_t>(kMaxDigits);
    return w;
}

// Results: sorted keys (null: not kept), the input position of each (null: not kept), and with `rec`
// cell-ordered records (x, y, z of pos, all +inf if one of them is not finite; input position as bits).
struct Out {
    int32_t *keys = nullptr;
    int32_t *idx = nullptr;
    const float *pos = nullptr;
    float4 *rec = nullptr;
};

// Histogram of the first digit for keys formed by the caller: kernels launched with s.tiles blocks of
// kThreads threads call this with key(i) for every index of their tile; keys go to `keys`.
template <int ITEMS, class Key>
__device__ __forceinline__ void key_tile(int64_t n, int rb, int32_t *__restrict__ keys,
                                         uint32_t *__restrict__ counts, uint32_t (&hist)[kMaxDigits], Key &&key) {
    const int D = 1 << rb;
    for (int d = threadIdx.x; d < D; d += kThreads) hist[d] = 0;
    __syncthreads();
    const int64_t base = static_cast<int64_t>(blockIdx.x) * (ITEMS * kThreads);
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int64_t i = base + r * kThreads + threadIdx.x;
        if (i < n) {
            const int32_t k = key(i);
            if (keys) keys[i] = k;
            atomicAdd(&hist[static_cast<uint32_t>(k) & (D - 1)], 1u);
        }
    }
    __syncthreads();
    for (int d = threadIdx.x; d < D; d += kThreads) counts[static_cast<int64_t>(blockIdx.x) * D + d] = hist[d];
}

// Histogram of the first digit of existing keys.
int launch_first_hist(const Shape &s, const int32_t *keys, const Ws &w, hipStream_t stream);

// Sort after the first histogram (launch_first_hist, or key_tile in a kernel of the caller's).
// `sorted` (optional) receives where the sorted keys are: out.keys, or the workspace.
int launch_sort(const Shape &s, const int32_t *keys, const Ws &w, const Out &out, const int32_t **sorted,
                hipStream_t stream);

// ptr[j] = first sorted position with key >= j, for j in [0, nkeys].
__device__ __forceinline__ int64_t lower_bound(const int32_t *__restrict__ sorted, int64_t n, int64_t j) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (static_cast<int64_t>(sorted[mid]) < j) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

}  // namespace radix
}  // namespace tiga
