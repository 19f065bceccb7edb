// Generated exact kNN relation with a fused neighbour sum (Section 4.9, generated relations: one
// program scans candidate tiles for its queries, keeps a power-of-two padded top-k state keyed by
// (squared distance, source index), and consumes the selected sources without storing adjacency;
// the exact-kNN workload of Section 7 is a neighbour sum with k = 16).
//   S_i = the k sources j != i with the smallest keys (d2_ij, j), d2 finite,
//   d2  = fl(fl(fl(dx*dx) + fl(dy*dy)) + fl(dz*dz)), dx = fl(p_j.x - p_i.x), ...
//   y_i = sum_{j in S_i} x_j
//
// MI355X design:
//  - A key is one 64-bit integer, (bits of d2) << 32 | index: d2 >= 0, so the float bits order like the
//    values, and one unsigned compare gives the lexicographic order with the index as the tie-break.
//    Keys of non-finite distances are >= the bits of +inf and are never selected.
//  - Build: points are ordered along a 30-bit Morton curve (radix sort) into records (x, y, z, original
//    index).  The curve's scale is chosen so that one of its levels is a grid of cubic cells holding
//    about cell_points(k) points each in a uniform cloud; a cell is one run of the records.
//  - Select (cell_select_kernel): a wavefront takes 8 consecutive queries; the candidates of a query are
//    the points of the 3 x 3 x 3 cells around its own, held in registers and shared by the queries of
//    the cell.  Every point closer than the block's nearest open face is among them, so a query with at
//    least k candidates inside that distance is decided: those candidates (38 of 246 on average for
//    k = 16) are compacted and ranked by counting.  Where a block holds more than 512 points the next finer
//    level of the curve is taken (the box is cut four standard deviations from the mean, so that far points
//    do not use up the levels).  Otherwise the query is listed, and a second launch
//    scans its 5 x 5 x 5 cells, then those of coarser levels, one wavefront per listed query (they sit
//    together at the cloud's faces, so a wavefront with eight of them would end long after the rest); a
//    block of more than 1,536 points is streamed through a list with one key per lane in a third launch.
//    131,072 points with a third of them in a clump of 0.002: 2,183 us with the tiles, 976 us now; a normal
//    cloud 499 and 462 us; one far outlier 9,286 and 1,161 us.
//  Measured, 131,072 uniform points, k = 16: the previous select (tiles of 64 queries, one per lane with its
//  keys sorted in registers, whose insertion ran for the whole wavefront whenever one lane accepted) took
//  366 us, the cell select takes 75 us and the second launch 15 us (k = 32, whole call: 1,424 us before,
//  174 us now).  The cell select is bound by VALU issue: about 8 tests per selected neighbour and 2
//  instructions per pair of compacted candidates.
#include "knn.hpp"

#include <cmath>

#include "common.hpp"
#include "radix.hpp"

namespace tiga {
namespace knn {

namespace {

constexpr int kBlock = 256;
constexpr int kBits = 10;                                 // Morton bits per axis
constexpr uint64_t kNone = 0x7f80000000000000ull;         // key (+inf, 0): above every finite key
constexpr int kPartials = 256;                            // read by every block of the key kernel

typedef float f4 __attribute__((ext_vector_type(4)));

// The curve: fine coordinate along axis a = floor((p - lo) * inv_f), clamped to [0, 2^kBits - 1].  The
// cells of level l are 2^(kBits - l) fine units wide, so a cell's id is the key without its low
// 3 (kBits - l) bits; the cells of level `base` have a table of their first records.
struct Curve {
    double lo[3];
    double inv_f;
    int base;
    int last[3];   // highest fine coordinate that holds a finite point
};

constexpr int kQueries = 8;       // queries per wavefront of the cell select
constexpr int kNear = 512;        // candidates of the 27 cells, held in registers (8 per lane)
constexpr int kFar = 1536;        // candidates of the 125 cells (24 per lane)
constexpr int kMaxK = 32;

// Undecided queries for the wider scan: kSegs lists (block b appends to list b % kSegs, so that the
// appends do not all wait for one counter), each as long as its blocks' queries.
constexpr int kSegs = 8;
struct alignas(256) SegCount {
    uint32_t v;
};
__host__ __device__ inline int64_t seg_size(int64_t n) {
    const int64_t blocks = (n + kQueries * (kBlock / kWave) - 1) / (kQueries * (kBlock / kWave));
    return (blocks + kSegs - 1) / kSegs * (kQueries * (kBlock / kWave));
}

struct Ws {
    float *part;        // [kPartials][6] box partials
    double *moments;    // [kPartials][6] sums of the finite coordinates and of their squares
    Curve *curve;
    int32_t *key, *key_sorted;
    radix::Ws sort;
    int32_t *start;     // [max_cells + 1] first record of each cell
    SegCount *seg_count;   // [2 kSegs] queries listed for the wider scan, then for the streaming scan
    int2 *seg, *far;    // [kSegs][seg_size(n)] their records and levels
    f4 *rec;            // [n] Morton-ordered (x, y, z, original index)
};

// The finest grid: the largest level with 8^level cells <= 4 n + 64.
int max_level(int64_t n) {
    int l = 0;
    while (l < kBits && (int64_t{8} << (3 * l)) <= 4 * n + 64) ++l;
    return l;
}

Ws carve(Carve &c, int64_t n) {
    Ws w;
    w.part = c.take<float>(kPartials * 6);
    w.moments = c.take<double>(kPartials * 6);
    w.curve = c.take<Curve>(1);
    w.key = c.take<int32_t>(n);
    w.key_sorted = c.take<int32_t>(n);
    w.sort = radix::carve(c, n);
    w.start = c.take<int32_t>((int64_t{1} << (3 * max_level(n))) + 1);
    w.seg_count = c.take<SegCount>(2 * kSegs);
    w.seg = c.take<int2>(kSegs * seg_size(n));
    w.far = c.take<int2>(kSegs * seg_size(n));
    w.rec = c.take<f4>(n);
    return w;
}

__device__ __forceinline__ bool finite3(float a, float b, float c) {
    return __builtin_isfinite(a) && __builtin_isfinite(b) && __builtin_isfinite(c);
}

__device__ __forceinline__ float wave_min(float v) {
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) v = fminf(v, __shfl_xor(v, m, kWave));
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) v = fmaxf(v, __shfl_xor(v, m, kWave));
    return v;
}

// ---- build

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) v += __shfl_xor(v, m, kWave);
    return v;
}

// Box and moments of the finite points: per-block partials (min xyz, max xyz; sums, sums of squares).
__global__ __launch_bounds__(kBlock) void box_partial_kernel(const float *__restrict__ pos, int64_t n,
                                                             float *__restrict__ part,
                                                             double *__restrict__ moments) {
    __shared__ float red[kBlock / kWave][6];
    __shared__ double sums[kBlock / kWave][6];
    float v[6] = {__builtin_inff(), __builtin_inff(), __builtin_inff(),
                  -__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
    double s[6] = {};
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < n; i += stride) {
        const float p[3] = {pos[i * 3], pos[i * 3 + 1], pos[i * 3 + 2]};
        if (!finite3(p[0], p[1], p[2])) continue;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            v[a] = fminf(v[a], p[a]);
            v[3 + a] = fmaxf(v[3 + a], p[a]);
            s[a] += p[a];
            s[3 + a] += static_cast<double>(p[a]) * p[a];
        }
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        v[a] = a < 3 ? wave_min(v[a]) : wave_max(v[a]);
        s[a] = wave_sum(s[a]);
    }
    const int w = threadIdx.x / kWave;
    if (lane_id() == 0)
        for (int a = 0; a < 6; ++a) {
            red[w][a] = v[a];
            sums[w][a] = s[a];
        }
    __syncthreads();
    if (threadIdx.x < 6) {
        float r = red[0][threadIdx.x];
        double t = sums[0][threadIdx.x];
        for (int q = 1; q < kBlock / kWave; ++q) {
            r = threadIdx.x < 3 ? fminf(r, red[q][threadIdx.x]) : fmaxf(r, red[q][threadIdx.x]);
            t += sums[q][threadIdx.x];
        }
        part[blockIdx.x * 6 + threadIdx.x] = r;
        moments[blockIdx.x * 6 + threadIdx.x] = t;
    }
}

__device__ __forceinline__ uint32_t spread3(uint32_t v) {
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__device__ __forceinline__ uint32_t morton(uint32_t x, uint32_t y, uint32_t z) {
    return spread3(x) | (spread3(y) << 1) | (spread3(z) << 2);
}

// The inverse of spread3: every third bit, from bit 0.
__device__ __forceinline__ uint32_t gather3(uint32_t v) {
    v &= 0x09249249u;
    v = (v | (v >> 2)) & 0x030c30c3u;
    v = (v | (v >> 4)) & 0x0300f00fu;
    v = (v | (v >> 8)) & 0x030000ffu;
    v = (v | (v >> 16)) & 0x3ffu;
    return v;
}

__device__ __forceinline__ uint32_t fine_axis(const Curve &c, int a, float v) {
    double t = (static_cast<double>(v) - c.lo[a]) * c.inv_f;
    const double top = static_cast<double>((1 << kBits) - 1);
    t = t >= 0.0 ? t : 0.0;
    return static_cast<uint32_t>(t < top ? t : top);
}

// Cell size for the box: `points` points per cell if the cloud were uniform, coarser where the table
// (base <= top) or the curve's scale (the longest axis) asks for it.  The box is cut four standard
// deviations from the mean: a few far points must not take the resolution from all others (points
// outside the cut share its border cells).
__device__ __forceinline__ Curve make_curve(const float (&lo)[3], const float (&hi)[3], const double (&mom)[6],
                                            int64_t n, double points, int top) {
    Curve c;
    double ext[3], vol = 1.0, longest = 0.0;
    for (int a = 0; a < 3; ++a) {
        double l = lo[a], u = hi[a];
        const double mean = mom[a] / static_cast<double>(n);
        const double var = mom[3 + a] / static_cast<double>(n) - mean * mean;
        if (var > 0.0) {
            const double cut = 4.0 * sqrt(var);
            if (mean - cut > l) l = mean - cut;
            if (mean + cut < u) u = mean + cut;
        }
        c.lo[a] = l;
        ext[a] = u - l;
        if (!(ext[a] > 0.0)) ext[a] = 0.0;   // no extent, or no finite point at all
        vol *= ext[a];
        longest = fmax(longest, ext[a]);
    }
    double h = cbrt(vol * points / static_cast<double>(n));
    const double finest = longest / static_cast<double>(1 << top);
    if (!(h > finest)) h = finest;
    if (!(h > 0.0)) h = 1.0;                 // coincident points
    int level = 0;
    while (level < top && longest >= h * static_cast<double>(1 << level)) ++level;
    c.base = level;
    c.inv_f = static_cast<double>(1 << (kBits - level)) / h;
    for (int a = 0; a < 3; ++a) c.last[a] = static_cast<int>(fine_axis(c, a, hi[a]));
    return c;
}

// Morton key of every point (non-finite points: the last key) and the sort's first histogram.  Every
// block reduces the box partials and forms the curve for itself; block 0 stores it.
template <int ITEMS>
__global__ __launch_bounds__(radix::kThreads) void key_kernel(const float *__restrict__ pos, int64_t n,
                                                              const float *__restrict__ part,
                                                              const double *__restrict__ moments, int nparts,
                                                              double points, int top, int rb,
                                                              Curve *__restrict__ curve, int32_t *__restrict__ key,
                                                              uint32_t *__restrict__ counts) {
    __shared__ uint32_t hist[radix::kMaxDigits];
    __shared__ float red[radix::kWaves][6];
    __shared__ double sums[radix::kWaves][6];
    __shared__ Curve sc;
    float v[6] = {__builtin_inff(), __builtin_inff(), __builtin_inff(),
                  -__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
    double m[6] = {};
    for (int p = threadIdx.x; p < nparts; p += radix::kThreads)
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            v[a] = a < 3 ? fminf(v[a], part[p * 6 + a]) : fmaxf(v[a], part[p * 6 + a]);
            m[a] += moments[p * 6 + a];
        }
    if (threadIdx.x < kPartials) {   // whole wavefronts
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            v[a] = a < 3 ? wave_min(v[a]) : wave_max(v[a]);
            m[a] = wave_sum(m[a]);
        }
        if (lane_id() == 0)
            for (int a = 0; a < 6; ++a) {
                red[threadIdx.x / kWave][a] = v[a];
                sums[threadIdx.x / kWave][a] = m[a];
            }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kPartials / kWave; ++w)
            for (int a = 0; a < 6; ++a) {
                v[a] = a < 3 ? fminf(v[a], red[w][a]) : fmaxf(v[a], red[w][a]);
                m[a] += sums[w][a];
            }
        const float lo[3] = {v[0], v[1], v[2]}, hi[3] = {v[3], v[4], v[5]};
        sc = make_curve(lo, hi, m, n, points, top);
        if (blockIdx.x == 0) *curve = sc;
    }
    __syncthreads();
    const Curve c = sc;
    radix::key_tile<ITEMS>(n, rb, key, counts, hist, [&](int64_t i) {
        const float px = pos[i * 3], py = pos[i * 3 + 1], pz = pos[i * 3 + 2];
        if (!finite3(px, py, pz)) return (1 << (3 * kBits)) - 1;
        return static_cast<int32_t>(morton(fine_axis(c, 0, px), fine_axis(c, 1, py), fine_axis(c, 2, pz)));
    });
}

// The table cells' first records (binary search over the sorted keys); also clears the list counters.
__global__ __launch_bounds__(kBlock) void cells_kernel(const Curve *__restrict__ curve,
                                                       const int32_t *__restrict__ sorted, int64_t n,
                                                       int32_t *__restrict__ start, SegCount *__restrict__ seg_count) {
    if (blockIdx.x == 0 && threadIdx.x < 2 * kSegs) seg_count[threadIdx.x].v = 0;
    const int64_t cells = int64_t{1} << (3 * curve->base);
    const int shift = 3 * (kBits - curve->base);
    for (int64_t c = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; c <= cells;
         c += static_cast<int64_t>(gridDim.x) * kBlock)
        start[c] = static_cast<int32_t>(radix::lower_bound(sorted, n, c << shift));
}

// ---- select and consume

__device__ __forceinline__ float sqdist(f4 pi, f4 pj) {
#pragma clang fp contract(off)
    const float dx = pj.x - pi.x, dy = pj.y - pi.y, dz = pj.z - pi.z;
    const float sx = dx * dx, sy = dy * dy, sz = dz * dz;
    const float s = sx + sy;
    return s + sz;
}

// ---- cell select

// 64-bit lane shift: lane t receives lane t - 1's value (lane 0 its own).
__device__ __forceinline__ uint64_t shift_up(uint64_t v) {
    const int src = lane_id() > 0 ? lane_id() - 1 : 0;
    const uint32_t lo = __builtin_amdgcn_ds_bpermute(src * 4, static_cast<int>(static_cast<uint32_t>(v)));
    const uint32_t hi = __builtin_amdgcn_ds_bpermute(src * 4, static_cast<int>(static_cast<uint32_t>(v >> 32)));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ uint64_t readlane64(uint64_t v, int l) {
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(v)), l);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(v >> 32)), l);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ float readlane_f(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// Insert the keys of `mask`'s lanes below `thr` into the ascending list L (one key per lane, lanes
// 0..kp-1) one at a time: each list lane takes its left neighbour's key or the new one.  `thr` is the
// list's last key.
__device__ __forceinline__ void insert_lanes(uint64_t mask, uint64_t key, int kp, uint64_t &L, uint64_t &thr) {
    const int lane = lane_id();
    while (mask) {
        const int b = __builtin_ctzll(mask);
        mask &= mask - 1;
        const uint64_t nk = readlane64(key, b);
        if (nk >= thr) continue;   // the list moved below it meanwhile
        const uint64_t left = shift_up(L);
        const uint64_t up = lane == 0 ? nk : (nk < left ? left : nk);
        L = lane < kp ? (nk < L ? up : L) : L;
        thr = readlane64(L, kp - 1);
    }
}

// Working set of one query: compacted candidates (distance bits, padded for 4-wide reads, and index) and
// the selected indices in key order (-1 past the end; one slot past k shows ties at the k-th key).
struct alignas(16) Pick {
    uint32_t d2[kWave + 4];
    int32_t id[kWave];
};
constexpr int kSelRow = kMaxK + 1;

__device__ __forceinline__ void lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The cell of level `level` with id m: its first record, and its number of records.
__device__ __forceinline__ void cell_range(const Curve &c, const int32_t *__restrict__ start,
                                           const int32_t *__restrict__ sorted, int level, uint32_t m, int &s,
                                           int &len) {
    if (level <= c.base) {   // a run of table cells
        const int up = 3 * (c.base - level);
        s = start[m << up];
        len = start[(m + 1) << up] - s;
    } else {                 // part of one table cell
        const uint32_t in = m >> (3 * (level - c.base));
        const int b = start[in], n = start[in + 1] - b, shift = 3 * (kBits - level);
        const int64_t f = radix::lower_bound(sorted + b, n, static_cast<int64_t>(m) << shift);
        s = b + static_cast<int>(f);
        len = static_cast<int>(radix::lower_bound(sorted + s, n - f, static_cast<int64_t>(m + 1) << shift));
    }
}

// Append the candidates of the cells i0 .. i0 + 63 (this lane: i0 + lane) of the (2R + 1)^3 block of
// level-`level` cells around cell m0 to the table of records `tab`, which holds `have` of at most `cap`;
// returns the new number, or -1 if they exceed `cap` (the table is then unfinished).
template <int R>
__device__ __forceinline__ int gather_cells(const Curve &c, const int32_t *__restrict__ start,
                                            const int32_t *__restrict__ sorted, int level, uint32_t m0, int i0,
                                            int have, int cap, int32_t *__restrict__ tab) {
    constexpr int W = 2 * R + 1;
    const int i = i0 + lane_id(), top = 1 << level;
    const int x = static_cast<int>(gather3(m0)) - R + i % W, y = static_cast<int>(gather3(m0 >> 1)) - R + (i / W) % W,
              z = static_cast<int>(gather3(m0 >> 2)) - R + i / (W * W);
    int s = 0, len = 0;
    if (i < W * W * W && x >= 0 && y >= 0 && z >= 0 && x < top && y < top && z < top)
        cell_range(c, start, sorted, level, morton(x, y, z), s, len);
    const int l = len < cap + 1 ? len : cap + 1;   // 64 of them cannot overflow the sum
    const int incl = wave_incl_scan(l);
    const int total = have + __builtin_amdgcn_readlane(incl, kWave - 1);
    if (total > cap) return -1;
    const int at = have + incl - l;
    for (int j = 0; __any(j < len); ++j)
        if (j < len) tab[at + j] = s + j;
    lds_fence();
    return total;
}

// Squared distance within which every point lies in the (2R + 1)^3 block of level-`level` cells around
// the cell of key `key`: the nearest face beyond which cells hold points, less a relative 2e-6 that covers
// the roundings of d2 (5 of 2^-24), and those of the fine coordinate and of this distance (2^-52 of the
// coordinate, which is at most 2^kBits times a distance of a cell or more).  FLT_MAX without such a face
// (then the block holds every finite point); -1 where the square could underflow.
__device__ __forceinline__ float block_reach2(const Curve &c, f4 at, int key, int level, int R) {
    const float p[3] = {at.x, at.y, at.z};
    const int sub = kBits - level;
    const uint32_t m = static_cast<uint32_t>(key) >> (3 * sub);
    const int cell[3] = {static_cast<int>(gather3(m)), static_cast<int>(gather3(m >> 1)),
                         static_cast<int>(gather3(m >> 2))};
    const double h = static_cast<double>(1 << sub) / c.inv_f;
    double g = __builtin_inf();
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double d = static_cast<double>(p[a]) - c.lo[a];
        if (cell[a] - R > 0) g = fmin(g, d - h * (cell[a] - R));
        if (cell[a] + R < (c.last[a] >> sub)) g = fmin(g, h * (cell[a] + R + 1) - d);
    }
    if (g == __builtin_inf()) return __FLT_MAX__;
    const double r2 = g > 0.0 ? g * g * (1.0 - 4e-6) : 0.0;
    return r2 < 1e-30 ? -1.0f : (r2 < static_cast<double>(__FLT_MAX__) ? static_cast<float>(r2) : __FLT_MAX__);
}

// Select the k smallest keys of one query from the candidates (d2[b], id[b]) of the lanes (no candidate:
// +inf) when they are decided by those within `reach` (FLT_MAX: always), and write their indices in key
// order to sel.  False: undecided.
template <int B>
__device__ __forceinline__ bool pick_query(Pick &pk, const float (&d2)[B], const int (&id)[B], float reach, int k,
                                           int32_t *__restrict__ sel) {
    const int lane = lane_id();
    auto within = [&](float r) __attribute__((always_inline)) {
        int m = 0;
#pragma unroll
        for (int b = 0; b < B; ++b) m += __popcll(__builtin_amdgcn_ballot_w64(d2[b] <= r));
        return m;
    };
    int m = within(reach);
    // fewer than k of them while points outside the block may be as close
    if (m < k && reach != __FLT_MAX__) return false;
    // more than a wavefront of them: shrink the bound (bisection of its bits) to one that still holds k
    if (m > kWave) {
        uint32_t hi = __float_as_uint(reach), lo = hi > (3u << 23) ? hi - (3u << 23) : 0;
        if (within(__uint_as_float(lo)) >= k) lo = 0;
        while (m > kWave && hi - lo > 1) {
            const uint32_t mid = lo + (hi - lo) / 2;
            const int mm = within(__uint_as_float(mid));
            if (mm >= k) hi = mid, m = mm;
            else lo = mid;
        }
        if (m > kWave) return false;   // that many equal distances
        reach = __uint_as_float(hi);
    }
    int base = 0;
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const bool in = d2[b] <= reach;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(in);
        if (in) {
            const int at = base + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                                            __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0));
            pk.d2[at] = __float_as_uint(d2[b]);
            pk.id[at] = id[b];
        }
        base += __popcll(mask);
    }
    if (lane < 4) pk.d2[m + lane] = ~0u;
    lds_fence();
    const uint32_t mine = lane < m ? pk.d2[lane] : ~0u;
    const int my_id = lane < m ? pk.id[lane] : 0;
    // rank = keys below this lane's; equal distances leave a slot of the first k + 1 unwritten
    int rank = 0;
#pragma unroll 2
    for (int j = 0; j < m; j += 4) {
        const i32x4 o = *reinterpret_cast<const i32x4 *>(&pk.d2[j]);
#pragma unroll
        for (int u = 0; u < 4; ++u) rank += static_cast<uint32_t>(o[u]) < mine;
    }
    if (lane < m && rank <= k) sel[rank] = my_id;
    lds_fence();
    const int slots = m < k + 1 ? m : k + 1;
    if (__any(lane < slots && sel[lane] < 0)) {
        for (int j = 0; j < m; ++j) rank += pk.d2[j] == mine && pk.id[j] < my_id;
        if (lane < m && rank <= k) sel[rank] = my_id;
        lds_fence();
    }
    return true;
}

// The queries q .. qe - 1 of one cell (lane q of `me`: the query's record, of `reach1`: how far the cells
// around it reach), whose `total` candidates are in `tab`, B 64-candidate steps held in registers.
// Returns the queries that stay undecided.  One instance per B: with a condition per step instead, the
// values merged at each of them took 364 registers.
template <int B>
__device__ __forceinline__ uint32_t pick_cell(Pick &pk, int32_t (*__restrict__ sel)[kSelRow],
                                              const f4 *__restrict__ rec, const int32_t *__restrict__ tab, int total,
                                              int k, int q, int qe, f4 me, uint64_t fin, float reach1) {
    const int lane = lane_id();
    f4 cand[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int j = b * kWave + lane;
        cand[b] = j < total ? rec[tab[j]] : f4{__builtin_inff(), __builtin_inff(), __builtin_inff(), 0.0f};
    }
    uint32_t left = 0;
    for (; q < qe; ++q) {
        if (lane < kSelRow) sel[q][lane] = -1;
        if (!((fin >> q) & 1)) continue;   // no finite distance: nothing is selected
        const f4 pq = f4{readlane_f(me.x, q), readlane_f(me.y, q), readlane_f(me.z, q), 0.0f};
        const int qid = __builtin_amdgcn_readlane(__float_as_int(me.w), q);
        float d2[B];
        int id[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const float v = sqdist(pq, cand[b]);
            id[b] = __float_as_int(cand[b].w);
            d2[b] = id[b] == qid ? __builtin_inff() : v;   // the query itself
        }
        if (!pick_query<B>(pk, d2, id, readlane_f(reach1, q), k, sel[q])) left |= 1u << q;
    }
    return left;
}

// Results of one query from its selected indices, by `lanes` lanes of which this is lane l.
__device__ __forceinline__ void put_query(const int32_t *__restrict__ sel, int64_t qid, int k, int feat, int l,
                                          int lanes, const float *__restrict__ x, float *__restrict__ y,
                                          int32_t *__restrict__ nbr) {
    if (nbr)
        for (int s = l; s < k; s += lanes) nbr[qid * k + s] = sel[s];
    for (int f = l; f < feat; f += lanes) {
        float acc = 0.0f;
#pragma unroll 8
        for (int s = 0; s < k; ++s) {
            const int32_t j = sel[s];
            if (j >= 0) acc += x[static_cast<int64_t>(j) * feat + f];
        }
        y[qid * feat + f] = acc;
    }
}

// Call item(list, entry index) for this wavefront's share (every nw-th, from w on) of the listed queries.
template <class F>
__device__ __forceinline__ void for_listed(const SegCount *__restrict__ count, int64_t w, int64_t nw, F &&item) {
    const uint32_t mine = lane_id() < kSegs ? count[lane_id()].v : 0u;   // all counters in one load
    int64_t before = 0;
    for (int s = 0; s < kSegs; ++s) {
        const int64_t c = static_cast<uint32_t>(__builtin_amdgcn_readlane(mine, s));
        if (c == 0) continue;
        for (int64_t i = (w - before % nw + nw) % nw; i < c; i += nw) item(s, i);
        before += c;
    }
}

// Wavefront w takes the records [8 w, 8 w + 8) as queries, cell by cell.
__global__ __launch_bounds__(kBlock, 6) void cell_select_kernel(const Curve *__restrict__ curve,
                                                                const int32_t *__restrict__ start,
                                                                const f4 *__restrict__ rec,
                                                                const int32_t *__restrict__ sorted, int64_t n, int k,
                                                                int feat, const float *__restrict__ x,
                                                                float *__restrict__ y, int32_t *__restrict__ nbr,
                                                                SegCount *__restrict__ seg_count,
                                                                int2 *__restrict__ seg,
                                                                SegCount *__restrict__ far_count,
                                                                int2 *__restrict__ far) {
    __shared__ Pick picks[kBlock / kWave];
    __shared__ int32_t tabs[kBlock / kWave][kNear];
    __shared__ int32_t sels[kBlock / kWave][kQueries][kSelRow];
    const int lane = lane_id(), wv = uniform(static_cast<int>(threadIdx.x) / kWave);
    Pick &pk = picks[wv];
    int32_t *tab = tabs[wv];
    const int64_t t = static_cast<int64_t>(xcd_block()) * (kBlock / kWave) + wv;
    const int64_t r0 = t * kQueries;
    if (r0 >= n) return;
    const int nq = static_cast<int>(n - r0 < kQueries ? n - r0 : kQueries);
    const Curve c = *curve;
    // lane q < nq: query q, its key, and how far the block of cells around it reaches
    const f4 me = rec[r0 + (lane < nq ? lane : 0)];
    const int key = lane < nq ? sorted[r0 + lane] : -1;
    const uint64_t fin = __builtin_amdgcn_ballot_w64(finite3(me.x, me.y, me.z));
    uint32_t wide = 0;       // undecided queries
    uint32_t over = 0;       // queries whose finest block holds more than kNear points
    int at_level = c.base;   // lane q: the level that left query q undecided
    for (int q = 0; q < nq;) {
        if (!((fin >> q) & 1)) {   // no finite distance: nothing is selected, whatever lies around
            if (lane < kSelRow) sels[wv][q][lane] = -1;
            ++q;
            continue;
        }
        // the table's level, or a finer one whose block is small enough (starting where the query's own
        // cell holds at most a quarter of it: lane l looks at l levels below the table's)
        int level = c.base, total = -1, qe = q;
        const uint32_t qkey = static_cast<uint32_t>(__builtin_amdgcn_readlane(key, q));
        while (true) {
            const int down = 3 * (kBits - level);
            const uint32_t cell = qkey >> down;
            // sorted: the queries of a cell are consecutive lanes
            const uint64_t same = __builtin_amdgcn_ballot_w64(lane < nq && static_cast<uint32_t>(key) >> down == cell);
            qe = kWave - __builtin_clzll(same);
            lds_fence();
            total = gather_cells<1>(c, start, sorted, level, cell, 0, 0, kNear, tab);
            if (total >= 0 || level == kBits) break;
            if (level++ == c.base) {
                const int l = c.base + lane;
                int b, len = kNear;
                if (lane > 0 && l <= kBits) cell_range(c, start, sorted, l, qkey >> (3 * (kBits - l)), b, len);
                const uint64_t small = __builtin_amdgcn_ballot_w64(len <= kNear / 4);
                level = small ? c.base + __builtin_ctzll(small) : kBits;
            }
        }
        uint32_t w = 0;
        if (total < 0) {
            over |= ((1u << qe) - 1) & ~((1u << q) - 1) & static_cast<uint32_t>(fin);
            for (int u = q; u < qe; ++u)
                if (lane < kSelRow) sels[wv][u][lane] = -1;
        } else {
            const float reach1 = block_reach2(c, me, key, level, 1);
            int32_t(*sel)[kSelRow] = sels[wv];
            switch ((total + kWave - 1) / kWave) {
                case 0:
                case 1: w = pick_cell<1>(pk, sel, rec, tab, total, k, q, qe, me, fin, reach1); break;
                case 2: w = pick_cell<2>(pk, sel, rec, tab, total, k, q, qe, me, fin, reach1); break;
                case 3: w = pick_cell<3>(pk, sel, rec, tab, total, k, q, qe, me, fin, reach1); break;
                case 4: w = pick_cell<4>(pk, sel, rec, tab, total, k, q, qe, me, fin, reach1); break;
                case 5: w = pick_cell<5>(pk, sel, rec, tab, total, k, q, qe, me, fin, reach1); break;
                case 6: w = pick_cell<6>(pk, sel, rec, tab, total, k, q, qe, me, fin, reach1); break;
                default: w = pick_cell<8>(pk, sel, rec, tab, total, k, q, qe, me, fin, reach1); break;
            }
        }
        wide |= w;
        if (lane < kQueries && ((w >> lane) & 1)) at_level = level;
        q = qe;
    }
    auto append = [&](uint32_t mask, SegCount *count, int2 *list, int level) __attribute__((always_inline)) {
        if (!mask) return;
        uint32_t at = 0;
        const int s = blockIdx.x % kSegs;
        if (lane == 0) at = atomicAdd(&count[s].v, static_cast<uint32_t>(__popc(mask)));
        at = uniform(at);
        if (lane < kQueries && ((mask >> lane) & 1))
            list[seg_size(n) * s + at + __popc(mask & ((1u << lane) - 1))] =
                make_int2(static_cast<int32_t>(r0 + lane), level);
    };
    append(wide, seg_count, seg, at_level);
    append(over, far_count, far, kBits);
    lds_fence();
    const int q = lane / 8;
    const int64_t qid = __float_as_int(__shfl(me.w, q, kWave));
    if (q < nq && !(((wide | over) >> q) & 1)) put_query(sels[wv][q], qid, k, feat, lane % 8, 8, x, y, nbr);
}

// The listed queries, one wavefront per query: the 5 x 5 x 5 cells, from the level that left the query
// undecided to coarser ones while the block has at most kFar points, held in registers.  What stays
// undecided is listed for the streaming scan (a list of the same segment, so that it cannot overflow).
__global__ __launch_bounds__(kBlock) void wide_select_kernel(const Curve *__restrict__ curve,
                                                             const int32_t *__restrict__ start,
                                                             const f4 *__restrict__ rec,
                                                             const int32_t *__restrict__ sorted, int64_t n, int k,
                                                             int feat, const float *__restrict__ x,
                                                             float *__restrict__ y, int32_t *__restrict__ nbr,
                                                             const SegCount *__restrict__ seg_count,
                                                             const int2 *__restrict__ seg,
                                                             SegCount *__restrict__ far_count,
                                                             int2 *__restrict__ far) {
    constexpr int B = kFar / kWave;
    __shared__ Pick picks[kBlock / kWave];
    __shared__ int32_t tabs[kBlock / kWave][kFar];
    __shared__ int32_t sels[kBlock / kWave][kSelRow];
    const int lane = lane_id(), wv = uniform(static_cast<int>(threadIdx.x) / kWave);
    int32_t *tab = tabs[wv], *sel = sels[wv];
    const int64_t w = static_cast<int64_t>(blockIdx.x) * (kBlock / kWave) + wv;
    const int64_t nw = static_cast<int64_t>(gridDim.x) * (kBlock / kWave);
    const Curve c = *curve;
    for_listed(seg_count, w, nw, [&](int s, int64_t i) __attribute__((always_inline)) {
        const int2 e = seg[seg_size(n) * s + i];
        const int64_t r = e.x;
        const f4 me = rec[r];
        const int key = sorted[r];
        const int qid = __float_as_int(me.w);
        bool done = false;
        int level = e.y;
        for (; !done && level >= 0; --level) {
            const uint32_t cell = static_cast<uint32_t>(key) >> (3 * (kBits - level));
            lds_fence();
            int total = 0;
            for (int i0 = 0; i0 < 125 && total >= 0; i0 += kWave)
                total = gather_cells<2>(c, start, sorted, level, cell, i0, total, kFar, tab);
            if (total < 0) break;
            if (lane < kSelRow) sel[lane] = -1;
            float d2[B];
            int id[B];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int j = b * kWave + lane;
                const f4 p = rec[j < total ? tab[j] : r];
                id[b] = __float_as_int(p.w);
                const float v = sqdist(me, p);
                d2[b] = id[b] == qid ? __builtin_inff() : v;   // the query itself, or no candidate
            }
            done = pick_query<B>(picks[wv], d2, id, block_reach2(c, me, key, level, 2), k, sel);
        }
        if (!done) {
            // a coarser block must be looked at as a whole, from the level whose reach is larger
            if (lane == 0)
                far[seg_size(n) * s + atomicAdd(&far_count[s].v, 1u)] = make_int2(e.x, level > 0 ? level - 1 : 0);
            return;
        }
        put_query(sel, qid, k, feat, lane, kWave, x, y, nbr);
    });
}

// Lower bound of the squared distance from a point to the points of one level-`level` cell (border cells
// hold the points beyond them too), with the relative margin of block_reach2.  The cell's face may be as
// near as the roundings of the coordinates on both sides of it (each some 2^-52 of its size), so the
// distance also gives way by 2^-50 of them.
__device__ __forceinline__ float cell_gap2(const Curve &c, f4 at, int level, int x, int y, int z) {
    const float p[3] = {at.x, at.y, at.z};
    const int cell[3] = {x, y, z}, sub = kBits - level;
    const double h = static_cast<double>(1 << sub) / c.inv_f;
    double g2 = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double d = static_cast<double>(p[a]) - c.lo[a], slack = (fabs(d) + h * (cell[a] + 1)) * 0x1p-50;
        double g = 0.0;
        if (cell[a] > 0) g = fmax(g, h * cell[a] - d - slack);
        if (cell[a] < (c.last[a] >> sub)) g = fmax(g, d - h * (cell[a] + 1) - slack);
        g2 += g * g;
    }
    return g2 > 1e-30 ? static_cast<float>(fmin(g2 * (1.0 - 4e-6), static_cast<double>(__FLT_MAX__))) : 0.0f;
}

// Fold the records [b, e) into the one-key-per-lane list L (k keys, the k-th is thr), 64 per step; the
// next step's records are loaded ahead.  Lanes past the end hold the query itself, which is never selected.
__device__ __forceinline__ void stream_records(const f4 *__restrict__ rec, int b, int e, f4 me, int k, uint64_t &L,
                                               uint64_t &thr) {
    const int lane = lane_id();
    const int qid = __float_as_int(me.w);
    f4 nxt = b + lane < e ? rec[b + lane] : me;
    for (int j0 = b; j0 < e; j0 += kWave) {
        const f4 p = nxt;
        const int jn = j0 + kWave + lane;
        nxt = jn < e ? rec[jn] : me;
        const float d2 = sqdist(me, p);
        if (!__any(d2 <= __uint_as_float(static_cast<uint32_t>(thr >> 32)))) continue;
        const int id = __float_as_int(p.w);
        uint64_t key = (static_cast<uint64_t>(__float_as_uint(d2)) << 32) | static_cast<uint32_t>(id);
        if (id == qid) key = ~0ull;
        insert_lanes(__builtin_amdgcn_ballot_w64(key < thr), key, k, L, thr);
    }
}

// The queries that the wider scan leaves undecided, one wavefront per query: the 27 cells around it from
// the listed level to coarser ones, streamed through the list as their children (6 x 6 x 6 cells of the next
// finer level; the finest level as it is), the query's own first, those farther than the k-th key skipped.
// Level 0 is the whole cloud, so every query is decided.
__global__ __launch_bounds__(kBlock, 8) void stream_select_kernel(const Curve *__restrict__ curve,
                                                                  const int32_t *__restrict__ start,
                                                                  const f4 *__restrict__ rec,
                                                                  const int32_t *__restrict__ sorted, int64_t n,
                                                                  int k, int feat, const float *__restrict__ x,
                                                                  float *__restrict__ y, int32_t *__restrict__ nbr,
                                                                  const SegCount *__restrict__ seg_count,
                                                                  const int2 *__restrict__ seg) {
    __shared__ int32_t sels[kBlock / kWave][kSelRow];
    const int lane = lane_id(), wv = uniform(static_cast<int>(threadIdx.x) / kWave);
    int32_t *sel = sels[wv];
    const int64_t w = static_cast<int64_t>(blockIdx.x) * (kBlock / kWave) + wv;
    const int64_t nw = static_cast<int64_t>(gridDim.x) * (kBlock / kWave);
    const Curve c = *curve;
    for_listed(seg_count, w, nw, [&](int s, int64_t i) __attribute__((always_inline)) {
        const int2 e = seg[seg_size(n) * s + i];
        const int r = uniform(e.x);
        const f4 me = rec[r];
        const int key = uniform(sorted[r]);
        uint64_t L = kNone;
        for (int level = uniform(e.y);; --level) {
            const int cl = level < kBits ? level + 1 : kBits, W = level < kBits ? 6 : 3;
            const uint32_t m0 = static_cast<uint32_t>(key) >> (3 * (kBits - level));
            const int scale = W / 3, top = 1 << cl;
            const int x0 = scale * (static_cast<int>(gather3(m0)) - 1),
                      y0 = scale * (static_cast<int>(gather3(m0 >> 1)) - 1),
                      z0 = scale * (static_cast<int>(gather3(m0 >> 2)) - 1);
            const uint32_t own = static_cast<uint32_t>(key) >> (3 * (kBits - cl));
            uint64_t thr = kNone;
            L = kNone;
            int b = 0, len = 0;
            cell_range(c, start, sorted, cl, own, b, len);
            stream_records(rec, uniform(b), uniform(b + len), me, k, L, thr);
            for (int i0 = 0; i0 < W * W * W; i0 += kWave) {
                const int at = i0 + lane;
                const int cx = x0 + at % W, cy = y0 + (at / W) % W, cz = z0 + at / (W * W);
                b = len = 0;
                float gap = __builtin_inff();
                if (at < W * W * W && cx >= 0 && cy >= 0 && cz >= 0 && cx < top && cy < top && cz < top) {
                    const uint32_t m = morton(cx, cy, cz);
                    gap = cell_gap2(c, me, cl, cx, cy, cz);
                    if (m != own) cell_range(c, start, sorted, cl, m, b, len);
                }
                uint64_t todo = __builtin_amdgcn_ballot_w64(len > 0);
                while (true) {
                    todo &= __builtin_amdgcn_ballot_w64(gap <= __uint_as_float(static_cast<uint32_t>(thr >> 32)));
                    if (!todo) break;
                    const int o = __builtin_ctzll(todo);
                    todo &= todo - 1;
                    const int ob = __builtin_amdgcn_readlane(b, o);
                    stream_records(rec, ob, ob + __builtin_amdgcn_readlane(len, o), me, k, L, thr);
                }
            }
            const float reach = block_reach2(c, me, key, level, 1);
            // decided if the k-th key lies within reach, or the block holds every finite point
            if (level == 0 || reach == __FLT_MAX__ ||
                (thr < kNone && __uint_as_float(static_cast<uint32_t>(thr >> 32)) <= reach))
                break;
        }
        lds_fence();
        if (lane < kSelRow)
            sel[lane] = lane < k && L < kNone ? static_cast<int32_t>(static_cast<uint32_t>(L)) : -1;
        lds_fence();
        put_query(sel, __float_as_int(me.w), k, feat, lane, kWave, x, y, nbr);
    });
}

// ---- small relations: one wavefront per query, no build

// At or below this many points every query scans every point and no relation is built (box, curve keys,
// sort, index): the build's launches and the cell select's dependent chains cost more there than the
// quadratic distance work.  Measured with the build and without it: 4,096 points 72 and 37 us, 8,192
// points 73 and 84 us (k = 16); 8,192 points 66 and 63 us (k = 4), 81 and 109 us (k = 32).
constexpr int64_t kBruteMax = 7168;
// Up to this many points the queries that the wider scan leaves undecided scan every point too: a third of
// 12,000 points in a tight clump took 250 us in all with the streaming scan and 200 us this way.
constexpr int64_t kBruteFar = 16384;
constexpr int kBruteWaves = 4;   // queries per block

// Wavefront w of block b takes query q = kBruteWaves b + w; its lanes scan the points 64 at a
// time in input order, with the fp32 distance and the (distance, index) key of the cell select.
// The query's KP smallest keys are kept one per lane (lanes 0..KP-1, ascending); a step's keys
// below the current KP-th key are found by one ballot and inserted one at a time, so the list is
// exact whatever the order of the scan.  With a list (far_count) the queries are its records, and the
// neighbour sums are added in key order, as for the call's other queries.
template <int KP>
__global__ __launch_bounds__(kBruteWaves * kWave) void brute_kernel(const float *__restrict__ pos, int64_t n, int k,
                                                                    int feat, const float *__restrict__ x,
                                                                    float *__restrict__ y, int32_t *__restrict__ nbr,
                                                                    const SegCount *__restrict__ far_count,
                                                                    const int2 *__restrict__ far,
                                                                    const f4 *__restrict__ rec) {
    __shared__ int32_t sels[kBruteWaves][kMaxK];
    const int lane = lane_id(), wv = uniform(static_cast<int>(threadIdx.x) / kWave);
    int64_t q = static_cast<int64_t>(blockIdx.x) * kBruteWaves + wv;
    if (q >= n) return;
    if (far_count) {
        // at most n listed queries, one per wavefront
        int64_t listed = -1;
        for_listed(far_count, q, n, [&](int s, int64_t i) { listed = far[seg_size(n) * s + i].x; });
        if (listed < 0) return;
        q = uniform(__float_as_int(rec[listed].w));
    }
    const f4 me = f4{pos[q * 3], pos[q * 3 + 1], pos[q * 3 + 2], 0.0f};   // uniform: scalar loads
    uint64_t L = kNone;                                                      // lane t < KP: the t-th key
    if (finite3(me.x, me.y, me.z)) {
        uint64_t thr = kNone;                                                // the KP-th key (uniform)
        // candidates of the next step are loaded before the current step is tested
        int64_t j = lane;
        f4 pj = j < n ? f4{pos[j * 3], pos[j * 3 + 1], pos[j * 3 + 2], 0.0f} : f4{0.0f, 0.0f, 0.0f, 0.0f};
        for (int64_t c0 = 0; c0 < n; c0 += kWave) {
            const f4 cur = pj;
            const int64_t jc = c0 + lane;
            j = jc + kWave;
            if (j < n) pj = f4{pos[j * 3], pos[j * 3 + 1], pos[j * 3 + 2], 0.0f};
            const float d2 = sqdist(me, cur);
            uint64_t key = (static_cast<uint64_t>(__float_as_uint(d2)) << 32) | static_cast<uint32_t>(jc);
            key = (jc >= n || jc == q) ? ~0ull : key;   // past the end, or the query itself
            insert_lanes(__builtin_amdgcn_ballot_w64(key < thr), key, KP, L, thr);
        }
    }
    const bool has = lane < k && L < kNone;
    const int32_t sel = has ? static_cast<int32_t>(static_cast<uint32_t>(L)) : -1;
    if (far_count) {
        if (lane < kMaxK) sels[wv][lane] = sel;
        lds_fence();
        put_query(sels[wv], q, k, feat, lane, kWave, x, y, nbr);
        return;
    }
    if (nbr && lane < k) nbr[q * k + lane] = sel;
    for (int f = 0; f < feat; ++f) {
        float v = has ? x[static_cast<int64_t>(sel) * feat + f] : 0.0f;
        // fixed shuffle tree over the lanes (the selected rows in key order, then zeros)
#pragma unroll
        for (int o = kWave / 2; o >= 1; o /= 2) v += __shfl_xor(v, o);
        if (lane == 0) y[q * feat + f] = v;
    }
}

template <int KP>
int launch_brute(int64_t n, int k, int feat, const float *pos, const float *x, float *y, int32_t *nbr,
                 hipStream_t stream, const SegCount *far_count = nullptr, const int2 *far = nullptr,
                 const f4 *rec = nullptr) {
    if (!far) prof_before(stream);
    hipLaunchKernelGGL(brute_kernel<KP>, dim3(static_cast<unsigned>(ceil_div(n, kBruteWaves))),
                       dim3(kBruteWaves * kWave), 0, stream, pos, n, k, feat, x, y, nbr, far_count, far, rec);
    if (!far) prof_after(stream);
    return check_launch("kNN brute force");
}

}  // namespace

// Points per cell: the ball of one cell width around a query then holds about k + 4 sqrt(k) + 6 points
// (so k of them nearly always), at most 50 (so that they nearly always fit one wavefront).
double cell_points(int k) {
    const double ball = k + 4.0 * std::sqrt(static_cast<double>(k)) + 6.0;
    return (ball < 50.0 ? ball : 50.0) * 3.0 / (4.0 * 3.14159265358979);
}

size_t workspace_bytes(int64_t n) {
    Carve c(nullptr);
    carve(c, n);
    return c.bytes();
}

int forward(int64_t n, int32_t feat, const float *pos, const float *x, int32_t k, float *y, int32_t *nbr, void *ws,
            hipStream_t stream) {
    const int kp = k <= 1 ? 1 : k <= 2 ? 2 : k <= 4 ? 4 : k <= 8 ? 8 : k <= 16 ? 16 : 32;
    auto brute = [&](const SegCount *far_count, const int2 *far, const f4 *rec) {
        switch (kp) {
            case 1: return launch_brute<1>(n, k, feat, pos, x, y, nbr, stream, far_count, far, rec);
            case 2: return launch_brute<2>(n, k, feat, pos, x, y, nbr, stream, far_count, far, rec);
            case 4: return launch_brute<4>(n, k, feat, pos, x, y, nbr, stream, far_count, far, rec);
            case 8: return launch_brute<8>(n, k, feat, pos, x, y, nbr, stream, far_count, far, rec);
            case 16: return launch_brute<16>(n, k, feat, pos, x, y, nbr, stream, far_count, far, rec);
            default: return launch_brute<32>(n, k, feat, pos, x, y, nbr, stream, far_count, far, rec);
        }
    };
    if (n <= kBruteMax) return brute(nullptr, nullptr, nullptr);
    Carve c(ws);
    Ws w = carve(c, n);
    const int np = static_cast<int>(ceil_div(n, kBlock) < kPartials ? ceil_div(n, kBlock) : kPartials);
    hipLaunchKernelGGL(box_partial_kernel, dim3(np), dim3(kBlock), 0, stream, pos, n, w.part, w.moments);
    if (int rc = check_launch("kNN box")) return rc;
    const radix::Shape s = radix::shape_for(n, int64_t{1} << (3 * kBits));
    const int top = max_level(n);
    auto *kern = s.items == 2 ? key_kernel<2> : s.items == 4 ? key_kernel<4> : key_kernel<8>;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(s.tiles)), dim3(radix::kThreads), 0, stream, pos, n, w.part,
                       w.moments, np, cell_points(k), top, s.rb, w.curve, w.key, w.sort.counts);
    if (int rc = check_launch("kNN keys")) return rc;
    radix::Out out;
    out.keys = w.key_sorted;
    out.pos = pos;
    out.rec = reinterpret_cast<float4 *>(w.rec);
    if (int rc = radix::launch_sort(s, w.key, w.sort, out, nullptr, stream)) return rc;
    const int64_t cells = (int64_t{1} << (3 * top)) + 1;
    const int64_t cb = ceil_div(cells, kBlock) < 1024 ? ceil_div(cells, kBlock) : 1024;
    hipLaunchKernelGGL(cells_kernel, dim3(static_cast<unsigned>(cb)), dim3(kBlock), 0, stream, w.curve, w.key_sorted, n,
                       w.start, w.seg_count);
    if (int rc = check_launch("kNN cells")) return rc;
    prof_before(stream);
    hipLaunchKernelGGL(cell_select_kernel, dim3(static_cast<unsigned>(ceil_div(n, kQueries * (kBlock / kWave)))),
                       dim3(kBlock), 0, stream, w.curve, w.start, w.rec, w.key_sorted, n, k, feat, x, y, nbr,
                       w.seg_count, w.seg, w.seg_count + kSegs, w.far);
    prof_after(stream);
    if (int rc = check_launch("kNN cell select")) return rc;
    // persistent grids: how many queries are listed is known on the device only
    static const int wide_blocks = resident_blocks(reinterpret_cast<const void *>(&wide_select_kernel), kBlock);
    static const int far_blocks = resident_blocks(reinterpret_cast<const void *>(&stream_select_kernel), kBlock);
    const int64_t most = ceil_div(n, kBlock / kWave), cus = device_cus();
    const int64_t wb = wide_blocks * cus < most ? wide_blocks * cus : most;
    hipLaunchKernelGGL(wide_select_kernel, dim3(static_cast<unsigned>(wb)), dim3(kBlock), 0, stream, w.curve, w.start,
                       w.rec, w.key_sorted, n, k, feat, x, y, nbr, w.seg_count, w.seg, w.seg_count + kSegs, w.far);
    if (int rc = check_launch("kNN wide select")) return rc;
    if (n <= kBruteFar) return brute(w.seg_count + kSegs, w.far, w.rec);
    const int64_t fb = far_blocks * cus < most ? far_blocks * cus : most;
    hipLaunchKernelGGL(stream_select_kernel, dim3(static_cast<unsigned>(fb)), dim3(kBlock), 0, stream, w.curve,
                       w.start, w.rec, w.key_sorted, n, k, feat, x, y, nbr, w.seg_count + kSegs, w.far);
    return check_launch("kNN streaming select");
}

}  // namespace knn
}  // namespace tiga
