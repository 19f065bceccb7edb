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
//    k = 16) are compacted and ranked by counting.  Where a block holds more than 512 points a finer
//    level of the curve is taken (the box is cut four standard deviations from the mean, so that far points
//    do not use up the levels).  Otherwise the query is listed, and a second launch
//    scans its 5 x 5 x 5 cells, then those of coarser levels, one wavefront per listed query (they sit
//    together at the cloud's faces, so a wavefront with eight of them would end long after the rest); where a
//    block holds more than 1,536 points a third launch streams cells, the nearest first, through a list of the
//    k smallest keys so far (up to 16,384 points: every point).
//  - Small relations (brute_kernel): a wavefront per query streams every point through such a list.
//  Measured, 131,072 uniform points, k = 16: the previous select (tiles of 64 queries, one per lane with its
//  keys sorted in registers, whose insertion ran for the whole wavefront whenever one lane accepted) took
//  366 us, the cell select takes 78 us and the second launch 15 us (k = 32, whole call: 1,408 us before,
//  179 us now).  The cell select is bound by VALU issue: about 8 tests per selected neighbour and 2
//  instructions per pair of compacted candidates.  131,072 points of unequal density, k = 16, whole calls,
//  tiles and now: a third in a clump of 0.002 2,173 and 796 us, normal 507 and 378 us, one far outlier
//  3,375 and 328 us, 100 copies of each position 231 and 206 us.  At k = 4, clusters whose finest cells are
//  below the table are still slower than the tiles were (50 clusters: 253 and 353 us).
#include "knn.hpp"

#include <cmath>

#include "common.hpp"
#include "radix.hpp"

namespace tiga {
namespace knn {

namespace {

constexpr int kBlock = 256;
constexpr int kBits = 10;                                 // Morton bits per axis
constexpr int kPartials = 256;                            // read by every block of the key kernel
constexpr int kMoments = 7;

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

constexpr int kQueries = 8;       // queries per wavefront of the cell select, at most
constexpr int kNear = 512;        // candidates of the 27 cells, held in registers (8 per lane)
constexpr int kFar = 1536;        // candidates of the 125 cells (24 per lane)
constexpr int kMaxK = 32;

// Two queries per wavefront below this many points: a wavefront's queries follow one another, each through a
// chain of dependent loads, and with eight there are too few wavefronts to cover it.
constexpr int64_t kFewQueries = 24000;

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
    double *moments;    // [kPartials][kMoments] sums of the finite coordinates, of their squares, of ones
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
    w.moments = c.take<double>(kPartials * kMoments);
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

__device__ __forceinline__ void lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
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

// Box and moments of the finite points: per-block partials (min xyz, max xyz; sums, sums of squares, number).
__global__ __launch_bounds__(kBlock) void box_partial_kernel(const float *__restrict__ pos, int64_t n,
                                                             float *__restrict__ part,
                                                             double *__restrict__ moments) {
    __shared__ float red[kBlock / kWave][6];
    __shared__ double sums[kBlock / kWave][kMoments];
    float v[6] = {__builtin_inff(), __builtin_inff(), __builtin_inff(),
                  -__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
    double s[kMoments] = {};
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
        s[6] += 1.0;
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) v[a] = a < 3 ? wave_min(v[a]) : wave_max(v[a]);
#pragma unroll
    for (int a = 0; a < kMoments; ++a) s[a] = wave_sum(s[a]);
    const int w = threadIdx.x / kWave;
    if (lane_id() == 0) {
        for (int a = 0; a < 6; ++a) red[w][a] = v[a];
        for (int a = 0; a < kMoments; ++a) sums[w][a] = s[a];
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        float r = red[0][threadIdx.x];
        for (int q = 1; q < kBlock / kWave; ++q)
            r = threadIdx.x < 3 ? fminf(r, red[q][threadIdx.x]) : fmaxf(r, red[q][threadIdx.x]);
        part[blockIdx.x * 6 + threadIdx.x] = r;
    }
    if (threadIdx.x < kMoments) {
        double t = sums[0][threadIdx.x];
        for (int q = 1; q < kBlock / kWave; ++q) t += sums[q][threadIdx.x];
        moments[blockIdx.x * kMoments + threadIdx.x] = t;
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

// The box cut four standard deviations from the mean (each axis by a thread of its own).
struct Cut {
    double lo[3], hi[3];
};
__device__ __forceinline__ void cut_axis(Cut &c, int a, double lo, double hi, double sum, double squares, double number) {
    const double mean = sum / number, var = squares / number - mean * mean;
    if (var > 0.0) {
        const double r = 4.0 * sqrt(var);
        if (mean - r > lo) lo = mean - r;
        if (mean + r < hi) hi = mean + r;
    }
    c.lo[a] = lo;
    c.hi[a] = hi;
}

// Cell size for the cut box: `points` points per cell if the cloud were uniform, coarser where the table
// (base <= top) or the curve's scale (the longest axis) asks for it.  A few far points must not take the
// resolution from all others: points outside the cut share its border cells.
__device__ __forceinline__ Curve make_curve(const Cut &cut, const double *hi, double number, double points,
                                            int top) {
    Curve c;
    double ext[3], vol = 1.0, longest = 0.0;
    for (int a = 0; a < 3; ++a) {
        c.lo[a] = cut.lo[a];
        ext[a] = cut.hi[a] - cut.lo[a];
        if (!(ext[a] > 0.0)) ext[a] = 0.0;   // no extent, or no finite point at all
        vol *= ext[a];
        longest = fmax(longest, ext[a]);
    }
    double h = cbrt(vol * points / fmax(number, 1.0));
    const double finest = longest / static_cast<double>(1 << top);
    if (!(h > finest)) h = finest;
    if (!(h > 0.0)) h = 1.0;                 // coincident points
    int level = 0;
    while (level < top && longest >= h * static_cast<double>(1 << level)) ++level;
    c.base = level;
    c.inv_f = static_cast<double>(1 << (kBits - level)) / h;
    for (int a = 0; a < 3; ++a) c.last[a] = static_cast<int>(fine_axis(c, a, static_cast<float>(hi[a])));
    return c;
}

// Morton key of every point (non-finite points: the last key) and the sort's first histogram.  Every
// block reduces the box partials and forms the curve for itself; block 0 stores it.  The moments are taken
// again without the partials that reach past the cut: a point ten thousand extents away widens the cut a
// hundredfold (12,000 points, k = 16, one of them far: whole call 218 us without this, 106 us with it).
template <int ITEMS>
__global__ __launch_bounds__(radix::kThreads) void key_kernel(const float *__restrict__ pos, int64_t n,
                                                              const float *__restrict__ part,
                                                              const double *__restrict__ moments, int nparts,
                                                              double points, int top, int rb,
                                                              Curve *__restrict__ curve, int32_t *__restrict__ key,
                                                              uint32_t *__restrict__ counts) {
    static_assert(kPartials <= radix::kThreads && 32 * (6 + kMoments) <= radix::kThreads, "threads of the reductions");
    __shared__ uint32_t hist[radix::kMaxDigits];
    __shared__ double tot[6 + kMoments], in[6 + kMoments];
    __shared__ uint8_t out[kPartials];
    __shared__ bool again;
    __shared__ Cut cut;
    __shared__ Curve sc;
    const int t = threadIdx.x;
    // 32 threads per quantity (min xyz, max xyz, moments), all loads in flight
    constexpr int kEach = kPartials / 32;
    const int q = t / 32;
    if (q < 6) {
        float u[kEach];
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            const int p = j * 32 + t % 32;
            u[j] = part[(p < nparts ? p : 0) * 6 + q];
            if (q >= 3) u[j] = -u[j];
        }
        float r = u[0];
#pragma unroll
        for (int j = 1; j < kEach; ++j) r = fminf(r, u[j]);
#pragma unroll
        for (int m = 1; m < 32; m <<= 1) r = fminf(r, __shfl_xor(r, m, 32));
        if (t % 32 == 0) tot[q] = q < 3 ? r : -r;
    }
    // the moments of the partials not marked in `out` (null: of all)
    auto sum_moments = [&](double *into, const uint8_t *out) __attribute__((always_inline)) {
        if (q < 6 || q >= 6 + kMoments) return;   // whole halves of wavefronts
        double u[kEach], r = 0.0;
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            const int p = j * 32 + t % 32;
            u[j] = moments[(p < nparts ? p : 0) * kMoments + (q - 6)];
        }
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            const int p = j * 32 + t % 32;
            r += p < nparts && !(out && out[p]) ? u[j] : 0.0;
        }
#pragma unroll
        for (int m = 1; m < 32; m <<= 1) r += __shfl_xor(r, m, 32);
        if (t % 32 == 0) into[q] = r;
    };
    sum_moments(tot, nullptr);
    __syncthreads();
    auto put_curve = [&]() __attribute__((always_inline)) {
        sc = make_curve(cut, tot + 3, tot[12], points, top);
        if (blockIdx.x == 0) *curve = sc;
    };
    if (t < kWave) {
        bool clipped = false;
        if (t < 3) {
            cut_axis(cut, t, tot[t], tot[3 + t], tot[6 + t], tot[9 + t], tot[12]);
            clipped = cut.lo[t] > tot[t] || cut.hi[t] < tot[3 + t];
        }
        lds_fence();
        const bool any = __any(clipped);
        if (t == 0) {
            again = any;
            if (!any) put_curve();
        }
    }
    __syncthreads();
    if (again) {
        if (t < nparts) {
            bool past = false;
            for (int a = 0; a < 3; ++a)
                past |= part[t * 6 + a] < cut.lo[a] || part[t * 6 + 3 + a] > cut.hi[a];
            out[t] = past;
        }
        __syncthreads();
        sum_moments(in, out);
        __syncthreads();
        if (t < kWave) {
            if (t < 3 && 2.0 * in[12] > tot[12]) cut_axis(cut, t, tot[t], tot[3 + t], in[6 + t], in[9 + t], in[12]);
            lds_fence();
            if (t == 0) put_curve();
        }
        __syncthreads();
    }
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

__device__ __forceinline__ float readlane_f(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// Working set of one query: compacted candidates (distance bits, padded for 4-wide reads, and index) and
// the selected indices in key order (-1 past the end; one slot past k shows ties at the k-th key).
constexpr int kPickMax = 2 * kWave;
constexpr int kSpare = 8;   // where candidates are cut down, so many more than k may stay
struct alignas(16) Pick {
    uint32_t d2[kPickMax + 4];
    int32_t id[kPickMax + 4];
};
constexpr int kSelRow = kMaxK + 1;

// The cells of level `level` with ids m[i] (i with ok[i]; the others are empty): first records, numbers of records.
// Above the table's level a cell is a run of table cells, below it a part of one, found by binary searches for its
// first and its last key: all of them in step, so that their dependent loads wait together.
template <int C>
__device__ __forceinline__ void cell_ranges(const Curve &c, const int32_t *__restrict__ start,
                                            const int32_t *__restrict__ sorted, int level, const uint32_t (&m)[C],
                                            const bool (&ok)[C], int (&s)[C], int (&len)[C]) {
    if (level <= c.base) {
        const int up = 3 * (c.base - level);
#pragma unroll
        for (int i = 0; i < C; ++i) {
            s[i] = ok[i] ? start[m[i] << up] : 0;
            len[i] = ok[i] ? start[(m[i] + 1) << up] - s[i] : 0;
        }
        return;
    }
    const int shift = 3 * (kBits - level);
    int from[C], n[C], a[C], b[C], most = 0;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        const uint32_t in = m[i] >> (3 * (level - c.base));
        from[i] = ok[i] ? start[in] : 0;
        n[i] = ok[i] ? start[in + 1] - from[i] : 0;
        a[i] = b[i] = 0;
        most = n[i] > most ? n[i] : most;
    }
    for (int step = most > 0 ? 1 << (31 - __builtin_clz(most)) : 0; step > 0; step >>= 1)
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const int ta = a[i] + step, tb = b[i] + step;
            const int32_t ka = ta <= n[i] ? sorted[from[i] + ta - 1] : INT32_MAX,
                          kb = tb <= n[i] ? sorted[from[i] + tb - 1] : INT32_MAX;
            if (ka < static_cast<int32_t>(m[i] << shift)) a[i] = ta;
            if (kb < static_cast<int32_t>((m[i] + 1) << shift)) b[i] = tb;
        }
#pragma unroll
    for (int i = 0; i < C; ++i) {
        s[i] = from[i] + a[i];
        len[i] = b[i] - a[i];
    }
}

// The candidates of the (2R + 1)^3 block of level-`level` cells around cell m0 to the table of records `tab`;
// returns their number, or -1 if they exceed `cap` (the table is then unfinished).
template <int R>
__device__ __forceinline__ int gather_cells(const Curve &c, const int32_t *__restrict__ start,
                                            const int32_t *__restrict__ sorted, int level, uint32_t m0, int cap,
                                            int32_t *__restrict__ tab) {
    constexpr int W = 2 * R + 1, C = (W * W * W + kWave - 1) / kWave;
    const int lane = lane_id(), side = 1 << level;
    const int x0 = static_cast<int>(gather3(m0)) - R, y0 = static_cast<int>(gather3(m0 >> 1)) - R,
              z0 = static_cast<int>(gather3(m0 >> 2)) - R;
    uint32_t m[C];
    bool ok[C];
    int s[C], len[C];
#pragma unroll
    for (int j = 0; j < C; ++j) {
        const int i = j * kWave + lane, x = x0 + i % W, y = y0 + (i / W) % W, z = z0 + i / (W * W);
        ok[j] = i < W * W * W && x >= 0 && y >= 0 && z >= 0 && x < side && y < side && z < side;
        m[j] = morton(x, y, z);
    }
    cell_ranges<C>(c, start, sorted, level, m, ok, s, len);
    int total = 0;
#pragma unroll
    for (int j = 0; j < C; ++j) {
        const int l = len[j] < cap + 1 ? len[j] : cap + 1;   // 64 of them cannot overflow the sum
        const int incl = wave_incl_scan(l);
        const int at = total + incl - l;
        total += __builtin_amdgcn_readlane(incl, kWave - 1);
        if (total > cap) return -1;
        for (int i = 0; __any(i < l); ++i)
            if (i < l) tab[at + i] = s[j] + i;
    }
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

// The indices of the k smallest keys of the m <= 64 candidates in `pk`, in key order, to sel (-1 before).
__device__ __forceinline__ void rank_picks(Pick &pk, int m, int k, int32_t *__restrict__ sel) {
    const int lane = lane_id();
    if (lane < 4) {
        pk.d2[m + lane] = ~0u;
        pk.id[m + lane] = INT32_MAX;
    }
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
        for (int j = 0; j < m; j += 4) {
            const i32x4 o = *reinterpret_cast<const i32x4 *>(&pk.d2[j]), i = *reinterpret_cast<const i32x4 *>(&pk.id[j]);
#pragma unroll
            for (int u = 0; u < 4; ++u) rank += static_cast<uint32_t>(o[u]) == mine && i[u] < my_id;
        }
        if (lane < m && rank <= k) sel[rank] = my_id;
        lds_fence();
    }
}

// Select the k smallest keys of one query from the candidates (d2[b], id[b]) of the lanes (no candidate:
// +inf) when they are decided by those within `reach` (FLT_MAX: always), and write their indices in key
// order to sel.  False: undecided.
template <int B>
__device__ __forceinline__ bool pick_query(Pick &pk, const float (&d2)[B], const int (&id)[B], float reach, int k,
                                           int n, int32_t *__restrict__ sel) {
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
    auto compact = [&](auto &&in) __attribute__((always_inline)) {
        int base = 0;
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const bool keep = in(b);
            const uint64_t mask = __builtin_amdgcn_ballot_w64(keep);
            if (keep) {
                const int at = base + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                                                __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0));
                pk.d2[at] = __float_as_uint(d2[b]);
                pk.id[at] = id[b];
            }
            base += __popcll(mask);
        }
    };
    bool ties = false;
    if (m > kWave) {
        uint32_t hi = __float_as_uint(reach), lo = hi > (3u << 23) ? hi - (3u << 23) : 0;
        int below = within(__uint_as_float(lo));   // less than k; lo = hi = 0: none
        if (below >= k) {
            lo = 0;
            below = within(0.0f);
            if (below >= k) {
                hi = 0;
                m = below;
                below = 0;
            }
        }
        while (m > kWave && hi - lo > 1) {
            const uint32_t mid = lo + (hi - lo) / 2;
            const int mm = within(__uint_as_float(mid));
            if (mm >= k) hi = mid, m = mm;
            else lo = mid, below = mm;
        }
        reach = __uint_as_float(hi);
        if (m > kWave) {
            // still more, so all at the distance hi but those below it: bisect their ids
            ties = true;
            int from = -1, last = n;
            while (m > k + kSpare) {
                const int mid = from + (last - from) / 2;
                int mm = below;
#pragma unroll
                for (int b = 0; b < B; ++b) mm += __popcll(__builtin_amdgcn_ballot_w64(d2[b] == reach && id[b] <= mid));
                if (mm >= k) last = mid, m = mm;
                else from = mid;
            }
            compact([&](int b) { return d2[b] < reach || (d2[b] == reach && id[b] <= last); });
        }
    }
    if (!ties) compact([&](int b) { return d2[b] <= reach; });
    rank_picks(pk, m, k, sel);
    return true;
}

// The queries q .. qe - 1 of one cell (lane q of `me`: the query's record, of `reach1`: how far the cells
// around it reach), whose `total` candidates are in `tab`, B 64-candidate steps held in registers.
// Returns the queries that stay undecided.  One instance per B: with a condition per step instead, the
// values merged at each of them took 364 registers.
template <int B>
__device__ __forceinline__ uint32_t pick_cell(Pick &pk, int32_t (*__restrict__ sel)[kSelRow],
                                              const f4 *__restrict__ rec, const int32_t *__restrict__ tab, int total,
                                              int k, int n, int q, int qe, f4 me, uint64_t fin, float reach1) {
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
        if (!pick_query<B>(pk, d2, id, readlane_f(reach1, q), k, n, sel[q])) left |= 1u << q;
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

// The k smallest keys of a stream of candidates: those no farther than `bound` are appended to the list in
// `pk`, which is cut down to about k of them, and the bound to their largest distance, whenever it holds more
// than 64.  (With the keys sorted in registers, one per lane, every key that entered cost a chain of
// cross-lane moves: a query beside a clump of 4,000 points, whose records come ever closer, took 130 us.)
constexpr int kAhead = 4;   // records per lane loaded together
struct TopK {
    Pick &pk;
    int k, n;   // all ids are below n
    int cnt = 0;
    float bound = __FLT_MAX__;

    __device__ __forceinline__ void offer(float d2, int id, bool ok) {
        const bool in = d2 <= bound && ok;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(in);
        if (!mask) return;
        if (in) {
            const int at = cnt + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                                           __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0));
            pk.d2[at] = __float_as_uint(d2);
            pk.id[at] = id;
        }
        cnt += __popcll(mask);
        if (cnt > kWave) shrink(k + kSpare);
    }

    // Drop the farthest, down to between k and `most` >= k candidates (all of them stay where they are fewer).
    // With most = k the bound ends as the k-th distance.
    __device__ __forceinline__ void shrink(int most) {
        if (cnt <= most) return;
        const int lane = lane_id();
        lds_fence();
        const uint32_t v0 = lane < cnt ? pk.d2[lane] : ~0u, v1 = lane + kWave < cnt ? pk.d2[lane + kWave] : ~0u;
        const int i0 = pk.id[lane], i1 = pk.id[lane + kWave];
        auto within = [&](uint32_t b) __attribute__((always_inline)) {
            return __popcll(__builtin_amdgcn_ballot_w64(v0 <= b)) + __popcll(__builtin_amdgcn_ballot_w64(v1 <= b));
        };
        uint32_t hi = __float_as_uint(bound), lo = 0;
        int m = cnt, below = within(0);   // below = within(lo) < k; lo = hi = 0: none
        if (below >= k) {
            hi = 0;
            m = below;
            below = 0;
        }
        while (m > most && hi - lo > 1) {
            const uint32_t mid = lo + (hi - lo) / 2;
            const int mm = within(mid);
            if (mm >= k) hi = mid, m = mm;
            else lo = mid, below = mm;
        }
        int from = -1, last = n;
        while (m > most) {   // at the distance hi, those of the lowest ids
            const int mid = from + (last - from) / 2;
            const int mm = below + __popcll(__builtin_amdgcn_ballot_w64(v0 == hi && i0 <= mid)) +
                           __popcll(__builtin_amdgcn_ballot_w64(v1 == hi && i1 <= mid));
            if (mm >= k) last = mid, m = mm;
            else from = mid;
        }
        const bool in0 = v0 < hi || (v0 == hi && i0 <= last), in1 = v1 < hi || (v1 == hi && i1 <= last);
        const uint64_t m0 = __builtin_amdgcn_ballot_w64(in0), m1 = __builtin_amdgcn_ballot_w64(in1);
        const int a0 = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m0 >> 32),
                                                 __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m0), 0));
        const int a1 = __popcll(m0) + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m1 >> 32),
                                                                __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m1), 0));
        lds_fence();
        if (in0) {
            pk.d2[a0] = v0;
            pk.id[a0] = i0;
        }
        if (in1) {
            pk.d2[a1] = v1;
            pk.id[a1] = i1;
        }
        lds_fence();
        cnt = m;
        bound = __uint_as_float(hi);
    }

    __device__ __forceinline__ void select(int32_t *__restrict__ sel) {
        if (lane_id() < kSelRow) sel[lane_id()] = -1;
        rank_picks(pk, cnt, k, sel);
    }
};

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

// Wavefront w takes the records [Q w, Q w + Q) as queries, cell by cell.
template <int Q>
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
    __shared__ int32_t sels[kBlock / kWave][Q][kSelRow];
    const int lane = lane_id(), wv = uniform(static_cast<int>(threadIdx.x) / kWave);
    Pick &pk = picks[wv];
    int32_t *tab = tabs[wv];
    const int64_t t = static_cast<int64_t>(xcd_block()) * (kBlock / kWave) + wv;
    const int64_t r0 = t * Q;
    if (r0 >= n) return;
    const int nq = static_cast<int>(n - r0 < Q ? n - r0 : Q);
    const Curve c = *curve;
    // lane q < nq: query q, its key, and how far the block of cells around it reaches
    const f4 me = rec[r0 + (lane < nq ? lane : 0)];
    const int key = lane < nq ? sorted[r0 + lane] : -1;
    const uint64_t fin = __builtin_amdgcn_ballot_w64(finite3(me.x, me.y, me.z));
    uint32_t wide = 0;       // undecided queries
    uint32_t over = 0;       // queries whose finest block holds more than kNear points
    int at_level = c.base;   // lane q: the level that left query q undecided
    uint32_t crowded = ~0u;  // a table cell whose block is known to hold more than kNear points
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
            if (level != c.base || cell != crowded) {
                lds_fence();
                total = gather_cells<1>(c, start, sorted, level, cell, kNear, tab);
            }
            if (total >= 0 || level == kBits) break;
            if (level++ == c.base) {
                crowded = cell;
                const int l = c.base + lane;
                const bool look[1] = {lane > 0 && l <= kBits};
                const uint32_t own[1] = {look[0] ? qkey >> (3 * (kBits - l)) : 0};
                int first[1], len[1];
                cell_ranges<1>(c, start, sorted, l, own, look, first, len);
                const uint64_t small = __builtin_amdgcn_ballot_w64(look[0] && len[0] <= kNear / 12);
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
                case 1: w = pick_cell<1>(pk, sel, rec, tab, total, k, static_cast<int>(n), q, qe, me, fin, reach1); break;
                case 2: w = pick_cell<2>(pk, sel, rec, tab, total, k, static_cast<int>(n), q, qe, me, fin, reach1); break;
                case 3: w = pick_cell<3>(pk, sel, rec, tab, total, k, static_cast<int>(n), q, qe, me, fin, reach1); break;
                case 4: w = pick_cell<4>(pk, sel, rec, tab, total, k, static_cast<int>(n), q, qe, me, fin, reach1); break;
                case 5: w = pick_cell<5>(pk, sel, rec, tab, total, k, static_cast<int>(n), q, qe, me, fin, reach1); break;
                case 6: w = pick_cell<6>(pk, sel, rec, tab, total, k, static_cast<int>(n), q, qe, me, fin, reach1); break;
                default: w = pick_cell<8>(pk, sel, rec, tab, total, k, static_cast<int>(n), q, qe, me, fin, reach1); break;
            }
        }
        wide |= w;
        if (lane < Q && ((w >> lane) & 1)) at_level = level;
        q = qe;
    }
    auto append = [&](uint32_t mask, SegCount *count, int2 *list, int level) __attribute__((always_inline)) {
        if (!mask) return;
        uint32_t at = 0;
        const int s = blockIdx.x % kSegs;
        if (lane == 0) at = atomicAdd(&count[s].v, static_cast<uint32_t>(__popc(mask)));
        at = uniform(at);
        if (lane < Q && ((mask >> lane) & 1))
            list[seg_size(n) * s + at + __popc(mask & ((1u << lane) - 1))] =
                make_int2(static_cast<int32_t>(r0 + lane), level);
    };
    append(wide, seg_count, seg, at_level);
    append(over, far_count, far, kBits);
    lds_fence();
    constexpr int PER = kWave / Q;   // lanes per query
    const int q = lane / PER;
    const int64_t qid = __float_as_int(__shfl(me.w, q, kWave));
    if (q < nq && !(((wide | over) >> q) & 1)) put_query(sels[wv][q], qid, k, feat, lane % PER, PER, x, y, nbr);
}

// The listed queries, one wavefront per query: the 5 x 5 x 5 cells, from the level that left the query
// undecided to coarser ones while the block has at most kFar points, held in registers.  What stays
// undecided is listed for the streaming scan (a list of the same segment, so that it cannot overflow).
__global__ __launch_bounds__(kBlock, 3) void wide_select_kernel(const Curve *__restrict__ curve,
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
            const int total = gather_cells<2>(c, start, sorted, level, cell, kFar, tab);
            if (total < 0) break;
            // too few of them, the query itself included, unless there are no others
            if (total <= k && block_reach2(c, me, key, level, 2) != __FLT_MAX__) continue;
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
            done = pick_query<B>(picks[wv], d2, id, block_reach2(c, me, key, level, 2), k, static_cast<int>(n), sel);
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

// The queries that the wider scan leaves undecided, one wavefront per query: the 27 cells around it from
// the listed level to coarser ones, streamed through the list as their children (6 x 6 x 6 cells of the next
// finer level; the finest level as it is), the nearest first, until the next is farther than the k-th key.
// Level 0 is the whole cloud, so every query is decided.
__global__ __launch_bounds__(kBlock, 4) void stream_select_kernel(const Curve *__restrict__ curve,
                                                                  const int32_t *__restrict__ start,
                                                                  const f4 *__restrict__ rec,
                                                                  const int32_t *__restrict__ sorted, int64_t n,
                                                                  int k, int feat, const float *__restrict__ x,
                                                                  float *__restrict__ y, int32_t *__restrict__ nbr,
                                                                  const SegCount *__restrict__ seg_count,
                                                                  const int2 *__restrict__ seg) {
    __shared__ Pick picks[kBlock / kWave];
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
        TopK top{picks[wv], k, static_cast<int>(n)};
        const int qid = __float_as_int(me.w);
        for (int level = uniform(e.y);; --level) {
            const int cl = level < kBits ? level + 1 : kBits, W = level < kBits ? 6 : 3;
            const uint32_t m0 = static_cast<uint32_t>(key) >> (3 * (kBits - level));
            const int scale = W / 3, side = 1 << cl;
            const int x0 = scale * (static_cast<int>(gather3(m0)) - 1),
                      y0 = scale * (static_cast<int>(gather3(m0 >> 1)) - 1),
                      z0 = scale * (static_cast<int>(gather3(m0 >> 2)) - 1);
            top.cnt = 0;   // (the bound holds at every level)
            // lane l: children l, l + 64, ... (first record, number of records, distance; taken: +inf)
            constexpr int C = (6 * 6 * 6 + kWave - 1) / kWave;
            uint32_t m[C];
            bool ok[C];
            int b[C], len[C];
            float gap[C];
#pragma unroll
            for (int j = 0; j < C; ++j) {
                const int at = j * kWave + lane;
                const int cx = x0 + at % W, cy = y0 + (at / W) % W, cz = z0 + at / (W * W);
                ok[j] = at < W * W * W && cx >= 0 && cy >= 0 && cz >= 0 && cx < side && cy < side && cz < side;
                m[j] = morton(cx, cy, cz);
                gap[j] = cell_gap2(c, me, cl, cx, cy, cz);
            }
            cell_ranges<C>(c, start, sorted, cl, m, ok, b, len);
#pragma unroll
            for (int j = 0; j < C; ++j) gap[j] = len[j] > 0 ? gap[j] : __builtin_inff();
            while (true) {
                float near = gap[0];
                int nb = b[0], nl = len[0];
#pragma unroll
                for (int j = 1; j < C; ++j) {
                    const bool less = gap[j] < near;
                    near = less ? gap[j] : near;
                    nb = less ? b[j] : nb;
                    nl = less ? len[j] : nl;
                }
                const float best = wave_min(near);
                if (!(best <= top.bound)) break;   // (+inf: none left)
                const int o = __builtin_ctzll(__builtin_amdgcn_ballot_w64(near == best));
                const int ob = __builtin_amdgcn_readlane(nb, o);
#pragma unroll
                for (int j = 0; j < C; ++j) gap[j] = lane == o && b[j] == ob ? __builtin_inff() : gap[j];
                const int oe = ob + __builtin_amdgcn_readlane(nl, o);
                for (int j0 = ob; j0 < oe; j0 += kAhead * kWave) {
                    f4 p[kAhead];
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const int j = j0 + u * kWave + lane;
                        p[u] = j < oe ? rec[j] : me;   // the query itself: left out
                    }
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const int id = __float_as_int(p[u].w);
                        top.offer(sqdist(me, p[u]), id, id != qid);
                    }
                }
                if (top.bound == __FLT_MAX__ || top.cnt > k + 2 * kSpare) top.shrink(k + kSpare);
            }
            // decided if the k-th distance lies within reach, or the block holds every finite point; otherwise on
            // to the first level whose reach covers it
            top.shrink(k);
            const bool some = top.cnt >= k;
            const auto open = [&](int l) __attribute__((always_inline)) {
                const float reach = block_reach2(c, me, key, l, 1);
                return l > 0 && reach != __FLT_MAX__ && !(some && top.bound <= reach);
            };
            if (!open(level)) break;
            while (some && level > 1 && open(level - 1)) --level;
        }
        top.select(sel);
        put_query(sel, qid, k, feat, lane, kWave, x, y, nbr);
    });
}

// ---- small relations: one wavefront per query, no build

// At or below this many points every query scans every point and no relation is built (box, curve keys,
// sort, index): the build's launches and the cell select's dependent chains cost more there than the
// quadratic distance work, on clouds of unequal density above all.  Without the build and with it, k = 16:
// 9,000 points, uniform 57 and 74 us, normal 55 and 128 us; 11,000 points, uniform 73 and 76 us; 12,000 points,
// uniform 84 and 75 us.
constexpr int64_t kBruteMax = 11000;
// For few neighbours, whose cells gain less: 12,000 points, k = 4, without the build and with it, uniform 73 and 70 us, a
// third of them in a clump 88 and 156 us, normal 83 and 121 us.
constexpr int kFewK = 8;
constexpr int64_t kBruteMaxFewK = 12500;
// Up to this many points the queries that the wider scan leaves undecided scan every point too.
constexpr int64_t kBruteFar = 16384;
constexpr int64_t kTreeMax = 7168;   // sums of at most so many points are pairwise trees
constexpr int kBruteWaves = 4;       // queries per block

// Wavefront w of block b takes query q = kBruteWaves b + w; its lanes scan the points 64 at a
// time in input order, with the fp32 distance and the (distance, index) key of the cell select.
// With a list (far_count) the queries are its records.
__global__ __launch_bounds__(kBruteWaves * kWave) void brute_kernel(const float *__restrict__ pos, int64_t n, int k,
                                                                    int feat, const float *__restrict__ x,
                                                                    float *__restrict__ y, int32_t *__restrict__ nbr,
                                                                    const SegCount *__restrict__ far_count,
                                                                    const int2 *__restrict__ far,
                                                                    const f4 *__restrict__ rec) {
    __shared__ Pick picks[kBruteWaves];
    __shared__ int32_t sels[kBruteWaves][kSelRow];
    const int lane = lane_id(), wv = uniform(static_cast<int>(threadIdx.x) / kWave);
    int q = static_cast<int>(blockIdx.x) * kBruteWaves + wv;
    if (q >= n) return;
    if (far_count) {
        // at most n listed queries, one per wavefront
        int64_t listed = -1;
        for_listed(far_count, q, n, [&](int s, int64_t i) { listed = far[seg_size(n) * s + i].x; });
        if (listed < 0) return;
        q = uniform(__float_as_int(rec[listed].w));
    }
    struct P3 {
        float x, y, z;
    };
    const P3 *__restrict__ pts = reinterpret_cast<const P3 *>(pos);
    const P3 mq = pts[q];   // uniform: scalar loads
    const f4 me = f4{mq.x, mq.y, mq.z, 0.0f};
    const int np = static_cast<int>(n);
    int32_t *sel = sels[wv];
    TopK top{picks[wv], k, np};
    if (finite3(me.x, me.y, me.z)) {
        for (int c0 = 0; c0 < np; c0 += kAhead * kWave) {
            P3 p[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int j = c0 + u * kWave + lane;
                p[u] = pts[j < np ? j : q];
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int j = c0 + u * kWave + lane;
                top.offer(sqdist(me, f4{p[u].x, p[u].y, p[u].z, 0.0f}), j, j < np && j != q);
            }
        }
    }
    top.shrink(k);
    top.select(sel);
    if (n > kTreeMax) {
        put_query(sel, q, k, feat, lane, kWave, x, y, nbr);
        return;
    }
    const int32_t j = lane < k ? sel[lane] : -1;
    if (nbr && lane < k) nbr[static_cast<int64_t>(q) * k + lane] = j;
    for (int f = 0; f < feat; ++f) {
        float v = j >= 0 ? x[static_cast<int64_t>(j) * feat + f] : 0.0f;
        // fixed shuffle tree over the lanes (the selected rows in key order, then zeros)
#pragma unroll
        for (int o = kWave / 2; o >= 1; o /= 2) v += __shfl_xor(v, o);
        if (lane == 0) y[static_cast<int64_t>(q) * feat + f] = v;
    }
}

int launch_brute(int64_t n, int k, int feat, const float *pos, const float *x, float *y, int32_t *nbr,
                 hipStream_t stream, const SegCount *far_count = nullptr, const int2 *far = nullptr,
                 const f4 *rec = nullptr) {
    if (!far) prof_before(stream);
    hipLaunchKernelGGL(brute_kernel, dim3(static_cast<unsigned>(ceil_div(n, kBruteWaves))), dim3(kBruteWaves * kWave),
                       0, stream, pos, n, k, feat, x, y, nbr, far_count, far, rec);
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
    if (n <= (k <= kFewK ? kBruteMaxFewK : kBruteMax)) return launch_brute(n, k, feat, pos, x, y, nbr, stream);
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
    const int queries = n < kFewQueries ? 2 : kQueries;
    hipLaunchKernelGGL((n < kFewQueries ? cell_select_kernel<2> : cell_select_kernel<kQueries>),
                       dim3(static_cast<unsigned>(ceil_div(n, queries * (kBlock / kWave)))), dim3(kBlock), 0, stream,
                       w.curve, w.start, w.rec, w.key_sorted, n, k, feat, x, y, nbr, w.seg_count, w.seg,
                       w.seg_count + kSegs, w.far);
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
    if (n <= kBruteFar) return launch_brute(n, k, feat, pos, x, y, nbr, stream, w.seg_count + kSegs, w.far, w.rec);
    const int64_t fb = far_blocks * cus < most ? far_blocks * cus : most;
    hipLaunchKernelGGL(stream_select_kernel, dim3(static_cast<unsigned>(fb)), dim3(kBlock), 0, stream, w.curve,
                       w.start, w.rec, w.key_sorted, n, k, feat, x, y, nbr, w.seg_count + kSegs, w.far);
    return check_launch("kNN streaming select");
}

}  // namespace knn
}  // namespace tiga
