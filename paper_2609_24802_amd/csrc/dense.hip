// Dense all-pairs relation without an edge array (Section 1 of the paper: a
// dense relation may need no edge array), softened inverse-square message:
//   y_i = sum_{j != i} q_j (p_j - p_i) (|p_j - p_i|^2 + eps^2)^(-3/2)
//
// VALU-bound, so the work per pair decides.  Evaluated for one destination, a
// pair takes 13 vector instructions (pairs_kernel); the distance, the reciprocal
// root and its cube serve both directions, so evaluated once for both it takes
// 17, 8.5 per direction (both_kernel).
//
// pairs_kernel (few points): each thread owns one destination i; the j range is
// split into slices (grid.y) so that enough wavefronts are resident, and each
// slice is streamed through LDS in tiles of kTile (p_j, q_j) records.
// both_kernel (kBothMin to kBothMax points): see there.
// The j = i term is exactly zero (zero displacement, eps > 0), so no branch is
// needed.  Summation is two-level (64 terms per inner sum) and partial sums are
// merged in a fixed order, so every output's serial run stays short and results
// do not depend on scheduling.
#include "dense.hpp"

namespace tiga {
namespace dense {

namespace {

constexpr int kBlock = 256;
constexpr int kTile = 256;
constexpr int kInner = 64;

__global__ __launch_bounds__(kBlock) void pack_kernel(const float *__restrict__ pos, const float *__restrict__ q,
                                                      int64_t n, int64_t npad, float4 *__restrict__ pq) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < npad; i += stride) {
        // padding records carry zero charge: they contribute exactly zero
        pq[i] = i < n ? make_float4(pos[i * 3 + 0], pos[i * 3 + 1], pos[i * 3 + 2], q[i])
                      : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
}

__global__ __launch_bounds__(kBlock) void pairs_kernel(const float4 *__restrict__ pq, int64_t n, int64_t slice,
                                                       float eps2, float *__restrict__ part) {
    __shared__ float4 tile[kTile];
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const float4 pi = pq[i < n ? i : 0];
    const int64_t j0 = static_cast<int64_t>(blockIdx.y) * slice;
    const int64_t j1 = j0 + slice;
    float ox = 0.0f, oy = 0.0f, oz = 0.0f;
    for (int64_t jt = j0; jt < j1; jt += kTile) {
        __syncthreads();
        tile[threadIdx.x] = pq[jt + threadIdx.x];
        __syncthreads();
#pragma unroll 1
        for (int jb = 0; jb < kTile; jb += kInner) {
            float ax = 0.0f, ay = 0.0f, az = 0.0f;
#pragma unroll 8
            for (int j = jb; j < jb + kInner; ++j) {
                const float4 pj = tile[j];
                const float dx = pj.x - pi.x;
                const float dy = pj.y - pi.y;
                const float dz = pj.z - pi.z;
                const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, eps2)));
                const float inv = __builtin_amdgcn_rsqf(r2);
                const float s = pj.w * (inv * inv * inv);
                ax = fmaf(s, dx, ax);
                ay = fmaf(s, dy, ay);
                az = fmaf(s, dz, az);
            }
            ox += ax;
            oy += ay;
            oz += az;
        }
    }
    if (i < n) {
        float *o = part + (static_cast<int64_t>(blockIdx.y) * n + i) * 3;
        o[0] = ox;
        o[1] = oy;
        o[2] = oz;
    }
}

__global__ __launch_bounds__(kBlock) void merge_kernel(const float *__restrict__ part, int64_t n, int nsplit,
                                                       float *__restrict__ y) {
    const int64_t k = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (k >= 3 * n) return;
    // pairwise tree over the slices (fixed order)
    float v[64];
    int m = nsplit;
    for (int s = 0; s < m; ++s) v[s] = part[static_cast<int64_t>(s) * 3 * n + k];
    while (m > 1) {
        const int h = (m + 1) / 2;
        for (int s = 0; s + h < m; ++s) v[s] += v[s + h];
        m = h;
    }
    y[k] = v[0];
}

// Both directions of a pair at once.  A block of 4 wavefronts holds kRows = 256 R destinations (R per lane, in
// registers) and walks tiles of 64 points: lane l meets the tile's points in the order l, l + 1, ... (the tile
// lies twice in LDS, so a step's address is the lane's plus a constant), R pairs per step.  The sums of the
// destinations stay in registers; a point's sum travels through the lanes with it, one lane per step (the
// rotation is an operand modifier of the add; LDS atomics instead made the kernel 5 times slower), and after
// the tile the four wavefronts' sums are added and written as the point's partial sum for this block of rows.
//
// Work items are (row block b, tile t) with t at or after the block's own tiles, row by row; a tile of the block
// itself is done one way (every ordered pair inside the block is met).  `per` consecutive items go to one
// block, which writes its rows' sums to slot (block + b) when the row block changes or it ends.  merge_both
// adds a point's row sums over the slots of its row block and subtracts its partial sums of the earlier row
// blocks (the force on the other end is the opposite one).
// Measured, whole calls, one way and both ways: 12,288 points 78 and 69 us, 16,384 124 and 94 us, 32,768 362 and
// 300 us, 65,536 1,208 and 906 us, 262,144 19.1 and
// 13.6 ms.  8,192 points (44 us one way) do not give every compute unit its share of row blocks.
constexpr int kWaves = kBlock / kWave;
constexpr int kJ = kWave;   // points per tile

// Items of the row blocks before b (ntile tiles, rt tiles per row block).
__host__ __device__ inline int64_t items_before(int64_t b, int64_t ntile, int64_t rt) {
    return b * ntile - rt * (b * (b - 1) / 2);
}
// First partial sum (float) of row block b: its row holds 3 x (points from the block's first on).
__host__ __device__ inline int64_t row_offset(int64_t b, int64_t npad, int64_t rows) {
    return 3 * (b * npad - rows * (b * (b - 1) / 2));
}

// The value of lane l + 1 (of lane 0 in lane 63): a whole-wavefront rotation, part of the add that uses it.
__device__ __forceinline__ float from_next(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x134, 0xf, 0xf, false));
}

template <int R>
__global__ __launch_bounds__(kBlock, R == 8 ? 4 : 5) void both_kernel(const float4 *__restrict__ pq, int64_t npad,
                                                                       int64_t ntile, int64_t items, int per,
                                                                       float eps2, float *__restrict__ part_i,
                                                                       float *__restrict__ part_j) {
    constexpr int kRows = kBlock * R, RT = kRows / kJ;
    __shared__ float4 tiles[kWaves][2 * kJ];
    __shared__ float comb[2][kWaves][3][kJ];
    const int lane = lane_id(), w = uniform(static_cast<int>(threadIdx.x) / kWave);
    float4 *tile = tiles[w];
    int64_t u = static_cast<int64_t>(blockIdx.x) * per;
    const int64_t end = u + per < items ? u + per : items;
    if (u >= end) return;
    int64_t b = 0;
    while (items_before(b + 1, ntile, RT) <= u) ++b;
    int flip = 0;
    while (u < end) {
        const int64_t row_end = items_before(b + 1, ntile, RT) < end ? items_before(b + 1, ntile, RT) : end;
        float4 pi[R];
        float o[R][3];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            pi[r] = pq[b * kRows + w * (R * kWave) + r * kWave + lane];
            o[r][0] = o[r][1] = o[r][2] = 0.0f;
        }
        int64_t t = b * RT + (u - items_before(b, ntile, RT));
        float4 nxt = pq[t * kJ + lane];
        for (; u < row_end; ++u, ++t) {
            // the tile and its sums are this wavefront's alone: its LDS operations stay in order
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            tile[lane] = nxt;
            tile[lane + kJ] = nxt;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (u + 1 < row_end) nxt = pq[(t + 1) * kJ + lane];
            const bool both = t >= (b + 1) * RT;   // the same for the whole block
            float a[R][3];
#pragma unroll
            for (int r = 0; r < R; ++r) a[r][0] = a[r][1] = a[r][2] = 0.0f;
            if (both) {
                float f[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll 2
                for (int s = 0; s < kJ; ++s) {
                    const float4 pj = tile[lane + s];
                    float gx = 0.0f, gy = 0.0f, gz = 0.0f;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const float dx = pj.x - pi[r].x, dy = pj.y - pi[r].y, dz = pj.z - pi[r].z;
                        const float inv = __builtin_amdgcn_rsqf(fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, eps2))));
                        const float inv3 = inv * inv * inv;
                        const float si = pj.w * inv3, sj = pi[r].w * inv3;
                        a[r][0] = fmaf(si, dx, a[r][0]);
                        a[r][1] = fmaf(si, dy, a[r][1]);
                        a[r][2] = fmaf(si, dz, a[r][2]);
                        gx = fmaf(sj, dx, gx);
                        gy = fmaf(sj, dy, gy);
                        gz = fmaf(sj, dz, gz);
                    }
                    // the point's sum comes from lane l + 1, which met the point one step earlier
                    f[0] = from_next(f[0]) + gx;
                    f[1] = from_next(f[1]) + gy;
                    f[2] = from_next(f[2]) + gz;
                }
                // after 64 steps lane l holds the sum of point l - 1
#pragma unroll
                for (int c = 0; c < 3; ++c) comb[flip][w][c][lane] = from_next(f[c]);
                __syncthreads();
                // the next tile writes the other half of comb, and only after this barrier's successor the same one
                if (w < 3) {
                    float v = comb[flip][0][w][lane];
#pragma unroll
                    for (int k = 1; k < kWaves; ++k) v += comb[flip][k][w][lane];
                    const int64_t len = npad - b * kRows;
                    part_j[row_offset(b, npad, kRows) + w * len + (t * kJ - b * kRows) + lane] = v;
                }
                flip ^= 1;
            } else {
#pragma unroll 2
                for (int s = 0; s < kJ; ++s) {
                    const float4 pj = tile[s];
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const float dx = pj.x - pi[r].x, dy = pj.y - pi[r].y, dz = pj.z - pi[r].z;
                        const float inv = __builtin_amdgcn_rsqf(fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, eps2))));
                        const float si = pj.w * (inv * inv * inv);
                        a[r][0] = fmaf(si, dx, a[r][0]);
                        a[r][1] = fmaf(si, dy, a[r][1]);
                        a[r][2] = fmaf(si, dz, a[r][2]);
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int c = 0; c < 3; ++c) o[r][c] += a[r][c];
        }
        float *out = part_i + (static_cast<int64_t>(blockIdx.x) + b) * (3 * kRows);
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c) out[c * kRows + w * (R * kWave) + r * kWave + lane] = o[r][c];
        ++b;
    }
}

// y of point i, component c = blockIdx.y: the partial sums in a fixed order, in 64 bits (a few hundred terms).
__global__ __launch_bounds__(kBlock) void merge_both_kernel(const float *__restrict__ part_i,
                                                            const float *__restrict__ part_j, int64_t n, int64_t npad,
                                                            int64_t ntile, int rows, int per, float *__restrict__ y) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= n) return;
    const int c = blockIdx.y;
    const int64_t b = i / rows, rt = rows / kJ;   // rows is a multiple of kBlock: b is the same for the block
    double v = 0.0;
    const int64_t g0 = items_before(b, ntile, rt) / per, g1 = (items_before(b + 1, ntile, rt) - 1) / per;
    const float *pi = part_i + (g0 + b) * (3 * rows) + c * static_cast<int64_t>(rows) + (i - b * rows);
#pragma unroll 4
    for (int64_t g = g0; g <= g1; ++g, pi += 3 * rows) v += *pi;
#pragma unroll 4
    for (int64_t a = 0; a < b; ++a)
        v -= part_j[row_offset(a, npad, rows) + c * (npad - a * rows) + (i - a * rows)];
    y[i * 3 + c] = static_cast<float>(v);
}

int64_t padded(int64_t n, int64_t unit) { return ceil_div(n > 0 ? n : 1, unit) * unit; }

int splits_for(int64_t n) {
    // enough wavefronts to fill the chip, at least one tile per slice, at most 64
    const int64_t tiles = padded(n, kTile) / kTile;
    int64_t want = ceil_div(static_cast<int64_t>(device_cus()) * 64, ceil_div(n, kBlock) * (kBlock / kWave));
    if (want < 1) want = 1;
    if (want > 64) want = 64;
    if (want > tiles) want = tiles;
    // slices must be whole tiles
    while (tiles % want) --want;
    return static_cast<int>(want);
}

// Both directions at once from kBothMin points on, below which the row blocks are too few to share out evenly,
// up to kBothMax, above which the partial sums (n^2 / 4096 x 12 bytes) outgrow the slices' (768 n bytes); 8
// destinations per lane from kBothWide on, 4 below (more, smaller items).
constexpr int64_t kBothMin = 12288;
constexpr int64_t kBothWide = 40960;
constexpr int64_t kBothMax = int64_t{1} << 18;

bool use_both(int64_t n) { return n >= kBothMin && n <= kBothMax; }

// The division of the work of both_kernel: rows per block, items, items per block, blocks.
struct Both {
    int R, rows;
    int64_t npad, ntile, nb, items;
    int per;
    int64_t most, grid;   // blocks: bound, and how many are launched
};

Both both_for(int64_t n) {
    Both s;
    s.R = n >= kBothWide ? 8 : 4;
    s.rows = kBlock * s.R;
    s.npad = padded(n, s.rows);
    s.ntile = s.npad / kJ;
    s.nb = s.npad / s.rows;
    s.items = items_before(s.nb, s.ntile, s.rows / kJ);
    // four blocks per compute unit, each the same number of items
    s.most = 4 * static_cast<int64_t>(device_cus());
    s.per = static_cast<int>(ceil_div(s.items, s.most));
    s.grid = ceil_div(s.items, s.per);
    return s;
}

struct Ws {
    float4 *pq;
    float *part;     // slices, or the row sums
    float *part_j;
};

Ws carve(Carve &c, int64_t n, int nsplit) {
    Ws w;
    w.pq = c.take<float4>(padded(n, kTile));
    w.part = c.take<float>(static_cast<size_t>(nsplit) * 3 * n);
    w.part_j = nullptr;
    return w;
}

Ws carve(Carve &c, const Both &s) {
    Ws w;
    w.pq = c.take<float4>(s.npad);
    // for the most blocks: `grid` falls and rises with n, the workspace must not
    w.part = c.take<float>((s.most + s.nb) * 3 * s.rows);
    w.part_j = c.take<float>(row_offset(s.nb, s.npad, s.rows));
    return w;
}

int pack(int64_t n, int64_t npad, const float *pos, const float *q, float4 *pq, hipStream_t stream) {
    hipLaunchKernelGGL(pack_kernel, dim3(static_cast<unsigned>(ceil_div(npad, kBlock))), dim3(kBlock), 0, stream, pos,
                       q, n, npad, pq);
    return check_launch("dense pack");
}

int forward_both(int64_t n, const float *pos, const float *q, float eps2, float *y, void *ws, hipStream_t stream) {
    const Both s = both_for(n);
    Carve c(ws);
    const Ws w = carve(c, s);
    if (int rc = pack(n, s.npad, pos, q, w.pq, stream)) return rc;
    prof_before(stream);
    if (s.R == 8)
        hipLaunchKernelGGL(both_kernel<8>, dim3(static_cast<unsigned>(s.grid)), dim3(kBlock), 0, stream, w.pq, s.npad,
                           s.ntile, s.items, s.per, eps2, w.part, w.part_j);
    else
        hipLaunchKernelGGL(both_kernel<4>, dim3(static_cast<unsigned>(s.grid)), dim3(kBlock), 0, stream, w.pq, s.npad,
                           s.ntile, s.items, s.per, eps2, w.part, w.part_j);
    prof_after(stream);
    if (int rc = check_launch("dense pairs")) return rc;
    hipLaunchKernelGGL(merge_both_kernel, dim3(static_cast<unsigned>(ceil_div(n, kBlock)), 3), dim3(kBlock), 0, stream,
                       w.part, w.part_j, n, s.npad, s.ntile, s.rows, s.per, y);
    return check_launch("dense merge");
}

}  // namespace

size_t workspace_bytes(int64_t n) {
    Carve c(nullptr);
    if (use_both(n)) carve(c, both_for(n));
    else carve(c, n, 64);
    // a workspace for n points holds every smaller problem, so above kBothMax no less than at kBothMax
    if (n <= kBothMax) return c.bytes();
    const size_t least = workspace_bytes(kBothMax);
    return c.bytes() > least ? c.bytes() : least;
}

int forward(int64_t n, const float *pos, const float *q, float eps, float *y, void *ws, hipStream_t stream) {
    if (use_both(n)) return forward_both(n, pos, q, eps * eps, y, ws, stream);
    const int nsplit = splits_for(n);
    Carve c(ws);
    Ws w = carve(c, n, nsplit);
    const int64_t npad = padded(n, kTile);
    if (int rc = pack(n, npad, pos, q, w.pq, stream)) return rc;
    const int64_t slice = npad / nsplit;
    const dim3 grid(static_cast<unsigned>(ceil_div(n, kBlock)), static_cast<unsigned>(nsplit));
    prof_before(stream);
    hipLaunchKernelGGL(pairs_kernel, grid, dim3(kBlock), 0, stream, w.pq, n, slice, eps * eps, w.part);
    prof_after(stream);
    if (int rc = check_launch("dense pairs")) return rc;
    hipLaunchKernelGGL(merge_kernel, dim3(static_cast<unsigned>(ceil_div(3 * n, kBlock))), dim3(kBlock), 0, stream,
                       w.part, n, nsplit, y);
    return check_launch("dense merge");
}

}  // namespace dense
}  // namespace tiga
