// Radius relation, tiles of 16 destinations.
//
// A wavefront owns 16 consecutive cell-ordered points.  Lane (g, m), g = lane / 16, m = lane % 16, tests
// destination m against the candidates of its group g, so the 16 destinations share every candidate row and
// no list of accepted pairs is built:
//   - the points of a tile that lie in one x-row of cells, with no more than kGap cells from one to the next, form
//     a segment (nearly always the whole tile; a tile that crosses the end of a row has two); the segment's
//     candidates are the 9 runs of cells around its x-range, all of them in cells next to a point's;
//   - a candidate is kept (LDS list: position, byte offset of its feature row) when the box of the segment's
//     destinations is within the radius of it: 205 of 331 (1M uniform points of degree 32, cells of the
//     radius).  The box distance is formed with the predicate's own operations, and every rounding is
//     monotone, so no accepted pair is dropped;
//   - each lane evaluates the exact predicate and the weight of its pairs (0 if rejected), which is the A
//     operand of v_mfma_f32_16x16x4_f32 as it stands: the weighted sum over candidates is a matrix product
//     with the candidates' rows (read in place, 16 lanes on one row) on the matrix cores, in fp32.  Rows of
//     one or two features are summed by the vector units instead, from values kept in LDS.
//   - Backward: dx is the same product with dy; the inner products <dy_i, x_j> + <dy_j, x_i> of the tile
//     with 16 candidates are two more products, whose result has lane (g, m) hold its own pairs' values.
// The matrix product also multiplies rejected pairs' rows by zero, which a non-finite row would turn into
// NaN: a tile with a non-finite result is evaluated again pair by pair (slow_*), so results are those of the
// accepted pairs alone.
//
// The kernels are bound by VALU issue: fp32 matrix products share it (their cycles and the vector units' add up
// to the kernel's time), at twice the rate of plain fused multiply-adds.  Per 16 candidates a wavefront issues 53
// vector and 8 matrix instructions (forward, 32 features).
// Measured against the previous kernels, which tested one cell's destinations in turn and appended accepted pairs
// to LDS lists (kept for wider rows): 1M uniform points, mean degree 31, 32 features 345 -> 281 us forward and
// 810 -> 737 us backward; 131,072 points, 1 feature 50 -> 25 us; 300,000 points of a normal cloud (whole calls,
// 32 features) 1,771 -> 215 us and 2,376 -> 374 us, since a dense cell is now many wavefronts' work.
#include "radius_tile.hpp"

namespace tiga {
namespace radius {

namespace {

constexpr int kBlock = 256;
constexpr int kTile = 16;
constexpr int kList = 256;   // candidates between two passes
// Cells from one point of a segment to the next, at most: the runs around them then leave no cell between.  Without
// this bound the few points of a sparse row of cells had a dense row beside it for candidates, whole: 1M points on
// a line, 16 of them one cell beside it, forward of 1 and 32 features 18 and 27 ms, now 0.18 and 0.25 ms (lists that
// test cell by cell: 0.31 and 0.36 ms).
constexpr int kGap = 3;

struct alignas(16) Work {
    f32x4 list[kList];       // x, y, z, byte offset of the row (bits)
};

__device__ __forceinline__ void lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

template <int CTRL>
__device__ __forceinline__ float row_rot(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
// Minimum over the 16 lanes of a row, in every lane (row rotations by 8, 4, 2, 1).
__device__ __forceinline__ float row_min(float v) {
    v = fminf(v, row_rot<0x128>(v));
    v = fminf(v, row_rot<0x124>(v));
    v = fminf(v, row_rot<0x122>(v));
    return fminf(v, row_rot<0x121>(v));
}

__device__ __forceinline__ bool finite(float v) { return __builtin_fabsf(v) <= __FLT_MAX__; }

// Destination of this lane: position, whether it belongs to the segment.
struct Dst {
    float x, y, z;
    bool in;
};

// Predicate and weight of one pair of distinct points; also the differences (for the position gradient).
__device__ __forceinline__ float weight(const Dst &d, f32x4 e, float r2, float nis, float (&diff)[3], bool &near) {
#pragma clang fp contract(off)
    diff[0] = e.x - d.x;
    diff[1] = e.y - d.y;
    diff[2] = e.z - d.z;
    const float sx = diff[0] * diff[0], sy = diff[1] * diff[1], sz = diff[2] * diff[2];
    const float d2 = (sx + sy) + sz;
    near = d2 < r2 && d.in;
    const float k = __builtin_amdgcn_exp2f(d2 * nis);
    return near ? k : 0.0f;
}

// Visit the candidates of every segment of the tile whose first record is s0: pass(cnt, own) is called with
// up to kList candidates in wk.list, whose entries up to the next multiple of 16 repeat one of them (the
// pass masks them).  The tile's own points come first, as a list of their own (own: entry m is destination
// m, a pair that the pass leaves out), so that no other pair needs the test for the point itself.
// keep(slot, offset) is called by the lane that stores a candidate.
template <class Keep, class Pass>
__device__ __forceinline__ void for_tile(const Params &p, const int64_t *__restrict__ start,
                                         const f32x4 *__restrict__ rec, const int32_t *__restrict__ cells, int64_t n,
                                         int64_t s0, uint32_t row_bytes, float r2, Work &wk, Dst &dst, int32_t &id,
                                         Keep &&keep, Pass &&pass) {
    const int lane = lane_id(), m = lane % kTile;
    const bool valid = s0 + m < n;
    const f32x4 me = rec[valid ? s0 + m : s0];
    const int32_t cell = cells[valid ? s0 + m : s0];
    id = valid ? __float_as_int(me.w) : -1;
    dst.x = me.x;
    dst.y = me.y;
    dst.z = me.z;
    // the tile's own points among themselves
    const uint32_t own_off = static_cast<uint32_t>(__float_as_int(me.w)) * row_bytes;
    if (lane < kTile) {
        wk.list[lane] = f32x4{me.x, me.y, me.z, __uint_as_float(own_off)};
        keep(lane, own_off);
    }
    lds_fence();
    dst.in = valid;
    pass(static_cast<int>(n - s0 < kTile ? n - s0 : kTile), std::true_type{});
    lds_fence();
    const uint32_t dx = p.dim[0], dy = p.dim[1], ucell = cell;   // unsigned divisions are the shorter ones
    // cells ascend along the tile: bit m of `ends` where point m is a segment's last
    const uint32_t all = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(valid)) & 0xffffu;
    const int step = __builtin_amdgcn_update_dpp(0, cell, 0x101, 0xf, 0xf, true) - cell;   // of lane m + 1's cell
    const bool last = step > kGap || static_cast<int>(ucell % dx) + step >= p.dim[0];
    const uint32_t ends = (static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(last)) | ~(all >> 1)) & all;
    uint32_t todo = all;
    const float inf = __builtin_inff();
    while (todo) {
        const int f = __builtin_ctz(todo), l = __builtin_ctz(todo & ends);
        const int first_cell = __builtin_amdgcn_readlane(cell, f), srow = static_cast<uint32_t>(first_cell) / dx;
        dst.in = m >= f && m <= l;
        todo &= ~0u << (l + 1);
        // the segment's x-range, one cell more on each side
        const int x0 = first_cell - srow * p.dim[0], x1 = x0 + (__builtin_amdgcn_readlane(cell, l) - first_cell);
        const int xa = x0 > 0 ? x0 - 1 : 0, xb = x1 + 1 < p.dim[0] ? x1 + 1 : p.dim[0] - 1;
        const int cz = static_cast<uint32_t>(srow) / dy, cy = srow - cz * p.dim[1];
        // box of the segment's destinations (records of non-finite points are all +inf: within the radius of
        // nothing)
        const bool box = dst.in && finite(dst.x);
        const float lx = row_min(box ? dst.x : inf), ly = row_min(box ? dst.y : inf), lz = row_min(box ? dst.z : inf);
        const float hx = -row_min(box ? -dst.x : inf), hy = -row_min(box ? -dst.y : inf),
                    hz = -row_min(box ? -dst.z : inf);
        // lanes 0..8: the runs (z, y) of the neighbourhood
        int32_t first = 0, len = 0;
        if (lane < 9) {
            const int z = cz - 1 + lane / 3, y = cy - 1 + lane % 3;
            if (z >= 0 && z < p.dim[2] && y >= 0 && y < p.dim[1]) {
                const int64_t rowc = (static_cast<int64_t>(z) * p.dim[1] + y) * p.dim[0];
                first = static_cast<int32_t>(start[rowc + xa]);
                len = static_cast<int32_t>(start[rowc + xb + 1]) - first;
            }
        }
        int cnt = 0;
        // run the pass on the list, filled up to a multiple of 16 with its first candidate
        auto flush = [&]() __attribute__((always_inline)) {
            lds_fence();
            const int pad = (kTile - cnt % kTile) % kTile;
            const f32x4 e = wk.list[0];
            if (lane < pad) {
                wk.list[cnt + lane] = e;
                keep(cnt + lane, __float_as_uint(e.w));
            }
            lds_fence();
            pass(cnt, std::false_type{});
            lds_fence();
            cnt = 0;
        };
        // keep the lanes' candidates `e` (records t) that the box is within the radius of
        auto offer = [&](f32x4 e, int32_t t, bool live) __attribute__((always_inline)) {
            bool take;
            {
#pragma clang fp contract(off)
                const float gx = fmaxf(fmaxf(lx - e.x, e.x - hx), 0.0f), gy = fmaxf(fmaxf(ly - e.y, e.y - hy), 0.0f),
                            gz = fmaxf(fmaxf(lz - e.z, e.z - hz), 0.0f);
                const float sx = gx * gx, sy = gy * gy, sz = gz * gz;
                take = (sx + sy) + sz < r2 && live && static_cast<uint32_t>(t - static_cast<int32_t>(s0)) >= kTile;
            }
            const uint64_t mask = __builtin_amdgcn_ballot_w64(take);
            const int nnew = __popcll(mask);
            if (cnt + nnew > kList) flush();
            if (take) {
                const int slot = cnt + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                                                 __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0));
                const uint32_t ro = static_cast<uint32_t>(__float_as_int(e.w)) * row_bytes;
                wk.list[slot] = f32x4{e.x, e.y, e.z, __uint_as_float(ro)};
                keep(slot, ro);
            }
            cnt += nnew;
        };
        // three runs at a time (one z), their first 64 records loaded together.  (One loop over steps of 64
        // with a single copy of the pass has a third of the code, but is slower: 34 against 27 us for 131,072
        // points and 1 feature, 272 against 262 us for 1M points and 32 features.)
#pragma unroll 1
        for (int k = 0; k < 9; k += 3) {
            int32_t fk[3], lk[3];
            f32x4 e[3];
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                fk[u] = __builtin_amdgcn_readlane(first, k + u);
                lk[u] = __builtin_amdgcn_readlane(len, k + u);
                e[u] = rec[lane < lk[u] ? fk[u] + lane : static_cast<int32_t>(s0)];
            }
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                if (lk[u] == 0) continue;
                offer(e[u], fk[u] + lane, lane < lk[u]);
                for (int j = kWave; j < lk[u]; j += kWave) {
                    const bool live = j + lane < lk[u];
                    const int32_t t = live ? fk[u] + j + lane : static_cast<int32_t>(s0);
                    offer(rec[t], t, live);
                }
            }
        }
        if (cnt > 0) flush();
    }
}

// T at a byte offset; rows of any width need only be aligned to their floats (the memory unit takes wider
// loads and stores at 4-byte addresses).
template <class T>
__device__ __forceinline__ void put_bytes(float *p, T v) {
    __builtin_memcpy(p, &v, sizeof(T));
}
template <class T>
__device__ __forceinline__ T at_bytes(const float *__restrict__ base, uint32_t off) {
    T v;
    __builtin_memcpy(&v, reinterpret_cast<const char *>(base) + off, sizeof(T));
    return v;
}

// Accepted candidates of record s, in candidate order: each(offset of the row, weight, differences), the
// arguments uniform over the wavefront.
template <class Each>
__device__ void slow_row(const Params &p, const int64_t *__restrict__ start, const f32x4 *__restrict__ rec, int64_t s,
                         uint32_t row_bytes, float r2, float nis, Each &&each) {
    const f32x4 me = rec[s];
    const Dst d{me.x, me.y, me.z, true};
    for_runs(p, start, make_float4(me.x, me.y, me.z, me.w), [&](int64_t b, int64_t e) {
        for (int64_t c0 = b; c0 < e; c0 += kWave) {
            const int64_t t = c0 + lane_id() < e ? c0 + lane_id() : s;   // past the end: the point itself
            f32x4 c = rec[t];
            c.w = __uint_as_float(static_cast<uint32_t>(__float_as_int(c.w)) * row_bytes);
            float diff[3];
            bool near;
            const float w = weight(d, c, r2, nis, diff, near);
            for (uint64_t mask = __builtin_amdgcn_ballot_w64(near && t != s); mask; mask &= mask - 1) {
                const int l = __builtin_ctzll(mask);
                const float dl[3] = {__shfl(diff[0], l), __shfl(diff[1], l), __shfl(diff[2], l)};
                each(static_cast<uint32_t>(__builtin_amdgcn_readlane(__float_as_int(c.w), l)), __shfl(w, l), dl);
            }
        }
    });
}

// Weighted sums over the candidates as matrix products, NB blocks of 16 features.  Each of a lane group's four
// candidates per step has accumulators of its own (NB = 1; the even and the odd ones otherwise, where more would cost a
// wavefront per SIMD), which are added in 64 bits.  Distance from 64 bits (norms of difference and result), 31
// neighbours, 16 and 32 features: 8.1e-8 and 9.8e-8, in one run of roundings 1.21e-7, as trees over lane groups (the
// lists' sums) 9.1e-8 and 1.10e-7.  Times before and now, 1M points of degree 32: 16 features 272 and 287 us, 32
// features 358 and 361 us (whole calls).
template <int NB>
struct Sums {
    static constexpr int A = NB == 1 ? 4 : 2;
    f32x4 a[A][NB];
    __device__ __forceinline__ Sums() {
#pragma unroll
        for (int i = 0; i < A; ++i)
#pragma unroll
            for (int b = 0; b < NB; ++b) a[i][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    __device__ __forceinline__ void add(int s, float w, const float (&v)[NB]) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
            a[s % A][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, v[b], a[s % A][b], 0, 0, 0);
    }
    // whether all are finite
    __device__ __forceinline__ bool total(f32x4 (&out)[NB]) const {
        bool ok = true;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double v = static_cast<double>(a[0][b][r]) + a[1][b][r];
                if constexpr (A == 4) v += static_cast<double>(a[2][b][r]) + a[3][b][r];
                out[b][r] = static_cast<float>(v);
                ok &= finite(out[b][r]);
            }
        }
        return ok;
    }
};

// Forward.  NB = 0: rows of SF features, summed by the vector units.  NB > 0: NB blocks of 16 features;
// lane m holds the features NB m .. NB m + NB - 1 of a row in one load (VEC: feat a multiple of NB), or the
// features m, m + 16, ... (any feat).
template <int NB, int SF, bool VEC, bool CNT>
__global__ __launch_bounds__(kBlock, NB == 0 && SF == 1 ? 8 : 1)   // one feature: 8 wavefronts per SIMD hide its loads
    void tile_fwd_kernel(const Params *__restrict__ prm,
                                                          const int64_t *__restrict__ start,
                                                          const f32x4 *__restrict__ rec,
                                                          const int32_t *__restrict__ cells, int64_t n, int feat,
                                                          const float *__restrict__ x, float r2, float nis,
                                                          float *__restrict__ y, int32_t *__restrict__ count) {
    constexpr int W = kBlock / kWave, AB = NB > 0 ? NB : 1, AS = NB == 0 ? SF : 1;
    __shared__ Work works[W];
    __shared__ float vals[NB == 0 ? W : 1][AS][NB == 0 ? kList : 1];   // NB = 0: the candidates' features
    const int wv = uniform(static_cast<int>(threadIdx.x) / kWave), lane = lane_id(), m = lane % kTile, g = lane / kTile;
    const int64_t s0 = (static_cast<int64_t>(xcd_block()) * W + wv) * kTile;
    if (s0 >= n) return;
    const Params p = *prm;
    Work &wk = works[wv];
    const uint32_t row_bytes = static_cast<uint32_t>(feat) * 4;
    // byte offsets of this lane's features in a row (past the end: the last one, whose sums are not stored)
    uint32_t fo[AB];
#pragma unroll
    for (int b = 0; b < AB; ++b) {
        const int f = VEC ? NB * m : m + 16 * b;
        fo[b] = static_cast<uint32_t>(f < feat ? f : (VEC ? feat - NB : feat - 1)) * 4;
    }
    Sums<AB> acc;
    float sum[AS][2];   // like acc
#pragma unroll
    for (int f = 0; f < AS; ++f) sum[f][0] = sum[f][1] = 0.0f;
    int deg = 0;
    Dst dst;
    int32_t id;
    auto keep = [&](int slot, uint32_t off) __attribute__((always_inline)) {
        if constexpr (NB == 0) {
#pragma unroll
            for (int f = 0; f < AS; ++f) vals[wv][f][slot] = at_bytes<float>(x, off + 4 * f);
        }
    };
    auto pass = [&](int cnt, auto own) __attribute__((always_inline)) {
        auto step = [&](int j, auto full) __attribute__((always_inline)) {
            constexpr bool FULL = decltype(full)::value;
            f32x4 e[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) e[s] = wk.list[j + 4 * g + s];
            float xv[4][AB];
            if constexpr (NB > 0) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const uint32_t ro = __float_as_uint(e[s].w);
                    if constexpr (VEC && NB == 2) {
                        const float2 t = at_bytes<float2>(x, ro + fo[0]);
                        xv[s][0] = t.x, xv[s][1] = t.y;
                    } else if constexpr (VEC && NB == 4) {
                        const float4 t = at_bytes<float4>(x, ro + fo[0]);
                        xv[s][0] = t.x, xv[s][1] = t.y, xv[s][2] = t.z, xv[s][3] = t.w;
                    } else {
#pragma unroll
                        for (int b = 0; b < NB; ++b) xv[s][b] = at_bytes<float>(x, ro + fo[b]);
                    }
                }
            }
            float w[4];
            bool near[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                float diff[3];
                w[s] = weight(dst, e[s], r2, nis, diff, near[s]);
                const int i = j + 4 * g + s;
                if (!FULL && (i >= cnt || (own && i == m))) w[s] = 0.0f, near[s] = false;
                if (CNT) deg += near[s];
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if constexpr (NB > 0) {
                    acc.add(s, w[s], xv[s]);
                } else {
#pragma unroll
                    for (int f = 0; f < AS; ++f)
                        if (near[s]) sum[f][s & 1] = fmaf(w[s], vals[wv][f][j + 4 * g + s], sum[f][s & 1]);
                }
            }
        };
        int j = 0;
        if constexpr (!own)
            for (; j + kTile <= cnt; j += kTile) step(j, std::true_type{});
        if (j < cnt) step(j, std::false_type{});
    };
    for_tile(p, start, rec, cells, n, s0, row_bytes, r2, wk, dst, id, keep, pass);
    if constexpr (CNT) {
        deg += shfl_xor_i(deg, 16);
        deg += shfl_xor_i(deg, 32);
        if (lane < kTile && id >= 0) count[id] = deg;
    }
    if constexpr (NB == 0) {
#pragma unroll
        for (int f = 0; f < AS; ++f) {
            double v = static_cast<double>(sum[f][0]) + sum[f][1];
            v += __shfl_xor(v, 16, kWave);
            v += __shfl_xor(v, 32, kWave);
            if (lane < kTile && id >= 0) y[static_cast<int64_t>(id) * AS + f] = static_cast<float>(v);
        }
    } else {
        f32x4 out[AB];
        if (__any(!acc.total(out))) {
            for (int64_t s = s0; s < s0 + kTile && s < n; ++s) {
                float a = 0.0f;
                slow_row(p, start, rec, s, row_bytes, r2, nis, [&](uint32_t off, float w, const float (&)[3]) {
                    if (lane < feat) a = fmaf(w, at_bytes<float>(x, off + 4 * lane), a);
                });
                if (lane < feat) y[static_cast<int64_t>(__float_as_int(rec[s].w)) * feat + lane] = a;
            }
            return;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t row = __shfl(id, 4 * g + r, kWave);
            if (row < 0) continue;
            float *o = y + row * feat;
            if constexpr (VEC && NB == 2) {
                if (2 * m < feat) put_bytes(o + 2 * m, make_float2(out[0][r], out[1][r]));
            } else if constexpr (VEC && NB == 4) {
                if (4 * m < feat) put_bytes(o + 4 * m, make_float4(out[0][r], out[1][r], out[2][r], out[3][r]));
            } else {
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    if (m + 16 * b < feat) o[m + 16 * b] = out[b][r];
            }
        }
    }
}

template <int KS>
__device__ __forceinline__ void load_part(const float *__restrict__ base, uint32_t off, float (&v)[KS]) {
    struct Part {
        float v[KS];
    };
    const Part t = at_bytes<Part>(base, off);
#pragma unroll
    for (int k = 0; k < KS; ++k) v[k] = t.v[k];
}

// Backward.  The inner products run over 4 KS >= feat features: lane group g takes KS features from KS g on,
// in one load; where those would pass the row's end it takes the row's last KS, and the destinations' operand
// is 0 for the features that another group has (KS <= feat).  dx is summed in NB blocks of 16 features (PAIR:
// even feat, two adjacent features per lane).
// Wavefronts per SIMD are asked for where the accumulators would cost one (1M points, 32 features, whole calls: 707 us
// with the 4, 793 us with 3; 16 features spill with 5: 510 us, 468 us with 4).
template <int KS, bool PAIR, bool DX, bool DP>
__global__ __launch_bounds__(kBlock, DX && DP ? (KS >= 4 ? 4 : 5) : 1) void tile_bwd_kernel(const Params *__restrict__ prm,
                                                          const int64_t *__restrict__ start,
                                                          const f32x4 *__restrict__ rec,
                                                          const int32_t *__restrict__ cells, int64_t n, int feat,
                                                          const float *__restrict__ x, const float *__restrict__ dy,
                                                          float r2, float nis, float tis, float *__restrict__ dx,
                                                          float *__restrict__ dp) {
    constexpr int W = kBlock / kWave, NB = KS > 4 ? 2 : 1;
    __shared__ Work works[W];
    const int wv = uniform(static_cast<int>(threadIdx.x) / kWave), lane = lane_id(), m = lane % kTile, g = lane / kTile;
    const int64_t s0 = (static_cast<int64_t>(xcd_block()) * W + wv) * kTile;
    if (s0 >= n) return;
    const Params p = *prm;
    Work &wk = works[wv];
    const uint32_t row_bytes = static_cast<uint32_t>(feat) * 4;
    uint32_t fo[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int f = PAIR ? 2 * m : m + 16 * b;
        fo[b] = static_cast<uint32_t>(f < feat ? f : (PAIR ? feat - 2 : feat - 1)) * 4;
    }
    const int part = KS * g + KS <= feat ? KS * g : feat - KS;   // this group's first feature
    Sums<NB> acc;
    float gp[3] = {0.0f, 0.0f, 0.0f};
    // the destinations' rows, as operands of the inner products
    float yi[KS], xi[KS];
    if constexpr (DP) {
        const int64_t s = s0 + m < n ? s0 + m : s0;
        const uint32_t off = static_cast<uint32_t>(__float_as_int(rec[s].w)) * row_bytes;
        load_part<KS>(dy, off + 4 * part, yi);
        load_part<KS>(x, off + 4 * part, xi);
#pragma unroll
        for (int t = 0; t < KS; ++t)
            if (part + t < KS * g) yi[t] = xi[t] = 0.0f;
    }
    Dst dst;
    int32_t id;
    auto pass = [&](int cnt, auto own) __attribute__((always_inline)) {
        auto step = [&](int j, auto full) __attribute__((always_inline)) {
            constexpr bool FULL = decltype(full)::value;
            f32x4 e[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) e[s] = wk.list[j + 4 * g + s];
            float xj[KS], yj[KS];
            if constexpr (DP) {
                const uint32_t off = __float_as_uint(wk.list[j + m].w);
                load_part<KS>(x, off + 4 * part, xj);
                load_part<KS>(dy, off + 4 * part, yj);
            }
            float gv[4][NB];
            if constexpr (DX) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const uint32_t ro = __float_as_uint(e[s].w);
                    if constexpr (PAIR) {
                        const float2 t = at_bytes<float2>(dy, ro + fo[0]);
                        gv[s][0] = t.x, gv[s][1] = t.y;
                    } else {
#pragma unroll
                        for (int b = 0; b < NB; ++b) gv[s][b] = at_bytes<float>(dy, ro + fo[b]);
                    }
                }
            }
            float w[4], diff[4][3];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                bool near;
                w[s] = weight(dst, e[s], r2, nis, diff[s], near);
                const int i = j + 4 * g + s;
                if (!FULL && (i >= cnt || (own && i == m))) w[s] = 0.0f;
            }
            if constexpr (DP) {
                // both products of 4 features add to the same accumulator, of several for shorter runs of roundings:
                // the position gradient of 32 features ends 1.38e-7 from 64 bits, 1.50e-7 with two accumulators (the
                // lists: 1.45e-7); a fourth costs 3% of the time
                constexpr int A = KS == 8 ? 3 : KS;
                f32x4 a[A];
#pragma unroll
                for (int t = 0; t < KS; ++t) {
                    const f32x4 c = t < A ? f32x4{0.0f, 0.0f, 0.0f, 0.0f} : a[t % A];
                    a[t % A] = __builtin_amdgcn_mfma_f32_16x16x4f32(xj[t], yi[t], c, 0, 0, 0);
                    a[t % A] = __builtin_amdgcn_mfma_f32_16x16x4f32(yj[t], xi[t], a[t % A], 0, 0, 0);
                }
                if constexpr (A >= 2) a[0] += a[1];
                if constexpr (A == 3) a[0] += a[2];
                if constexpr (A == 4) a[0] += a[2] + a[3];
                // lane (g, m), register s: candidate j + 4 g + s with destination m
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const float cc = tis * w[s] * a[0][s];
#pragma unroll
                    for (int q = 0; q < 3; ++q) gp[q] = fmaf(cc, diff[s][q], gp[q]);
                }
            }
            if constexpr (DX) {
#pragma unroll
                for (int s = 0; s < 4; ++s) acc.add(s, w[s], gv[s]);
            }
        };
        int j = 0;
        if constexpr (!own)
            for (; j + kTile <= cnt; j += kTile) step(j, std::true_type{});
        if (j < cnt) step(j, std::false_type{});
    };
    for_tile(p, start, rec, cells, n, s0, row_bytes, r2, wk, dst, id, [](int, uint32_t) {}, pass);
    bool bad = false;
    f32x4 out[NB];
    if constexpr (DX) bad |= !acc.total(out);
    if constexpr (DP) {
#pragma unroll
        for (int q = 0; q < 3; ++q) bad |= !finite(gp[q]);
    }
    if (__any(bad)) {
        for (int64_t s = s0; s < s0 + kTile && s < n; ++s) {
            const int64_t i = __float_as_int(rec[s].w);
            const bool mine = lane < feat;
            const float gi = DP && mine ? dy[i * feat + lane] : 0.0f, vi = DP && mine ? x[i * feat + lane] : 0.0f;
            float a = 0.0f, gq[3] = {0.0f, 0.0f, 0.0f};
            slow_row(p, start, rec, s, row_bytes, r2, nis, [&](uint32_t off, float w, const float (&d)[3]) {
                const float gj = mine ? at_bytes<float>(dy, off + 4 * lane) : 0.0f;
                if (DX) a = fmaf(w, gj, a);
                if constexpr (DP) {
                    const float vj = mine ? at_bytes<float>(x, off + 4 * lane) : 0.0f;
                    float dot = mine ? fmaf(gi, vj, gj * vi) : 0.0f;
#pragma unroll
                    for (int o = 1; o < kWave; o <<= 1) dot += shfl_xor_f(dot, o);
                    const float cc = tis * w * dot;
#pragma unroll
                    for (int q = 0; q < 3; ++q) gq[q] = fmaf(cc, d[q], gq[q]);
                }
            });
            if (DX && mine) dx[i * feat + lane] = a;
            if (DP && lane == 0)
                for (int q = 0; q < 3; ++q) dp[i * 3 + q] = gq[q];
        }
        return;
    }
    if constexpr (DP) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            double v = static_cast<double>(gp[q]);
            v += __shfl_xor(v, 16, kWave);
            v += __shfl_xor(v, 32, kWave);
            if (lane < kTile && id >= 0) dp[static_cast<int64_t>(id) * 3 + q] = static_cast<float>(v);
        }
    }
    if constexpr (DX) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t row = __shfl(id, 4 * g + r, kWave);
            if (row < 0) continue;
            float *o = dx + row * feat;
            if constexpr (PAIR) {
                if (2 * m < feat) put_bytes(o + 2 * m, make_float2(out[0][r], out[1][r]));
            } else {
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    if (m + 16 * b < feat) o[m + 16 * b] = out[b][r];
            }
        }
    }
}

dim3 tile_grid(int64_t n) { return dim3(static_cast<unsigned>(ceil_div(n, kTile * (kBlock / kWave)))); }

}  // namespace

int tile_forward(int64_t n, int32_t feat, const Cells &c, const int32_t *cells, const float *x, float r2, float nis,
                 float *y, int32_t *count, hipStream_t stream) {
    const f32x4 *rec = reinterpret_cast<const f32x4 *>(c.rec);
    prof_before(stream);
#define TIGA_FWD(NB, SF, VEC)                                                                                        \
    hipLaunchKernelGGL((count ? tile_fwd_kernel<NB, SF, VEC, true> : tile_fwd_kernel<NB, SF, VEC, false>),           \
                       tile_grid(n), dim3(kBlock), 0, stream, c.prm, c.start, rec, cells, n, feat, x, r2, nis, y,    \
                       count)
    // One or two features: vector units, 27 us where 16-feature blocks take 31 us (131,072 points, 1 feature);
    // from three on the reads of the candidates' values cost more than the unused columns of a block (1M points:
    // 279 and 320 us for 3 and 4 features, 258 us for a block).
    if (feat == 1) TIGA_FWD(0, 1, false);
    else if (feat == 2) TIGA_FWD(0, 2, false);
    else if (feat <= 16) TIGA_FWD(1, 0, false);
    else if (feat <= 32 && feat % 2 == 0) TIGA_FWD(2, 0, true);
    else if (feat <= 32) TIGA_FWD(2, 0, false);
    else if (feat % 4 == 0) TIGA_FWD(4, 0, true);
    else TIGA_FWD(4, 0, false);
#undef TIGA_FWD
    prof_after(stream);
    return check_launch("radius forward (tiles)");
}

namespace {

template <int KS, bool PAIR>
void launch_bwd(int64_t n, int32_t feat, const Cells &c, const int32_t *cells, const float *x, const float *dy,
                float r2, float nis, float tis, float *dx, float *dpos, hipStream_t stream) {
    const f32x4 *rec = reinterpret_cast<const f32x4 *>(c.rec);
    auto *kern = dx && dpos ? tile_bwd_kernel<KS, PAIR, true, true>
                 : dx       ? tile_bwd_kernel<KS, PAIR, true, false>
                            : tile_bwd_kernel<KS, PAIR, false, true>;
    hipLaunchKernelGGL(kern, tile_grid(n), dim3(kBlock), 0, stream, c.prm, c.start, rec, cells, n, feat, x, dy, r2,
                       nis, tis, dx, dpos);
}

}  // namespace

int tile_backward(int64_t n, int32_t feat, const Cells &c, const int32_t *cells, const float *x, const float *dy,
                  float r2, float nis, float tis, float *dx, float *dpos, hipStream_t stream) {
    prof_before(stream);
#define TIGA_BWD(KS, PAIR) launch_bwd<KS, PAIR>(n, feat, c, cells, x, dy, r2, nis, tis, dx, dpos, stream)
    if (feat <= 4) TIGA_BWD(1, false);
    else if (feat <= 8) TIGA_BWD(2, false);
    else if (feat <= 16) TIGA_BWD(4, false);
    else if (feat % 2 == 0) TIGA_BWD(8, true);
    else TIGA_BWD(8, false);
#undef TIGA_BWD
    prof_after(stream);
    return check_launch("radius backward (tiles)");
}

}  // namespace radius
}  // namespace tiga
