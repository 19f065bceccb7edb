// Degree-aware row plan, one pass over the rows.
//
// init: clear the counters and record where classes 1 and 2 start in the
//       chunk array (each class has a region of its own capacity);
// plan: each block takes a tile of 8 rows per thread, scans the chunks of each
//       class, partial slots and split rows its rows need (block-local scan),
//       reserves those ranges with one atomic add per counter, and writes the
//       descriptors in row order within its ranges.
// Only rows longer than the short-row bound get descriptors; short rows are
// taken in natural order by the traversal itself.
#include "csr_common.hpp"

namespace tiga {
namespace csr {

namespace {

// Tile-local counts are 32-bit: a partial slot is an int32 id, so no tile can need more.
struct Need {
    int32_t v[kPlanVals];  // chunks per class, partial slots, split rows
};

// Chunks per class, partial slots and split rows needed by a row of degree deg.
__device__ __forceinline__ Need need_of(const Geom &g, int64_t deg) {
    Need r;
#pragma unroll
    for (int k = 0; k < kPlanVals; ++k) r.v[k] = 0;
    if (deg > g.DS) {
        const int32_t nch = static_cast<int32_t>((deg + g.CH - 1) / g.CH);
        const int64_t last = deg - static_cast<int64_t>(nch - 1) * g.CH;
        const int c = chunk_class(g, last);
        r.v[0] += nch - 1 + (c == 0);
        r.v[1] += (c == 1);
        r.v[2] += (c == 2);
        if (nch > 1) {
            r.v[kClasses] = nch;
            r.v[kClasses + 1] = 1;
        }
    }
    return r;
}

// Block-wide exclusive scan of kPlanVals counters over BLOCK threads; returns
// the block totals.
template <int BLOCK>
__device__ __forceinline__ Need block_excl_scan(const Need &v, Need &excl) {
    constexpr int W = BLOCK / kWave;
    __shared__ int32_t sh[kPlanVals][W];
    const int lane = lane_id();
    const int wave = threadIdx.x / kWave;
    Need inc, tot;
#pragma unroll
    for (int k = 0; k < kPlanVals; ++k) {
        inc.v[k] = wave_incl_scan(v.v[k]);
        if (lane == kWave - 1) sh[k][wave] = inc.v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPlanVals; ++k) {
        int32_t off = 0, t = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            if (w < wave) off += sh[k][w];
            t += sh[k][w];
        }
        excl.v[k] = off + inc.v[k] - v.v[k];
        tot.v[k] = t;
    }
    __syncthreads();
    return tot;
}

__global__ void plan_init_kernel(PlanCounts *__restrict__ counts, int64_t off1, int64_t off2) {
    if (threadIdx.x < kPlanVals) counts->ctr[threadIdx.x].v = 0;
    if (threadIdx.x == 0) {
        counts->off[0] = static_cast<unsigned long long>(off1);
        counts->off[1] = static_cast<unsigned long long>(off2);
    }
}

// Descriptors of a tile in row order: thread t owns the kPlanRowsPerThread
// consecutive rows base + t * kPlanRowsPerThread + r and writes them after the
// rows of threads 0..t-1, so consecutive descriptors of a class are rows in
// ascending order (a work item of several chunks writes neighbouring output
// rows).  The tile's row pointers are staged in LDS first (coalesced loads;
// one pad slot per 8 entries keeps the per-thread reads off a single bank).
__host__ __device__ constexpr int pad_ix(int i) { return i + (i >> 3); }

// A row of more than kHubChunks chunks is written by its whole wavefront (64 descriptors per step):
// written by its own thread, a 320,000-edge row (1,250 chunks) kept one lane storing for 150 us while
// the rest of the plan took 19 us (1M rows, 16M edges, 64 features).
//
// The tiles' reservations on one counter are served one after another (about 13 ns each, measured with
// one counter per XCD), so the tile grows with the relation: BLOCK = 256 (2,048 rows) keeps all compute
// units busy on small relations, BLOCK = 1024 (8,192 rows) needs a quarter of the atomics.
constexpr int kHubChunks = 16;

template <int L, int BLOCK>
__global__ __launch_bounds__(BLOCK) void plan_kernel(const int64_t *__restrict__ ptr, int64_t nrows,
                                                     PlanCounts *__restrict__ counts, Desc *__restrict__ chunks,
                                                     Split *__restrict__ splits) {
    constexpr Geom g = make_geom(L);
    constexpr int TILE = BLOCK * kPlanRowsPerThread;
    __shared__ int64_t sptr[pad_ix(TILE) + 1];
    __shared__ int64_t sbase[kPlanVals];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * TILE;
    for (int i = threadIdx.x; i <= TILE; i += BLOCK) {
        const int64_t row = base + i;
        sptr[pad_ix(i)] = ptr[row < nrows ? row : nrows];
    }
    __syncthreads();
    const int64_t cbase[kClasses] = {0, static_cast<int64_t>(counts->off[0]), static_cast<int64_t>(counts->off[1])};
    Need mine;
#pragma unroll
    for (int k = 0; k < kPlanVals; ++k) mine.v[k] = 0;
    const int i0 = threadIdx.x * kPlanRowsPerThread;
    // rows past the end have equal staged pointers: degree 0
#pragma unroll
    for (int r = 0; r < kPlanRowsPerThread; ++r) {
        const Need n = need_of(g, sptr[pad_ix(i0 + r + 1)] - sptr[pad_ix(i0 + r)]);
#pragma unroll
        for (int k = 0; k < kPlanVals; ++k) mine.v[k] += n.v[k];
    }
    Need excl;
    const Need tot = block_excl_scan<BLOCK>(mine, excl);
    // one reservation per counter for the whole tile: thread k adds the tile's total of counter k
    // (vector atomics, all in flight together)
    if (threadIdx.x < kPlanVals) {
        int32_t t = 0;
#pragma unroll
        for (int k = 0; k < kPlanVals; ++k) t = threadIdx.x == k ? tot.v[k] : t;
        sbase[threadIdx.x] =
            t > 0 ? static_cast<int64_t>(atomicAdd(&counts->ctr[threadIdx.x].v, static_cast<unsigned long long>(t))) : 0;
    }
    __syncthreads();
    int64_t run[kPlanVals];
#pragma unroll
    for (int k = 0; k < kPlanVals; ++k) run[k] = sbase[k] + excl.v[k];
#pragma unroll
    for (int k = 0; k < kClasses; ++k) run[k] += cbase[k];
#pragma unroll 1
    for (int r = 0; r < kPlanRowsPerThread; ++r) {
        const int64_t e0 = sptr[pad_ix(i0 + r)];
        const int64_t deg = sptr[pad_ix(i0 + r + 1)] - e0;
        const bool planned = deg > g.DS;
        const int32_t nch = planned ? static_cast<int32_t>((deg + g.CH - 1) / g.CH) : 0;
        const int32_t row = static_cast<int32_t>(base + i0 + r);
        const int slot0 = nch > 1 ? static_cast<int>(run[kClasses]) : -1;
        // the full chunks of hub rows, one row at a time by the whole wavefront (run[0] is where a
        // row's class-0 descriptors start)
        uint64_t hubs = __builtin_amdgcn_ballot_w64(nch > kHubChunks);
        while (hubs) {
            const int src = __builtin_ctzll(hubs);
            hubs &= hubs - 1;
            const int32_t h_n = __builtin_amdgcn_readlane(nch, src) - 1;
            const int32_t h_row = __builtin_amdgcn_readlane(row, src);
            const int32_t h_slot = __builtin_amdgcn_readlane(slot0, src);
            const int64_t h_e0 = __shfl(e0, src, kWave);
            const int64_t h_pos = __shfl(run[0], src, kWave);
            for (int32_t k = lane_id(); k < h_n; k += kWave)
                chunks[h_pos + k] =
                    Desc{h_row, h_slot + k, pack_range(h_e0 + static_cast<int64_t>(k) * g.CH, g.CH)};
        }
        if (!planned) continue;
        int32_t k = 0;
        if (nch > kHubChunks) {
            k = nch - 1;
            run[0] += k;
        }
        for (; k < nch; ++k) {
            const int64_t at = static_cast<int64_t>(k) * g.CH;
            const int64_t len = (k + 1 < nch) ? g.CH : deg - at;
            const int c = (k + 1 < nch) ? 0 : chunk_class(g, len);
            const int64_t pos = c == 0 ? run[0] : (c == 1 ? run[1] : run[2]);
            chunks[pos] = Desc{row, slot0 >= 0 ? slot0 + k : -1, pack_range(e0 + at, len)};
            run[0] += (c == 0);
            run[1] += (c == 1);
            run[2] += (c == 2);
        }
        if (nch > 1) {
            splits[run[kClasses + 1]] = Split{row, slot0, nch, 0};
            run[kClasses] += nch;
            run[kClasses + 1] += 1;
        }
    }
}

}  // namespace

namespace {

// Tiles of 8,192 rows from 4M rows on (512 tiles of them still cover the compute units twice).
constexpr int kPlanBig = 1024;
constexpr int64_t kPlanBigRows = int64_t{1} << 22;

template <int L>
int launch_plan_t(const int64_t *ptr, int64_t nrows, const PlanBounds &b, const PlanWs &w, hipStream_t stream) {
    hipLaunchKernelGGL(plan_init_kernel, dim3(1), dim3(kWave), 0, stream, w.counts, b.cap[0], b.cap[0] + b.cap[1]);
    if (int rc = check_launch("plan init")) return rc;
    const bool big = nrows >= kPlanBigRows;
    const int block = big ? kPlanBig : kBlock;
    const dim3 tiles(static_cast<unsigned>(ceil_div(nrows > 0 ? nrows : 1, block * kPlanRowsPerThread)));
    if (big)
        hipLaunchKernelGGL((plan_kernel<L, kPlanBig>), tiles, dim3(kPlanBig), 0, stream, ptr, nrows, w.counts,
                           w.chunks, w.splits);
    else
        hipLaunchKernelGGL((plan_kernel<L, kBlock>), tiles, dim3(kBlock), 0, stream, ptr, nrows, w.counts, w.chunks,
                           w.splits);
    return check_launch("plan");
}
}  // namespace

int launch_plan(const int64_t *ptr, int64_t nrows, const Geom &g, const PlanBounds &b, const PlanWs &w,
                hipStream_t stream) {
    switch (g.L) {
        case 1: return launch_plan_t<1>(ptr, nrows, b, w, stream);
        case 2: return launch_plan_t<2>(ptr, nrows, b, w, stream);
        case 4: return launch_plan_t<4>(ptr, nrows, b, w, stream);
        case 8: return launch_plan_t<8>(ptr, nrows, b, w, stream);
        case 16: return launch_plan_t<16>(ptr, nrows, b, w, stream);
        case 32: return launch_plan_t<32>(ptr, nrows, b, w, stream);
        case 64: return launch_plan_t<64>(ptr, nrows, b, w, stream);
        default: return fail(TIGA_EINVAL, "internal: plan for %d lanes per edge", g.L);
    }
}

}  // namespace csr
}  // namespace tiga
