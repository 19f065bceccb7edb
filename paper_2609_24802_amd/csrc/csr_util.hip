// Topology utilities: the stable CSR transpose (a radix sort of edge positions keyed by source id), the
// per-edge records of the gather-mode backward and full validation.
#include "csr_bwd.hpp"
#include "radix.hpp"

namespace tiga {
namespace csr {

namespace {

// rec[e] = (bits of w[e], or of 1.0 without weights; the destination row of e).  Block b takes the edges
// [b * kBlock * ITEMS, (b + 1) * kBlock * ITEMS), so hub rows cost no more than others (split by tiles of rows, the
// 16 blocks of a tile with a 320,000-edge row set the time: 162 us for 16M edges).  It stages windows of
// kRecRows row pointers, each starting within 64 rows before that of the first edge not yet written (found by a
// search over row_ptr by one wavefront, 64 probes per step; a short row_ptr is staged whole), so runs of empty
// rows are skipped; a thread finds the rows of its edges by binary search in LDS, ITEMS edges at a time
// (independent chains): 8 where that gives every compute unit two blocks, 1 below (8,192 edges of 1,024 rows: 8.6 us
// in 4 blocks, 3.6 us in 32; 500,000 edges 7 us with one; 1.2M edges 13 us with 8, 15 us with one).
// Bound: the 8-byte writes and the 4-byte reads of w.
constexpr int kRecRows = 1024;
constexpr int kRecItems = 8;
constexpr int kRecBlocks = 2;   // per compute unit

template <int ITEMS>
__global__ __launch_bounds__(kBlock) void edge_records_kernel(const int64_t *__restrict__ row_ptr, int64_t nrows,
                                                              int64_t nedges, const float *__restrict__ w,
                                                              int2 *__restrict__ rec) {
    constexpr int kEdges = kBlock * ITEMS;
    __shared__ int64_t sp[kRecRows + 1];
    __shared__ int64_t first_row;
    const int64_t e1 = static_cast<int64_t>(blockIdx.x + 1) * kEdges < nedges
                           ? static_cast<int64_t>(blockIdx.x + 1) * kEdges
                           : nedges;
    int64_t r_known = 0;   // row_ptr[r_known] <= the next edge
    for (int64_t e0 = static_cast<int64_t>(blockIdx.x) * kEdges; e0 < e1;) {
        if (threadIdx.x < kWave) {
            // [lo, lo + len) holds the last row r with row_ptr[r] <= e0; row_ptr[lo] <= e0
            int64_t lo = r_known, len = nrows - r_known;
            while (len > kWave && nrows > kRecRows) {
                const int64_t step = (len + kWave - 1) / kWave;
                const int64_t at = lo + step * lane_id();
                const bool below = at < lo + len && row_ptr[at] <= e0;
                const int n_below = __popcll(__builtin_amdgcn_ballot_w64(below));
                const int last = n_below > 0 ? n_below - 1 : 0;
                const int64_t nlo = lo + step * last;
                len = step < lo + len - nlo ? step : lo + len - nlo;
                lo = nlo;
            }
            if (threadIdx.x == 0) first_row = lo;
        }
        __syncthreads();
        const int64_t r0 = first_row;
        const int nr = static_cast<int>(nrows - r0 < kRecRows ? nrows - r0 : kRecRows);
        for (int i = threadIdx.x; i <= nr; i += kBlock) sp[i] = row_ptr[r0 + i];
        __syncthreads();
        const int64_t end = sp[nr] < e1 ? sp[nr] : e1;   // > e0: row r0 holds e0
        if (end <= e0) return;                           // (unless row_ptr ends before num_edges)
        int lo[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) lo[k] = 0;
        // the last row i of the window with sp[i] <= e: descending powers of two
        for (int step = kRecRows / 2; step >= 1; step >>= 1)
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int i = lo[k] + step;
                if (i < nr && sp[i] <= e0 + k * kBlock + threadIdx.x) lo[k] = i;
            }
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int64_t e = e0 + k * kBlock + threadIdx.x;
            if (e < end) rec[e] = make_int2(__float_as_int(w ? w[e] : 1.0f), static_cast<int32_t>(r0 + lo[k]));
        }
        __syncthreads();
        e0 = end;
        r_known = r0 + nr < nrows ? r0 + nr : r0;
    }
}

// ptr[j] = first sorted position with key >= j, for j in [0, nkeys]: one
// binary search per j, so long runs of absent keys cost no serial work.
__global__ __launch_bounds__(kBlock) void ptr_from_sorted_kernel(const int32_t *__restrict__ sorted, int64_t n,
                                                                 int64_t nkeys, int64_t *__restrict__ ptr) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t j = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; j <= nkeys; j += stride)
        ptr[j] = radix::lower_bound(sorted, n, j);
}

// ---------------------------------------------------------------- validation

struct Violations {
    unsigned long long first_row;    // first i with row_ptr[i] > row_ptr[i+1]
    unsigned long long first_col;    // first e with col out of range
    long long rp0, rpn;              // row_ptr[0], row_ptr[num_dst]
};

__global__ __launch_bounds__(kBlock) void validate_kernel(const int64_t *__restrict__ row_ptr,
                                                          const int32_t *__restrict__ col, int64_t nrows,
                                                          int64_t nedges, int64_t nsrc, Violations *v) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    const int64_t tid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (tid == 0) {
        v->rp0 = row_ptr[0];
        v->rpn = row_ptr[nrows];
    }
    for (int64_t i = tid; i < nrows; i += stride)
        if (row_ptr[i] > row_ptr[i + 1]) atomicMin(&v->first_row, static_cast<unsigned long long>(i));
    for (int64_t e = tid; e < nedges; e += stride) {
        const int32_t c = col[e];
        if (c < 0 || c >= nsrc) atomicMin(&v->first_col, static_cast<unsigned long long>(e));
    }
}

__global__ void validate_init_kernel(Violations *v) {
    v->first_row = ~0ull;
    v->first_col = ~0ull;
    v->rp0 = 0;
    v->rpn = 0;
}

}  // namespace

size_t transpose_ws_bytes(int64_t num_dst, int64_t num_src, int64_t num_edges) {
    (void)num_dst;
    (void)num_src;
    Carve c(nullptr);
    radix::carve(c, num_edges);
    return c.bytes();
}

int launch_transpose(const tiga_csr *rel, int64_t *src_ptr, int32_t *edge_id, void *ws, hipStream_t stream) {
    const int64_t n = rel->num_edges;
    if (n == 0) return fill_u32(src_ptr, 0u, 2 * (rel->num_src + 1), stream);
    Carve c(ws);
    const radix::Ws w = radix::carve(c, n);
    const radix::Shape s = radix::shape_for(n, rel->num_src);
    radix::Out out;
    out.idx = edge_id;
    const int32_t *sorted = nullptr;
    if (int rc = radix::launch_first_hist(s, rel->col_idx, w, stream)) return rc;
    if (int rc = radix::launch_sort(s, rel->col_idx, w, out, &sorted, stream)) return rc;
    const int pb = persistent_blocks(ceil_div(rel->num_src + 1, kWave), 8);
    hipLaunchKernelGGL(ptr_from_sorted_kernel, dim3(pb), dim3(kBlock), 0, stream, sorted, n, rel->num_src, src_ptr);
    return check_launch("pointers from sorted keys");
}

int launch_edge_records(const tiga_csr *rel, const float *w, int2 *rec, hipStream_t stream) {
    if (rel->num_edges == 0 || rel->num_dst == 0) return TIGA_OK;
    const bool few = ceil_div(rel->num_edges, kBlock * kRecItems) < kRecBlocks * device_cus();
    const unsigned blocks = static_cast<unsigned>(ceil_div(rel->num_edges, few ? kBlock : kBlock * kRecItems));
    hipLaunchKernelGGL((few ? edge_records_kernel<1> : edge_records_kernel<kRecItems>), dim3(blocks), dim3(kBlock), 0,
                       stream, rel->row_ptr, rel->num_dst, rel->num_edges, w, rec);
    return check_launch("edge records");
}

int launch_validate(const tiga_csr *rel, hipStream_t stream) {
    Violations *dv = nullptr;
    if (int rc = check_hip(hipMalloc(&dv, sizeof(Violations)), "validate: hipMalloc")) return rc;
    Violations hv{};
    int rc = TIGA_OK;
    hipLaunchKernelGGL(validate_init_kernel, dim3(1), dim3(1), 0, stream, dv);
    rc = check_launch("validate init");
    if (!rc) {
        const int blocks = persistent_blocks(ceil_div(rel->num_dst + rel->num_edges, kWave), 8);
        hipLaunchKernelGGL(validate_kernel, dim3(blocks), dim3(kBlock), 0, stream, rel->row_ptr, rel->col_idx,
                           rel->num_dst, rel->num_edges, rel->num_src, dv);
        rc = check_launch("validate");
    }
    if (!rc) rc = check_hip(hipMemcpyAsync(&hv, dv, sizeof hv, hipMemcpyDeviceToHost, stream), "validate: copy");
    if (!rc) rc = check_hip(hipStreamSynchronize(stream), "validate: synchronize");
    (void)hipFree(dv);
    if (rc) return rc;
    if (hv.rp0 != 0) return fail(TIGA_EGRAPH, "row_ptr[0] = %lld, expected 0", hv.rp0);
    if (hv.first_row != ~0ull)
        return fail(TIGA_EGRAPH, "row_ptr decreases at row %llu (row_ptr[i] > row_ptr[i+1])", hv.first_row);
    if (hv.rpn != rel->num_edges)
        return fail(TIGA_EGRAPH, "row_ptr[num_dst] = %lld, expected num_edges = %lld", hv.rpn,
                    (long long)rel->num_edges);
    if (hv.first_col != ~0ull)
        return fail(TIGA_EGRAPH, "col_idx[%llu] is outside [0, %lld)", hv.first_col, (long long)rel->num_src);
    return TIGA_OK;
}

}  // namespace csr
}  // namespace tiga
