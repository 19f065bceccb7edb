// Kernels of the stable radix sort.
#include "radix.hpp"

namespace tiga {
namespace radix {

namespace {

template <int ITEMS>
__global__ __launch_bounds__(kThreads) void hist_kernel(const int32_t *__restrict__ keys, int64_t n, int shift, int rb,
                                                        uint32_t *__restrict__ counts) {
    __shared__ uint32_t hist[kMaxDigits];
    key_tile<ITEMS>(n, rb, nullptr, counts, hist,
                    [&](int64_t i) { return static_cast<int32_t>(static_cast<uint32_t>(keys[i]) >> shift); });
}

// Column scan of counts [tiles][D]: block b takes 64 digits (a lane each); its 16 wavefronts take equal
// runs of tiles, sum them, and write the exclusive prefixes on a second walk.
constexpr int kScanThreads = 1024;
constexpr int kScanWaves = kScanThreads / kWave;
constexpr int kScanBatch = 8;

__global__ __launch_bounds__(kScanThreads) void scan_kernel(uint32_t *__restrict__ counts, int64_t tiles, int D,
                                                            uint32_t *__restrict__ totals) {
    __shared__ uint32_t sums[kScanWaves][kWave];
    const int lane = lane_id(), wv = threadIdx.x / kWave;
    const int d = blockIdx.x * kWave + lane;
    const bool ok = d < D;
    const int64_t per = (tiles + kScanWaves - 1) / kScanWaves;
    const int64_t t0 = per * wv < tiles ? per * wv : tiles, t1 = t0 + per < tiles ? t0 + per : tiles;
    uint32_t s = 0;
    for (int64_t t = t0; t < t1; t += kScanBatch) {
        uint32_t v[kScanBatch];
#pragma unroll
        for (int b = 0; b < kScanBatch; ++b) v[b] = ok && t + b < t1 ? counts[(t + b) * D + d] : 0u;
#pragma unroll
        for (int b = 0; b < kScanBatch; ++b) s += v[b];
    }
    sums[wv][lane] = s;
    __syncthreads();
    uint32_t run = 0;
    for (int w = 0; w < wv; ++w) run += sums[w][lane];
    if (wv == kScanWaves - 1 && ok) totals[d] = run + s;
    for (int64_t t = t0; t < t1; t += kScanBatch) {
        uint32_t v[kScanBatch];
#pragma unroll
        for (int b = 0; b < kScanBatch; ++b) v[b] = ok && t + b < t1 ? counts[(t + b) * D + d] : 0u;
#pragma unroll
        for (int b = 0; b < kScanBatch; ++b)
            if (ok && t + b < t1) {
                counts[(t + b) * D + d] = run;
                run += v[b];
            }
    }
}

template <int ITEMS>
__global__ __launch_bounds__(kThreads) void scatter_kernel(const int32_t *__restrict__ keys_in,
                                                           const int32_t *__restrict__ idx_in, int64_t n, int shift,
                                                           int rb, int64_t tiles, bool direct,
                                                           const uint32_t *__restrict__ counts,
                                                           const uint32_t *__restrict__ totals, Out out) {
    constexpr int TILE = ITEMS * kThreads;
    constexpr int PIECE = ITEMS * kWave;   // keys of one wavefront
    // per-wavefront digit counters while ranking, then the tile grouped by digit
    __shared__ union {
        uint32_t cnt[kWaves][kMaxDigits];
        struct {
            int32_t key[TILE], idx[TILE];
        } st;
    } sh;
    __shared__ uint32_t first[kMaxDigits];   // LDS slot of the tile's first key of each digit
    __shared__ uint32_t delta[kMaxDigits];   // output position - LDS slot, per digit
    __shared__ uint32_t wsum[2][kWaves];
    const int D = 1 << rb;
    const int t = threadIdx.x, lane = lane_id(), wv = t / kWave;
    const int64_t tile = blockIdx.x;
    const int64_t base = tile * TILE;
    const int total = static_cast<int>(n - base < TILE ? n - base : TILE);
    const uint64_t lt = (uint64_t{1} << lane) - 1;
    int32_t key[ITEMS], idx[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int j = wv * PIECE + r * kWave + lane;
        const int64_t i = base + (j < total ? j : 0);
        key[r] = keys_in[i];
        idx[r] = idx_in ? idx_in[i] : static_cast<int32_t>(i);
    }
    // this thread's two digits: keys of earlier tiles and of all tiles
    const int d0 = 2 * t;
    uint32_t pre[2] = {0, 0}, tot[2] = {0, 0};
    if (d0 < D) {
        if (direct) {
            const uint2 *col = reinterpret_cast<const uint2 *>(counts + d0);
#pragma unroll 8
            for (int b = 0; b < static_cast<int>(tiles); ++b) {
                const uint2 c = col[static_cast<int64_t>(b) * (D / 2)];
                tot[0] += c.x;
                tot[1] += c.y;
                pre[0] += b < tile ? c.x : 0u;
                pre[1] += b < tile ? c.y : 0u;
            }
        } else {
            pre[0] = counts[tile * D + d0];
            pre[1] = counts[tile * D + d0 + 1];
            tot[0] = totals[d0];
            tot[1] = totals[d0 + 1];
        }
    }
    for (int i = t; i < kWaves * kMaxDigits; i += kThreads) (&sh.cnt[0][0])[i] = 0;
    __syncthreads();
    uint32_t off[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const bool valid = wv * PIECE + r * kWave + lane < total;
        const uint32_t d = (static_cast<uint32_t>(key[r]) >> shift) & (D - 1);
        uint64_t peers = __builtin_amdgcn_ballot_w64(valid);
        for (int bit = 0; bit < rb; ++bit) {
            const bool on = (d >> bit) & 1;
            const uint64_t m = __builtin_amdgcn_ballot_w64(on);
            peers &= on ? m : ~m;
        }
        const uint32_t rank = __popcll(peers & lt);
        const uint32_t seen = sh.cnt[wv][d];
        off[r] = seen + rank;
        __builtin_amdgcn_wave_barrier();
        if (valid && rank == 0) sh.cnt[wv][d] = seen + __popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // exclusive prefixes: over the wavefronts per digit, over the digits for the tile and for the output
    uint32_t mine[2] = {0, 0};
    if (d0 < D) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint32_t c = sh.cnt[w][d0 + k];
                sh.cnt[w][d0 + k] = mine[k];
                mine[k] += c;
            }
    }
    const uint32_t here = mine[0] + mine[1], all = tot[0] + tot[1];
    const uint32_t inc_here = wave_incl_scan(here), inc_all = wave_incl_scan(all);
    if (lane == kWave - 1) {
        wsum[0][wv] = inc_here;
        wsum[1][wv] = inc_all;
    }
    __syncthreads();
    uint32_t b_here = inc_here - here, b_all = inc_all - all;
    for (int w = 0; w < wv; ++w) {
        b_here += wsum[0][w];
        b_all += wsum[1][w];
    }
    if (d0 < D) {
        first[d0] = b_here;
        first[d0 + 1] = b_here + mine[0];
        delta[d0] = b_all + pre[0] - b_here;
        delta[d0 + 1] = b_all + tot[0] + pre[1] - (b_here + mine[0]);
    }
    __syncthreads();
    uint32_t slot[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t d = (static_cast<uint32_t>(key[r]) >> shift) & (D - 1);
        slot[r] = first[d] + sh.cnt[wv][d] + off[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
        if (wv * PIECE + r * kWave + lane < total) {
            sh.st.key[slot[r]] = key[r];
            sh.st.idx[slot[r]] = idx[r];
        }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int s = r * kThreads + t;
        if (s < total) {
            const int32_t k = sh.st.key[s], i = sh.st.idx[s];
            const uint32_t pos = s + delta[(static_cast<uint32_t>(k) >> shift) & (D - 1)];
            if (pos < n) {
                if (out.keys) out.keys[pos] = k;
                if (out.idx) out.idx[pos] = i;
                if (out.rec) {
                    const float *p = out.pos + static_cast<int64_t>(i) * 3;
                    // a point with a non-finite coordinate is within the radius of, and near, nothing: all +inf
                    const bool ok = __builtin_isfinite(p[0]) && __builtin_isfinite(p[1]) && __builtin_isfinite(p[2]);
                    const float inf = __builtin_inff();
                    out.rec[pos] = make_float4(ok ? p[0] : inf, ok ? p[1] : inf, ok ? p[2] : inf, __int_as_float(i));
                }
            }
        }
    }
}

int hist(const Shape &s, const int32_t *keys, int shift, const Ws &w, hipStream_t stream) {
    const dim3 grid(static_cast<unsigned>(s.tiles)), block(kThreads);
    if (s.items == 2)
        hipLaunchKernelGGL(hist_kernel<2>, grid, block, 0, stream, keys, s.n, shift, s.rb, w.counts);
    else if (s.items == 4)
        hipLaunchKernelGGL(hist_kernel<4>, grid, block, 0, stream, keys, s.n, shift, s.rb, w.counts);
    else
        hipLaunchKernelGGL(hist_kernel<8>, grid, block, 0, stream, keys, s.n, shift, s.rb, w.counts);
    return check_launch("radix histogram");
}

}  // namespace

int launch_first_hist(const Shape &s, const int32_t *keys, const Ws &w, hipStream_t stream) {
    return hist(s, keys, 0, w, stream);
}

int launch_sort(const Shape &s, const int32_t *keys, const Ws &w, const Out &out, const int32_t **sorted,
                hipStream_t stream) {
    const int32_t *kin = keys, *ain = nullptr;
    const int D = 1 << s.rb;
    for (int p = 0; p < s.passes; ++p) {
        const int shift = p * s.rb;
        if (p > 0)
            if (int rc = hist(s, kin, shift, w, stream)) return rc;
        if (!s.direct) {
            hipLaunchKernelGGL(scan_kernel, dim3(static_cast<unsigned>(ceil_div(D, kWave))), dim3(kScanThreads), 0,
                               stream, w.counts, s.tiles, D, w.totals);
            if (int rc = check_launch("radix scan")) return rc;
        }
        // ping-pong through the workspace; the last pass writes the caller's arrays
        const bool last = p == s.passes - 1;
        Out o;
        o.keys = last && out.keys ? out.keys : w.k[p & 1];
        o.idx = last ? out.idx : w.a[p & 1];
        if (last) {
            o.pos = out.pos;
            o.rec = out.rec;
        }
        const dim3 grid(static_cast<unsigned>(s.tiles)), block(kThreads);
        if (s.items == 2)
            hipLaunchKernelGGL(scatter_kernel<2>, grid, block, 0, stream, kin, ain, s.n, shift, s.rb, s.tiles,
                               s.direct, w.counts, w.totals, o);
        else if (s.items == 4)
            hipLaunchKernelGGL(scatter_kernel<4>, grid, block, 0, stream, kin, ain, s.n, shift, s.rb, s.tiles,
                               s.direct, w.counts, w.totals, o);
        else
            hipLaunchKernelGGL(scatter_kernel<8>, grid, block, 0, stream, kin, ain, s.n, shift, s.rb, s.tiles,
                               s.direct, w.counts, w.totals, o);
        if (int rc = check_launch("radix scatter")) return rc;
        kin = o.keys;
        ain = o.idx;
    }
    if (sorted) *sorted = kin;
    return TIGA_OK;
}

}  // namespace radix
}  // namespace tiga
