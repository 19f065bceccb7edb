// Edge-local MLP message over the generated radius relation, with its vector-Jacobian product
// (appendix "A differentiable EdgeNN example"; Section 5 for the VJP with the relation held fixed):
//   in_ij = [p_j - p_i ; x_j],  m_ij = W2 ReLU(W1 in_ij + b1) + b2,  y_i = sum_{j in N(i)} m_ij
// with N(i) the radius relation (j != i, fp32 squared distance strictly below fl(r*r)).
//
// MI355X design: a persistent grid of wavefronts walks the cell-ordered points, one point per
// wavefront at a time.  The point's candidates are tested 64 at a time, one per lane, and the accepted
// ones compacted into an LDS list (for_pairs).  Then lanes are (neighbour slot, hidden unit): HP lanes
// per neighbour (HP >= the hidden width, a power of two), 64 / HP neighbours per step.  Each lane keeps its row of W1 and
// its column of W2 in registers, so a message costs one lane 3 + F multiply-adds for its hidden
// unit and `out` for its share of the output; the output is summed over hidden units and
// neighbours by one wave reduction per point.  No edge, message or activation is stored.
//
// The VJP uses the symmetry of the radius relation (j in N(i) iff i in N(j)).  At point k, with
// neighbour l, a lane recomputes its hidden unit for both directed messages:
//   l -> k (k the destination, cotangent dy_k): the parameter gradients, and -W1[:, 0:3]^T da for
//     the position of k; every directed pair is the "l -> k" pair of exactly one point, so the
//     parameter gradients count each message once;
//   k -> l (k the source, cotangent dy_l): W1^T da gives the feature gradient of k and +W1[:, 0:3]^T
//     da its position gradient.
// The input gradients are W1^T times per-lane sums of da, so they need one wave reduction per point
// and no atomics.  Parameter gradients are summed in registers across a wavefront's points, written
// as one partial per wavefront, and reduced in a fixed order (deterministic).
#include "edgenn.hpp"

#include "radius_cells.hpp"

namespace tiga {
namespace edgenn {

using radius::Cells;
using radius::Params;

namespace {

constexpr int kBlock = 256;
constexpr int kMaxBlocks = 1024;                       // persistent grid cap
constexpr int kMaxWaves = kMaxBlocks * (kBlock / kWave);

// Sums over the wavefront of N values (N a power of two up to 64): at each of the first log2 N steps a lane
// keeps one half of its values and hands over the other, so N values take N - 1 + 6 - log2 N shuffles, not
// 6 N.  Lane l ends with the sum of value l / (64 / N) (in all 64 / N lanes of that value).
// (Recursive, so that every index is a constant: as loops, the compiler selected among the values at run time.)
template <int N, int M = kWave / 2>
__device__ __forceinline__ float wave_sums(const float (&v)[N]) {
    if constexpr (M == 0) {
        return v[0];
    } else if constexpr (N == 1) {
        const float r[1] = {v[0] + __shfl_xor(v[0], M, kWave)};
        return wave_sums<1, M / 2>(r);
    } else {
        const bool up = (lane_id() & M) != 0;
        float h[N / 2];
#pragma unroll
        for (int k = 0; k < N / 2; ++k) {
            const float give = up ? v[k] : v[k + N / 2], own = up ? v[k + N / 2] : v[k];
            h[k] = own + __shfl_xor(give, M, kWave);
        }
        return wave_sums<N / 2, M / 2>(h);
    }
}

constexpr int kPairs = 64;   // accepted pairs between two passes

// The accepted pairs of the point with record s, as entries (p_j - p_i, point id j) of `list`, at most kPairs at
// a time: pass(count).  The candidates (9 runs of the cell order, laid end to end) are decoded by comparing the
// position with the runs' first positions.  (The previous form tested the 64 / HP candidates of a step, two at
// hidden width 32, each step waiting for its records: 75 us forward and 140 us backward for 35,947 surface
// points, 8 features, hidden width 32; 36 and 55 us now.)
template <class Pass>
__device__ __forceinline__ int for_pairs(const Params &p, const int64_t *__restrict__ start,
                                         const float4 *__restrict__ rec, int64_t s, float4 pi, float r2,
                                         float4 *__restrict__ list, Pass &&pass) {
    const int lane = lane_id();
    const int cx = radius::cell_axis(p, 0, pi.x), cy = radius::cell_axis(p, 1, pi.y), cz = radius::cell_axis(p, 2, pi.z);
    const int x0 = cx > 0 ? cx - 1 : 0, x1 = cx + 1 < p.dim[0] ? cx + 1 : p.dim[0] - 1;
    int32_t first = 0, len = 0;
    if (lane < 9) {
        const int z = cz - 1 + lane / 3, y = cy - 1 + lane % 3;
        if (z >= 0 && z < p.dim[2] && y >= 0 && y < p.dim[1]) {
            const int64_t rowc = (static_cast<int64_t>(z) * p.dim[1] + y) * p.dim[0];
            first = static_cast<int32_t>(start[rowc + x0]);
            len = static_cast<int32_t>(start[rowc + x1 + 1]) - first;
        }
    }
    int32_t at[9], off[9], total = 0;   // first position of run k, record of a position less the position
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        at[k] = total;
        off[k] = __builtin_amdgcn_readlane(first, k) - total;
        total += __builtin_amdgcn_readlane(len, k);
    }
    int cnt = 0, deg = 0;
    for (int32_t c0 = 0; c0 < total; c0 += kWave) {
        const int32_t q = c0 + lane;
        int32_t o = off[0];
#pragma unroll
        for (int k = 1; k < 9; ++k) o = q >= at[k] ? off[k] : o;
        const int64_t t = q < total ? q + o : s;   // past the end: the point itself, which is not accepted
        const float4 pj = rec[t];
        float d2;
        const bool take = radius::accept(pi, pj, r2, d2) && t != s;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(take);
        const int nnew = __popcll(mask);
        if (cnt + nnew > kPairs) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            pass(cnt);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            cnt = 0;
        }
        if (take) {
            const int slot = cnt + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                                             __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0));
            list[slot] = make_float4(pj.x - pi.x, pj.y - pi.y, pj.z - pi.z, pj.w);
        }
        cnt += nnew;
        deg += nnew;
    }
    if (cnt > 0) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        pass(cnt);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    return deg;
}

// Sum over the lanes that hold the same hidden unit (the SL = 64 / HP neighbour slots).
template <int HP>
__device__ __forceinline__ float slot_sum(float v) {
#pragma unroll
    for (int m = HP; m < kWave; m <<= 1) v += __shfl_xor(v, m, kWave);
    return v;
}

int64_t param_count(const Net &net) {
    const int64_t D = 3 + net.feat;
    return net.hidden * D + net.hidden + net.out * net.hidden + net.out;
}

// The lane's weights: row h of W1, b1[h], column h of W2 (zero for h >= hidden).
template <int FP, int OP>
struct LaneNet {
    float w1[3 + FP];
    float bh;
    float w2[OP];
    __device__ __forceinline__ void load(const Net &net, int h) {
        const bool hv = h < net.hidden;
        const int D = 3 + net.feat;
#pragma unroll
        for (int c = 0; c < 3 + FP; ++c) w1[c] = hv && c < D ? net.W1[h * D + c] : 0.0f;
        bh = hv ? net.b1[h] : 0.0f;
#pragma unroll
        for (int o = 0; o < OP; ++o) w2[o] = hv && o < net.out ? net.W2[o * net.hidden + h] : 0.0f;
    }
};

template <int FP>
__device__ __forceinline__ void load_row(const float *__restrict__ x, int64_t j, int F, float (&v)[FP]) {
    const float *r = x + j * F;
    if (F == FP) {   // whole rows: 16-byte loads, which need only the floats' alignment
        __builtin_memcpy(v, r, sizeof v);
        return;
    }
#pragma unroll
    for (int c = 0; c < FP; ++c) v[c] = c < F ? r[c] : 0.0f;
}

template <int HP, int FP, int OP>
__global__ __launch_bounds__(kBlock) void fwd_kernel(const Params *__restrict__ prm, const int64_t *__restrict__ start,
                                                     const float4 *__restrict__ rec, int64_t n, float r2,
                                                     const float *__restrict__ x, Net net, float *__restrict__ y) {
    constexpr int SL = kWave / HP, U = FP <= 8 ? 2 : 1;   // U pairs per slot in flight
    __shared__ float4 lists[kBlock / kWave][kPairs];
    const Params p = *prm;
    const int wv = uniform(static_cast<int>(threadIdx.x) / kWave);
    float4 *list = lists[wv];
    const int lane = lane_id(), slot = lane / HP, h = lane % HP;
    LaneNet<FP, OP> L;
    L.load(net, h);
    const int F = net.feat, O = net.out;
    const int64_t nw = static_cast<int64_t>(gridDim.x) * (kBlock / kWave);
    for (int64_t s = static_cast<int64_t>(xcd_block()) * (kBlock / kWave) + wv; s < n; s += nw) {
        const float4 pi = rec[s];
        const int32_t i = __float_as_int(pi.w);
        float acc[OP] = {};
        const int deg = for_pairs(p, start, rec, s, pi, r2, list, [&](int cnt) __attribute__((always_inline)) {
            for (int k0 = slot; k0 < cnt; k0 += SL * U) {
                float4 e[U];
                float xj[U][FP];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    e[u] = list[k0 + u * SL < cnt ? k0 + u * SL : k0];
                    load_row<FP>(x, __float_as_int(e[u].w), F, xj[u]);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    float a = L.bh + L.w1[0] * e[u].x + L.w1[1] * e[u].y + L.w1[2] * e[u].z;
#pragma unroll
                    for (int c = 0; c < FP; ++c) a += L.w1[3 + c] * xj[u][c];
                    const float r = k0 + u * SL < cnt ? fmaxf(a, 0.0f) : 0.0f;
#pragma unroll
                    for (int o = 0; o < OP; ++o) acc[o] += L.w2[o] * r;
                }
            }
        });
        const float v = wave_sums(acc);
        const int o = lane / (kWave / OP);
        if (lane % (kWave / OP) == 0 && o < O)
            y[static_cast<int64_t>(i) * O + o] = v + static_cast<float>(deg) * net.b2[o];
    }
}

// At feature width 32 the kernel is held to 168 registers (3 waves per SIMD instead of 2 at 179);
// the 8 values this spills cost less than the third wave gains. Other widths keep their registers.
template <int HP, int FP, int OP>
__global__ __launch_bounds__(kBlock, FP == 32 ? 3 : 1) void bwd_kernel(const Params *__restrict__ prm, const int64_t *__restrict__ start,
                                                     const float4 *__restrict__ rec, int64_t n, float r2,
                                                     const float *__restrict__ x, Net net, const float *__restrict__ dyv,
                                                     float *__restrict__ dxo, float *__restrict__ dpo,
                                                     float *__restrict__ part, int64_t P) {
    constexpr int SL = kWave / HP, U = 1;   // U pairs per slot in flight
    __shared__ float4 lists[kBlock / kWave][kPairs];
    const Params p = *prm;
    const int lane = lane_id(), slot = lane / HP, h = lane % HP;
    LaneNet<FP, OP> L;
    L.load(net, h);
    const int F = net.feat, O = net.out, H = net.hidden, D = 3 + F;
    float gW1[3 + FP] = {}, gb1 = 0.0f, gW2[OP] = {}, gb2[OP] = {};
    const int wb = uniform(static_cast<int>(threadIdx.x) / kWave);
    float4 *list = lists[wb];
    const int64_t wv = static_cast<int64_t>(xcd_block()) * (kBlock / kWave) + wb;
    const int64_t nw = static_cast<int64_t>(gridDim.x) * (kBlock / kWave);
    for (int64_t s = wv; s < n; s += nw) {
        const float4 pi = rec[s];
        const int32_t i = __float_as_int(pi.w);
        float dyk[OP];
#pragma unroll
        for (int o = 0; o < OP; ++o) dyk[o] = o < O ? dyv[static_cast<int64_t>(i) * O + o] : 0.0f;
        float dhk = 0.0f;   // this lane's (W2^T dy_k)[h]
#pragma unroll
        for (int o = 0; o < OP; ++o) dhk += L.w2[o] * dyk[o];
        float xi[FP];
        load_row<FP>(x, i, F, xi);
        float ck = L.bh;    // the k -> l pre-activation without its displacement part
#pragma unroll
        for (int c = 0; c < FP; ++c) ck += L.w1[3 + c] * xi[c];
        float S = 0.0f, T = 0.0f;
        const int deg = for_pairs(p, start, rec, s, pi, r2, list, [&](int cnt) __attribute__((always_inline)) {
            for (int k0 = slot; k0 < cnt; k0 += SL * U) {
                float4 e[U];
                float xj[U][FP], dyl[U][OP];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    e[u] = list[k0 + u * SL < cnt ? k0 + u * SL : k0];
                    const int32_t j = __float_as_int(e[u].w);
                    load_row<FP>(x, j, F, xj[u]);
#pragma unroll
                    for (int o = 0; o < OP; ++o) dyl[u][o] = o < O ? dyv[static_cast<int64_t>(j) * O + o] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool live = k0 + u * SL < cnt;
                    const float dx = e[u].x, dy = e[u].y, dz = e[u].z;
                    const float wd = L.w1[0] * dx + L.w1[1] * dy + L.w1[2] * dz;
                    // l -> k: input [d; x_l], cotangent dy_k
                    float a = L.bh + wd;
#pragma unroll
                    for (int c = 0; c < FP; ++c) a += L.w1[3 + c] * xj[u][c];
                    const float r = live ? fmaxf(a, 0.0f) : 0.0f;
#pragma unroll
                    for (int o = 0; o < OP; ++o) gW2[o] += dyk[o] * r;
                    const float da = live && a > 0.0f ? dhk : 0.0f;
                    gW1[0] += da * dx;
                    gW1[1] += da * dy;
                    gW1[2] += da * dz;
#pragma unroll
                    for (int c = 0; c < FP; ++c) gW1[3 + c] += da * xj[u][c];
                    gb1 += da;
                    T += da;
                    // k -> l: input [-d; x_k], cotangent dy_l
                    float dhl = 0.0f;
#pragma unroll
                    for (int o = 0; o < OP; ++o) dhl += L.w2[o] * dyl[u][o];
                    S += live && ck - wd > 0.0f ? dhl : 0.0f;
                }
            }
        });
        // input gradients of point i: W1^T times the lane sums of da (over hidden units and slots)
        constexpr int NV = FP <= 8 ? 16 : (FP <= 16 ? 32 : 64);   // 3 position and FP feature values (FP = 64: below)
        float v[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = 0.0f;
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] = L.w1[q] * (S - T);
#pragma unroll
        for (int q = 0; q < FP; ++q)
            if (3 + q < NV) v[3 + q] = L.w1[3 + q] * S;
        const float g = wave_sums(v);
        const int q = lane / (kWave / NV);
        if (lane % (kWave / NV) == 0) {
            if (dpo && q < 3) dpo[static_cast<int64_t>(i) * 3 + q] = g;
            if (dxo && q >= 3 && q < 3 + F) dxo[static_cast<int64_t>(i) * F + (q - 3)] = g;
        }
        if constexpr (3 + FP > NV) {   // the last features of FP = 64
            float u[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) u[k] = NV - 3 + k < FP ? L.w1[NV + k < 3 + FP ? NV + k : 0] * S : 0.0f;
            const float t = wave_sums(u);
            const int f = NV - 3 + lane / (kWave / 4);
            if (lane % (kWave / 4) == 0 && dxo && f < F) dxo[static_cast<int64_t>(i) * F + f] = t;
        }
        // every message into i carries b2: db2 += deg(i) dy_i
#pragma unroll
        for (int o = 0; o < OP; ++o) gb2[o] += static_cast<float>(deg) * dyk[o];
    }
    if (!part) return;
    // this wavefront's parameter-gradient partial: [dW1 | db1 | dW2 | db2]
    float *pw = part + wv * P;
#pragma unroll
    for (int c = 0; c < 3 + FP; ++c) {
        const float v = slot_sum<HP>(gW1[c]);
        if (slot == 0 && h < H && c < D) pw[h * D + c] = v;
    }
    {
        const float v = slot_sum<HP>(gb1);
        if (slot == 0 && h < H) pw[H * D + h] = v;
    }
#pragma unroll
    for (int o = 0; o < OP; ++o) {
        const float v = slot_sum<HP>(gW2[o]);
        if (slot == 0 && h < H && o < O) pw[H * D + H + o * H + h] = v;
    }
    if (lane == 0)
        for (int o = 0; o < O; ++o) pw[H * D + H + O * H + o] = gb2[o];
}

// Sum the per-wavefront partials into the parameter gradients in two fixed-order stages: each of
// kGroups groups of wavefronts per parameter (consecutive wavefronts, in order), then the groups;
// 64 x 64 balances the two stages' serial sums for 4096 partials.
constexpr int kGroups = 64;

__global__ __launch_bounds__(kWave) void reduce_groups_kernel(const float *__restrict__ part, int64_t nw, int64_t P,
                                                              float *__restrict__ grp) {
    const int64_t q = static_cast<int64_t>(blockIdx.x) * kWave + threadIdx.x;
    if (q >= P) return;
    const int64_t per = (nw + kGroups - 1) / kGroups;
    const int64_t w0 = blockIdx.y * per, w1 = w0 + per < nw ? w0 + per : nw;
    float s = 0.0f;
#pragma unroll 8
    for (int64_t w = w0; w < w1; ++w) s += part[w * P + q];   // 8 loads in flight, summed in order
    grp[static_cast<int64_t>(blockIdx.y) * P + q] = s;
}

__global__ __launch_bounds__(kBlock) void reduce_params_kernel(const float *__restrict__ grp, int64_t P, Net net,
                                                               Grads g) {
    const int64_t q = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (q >= P) return;
    float s = 0.0f;
#pragma unroll 16
    for (int gi = 0; gi < kGroups; ++gi) s += grp[gi * P + q];
    const int64_t D = 3 + net.feat, H = net.hidden, O = net.out;
    if (q < H * D) {
        if (g.dW1) g.dW1[q] = s;
    } else if (q < H * D + H) {
        if (g.db1) g.db1[q - H * D] = s;
    } else if (q < H * D + H + O * H) {
        if (g.dW2) g.dW2[q - H * D - H] = s;
    } else if (g.db2) {
        g.db2[q - H * D - H - O * H] = s;
    }
}

int grid_blocks(int64_t n) {
    const int64_t b = ceil_div(n, kBlock / kWave);
    return static_cast<int>(b < kMaxBlocks ? b : kMaxBlocks);
}

template <int HP, int FP, int OP>
int launch_fwd(int64_t n, const Cells &cl, float r2, const float *x, const Net &net, float *y, hipStream_t stream) {
    // the forward keeps no per-wavefront partials, so its grid is as large as stays resident
    // (more wavefronts in flight hide the dependent record and row loads of each point)
    static const int per_cu = resident_blocks(reinterpret_cast<const void *>(&fwd_kernel<HP, FP, OP>), kBlock);
    const int64_t cap = static_cast<int64_t>(device_cus()) * per_cu;
    const int64_t need = ceil_div(n, kBlock / kWave);
    const int blocks = static_cast<int>(need < cap ? need : cap);
    prof_before(stream);
    hipLaunchKernelGGL((fwd_kernel<HP, FP, OP>), dim3(blocks), dim3(kBlock), 0, stream, cl.prm, cl.start, cl.rec,
                       n, r2, x, net, y);
    prof_after(stream);
    return check_launch("edge MLP forward");
}

template <int HP, int FP, int OP>
int launch_bwd(int64_t n, const Cells &cl, float r2, const float *x, const Net &net, const float *dy, const Grads &g,
               float *part, float *grp, hipStream_t stream) {
    const int blocks = grid_blocks(n);
    const int64_t P = param_count(net);
    const bool params = g.dW1 || g.db1 || g.dW2 || g.db2;
    prof_before(stream);
    hipLaunchKernelGGL((bwd_kernel<HP, FP, OP>), dim3(blocks), dim3(kBlock), 0, stream, cl.prm, cl.start, cl.rec, n, r2,
                       x, net, dy, g.dx, g.dpos, params ? part : nullptr, P);
    prof_after(stream);
    if (int rc = check_launch("edge MLP backward")) return rc;
    if (!params) return TIGA_OK;
    hipLaunchKernelGGL(reduce_groups_kernel, dim3(static_cast<unsigned>(ceil_div(P, kWave)), kGroups), dim3(kWave), 0,
                       stream, part, static_cast<int64_t>(blocks) * (kBlock / kWave), P, grp);
    if (int rc = check_launch("edge MLP parameter reduction")) return rc;
    hipLaunchKernelGGL(reduce_params_kernel, dim3(static_cast<unsigned>(ceil_div(P, kBlock))), dim3(kBlock), 0,
                       stream, grp, P, net, g);
    return check_launch("edge MLP parameter reduction");
}

template <int HP, class Fn>
int by_feat(int F, Fn &&fn) {
    if (F <= 8) return fn(std::integral_constant<int, 8>{});
    if (F <= 16) return fn(std::integral_constant<int, 16>{});
    if (F <= 32) return fn(std::integral_constant<int, 32>{});
    return fn(std::integral_constant<int, 64>{});
}

template <int OP, class Fn>
int by_hidden(const Net &net, Fn &&fn) {
    const std::integral_constant<int, OP> op;
    if (net.hidden <= 16)
        return by_feat<16>(net.feat, [&](auto fp) { return fn(std::integral_constant<int, 16>{}, fp, op); });
    if (net.hidden <= 32)
        return by_feat<32>(net.feat, [&](auto fp) { return fn(std::integral_constant<int, 32>{}, fp, op); });
    return by_feat<64>(net.feat, [&](auto fp) { return fn(std::integral_constant<int, 64>{}, fp, op); });
}

// Outputs padded to 4 or 8: at 3 outputs the instructions of the other five were a third of a message's.
template <class Fn>
int dispatch(const Net &net, Fn &&fn) {
    if (net.out <= 4) return by_hidden<4>(net, fn);
    return by_hidden<kMaxOut>(net, fn);
}

}  // namespace

size_t workspace_bytes(int64_t n, const Net &net) {
    Carve c(nullptr);
    c.take<char>(radius::cells_ws_bytes(n));
    c.take<float>(static_cast<size_t>(kMaxWaves) * param_count(net));
    c.take<float>(static_cast<size_t>(kGroups) * param_count(net));
    return c.bytes();
}

int forward(int64_t n, const float *pos, const float *x, float radius, const Net &net, float *y, void *ws,
            hipStream_t stream) {
    Carve c(ws);
    void *cws = c.take<char>(radius::cells_ws_bytes(n));
    Cells cl;
    if (int rc = radius::build_cells(n, pos, radius, cws, cl, stream)) return rc;
    const float r2 = radius * radius;
    return dispatch(net, [&](auto hp, auto fp, auto op) {
        return launch_fwd<decltype(hp)::value, decltype(fp)::value, decltype(op)::value>(n, cl, r2, x, net, y, stream);
    });
}

int backward(int64_t n, const float *pos, const float *x, float radius, const Net &net, const float *dy,
             const Grads &g, void *ws, hipStream_t stream) {
    Carve c(ws);
    void *cws = c.take<char>(radius::cells_ws_bytes(n));
    float *part = c.take<float>(static_cast<size_t>(kMaxWaves) * param_count(net));
    float *grp = c.take<float>(static_cast<size_t>(kGroups) * param_count(net));
    Cells cl;
    if (int rc = radius::build_cells(n, pos, radius, cws, cl, stream)) return rc;
    const float r2 = radius * radius;
    return dispatch(net, [&](auto hp, auto fp, auto op) {
        return launch_bwd<decltype(hp)::value, decltype(fp)::value, decltype(op)::value>(n, cl, r2, x, net, dy, g, part, grp, stream);
    });
}

}  // namespace edgenn
}  // namespace tiga
