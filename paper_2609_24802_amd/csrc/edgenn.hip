// Edge-local MLP message over the generated radius relation, with its vector-Jacobian product
// (appendix "A differentiable EdgeNN example"; Section 5 for the VJP with the relation held fixed):
//   in_ij = [p_j - p_i ; x_j],  m_ij = W2 ReLU(W1 in_ij + b1) + b2,  y_i = sum_{j in N(i)} m_ij
// with N(i) the radius relation (j != i, fp32 squared distance strictly below fl(r*r)).
//
// MI355X design: a persistent grid of wavefronts walks the cell-ordered points, one point per
// wavefront at a time.  The point's candidates are tested 64 at a time, one per lane, and the accepted
// ones compacted into LDS lists, one per neighbour slot (for_pairs).  Then lanes are (neighbour slot,
// hidden unit): HP lanes per neighbour (HP >= the hidden width, a power of two), 64 / HP neighbours per
// step.  Each lane keeps its row of W1 and its column of W2 in registers, so a message costs one lane
// 3 + F products for its hidden unit and `out` for its share of the output; the output is summed over
// hidden units and neighbours by one wave reduction per point.  No edge, message or activation is stored.
//
// Every sum has one fixed order, which depends on the hidden width alone: with few outputs and a
// cancelling cotangent the parameter gradients amplify a change of order a hundredfold (2e-5 relative
// between two orders of the same pairs).
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

// The value of lane l ^ M: within 4 lanes an operand modifier (DPP), else a cross-lane read.
template <int M>
__device__ __forceinline__ float from_xor(float v) {
    if constexpr (M == 1 || M == 2)
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), M == 1 ? 0xb1 : 0x4e, 0xf, 0xf, false));
    else
        return __shfl_xor(v, M, kWave);
}

// Sums of N values (a power of two) over the lanes at distances M, 2 M, ..., 32: at each of the first log2 N
// steps a lane keeps one half of its values and hands over the other, so the values cost N - 1 + the steps
// left over in shuffles, not N per step.  Each sum adds what a butterfly over the same distances adds, in its
// order.  Lane l ends with the sum of value sum_index<N, M>(l).
// (Recursive, so that every index is a constant: as loops, the compiler selected among the values at run time.)
template <int N, int M>
__device__ __forceinline__ float exchange_sums(const float (&v)[N]) {
    if constexpr (M == kWave) {
        static_assert(N == 1, "more values than the lanes can hold");
        return v[0];
    } else if constexpr (N == 1) {
        const float r[1] = {v[0] + from_xor<M>(v[0])};
        return exchange_sums<1, 2 * M>(r);
    } else {
        const bool up = (lane_id() & M) != 0;
        float h[N / 2];
#pragma unroll
        for (int k = 0; k < N / 2; ++k) {
            const float give = up ? v[k] : v[k + N / 2], own = up ? v[k + N / 2] : v[k];
            h[k] = own + from_xor<M>(give);
        }
        return exchange_sums<N / 2, 2 * M>(h);
    }
}

template <int N, int M>
__device__ __forceinline__ int sum_index(int lane) {
    int q = 0;
#pragma unroll
    for (int n = N / 2, m = M; n >= 1; n /= 2, m *= 2) q += lane & m ? n : 0;
    return q;
}

constexpr int kPairs = 64;             // accepted pairs of a slot between two passes
constexpr int kListRow = kPairs + 1;   // the slots' lists start on different LDS banks

// The accepted pairs of the point with record s, as entries (p_j - p_i, point id j) of a list per neighbour slot,
// at most kPairs each at a time: pass(count of this lane's slot).  The candidates are 9 runs of the cell order,
// laid end to end, each from a multiple of SL on, and decoded by comparing the position with the runs' bounds.
// Slot (position in its run) mod SL takes a pair, whatever became of the others: every sum over pairs then has
// one order for all widths of the kernels, that of testing SL candidates of a run per step.  (That form, which
// waits for the records of every step, took 75 us forward and 140 us backward for 35,947 surface points,
// 8 features, hidden width 32; 37 and 65 us now.)
template <int SL, class Pass>
__device__ __forceinline__ int for_pairs(const Params &p, const int64_t *__restrict__ start,
                                         const float4 *__restrict__ rec, int64_t s, float4 pi, float r2,
                                         float4 *__restrict__ list, Pass &&pass) {
    static_assert(SL == 1 || SL == 2 || SL == 4, "neighbour slots");
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
    // run k: first position, position past its last, record of a position less the position
    int32_t at[9], end[9], off[9], total = 0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        total = (total + SL - 1) & -SL;
        at[k] = total;
        off[k] = __builtin_amdgcn_readlane(first, k) - total;
        total += __builtin_amdgcn_readlane(len, k);
        end[k] = total;
    }
    // lanes l, l + SL, ... hold the candidates of slot l
    constexpr uint64_t kSlotLanes = SL == 1 ? ~0ull : (SL == 2 ? 0x5555555555555555ull : 0x1111111111111111ull);
    const int to = lane % SL, slot = lane / (kWave / SL);
    const uint64_t mine = kSlotLanes << to;
    uint32_t cnt = 0;   // entries of each list, a byte per slot (at most kPairs, 128 before a pass)
    int deg = 0;
    auto count_of = [&](int k) __attribute__((always_inline)) { return static_cast<int>((cnt >> (8 * k)) & 0xffu); };
    for (int32_t c0 = 0; c0 < total; c0 += kWave) {
        const int32_t q = c0 + lane;
        int32_t o = off[0], e = end[0];
#pragma unroll
        for (int k = 1; k < 9; ++k) {
            o = q >= at[k] ? off[k] : o;
            e = q >= at[k] ? end[k] : e;
        }
        const int64_t t = q < e ? q + o : s;   // past a run's end: the point itself, which is not accepted
        const float4 pj = rec[t];
        float d2;
        const bool take = radius::accept(pi, pj, r2, d2) && t != s;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(take);
        uint32_t nnew = 0;
#pragma unroll
        for (int k = 0; k < SL; ++k)
            nnew |= static_cast<uint32_t>(__popcll(mask & (kSlotLanes << k))) << (8 * k);
        static_assert(kPairs == 64, "a byte's top bit shows a list above 64");
        if ((cnt + nnew + 0x3f3f3f3fu) & 0x80808080u) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            pass(count_of(slot));
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            cnt = 0;
        }
        if (take) {
            const uint64_t before = mask & mine;
            const int pos = count_of(to) +
                           __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(before >> 32),
                                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(before), 0));
            list[to * kListRow + pos] = make_float4(pj.x - pi.x, pj.y - pi.y, pj.z - pi.z, pj.w);
        }
        cnt += nnew;
        deg += __popcll(mask);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    pass(count_of(slot));
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
    __shared__ float4 lists[kBlock / kWave][SL * kListRow];
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
        const int deg = for_pairs<SL>(p, start, rec, s, pi, r2, list, [&](int cnt) __attribute__((always_inline)) {
            for (int k0 = 0; k0 < cnt; k0 += U) {
                float4 e[U];
                float xj[U][FP];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    e[u] = list[slot * kListRow + (k0 + u < cnt ? k0 + u : k0)];
                    load_row<FP>(x, __float_as_int(e[u].w), F, xj[u]);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    // products and sums rounded one by one, here and in the backward's parameter gradients: both
                    // decide alike which hidden units are active
#pragma clang fp contract(off)
                    float a = L.bh + L.w1[0] * e[u].x + L.w1[1] * e[u].y + L.w1[2] * e[u].z;
#pragma unroll
                    for (int c = 0; c < FP; ++c) a += L.w1[3 + c] * xj[u][c];
                    const float r = fmaxf(a, 0.0f);
#pragma unroll
                    for (int o = 0; o < OP; ++o) {
                        const float t = acc[o] + L.w2[o] * r;
                        acc[o] = k0 + u < cnt ? t : acc[o];
                    }
                }
            }
        });
        const float v = exchange_sums<OP, 1>(acc);
        const int o = sum_index<OP, 1>(lane);
        if (lane < OP && o < O) y[static_cast<int64_t>(i) * O + o] = fmaf(static_cast<float>(deg), net.b2[o], v);
    }
}

// The input gradients of a point, values Q, Q + 1, ... of 3 + FP: position (W1 column times S - T), then features
// (column times S), each summed over the lanes.  The first step adds a lane's product unrounded to that of its odd
// neighbour, in every even lane; the others go by exchange among the even lanes, up to 32 values at a time.
template <int FP, int Q = 0>
__device__ __forceinline__ void put_input_grads(const float (&w1)[3 + FP], float S, float T, int64_t i, int F,
                                                float *__restrict__ dxo, float *__restrict__ dpo) {
    constexpr int rest = 3 + FP - Q, N = rest <= 4 ? 4 : (rest <= 16 ? 16 : 32);
    const int lane = lane_id();
    float v[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const float w = k < rest ? w1[k < rest ? Q + k : 0] : 0.0f, d = Q + k < 3 ? S - T : S;
        v[k] = fmaf(w, d, from_xor<1>(w * d));
    }
    const float g = exchange_sums<N, 2>(v);
    const int q = Q + sum_index<N, 2>(lane);
    if (lane % 2 == 0 && lane < 2 * N) {
        if (dpo && q < 3) dpo[i * 3 + q] = g;
        if (dxo && q >= 3 && q < 3 + F) dxo[i * F + (q - 3)] = g;
    }
    if constexpr (rest > N) put_input_grads<FP, Q + N>(w1, S, T, i, F, dxo, dpo);
}

// At feature width 32 the kernel is held to 168 registers (3 waves per SIMD instead of 2 at 179);
// the 8 values this spills cost less than the third wave gains. Other widths keep their registers.
template <int HP, int FP, int OP>
__global__ __launch_bounds__(kBlock, FP == 32 ? 3 : 1) void bwd_kernel(const Params *__restrict__ prm, const int64_t *__restrict__ start,
                                                     const float4 *__restrict__ rec, int64_t n, float r2,
                                                     const float *__restrict__ x, Net net, const float *__restrict__ dyv,
                                                     float *__restrict__ dxo, float *__restrict__ dpo,
                                                     float *__restrict__ part, int64_t P) {
    constexpr int SL = kWave / HP;
    __shared__ float4 lists[kBlock / kWave][SL * kListRow];
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
        for (int o = 0; o < OP; ++o) dhk = fmaf(L.w2[o], dyk[o], dhk);
        float xi[FP];
        load_row<FP>(x, i, F, xi);
        float ck = L.bh;    // the k -> l pre-activation without its displacement part
#pragma unroll
        for (int c = 0; c < FP; ++c) ck = fmaf(L.w1[3 + c], xi[c], ck);
        float S = 0.0f, T = 0.0f;
        const int deg = for_pairs<SL>(p, start, rec, s, pi, r2, list, [&](int cnt) __attribute__((always_inline)) {
            for (int k0 = 0; k0 < cnt; ++k0) {
#pragma clang fp contract(off)
                const float4 e = list[slot * kListRow + k0];
                const int32_t j = __float_as_int(e.w);
                const float dx = e.x, dy = e.y, dz = e.z;
                float xj[FP], dyl[OP];
                load_row<FP>(x, j, F, xj);
#pragma unroll
                for (int o = 0; o < OP; ++o) dyl[o] = o < O ? dyv[static_cast<int64_t>(j) * O + o] : 0.0f;
                const float wd = L.w1[0] * dx + L.w1[1] * dy + L.w1[2] * dz;
                // l -> k: input [d; x_l], cotangent dy_k
                float a = L.bh + wd;
#pragma unroll
                for (int c = 0; c < FP; ++c) a += L.w1[3 + c] * xj[c];
                const float r = fmaxf(a, 0.0f);
#pragma unroll
                for (int o = 0; o < OP; ++o) gW2[o] += dyk[o] * r;
                const float da = a > 0.0f ? dhk : 0.0f;
                gW1[0] += da * dx;
                gW1[1] += da * dy;
                gW1[2] += da * dz;
#pragma unroll
                for (int c = 0; c < FP; ++c) gW1[3 + c] += da * xj[c];
                gb1 += da;
                T += da;
                // k -> l: input [-d; x_k], cotangent dy_l
                float dhl = 0.0f;
#pragma unroll
                for (int o = 0; o < OP; ++o) dhl += L.w2[o] * dyl[o];
                S += ck - wd > 0.0f ? dhl : 0.0f;
            }
        });
        // input gradients of point i: W1^T times the lane sums of da (over hidden units and slots)
        if (dxo || dpo) put_input_grads<FP>(L.w1, S, T, i, F, dxo, dpo);
        // every message into i carries b2: db2 += deg(i) dy_i
#pragma unroll
        for (int o = 0; o < OP; ++o) gb2[o] = fmaf(static_cast<float>(deg), dyk[o], gb2[o]);
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
