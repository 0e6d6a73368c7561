// Learned closure of the treecode: training data, the network, training.
//
// The paper's treecode represents an accepted cell by its monopole (§3.1).
// The closure adds, for a body x and an accepted cell c (centre of mass C,
// mass M, side s, traceless quadrupole Q), a correction predicted by a small
// network from features of the pair:
//   f = [(x - C)/s (3), Q/(M s^2) (6), ln(M/mbar) (1)],  mbar = total mass / n,
//   yhat = MLP(f) (3),  a += G [ a_mono + (M s^2/|x - C|^4) yhat ].
// The training target is the residual in units of the quadrupole scale
//   y = (a_exact - a_mono) |x - C|^4 / (M s^2)   (G = 1),
// where a_exact sums the cell's bodies directly.  The network is
// 10-64-64-3 with GELU (tanh form); its products run on BF16 matrix-core
// instructions with FP32 accumulation (training: 16x16x16 tiles;
// inference: net_tile in closure.h) with FP32 master weights, trained
// by mean squared error and Adam.
//
// This file: residual generation (one wave per target body lists its accepted
// cells by the batched level-order walk of the force kernel with the box shrunk
// to the body; then the pairs are computed side by side), the network's forward and backward passes, the Adam update.
#include "tc_internal.h"
#include "closure.h"
#include "walk_common.h"

#include <math.h>

namespace tc {

namespace {

// ------------------------------------------------------------ residuals ----

constexpr int kStack = 320;                       // range stack per wave (bound as in force.hip)

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Walk for one body (the box shrunk to a point) at the prepared opening
// radii; on_round(accept, b) runs with the whole wave once per round: lane j
// tested the cell at level-order index b, and accept says whether the body is
// far enough from it.  3D.
template <typename F>
__device__ void walk_point(const WalkCell* __restrict__ walk, uint32_t* S, double px, double py, double pz,
                           F&& on_round) {
    constexpr int R = 8, RP = kWave / R;
    constexpr int kReserve = (R - 1) * 21 + R;
    static_assert(kStack >= kWave + kReserve + kWave, "stack bound");
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
    if (lane == 0) S[0] = 0u;
    wave_lds_sync();
    int top = 1;
    while (top > 0) {
        const int nr = (top + kWave + kReserve <= kStack) ? min(top, RP) : 1;
        const int rr = lane / R, j = lane % R;
        uint32_t packed = 0;
        if (rr < nr) packed = S[top - 1 - rr];
        top -= nr;
        const int rlen = (int)(packed & 7u) + 1;
        const bool vc = rr < nr && j < rlen;
        const uint32_t b = (packed >> 3) + (uint32_t)j;
        wave_lds_sync();
        WalkCell wc;
        if (vc) {
            wc = walk[b];
        } else {
            wc.cx = wc.cy = wc.cz = 0.0;
            wc.rcrit2 = INFINITY;
            wc.m = 0.f;
            wc.a = 0;
            wc.b = 0;
            wc.pad = 0;
        }
        const double dx = wc.cx - px, dy = wc.cy - py, dz = wc.cz - pz;
        const double d2 = (dx * dx + dy * dy) + dz * dz;
        const bool leaf = vc && wc.b < 0;
        const bool accept = vc && d2 > wc.rcrit2;
        const bool opened = vc && !accept && !leaf;
        const uint64_t O = __ballot(opened);
        if (opened) S[top + __popcll(O & below)] = ((uint32_t)wc.a << 3) | (uint32_t)(wc.b - 1);
        top += __popcll(O);
        wave_lds_sync();
        on_round(accept, b);
    }
}

// A pair's key in the order by cell: its cell's level-order index, or for the
// cells from `hot` on one of kResidColdKeys by its target (only there if there
// are such cells).
__device__ __forceinline__ uint32_t pair_key(uint32_t b, uint32_t t, uint32_t hot) {
    return b < hot ? b : hot + t % kResidColdKeys;
}

// One wave per target.  Count pass: pairs per target; list pass (LIST): the
// accepted cells (pre-order) at the scanned offsets, the pairs per key, and in
// the first two words of the pair's y the target's number and the pair's rank
// within its key.
template <bool LIST>
__global__ void __launch_bounds__(256) k_resid_walk(const WalkCell* __restrict__ walk, const Body* __restrict__ bodies,
                                                    const uint32_t* __restrict__ bfs2pre,
                                                    const uint32_t* __restrict__ inv_perm,
                                                    DevParams* __restrict__ prm, int64_t n,
                                                    const int32_t* __restrict__ targets, int nt,
                                                    uint32_t* __restrict__ counts, const uint32_t* __restrict__ offs,
                                                    int64_t cap, float* __restrict__ yout,
                                                    int32_t* __restrict__ cell_out, uint32_t* __restrict__ key_count,
                                                    uint32_t hot) {
    __shared__ uint32_t s_stack[4][kStack];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & (kWave - 1);
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
    const int t = blockIdx.x * 4 + wv;
    if (t >= nt) return;
    const int64_t o = targets[t];
    if (o < 0 || o >= n) {                     // no pairs for an index outside the bodies
        if (lane == 0) {
            atomicOr(&prm->status, kFlagBadIndex);
            if (!LIST) counts[t] = 0u;
        }
        return;
    }
    int64_t k = LIST ? (int64_t)offs[t] : 0;
    if (LIST && k >= cap) return;
    const Body me = bodies[inv_perm[o]];
    walk_point(walk, s_stack[wv], me.x, me.y, me.z, [&](bool accept, uint32_t b) {
        const uint64_t A = __ballot(accept);
        if (LIST) {
            const int64_t at = k + __popcll(A & below);
            const bool write = accept && at < cap;
            const uint64_t cold = __ballot(write && b >= hot);
            uint32_t rank = 0;
            if (cold) {
                if (lane == 0) rank = atomicAdd(&key_count[pair_key(hot, (uint32_t)t, hot)], (uint32_t)__popcll(cold));
                rank = (uint32_t)__builtin_amdgcn_readfirstlane((int)rank) + (uint32_t)__popcll(cold & below);
            }
            if (write) {
                if (b < hot) rank = atomicAdd(&key_count[b], 1u);
                cell_out[at] = (int32_t)bfs2pre[b];
                yout[at * 3] = __int_as_float(t);
                yout[at * 3 + 1] = __uint_as_float(rank);
            }
        }
        k += __popcll(A);
    });
    if (!LIST && lane == 0) counts[t] = (uint32_t)k;
}

// Counters of k_resid_pairs, zeroed beforehand: [0] the groups listed, then a
// line per queue for the groups and for the lots handed out.
constexpr int kQueues = 16, kLine = 32, kCounters = (1 + 2 * kQueues) * kLine;
static_assert(kCounters <= kResidMaxTargets, "the counters lie where the targets' counts were");

// The pairs by key.  Their order within a key varies from run to run; no
// pair's result depends on it.
__global__ void __launch_bounds__(256) k_resid_order(const int32_t* __restrict__ cell, const float* __restrict__ y,
                                                     const uint32_t* __restrict__ total, int64_t cap,
                                                     const uint32_t* __restrict__ pre2bfs,
                                                     const uint32_t* __restrict__ key_off, uint32_t hot,
                                                     uint32_t* __restrict__ order, uint32_t* __restrict__ ctr) {
    const int64_t P = (int64_t)*total < cap ? (int64_t)*total : cap;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    for (int64_t k = i; k < kCounters; k += (int64_t)gridDim.x * blockDim.x) ctr[k] = 0u;
    for (int64_t k = i; k < P; k += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t b = pre2bfs[cell[k]], t = __float_as_uint(y[k * 3]);
        order[key_off[pair_key(b, t, hot)] + __float_as_uint(y[k * 3 + 1])] = (uint32_t)k;
    }
}

// The sums of the pairs: the exact softened sum over the cell's bodies (FP64,
// fixed order) against the monopole.  Pairs of one cell are taken up to four at
// once, each body read once for all of them: those of a cell with more than
// kPairHuge bodies by a block, of more than kPairLong by a wave; the others go
// four to a wave on 16 lanes each.  Which way a pair goes, and so the order of
// its sum, depends on its cell only (and on the system's size: k_resid_small).  The blocks first take the groups of four
// in the order by cell that hold pairs of huge cells (k_resid_huge lists them),
// then their waves take the other pairs, kTask at a time; big cells come first.
// Both are handed out by kQueues counters, each the places of one remainder:
// from a single one, at some 15 ns a claim, the claims alone took 0.5 ms.
//
// Bound by the FP64 units, about 21 instructions per body and pair, for the
// large cells and by the latency of their few reads for the small ones: 1.05M
// pairs of 5.4e8 bodies (4,096 targets, 262,144 bodies) in 0.6 ms.  One wave per
// target going through its cells in turn, with sqrt and divide, took 3.1 ms; 16
// lanes or a wave per pair 2.1 ms, as one cell of four fifths of the bodies kept
// a wave busy that long.  kPairHuge: 4096 and 2048 are alike at 262,144 bodies
// (852 and 891 us for everything), at 1,000,001 4096 wins (1.96 and 2.11 ms).
constexpr int kTask = 8;                        // pairs a wave takes at a time
constexpr int kPairLanes = 16;
constexpr int kPairLong = 128;
constexpr int kPairHuge = 4096;
constexpr int kPairBlock = 512;
constexpr int kPairGrid = 512;                  // blocks the chip holds at once, two per CU

// The list follows the P pairs of the order.
__global__ void __launch_bounds__(256) k_resid_huge(const Cell* __restrict__ cells, const int32_t* __restrict__ cell,
                                                    uint32_t* order, const uint32_t* __restrict__ total, int64_t cap,
                                                    uint32_t* __restrict__ ctr) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t P = (int64_t)*total < cap ? (int64_t)*total : cap;
    uint32_t* list = order + P;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i0 = blockIdx.x * (int64_t)blockDim.x + (threadIdx.x & ~(kWave - 1)); i0 < P; i0 += stride) {
        const int64_t i = i0 + lane;
        const uint64_t H = __ballot(i < P && cells[cell[order[i]]].count > kPairHuge);
        const bool mine = lane < 16 && ((H >> (4 * lane)) & 15ull);
        const uint64_t G = __ballot(mine);
        if (!G) continue;
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&ctr[0], (uint32_t)__popcll(G));
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__popcll(G & ((1ull << lane) - 1ull));
        if (mine) list[at] = (uint32_t)(i0 / 4 + lane);
    }
}

struct Sum3 {
    double x, y, z;
};

__device__ __forceinline__ void add_body(Sum3& e, const Body& b, double x, double y, double z, double eps2) {
    const double dx = b.x - x, dy = b.y - y, dz = b.z - z;
    const double inv = walk::rsqrt64(fma(dz, dz, fma(dy, dy, fma(dx, dx, eps2))));
    const double w3 = b.m * inv * inv * inv;
    e.x = fma(w3, dx, e.x);
    e.y = fma(w3, dy, e.y);
    e.z = fma(w3, dz, e.z);
}

// Body j of the sums: FP32 inputs have a copy of 16 bytes a body, exactly the
// input, which halves what the sums read.
template <bool F32>
__device__ __forceinline__ Body sum_body(const Body* __restrict__ bodies, const float4* __restrict__ bodies32, int64_t j) {
    if (!F32) return bodies[j];
    const float4 b = bodies32[j];
    Body o;
    o.x = b.x;
    o.y = b.y;
    o.z = b.z;
    o.m = b.w;
    return o;
}

__device__ __forceinline__ Sum3 shfl3(const Sum3& v, int l) {
    return {__shfl(v.x, l, kWave), __shfl(v.y, l, kWave), __shfl(v.z, l, kWave)};
}

// One step of the sum over the wave: lanes o apart add up.
__device__ __forceinline__ void fold(Sum3& v, int o) {
    v.x += __shfl_xor(v.x, o, kWave);
    v.y += __shfl_xor(v.y, o, kWave);
    v.z += __shfl_xor(v.z, o, kWave);
}

// The same of two sums at once: lanes with bit o keep b, the others a.
__device__ __forceinline__ Sum3 fold2(const Sum3& a, const Sum3& b, int o, bool hi) {
    const double x = __shfl_xor(hi ? a.x : b.x, o, kWave), y = __shfl_xor(hi ? a.y : b.y, o, kWave),
                 z = __shfl_xor(hi ? a.z : b.z, o, kWave);
    return {(hi ? b.x : a.x) + x, (hi ? b.y : a.y) + y, (hi ? b.z : a.z) + z};
}

// The whole wave over the bodies [b0, b1) for T targets; afterwards the lanes
// from m * 64 / T on hold the sum of target m.
template <bool F32, int T>
__device__ __forceinline__ Sum3 wide_sum(const Body* __restrict__ bodies, const float4* __restrict__ bodies32, int64_t b0, int64_t b1, const Sum3 (&at)[T],
                                         double eps2) {
    const int lane = threadIdx.x & (kWave - 1);
    Sum3 e[T];
#pragma unroll
    for (int m = 0; m < T; ++m) e[m] = {0.0, 0.0, 0.0};
    for (int64_t j = b0 + lane; j < b1; j += 2 * kWave) {
        const Body b = sum_body<F32>(bodies, bodies32, j);
        Body c = sum_body<F32>(bodies, bodies32, min(j + kWave, b1 - 1));
        if (j + kWave >= b1) c.m = 0.0;                                      // adds nothing
#pragma unroll
        for (int m = 0; m < T; ++m) add_body(e[m], b, at[m].x, at[m].y, at[m].z, eps2);
#pragma unroll
        for (int m = 0; m < T; ++m) add_body(e[m], c, at[m].x, at[m].y, at[m].z, eps2);
    }
    const bool h5 = (lane & 32) != 0, h4 = (lane & 16) != 0;
    Sum3 v;
    if constexpr (T == 4) {
        v = fold2(fold2(e[0], e[2], 32, h5), fold2(e[1], e[3], 32, h5), 16, h4);
    } else if constexpr (T == 2) {
        v = fold2(e[0], e[1], 32, h5);
        fold(v, 16);
    } else {
        v = e[0];
        fold(v, 32);
        fold(v, 16);
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) fold(v, o);
    return v;
}

__device__ __forceinline__ double readlane64(double v, int l) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l),
                   hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// One lane's pair: its number, cell and target.
struct Pair {
    int64_t k;
    int cell, begin, count, level;
    Sum3 at;
};

__device__ __forceinline__ void put_pair(const Pair& p, const Sum3& r, const Moments* __restrict__ mom, double size,
                                         double eps2, float* yout) {
    const Moments& mo = mom[p.cell];
    const double M = mo.M, s = ldexp(size, -p.level);
    const double dcx = mo.com[0] - p.at.x, dcy = mo.com[1] - p.at.y, dcz = mo.com[2] - p.at.z;
    const double d2 = (dcx * dcx + dcy * dcy) + dcz * dcz;
    const double inv = 1.0 / sqrt(d2 + eps2);
    const double w3 = M * inv * inv * inv;
    // residual in units of the quadrupole scale M s^2 / d^4
    const double nrm = (d2 * d2) / (M * s * s);
    yout[p.k * 3] = (float)((r.x - w3 * dcx) * nrm);
    yout[p.k * 3 + 1] = (float)((r.y - w3 * dcy) * nrm);
    yout[p.k * 3 + 2] = (float)((r.z - w3 * dcz) * nrm);
}

// The wave's part (wave wv of nw) of the sums of `take` pairs from lane i on,
// all of one cell; the sum of pair i + m is at the returned lane shift m << shift.
template <bool F32>
__device__ __forceinline__ Sum3 run_sum(const Body* __restrict__ bodies, const float4* __restrict__ bodies32, const Pair& p, int i, int take, int wv, int nw,
                                        double eps2, int& shift) {
    const int64_t c0 = __builtin_amdgcn_readlane(p.begin, i), cn = __builtin_amdgcn_readlane(p.count, i);
    const int64_t part = (cn + nw - 1) / nw;
    const int64_t b0 = c0 + min(wv * part, cn), b1 = c0 + min((wv + 1) * part, cn);
    auto target = [&](int m) {
        return Sum3{readlane64(p.at.x, m), readlane64(p.at.y, m), readlane64(p.at.z, m)};
    };
    if (take >= 3) {
        const Sum3 a[4] = {target(i), target(i + 1), target(i + 2), target(i + take - 1)};
        shift = 4;
        return wide_sum<F32, 4>(bodies, bodies32, b0, b1, a, eps2);
    }
    shift = 5;
    if (take == 2) {
        const Sum3 a[2] = {target(i), target(i + 1)};
        return wide_sum<F32, 2>(bodies, bodies32, b0, b1, a, eps2);
    }
    const Sum3 a[1] = {target(i)};
    return wide_sum<F32, 1>(bodies, bodies32, b0, b1, a, eps2);
}

// Loads the pair at p0 + lane (lane < np) if its cell is on this side of
// kPairHuge: the other side's y may hold its result already.
template <bool HUGE>
__device__ __forceinline__ bool load_pair(Pair& p, int64_t p0, int np, const Body* __restrict__ bodies,
                                          const Cell* __restrict__ cells, const uint32_t* __restrict__ inv_perm,
                                          const int32_t* __restrict__ targets, const float* yout,
                                          const int32_t* __restrict__ cell_out, const uint32_t* __restrict__ order) {
    const int lane = threadIdx.x & (kWave - 1);
    p = {0, -1, 0, 0, 0, {0.0, 0.0, 0.0}};
    if (lane >= np) return false;
    p.k = order[p0 + lane];
    const int kc = cell_out[p.k];
    const Cell c = cells[kc];
    if ((c.count > kPairHuge) != HUGE) return false;
    p.cell = kc;
    p.begin = c.begin;
    p.count = c.count;
    p.level = c.level;
    const Body me = bodies[inv_perm[targets[__float_as_int(yout[p.k * 3])]]];
    p.at = {me.x, me.y, me.z};
    return true;
}

template <bool F32>
__global__ void __launch_bounds__(kPairBlock) k_resid_pairs(const Body* __restrict__ bodies,
                                                            const float4* __restrict__ bodies32,
                                                            const Cell* __restrict__ cells,
                                                            const Moments* __restrict__ mom,
                                                            const uint32_t* __restrict__ inv_perm,
                                                            const DevParams* __restrict__ prm,
                                                            const int32_t* __restrict__ targets, double eps2,
                                                            const uint32_t* __restrict__ total, int64_t cap,
                                                            float* yout, const int32_t* __restrict__ cell_out,
                                                            const uint32_t* __restrict__ order, uint32_t* ctr) {
    constexpr int kWaves = kPairBlock / kWave;
    __shared__ Sum3 s_part[kWaves][4];
    __shared__ uint32_t s_task;
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
    const int64_t P = (int64_t)*total < cap ? (int64_t)*total : cap;
    const double size = prm->size;
    const uint32_t* list = order + P;
    const uint32_t nlist = ctr[0], nq = min((uint32_t)kQueues, gridDim.x), queue = blockIdx.x % nq;
    uint32_t *groups = ctr + (1 + queue) * kLine, *lots = groups + kQueues * kLine;
    Pair p;
    for (;;) {
        if (threadIdx.x == 0) s_task = atomicAdd(groups, 1u) * nq + queue;
        __syncthreads();
        const uint32_t task = s_task;
        __syncthreads();
        if (task >= nlist) break;
        const int64_t p0 = (int64_t)list[task] * 4;
        uint64_t left = __ballot(load_pair<true>(p, p0, (int)min((int64_t)4, P - p0), bodies, cells, inv_perm, targets,
                                                 yout, cell_out, order));
        while (left) {
            const int i = __builtin_ctzll(left);
            const int take = __builtin_ctzll(~__ballot(p.cell == __builtin_amdgcn_readlane(p.cell, i)) >> i);
            int shift;
            const Sum3 v = run_sum<F32>(bodies, bodies32, p, i, take, wv, kWaves, eps2, shift);
            if ((lane & ((1 << shift) - 1)) == 0) s_part[wv][lane >> shift] = v;
            __syncthreads();
            if (wv == 0 && lane >= i && lane < i + take) {
                Sum3 r = s_part[0][lane - i];
                for (int w = 1; w < kWaves; ++w) {
                    const Sum3& q = s_part[w][lane - i];
                    r.x += q.x;
                    r.y += q.y;
                    r.z += q.z;
                }
                put_pair(p, r, mom, size, eps2, yout);
            }
            left &= ~(((1ull << take) - 1ull) << i);
            __syncthreads();
        }
    }
    for (;;) {
        uint32_t next = 0;
        if (lane == 0) next = atomicAdd(lots, 1u);
        next = (uint32_t)__builtin_amdgcn_readfirstlane((int)next);
        const int64_t p0 = ((int64_t)next * nq + queue) * kTask;
        if (p0 >= P) break;
        const int np = (int)min((int64_t)kTask, P - p0);
        const bool mine = load_pair<false>(p, p0, np, bodies, cells, inv_perm, targets, yout, cell_out, order);
        const uint32_t mask = (uint32_t)__ballot(mine), wide = (uint32_t)__ballot(mine && p.count > kPairLong);
        Sum3 r = {0.0, 0.0, 0.0};
        for (int i = 0; i < np;) {
            Sum3 v;
            int take, shift;
            if (!((mask >> i) & 1u)) {
                ++i;
                continue;
            }
            if ((wide >> i) & 1u) {
                const uint32_t other = ~(uint32_t)__ballot(p.cell == __builtin_amdgcn_readlane(p.cell, i)) >> i;
                take = min(__builtin_ctz(other), 4);
                v = run_sum<F32>(bodies, bodies32, p, i, take, 0, 1, eps2, shift);
            } else {
                constexpr int kPairs = kWave / kPairLanes;
                take = min(__builtin_ctz((wide | ~mask) >> i), kPairs);
                const int src = i + min(lane / kPairLanes, take - 1);
                const Sum3 a = shfl3(p.at, src);
                const int64_t b0 = __shfl(p.begin, src, kWave), b1 = b0 + __shfl(p.count, src, kWave);
                v = {0.0, 0.0, 0.0};
                // four bodies of a lane are read together: one after the
                // other, the groups waited for each
                for (int64_t j = b0 + lane % kPairLanes; j < b1; j += 4 * kPairLanes) {
                    Body b[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        b[u] = sum_body<F32>(bodies, bodies32, min(j + u * kPairLanes, b1 - 1));
                        if (j + u * kPairLanes >= b1) b[u].m = 0.0;      // adds nothing
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) add_body(v, b[u], a.x, a.y, a.z, eps2);
                }
#pragma unroll
                for (int o = kPairLanes / 2; o > 0; o >>= 1) fold(v, o);
                shift = 4;
            }
            const Sum3 got = shfl3(v, ((lane - i) << shift) & (kWave - 1));
            if (lane >= i && lane < i + take) r = got;
            i += take;
        }
        if (mine) put_pair(p, r, mom, size, eps2, yout);
    }
}

// The features of a pair.
__device__ __forceinline__ void put_features(float* __restrict__ f, const Sum3& at, const Moments& mo, int level,
                                             double size, double mbar) {
    const double s = ldexp(size, -level);
    const double M = mo.M;
    f[0] = (float)((at.x - mo.com[0]) / s);
    f[1] = (float)((at.y - mo.com[1]) / s);
    f[2] = (float)((at.z - mo.com[2]) / s);
    for (int q = 0; q < 6; ++q) f[3 + q] = (float)(mo.Q[q] / (M * s * s));
    f[9] = (float)log(M / mbar);
}

// The features, one block per target.
__global__ void __launch_bounds__(256) k_resid_features(const Body* __restrict__ bodies,
                                                        const Cell* __restrict__ cells,
                                                        const Moments* __restrict__ mom,
                                                        const uint32_t* __restrict__ inv_perm,
                                                        const DevParams* __restrict__ prm, int64_t n,
                                                        const int32_t* __restrict__ targets,
                                                        const uint32_t* __restrict__ offs, int64_t cap,
                                                        const int32_t* __restrict__ cell_out,
                                                        float* __restrict__ feat) {
    const int t = blockIdx.x;
    const int64_t e = min((int64_t)offs[t + 1], cap);
    int64_t k = (int64_t)offs[t] + threadIdx.x;
    if (k >= e) return;
    const Body me = bodies[inv_perm[targets[t]]];
    const double mbar = mom[0].M / (double)n;
    const double size = prm->size;
    for (; k < e; k += blockDim.x) {
        const int64_t kc = cell_out[k];
        put_features(feat + k * 10, {me.x, me.y, me.z}, mom[kc], cells[kc].level, size, mbar);
    }
}

// The smallest systems' pairs in one launch: a wave per target, a lane per
// accepted cell and its few bodies, in order.  Bound by latency and launches; by
// way of the order by cell 50 bodies and one target took 95 us, 48 so (kResidSmall).
__global__ void __launch_bounds__(256) k_resid_small(const WalkCell* __restrict__ walk, const Body* __restrict__ bodies,
                                                     const Cell* __restrict__ cells, const Moments* __restrict__ mom,
                                                     const uint32_t* __restrict__ bfs2pre,
                                                     const uint32_t* __restrict__ inv_perm,
                                                     const DevParams* __restrict__ prm, int64_t n,
                                                     const int32_t* __restrict__ targets, int nt, double eps2,
                                                     const uint32_t* __restrict__ offs, int64_t cap,
                                                     float* __restrict__ feat, float* __restrict__ yout,
                                                     int32_t* __restrict__ cell_out) {
    __shared__ uint32_t s_stack[4][kStack];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & (kWave - 1);
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
    const int t = blockIdx.x * 4 + wv;
    if (t >= nt) return;
    int64_t k = offs[t];
    if ((int64_t)offs[t + 1] == k || k >= cap) return;   // no pairs (an index outside the bodies has none)
    const Body me = bodies[inv_perm[targets[t]]];
    const double mbar = mom[0].M / (double)n, size = prm->size;
    walk_point(walk, s_stack[wv], me.x, me.y, me.z, [&](bool accept, uint32_t b) {
        const uint64_t A = __ballot(accept);
        const int64_t at = k + __popcll(A & below);
        if (accept && at < cap) {
            const int kc = (int)bfs2pre[b];
            const Cell c = cells[kc];
            const Pair p = {at, kc, c.begin, c.count, c.level, {me.x, me.y, me.z}};
            Sum3 r = {0.0, 0.0, 0.0};
#pragma unroll 4
            for (int64_t j = c.begin; j < (int64_t)c.begin + c.count; ++j) add_body(r, bodies[j], me.x, me.y, me.z, eps2);
            put_pair(p, r, mom, size, eps2, yout);
            put_features(feat + at * 10, p.at, mom[kc], c.level, size, mbar);
            cell_out[at] = kc;
        }
        k += __popcll(A);
    });
}

__global__ void k_inverse_perm(const uint32_t* __restrict__ perm, int64_t n, uint32_t* __restrict__ inv) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        inv[perm[i]] = (uint32_t)i;
}

// --------------------------------------------------------------- network ----

__device__ __forceinline__ uint16_t f2bf(float f) {        // round to nearest, ties to even
    return __builtin_bit_cast(uint16_t, (__bf16)f);
}

// Inference on rows of stored features, with the matrix-core routine of
// the learned walk (net_tile): one wave per 64 samples, 16 at a time.
__global__ void __launch_bounds__(256) k_mlp_forward(const float* __restrict__ feat, int64_t nrows,
                                                     const int32_t* __restrict__ idx, int64_t nb,
                                                     const MlpState* __restrict__ st, float* __restrict__ yhat,
                                                     uint32_t* status) {
    __shared__ NetF N;
    load_net_frags(st, N, threadIdx.x, blockDim.x);
    __syncthreads();
    const int wv = threadIdx.x >> 6, l = threadIdx.x & (kWave - 1), g = l >> 4, r = l & 15;
    const int64_t s0 = ((int64_t)blockIdx.x * 4 + wv) * kWave;
    if (s0 >= nb) return;
    for (int tile = 0; tile < 4; ++tile) {
        const int64_t s = s0 + 16 * tile + r;
        bool valid = s < nb;
        int64_t src = valid ? (idx ? (int64_t)idx[s] : s) : 0;
        if (valid && (src < 0 || src >= nrows)) {  // a row outside feat: left out, flagged
            atomicOr(status, kFlagBadIndex);
            valid = false;
            src = 0;
        }
        short4_t x;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 4 * g + j;
            x[j] = (valid && k < kNIn) ? bf16_bits(feat[src * kNIn + k]) : (short)0;
        }
        const float4_t y = net_tile(N, x);
        if (g == 0 && valid)
            for (int q = 0; q < kNOut; ++q) yhat[s * kNOut + q] = y[q];
    }
}

// One training block: forward, squared error, backward for 64 samples; writes
// this block's gradient sums (canonical order) and squared error.
//
// A wave does 16 samples, and every layer is computed transposed (Z^T = W^T
// H^T, as in net_tile): lane 16 g + r holds the units 16 t + 4 g + q (q < 4) of
// sample r for each tile t of 16 units, which is both what a 16x16x16 product
// gives it and what the next one takes from it as its operand, forward and
// backward, so activations and their gradients stay in registers.  The
// weights' gradients are sums over the samples: for those the block's four
// waves leave their values in LDS by unit, and each takes a quarter of the
// output tiles.  Bound by latency at the batches in use (64 blocks for 4,096
// samples).  One wave per 64 samples with every layer going through LDS and
// the operands read from it two bytes at a time took 28 us for 4,096 samples.
constexpr int kTrainWaves = 4;
constexpr int kTrainPad = kMlpBlock + 4;         // samples per unit's row (8-byte aligned rows)

struct __align__(16) TrainLds {
    uint16_t w2[kNHid][kNHid + 4];
    uint16_t x[16][kTrainPad], dy[16][kTrainPad];                       // [feature or output][sample]
    uint16_t h1[kNHid][kTrainPad], h2[kNHid][kTrainPad];                // [unit][sample]
    uint16_t d1[kNHid][kTrainPad], d2[kNHid][kTrainPad];
    float f1[kNHid][kMlpBlock + 1], f2[kNHid][kMlpBlock + 1];           // the same gradients, FP32
    float out[4][kMlpBlock + 1];                                        // output gradients and squared errors
};

__device__ __forceinline__ float4_t mfma16(short4_t a, short4_t b, float4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// Reads of the network state, whose arrays are only aligned to 4 bytes.
typedef short short4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef short short8_a4 __attribute__((ext_vector_type(8), aligned(4)));
typedef float float4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// Four consecutive samples of a unit.
__device__ __forceinline__ short4_t row4(const uint16_t* p) { return *reinterpret_cast<const short4_t*>(p); }

// The sum over the 64 samples of A(i, s) B(s, j), rows i0 and j0 of unit-major
// arrays: samples in order.
__device__ __forceinline__ float4_t over_samples(const uint16_t (*A)[kTrainPad], int i0, const uint16_t (*B)[kTrainPad],
                                                 int j0) {
    const int l = threadIdx.x & (kWave - 1), r = l & 15, kq = 4 * (l >> 4);
    float4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k0 = 0; k0 < kMlpBlock; k0 += 16) acc = mfma16(row4(&A[i0 + r][k0 + kq]), row4(&B[j0 + r][k0 + kq]), acc);
    return acc;
}

__global__ void __launch_bounds__(kTrainWaves * kWave) k_mlp_train(const float* __restrict__ feat,
                                                                   const float* __restrict__ ytrue, int64_t nrows,
                                                                   const int32_t* __restrict__ idx, int64_t nb,
                                                                   MlpState* __restrict__ st, uint32_t* status) {
    __shared__ TrainLds L;
    const int t = threadIdx.x, w = t / kWave, l = t & (kWave - 1), g = l >> 4, r = l & 15;
    const int sl = 16 * w + r;                       // this lane's sample in the block
    // the sample's row, features 4 g .. 4 g + 3
    const int64_t s = (int64_t)blockIdx.x * kMlpBlock + sl;
    bool valid = s < nb;
    int64_t src = valid ? (idx ? (int64_t)idx[s] : s) : 0;
    if (valid && (src < 0 || src >= nrows)) {        // a row outside feat: left out, flagged
        if (g == 0) atomicOr(status, kFlagBadIndex);
        valid = false;
        src = 0;
    }
    short4_t x = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (valid && 4 * g + j < kNIn) x[j] = (short)f2bf(feat[src * kNIn + 4 * g + j]);
    float yt[kNOut];
#pragma unroll
    for (int q = 0; q < kNOut; ++q) yt[q] = valid && g == 0 ? ytrue[src * kNOut + q] : 0.f;
    // weights: W2 to LDS (read both ways), the others' operands from memory
    for (int i = t; i < kNHid * kNHid / 8; i += kTrainWaves * kWave) {
        const short8_t v = reinterpret_cast<const short8_a4*>(st->w2)[i];
        const int row = i / (kNHid / 8), c = 8 * (i % (kNHid / 8));
        *reinterpret_cast<short4_t*>(&L.w2[row][c]) = __builtin_shufflevector(v, v, 0, 1, 2, 3);
        *reinterpret_cast<short4_t*>(&L.w2[row][c + 4]) = __builtin_shufflevector(v, v, 4, 5, 6, 7);
    }
    short4_t a1[4], a3[4], a3t[4];                   // W1^T, W3^T and W3 by tile
    float4_t b1[4], b2[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            a1[h][j] = (short)st->w1[(4 * g + j) * kNHid + 16 * h + r];
            a3[h][j] = (short)st->w3[(16 * h + 4 * g + j) * 16 + r];
        }
        a3t[h] = *reinterpret_cast<const short4_a4*>(&st->w3[(16 * h + r) * 16 + 4 * g]);
        b1[h] = *reinterpret_cast<const float4_a4*>(&st->b1[16 * h + 4 * g]);
        b2[h] = *reinterpret_cast<const float4_a4*>(&st->b2[16 * h + 4 * g]);
    }
    const float4_t b3 = *reinterpret_cast<const float4_a4*>(&st->b3[4 * g]);
#pragma unroll
    for (int j = 0; j < 4; ++j) L.x[4 * g + j][sl] = (uint16_t)x[j];
    const float4_t zero = {0.f, 0.f, 0.f, 0.f};

    // forward
    float4_t z1[4], z2[4];
    short4_t h1[4], h2[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        z1[h] = mfma16(a1[h], x, zero) + b1[h];
        h1[h] = gelu_pack(z1[h]);
#pragma unroll
        for (int q = 0; q < 4; ++q) L.h1[16 * h + 4 * g + q][sl] = (uint16_t)h1[h][q];
    }
    __syncthreads();                                 // W2
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        float4_t d = zero;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            short4_t a;
#pragma unroll
            for (int j = 0; j < 4; ++j) a[j] = (short)L.w2[16 * k + 4 * g + j][16 * h + r];
            d = mfma16(a, h1[k], d);
        }
        z2[h] = d + b2[h];
        h2[h] = gelu_pack(z2[h]);
#pragma unroll
        for (int q = 0; q < 4; ++q) L.h2[16 * h + 4 * g + q][sl] = (uint16_t)h2[h][q];
    }
    float4_t y = zero;
#pragma unroll
    for (int k = 0; k < 4; ++k) y = mfma16(a3[k], h2[k], y);
    y = y + b3;

    // loss gradient (outputs 0..2 are in lane group 0)
    const float scale = 2.0f / (float)(nb * kNOut);
    short4_t dy = {0, 0, 0, 0};
    if (g == 0) {
        float se = 0.f;
#pragma unroll
        for (int q = 0; q < kNOut; ++q) {
            const float d = valid ? y[q] - yt[q] : 0.f;
            se += d * d;
            const float df = d * scale;
            L.out[q][sl] = df;
            dy[q] = (short)f2bf(df);
        }
        L.out[kNOut][sl] = se;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) L.dy[4 * g + q][sl] = (uint16_t)dy[q];

    // backward: dz2 = (dy W3^T) gelu'(z2), dz1 = (dz2 W2^T) gelu'(z1)
    short4_t d2[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const float4_t d = mfma16(a3t[h], dy, zero);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float v = d[q] * gelu_grad_f(z2[h][q]);
            const int u = 16 * h + 4 * g + q;
            L.f2[u][sl] = v;
            d2[h][q] = (short)f2bf(v);
            L.d2[u][sl] = (uint16_t)d2[h][q];
        }
    }
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        float4_t d = zero;
#pragma unroll
        for (int k = 0; k < 4; ++k) d = mfma16(row4(&L.w2[16 * h + r][16 * k + 4 * g]), d2[k], d);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float v = d[q] * gelu_grad_f(z1[h][q]);
            const int u = 16 * h + 4 * g + q;
            L.f1[u][sl] = v;
            L.d1[u][sl] = f2bf(v);
        }
    }
    __syncthreads();

    // gradients over the 64 samples, in sample order
    float* part = st->partials[blockIdx.x];
#pragma unroll
    for (int c = 0; c < 4; ++c) {                    // dW2 = h1^T dz2
        const float4_t d = over_samples(L.h1, 16 * w, L.d2, 16 * c);
#pragma unroll
        for (int q = 0; q < 4; ++q) part[kOffW2 + (16 * w + 4 * g + q) * kNHid + 16 * c + r] = d[q];
    }
    {                                                // dW3 = h2^T dy
        const float4_t d = over_samples(L.h2, 16 * w, L.dy, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (r < kNOut) part[kOffW3 + (16 * w + 4 * g + q) * kNOut + r] = d[q];
    }
    {                                                // dW1 = x^T dz1
        const float4_t d = over_samples(L.x, 0, L.d1, 16 * w);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (4 * g + q < kNIn) part[kOffW1 + (4 * g + q) * kNHid + 16 * w + r] = d[q];
    }
    // biases and the squared error: a thread each
    const float* row = nullptr;
    int to = 0;
    if (t < kNHid) {
        row = L.f2[t];
        to = kOffB2 + t;
    } else if (t < 2 * kNHid) {
        row = L.f1[t - kNHid];
        to = kOffB1 + t - kNHid;
    } else if (t < 2 * kNHid + kNOut + 1) {
        row = L.out[t - 2 * kNHid];
        to = t < 2 * kNHid + kNOut ? kOffB3 + t - 2 * kNHid : kNParam;
    }
    if (row) {
        float acc = 0.f;
#pragma unroll 16
        for (int k = 0; k < kMlpBlock; ++k) acc += row[k];
        part[to] = acc;
    }
}

// Refresh the padded BF16 weights and the biases from the FP32 masters.
__device__ void refresh_copy(MlpState* st, int p) {
    const float w = st->master[p];
    if (p < kOffB1) {
        st->w1[(p / kNHid) * kNHid + p % kNHid] = f2bf(w);
    } else if (p < kOffW2) {
        st->b1[p - kOffB1] = w;
    } else if (p < kOffB2) {
        st->w2[p - kOffW2] = f2bf(w);
    } else if (p < kOffW3) {
        st->b2[p - kOffB2] = w;
    } else if (p < kOffB3) {
        const int q = p - kOffW3;
        st->w3[(q / kNOut) * 16 + q % kNOut] = f2bf(w);
    } else {
        st->b3[p - kOffB3] = w;
    }
}

// Sum the blocks' gradients in block order, then one Adam step on the
// masters (step counts from 1) and a refresh of the BF16 copies.  The
// partials are read sixteen blocks at a time: one after the other they took
// 17 us for 64 blocks.
constexpr int kAdamThreads = 64;

__global__ void __launch_bounds__(kAdamThreads) k_mlp_adam(MlpState* __restrict__ st, int nblocks, int64_t nb, float lr,
                                                           int step, float* __restrict__ grad_out) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p > kNParam) return;
    float g = 0.f;
    int b = 0;
    for (; b + 16 <= nblocks; b += 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = st->partials[b + u][p];
#pragma unroll
        for (int u = 0; u < 16; ++u) g += v[u];
    }
    for (; b < nblocks; ++b) g += st->partials[b][p];
    if (p == kNParam) {
        st->loss = g / (float)(nb * kNOut);
        return;
    }
    if (grad_out) grad_out[p] = g;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float m = b1 * st->m[p] + (1.f - b1) * g;
    const float v = b2 * st->v[p] + (1.f - b2) * g * g;
    st->m[p] = m;
    st->v[p] = v;
    const float mh = m / (1.f - powf(b1, (float)step));
    const float vh = v / (1.f - powf(b2, (float)step));
    st->master[p] = st->master[p] - lr * mh / (sqrtf(vh) + eps);
    refresh_copy(st, p);
}

__global__ void __launch_bounds__(256) k_mlp_load(MlpState* __restrict__ st, const float* __restrict__ params) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p == 0) st->loss = 0.f;
    if (p >= kNParam) return;
    st->master[p] = params[p];
    st->m[p] = 0.f;
    st->v[p] = 0.f;
    refresh_copy(st, p);
    // padding of the BF16 tiles and b3
    if (p < (16 - kNIn) * kNHid) st->w1[kNIn * kNHid + p] = 0;
    if (p < kNHid * 16) {
        const int c = p % 16;
        if (c >= kNOut) st->w3[p] = 0;
    }
    if (p < 16 - kNOut) st->b3[kNOut + p] = 0.f;
}

__global__ void __launch_bounds__(256) k_mlp_get(const MlpState* __restrict__ st, float* __restrict__ params) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < kNParam) params[p] = st->master[p];
}

}  // namespace

// ------------------------------------------------------------ launchers ----

hipError_t launch_inverse_perm(const uint32_t* perm, int64_t n, uint32_t* inv, hipStream_t s) {
    hipLaunchKernelGGL(k_inverse_perm, dim3(grid_for(n)), dim3(256), 0, s, perm, n, inv);
    return hipGetLastError();
}

hipError_t launch_resid_count(const WalkCell* walk, const Body* bodies, const uint32_t* bfs2pre,
                              const uint32_t* inv_perm, DevParams* prm, int64_t n, const int32_t* targets, int nt,
                              uint32_t* counts, hipStream_t s) {
    hipLaunchKernelGGL(k_resid_walk<false>, dim3((unsigned)((nt + 3) / 4)), dim3(256), 0, s, walk, bodies, bfs2pre,
                       inv_perm, prm, n, targets, nt, counts, (const uint32_t*)nullptr, (int64_t)0, (float*)nullptr,
                       (int32_t*)nullptr, (uint32_t*)nullptr, 0u);
    return hipGetLastError();
}

hipError_t launch_resid_pairs(const WalkCell* walk, const Body* bodies, const float4* bodies32, const Cell* cells, const Moments* mom,
                              const uint32_t* bfs2pre, const uint32_t* pre2bfs, const uint32_t* inv_perm,
                              DevParams* prm, int64_t n, int64_t cmax, const int32_t* targets, int nt, double eps2,
                              const uint32_t* offs, int64_t cap, uint32_t* key_count, uint32_t* key_off,
                              uint32_t* key_part, uint32_t* ctr, float* feat, float* y, int32_t* cell_out,
                              hipStream_t s) {
    if (cap <= 0) return hipSuccess;
    if (n <= kResidSmall) {
        hipLaunchKernelGGL(k_resid_small, dim3((unsigned)((nt + 3) / 4)), dim3(256), 0, s, walk, bodies, cells, mom,
                           bfs2pre, inv_perm, (const DevParams*)prm, n, targets, nt, eps2, offs, cap, feat, y,
                           cell_out);
        return hipGetLastError();
    }
    const bool cold = cmax > kResidKeys;
    const int64_t nkeys = cold ? kResidKeys : cmax;
    const uint32_t hot = (uint32_t)(cold ? nkeys - kResidColdKeys : nkeys);
    const uint32_t* total = offs + nt;
    // The order and the list lie in the P pairs' features until these are written.
    uint32_t* order = reinterpret_cast<uint32_t*>(feat);
    hipError_t e = launch_fill_u32(key_count, nkeys, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_resid_walk<true>, dim3((unsigned)((nt + 3) / 4)), dim3(256), 0, s, walk, bodies, bfs2pre,
                       inv_perm, prm, n, targets, nt, (uint32_t*)nullptr, offs, cap, y, cell_out, key_count, hot);
    e = launch_scan_u32(key_count, nkeys, key_off, key_part, (nkeys + kScanTile - 1) / kScanTile, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_resid_order, dim3(grid_for(cap)), dim3(256), 0, s, (const int32_t*)cell_out, (const float*)y,
                       total, cap, pre2bfs, (const uint32_t*)key_off, hot, order, ctr);
    hipLaunchKernelGGL(k_resid_huge, dim3(grid_for(cap)), dim3(256), 0, s, cells, (const int32_t*)cell_out,
                       order, total, cap, ctr);
    const int64_t groups = (cap + 3) / 4;
    const dim3 grid((unsigned)(groups < kPairGrid ? groups : kPairGrid));
    const auto pairs = bodies32 ? k_resid_pairs<true> : k_resid_pairs<false>;
    hipLaunchKernelGGL(pairs, grid, dim3(kPairBlock), 0, s, bodies, bodies32, cells, mom, inv_perm,
                       (const DevParams*)prm, targets, eps2, total, cap, y, (const int32_t*)cell_out,
                       (const uint32_t*)order, ctr);
    hipLaunchKernelGGL(k_resid_features, dim3((unsigned)nt), dim3(256), 0, s, bodies, cells, mom, inv_perm,
                       (const DevParams*)prm, n, targets, offs, cap, (const int32_t*)cell_out, feat);
    return hipGetLastError();
}

hipError_t launch_mlp_load(MlpState* st, const float* params, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_load, dim3((kNParam + 255) / 256), dim3(256), 0, s, st, params);
    return hipGetLastError();
}

hipError_t launch_mlp_get(const MlpState* st, float* params, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_get, dim3((kNParam + 255) / 256), dim3(256), 0, s, st, params);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const MlpState* st, const float* feat, int64_t nrows, const int32_t* idx, int64_t nb,
                              float* yhat, uint32_t* status, hipStream_t s) {
    const unsigned blocks = (unsigned)((nb + 4 * kWave - 1) / (4 * kWave));
    hipLaunchKernelGGL(k_mlp_forward, dim3(blocks), dim3(256), 0, s, feat, nrows, idx, nb, st, yhat, status);
    return hipGetLastError();
}

hipError_t launch_mlp_step(MlpState* st, const float* feat, const float* y, int64_t nrows, const int32_t* idx,
                           int64_t nb, float lr, int step, float* grad_out, uint32_t* status, hipStream_t s) {
    const int blocks = (int)((nb + kMlpBlock - 1) / kMlpBlock);
    hipLaunchKernelGGL(k_mlp_train, dim3(blocks), dim3(kTrainWaves * kWave), 0, s, feat, y, nrows, idx, nb, st, status);
    hipLaunchKernelGGL(k_mlp_adam, dim3((kNParam + kAdamThreads) / kAdamThreads), dim3(kAdamThreads), 0, s, st, blocks, nb, lr, step,
                       grad_out);
    return hipGetLastError();
}

}  // namespace tc
