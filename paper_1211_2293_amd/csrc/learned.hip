// Walk and force summation with the learned closure (3D).
//
// The walk of the plain kernel with two opening radii, theta_L (large, the
// learned walk) and theta_P (the plain walk it stands in for), and a mode
// per stacked range:
//   mode L: a cell accepted at both radii is a plain monopole entry; a cell
//           accepted at theta_L but opened at theta_P is a learned cell; a
//           cell opened at theta_L is opened (children stay in mode L);
//   mode P: the plain walk at theta_P (children stay in mode P).
// For a learned cell the network predicts the normalised residual for each
// of the group's bodies; if the largest predicted residual relative to the
// monopole, |yhat| s^2 / |x - C|^2, over the group exceeds tau the cell falls
// back to the plain walk of its subtree at theta_P (its
// children in mode P, or its bodies directly if it is a leaf), otherwise it
// enters as a monopole entry plus, per body, G M s^2 yhat / |x - C|^4 (the
// network predicts the residual in units of the quadrupole scale).  With
// tau = 0 every learned cell falls back and the walk is exactly the plain
// walk at theta_P; with tau = inf it is the plain walk at theta_L plus the
// corrections.  The potential keeps the monopoles.
//
// One block of eight waves per group, as in the shared plain walk: each round
// tests one cell per thread, plain entries and the bodies of unaccepted leaves
// go to one LDS list that the waves sum in equal parts, and learned cells to a
// queue.  When the walk has no ranges left (or the queue is full) the queued
// cells' features are computed one cell per thread, the waves deal the cells
// among them, one network pass over the group's bodies each in tiles of 16
// samples (net_tiles in closure.h: activations stay in registers, weights are
// matrix-core fragments in LDS), and what falls back returns to the stack or
// the queue of leaves.  Places come from prefix sums, so every sum runs in the
// same order each time; the waves' sums are added in FP64 in wave order.
//
// What bounds it: the activations, 128 GELUs a body and learned cell at nine
// issue slots each, 32 of them per lane and tile.  With one wave per group
// (131,072 bodies, theta 0.8 / 0.5: some 400 learned cells a group) there was
// less than one wave per SIMD, every wave computed each cell's FP64 features,
// and the kernel took 6.8 ms; a block per group takes 2.5, four fifths of it
// issuing vector instructions (1,048,576 bodies, build included: 23.5 -> 18.6 ms).
#include "tc_internal.h"
#include "closure.h"
#include "walk_common.h"

#include <math.h>

namespace tc {
namespace {

using namespace walk;

constexpr int kNW = 8;                                // waves per block
constexpr int kThreads = kNW * kWave;
constexpr int kR = 8;                                 // cells per range
constexpr int kReserve = (kR - 1) * 21 + kR;          // ranges a depth-first descent adds at most
constexpr int kRanges = 4 * kThreads;
// Batches of ranges are popped up to here.  Above it lie, at the worst, one
// depth-first descent in mode L, a full queue's fallbacks, and one descent of
// these in mode P, which queues no learned cell; they are popped before the
// mode L ranges beneath them.
constexpr int kBatchTop = kRanges - 2 * kReserve - kThreads;
constexpr int kEntries = 1024;                        // list entries
constexpr int kFeat = 256;                            // learned cells whose features are held at once
static_assert(kBatchTop > kThreads, "stack too small for its bound");
static_assert(kEntries >= kThreads, "a round's cells must fit the list");
static_assert(kEntries * sizeof(float4) >= kNW * 4 * kWave * sizeof(double), "the waves' sums reuse the list");

// What the waves need of a learned cell: centre of mass, 1 / s, s^2, M s^2 and
// the BF16 features that do not depend on the body: a = Q_yy, Q_zz, Q_xy, Q_xz;
// b = Q_yz, ln(M / mbar), Q_xx and, afterwards, whether the cell was kept.
struct LearnedCell {
    double c[3], inv_s, ss, mss;
    short4_t a, b;
};

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) k_walk_force_learned(
    const WalkCell* __restrict__ walk, const double* __restrict__ rcp2, const Body* __restrict__ bodies,
    const float4* __restrict__ bodies32, const Cell* __restrict__ cells, const Moments* __restrict__ mom,
    const uint32_t* __restrict__ bfs2pre, const uint32_t* __restrict__ perm, const int32_t* __restrict__ gbeg,
    const int32_t* __restrict__ gcnt, uint32_t* queue, const MlpState* __restrict__ st, int lpl_log2, float G,
    float eps2, float tau, int64_t n, const DevParams* __restrict__ prm, float* __restrict__ acc,
    float* __restrict__ pot, int64_t* __restrict__ m2p_out, int64_t* __restrict__ p2p_out,
    int64_t* __restrict__ learned_out, int64_t* __restrict__ fallback_out) {
    __shared__ NetF N;
    __shared__ float4 L[kEntries];
    __shared__ uint32_t S[kRanges];
    __shared__ int2 s_leaf[kThreads];                 // queued leaves: first body, count
    __shared__ uint32_t s_loff[kThreads];             // their first places
    __shared__ uint32_t s_lrn[kThreads];              // queued learned cells
    __shared__ LearnedCell s_feat[kFeat];
    __shared__ short4_t s_x[kNW][kWave];              // features 0..3 per body
    __shared__ float4_t s_y[kNW][kWave];              // network outputs per body
    __shared__ double s_pos[3][kWave];                // the group's FP64 positions
    __shared__ uint64_t s_cnt[kNW];
    __shared__ uint32_t s_sum[kNW];
    __shared__ uint32_t s_next;
    load_net_frags(st, N, threadIdx.x, kThreads);

    const int t = (int)threadIdx.x, lane = t & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int lg = lane >> 4, lr = lane & 15;
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
    const int lpl = 1 << lpl_log2, slot = t >> lpl_log2, jj = t & (lpl - 1), slots = kThreads >> lpl_log2;
    const double size = prm->size;
    const double mbar = mom[0].M / (double)n;          // mean body mass (root cell)

    // four counts per wave, 16 bits apart: those of the waves before and of all
    auto block_counts = [&](uint64_t A, uint64_t B, uint64_t C, uint64_t D, uint64_t& before, uint64_t& total) {
        if (lane == 0)
            s_cnt[wv] = (uint64_t)__popcll(A) | (uint64_t)__popcll(B) << 16 | (uint64_t)__popcll(C) << 32 |
                        (uint64_t)__popcll(D) << 48;
        __syncthreads();
        before = total = 0;
#pragma unroll
        for (int w = 0; w < kNW; ++w) {
            const uint64_t v = s_cnt[w];
            if (w < wv) before += v;
            total += v;
        }
    };

    const GroupSched sched{queue, prm->ngroups, blockIdx.x / kXcd, (int)(blockIdx.x % kXcd), 1};
    for (int hop = 0; hop < kXcd; ++hop) {
        const int xq = (sched.home + hop) % kXcd;
        const uint32_t g_hi = sched.share_lo(xq + 1);
        if (wv == 0) {
            const uint32_t f = sched.first(xq, hop);
            if (lane == 0) s_next = f;
        }
        __syncthreads();
        uint32_t g = s_next;
        while (g < g_hi) {
            const int64_t i0 = gbeg[g];
            const int gn = gcnt[g];
            const int64_t i = i0 + lane;
            const bool valid = lane < gn;
            const Body me = bodies[valid ? i : i0];
            const double lox = uniform(wave_min(me.x)), hix = uniform(wave_max(me.x));
            const double loy = uniform(wave_min(me.y)), hiy = uniform(wave_max(me.y));
            const double loz = uniform(wave_min(me.z)), hiz = uniform(wave_max(me.z));
            const double rx = (lox + hix) * 0.5, ry = (loy + hiy) * 0.5, rz = (loz + hiz) * 0.5;
            const float xi = (float)(me.x - rx), yi = (float)(me.y - ry), zi = (float)(me.z - rz);
            const int ntiles = (gn + 15) >> 4;              // sample tiles holding bodies

            Acc a = {0.0, 0.0, 0.0, 0.0};
            double kx = 0.0, ky = 0.0, kz = 0.0;              // closure corrections
            int64_t nm2p = 0, np2p = 0, nlearn = 0, nfall = 0;
            int len = 0, nleaf = 0, nlrn = 0, top = 1;
            bool drain = false, full = false;                 // a list or queue is full; the learned cells' queue is
            if (wv == 0) {
                s_pos[0][lane] = me.x;
                s_pos[1][lane] = me.y;
                s_pos[2][lane] = me.z;
            }
            if (t == 0) S[0] = 0u;                            // root, mode L
            __syncthreads();
            for (;;) {
                if (drain || top == 0) {
                    // the queued leaves' bodies into the list: lpl lanes per
                    // leaf, places from the scanned counts, in windows that
                    // fit the list; each window is summed with what is there
                    const uint32_t c = t < nleaf ? (uint32_t)s_leaf[t].y : 0u;
                    uint32_t x = c;
#pragma unroll
                    for (int o = 1; o < kWave; o <<= 1) {
                        const uint32_t y = __shfl_up(x, o, kWave);
                        if (lane >= o) x += y;
                    }
                    if (lane == kWave - 1) s_sum[wv] = x;
                    __syncthreads();
                    uint32_t before = 0, total = 0, done = 0;
                    for (int w = 0; w < kNW; ++w) {
                        const uint32_t v = s_sum[w];
                        if (w < wv) before += v;
                        total += v;
                    }
                    s_loff[t] = before + x - c;
                    __syncthreads();
                    do {
                        const uint32_t end = min(total, done + (uint32_t)(kEntries - len));
                        for (int s = slot; s < nleaf; s += slots) {
                            const int2 lf = s_leaf[s];
                            const int32_t o = (int32_t)s_loff[s], k0 = max(0, (int32_t)done - o);
                            const int32_t to = lf.x + min(lf.y, (int32_t)end - o);
                            for (int32_t j = lf.x + k0 + jj, p = len + o + k0 + jj - (int32_t)done; j < to;
                                 j += lpl, p += lpl)
                                L[p] = body_entry(bodies, bodies32, j, rx, ry, rz);
                        }
                        len += (int)(end - done);
                        done = end;
                        __syncthreads();
                        const int per = ((len + kNW - 1) / kNW + 7) & ~7;
                        const int cnt = min(per, len - wv * per);
                        if (cnt > 0) flush<3, false, true>(L + wv * per, cnt, xi, yi, zi, eps2, a);
                        len = 0;
                        __syncthreads();
                    } while (done < total);
                    np2p += total;
                    nleaf = 0;
                    drain = false;
                    if (nlrn == 0 && top == 0) break;
                    if (top == 0 || full) {
                        for (int c0 = 0; c0 < nlrn; c0 += kFeat) {
                            const int m = min(kFeat, nlrn - c0);
                            if (t < m) {
                                const int64_t kc = bfs2pre[s_lrn[c0 + t]];
                                const Moments& mo = mom[kc];
                                const int lev = cells[kc].level;
                                const double s = ldexp(size, -lev), M = mo.M;
                                const double iq = 1.0 / (M * s * s);
                                LearnedCell q;
                                q.c[0] = mo.com[0];
                                q.c[1] = mo.com[1];
                                q.c[2] = mo.com[2];
                                q.inv_s = ldexp(1.0 / size, lev);   // exact: size is a power of two
                                q.ss = s * s;
                                q.mss = M * s * s;
                                q.a = short4_t{bf16_bits((float)(mo.Q[1] * iq)), bf16_bits((float)(mo.Q[2] * iq)),
                                               bf16_bits((float)(mo.Q[3] * iq)), bf16_bits((float)(mo.Q[4] * iq))};
                                q.b = short4_t{bf16_bits((float)(mo.Q[5] * iq)), bf16_bits((float)log(M / mbar)),
                                               bf16_bits((float)(mo.Q[0] * iq)), 0};
                                s_feat[t] = q;
                            }
                            __syncthreads();
                            for (int k = wv; k < m; k += kNW) {
                                const LearnedCell& q = s_feat[k];
                                const short4_t qb = q.b;
                                {
                                    const double ux = (s_pos[0][lane] - q.c[0]) * q.inv_s,
                                                 uy = (s_pos[1][lane] - q.c[1]) * q.inv_s,
                                                 uz = (s_pos[2][lane] - q.c[2]) * q.inv_s;
                                    s_x[wv][lane] =
                                        short4_t{bf16_bits((float)ux), bf16_bits((float)uy), bf16_bits((float)uz), qb[2]};
                                }
                                wave_lds_sync();
                                // the features a lane group feeds: g = 0: u (3) and Q_xx; g = 1: Q_yy,
                                // Q_zz, Q_xy, Q_xz; g = 2: Q_yz and ln(M / mbar); g = 3: zero padding
                                short4_t xc = {0, 0, 0, 0};
                                if (lg == 1) xc = q.a;
                                else if (lg == 2) xc = short4_t{qb[0], qb[1], 0, 0};
                                for (int tl = 0; tl < ntiles; tl += 2) {
                                    // the weight fragments are read from LDS per pair of tiles, not held in registers
                                    __asm__ volatile("" ::: "memory");
                                    const short4_t x0 = s_x[wv][16 * tl + lr], x1 = s_x[wv][(16 * tl + 16 + lr) & 63];
                                    short4_t xs[2] = {lg == 0 ? x0 : xc, lg == 0 ? x1 : xc};
                                    float4_t ys[2];
                                    if (tl + 1 < ntiles) net_tiles<2>(N, xs, ys);
                                    else net_tiles<1>(N, xs, ys);
                                    if (lg == 0) {
                                        s_y[wv][16 * tl + lr] = ys[0];
                                        if (tl + 1 < ntiles) s_y[wv][16 * tl + 16 + lr] = ys[1];
                                    }
                                }
                                wave_lds_sync();
                                const float4_t yo = s_y[wv][lane];
                                wave_lds_sync();
                                // predicted residual relative to the monopole: |yhat| s^2 / |x - C|^2
                                const double ex = s_pos[0][lane] - q.c[0], ey = s_pos[1][lane] - q.c[1],
                                             ez = s_pos[2][lane] - q.c[2];
                                const double r = 1.0 / ((ex * ex + ey * ey) + ez * ez);
                                const float ratio =
                                    sqrtf(yo[0] * yo[0] + yo[1] * yo[1] + yo[2] * yo[2]) * (float)(q.ss * r);
                                const bool keep = __ballot(valid && ratio > tau) == 0ull;
                                if (keep) {
                                    const float w = (float)(q.mss * r * r);     // quadrupole scale
                                    kx += (double)(w * yo[0]);
                                    ky += (double)(w * yo[1]);
                                    kz += (double)(w * yo[2]);
                                }
                                if (lane == 0) s_feat[k].b[3] = keep;
                            }
                            __syncthreads();
                            // kept cells are monopole entries, the others the plain
                            // walk of the cell at theta_P
                            WalkCell wc = load_cell(walk, t < m ? s_lrn[c0 + t] : 0u, t < m);
                            const bool kept = t < m && s_feat[t < m ? t : 0].b[3] != 0;
                            const bool leaf = t < m && !kept && wc.b < 0, open = t < m && !kept && !leaf;
                            const uint64_t K = __ballot(kept), P = __ballot(leaf), O = __ballot(open);
                            uint64_t bc, tc;
                            block_counts(O, K, P, 0ull, bc, tc);
                            if (kept)
                                L[len + (int)(bc >> 16 & 0xffffu) + __popcll(K & below)] =
                                    make_float4((float)(wc.cx - rx), (float)(wc.cy - ry), (float)(wc.cz - rz), wc.m);
                            if (leaf)
                                s_leaf[nleaf + (int)(bc >> 32 & 0xffffu) + __popcll(P & below)] =
                                    make_int2(wc.a, wc.b & 0x7fffffff);
                            if (open)
                                S[top + (int)(bc & 0xffffu) + __popcll(O & below)] =
                                    ((uint32_t)wc.a << 4) | 8u | (uint32_t)(wc.b - 1);
                            const int no = (int)(tc & 0xffffu), nk = (int)(tc >> 16 & 0xffffu),
                                      np = (int)(tc >> 32 & 0xffffu);
                            len += nk;
                            nleaf += np;
                            top += no;
                            nlearn += nk;
                            nm2p += nk;
                            nfall += no + np;
                            __syncthreads();
                        }
                        nlrn = 0;
                        full = false;
                        if (top == 0) continue;
                    }
                }
                // pop as many ranges as the stack's reserve allows
                const int nr = max(1, min(min(top, kThreads / kR), (kBatchTop - top) / (kR - 1)));
                const int rr = t / kR, j = t % kR;
                uint32_t packed = 0;
                if (rr < nr) packed = S[top - 1 - rr];
                const bool modeP = (packed >> 3) & 1u;
                const bool vc = rr < nr && j < (int)(packed & 7u) + 1;
                const uint32_t bidx = (packed >> 4) + (uint32_t)j;
                const WalkCell wc = load_cell(walk, bidx, vc);
                const double rp = vc ? rcp2[bidx] : INFINITY;
                const double dxm = fmax(fmax(lox - wc.cx, 0.0), wc.cx - hix);
                const double dym = fmax(fmax(loy - wc.cy, 0.0), wc.cy - hiy);
                const double dzm = fmax(fmax(loz - wc.cz, 0.0), wc.cz - hiz);
                const double d2 = (dxm * dxm + dym * dym) + dzm * dzm;
                const bool leaf = vc && wc.b < 0;
                const bool accL = vc && d2 > wc.rcrit2;
                const bool accP = vc && d2 > rp;
                const bool plain = modeP ? accP : accL && accP;
                const bool learned = !modeP && accL && !accP;
                const bool closed = modeP ? accP : accL;   // accepted in its own mode
                const bool opened = vc && !closed && !leaf;
                const bool direct = leaf && !closed;
                const uint64_t O = __ballot(opened), A = __ballot(plain), P = __ballot(direct), W = __ballot(learned);
                uint64_t before, total;
                block_counts(O, A, P, W, before, total);
                const int na = (int)(total >> 16 & 0xffffu), np = (int)(total >> 32 & 0xffffu),
                          nw = (int)(total >> 48);
                if (len + na > kEntries || nleaf + np > kThreads || nlrn + nw > kThreads) {
                    drain = true;                          // make room, then this round again
                    full = nlrn + nw > kThreads;
                    __syncthreads();
                    continue;
                }
                top -= nr;
                if (opened)
                    S[top + (int)(before & 0xffffu) + __popcll(O & below)] =
                        ((uint32_t)wc.a << 4) | (modeP ? 8u : 0u) | (uint32_t)(wc.b - 1);
                if (plain)
                    L[len + (int)(before >> 16 & 0xffffu) + __popcll(A & below)] =
                        make_float4((float)(wc.cx - rx), (float)(wc.cy - ry), (float)(wc.cz - rz), wc.m);
                if (direct)
                    s_leaf[nleaf + (int)(before >> 32 & 0xffffu) + __popcll(P & below)] =
                        make_int2(wc.a, wc.b & 0x7fffffff);
                if (learned) s_lrn[nlrn + (int)(before >> 48) + __popcll(W & below)] = bidx;
                top += (int)(total & 0xffffu);
                len += na;
                nleaf += np;
                nlrn += nw;
                nm2p += na;
                __syncthreads();
            }

            // the waves' sums, added in FP64 in wave order: one thread per
            // body and component
            double* part = reinterpret_cast<double*>(L);
            part[(wv * 4 + 0) * kWave + lane] = a.sx + kx;
            part[(wv * 4 + 1) * kWave + lane] = a.sy + ky;
            part[(wv * 4 + 2) * kWave + lane] = a.sz + kz;
            part[(wv * 4 + 3) * kWave + lane] = a.sp;
            if (wv == 0) {
                const uint32_t nx = sched.pop(xq);
                if (lane == 0) s_next = nx;
            }
            __syncthreads();
            for (int c = wv; c < 4 && valid; c += kNW) {
                double v = 0.0;
                for (int w = 0; w < kNW; ++w) v += part[(w * 4 + c) * kWave + lane];
                const int64_t o = perm[i];
                if (c < 3) {
                    acc[o * 3 + c] = (float)((double)G * v);
                } else {
                    const float mself = (float)bodies[i].m;
                    v += (double)(mself * __builtin_amdgcn_rsqf(eps2));
                    pot[o] = (float)((double)G * v);
                }
            }
            if (t == 0) {
                m2p_out[g] = nm2p;
                p2p_out[g] = np2p;
                learned_out[g] = nlearn;
                fallback_out[g] = nfall;
            }
            g = s_next;
            __syncthreads();                         // the list is reused by the next group
        }
        __syncthreads();                             // s_next is rewritten
    }
}

__global__ void k_reset_queue_l(uint32_t* queue) { reset_sched(queue); }

}  // namespace

hipError_t launch_walk_force_learned(const WalkCell* walk, const double* rcp2, const Body* bodies,
                                     const float4* bodies32, const Cell* cells, const Moments* mom,
                                     const uint32_t* bfs2pre, const uint32_t* perm, const int32_t* gbeg,
                                     const int32_t* gcnt, int64_t gmax, uint32_t* queue, const MlpState* st,
                                     int leaf_cap, float G, float eps2, float tau, int64_t n,
                                     const DevParams* prm, float* acc, float* pot, int64_t* m2p, int64_t* p2p,
                                     int64_t* learned, int64_t* fallback, hipStream_t s) {
    static int resident = 0;
    if (resident == 0) {
        int dev = 0, cus = 0, per_cu = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess)
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_walk_force_learned, kThreads, 0);
        if (e != hipSuccess) return e;
        resident = cus * (per_cu > 0 ? per_cu : 1);
    }
    int64_t want = gmax;
    if (want > resident) want = resident;
    if (want < kXcd) want = kXcd;
    int lpl_log2 = 0;
    while ((1 << lpl_log2) < leaf_cap && lpl_log2 < 6) ++lpl_log2;
    hipLaunchKernelGGL(k_reset_queue_l, dim3(1), dim3(64), 0, s, queue);
    hipLaunchKernelGGL(k_walk_force_learned, dim3((unsigned)want), dim3(kThreads), 0, s, walk, rcp2, bodies,
                       bodies32, cells, mom, bfs2pre, perm, gbeg, gcnt, queue, st, lpl_log2, G, eps2, tau, n, prm, acc,
                       pot, m2p, p2p, learned, fallback);
    return hipGetLastError();
}

}  // namespace tc
