// Fused tree walk and force summation (§3.1: a cell goes on a body's
// interaction list when it is distant enough, otherwise the walk descends
// into its children; the list is then summed to give the force; §3.2: the
// per-body sums are independent of each other).
//
// One wavefront per walk group (at most 64 consecutive bodies in key order,
// never straddling a cluster cell), one lane per body.  The walk tests whole batches of cells at once: a per-wave LDS
// stack holds ranges of sibling cells (the children of one opened cell are
// contiguous in level order), and each round pops up to 8 ranges (4 in 2D),
// gives every lane one cell, and runs the opening test for all of them in
// FP64.  Accepted cells become list entries, leaves that are not accepted
// contribute their bodies (copied by all lanes together, 16 bodies per leaf
// side by side), opened cells push the range of their children.  The list
// lives in LDS; when it is full it is flushed: every lane sums it for its
// own body in FP32, reading each entry as an LDS broadcast.  Coordinates are
// relative to the group's box centre (FP64 difference, then rounded) so FP32
// keeps the significant digits; chunks of 64 entries are summed plainly and
// added to FP64 totals.  Each group's walk also counts
// the cells it tests (the root and every child of an opened cell), a
// measure of the walk's work that is kept per group.
//
// Stack bound: a round pushes at most 64 ranges; popping a single range at a
// time is a depth-first descent that adds at most (R-1) ranges per level
// plus R (R = cells per range, 8 in 3D, 4 in 2D), so full batches are popped
// only while that reserve is free and the stack can never overflow.
#include "tc_internal.h"
#include "walk_common.h"

#include <math.h>

#include <algorithm>
#include <atomic>

namespace tc {
namespace {

using namespace walk;
constexpr int kWavesPerBlock = 4;

// Walk for one group from the batch of cells [first, first + first_len) (the
// root alone for a whole walk) and sum its list into a, counting the cell
// entries in nm2p and the body entries in np2p.  The group's box is
// [lo, hi], its FP32 origin (rx, ry, rz), this lane's body (xi, yi, zi).
template <int D, bool PLAIN, bool QUAD, int STEP = 8>
__device__ __forceinline__ void walk_group(const WalkCell* __restrict__ walk, const float4* __restrict__ walkq,
                                           const Body* __restrict__ bodies, const float4* __restrict__ bodies32,
                                           float4* L, uint32_t* S, float4* LQ, int lpl_log2, float eps2,
                                           double lox, double hix, double loy, double hiy, double loz, double hiz,
                                           double rx, double ry, double rz, float xi, float yi, float zi,
                                           uint32_t first, int first_len, Acc& a, int64_t& nm2p, int64_t& np2p,
                                           int64_t& ntest) {
    constexpr int R = D == 3 ? 8 : 4;                    // lanes (cells) per popped range
    constexpr int RP = kWave / R;                        // ranges per full round
    constexpr int kReserve = (R - 1) * (D == 3 ? 21 : 31) + R;
    static_assert(kStackCap >= kWave + kReserve + kWave, "stack too small for its bound");
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t lanes_below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
    const int lpl = 1 << lpl_log2;                       // lanes per leaf in a copy batch
    const int slot = lane >> lpl_log2, jj = lane & (lpl - 1);
        int len = 0, qlen = 0;

        // The first batch is the range [first, first + first_len).  Each round: opening tests, pushes,
        // then the NEXT batch is popped and its cell loads issued before
        // this round's entries and leaf bodies are staged, so the two
        // memory round trips of a round overlap.
        int top = 0;
        bool vc = lane < first_len;
        WalkCell wc = load_cell(walk, first + (uint32_t)lane, vc);
        float4 q0 = make_float4(0.f, 0.f, 0.f, 0.f), q1 = q0;   // quadrupole of the tested cell
        if (QUAD && vc) {
            q0 = walkq[2 * (size_t)(first + lane)];
            q1 = walkq[2 * (size_t)(first + lane) + 1];
        }
        bool more = true;
        while (more) {
            // opening test: squared distance from the centre of mass to the box
            const double dxm = fmax(fmax(lox - wc.cx, 0.0), wc.cx - hix);
            const double dym = fmax(fmax(loy - wc.cy, 0.0), wc.cy - hiy);
            double d2 = dxm * dxm + dym * dym;
            if (D == 3) {
                const double dzm = fmax(fmax(loz - wc.cz, 0.0), wc.cz - hiz);
                d2 = d2 + dzm * dzm;
            }
            const bool leaf = vc && wc.b < 0;
            const bool accept = vc && d2 > wc.rcrit2;
            const bool opened = vc && !accept && !leaf;
            const bool direct = leaf && !accept;
            ntest += __popcll(__ballot(vc));

            // push the children ranges of opened cells
            const uint64_t O = __ballot(opened);
            if (opened) S[top + __popcll(O & lanes_below)] = ((uint32_t)wc.a << 3) | (uint32_t)(wc.b - 1);
            top += __popcll(O);
            wave_lds_sync();

            // pop the next batch (full batches only while the depth-first
            // reserve is free) and start loading its cells
            more = top > 0;
            bool vcn = false;
            WalkCell wcn;
            float4 q0n = make_float4(0.f, 0.f, 0.f, 0.f), q1n = q0n;
            if (more) {
                const int nr = (top + kWave + kReserve <= kStackCap) ? min(top, RP) : 1;
                const int rr = lane / R, j = lane % R;
                uint32_t packed = 0;
                if (rr < nr) packed = S[top - 1 - rr];
                top -= nr;
                const int rlen = (int)(packed & 7u) + 1;
                vcn = rr < nr && j < rlen;
                wcn = load_cell(walk, (packed >> 3) + j, vcn);
                if (QUAD && vcn) {
                    const uint32_t bq = (packed >> 3) + j;
                    q0n = walkq[2 * (size_t)bq];
                    q1n = walkq[2 * (size_t)bq + 1];
                }
            }
            wave_lds_sync();

            // accepted cells: one entry each, at their centre of mass
            const uint64_t A = __ballot(accept);
            const int na = __popcll(A);
            if (QUAD && na) {
                // with their quadrupole: 3 float4 per entry in the second list
                if (qlen + na > kQuadCap) {
                    flush_quad<PLAIN>(LQ, qlen, xi, yi, zi, eps2, a);
                    qlen = 0;
                }
                if (accept) {
                    const int at = 3 * (qlen + __popcll(A & lanes_below));
                    LQ[at] = make_float4((float)(wc.cx - rx), (float)(wc.cy - ry), (float)(wc.cz - rz), wc.m);
                    LQ[at + 1] = q0;
                    LQ[at + 2] = q1;
                }
                qlen += na;
                nm2p += na;
            } else if (na) {
                if (len + na > kListCap) {
                    flush<D, PLAIN, false, STEP>(L, len, xi, yi, zi, eps2, a);
                    len = 0;
                }
                if (accept)
                    L[len + __popcll(A & lanes_below)] =
                        make_float4((float)(wc.cx - rx), (float)(wc.cy - ry), (float)(wc.cz - rz), wc.m);
                len += na;
                nm2p += na;
            }

            // leaves that are not accepted: their bodies, copied cooperatively
            const int cnt = direct ? (wc.b & 0x7fffffff) : 0;
            const uint64_t P = __ballot(direct);
            if (P) {
                const uint64_t big = __ballot(direct && cnt > lpl);
                uint64_t small = P & ~big;
                while (small) {
                    int my_begin = 0, my_cnt = 0, my_off = 0, tot = 0;
                    for (int s = 0; s < (kWave >> lpl_log2) && small; ++s) {
                        const int l = __builtin_ctzll(small);
                        small &= small - 1;
                        const int cl = __builtin_amdgcn_readlane(cnt, l);
                        const int bl = __builtin_amdgcn_readlane(wc.a, l);
                        if (slot == s) {
                            my_begin = bl;
                            my_cnt = cl;
                            my_off = tot;
                        }
                        tot += cl;
                    }
                    if (len + tot > kListCap) {
                        flush<D, PLAIN, false, STEP>(L, len, xi, yi, zi, eps2, a);
                        len = 0;
                    }
                    if (jj < my_cnt)
                        L[len + my_off + jj] = body_entry(bodies, bodies32, my_begin + jj, rx, ry, rz);
                    len += tot;
                    np2p += tot;
                }
                uint64_t bg = big;
                while (bg) {                                   // leaves larger than a batch slot
                    const int l = __builtin_ctzll(bg);
                    bg &= bg - 1;
                    const int cl = __builtin_amdgcn_readlane(cnt, l);
                    const int bl = __builtin_amdgcn_readlane(wc.a, l);
                    for (int o = 0; o < cl; o += kWave) {
                        const int m = min(kWave, cl - o);
                        if (len + m > kListCap) {
                            flush<D, PLAIN, false, STEP>(L, len, xi, yi, zi, eps2, a);
                            len = 0;
                        }
                        if (lane < m) L[len + lane] = body_entry(bodies, bodies32, bl + o + lane, rx, ry, rz);
                        len += m;
                    }
                    np2p += cl;
                }
            }
            wave_lds_sync();
            wc = wcn;
            vc = vcn;
            if (QUAD) {
                q0 = q0n;
                q1 = q1n;
            }
        }
        flush<D, PLAIN, false, STEP>(L, len, xi, yi, zi, eps2, a);
        if (QUAD) flush_quad<PLAIN>(LQ, qlen, xi, yi, zi, eps2, a);
}

template <int D, bool PLAIN, bool QUAD, int STEP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(QUAD ? 4 : 5, 8))) k_walk_force(const WalkCell* __restrict__ walk,
                                                    const float4* __restrict__ walkq,
                                                    const Body* __restrict__ bodies,
                                                    const float4* __restrict__ bodies32,
                                                    const uint32_t* __restrict__ perm,
                                                    const int32_t* __restrict__ gbeg,
                                                    const int32_t* __restrict__ gcnt,
                                                    const uint32_t* __restrict__ order, uint32_t* queue,
                                                    uint32_t* __restrict__ bcost,
                                                    int lpl_log2, float G, float eps2,
                                                    const DevParams* __restrict__ prm,
                                                    ForceOut out,
                                                    int64_t* __restrict__ m2p_out,
                                                    int64_t* __restrict__ p2p_out,
                                                    int64_t* __restrict__ tst_out) {
    static_assert(!QUAD || D == 3, "quadrupole terms are 3D");
    __shared__ float4 s_list[kWavesPerBlock][kListCap];
    __shared__ uint32_t s_stack[kWavesPerBlock][kStackCap];
    __shared__ float4 s_qlist[kWavesPerBlock][QUAD ? 3 * kQuadCap : 1];   // accepted cells with Q
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & (kWave - 1);
    float4* L = s_list[wv];
    uint32_t* S = s_stack[wv];
    float4* LQ = s_qlist[wv];

    // Persistent waves, scheduled by GroupSched over the positions of
    // order (a permutation of the groups within each XCD share).
    const GroupSched sched = make_sched(queue, prm->ngroups, kWavesPerBlock);
    for (int hop = 0; hop < kXcd; ++hop) {
        const int xq = (sched.home + hop) % kXcd;
        const uint32_t g_hi = sched.share_lo(xq + 1);
        uint32_t g = sched.first(xq, hop);
        while (g < g_hi) {

            const uint32_t gi = order[g];
            const int64_t i0 = gbeg[gi];
            const int gn = gcnt[gi];
            const int64_t i = i0 + lane;
            const bool valid = lane < gn;
            const Body me = bodies[valid ? i : i0];

            // group bounding box (exact) and its centre, the group's FP32 origin
            const double lox = uniform(wave_min(me.x)), hix = uniform(wave_max(me.x));
            const double loy = uniform(wave_min(me.y)), hiy = uniform(wave_max(me.y));
            const double loz = D == 3 ? uniform(wave_min(me.z)) : 0.0;
            const double hiz = D == 3 ? uniform(wave_max(me.z)) : 0.0;
            const double rx = (lox + hix) * 0.5, ry = (loy + hiy) * 0.5, rz = (loz + hiz) * 0.5;
            const float xi = (float)(me.x - rx), yi = (float)(me.y - ry), zi = (float)(me.z - rz);

            Acc a = {0.0, 0.0, 0.0, 0.0};
            int64_t nm2p = 0, np2p = 0, ntest = 0;
            walk_group<D, PLAIN, QUAD, STEP>(walk, walkq, bodies, bodies32, L, S, LQ, lpl_log2, eps2, lox,
                                                       hix, loy, hiy, loz, hiz, rx, ry, rz, xi, yi, zi, 0u, 1, a, nm2p,
                                                       np2p, ntest);

            if (valid) {
                // the body met itself once as a direct entry: no force (zero
                // displacement) but a -m/eps potential term, removed here exactly as
                // it was formed
                const float mself = (float)me.m;
                const float sself = __builtin_amdgcn_rsqf(eps2);
                const float ph = (float)(a.sp + (double)(mself * sself));
                const int64_t o = perm[i];
                out.put<D>(o, G * (float)a.sx, G * (float)a.sy, G * (float)a.sz, G * ph);
                // the list length, for the next evaluation's schedule
                const int64_t lc = nm2p + np2p;
                bcost[o] = lc > 0xffffffffll ? 0xffffffffu : (uint32_t)lc;
            }
            if (lane == 0) {
                m2p_out[gi] = nm2p;
                p2p_out[gi] = np2p;
                tst_out[gi] = ntest;
            }
            g = sched.pop(xq);
        }
    }
}

// Small and mid-size problems: with fewer groups than resident waves, every
// wave walks its group alone on its SIMD and the walk's latency sets the
// time.  Here a block of NW waves takes one group at a time and shares both
// halves of its work evenly: the walk goes breadth first with one lane per
// cell over the whole block (NW 64 cells a round, from one LDS stack of
// ranges), and what it finds goes to one LDS list (cells at once, unaccepted
// leaves to a queue whose bodies are copied together), which the waves sum
// in equal contiguous parts whenever it is full.  Places come from prefix
// sums over the lanes and waves, so the list's order, and with it every sum,
// is the same in each run; the waves' FP32 sums are added in FP64 in wave
// order.  The interactions and counts are those of the one-wave walk; only
// the summation order differs.
// What bounds it: about a dozen dependent rounds (the tree's depth; a cell
// load and two barriers each) and then the list's arithmetic.  Dealing the
// cells of one level among waves that each walk and sum alone instead left
// the parts unequal, the near field lying in a few cells around the group
// (3D Plummer, theta 0.5, whole force evaluation: 110 us at 10,000 bodies,
// 239 at 50,000, 334 at 100,000 and 510 at 160,000 so; 61, 149, 219 and 345
// shared evenly).  coop_shape holds the measured NW and H.
template <int D, bool QUAD, int NW>
struct BlockWalk {
    static constexpr int kThreads = NW * kWave;
    static constexpr int R = D == 3 ? 8 : 4;                          // cells per range
    static constexpr int kReserve = (R - 1) * (D == 3 ? 21 : 31) + R;
    static constexpr int kStack = NW <= 2 ? 512 : 4 * kThreads;       // ranges
    static constexpr int kList = NW <= 2 || (QUAD && NW <= 4) ? 512 : NW <= 4 || QUAD ? 1024 : 2048;   // entries (16 B)
    static constexpr int kQuad = QUAD ? kThreads : 0;                 // entries with quadrupole (48 B)
    static_assert(kStack > kReserve + kThreads, "stack too small for its bound");
    static_assert(kList >= kThreads && kList % 8 == 0, "a round's cells must fit the list");
    static_assert(kList * sizeof(float4) >= NW * 4 * kWave * sizeof(double), "the waves' sums reuse the list");
};

template <int D, bool PLAIN, bool QUAD, int NW, int H>
__global__ void __launch_bounds__(NW * kWave) __attribute__((amdgpu_waves_per_eu(NW <= 4 ? 5 : 4, 8))) k_walk_force_coop(
    const WalkCell* __restrict__ walk, const float4* __restrict__ walkq, const Body* __restrict__ bodies,
    const float4* __restrict__ bodies32, const uint32_t* __restrict__ perm, const int32_t* __restrict__ gbeg,
    const int32_t* __restrict__ gcnt, const uint32_t* __restrict__ order, uint32_t* queue,
    uint32_t* __restrict__ bcost, int lpl_log2, float G, float eps2, const DevParams* __restrict__ prm,
    ForceOut out, int64_t* __restrict__ m2p_out, int64_t* __restrict__ p2p_out,
    int64_t* __restrict__ tst_out) {
    using B = BlockWalk<D, QUAD, NW>;
    constexpr int R = B::R, T = B::kThreads;
    __shared__ float4 L[B::kList];
    __shared__ uint32_t S[B::kStack];
    __shared__ float4 LQ[QUAD ? 3 * B::kQuad : 1];
    __shared__ int2 s_leaf[T];                       // queued leaves: first body, count
    __shared__ uint32_t s_loff[T];                   // their first places
    __shared__ uint64_t s_cnt[NW];
    __shared__ uint32_t s_sum[NW];
    __shared__ uint32_t s_next;
    const int t = (int)threadIdx.x, lane = t & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
    const int lpl = 1 << lpl_log2, slot = t >> lpl_log2, jj = t & (lpl - 1), slots = T >> lpl_log2;

    // Blocks are scheduled like the one-wave kernel's waves (GroupSched over
    // the positions of order, longest walks first in each XCD's share).
    // With H > 1 a group is H tasks of 64 / H bodies each: every task walks
    // for the whole group, and each of a wave's H lane parts sums its share
    // of the list for the task's bodies.
    const GroupSched sched{queue, prm->ngroups * (uint32_t)H, blockIdx.x / kXcd, (int)(blockIdx.x % kXcd), 1};
    // Without an order the tasks are dealt out in strides of the grid.
    constexpr int kBodies = kWave / H;
    for (int hop = 0; hop < (order ? kXcd : 1); ++hop) {
        const int xq = (sched.home + hop) % kXcd;
        const uint32_t g_hi = order ? sched.share_lo(xq + 1) : sched.ng;
        if (wv == 0) {
            const uint32_t f = order ? sched.first(xq, hop) : blockIdx.x;
            if (lane == 0) s_next = f;
        }
        __syncthreads();
        uint32_t pos = s_next;
        while (pos < g_hi) {
            const uint32_t g = order ? order[pos / H] : pos / H;
            const int64_t i0 = gbeg[g];
            const int gn = gcnt[g];
            const Body me = bodies[lane < gn ? i0 + lane : i0];
            const double lox = uniform(wave_min(me.x)), hix = uniform(wave_max(me.x));
            const double loy = uniform(wave_min(me.y)), hiy = uniform(wave_max(me.y));
            const double loz = D == 3 ? uniform(wave_min(me.z)) : 0.0;
            const double hiz = D == 3 ? uniform(wave_max(me.z)) : 0.0;
            const double rx = (lox + hix) * 0.5, ry = (loy + hiy) * 0.5, rz = (loz + hiz) * 0.5;
            // the body this lane sums for, and whether it is the one to store it
            const int own = (int)(pos % H) * kBodies + lane % kBodies;
            const bool valid = own < gn && lane < kBodies;
            float xi = (float)(me.x - rx), yi = (float)(me.y - ry), zi = (float)(me.z - rz);
            if (H > 1) {
                xi = __shfl(xi, own, kWave);
                yi = __shfl(yi, own, kWave);
                zi = __shfl(zi, own, kWave);
            }

            Acc a = {0.0, 0.0, 0.0, 0.0};
            int64_t nm2p = 0, np2p = 0, ntest = 0;
            int len = 0, qlen = 0, nleaf = 0, top = 1;

            bool drain = false;                      // the list or the leaf queue is full

            if (t == 0) S[0] = 0u;                   // the root alone
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
                    for (int w = 0; w < NW; ++w) {
                        const uint32_t v = s_sum[w];
                        if (w < wv) before += v;
                        total += v;
                    }
                    s_loff[t] = before + x - c;
                    __syncthreads();
                    do {
                        const uint32_t end = min(total, done + (uint32_t)(B::kList - len));
                        for (int s0 = slot; s0 < nleaf; s0 += 2 * slots) {
                            int32_t from[2], to[2], at[2];
                            float4 e[2];
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                const int s = s0 + u * slots;
                                const int2 lf = s < nleaf ? s_leaf[s] : make_int2(0, 0);
                                const int32_t o = s < nleaf ? (int32_t)s_loff[s] : 0;
                                const int32_t k0 = max(0, (int32_t)done - o);
                                from[u] = lf.x + k0 + jj;
                                to[u] = lf.x + min(lf.y, (int32_t)end - o);
                                at[u] = len + o + k0 + jj - (int32_t)done;
                            }
#pragma unroll
                            for (int u = 0; u < 2; ++u)
                                if (from[u] < to[u]) e[u] = body_entry(bodies, bodies32, from[u], rx, ry, rz);
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                if (from[u] < to[u]) L[at[u]] = e[u];
                                // leaves larger than lpl
                                for (int32_t j = from[u] + lpl, p = at[u] + lpl; j < to[u]; j += lpl, p += lpl)
                                    L[p] = body_entry(bodies, bodies32, j, rx, ry, rz);
                            }
                        }
                        len += (int)(end - done);
                        done = end;
                        __syncthreads();
                        // the waves' parts of the list: contiguous, equal, whole rounds of 8 H
                        const int per = ((len + NW - 1) / NW + 8 * H - 1) & ~(8 * H - 1);
                        const int cnt = min(per, len - wv * per);
                        if (cnt > 0) flush<D, PLAIN, true, 8, H>(L + wv * per, cnt, xi, yi, zi, eps2, a);
                        len = 0;
                        __syncthreads();
                    } while (done < total);
                    np2p += total;
                    nleaf = 0;
                    if (QUAD) {
                        const int per = ((qlen + NW - 1) / NW + 8 * H - 1) & ~(8 * H - 1);
                        const int cnt = min(per, qlen - wv * per);
                        if (cnt > 0) flush_quad<PLAIN, H>(LQ + 3 * wv * per, cnt, xi, yi, zi, eps2, a);
                        qlen = 0;
                        __syncthreads();
                    }
                    drain = false;
                    if (top == 0) break;
                }
                // pop as many ranges as the stack's depth-first reserve allows
                const int fit = (B::kStack - B::kReserve - top) / (R - 1);
                const int nr = max(1, min(min(top, T / R), fit));
                const int rr = t / R, j = t % R;
                uint32_t packed = 0;
                if (rr < nr) packed = S[top - 1 - rr];
                const bool vc = rr < nr && j < (int)(packed & 7u) + 1;
                const uint32_t cidx = (packed >> 3) + (uint32_t)j;
                const WalkCell wc = load_cell(walk, cidx, vc);
                // opening test: squared distance from the centre of mass to the box
                const double dxm = fmax(fmax(lox - wc.cx, 0.0), wc.cx - hix);
                const double dym = fmax(fmax(loy - wc.cy, 0.0), wc.cy - hiy);
                double d2 = dxm * dxm + dym * dym;
                if (D == 3) {
                    const double dzm = fmax(fmax(loz - wc.cz, 0.0), wc.cz - hiz);
                    d2 = d2 + dzm * dzm;
                }
                const bool leaf = vc && wc.b < 0;
                const bool accept = vc && d2 > wc.rcrit2;
                const bool opened = vc && !accept && !leaf;
                const bool direct = leaf && !accept;
                const uint64_t O = __ballot(opened), A = __ballot(accept), P = __ballot(direct), V = __ballot(vc);
                // four counts of at most kThreads each, 16 bits apart
                if (lane == 0)
                    s_cnt[wv] = (uint64_t)__popcll(O) | (uint64_t)__popcll(A) << 16 | (uint64_t)__popcll(P) << 32 |
                                (uint64_t)__popcll(V) << 48;
                __syncthreads();
                uint64_t before = 0, total = 0;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const uint64_t v = s_cnt[w];
                    if (w < wv) before += v;
                    total += v;
                }
                const int na = (int)(total >> 16 & 0xffffu), np = (int)(total >> 32 & 0xffffu);
                if ((QUAD ? qlen + na > B::kQuad : len + na > B::kList) || nleaf + np > T) {
                    drain = true;                    // make room, then this round again
                    __syncthreads();
                    continue;
                }
                top -= nr;
                if (opened)
                    S[top + (int)(before & 0xffffu) + __popcll(O & below)] =
                        ((uint32_t)wc.a << 3) | (uint32_t)(wc.b - 1);
                if (accept) {
                    const int at = (int)(before >> 16 & 0xffffu) + __popcll(A & below);
                    const float4 e =
                        make_float4((float)(wc.cx - rx), (float)(wc.cy - ry), (float)(wc.cz - rz), wc.m);
                    if (QUAD) {
                        LQ[3 * (qlen + at)] = e;
                        LQ[3 * (qlen + at) + 1] = walkq[2 * (size_t)cidx];
                        LQ[3 * (qlen + at) + 2] = walkq[2 * (size_t)cidx + 1];
                    } else {
                        L[len + at] = e;
                    }
                }
                if (direct)
                    s_leaf[nleaf + (int)(before >> 32 & 0xffffu) + __popcll(P & below)] =
                        make_int2(wc.a, wc.b & 0x7fffffff);
                top += (int)(total & 0xffffu);
                if (QUAD) qlen += na;
                else len += na;
                nleaf += np;
                nm2p += na;
                ntest += (int)(total >> 48);
                __syncthreads();
            }

            // the waves' sums, added in FP64 in wave order: one thread per
            // body and component
            double* part = reinterpret_cast<double*>(L);
            part[(wv * 4 + 0) * kWave + lane] = a.sx;
            part[(wv * 4 + 1) * kWave + lane] = a.sy;
            part[(wv * 4 + 2) * kWave + lane] = a.sz;
            part[(wv * 4 + 3) * kWave + lane] = a.sp;
            if (wv == 0) {
                const uint32_t nx = order ? sched.pop(xq) : pos + gridDim.x;
                if (lane == 0) s_next = nx;
            }
            __syncthreads();
            for (int c = wv; c < 4 && valid; c += NW) {
                double v = 0.0;
                for (int q = 0; q < H; ++q)
                    for (int w = 0; w < NW; ++w) v += part[(w * 4 + c) * kWave + q * kBodies + lane];
                const int64_t o = perm[i0 + own];
                if (c < 3) {
                    if (c < D) out.put_acc(o * D + c, (float)((double)G * v));
                } else {
                    // the body met itself once as a direct entry: its -m/eps
                    // potential term is removed as in the one-wave kernel
                    const float mself = (float)bodies[i0 + own].m;
                    v += (double)(mself * __builtin_amdgcn_rsqf(eps2));
                    out.put_pot(o, (float)((double)G * v));
                    const int64_t lc = nm2p + np2p;
                    bcost[o] = lc > 0xffffffffll ? 0xffffffffu : (uint32_t)lc;
                }
            }
            if (t == 0 && pos % H == 0) {
                m2p_out[g] = nm2p;
                p2p_out[g] = np2p;
                tst_out[g] = ntest;
            }
            pos = s_next;
            __syncthreads();                         // the list is reused by the next group
        }
        __syncthreads();                             // s_next is rewritten
    }
}

// Split walks for small N, where the longest single group otherwise bounds
// the kernel: the walk of group g is cut into kSplitTasks<D> tasks, one per
// (level-1 cell k, child slot j).  If cell k is accepted or is a leaf, task
// (k, 0) walks it and the other slots of k do nothing; if k is opened, task
// (k, j) walks its j-th child.  Together the tasks visit exactly the cells
// and bodies of the unsplit walk (the root is never accepted for a group
// inside it).  Each task writes its FP32 sums for the group's bodies to its
// own slice of part; k_split_reduce adds the slices in FP64 in task order.
template <int D>
constexpr int kSplitTasks = D == 3 ? 64 : 16;

template <int D, bool PLAIN, bool QUAD>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(QUAD ? 4 : 5, 8))) k_walk_force_split(
    const WalkCell* __restrict__ walk, const float4* __restrict__ walkq, const Body* __restrict__ bodies,
    const float4* __restrict__ bodies32, const int32_t* __restrict__ gbeg, const int32_t* __restrict__ gcnt,
    int lpl_log2, float eps2, const DevParams* __restrict__ prm, int64_t n, float4* __restrict__ part,
    unsigned long long* __restrict__ m2p_out, unsigned long long* __restrict__ p2p_out) {
    constexpr int R = D == 3 ? 8 : 4;
    constexpr int T = kSplitTasks<D>;
    __shared__ float4 s_list[kWavesPerBlock][kListCap];
    __shared__ uint32_t s_stack[kWavesPerBlock][kStackCap];
    __shared__ float4 s_qlist[kWavesPerBlock][QUAD ? 3 * kQuadCap : 1];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & (kWave - 1);
    const int64_t task = (int64_t)blockIdx.x * kWavesPerBlock + wv;
    const int64_t g = task / T;
    const int t = (int)(task % T);
    if (g >= (int64_t)prm->ngroups) return;
    const int64_t i0 = gbeg[g];
    const int gn = gcnt[g];
    const int64_t i = i0 + lane;
    const bool valid = lane < gn;
    const Body me = bodies[valid ? i : i0];
    const double lox = uniform(wave_min(me.x)), hix = uniform(wave_max(me.x));
    const double loy = uniform(wave_min(me.y)), hiy = uniform(wave_max(me.y));
    const double loz = D == 3 ? uniform(wave_min(me.z)) : 0.0;
    const double hiz = D == 3 ? uniform(wave_max(me.z)) : 0.0;
    const double rx = (lox + hix) * 0.5, ry = (loy + hiy) * 0.5, rz = (loz + hiz) * 0.5;
    const float xi = (float)(me.x - rx), yi = (float)(me.y - ry), zi = (float)(me.z - rz);

    // this task's first batch: one cell or nothing
    uint32_t first = 0;
    int first_len = 0;
    const WalkCell root = walk[0];
    if (root.b < 0) {                                    // the root is a leaf
        first_len = t == 0 ? 1 : 0;
    } else {
        const int k = t / R, j = t % R;
        if (k < root.b) {
            const uint32_t c1 = (uint32_t)root.a + (uint32_t)k;
            const WalkCell w1 = walk[c1];
            const double dxm = fmax(fmax(lox - w1.cx, 0.0), w1.cx - hix);
            const double dym = fmax(fmax(loy - w1.cy, 0.0), w1.cy - hiy);
            double d2 = dxm * dxm + dym * dym;
            if (D == 3) {
                const double dzm = fmax(fmax(loz - w1.cz, 0.0), w1.cz - hiz);
                d2 = d2 + dzm * dzm;
            }
            if (d2 > w1.rcrit2 || w1.b < 0) {
                first = c1;
                first_len = j == 0 ? 1 : 0;
            } else if (j < w1.b) {
                first = (uint32_t)w1.a + (uint32_t)j;
                first_len = 1;
            }
        }
    }
    Acc a = {0.0, 0.0, 0.0, 0.0};
    int64_t nm2p = 0, np2p = 0, ntest = 0;   // tested cells are not kept for split walks
    walk_group<D, PLAIN, QUAD>(walk, walkq, bodies, bodies32, s_list[wv], s_stack[wv], s_qlist[wv], lpl_log2, eps2,
                               lox, hix, loy, hiy, loz, hiz, rx, ry, rz, xi, yi, zi, first, first_len, a, nm2p,
                               np2p, ntest);
    if (valid)
        part[(int64_t)t * n + i] = make_float4((float)a.sx, (float)a.sy, (float)a.sz, (float)a.sp);
    if (lane == 0 && (nm2p | np2p)) {
        atomicAdd(&m2p_out[g], (unsigned long long)nm2p);
        atomicAdd(&p2p_out[g], (unsigned long long)np2p);
    }
}

template <int D>
__global__ void __launch_bounds__(256) k_split_reduce(const float4* __restrict__ part, const Body* __restrict__ bodies,
                                                      const uint32_t* __restrict__ perm, int64_t n, float G,
                                                      float eps2, ForceOut out) {
    constexpr int T = kSplitTasks<D>;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double ax = 0.0, ay = 0.0, az = 0.0, ap = 0.0;
        for (int t = 0; t < T; ++t) {
            const float4 v = part[(int64_t)t * n + i];
            ax += v.x;
            ay += v.y;
            az += v.z;
            ap += v.w;
        }
        // the body met itself once as a direct entry: its -m/eps potential
        // term is removed as in the unsplit kernel
        const float mself = (float)bodies[i].m;
        ap += (double)(mself * __builtin_amdgcn_rsqf(eps2));
        const int64_t o = perm[i];
        out.put<D>(o, (float)((double)G * ax), (float)((double)G * ay), (float)((double)G * az),
                   (float)((double)G * ap));
    }
}

__global__ void k_zero_u64(unsigned long long* __restrict__ a, unsigned long long* __restrict__ b,
                           unsigned long long* __restrict__ c, int64_t k) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < k; i += (int64_t)gridDim.x * blockDim.x) {
        a[i] = 0ull;
        b[i] = 0ull;
        c[i] = 0ull;
    }
}

// FP32 copy of each cell's traceless quadrupole in level order, two float4
// per cell: (xx, yy, zz, xy), (xz, yz, 0, 0).
__global__ void __launch_bounds__(256) k_quad_pack(const Moments* __restrict__ mom,
                                                   const uint32_t* __restrict__ pre2bfs,
                                                   const DevParams* __restrict__ prm, int64_t cmax,
                                                   float4* __restrict__ walkq) {
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < C; k += (int64_t)gridDim.x * blockDim.x) {
        const Moments& mo = mom[k];
        const size_t b = 2 * (size_t)pre2bfs[k];
        walkq[b] = make_float4((float)mo.Q[0], (float)mo.Q[1], (float)mo.Q[2], (float)mo.Q[3]);
        walkq[b + 1] = make_float4((float)mo.Q[4], (float)mo.Q[5], 0.f, 0.f);
    }
}


// The order in which the persistent waves take the groups of each XCD
// share: runs of consecutive groups, by decreasing cost.  A
// group's cost is the list length that its middle body had in the previous
// force evaluation (bodies are named by their input index, so this survives
// a rebuild; group boundaries move from step to step, so neither a group
// index nor a group's first body, often the previous group's last, does as
// well).  Long walks then start first and the walks still running when a
// share drains are short ones.  Longer runs keep more neighbouring groups,
// which read the same cells and bodies, running side by side in one XCD's
// L2, but they lengthen the tail, which matters less the more groups each
// wave takes.  Runs are max(1, groups / (4 waves)) long, and from 16 groups
// per wave on the groups are taken in key order.  Measured: on a 1M-body
// Plummer sphere (3.5 groups per wave) runs of 1, 4, 16, 64 and 256 groups
// fetched 560, 500, 400, 320 and 275 MB from HBM per launch (280 GB/s at
// most: the kernel is ALU-bound) and took 2.0, 2.11, 2.09, 2.16 and
// 2.19 ms (2.2 ms in key order); on 4.2M bodies of two Plummer spheres (14
// groups per wave) runs of 3 took 1% less than key order; on 16.7M
// clustered bodies (57 groups per wave) single groups took 15.7 ms, runs of
// 14, 16 or 64 14.9-15.3 ms, key order 14.7-15.2 ms.  Only the schedule
// depends on the costs: each group's walk and sums are the same in any order, so stale
// or missing costs cost time, never accuracy.  k_group_order gathers the
// costs of one share's groups and sorts its runs, one share per block (and
// zeroes that share's work counter), by the mean cost of a run in buckets
// of 1/16 of an octave (log2 with four fraction bits);
// places within a bucket are taken with LDS atomics, so they may differ
// from run to run.
constexpr int kOrderBuckets = 512;
constexpr int kOrderThreads = 1024;

__device__ __forceinline__ int cost_bucket(uint32_t v) {
    if (v < 1) return 0;
    const int e = 31 - __builtin_clz(v);
    const uint32_t frac = (e >= 4 ? (v >> (e - 4)) : (v << (4 - e))) & 15u;
    const int b = 16 * e + (int)frac;
    return b < kOrderBuckets ? b : kOrderBuckets - 1;
}

__global__ void __launch_bounds__(kOrderThreads) k_group_order(const uint32_t* __restrict__ bcost,
                                                               const uint32_t* __restrict__ perm,
                                                               const int32_t* __restrict__ gbeg,
                                                               const int32_t* __restrict__ gcnt,
                                                               const DevParams* __restrict__ prm,
                                                               uint32_t* __restrict__ gcost,
                                                               uint16_t* __restrict__ ckey,
                                                               uint32_t* __restrict__ order,
                                                               uint32_t* __restrict__ queue, uint32_t waves) {
    __shared__ uint32_t hist[kOrderBuckets];
    __shared__ uint32_t scan[2][kOrderBuckets];
    const uint32_t NG = prm->ngroups;
    const int x = (int)blockIdx.x;
    const uint32_t lo = (uint32_t)(((uint64_t)NG * x) / kXcd), hi = (uint32_t)(((uint64_t)NG * (x + 1)) / kXcd);
    const uint32_t W = max(waves, 1u);
    const int t = (int)threadIdx.x;
    if (t == 0) queue[x * kQueueStride] = 0u;
    if (NG >= 16u * W) {                                 // key order
        for (uint32_t g = lo + (uint32_t)t; g < hi; g += kOrderThreads) order[g] = g;
        return;
    }
    const uint32_t run = max(1u, NG / (4u * W));
    const uint32_t nc = (hi - lo + run - 1) / run;
    if (t < kOrderBuckets) hist[t] = 0u;
    // the share's group costs, four groups per thread with their loads
    // issued together (three dependent loads each)
    for (uint32_t g0 = lo + (uint32_t)t; g0 < hi; g0 += 4 * kOrderThreads) {
        int32_t gb[4], gc[4];
        uint32_t pb[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t g = g0 + u * kOrderThreads;
            gb[u] = g < hi ? gbeg[g] : 0;
            gc[u] = g < hi ? gcnt[g] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) pb[u] = g0 + u * kOrderThreads < hi ? perm[gb[u] + gc[u] / 2] : 0u;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t g = g0 + u * kOrderThreads;
            if (g < hi) gcost[g] = bcost[pb[u]];
        }
    }
    __syncthreads();
    // each run's bucket (kept at its first group's key) and the groups per bucket
    for (uint32_t c = (uint32_t)t; c < nc; c += kOrderThreads) {
        const uint32_t c0 = lo + c * run, c1 = min(hi, c0 + run);
        uint64_t sum = 0;
        for (uint32_t g = c0; g < c1; ++g) sum += gcost[g];
        const uint64_t mean = sum / (c1 - c0);
        const int b = cost_bucket(mean > 0xffffffffull ? 0xffffffffu : (uint32_t)mean);
        ckey[c0] = (uint16_t)b;
        atomicAdd(&hist[b], c1 - c0);
    }
    __syncthreads();
    // inclusive scan over the buckets from the most expensive down
    int cur = 0;
    if (t < kOrderBuckets) scan[0][t] = hist[kOrderBuckets - 1 - t];
    __syncthreads();
    for (int d = 1; d < kOrderBuckets; d <<= 1) {
        if (t < kOrderBuckets) scan[cur ^ 1][t] = scan[cur][t] + (t >= d ? scan[cur][t - d] : 0u);
        cur ^= 1;
        __syncthreads();
    }
    // hist becomes the next free place of each bucket
    if (t < kOrderBuckets) {
        const int r = kOrderBuckets - 1 - t;             // bucket of scan position t
        hist[r] = scan[cur][t] - hist[r];
    }
    __syncthreads();
    // the same runs as above, each read back by the thread that keyed it
    for (uint32_t c = (uint32_t)t; c < nc; c += kOrderThreads) {
        const uint32_t c0 = lo + c * run, c1 = min(hi, c0 + run);
        const uint32_t at = lo + atomicAdd(&hist[ckey[c0]], c1 - c0);
        for (uint32_t g = c0; g < c1; ++g) order[at + (g - c0)] = g;
    }
}

}  // namespace

hipError_t launch_quad_pack(const Moments* mom, const uint32_t* pre2bfs, const DevParams* prm, int64_t cmax,
                            float4* walkq, hipStream_t s) {
    int64_t nb = (cmax + 255) / 256;
    if (nb > 4096) nb = 4096;
    hipLaunchKernelGGL(k_quad_pack, dim3((unsigned)nb), dim3(256), 0, s, mom, pre2bfs, prm, cmax, walkq);
    return hipGetLastError();
}

hipError_t launch_walk_force_split(const WalkCell* walk, const float4* walkq, const Body* bodies,
                                   const float4* bodies32, const uint32_t* perm, const int32_t* gbeg,
                                   const int32_t* gcnt, int64_t gmax, int64_t n, int dim, int leaf_cap, float G,
                                   float eps2, const DevParams* prm, float4* part, const ForceOut& out,
                                   int64_t* m2p, int64_t* p2p, int64_t* tests, bool plain, hipStream_t s) {
    int lpl_log2 = 0;
    while ((1 << lpl_log2) < leaf_cap && lpl_log2 < 6) ++lpl_log2;
    unsigned long long* c1 = reinterpret_cast<unsigned long long*>(m2p);
    unsigned long long* c2 = reinterpret_cast<unsigned long long*>(p2p);
    hipLaunchKernelGGL(k_zero_u64, dim3((unsigned)((gmax + 255) / 256)), dim3(256), 0, s, c1, c2,
                       reinterpret_cast<unsigned long long*>(tests), gmax);
    const int T = dim == 3 ? kSplitTasks<3> : kSplitTasks<2>;
    const unsigned nb = (unsigned)((gmax * T + kWavesPerBlock - 1) / kWavesPerBlock);
#define TC_LAUNCH_SPLIT(DIM, PL, QU)                                                                               \
    hipLaunchKernelGGL((k_walk_force_split<DIM, PL, QU>), dim3(nb), dim3(256), 0, s, walk, walkq, bodies, bodies32, \
                       gbeg, gcnt, lpl_log2, eps2, prm, n, part, c1, c2)
    if (dim == 3 && walkq) {
        if (plain) TC_LAUNCH_SPLIT(3, true, true);
        else TC_LAUNCH_SPLIT(3, false, true);
    } else if (dim == 3) {
        if (plain) TC_LAUNCH_SPLIT(3, true, false);
        else TC_LAUNCH_SPLIT(3, false, false);
    } else {
        if (plain) TC_LAUNCH_SPLIT(2, true, false);
        else TC_LAUNCH_SPLIT(2, false, false);
    }
#undef TC_LAUNCH_SPLIT
    const unsigned rb = (unsigned)std::min<int64_t>((n + 255) / 256, 4096);
    if (dim == 3)
        hipLaunchKernelGGL(k_split_reduce<3>, dim3(rb), dim3(256), 0, s, part, bodies, perm, n, G, eps2, out);
    else
        hipLaunchKernelGGL(k_split_reduce<2>, dim3(rb), dim3(256), 0, s, part, bodies, perm, n, G, eps2, out);
    return hipGetLastError();
}

// Blocks of a shared-walk kernel that can be resident at once, at most one
// per group and at least one per XCD share (k_group_order's eight shares).
template <auto kKernel>
static hipError_t coop_blocks(int threads, int64_t gmax, unsigned* out) {
    static std::atomic<int> resident{0};
    int64_t want = resident.load(std::memory_order_relaxed);
    if (want == 0) {
        int dev = 0, cus = 0, per_cu = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kKernel, threads, 0);
        if (e != hipSuccess) return e;
        want = (int64_t)cus * (per_cu > 0 ? per_cu : 1);
        resident.store((int)want, std::memory_order_relaxed);
    }
    if (want > gmax) want = gmax;
    if (want < kXcd) want = kXcd;
    *out = (unsigned)want;
    return hipSuccess;
}

hipError_t launch_walk_force(const WalkCell* walk, const float4* walkq, const Body* bodies, const float4* bodies32,
                             const uint32_t* perm,
                             const int32_t* gbeg, const int32_t* gcnt, int64_t gmax, uint32_t* order,
                             uint32_t* queue, uint32_t* bcost,
                             int64_t n, int dim, int leaf_cap, float G, float eps2,
                             const DevParams* prm, const ForceOut& out, int64_t* m2p,
                             int64_t* p2p, int64_t* tests, bool plain, bool share,
                             double theta, hipStream_t s) {
    // as many blocks as can be resident at once (the waves are persistent)
    static int resident[3] = {0, 0, 0};                // 2D, 3D, 3D with quadrupoles
    const int kind = dim == 3 ? (walkq ? 2 : 1) : 0;
    int& res = resident[kind];
    if (res == 0) {
        int dev = 0, cus = 0, per_cu = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess)
            e = kind == 2   ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_walk_force<3, false, true, 8>, 256, 0)
                : kind == 1 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_walk_force<3, false, false, 8>, 256, 0)
                            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_walk_force<2, false, false, 8>, 256, 0);
        if (e != hipSuccess) return e;
        res = cus * (per_cu > 0 ? per_cu : 1);
    }
    int64_t want = (gmax + kWavesPerBlock - 1) / kWavesPerBlock;
    if (want > res) want = res;
    if (want < kXcd) want = kXcd;
    const unsigned nb = (unsigned)want;
    int lpl_log2 = 0;                                   // lanes per leaf: next power of two, <= 64
    while ((1 << lpl_log2) < leaf_cap && lpl_log2 < 6) ++lpl_log2;
    // the group order: costs and run keys after the gmax places of order
    // (as the layout reserves), then the counting sort of each share
    uint32_t* gcost = order + gmax;
    uint16_t* ckey = reinterpret_cast<uint16_t*>(order + 2 * gmax);
    auto make_order = [&]() {
        hipLaunchKernelGGL(k_group_order, dim3(kXcd), dim3(kOrderThreads), 0, s, (const uint32_t*)bcost, perm, gbeg,
                           gcnt, prm, gcost, ckey, order, queue, (uint32_t)(nb * kWavesPerBlock));
    };
    if (share && n <= coop_max_n(dim, theta, walkq != nullptr)) {
        // one block per task at a time, as many blocks as can be resident;
        // with about one task per block (coop_shape) no order is made: it
        // would cost its launch and change nothing
        const CoopShape shape = coop_shape(n, dim, theta);
        if (shape.ordered) make_order();
        const uint32_t* places = shape.ordered ? order : nullptr;
        unsigned cb = 0;
#define TC_LAUNCH_COOP_NW(DIM, PL, QU, NW, H)                                                                       \
    do {                                                                                                            \
        const hipError_t e_ = coop_blocks<k_walk_force_coop<DIM, PL, QU, NW, H>>(NW * kWave, gmax * H, &cb);        \
        if (e_ != hipSuccess) return e_;                                                                            \
        hipLaunchKernelGGL((k_walk_force_coop<DIM, PL, QU, NW, H>), dim3(cb), dim3(NW * kWave), 0, s, walk, walkq,  \
                           bodies, bodies32, perm, gbeg, gcnt, places, queue, bcost, lpl_log2, G, eps2, prm, out,   \
                           m2p, p2p, tests);                                                                        \
    } while (0)
#define TC_LAUNCH_COOP(DIM, PL, QU)                                                                                 \
    do {                                                                                                            \
        if (DIM == 3 && shape.parts == 2) TC_LAUNCH_COOP_NW(3, PL, QU, 8, 2);                                       \
        else if (shape.waves == 8) TC_LAUNCH_COOP_NW(DIM, PL, QU, 8, 1);                                            \
        else if (DIM == 3 || shape.waves == 4) TC_LAUNCH_COOP_NW(DIM, PL, QU, 4, 1);                                \
        else TC_LAUNCH_COOP_NW(2, PL, false, 2, 1);                                                                 \
    } while (0)
        if (dim == 3 && walkq) {
            if (plain) TC_LAUNCH_COOP(3, true, true);
            else TC_LAUNCH_COOP(3, false, true);
        } else if (dim == 3) {
            if (plain) TC_LAUNCH_COOP(3, true, false);
            else TC_LAUNCH_COOP(3, false, false);
        } else {
            if (plain) TC_LAUNCH_COOP(2, true, false);
            else TC_LAUNCH_COOP(2, false, false);
        }
#undef TC_LAUNCH_COOP
#undef TC_LAUNCH_COOP_NW
        return hipGetLastError();
    }
    make_order();
    // With two to four groups per resident wave (counting n/64 groups) the
    // list sums go in rounds of 4 entries, else 8: the same sums either
    // way, and measured per force kernel (3D Plummer, rounds of 4 against
    // 8): 1.89 against 1.94 ms at 1M bodies, 2.29 against 2.32 at 1.25M,
    // but 0.86 against 0.85 at 400,000, 7.89 against 7.86 at 4M, 16.45
    // against 16.19 at 16.7M and 0.1145 against 0.1140 ms for the
    // 262,144-body disk.
    const int64_t groups_lo = (n + kGroup - 1) / kGroup, waves_all = (int64_t)nb * kWavesPerBlock;
    const bool short_rounds = groups_lo > 2 * waves_all && groups_lo <= 4 * waves_all;
#define TC_LAUNCH_WF_STEP(DIM, PL, QU, ST)                                                                           \
    hipLaunchKernelGGL((k_walk_force<DIM, PL, QU, ST>), dim3(nb), dim3(256), 0, s, walk, walkq, bodies, bodies32,  \
                       perm, gbeg, gcnt, order, queue, bcost, lpl_log2, G, eps2, prm, out, m2p, p2p, tests)
#define TC_LAUNCH_WF(DIM, PL, QU)                                                                                \
    do {                                                                                                         \
        if (short_rounds) TC_LAUNCH_WF_STEP(DIM, PL, QU, 4);                                                     \
        else TC_LAUNCH_WF_STEP(DIM, PL, QU, 8);                                                                  \
    } while (0)
    if (dim == 3 && walkq) {
        if (plain) TC_LAUNCH_WF(3, true, true);
        else TC_LAUNCH_WF(3, false, true);
    } else if (dim == 3) {
        if (plain) TC_LAUNCH_WF(3, true, false);
        else TC_LAUNCH_WF(3, false, false);
    } else {
        if (plain) TC_LAUNCH_WF(2, true, false);
        else TC_LAUNCH_WF(2, false, false);
    }
#undef TC_LAUNCH_WF
#undef TC_LAUNCH_WF_STEP
    return hipGetLastError();
}

}  // namespace tc
