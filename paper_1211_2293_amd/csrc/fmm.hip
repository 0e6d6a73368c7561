// Fast multipole method (§5 of the paper points to it as the step beyond the
// treecode): cell-cell interactions through Cartesian expansions, 3D.
//
//   * every cell has its multipole about its centre of mass (mass M and the
//     traceless quadrupole Q; the dipole vanishes there) and a local
//     expansion about its geometric centre z: 20 FP64 coefficients of
//       phi(z + dl) = -G sum_{n<=3} (1/n!) Lam_n[dl^n];
//   * a dual tree traversal, one level of pairs per launch, sorts every
//     (target A, source B) pair reached from (root, root): a cell with
//     itself becomes all pairs of its children (a leaf: a direct sum); A and
//     B are far enough for an expansion when |z_A - com_B| > (rho_A + rho_B)
//     / theta, rho_A and rho_B bounding their bodies about z_A and com_B
//     (from the bodies for a leaf, from the children for a cell, capped by
//     the geometric bounds); two leaves that are not sum
//     directly; otherwise the larger cell (smaller level, A on a tie, never
//     a leaf) is split;
//   * M2L: with g(R) = (|R|^2 + eps^2)^(-1/2), D_n its derivative tensors and
//     R = z_A - com_B, Lam_n += M D_n(R) + (1/6) Q:D_(n+2)(R), truncated at
//     total order 3 (the quadrupole acts on Lam_0 and Lam_1);
//   * L2L from every parent to its children, level by level;
//   * per leaf: the expansion at each body (L2P) plus the direct sums over
//     its partner leaves in FP32 (P2P), coordinates relative to the leaf
//     centre, chunks added in FP64 as in the treecode force loop.
//
// The traversal writes its pairs in a fixed order and a stable sort groups
// them by target, so every sum runs in a fixed order and results are
// reproducible bit for bit.
#include "tc_internal.h"
#include "walk_common.h"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace tc {
namespace {

using namespace walk;

constexpr double kHalfSqrt3 = 0.8660254037844386;   // sqrt(3)/2, rounded to FP64

// Symmetric tensor slots of a local expansion:
//   0: Lam_0;  1..3: x, y, z;  4..9: xx, yy, zz, xy, xz, yz;
//   10..19: xxx, yyy, zzz, xxy, xxz, xyy, yyz, xzz, yzz, xyz.
constexpr int kNL = 20;

__device__ __forceinline__ bool is_leaf(const Cell& c) { return c.leaf_nch < 0; }

__device__ __forceinline__ uint64_t pair_key(uint32_t a, uint32_t b) { return ((uint64_t)a << 32) | b; }

__device__ __forceinline__ double dist2(double ax, double ay, double az, double bx, double by, double bz) {
    const double dx = ax - bx, dy = ay - by, dz = az - bz;
    return (dx * dx + dy * dy) + dz * dz;
}

constexpr int kGeoLanes = 8;                // lanes per cell: bodies of a leaf, children of a cell

__device__ __forceinline__ double lanes_max(double v) {
#pragma unroll
    for (int o = kGeoLanes / 2; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, kWave));
    return v;
}

// Centres and radii: rho_A bounds the cell's bodies about its centre z, rho_B
// about its centre of mass; for a leaf the largest distance of one of its
// bodies (the root of the largest square, which is the same number), for an
// internal cell the largest (distance between the centres + the child's radius)
// over its children, from k_fmm_radii; each capped by the geometric bound.
__global__ void __launch_bounds__(256) k_fmm_geo(const Cell* __restrict__ cells, const Moments* __restrict__ mom,
                                                 const Body* __restrict__ bodies, const WalkCell* __restrict__ walk,
                                                 const uint32_t* __restrict__ pre2bfs,
                                                 const DevParams* __restrict__ prm, int64_t cmax,
                                                 FmmGeo* __restrict__ geo, DttCell* __restrict__ dc) {
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    const double size = prm->size;
    const int sub = threadIdx.x % kGeoLanes;
    const int64_t stride = (int64_t)gridDim.x * (blockDim.x / kGeoLanes);
    for (int64_t k = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kGeoLanes; k < C; k += stride) {
        const Cell c = cells[k];
        const int l = c.level;
        const double s = ldexp(size, -l);
        uint64_t org[3] = {0, 0, 0};
        for (int j = 1; j <= l; ++j) {
            const unsigned d = (unsigned)((c.prefix >> (3 * (l - j))) & 7u);
#pragma unroll
            for (int a = 0; a < 3; ++a) org[a] = (org[a] << 1) | ((d >> (2 - a)) & 1u);
        }
        FmmGeo g;
        double com[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            g.z[a] = prm->lo[a] + ((double)org[a] + 0.5) * s;
            com[a] = mom[k].com[a];
        }
        double rhoA = kHalfSqrt3 * s;
        double rhoB = kHalfSqrt3 * s + sqrt(dist2(com[0], com[1], com[2], g.z[0], g.z[1], g.z[2]));
        if (is_leaf(c)) {
            double ra = 0.0, rb = 0.0;
            for (int64_t j = c.begin + sub; j < (int64_t)c.begin + c.count; j += kGeoLanes) {
                const Body b = bodies[j];
                ra = fmax(ra, dist2(b.x, b.y, b.z, g.z[0], g.z[1], g.z[2]));
                rb = fmax(rb, dist2(b.x, b.y, b.z, com[0], com[1], com[2]));
            }
            rhoA = fmin(sqrt(lanes_max(ra)), rhoA);
            rhoB = fmin(sqrt(lanes_max(rb)), rhoB);
        }
        if (sub != 0) continue;
        geo[k] = g;
        const uint32_t kb = pre2bfs[k];
        DttCell t;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            t.z[a] = g.z[a];
            t.com[a] = com[a];
        }
        t.rhoA = rhoA;
        t.rhoB = rhoB;
        t.child = is_leaf(c) ? -1 : walk[kb].a;
        t.nch_leaf = c.leaf_nch;
        t.level = l;
        t.pre = (int32_t)k;
        dc[kb] = t;
    }
}

// The radii of the internal cells of one level (level-order range), deepest
// level first.  One lane per child: with a thread per cell and the leaves'
// bodies in the same kernel, a level was one thread's chain of up to 64 loads
// and roots (285 us for eleven levels of 60,850 cells; now 31, and 14 for
// k_fmm_geo with the leaves' bodies).
__global__ void __launch_bounds__(256) k_fmm_radii(const uint32_t* __restrict__ lvl_off, int level, DttCell* dc) {
    const int sub = threadIdx.x % kGeoLanes;
    const int64_t lo = lvl_off[level], hi = lvl_off[level + 1];
    const int64_t stride = (int64_t)gridDim.x * (blockDim.x / kGeoLanes);
    for (int64_t k = lo + (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kGeoLanes; k < hi; k += stride) {
        const DttCell g = dc[k];
        if (g.nch_leaf < 0) continue;
        double ra = 0.0, rb = 0.0;
        if (sub < g.nch_leaf) {
            const DttCell ch = dc[g.child + sub];
            ra = sqrt(dist2(ch.z[0], ch.z[1], ch.z[2], g.z[0], g.z[1], g.z[2])) + ch.rhoA;
            rb = sqrt(dist2(ch.com[0], ch.com[1], ch.com[2], g.com[0], g.com[1], g.com[2])) + ch.rhoB;
        }
        ra = lanes_max(ra);
        rb = lanes_max(rb);
        if (sub == 0) {
            dc[k].rhoA = fmin(ra, g.rhoA);
            dc[k].rhoB = fmin(rb, g.rhoB);
        }
    }
}

// One level of the traversal, on level-order cell indices: every input
// pair becomes an M2L pair, a P2P pair, or pairs of the next level.  Three
// launches per level keep the output order fixed: each wave counts the
// outputs of its contiguous chunk of the input and leaves every pair's kind in
// the pair's two spare bits, one block turns the counts into every wave's first
// slots (and advances the running totals), and each wave writes its outputs in
// lane order.  A slot at or beyond a capacity is counted but not written.  M2L
// and P2P pairs are stored as (source << 32) | target with pre-order indices,
// ready for the sort by target; pairs of the next level as (A << 32) | B in
// level order (indices below 2^31).  The levels' sizes stay on the device, so
// that the host waits once for a batch of levels; a level larger than its
// buffer counts as empty.
//
// Bound by the scattered reads of the cells in the count and by the pairs'
// traffic in the write.  Classifying again in the write, with up to eight
// 8-byte stores per lane that each touched another line, and a host wait per
// level took 243 + 192 + 513 us of kernels for the 17 levels of 1,048,576 bodies
// (theta 0.5, 27.2M M2L and 5.1M P2P pairs) and 0.9 ms of gaps; now 278 + 112 +
// 282 and one or two waits.
// kind 1: M2L, 2: P2P, 3: children x children, 4: children x B, 5: A x children;
// next: pairs of the next level.  Without branches, so that the loads of
// several pairs overlap.
struct DttOut {
    int kind;
    uint32_t next;
};

__device__ __forceinline__ DttOut dtt_classify(const DttCell& ca, const DttCell& cb, bool self, double theta) {
    const bool la = ca.nch_leaf < 0, lb = cb.nch_leaf < 0;
    const double dx = ca.z[0] - cb.com[0], dy = ca.z[1] - cb.com[1], dz = ca.z[2] - cb.com[2];
    const double r = (ca.rhoA + cb.rhoB) / theta;
    const bool acc = theta != 0.0 && (dx * dx + dy * dy) + dz * dz > r * r;
    const bool split_a = !la && (lb || ca.level <= cb.level);
    const uint32_t na = (uint32_t)ca.nch_leaf & 0x7fffffffu, nb = (uint32_t)cb.nch_leaf & 0x7fffffffu;
    DttOut o;
    o.kind = self ? (la ? 2 : 3) : acc ? 1 : la && lb ? 2 : split_a ? 4 : 5;
    o.next = o.kind < 3 ? 0u : o.kind == 3 ? na * na : o.kind == 4 ? na : nb;
    return o;
}

constexpr int kDttBlock = 256;
constexpr int kDttWaves = kDttBlock / kWave;
constexpr int kScanWaves = kFmmMaxWaves / 1024;
static_assert(kDttWaves == 4, "the scan takes a block's counts as one uint4");
constexpr uint64_t kKindA = 1ull << 63, kKindB = 1ull << 31;   // none: M2L; B: P2P; A: split A (or a cell's own pair); both: split B

// The chunk of the input of one of nw waves, the same in both sweeps.
__device__ __forceinline__ void dtt_chunk(int64_t nin, int64_t w, int64_t nw, int64_t& begin, int64_t& end) {
    const int64_t chunk = ((nin + nw - 1) / nw + kWave - 1) / kWave * kWave;
    begin = min(nin, w * chunk);
    end = min(nin, begin + chunk);
}

__device__ __forceinline__ int64_t dtt_size(const unsigned long long* size, int64_t capf) {
    const int64_t n = (int64_t)*size;
    return n > capf ? 0 : n;
}

__global__ void k_fmm_dtt_root(unsigned long long* __restrict__ ctr, uint64_t* __restrict__ fin) {
    if (threadIdx.x < kFmmCounters) ctr[threadIdx.x] = threadIdx.x == kFmmSizes ? 1ull : 0ull;
    if (threadIdx.x == 0) fin[0] = 0ull;        // the pair (root, root)
}

// Sweep 1: bt[k * waves + wave] = the wave's M2L (k = 0), P2P (1) and
// next-level (2) output counts; the kinds go into the pairs.
__global__ void __launch_bounds__(kDttBlock) k_fmm_dtt_count(const DttCell* __restrict__ dc, double theta,
                                                             uint64_t* __restrict__ fin,
                                                             const unsigned long long* __restrict__ size, int64_t capf,
                                                             uint32_t* __restrict__ bt) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t nw = (int64_t)gridDim.x * kDttWaves, w = (int64_t)blockIdx.x * kDttWaves + (threadIdx.x / kWave);
    int64_t begin, end;
    dtt_chunk(dtt_size(size, capf), w, nw, begin, end);
    uint32_t cm = 0, cp = 0, cn = 0;
    constexpr int kAhead = 2;
    for (int64_t i0 = begin + lane; i0 < end; i0 += kAhead * kWave) {
        uint64_t pr[kAhead];
        DttCell ca[kAhead], cb[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) pr[u] = fin[min(i0 + u * kWave, end - 1)];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            ca[u] = dc[(pr[u] >> 32) & 0x7fffffffu];
            cb[u] = dc[pr[u] & 0x7fffffffu];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const bool valid = i0 + u * kWave < end;
            const DttOut o = dtt_classify(ca[u], cb[u], pr[u] >> 32 == (uint32_t)pr[u], theta);
            cm += valid && o.kind == 1;
            cp += valid && o.kind == 2;
            cn += valid ? o.next : 0u;
            if (valid && o.kind != 1)
                fin[i0 + u * kWave] = pr[u] | (o.kind == 2 ? kKindB : o.kind == 5 ? kKindA | kKindB : kKindA);
        }
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        cm += __shfl_xor(cm, o, kWave);
        cp += __shfl_xor(cp, o, kWave);
        cn += __shfl_xor(cn, o, kWave);
    }
    if (lane < 3) bt[lane * nw + w] = lane == 0 ? cm : lane == 1 ? cp : cn;
}

// One block: every block's first output slots (M2L and P2P after the running
// totals ctr[1], ctr[2]; the next level from 0), then the next level's size
// and ctr[1], ctr[2] advanced.  nw is four per block, at most kScanWaves per
// thread.
__global__ void __launch_bounds__(1024) k_fmm_dtt_scan(const uint32_t* __restrict__ bt, int nw,
                                                       unsigned long long* __restrict__ ctr,
                                                       unsigned long long* __restrict__ next,
                                                       unsigned long long* __restrict__ base) {
    __shared__ unsigned long long s[3][1024 / kWave];
    const int t = threadIdx.x, lane = t & (kWave - 1), wv = t / kWave;
    uint4 c[3][kScanWaves / 4];
    unsigned long long mine[3], incl[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        mine[k] = 0;
#pragma unroll
        for (int j = 0; j < kScanWaves / 4; ++j) {
            const int w = kScanWaves * t + 4 * j;
            c[k][j] = w < nw ? *reinterpret_cast<const uint4*>(bt + (int64_t)k * nw + w) : make_uint4(0, 0, 0, 0);
            mine[k] += (unsigned long long)c[k][j].x + c[k][j].y + c[k][j].z + c[k][j].w;
        }
        incl[k] = mine[k];
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const unsigned long long y = __shfl_up(incl[k], o, kWave);
            if (lane >= o) incl[k] += y;
        }
        if (lane == kWave - 1) s[k][wv] = incl[k];
    }
    const unsigned long long m0 = ctr[1], p0 = ctr[2];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        unsigned long long run = k == 0 ? m0 : k == 1 ? p0 : 0ull;
        for (int w = 0; w < wv; ++w) run += s[k][w];
        run += incl[k] - mine[k];
#pragma unroll
        for (int j = 0; j < kScanWaves / 4; ++j) {
            const int w = kScanWaves * t + 4 * j;
            if (w < nw) base[(int64_t)k * (nw / 4) + w / 4] = run;
            run += (unsigned long long)c[k][j].x + c[k][j].y + c[k][j].z + c[k][j].w;
        }
        if (t == 1023) (k == 0 ? ctr[1] : k == 1 ? ctr[2] : *next) = run;
    }
}

// Sweep 2: the outputs in lane order from the wave's first slots, those of its
// block and the counts of the block's waves before it.  The pairs of
// the next level are written 64 at a time, side by side: a bit per splitting
// pair's first place tells every lane which pair its place belongs to.
__global__ void __launch_bounds__(kDttBlock) k_fmm_dtt_write(const DttCell* __restrict__ dc,
                                                             const uint32_t* __restrict__ bfs2pre,
                                                             const uint64_t* __restrict__ fin,
                                                             const unsigned long long* __restrict__ size,
                                                             const uint32_t* __restrict__ bt,
                                                             const unsigned long long* __restrict__ base,
                                                             uint64_t* __restrict__ fout, int64_t capf,
                                                             uint64_t* __restrict__ m2l, int64_t capm,
                                                             uint64_t* __restrict__ p2p, int64_t capp) {
    __shared__ int4 s_split[kDttWaves][kWave];       // first place, A, B, pairs per child of A (bits 24..) and its reciprocal
    __shared__ uint64_t s_start[kDttWaves][kWave];   // at most 64 places per pair
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const uint64_t below = (1ull << lane) - 1ull, upto = ~0ull >> (kWave - 1 - lane);
    const int64_t nw = (int64_t)gridDim.x * kDttWaves, w = (int64_t)blockIdx.x * kDttWaves + wv;
    int64_t begin, end;
    dtt_chunk(dtt_size(size, capf), w, nw, begin, end);
    if (begin >= end) return;
    const int64_t nb = gridDim.x, w0 = (int64_t)blockIdx.x * kDttWaves;
    int64_t om = (int64_t)base[blockIdx.x], op = (int64_t)base[nb + blockIdx.x], on = (int64_t)base[2 * nb + blockIdx.x];
    for (int j = 0; j < kDttWaves - 1; ++j)
        if (j < wv) {
            om += bt[w0 + j];
            op += bt[nw + w0 + j];
            on += bt[2 * nw + w0 + j];
        }
    uint64_t ahead = fin[min(begin + lane, end - 1)];
    for (int64_t i0 = begin; i0 < end; i0 += kWave) {
        const bool valid = i0 + lane < end;
        const uint64_t pr = ahead;
        ahead = fin[min(i0 + kWave + lane, end - 1)];
        const bool ka = (pr & kKindA) != 0, kb = (pr & kKindB) != 0;
        const uint32_t A = (uint32_t)(pr >> 32) & 0x7fffffffu, B = (uint32_t)pr & 0x7fffffffu;
        const bool split = valid && ka;
        const uint64_t M = __ballot(valid && !ka && !kb), P = __ballot(valid && !ka && kb), C = __ballot(split);
        if (valid && !ka) {
            const uint64_t key = ((uint64_t)bfs2pre[B] << 32) | bfs2pre[A];
            if (kb) {
                const int64_t at = op + __popcll(P & below);
                if (at < capp) p2p[at] = key;
            } else {
                const int64_t at = om + __popcll(M & below);
                if (at < capm) m2l[at] = key;
            }
        }
        om += __popcll(M);
        op += __popcll(P);
        if (!C) continue;
        int child = 0, nch = 0, per = 1;             // per: pairs per child of A
        if (split) {
            const DttCell& c = dc[kb ? B : A];
            child = c.child;
            nch = c.nch_leaf & 0x7fffffff;
            per = A == B ? nch : kb ? kWave : 1;
        }
        const int count = A == B ? nch * nch : nch;
        int incl = count;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int y = __shfl_up(incl, o, kWave);
            if (lane >= o) incl += y;
        }
        const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
        s_start[wv][lane] = 0ull;
        wave_lds_sync();
        if (split) {
            const int first = incl - count;
            s_split[wv][__popcll(C & below)] = make_int4(first, kb ? (int)A : child, kb || A == B ? child : (int)B,
                                                         per << 24 | (65536 + per - 1) / per);
            atomicOr(reinterpret_cast<uint32_t*>(s_start[wv]) + first / 32, 1u << (first % 32));
        }
        wave_lds_sync();
        int before = -1;
        for (int t0 = 0; t0 < total; t0 += kWave) {
            const uint64_t st = s_start[wv][t0 / kWave];
            const int4 q = s_split[wv][before + __popcll(st & upto)];
            before += __popcll(st);
            const int j = t0 + lane - q.x;
            const int x = (int)((uint32_t)(j * (q.w & 0xffffff)) >> 16), y = j - x * (q.w >> 24);
            const int64_t at = on + t0 + lane;
            if (t0 + lane < total && at < capf) fout[at] = pair_key((uint32_t)(q.y + x), (uint32_t)(q.z + y));
        }
        on += total;
        wave_lds_sync();
    }
}

// Start of every target's run in the keys sorted by target (the low 32
// bits): off[t] = the first key whose target is >= t, for t = 0..C
// (off[C] = n).
__global__ void __launch_bounds__(256) k_fmm_offsets(const uint64_t* __restrict__ keys, int64_t n, int64_t C,
                                                     uint32_t* __restrict__ off) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t <= C; t += (int64_t)gridDim.x * blockDim.x) {
        int64_t lo = 0, hi = n;
        while (lo < hi) {
            const int64_t mid = lo + (hi - lo) / 2;
            if ((int64_t)(uint32_t)keys[mid] < t) lo = mid + 1;
            else hi = mid;
        }
        off[t] = (uint32_t)lo;
    }
}

// ---- expansions, FP64

// Add the expansion of a source (M, traceless Q at its centre of mass) at
// R = centre - source to lam.
__device__ __forceinline__ void m2l_add(double M, const double* Q, double x, double y, double z, double eps2,
                                        double* lam) {
    const double xx = x * x, yy = y * y, zz = z * z;
    const double s = rsqrt64(((xx + yy) + zz) + eps2);
    const double s2 = s * s, s3 = s2 * s, s5 = s3 * s2, s7 = s5 * s2;
    const double Qxx = Q[0], Qyy = Q[1], Qzz = Q[2], Qxy = Q[3], Qxz = Q[4], Qyz = Q[5];
    const double qx = fma(Qxz, z, fma(Qxy, y, Qxx * x));
    const double qy = fma(Qyz, z, fma(Qyy, y, Qxy * x));
    const double qz = fma(Qzz, z, fma(Qyz, y, Qxz * x));
    const double rqr = fma(qz, z, fma(qy, y, qx * x));
    const double trq = Qxx + Qyy + Qzz;
    const double m3 = M * s3, m5 = 3.0 * M * s5, m7 = -15.0 * M * s7;
    // Lam_0: M D0 + (1/6) Q:D2, with Q:D2 = 3 RQR s^5 - tr(Q) s^3
    lam[0] += fma(M, s, fma(0.5 * rqr, s5, trq * s3 * (-1.0 / 6.0)));
    // Lam_1: M D1 + (1/6) Q:D3, with (Q:D3)_a = -15 R_a RQR s^7 + 3 (2 (QR)_a + R_a tr Q) s^5
    const double k1 = fma(0.5 * trq, s5, fma(-2.5 * rqr, s7, -m3));
    lam[1] += fma(x, k1, qx * s5);
    lam[2] += fma(y, k1, qy * s5);
    lam[3] += fma(z, k1, qz * s5);
    // Lam_2 = M D2: 3 R_a R_b s^5 - delta_ab s^3
    const double mx = m5 * x, my = m5 * y, mz = m5 * z;
    lam[4] += fma(mx, x, -m3);
    lam[5] += fma(my, y, -m3);
    lam[6] += fma(mz, z, -m3);
    lam[7] = fma(mx, y, lam[7]);
    lam[8] = fma(mx, z, lam[8]);
    lam[9] = fma(my, z, lam[9]);
    // Lam_3 = M D3: -15 R_a R_b R_c s^7 + 3 (delta_ab R_c + delta_ac R_b + delta_bc R_a) s^5
    const double ax = fma(m7, xx, m5), ay = fma(m7, yy, m5), az = fma(m7, zz, m5);
    lam[10] = fma(x, fma(2.0, m5, ax), lam[10]);
    lam[11] = fma(y, fma(2.0, m5, ay), lam[11]);
    lam[12] = fma(z, fma(2.0, m5, az), lam[12]);
    lam[13] = fma(y, ax, lam[13]);
    lam[14] = fma(z, ax, lam[14]);
    lam[15] = fma(x, ay, lam[15]);
    lam[16] = fma(z, ay, lam[16]);
    lam[17] = fma(x, az, lam[17]);
    lam[18] = fma(y, az, lam[18]);
    lam[19] = fma(m7 * x, y * z, lam[19]);
}

// Full-tensor views of the packed coefficients.
__device__ __forceinline__ double t2(const double* lam, int a, int b) {
    if (a == b) return lam[4 + a];
    const int s = a + b;   // (0,1) -> xy, (0,2) -> xz, (1,2) -> yz
    return lam[s == 1 ? 7 : s == 2 ? 8 : 9];
}

__device__ __forceinline__ double t3(const double* lam, int a, int b, int c) {
    int n[3] = {0, 0, 0};
    ++n[a];
    ++n[b];
    ++n[c];
    if (n[0] == 3) return lam[10];
    if (n[1] == 3) return lam[11];
    if (n[2] == 3) return lam[12];
    if (n[0] == 2) return n[1] == 1 ? lam[13] : lam[14];
    if (n[1] == 2) return n[0] == 1 ? lam[15] : lam[16];
    if (n[2] == 2) return n[0] == 1 ? lam[17] : lam[18];
    return lam[19];
}

// (acc / G, -pot / G) of an expansion at offset dl: g_a = Lam1_a + Lam2_ab dl_b
// + (1/2) Lam3_abc dl_b dl_c and p = Lam0 + Lam1.dl + (1/2) dl.Lam2.dl +
// (1/6) Lam3[dl, dl, dl].
__device__ __forceinline__ void l2p(const double* lam, const double* dl, double* g, double& p) {
    p = lam[0];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double h = 0.0, t = 0.0;                 // (Lam2 dl)_a and (Lam3[dl, dl])_a
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            double u = 0.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) u = fma(t3(lam, a, b, c), dl[c], u);
            h = fma(t2(lam, a, b), dl[b], h);
            t = fma(u, dl[b], t);
        }
        g[a] = lam[1 + a] + fma(0.5, t, h);
        p = fma(dl[a], lam[1 + a] + fma(1.0 / 6.0, t, 0.5 * h), p);
    }
}

// M2L: one wave per target cell; lane k takes the target's sorted sources
// k, k + 64, ...; the lanes' sums are added by a fixed butterfly, 22 exchanges
// for the 20 coefficients.  Bound by the gathered moments and the FP64 units:
// 27.2M pairs in 261 us; with a butterfly of six exchanges per coefficient,
// divisions and a root it was 374, half of it the exchanges.
// Overwrites lam.
__global__ void __launch_bounds__(256) k_fmm_m2l(const Moments* __restrict__ mom, const FmmGeo* __restrict__ geo,
                                                 const DevParams* __restrict__ prm, int64_t cmax,
                                                 const uint64_t* __restrict__ keys, const uint32_t* __restrict__ off,
                                                 double eps2, double* __restrict__ lam_out) {
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x / kWave);
    for (int64_t t = blockIdx.x * (int64_t)(blockDim.x / kWave) + (threadIdx.x / kWave); t < C; t += nwaves) {
        double lam[kNL];
#pragma unroll
        for (int k = 0; k < kNL; ++k) lam[k] = 0.0;
        const FmmGeo g = geo[t];
        const uint32_t q0 = off[t], q1 = off[t + 1];
        uint64_t ahead = q0 + lane < q1 ? keys[q0 + lane] : 0ull;
        for (uint32_t q = q0 + lane; q < q1; q += kWave) {
            const Moments& mb = mom[(uint32_t)(ahead >> 32)];
            ahead = keys[min(q + kWave, q1 - 1)];
            m2l_add(mb.M, mb.Q, g.z[0] - mb.com[0], g.z[1] - mb.com[1], g.z[2] - mb.com[2], eps2, lam);
        }
        // the sums over the lanes, xor 32 first: two coefficients share a step
        // as long as there are two, half the lanes keeping either
        auto fold = [&](double x, double y, int o) {
            const bool hi = (lane & o) != 0;
            return (hi ? y : x) + __shfl_xor(hi ? x : y, o, kWave);
        };
#pragma unroll
        for (int k = 0; k < 10; ++k) lam[k] = fold(lam[k], lam[k + 10], 32);
#pragma unroll
        for (int k = 0; k < 5; ++k) lam[k] = fold(lam[k], lam[k + 5], 16);
        lam[0] = fold(lam[0], lam[3], 8);
        lam[1] = fold(lam[1], lam[4], 8);
        lam[2] += __shfl_xor(lam[2], 8, kWave);
        lam[0] = fold(lam[0], lam[1], 4);
        lam[2] += __shfl_xor(lam[2], 4, kWave);
        lam[0] = fold(lam[0], lam[2], 2);
        lam[0] += __shfl_xor(lam[0], 1, kWave);
        const bool third = (lane & 2) != 0;
        const int k = (lane & 32 ? 10 : 0) + (lane & 16 ? 5 : 0) + (third ? 2 : (lane & 8 ? 3 : 0) + (lane & 4 ? 1 : 0));
        if (!(lane & 1) && !(third && (lane & 12))) lam_out[t * kNL + k] = lam[0];
    }
}

// L2L for the cells of one level (level-order range [lo, hi)): each adds its
// parent's expansion moved to its own centre.
__global__ void __launch_bounds__(256) k_fmm_l2l(const Cell* __restrict__ cells, const FmmGeo* __restrict__ geo,
                                                 const uint32_t* __restrict__ bfs2pre,
                                                 const uint32_t* __restrict__ lvl_off, int level,
                                                 double* __restrict__ lam) {
    const int64_t lo = lvl_off[level], hi = lvl_off[level + 1];
    for (int64_t k = lo + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < hi;
         k += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t c = bfs2pre[k];
        const int32_t p = cells[c].parent;
        if (p < 0) continue;
        double P[kNL];
#pragma unroll
        for (int j = 0; j < kNL; ++j) P[j] = lam[(int64_t)p * kNL + j];
        double t[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) t[a] = geo[c].z[a] - geo[p].z[a];
        double* out = lam + (int64_t)c * kNL;
        // Lam'_0 and Lam'_1 are the potential and its gradient at t
        double g[3], p0;
        l2p(P, t, g, p0);
        out[0] += p0;
        out[1] += g[0];
        out[2] += g[1];
        out[3] += g[2];
        // Lam'_2 = Lam2 + Lam3 . t
        const int ia[6] = {0, 1, 2, 0, 0, 1}, ib[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            double v = P[4 + j];
#pragma unroll
            for (int c3 = 0; c3 < 3; ++c3) v += t3(P, ia[j], ib[j], c3) * t[c3];
            out[4 + j] += v;
        }
#pragma unroll
        for (int j = 10; j < kNL; ++j) out[j] += P[j];
    }
}

constexpr int kFmmList = 256;
constexpr int kFmmWaves = 1;                // per block: their tasks differ in length
// Tasks per launch: a grid holds fewer than 2^32 threads, so one launch for all
// would be refused from 67M tasks on; a launch costs nothing beside 1M tasks.
constexpr int64_t kFmmLaunch = (int64_t)1 << 20;
static_assert(kFmmLaunch * kWave < (int64_t)1 << 32, "a launch's threads must fit its grid");

// A target leaf whose partner list is longer than kFmmChunk leaves is cut
// into chunks of kFmmChunk partners, one task each, so that no single wave
// carries a far-spread leaf's whole direct sum; the chunks' sums go to
// partial slots and k_fmm_leaf_finish adds them in chunk order.
constexpr uint32_t kFmmChunk = 256;

// Tasks of more partners than this are started first, so that the others fill
// the end of the launch: 1,048,576 bodies (leaf size 64, theta 0.5) 3.90 -> 3.67
// ms for everything, the leaf kernel 1.60 -> 1.37 (a line of 96 or 160 partners
// was 1% slower).  A task's
// sums do not depend on when it runs.
constexpr uint32_t kFmmLong = 128;

__device__ __forceinline__ bool long_task(uint32_t partners) { return partners > kFmmLong; }

// Tasks per cell (leaves: chunks of the partner list; other cells: none)
// and partial slots (chunks x bodies, for leaves cut into several chunks).
__global__ void __launch_bounds__(256) k_fmm_tasks_count(const Cell* __restrict__ cells,
                                                         const uint32_t* __restrict__ poff,
                                                         const DevParams* __restrict__ prm, int64_t cmax,
                                                         uint32_t* __restrict__ ntask, uint32_t* __restrict__ nslot,
                                                         unsigned long long* __restrict__ ctr) {
    __shared__ unsigned long long s_slots[4], s_tasks[4];
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    unsigned long long slots = 0, tasks = 0;          // tasks << 32 | long ones
    for (int64_t A = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; A < C; A += (int64_t)gridDim.x * blockDim.x) {
        const Cell ca = cells[A];
        uint32_t nt = 0, ns = 0;
        if (is_leaf(ca)) {
            const uint32_t np = poff[A + 1] - poff[A];
            nt = np > kFmmChunk ? (np + kFmmChunk - 1) / kFmmChunk : 1u;
            ns = nt > 1 ? nt * (uint32_t)ca.count : 0u;
            slots += ns;
            tasks += (unsigned long long)nt << 32 | (nt - 1 + (long_task(np - (nt - 1) * kFmmChunk) ? 1u : 0u));
        }
        ntask[A] = nt;
        nslot[A] = ns;
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        slots += __shfl_xor(slots, o, kWave);
        tasks += __shfl_xor(tasks, o, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        s_slots[threadIdx.x / kWave] = slots;
        s_tasks[threadIdx.x / kWave] = tasks;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        tasks = s_tasks[0] + s_tasks[1] + s_tasks[2] + s_tasks[3];
        slots = s_slots[0] + s_slots[1] + s_slots[2] + s_slots[3];
        if (tasks) atomicAdd(&ctr[3], tasks);
        if (slots) atomicAdd(&ctr[0], slots);
    }
}

// Every task's leaf, and the list of the long tasks (in any order; left_long:
// those still to be listed, taken by one claim per wave).
__global__ void __launch_bounds__(256) k_fmm_tasks_fill(const uint32_t* __restrict__ toff,
                                                        const uint32_t* __restrict__ poff,
                                                        const DevParams* __restrict__ prm, int64_t cmax,
                                                        uint32_t* __restrict__ task, uint32_t* __restrict__ longs,
                                                        uint32_t* __restrict__ left_long) {
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t A0 = blockIdx.x * (int64_t)blockDim.x + (threadIdx.x & ~(kWave - 1)); A0 < C; A0 += stride) {
        const int64_t A = A0 + lane;
        const uint32_t t0 = A < C ? toff[A] : 0u, t1 = A < C ? toff[A + 1] : 0u;
        const uint32_t np = t1 > t0 ? poff[A + 1] - poff[A] : 0u;
        const uint32_t full = t1 > t0 ? t1 - t0 - 1u : 0u;          // whole chunks before the last
        const uint32_t mine = full + (long_task(np - full * kFmmChunk) ? 1u : 0u);
        uint32_t incl = mine;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o, kWave);
            if (lane >= o) incl += y;
        }
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
        uint32_t at = 0;
        if (total) {
            if (lane == 0) at = atomicSub(left_long, total) - total;
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + incl - mine;
        }
        for (uint32_t k = t0; k < t1; ++k) {
            task[k] = (uint32_t)A;
            if (k - t0 < mine) longs[at + (k - t0)] = k;
        }
    }
}

// L2P + P2P: one wave per task (a target leaf, or one chunk of a long
// leaf's partner list).  Lanes are (two target bodies t and t + H, slice): with
// nA target bodies, H = ceil(nA / 2) lanes per slice, and slice k of
// S = floor(64 / H) sums list entries k, k + S, ...; the slices' sums are added
// in FP64 in a fixed order.  The partner leaves' bodies are gathered up to 256
// at a time: 64 partner cells are loaded together, their body counts scanned,
// and each lane finds its bodies' partners from a bit per partner's first slot,
// for four bodies at once where there are as many.
//
// Bound by the FP32 units, 14 instructions per pair of bodies: 2.9e9 pairs
// (1,048,576 bodies, leaf size 64, theta 0.5) in 1.4 ms.  Two targets per lane
// halve the LDS reads per interaction and leave few lanes idle (slices of the
// next power of two of nA lanes lost a quarter); four entries per lane are read
// ahead, where one at a time waited for each; chunks are added in FP64 (two
// instructions, where a compensated FP32 sum took eight); a wave per block, as
// tasks differ in length.  Before: 2.74 ms.
__device__ __forceinline__ void two_targets(const float4& q, const float (&x)[2][3], float eps2, float (&a)[2][4]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float dx = q.x - x[h][0], dy = q.y - x[h][1], dz = q.z - x[h][2];
        const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, eps2)));
        const float s = __builtin_amdgcn_rsqf(r2);
        const float ms = q.w * s;
        const float ms3 = ms * (s * s);
        a[h][0] = fmaf(ms3, dx, a[h][0]);
        a[h][1] = fmaf(ms3, dy, a[h][1]);
        a[h][2] = fmaf(ms3, dz, a[h][2]);
        a[h][3] -= ms;
    }
}

template <bool F32>
__global__ void __launch_bounds__(kFmmWaves * kWave, 4) k_fmm_leaf(const Cell* __restrict__ cells, const Body* __restrict__ bodies,
                                                  const float4* __restrict__ bodies32, const uint32_t* __restrict__ perm,
                                                  const FmmGeo* __restrict__ geo, const double* __restrict__ lam,
                                                  const uint64_t* __restrict__ pkeys, const uint32_t* __restrict__ poff,
                                                  const uint32_t* __restrict__ task, const uint32_t* __restrict__ toff,
                                                  const uint32_t* __restrict__ soff, int64_t first, int64_t ntasks,
                                                  const uint32_t* __restrict__ longs, int64_t nlong, double* __restrict__ part,
                                                  float G, float eps2, float* __restrict__ acc, float* __restrict__ pot) {
    constexpr int kAhead = 4;               // entries read ahead per lane
    constexpr int kPlain = 32;              // FP32 terms per lane between additions in FP64
    __shared__ float4 s_list[kFmmWaves][kFmmList];
    __shared__ int32_t s_beg[kFmmWaves][kWave];
    __shared__ uint64_t s_start[kFmmWaves][kFmmList / kWave];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & (kWave - 1);
    float4* L = s_list[wv];
    int32_t* SB = s_beg[wv];
    uint64_t* ST = s_start[wv];
    const uint64_t upto = ~0ull >> (kWave - 1 - lane);
    const int64_t at = first + blockIdx.x * (int64_t)kFmmWaves + __builtin_amdgcn_readfirstlane(wv);
    if (at >= nlong + ntasks) return;
    const int64_t tk = at < nlong ? (int64_t)longs[at] : at - nlong;
    {
        const uint32_t A = task[tk];
        const uint32_t chunk = (uint32_t)tk - toff[A], nchunks = toff[A + 1] - toff[A];
        const Cell ca = cells[A];
        const double zx = geo[A].z[0], zy = geo[A].z[1], zz = geo[A].z[2];
        const uint32_t q0 = poff[A] + chunk * kFmmChunk;
        const uint32_t q1 = nchunks > 1 ? min(poff[A + 1], q0 + kFmmChunk) : poff[A + 1];
        if (at >= nlong && long_task(q1 - q0)) return;       // done from the list
        for (int t0 = 0; t0 < ca.count; t0 += kWave) {
            const int nA = min(kWave, ca.count - t0);
            const int H = (nA + 1) / 2, S = kWave / H;
            const int t = lane % H;
            const int sl = min(lane / H, S - 1);             // lanes left over repeat the last slice
            float x[2][3];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const Body me = bodies[(int64_t)ca.begin + t0 + (t + h * H < nA ? t + h * H : t)];
                x[h][0] = (float)(me.x - zx);
                x[h][1] = (float)(me.y - zy);
                x[h][2] = (float)(me.z - zz);
            }
            double v[2][4] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
            int len = 0;
            auto flush = [&](int cnt) {
                wave_lds_sync();
                for (int e = 0; e < cnt; e += kPlain * S) {
                    const int lim = min(cnt, e + kPlain * S);
                    float a[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
                    int k = e;
                    for (; k + kAhead * S <= lim; k += kAhead * S) {
                        float4 q[kAhead];
#pragma unroll
                        for (int u = 0; u < kAhead; ++u) q[u] = L[k + u * S + sl];
#pragma unroll
                        for (int u = 0; u < kAhead; ++u) two_targets(q[u], x, eps2, a);
                    }
                    for (; k + sl < lim; k += S) two_targets(L[k + sl], x, eps2, a);
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int c = 0; c < 4; ++c) v[h][c] += (double)a[h][c];
                }
                wave_lds_sync();
            };
            for (uint32_t qb = q0; qb < q1; qb += kWave) {
                const int nq = (int)min((uint32_t)kWave, q1 - qb);
                int32_t pb = 0;
                uint32_t pc = 0;
                if (lane < nq) {
                    const Cell cb = cells[(uint32_t)(pkeys[qb + lane] >> 32)];
                    pb = cb.begin;
                    pc = (uint32_t)cb.count;
                }
                uint32_t incl = pc;
#pragma unroll
                for (int o = 1; o < kWave; o <<= 1) {
                    const uint32_t y = __shfl_up(incl, o, kWave);
                    if (lane >= o) incl += y;
                }
                const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
                const uint32_t first = incl - pc;  // slot of the partner's first body
                SB[lane] = pb - (int32_t)first;
                for (uint32_t base = 0; base < total;) {
                    const uint32_t m = min((uint32_t)(kFmmList - len), total - base);
                    // one bit per slot where a partner starts: a body's partner
                    // is the number of starts up to its slot, less one
                    if (lane < kFmmList / kWave) ST[lane] = 0ull;
                    wave_lds_sync();
                    if (lane < nq && first - base < m)
                        atomicOr(reinterpret_cast<uint32_t*>(ST) + (first - base) / 32, 1u << ((first - base) % 32));
                    int before = __popcll(__ballot(lane < nq && first < base)) - 1;
                    wave_lds_sync();
                    auto gather = [&](auto batch, uint32_t from) {
                        constexpr int B = decltype(batch)::value;
                        int lo[B];
                        float4 e[B];
#pragma unroll
                        for (int u = 0; u < B; ++u) {
                            const uint64_t st = ST[from / kWave + u];
                            lo[u] = before + __popcll(st & upto);
                            before += __popcll(st);
                        }
#pragma unroll
                        for (int u = 0; u < B; ++u) {
                            const int64_t j = SB[lo[u]] + (int32_t)(base + min(from + u * kWave + lane, m - 1));
                            if constexpr (F32) {
                                e[u] = bodies32[j];
                            } else {
                                const Body b = bodies[j];
                                e[u] = make_float4((float)(b.x - zx), (float)(b.y - zy), (float)(b.z - zz), (float)b.m);
                            }
                        }
#pragma unroll
                        for (int u = 0; u < B; ++u) {
                            const uint32_t off = from + u * kWave + lane;
                            if constexpr (F32)
                                e[u] = make_float4((float)((double)e[u].x - zx), (float)((double)e[u].y - zy),
                                                   (float)((double)e[u].z - zz), e[u].w);
                            if (off < m) L[len + off] = e[u];
                        }
                    };
                    constexpr uint32_t kBatch = kFmmList / kWave;
                    if (m > kWave * kBatch / 2) gather(std::integral_constant<int, (int)kBatch>{}, 0u);
                    else
                        for (uint32_t from = 0; from < m; from += kWave) gather(std::integral_constant<int, 1>{}, from);
                    len += (int)m;
                    base += m;
                    if (len == kFmmList) {
                        flush(len);
                        len = 0;
                    }
                }
                wave_lds_sync();
            }
            flush(len);
            // slices' sums in FP64, in a fixed order
            for (int left = S; left > 1;) {
                const int half = (left + 1) / 2;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const double w = __shfl(v[h][c], (lane + half * H) & (kWave - 1), kWave);
                        if (lane / H + half < left) v[h][c] += w;
                    }
                left = half;
            }
            // lane j now takes target j
            double w[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double lo = __shfl(v[0][c], lane, kWave), hi = __shfl(v[1][c], (lane - H) & (kWave - 1), kWave);
                w[c] = lane < H ? lo : hi;
            }
            if (lane < nA && nchunks > 1) {
                // the leaf's expansion and the self term: k_fmm_leaf_finish
                double* o = part + 4 * ((int64_t)soff[A] + (int64_t)chunk * ca.count + t0 + lane);
                o[0] = w[0];
                o[1] = w[1];
                o[2] = w[2];
                o[3] = w[3];
            } else if (lane < nA) {
                const int64_t i = (int64_t)ca.begin + t0 + lane;
                const Body me = bodies[i];
                double lamA[kNL], g[3], p;
                for (int k = 0; k < kNL; ++k) lamA[k] = lam[A * kNL + k];
                const double dl[3] = {me.x - zx, me.y - zy, me.z - zz};
                l2p(lamA, dl, g, p);
                // the body met itself in its own leaf: no force, a -m/eps
                // potential term removed as it was formed
                const float mself = (float)me.m;
                const double self = (double)(mself * __builtin_amdgcn_rsqf(eps2));
                const int64_t o = perm[i];
                acc[o * 3 + 0] = (float)((double)G * (g[0] + w[0]));
                acc[o * 3 + 1] = (float)((double)G * (g[1] + w[1]));
                acc[o * 3 + 2] = (float)((double)G * (g[2] + w[2]));
                pot[o] = (float)((double)G * (-p + w[3] + self));
            }
        }
    }
}

// Bodies of the leaves cut into chunks: the chunks' sums in chunk order,
// the leaf's expansion and the self term, as in k_fmm_leaf.  One wave per
// cell, lanes over its bodies.
__global__ void __launch_bounds__(256) k_fmm_leaf_finish(const Cell* __restrict__ cells, const Body* __restrict__ bodies,
                                                         const uint32_t* __restrict__ perm,
                                                         const FmmGeo* __restrict__ geo, const double* __restrict__ lam,
                                                         const uint32_t* __restrict__ toff,
                                                         const uint32_t* __restrict__ soff,
                                                         const double* __restrict__ part,
                                                         const DevParams* __restrict__ prm, int64_t cmax, float G,
                                                         float eps2, float* __restrict__ acc, float* __restrict__ pot) {
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x / kWave);
    for (int64_t A = blockIdx.x * (int64_t)(blockDim.x / kWave) + (threadIdx.x / kWave); A < C; A += nwaves) {
        const uint32_t nchunks = toff[A + 1] - toff[A];
        if (nchunks < 2) continue;
        const Cell ca = cells[A];
        const FmmGeo ga = geo[A];
        for (int t = lane; t < ca.count; t += kWave) {
            const int64_t i = (int64_t)ca.begin + t;
            const Body me = bodies[i];
            double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
            for (uint32_t j = 0; j < nchunks; ++j) {
                const double* q = part + 4 * ((int64_t)soff[A] + (int64_t)j * ca.count + t);
                v[0] += q[0];
                v[1] += q[1];
                v[2] += q[2];
                v[3] += q[3];
            }
            double lamA[kNL];
            for (int k = 0; k < kNL; ++k) lamA[k] = lam[A * kNL + k];
            const double dl[3] = {me.x - ga.z[0], me.y - ga.z[1], me.z - ga.z[2]};
            double g[3], p;
            l2p(lamA, dl, g, p);
            const float mself = (float)me.m;
            const double self = (double)(mself * __builtin_amdgcn_rsqf(eps2));
            const int64_t o = perm[i];
            acc[o * 3 + 0] = (float)((double)G * (g[0] + v[0]));
            acc[o * 3 + 1] = (float)((double)G * (g[1] + v[1]));
            acc[o * 3 + 2] = (float)((double)G * (g[2] + v[2]));
            pot[o] = (float)((double)G * (-p + v[3] + self));
        }
    }
}

// Pairs as (target, source) pre-order indices.
__global__ void __launch_bounds__(256) k_fmm_unpack(const uint64_t* __restrict__ keys, int64_t n,
                                                    int32_t* __restrict__ out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        out[2 * i] = (int32_t)(uint32_t)keys[i];
        out[2 * i + 1] = (int32_t)(keys[i] >> 32);
    }
}

__global__ void __launch_bounds__(256) k_fill_u32(uint32_t* __restrict__ p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

}  // namespace

hipError_t launch_fmm_geo(const Cell* cells, const Moments* mom, const Body* bodies, const WalkCell* walk,
                          const uint32_t* pre2bfs, const DevParams* prm, int64_t cmax, FmmGeo* geo, DttCell* dc,
                          hipStream_t s) {
    hipLaunchKernelGGL(k_fmm_geo, dim3(grid_for(cmax * kGeoLanes)), dim3(256), 0, s, cells, mom, bodies, walk, pre2bfs,
                       prm, cmax, geo, dc);
    return hipGetLastError();
}

hipError_t launch_fmm_radii(const uint32_t* lvl_off, int level, int64_t count, DttCell* dc, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fmm_radii, dim3(grid_for(count * kGeoLanes)), dim3(256), 0, s, lvl_off, level, dc);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(n)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_fmm_dtt_root(unsigned long long* ctr, uint64_t* fin, hipStream_t s) {
    hipLaunchKernelGGL(k_fmm_dtt_root, dim3(1), dim3(64), 0, s, ctr, fin);
    return hipGetLastError();
}

hipError_t launch_fmm_dtt(const DttCell* dc, const uint32_t* bfs2pre, double theta, uint64_t* fin, int64_t bound,
                          const unsigned long long* size, unsigned long long* next, uint64_t* fout, int64_t capf,
                          uint64_t* m2l, int64_t capm, uint64_t* p2p, int64_t capp, unsigned long long* ctr,
                          uint32_t* bt, unsigned long long* base, hipStream_t s) {
    const unsigned nb = grid_for(bound, kFmmMaxWaves / kDttWaves);
    const int nw = (int)nb * kDttWaves;
    hipLaunchKernelGGL(k_fmm_dtt_count, dim3(nb), dim3(kDttBlock), 0, s, dc, theta, fin, size, capf, bt);
    hipLaunchKernelGGL(k_fmm_dtt_scan, dim3(1), dim3(1024), 0, s, (const uint32_t*)bt, nw, ctr, next, base);
    hipLaunchKernelGGL(k_fmm_dtt_write, dim3(nb), dim3(kDttBlock), 0, s, dc, bfs2pre, (const uint64_t*)fin, size,
                       (const uint32_t*)bt, (const unsigned long long*)base, fout, capf, m2l, capm, p2p, capp);
    return hipGetLastError();
}

hipError_t launch_fmm_offsets(const uint64_t* keys, int64_t n, int64_t C, uint32_t* off, hipStream_t s) {
    hipLaunchKernelGGL(k_fmm_offsets, dim3(grid_for(C + 1)), dim3(256), 0, s, keys, n, C, off);
    return hipGetLastError();
}

hipError_t launch_fmm_m2l(const Moments* mom, const FmmGeo* geo, const DevParams* prm, int64_t cmax,
                          const uint64_t* keys, const uint32_t* off, double eps2, double* lam,
                          hipStream_t s) {
    int64_t blocks = (cmax + 3) / 4;   // one wave per cell
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fmm_m2l, dim3((unsigned)blocks), dim3(256), 0, s, mom, geo, prm, cmax, keys, off, eps2,
                       lam);
    return hipGetLastError();
}

hipError_t launch_fmm_l2l(const Cell* cells, const FmmGeo* geo, const uint32_t* bfs2pre, const uint32_t* lvl_off,
                          int level, int64_t count, double* lam, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fmm_l2l, dim3(grid_for(count)), dim3(256), 0, s, cells, geo, bfs2pre, lvl_off, level, lam);
    return hipGetLastError();
}

hipError_t launch_fmm_tasks(const Cell* cells, const uint32_t* poff, const DevParams* prm, int64_t cmax,
                            uint32_t* ntask, uint32_t* nslot, unsigned long long* ctr, hipStream_t s) {
    hipLaunchKernelGGL(k_fmm_tasks_count, dim3(grid_for(cmax)), dim3(256), 0, s, cells, poff, prm, cmax, ntask, nslot,
                       ctr);
    return hipGetLastError();
}

hipError_t launch_fmm_tasks_fill(const uint32_t* toff, const uint32_t* poff, const DevParams* prm, int64_t cmax,
                                 uint32_t* task, uint32_t* longs, unsigned long long* ctr, hipStream_t s) {
    hipLaunchKernelGGL(k_fmm_tasks_fill, dim3(grid_for(cmax)), dim3(256), 0, s, toff, poff, prm, cmax, task, longs,
                       reinterpret_cast<uint32_t*>(ctr + 3));
    return hipGetLastError();
}

hipError_t launch_fmm_leaf(const Cell* cells, const Body* bodies, const float4* bodies32, const uint32_t* perm,
                           const FmmGeo* geo, const double* lam, const uint64_t* pkeys, const uint32_t* poff,
                           const uint32_t* task, const uint32_t* toff, const uint32_t* soff, int64_t ntasks,
                           const uint32_t* longs, int64_t nlong, double* part, const DevParams* prm, int64_t cmax,
                           float G, float eps2, float* acc, float* pot, hipStream_t s) {
    const auto leaf = bodies32 ? k_fmm_leaf<true> : k_fmm_leaf<false>;
    for (int64_t first = 0; first < nlong + ntasks; first += kFmmLaunch) {
        const int64_t tasks = std::min(kFmmLaunch, nlong + ntasks - first);
        hipLaunchKernelGGL(leaf, dim3((unsigned)((tasks + kFmmWaves - 1) / kFmmWaves)), dim3(kFmmWaves * kWave), 0, s, cells,
                           bodies, bodies32, perm, geo, lam, pkeys, poff, task, toff, soff, first, ntasks, longs, nlong, part,
                           G, eps2, acc, pot);
    }
    int64_t fb = (cmax + 3) / 4;
    if (fb > 65536) fb = 65536;
    hipLaunchKernelGGL(k_fmm_leaf_finish, dim3((unsigned)fb), dim3(256), 0, s, cells, bodies, perm, geo, lam, toff,
                       soff, (const double*)part, prm, cmax, G, eps2, acc, pot);
    return hipGetLastError();
}

hipError_t launch_fmm_unpack(const uint64_t* keys, int64_t n, int32_t* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fmm_unpack, dim3(grid_for(n)), dim3(256), 0, s, keys, n, out);
    return hipGetLastError();
}

}  // namespace tc
