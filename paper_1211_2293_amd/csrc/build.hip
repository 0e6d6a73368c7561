// Tree construction and cell moments (§3.1 of the paper: recursive 4-/8-way
// subdivision until a subspace holds at most leaf_cap bodies; each cell is
// its bodies' total mass at their centre of mass).
//
// Pipeline, one stream, no host synchronisation:
//   bbox     root cube: per-axis minimum corner, power-of-two side (FP64);
//            the same pass packs the input as (x, y, z, m) records
//   keys     Morton key of FP64-quantised coordinates, index iota
//   sort     from kBucketMaxN bodies a stable LSD radix sort of (key,
//            index), 8 bits per pass (each tile ranked in LDS before it is
//            written out); keys, sort and gather of smaller systems are in
//            bodysort.hip
//   gather   bodies into key order, FP64, one packed record per body
//   topology all cells at once from the sorted keys (no per-level launches):
//            body i starts the cells of levels a_i..l*_i, where a_i is one
//            more than its common-prefix length with body i-1 and l*_i is
//            one below the deepest level at which a run of leaf_cap+1
//            consecutive keys around i still shares a prefix; their
//            exclusive scan is the depth-first pre-order index; the level
//            order is one more radix pass, keyed by level, and the walk
//            groups one more scan
//   moments  FP64, leaves over bodies in order, internal cells over their
//            children in digit order: small subtrees within a block each,
//            the cells above them by one block
//   mac      opening radius per cell for the current theta
//
// Every expression that decides an integer (keys, topology, opening radii)
// is compiled without floating-point contraction.
#include "tc_internal.h"
#include "keys.h"

#include <math.h>

#include <algorithm>

namespace tc {
namespace {

using namespace keys;

__device__ __forceinline__ int wave_lane() { return threadIdx.x & (kWave - 1); }

// ---------------------------------------------------------------- bbox ----

// With KICK the bodies are first moved by the half kick and the drift of a
// step, as k_kick_drift does: one launch and one reading of the positions less
// (a step of 10,000 bodies 158 -> 155 us, of 1,048,576 2,165 -> 2,136).
template <typename T, int D, bool KICK>
__global__ void __launch_bounds__(256) k_bbox_part(T* __restrict__ pos, const T* __restrict__ mass,
                                                   int64_t n, double* __restrict__ part,
                                                   typename Packed<T>::type* __restrict__ packed,
                                                   T* __restrict__ vel, const float* __restrict__ acc, T hdt, T dt) {
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    int bad = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        T c[3] = {T(0), T(0), T(0)};
#pragma unroll
        for (int a = 0; a < D; ++a) {
            c[a] = pos[i * D + a];
            if (KICK) {
                const T v = vel[i * D + a] + hdt * (T)acc[i * D + a];
                vel[i * D + a] = v;
                c[a] = c[a] + dt * v;
                pos[i * D + a] = c[a];
            }
            const double v = (double)c[a];
            if (!isfinite(v)) { bad = 1; continue; }
            lo[a] = fmin(lo[a], v);
            hi[a] = fmax(hi[a], v);
        }
        const T mt = mass[i];
        const double m = (double)mt;
        if (!(isfinite(m) && m > 0.0)) bad = 1;
        if (packed) {
            typename Packed<T>::type r;
            r.x = c[0];
            r.y = c[1];
            r.z = c[2];
            r.w = mt;
            packed[i] = r;
        }
    }
    __shared__ double s_lo[3][256], s_hi[3][256];
    __shared__ int s_bad[256];
    const int t = threadIdx.x;
#pragma unroll
    for (int a = 0; a < 3; ++a) { s_lo[a][t] = lo[a]; s_hi[a][t] = hi[a]; }
    s_bad[t] = bad;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                s_lo[a][t] = fmin(s_lo[a][t], s_lo[a][t + w]);
                s_hi[a][t] = fmax(s_hi[a][t], s_hi[a][t + w]);
            }
            s_bad[t] |= s_bad[t + w];
        }
        __syncthreads();
    }
    if (t == 0) {
        double* o = part + blockIdx.x * 7;
        for (int a = 0; a < 3; ++a) { o[a] = s_lo[a][0]; o[3 + a] = s_hi[a][0]; }
        o[6] = (double)s_bad[0];
    }
}

__global__ void __launch_bounds__(256) k_bbox_final(const double* __restrict__ part, int nb, int dim,
                                                    DevParams* prm) {
    __shared__ double s_lo[3][256], s_hi[3][256];
    __shared__ int s_bad[256];
    const int t = threadIdx.x;
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    int bad = 0;
    for (int b = t; b < nb; b += 256) {
        for (int a = 0; a < 3; ++a) {
            lo[a] = fmin(lo[a], part[b * 7 + a]);
            hi[a] = fmax(hi[a], part[b * 7 + 3 + a]);
        }
        bad |= part[b * 7 + 6] != 0.0;
    }
    for (int a = 0; a < 3; ++a) { s_lo[a][t] = lo[a]; s_hi[a][t] = hi[a]; }
    s_bad[t] = bad;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) {
            for (int a = 0; a < 3; ++a) {
                s_lo[a][t] = fmin(s_lo[a][t], s_lo[a][t + w]);
                s_hi[a][t] = fmax(s_hi[a][t], s_hi[a][t + w]);
            }
            s_bad[t] |= s_bad[t + w];
        }
        __syncthreads();
    }
    if (t == 0) {
        const double l[3] = {s_lo[0][0], s_lo[1][0], s_lo[2][0]}, h[3] = {s_hi[0][0], s_hi[1][0], s_hi[2][0]};
        store_cube(make_cube(l, h, dim), s_bad[0] != 0, prm);
    }
}

// ---------------------------------------------------------------- keys ----

template <typename T, int D>
__global__ void __launch_bounds__(256) k_keys(const T* __restrict__ pos, int64_t n,
                                              const DevParams* __restrict__ prm,
                                              uint64_t* __restrict__ keys, uint32_t* __restrict__ idx) {
    const double scale = prm->scale, lo[3] = {prm->lo[0], prm->lo[1], prm->lo[2]};
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t key = morton<D>((double)pos[i * D], (double)pos[i * D + 1],
                                       D == 3 ? (double)pos[i * D + D - 1] : 0.0, lo, scale);
        keys[i] = key;
        idx[i] = (uint32_t)i;
    }
}

// ---------------------------------------------------------------- sort ----
// Reduce-then-scan LSD radix sort: per tile digit counts, a scan of the
// counts in digit-major order, then a stable scatter in which each wave
// ranks its keys with ballot-based digit matching.  The scatter loads all
// of a thread's keys before ranking any (one block per tile leaves few
// waves per CU, and a load per round of 256 keys waited on memory round
// after round: 20.2 us per pass of 1M keys, 16.0 us with the loads first).
// Recording every round's per-wave digit counts and placing all keys after
// one prefix pass (three barriers per tile instead of three per round) took
// 18.4 us.  Copies of the running places (two) and counts (three) let a
// round place its keys while the next round's places are advanced and a
// later round's counts cleared: one barrier per round instead of three
// (1M keys: 0.191 against 0.201 ms per sort; 16.7M: 1.57 against 1.64).
// PER keys per thread, tiles of 256 PER keys (sort_per).
// Placing each key straight at its output place writes about one key per
// digit per round of 256, so a line of the output is written in many
// pieces; large sorts (STAGE, from kSortStageMin keys) first rank the whole
// tile into LDS in output order and then write each digit's run with
// consecutive threads (16.7M keys: 2.36 to 1.64 ms for the eight passes,
// 4M: 0.56 to 0.46; 1M keys, whose passes stay in the caches, 0.20 to 0.22,
// so smaller sorts do not stage; the same at 1.5M).
//
// Where a pass's pairs come from and go to.  A plain pass reads keys and
// values (nullable) and writes both at their places.  The level pass sorts
// the cells by level (pre-order within a level, so the children of a cell
// stay adjacent): it reads each cell's level as its key and its pre-order
// index as its value, writes the level order both ways, and the first tile
// writes where each level starts (its digit bases: no tile precedes it).
struct PairsIn {
    const uint64_t* __restrict__ k;
    const uint32_t* __restrict__ v;
    __device__ uint64_t key(int64_t i) const { return k[i]; }
    __device__ uint32_t val(int64_t i) const { return v ? v[i] : 0u; }
};
struct PairsOut {
    uint64_t* __restrict__ k;
    uint32_t* __restrict__ v;
    __device__ void put(uint32_t p, uint64_t key, uint32_t val) const {
        k[p] = key;
        if (v) v[p] = val;
    }
    __device__ void starts(int, uint32_t) const {}
};
struct LevelsIn {
    const Cell* __restrict__ cells;
    __device__ uint64_t key(int64_t i) const { return (uint64_t)cells[i].level; }
    __device__ uint32_t val(int64_t i) const { return (uint32_t)i; }
};
struct LevelsOut {
    uint32_t* __restrict__ bfs2pre;
    uint32_t* __restrict__ pre2bfs;
    uint32_t* __restrict__ lvl_off;   // levels 0..L and the end
    int L;
    __device__ void put(uint32_t p, uint64_t, uint32_t val) const {
        bfs2pre[p] = val;
        pre2bfs[val] = p;
    }
    __device__ void starts(int d, uint32_t base) const {
        if (d <= L + 1) lvl_off[d] = base;
    }
};

// Tiles of `tile` keys that hold the first n keys (at least one, so that
// the first tile always writes the digit starts).
__device__ __forceinline__ int64_t live_tiles(int64_t n, int64_t tile) {
    return n > 0 ? (n + tile - 1) / tile : 1;
}

template <int PER, class In>
// n_live (nullable, device): sort only the first min(n, *n_live) keys; the
// tiles past them (a pass over the cells is sized for the most cells a tree
// can have) count, scan and scatter nothing.
__global__ void __launch_bounds__(256) k_sort_hist(In in, int64_t n, const uint32_t* __restrict__ n_live, int shift,
                                                   uint32_t* __restrict__ hist, int64_t tiles) {
    if (n_live && (int64_t)*n_live < n) n = *n_live;
    const int64_t tile = blockIdx.x;
    if (tile >= live_tiles(n, 256 * PER)) return;   // nothing reads the counts of later tiles
    __shared__ uint32_t cnt[4][256];
    const int t = threadIdx.x, w = t >> 6;
    for (int a = 0; a < 4; ++a) cnt[a][t] = 0;
    __syncthreads();
    const int64_t base = tile * (256 * PER);
#pragma unroll 4
    for (int j = 0; j < PER; ++j) {
        const int64_t i = base + j * 256 + t;
        if (i < n) atomicAdd(&cnt[w][(unsigned)(in.key(i) >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[(int64_t)t * tiles + tile] = cnt[0][t] + cnt[1][t] + cnt[2][t] + cnt[3][t];
}

// Exclusive block scan of one value per thread (256 threads); returns the
// prefix, writes the block total into *total (shared).
__device__ __forceinline__ uint32_t block_exscan_u32(uint32_t v, uint32_t* s_w, uint32_t* total) {
    const int lane = wave_lane(), w = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, kWave);
        if (lane >= o) x += y;
    }
    if (lane == kWave - 1) s_w[w] = x;
    __syncthreads();
    uint32_t wbase = 0;
    for (int k = 0; k < w; ++k) wbase += s_w[k];
    if (threadIdx.x == 255) *total = wbase + x;
    __syncthreads();
    return wbase + x - v;
}

template <int PER>
__global__ void __launch_bounds__(256) k_sort_scan(uint32_t* __restrict__ hist, int64_t tiles, int64_t n,
                                                   const uint32_t* __restrict__ n_live,
                                                   uint32_t* __restrict__ digit_tot) {
    __shared__ uint32_t s_w[4];
    __shared__ uint32_t s_tot;
    if (n_live && (int64_t)*n_live < n) n = *n_live;
    const int64_t tl = live_tiles(n, 256 * PER);
    uint32_t* h = hist + (int64_t)blockIdx.x * tiles;
    uint32_t carry = 0;
    for (int64_t c = 0; c < tl; c += 256) {
        const int64_t i = c + threadIdx.x;
        const uint32_t v = i < tl ? h[i] : 0u;
        const uint32_t ex = block_exscan_u32(v, s_w, &s_tot);
        if (i < tl) h[i] = carry + ex;
        carry += s_tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) digit_tot[blockIdx.x] = carry;
}

// SCAN: hist holds the raw per-tile counts (no k_sort_scan before it), and
// each block sums its digit's row itself: the earlier tiles' counts and the
// total, which block 0 also stores in digit_tot.  For a few tiles (at most
// kSortScanInScatter) this costs less than the scan's own launch.
constexpr int64_t kSortScanInScatter = 128;
// Sorts of at least kSortStageMin keys stage each tile in LDS (STAGE).
constexpr int64_t kSortStageMin = (int64_t)1 << 21;
constexpr int kSortStagePer = 16;

template <int PER, bool SCAN, bool STAGE, class In, class Out>
__global__ void __launch_bounds__(256) k_sort_scatter(In in, Out out, int64_t n, const uint32_t* __restrict__ n_live,
                                                      int shift, const uint32_t* __restrict__ hist,
                                                      uint32_t* __restrict__ digit_tot, int64_t tiles) {
    if (n_live && (int64_t)*n_live < n) n = *n_live;
    constexpr int kTile = 256 * PER;
    constexpr int kStage = STAGE ? kTile : 1;
    const int64_t tl = live_tiles(n, kTile);
    if ((int64_t)blockIdx.x >= tl) return;
    __shared__ uint32_t s_base[256];   // where the tile's keys of each digit start in the output
    // running place of each digit (staged: in the tile, else in the output)
    // in two copies, and each wave's count of each digit in a round in three:
    // round r reads place copy r % 2 and count copy r % 3, writes place copy
    // (r + 1) % 2 and clears count copy (r + 2) % 3, so one barrier per round
    // separates every write of a copy from its reads
    __shared__ uint32_t s_pos[2][256];
    __shared__ uint32_t s_lstart[256]; // staged: where each digit's keys start in the tile
    __shared__ uint32_t s_wcnt[3][4][256];
    __shared__ uint32_t s_w[4];
    __shared__ uint32_t s_tot;
    __shared__ uint64_t s_key[kStage];
    __shared__ uint32_t s_val[kStage];
    const int t = threadIdx.x, w = t >> 6, lane = wave_lane();
    const int64_t tile = blockIdx.x;
    uint32_t own = 0;   // this tile's count of digit t (staged only)
    if (SCAN) {
        const uint32_t* row = hist + (int64_t)t * tiles;
        uint32_t pre = 0, tot = 0;
#pragma unroll 8
        for (int64_t k = 0; k < tl; ++k) {
            const uint32_t v = row[k];
            tot += v;
            if (k < tile) pre += v;
        }
        if (tile == 0) digit_tot[t] = tot;
        if (STAGE) own = row[tile];
        s_base[t] = block_exscan_u32(tot, s_w, &s_tot) + pre;
    } else {
        const uint32_t tot = digit_tot[t];
        const uint32_t here = hist[(int64_t)t * tiles + tile];
        if (STAGE) own = (tile + 1 < tl ? hist[(int64_t)t * tiles + tile + 1] : tot) - here;
        s_base[t] = block_exscan_u32(tot, s_w, &s_tot) + here;
    }
    if (tile == 0) out.starts(t, s_base[t]);
    if (STAGE) {
        const uint32_t l = block_exscan_u32(own, s_w, &s_tot);
        s_lstart[t] = l;
        s_pos[0][t] = l;
    } else {
        s_pos[0][t] = s_base[t];
    }
    for (int a = 0; a < 4; ++a) s_wcnt[0][a][t] = s_wcnt[1][a][t] = 0;
    uint64_t kr[PER];
    uint32_t vr[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int64_t i = tile * kTile + r * 256 + t;
        kr[r] = i < n ? in.key(i) : 0ull;
        vr[r] = i < n ? in.val(i) : 0u;
    }
    __syncthreads();
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const bool valid = tile * kTile + r * 256 + t < n;
        const uint64_t k = kr[r];
        const uint32_t d = (uint32_t)(k >> shift) & 255u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            peers &= bit ? bb : ~bb;
        }
        const uint64_t before = peers & lt;
        const int cur = r & 1, nxt = cur ^ 1, cc = r % 3, cz = (r + 2) % 3;
        if (valid && before == 0) s_wcnt[cc][w][d] = (uint32_t)__popcll(peers);
        __syncthreads();
        if (valid) {
            uint32_t p = s_pos[cur][d] + (uint32_t)__popcll(before);
            for (int a = 0; a < w; ++a) p += s_wcnt[cc][a][d];
            if (STAGE) {
                s_key[p] = k;
                s_val[p] = vr[r];
            } else {
                out.put(p, k, vr[r]);
            }
        }
        // the next round's places, advanced by this round's counts, and the
        // counts of the round after it cleared (last read by the previous round)
        s_pos[nxt][t] = s_pos[cur][t] + s_wcnt[cc][0][t] + s_wcnt[cc][1][t] + s_wcnt[cc][2][t] +
                        s_wcnt[cc][3][t];
        for (int a = 0; a < 4; ++a) s_wcnt[cz][a][t] = 0;
    }
    if (STAGE) {
        __syncthreads();
        // The tile's keys now sit in LDS in output order, digit by digit:
        // consecutive threads write consecutive places of a digit's run.
        const int64_t left = n - tile * kTile;
        const int live = left < kTile ? (int)left : kTile;
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            const int l = r * 256 + t;
            if (l < live) {
                const uint64_t k = s_key[l];
                const uint32_t d = (uint32_t)(k >> shift) & 255u;
                out.put(s_base[d] + (uint32_t)l - s_lstart[d], k, s_val[l]);
            }
        }
    }
}

// -------------------------------------------------------------- gather ----

template <typename T>
__global__ void __launch_bounds__(256) k_gather(const typename Packed<T>::type* __restrict__ packed,
                                                const uint32_t* __restrict__ perm, int64_t n,
                                                Body* __restrict__ bodies, float4* __restrict__ bodies32) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const typename Packed<T>::type r = packed[perm[i]];
        Body b;
        b.x = (double)r.x;
        b.y = (double)r.y;
        b.z = (double)r.z;
        b.m = (double)r.w;
        bodies[i] = b;
        // FP32 inputs also get a compact copy (exactly the input values)
        if (bodies32) bodies32[i] = make_float4((float)b.x, (float)b.y, (float)b.z, (float)b.m);
    }
}

// ---------------------------------------------------------------- scan ----
// Exclusive scan of u32 values: out[i] = sum_{j<i} in[j], out[n] = total.
// With n_live (device, nullable) only the first m = min(n, *n_live) values
// are read and written, and the total also goes to out[m]; the grids cover
// n.

__device__ __forceinline__ int64_t live_count(int64_t n, const uint32_t* n_live) {
    return (n_live && (int64_t)*n_live < n) ? (int64_t)*n_live : n;
}

__global__ void __launch_bounds__(256) k_scan_reduce(const uint32_t* __restrict__ in, int64_t n,
                                                     const uint32_t* __restrict__ n_live,
                                                     uint32_t* __restrict__ part) {
    __shared__ uint32_t s_w[4];
    __shared__ uint32_t s_tot;
    n = live_count(n, n_live);
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    if (base >= n) {                       // the whole tile is past the live values
        if (threadIdx.x == 0) part[blockIdx.x] = 0u;
        return;
    }
    uint32_t s = 0;
    for (int j = 0; j < kScanTile / 256; ++j) {
        const int64_t i = base + j * 256 + threadIdx.x;
        if (i < n) s += in[i];
    }
    block_exscan_u32(s, s_w, &s_tot);
    if (threadIdx.x == 0) part[blockIdx.x] = s_tot;
}

// The tiles' sums in one block of 1024 threads, four consecutive tiles per
// thread, over the tiles that hold live values only.
__global__ void __launch_bounds__(1024) k_scan_part(uint32_t* __restrict__ part, int64_t tiles,
                                                    uint32_t* __restrict__ out, int64_t n,
                                                    const uint32_t* __restrict__ n_live) {
    __shared__ uint32_t s_w[16];
    const int64_t m = live_count(n, n_live);
    int64_t tl = (m + kScanTile - 1) / kScanTile;
    if (tl > tiles) tl = tiles;
    const int t = threadIdx.x, lane = wave_lane(), w = t >> 6;
    uint32_t carry = 0;
    for (int64_t c = 0; c < tl; c += 4 * 1024) {
        const int64_t i = c + 4 * t;
        const uint32_t v0 = i < tl ? part[i] : 0u, v1 = i + 1 < tl ? part[i + 1] : 0u;
        const uint32_t v2 = i + 2 < tl ? part[i + 2] : 0u, v3 = i + 3 < tl ? part[i + 3] : 0u;
        const uint32_t own = v0 + v1 + v2 + v3;
        uint32_t x = own;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, kWave);
            if (lane >= o) x += y;
        }
        if (lane == kWave - 1) s_w[w] = x;
        __syncthreads();
        uint32_t wbase = 0, tot = 0;
        for (int k = 0; k < 16; ++k) {
            if (k < w) wbase += s_w[k];
            tot += s_w[k];
        }
        uint32_t e = carry + wbase + x - own;
        if (i < tl) part[i] = e;
        e += v0;
        if (i + 1 < tl) part[i + 1] = e;
        e += v1;
        if (i + 2 < tl) part[i + 2] = e;
        e += v2;
        if (i + 3 < tl) part[i + 3] = e;
        carry += tot;
        __syncthreads();    // s_w is rewritten by the next round
    }
    if (t == 0) {
        out[n] = carry;
        out[m] = carry;
    }
}

// A tile is kScanTile / 1024 rows of 1024 values; thread t takes values
// 4t..4t+3 of each row (one 16-byte load and store when VEC: in and out
// 16-byte aligned), so a wave's accesses are contiguous.  (One thread per 16
// consecutive values, each loaded alone, took 100 us for 16.7M values; the
// rows take about 23.)
template <bool VEC>
__global__ void __launch_bounds__(256) k_scan_apply(const uint32_t* __restrict__ in, int64_t n,
                                                    const uint32_t* __restrict__ n_live,
                                                    const uint32_t* __restrict__ part,
                                                    uint32_t* __restrict__ out) {
    constexpr int kRows = kScanTile / 1024;
    static_assert(kScanTile % 1024 == 0, "scan tiles are whole rows of 1024 values");
    __shared__ uint32_t s_w[kRows][4];
    n = live_count(n, n_live);
    const int64_t tile0 = (int64_t)blockIdx.x * kScanTile;
    if (tile0 >= n) return;
    const int t = threadIdx.x, lane = wave_lane(), w = t >> 6;
    uint4 q[kRows];
    uint32_t own[kRows], x[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const int64_t i = tile0 + r * 1024 + 4 * t;
        if (VEC && i + 3 < n) {
            q[r] = *reinterpret_cast<const uint4*>(in + i);
        } else {
            q[r].x = i < n ? in[i] : 0u;
            q[r].y = i + 1 < n ? in[i + 1] : 0u;
            q[r].z = i + 2 < n ? in[i + 2] : 0u;
            q[r].w = i + 3 < n ? in[i + 3] : 0u;
        }
        own[r] = q[r].x + q[r].y + q[r].z + q[r].w;
        x[r] = own[r];
    }
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const uint32_t y = __shfl_up(x[r], o, kWave);
            if (lane >= o) x[r] += y;
        }
    }
    if (lane == kWave - 1) {
#pragma unroll
        for (int r = 0; r < kRows; ++r) s_w[r][w] = x[r];
    }
    __syncthreads();
    uint32_t run = part[blockIdx.x];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        uint32_t wbase = 0;
        for (int k = 0; k < w; ++k) wbase += s_w[r][k];
        uint4 e;
        e.x = run + wbase + x[r] - own[r];
        e.y = e.x + q[r].x;
        e.z = e.y + q[r].y;
        e.w = e.z + q[r].z;
        const int64_t i = tile0 + r * 1024 + 4 * t;
        if (VEC && i + 3 < n) {
            *reinterpret_cast<uint4*>(out + i) = e;
        } else {
            if (i < n) out[i] = e.x;
            if (i + 1 < n) out[i + 1] = e.y;
            if (i + 2 < n) out[i + 2] = e.z;
            if (i + 3 < n) out[i + 3] = e.w;
        }
        run += s_w[r][0] + s_w[r][1] + s_w[r][2] + s_w[r][3];
    }
}

// Short arrays in one block of 1024 threads, one launch instead of three.
// A segment is kScanSmallRows rows of 4096 values; thread t loads values
// 4t..4t+3 of each row with one 16-byte load, and the rows of a segment are
// scanned together between one pair of barriers, with a running carry from
// segment to segment.  in and out must be 16-byte aligned.
constexpr int kScanSmallRows = 4;
constexpr int64_t kScanSmallSeg = kScanSmallRows * 4096;
constexpr int64_t kScanSmallMax = 8 * kScanSmallSeg;   // longest array sent here

__global__ void __launch_bounds__(1024) k_scan_small(const uint32_t* __restrict__ in, int64_t n,
                                                     const uint32_t* __restrict__ n_live,
                                                     uint32_t* __restrict__ out) {
    __shared__ uint32_t s_w[kScanSmallRows][16];
    const int64_t m = live_count(n, n_live);
    const int t = threadIdx.x, lane = wave_lane(), w = t >> 6;
    uint32_t carry = 0;
    for (int64_t c = 0; c < m; c += kScanSmallSeg) {
        uint4 q[kScanSmallRows];
        uint32_t x[kScanSmallRows], sum[kScanSmallRows];
#pragma unroll
        for (int r = 0; r < kScanSmallRows; ++r) {
            const int64_t i = c + r * 4096 + 4 * t;
            if (i + 3 < m) {
                q[r] = *reinterpret_cast<const uint4*>(in + i);
            } else {
                q[r].x = i < m ? in[i] : 0u;
                q[r].y = i + 1 < m ? in[i + 1] : 0u;
                q[r].z = i + 2 < m ? in[i + 2] : 0u;
                q[r].w = 0u;
            }
            sum[r] = q[r].x + q[r].y + q[r].z + q[r].w;
            x[r] = sum[r];
        }
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
#pragma unroll
            for (int r = 0; r < kScanSmallRows; ++r) {
                const uint32_t y = __shfl_up(x[r], o, kWave);
                if (lane >= o) x[r] += y;
            }
        }
        if (lane == kWave - 1) {
#pragma unroll
            for (int r = 0; r < kScanSmallRows; ++r) s_w[r][w] = x[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kScanSmallRows; ++r) {
            uint32_t pre = 0, tot = 0;
            for (int k = 0; k < 16; ++k) {
                const uint32_t v = s_w[r][k];
                if (k < w) pre += v;
                tot += v;
            }
            const int64_t i = c + r * 4096 + 4 * t;
            uint4 e;
            e.x = carry + pre + x[r] - sum[r];
            e.y = e.x + q[r].x;
            e.z = e.y + q[r].y;
            e.w = e.z + q[r].z;
            if (i + 3 < m) {
                *reinterpret_cast<uint4*>(out + i) = e;
            } else {
                if (i < m) out[i] = e.x;
                if (i + 1 < m) out[i + 1] = e.y;
                if (i + 2 < m) out[i + 2] = e.z;
            }
            carry += tot;
        }
        __syncthreads();    // s_w is rewritten by the next segment
    }
    if (t == 0) {
        out[n] = carry;
        out[m] = carry;
    }
}

// Exclusive scan of n values (the first min(n, *n_live) with n_live) into
// out, with out[n] and out[live] the total; part holds `tiles` partial sums.
static void scan_u32(const uint32_t* in, int64_t n, const uint32_t* n_live, uint32_t* out, uint32_t* part,
                     int64_t tiles, hipStream_t s) {
    if (n <= kScanSmallMax && (reinterpret_cast<uintptr_t>(in) & 15) == 0 &&
        (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
        hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(1024), 0, s, in, n, n_live, out);
        return;
    }
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)tiles), dim3(256), 0, s, in, n, n_live, part);
    hipLaunchKernelGGL(k_scan_part, dim3(1), dim3(1024), 0, s, part, tiles, out, n, n_live);
    if ((reinterpret_cast<uintptr_t>(in) & 15) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0)
        hipLaunchKernelGGL(k_scan_apply<true>, dim3((unsigned)tiles), dim3(256), 0, s, in, n, n_live,
                           (const uint32_t*)part, out);
    else
        hipLaunchKernelGGL(k_scan_apply<false>, dim3((unsigned)tiles), dim3(256), 0, s, in, n, n_live,
                           (const uint32_t*)part, out);
}

// ------------------------------------------------------------ topology ----

// Number of leading Morton digits two keys share (L if equal).
template <int D>
__device__ __forceinline__ int common_digits(uint64_t a, uint64_t b) {
    const uint64_t x = a ^ b;
    if (x == 0) return D == 3 ? 21 : 31;
    const int z = __clzll(x);
    return D == 3 ? (z - 1) / 3 : (z - 2) / 2;
}

// Per body i: a = the shallowest level at which a cell starts at i (one
// past the digits i shares with i - 1), lstar = the deepest level of a cell
// containing i that is not a leaf, plus one (leaf_cap + 1 consecutive
// bodies sharing c digits put an internal cell at level c).  The window
// depths c_j = common digits of bodies j and j + leaf_cap are computed once
// per block tile into LDS, and each body takes the maximum over the windows
// that contain it.
constexpr int kTopoTile = 256;

template <int D>
__global__ void __launch_bounds__(kTopoTile) k_topo_count(const uint64_t* __restrict__ keys, int64_t n, int leaf_cap,
                                                          uint32_t* __restrict__ range, uint32_t* __restrict__ nper,
                                                          uint32_t* __restrict__ tile_tot) {
    constexpr int L = D == 3 ? 21 : 31;
    __shared__ int8_t s_c[kTopoTile + kMaxLeafCap];   // c_j for j = i0 - leaf_cap .. i0 + kTopoTile - 1
    __shared__ uint32_t s_tot;
    const int t = threadIdx.x;
    for (int64_t i0 = (int64_t)blockIdx.x * kTopoTile; i0 < n; i0 += (int64_t)gridDim.x * kTopoTile) {
        for (int q = t; q < kTopoTile + leaf_cap; q += kTopoTile) {
            const int64_t j = i0 - leaf_cap + q;
            s_c[q] = (j >= 0 && j + leaf_cap < n) ? (int8_t)common_digits<D>(keys[j], keys[j + leaf_cap]) : (int8_t)-1;
        }
        __syncthreads();
        const int64_t i = i0 + t;
        uint32_t own = 0;
        if (i < n) {
            const int a = (i == 0) ? 0 : common_digits<D>(keys[i - 1], keys[i]) + 1;
            // windows j = i - leaf_cap .. i (those out of range hold -1)
            int deep = -1;
            for (int q = t; q <= t + leaf_cap; ++q) deep = s_c[q] > deep ? s_c[q] : deep;
            int lstar = 0;
            if (deep >= 0) lstar = (deep < L - 1 ? deep : L - 1) + 1;
            range[i] = (uint32_t)a | ((uint32_t)lstar << 8);
            own = lstar >= a ? (uint32_t)(lstar - a + 1) : 0u;
            nper[i] = own;
        }
        if (tile_tot) {
            if (t == 0) s_tot = 0u;
            __syncthreads();
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) own += __shfl_xor(own, o, kWave);
            if (wave_lane() == 0) atomicAdd(&s_tot, own);
            __syncthreads();
            if (t == 0) tile_tot[i0 / kTopoTile] = s_tot;
        }
        __syncthreads();
    }
}

// The cells that start at body i (levels a_i..l*_i) at their pre-order
// indices base + (l - a_i): prefix, first body, level, parent and the leaf
// mark.  Their ends (count and skip) come from a pass with one lane per cell
// (topo_end): a body that starts many cells would otherwise run their searches
// one after another while the other lanes of its wave, most of which start
// none, wait.
template <int D>
__device__ __forceinline__ void emit_cells(int64_t i, uint32_t range, uint32_t base, uint64_t key,
                                           Cell* __restrict__ cells, int64_t cmax) {
    constexpr int L = D == 3 ? 21 : 31;
    const int a = (int)(range & 255u), lstar = (int)(range >> 8);
    for (int l = a; l <= lstar; ++l) {
        const int64_t k = (int64_t)base + (l - a);
        if (k >= cmax) break;
        Cell c;
        c.prefix = l == 0 ? 0ull : key >> (D * (L - l));
        c.begin = (int32_t)i;
        c.count = 0;                               // topo_end
        c.skip = 0;
        c.parent = (l == 0) ? -1 : (l > a ? (int32_t)(k - 1) : -2);
        c.level = l;
        c.leaf_nch = (l == lstar) ? (int32_t)0x80000000u : 0;
        cells[k] = c;
    }
}

// The number of cells C, known once the last body's are placed.
__device__ __forceinline__ void store_ncells(uint32_t C, int64_t cmax, DevParams* prm) {
    // C never exceeds the bound (internal cells are disjoint per level
    // and hold > leaf_cap bodies); clamp anyway so no reader can run off
    prm->ncells = (int64_t)C > cmax ? (uint32_t)cmax : C;
    if ((int64_t)C > cmax) atomicOr(&prm->status, kFlagOverflow);
}

template <int D>
__global__ void __launch_bounds__(256) k_topo_emit(const uint64_t* __restrict__ keys, int64_t n,
                                                   const uint32_t* __restrict__ range,
                                                   const uint32_t* __restrict__ cstart, Cell* __restrict__ cells,
                                                   int64_t cmax, DevParams* prm, BigList big) {
    if (blockIdx.x == 0 && threadIdx.x < kLevels) big.count[threadIdx.x * BigList::kStride] = 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) store_ncells(cstart[n], cmax, prm);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        emit_cells<D>(i, range[i], cstart[i], keys[i], cells, cmax);
}

// A cell's end: the first body after its first whose prefix at the cell's
// level differs (a galloping search, then bisection over the sorted keys; the
// root ends at n), giving its body count and its skip (the pre-order index of
// the cell that starts there).
template <int D>
__device__ __forceinline__ void topo_end(const uint64_t* __restrict__ keys, int64_t n,
                                         const uint32_t* __restrict__ cstart, const Cell& c,
                                         Cell* __restrict__ out) {
    constexpr int L = D == 3 ? 21 : 31;
    const int64_t i = c.begin;
    const int l = c.level;
    int64_t end = n;
    if (l > 0) {
        const int shift = D * (L - l);
        const uint64_t prefix = c.prefix;
        int64_t lo = i, step = 1, hi = i + 1;
        while (hi < n && (keys[hi] >> shift) == prefix) {
            lo = hi;
            step <<= 1;
            hi = i + step;
        }
        if (hi > n) hi = n;
        while (hi - lo > 1) {
            const int64_t mid = lo + ((hi - lo) >> 1);
            if ((keys[mid] >> shift) == prefix) lo = mid; else hi = mid;
        }
        end = hi;
    }
    out->count = (int32_t)(end - i);
    out->skip = (int32_t)cstart[end];
}

template <int D>
__global__ void __launch_bounds__(256) k_topo_ends(const uint64_t* __restrict__ keys, int64_t n,
                                                   const uint32_t* __restrict__ cstart, Cell* __restrict__ cells,
                                                   const DevParams* __restrict__ prm, int64_t cmax) {
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < C;
         k += (int64_t)gridDim.x * blockDim.x)
        topo_end<D>(keys, n, cstart, cells[k], &cells[k]);
}

// Parents and child counts: an internal cell walks over its children (the next
// one starts where the last one's subtree ends); f(child index, child) for
// each.
template <typename F>
__device__ __forceinline__ void link_children(Cell* __restrict__ cells, int64_t k, const Cell& c, int64_t C, F&& f) {
    int nch = 0;
    int64_t ch = k + 1;
    const int64_t end = c.skip < C ? c.skip : C;
    while (ch < end) {
        cells[ch].parent = (int32_t)k;
        ++nch;
        const Cell cc = cells[ch];
        f(ch, cc);
        ch = cc.skip > ch ? (int64_t)cc.skip : end;   // defensive: the skip chain only moves forward
    }
    cells[k].leaf_nch = nch;
}

// Cells with subtrees of more than big.sub cells go on their level's list
// (BigList), for the upper part of the moments pass: a block counts its own
// per level and takes their places with one add per level (an add per cell
// would have thousands of adds on one address wait for each other).  All of
// the block's threads call this, level < 0 for no cell.
__device__ __forceinline__ void list_upper(int level, int64_t k, const BigList& big) {
    __shared__ uint32_t s_n[kLevels], s_at[kLevels];
    const int t = threadIdx.x;
    if (t < kLevels) s_n[t] = 0u;
    __syncthreads();
    uint32_t at = 0;
    if (level >= 0) at = atomicAdd(&s_n[level], 1u);
    __syncthreads();
    if (t < kLevels && s_n[t]) s_at[t] = atomicAdd(big.count + t * BigList::kStride, s_n[t]);
    __syncthreads();
    if (level >= 0 && s_at[level] + at < big.cap) big.cell[(size_t)level * big.cap + s_at[level] + at] = (uint32_t)k;
    __syncthreads();
}

constexpr int kLinkThreads = 1024;

__global__ void __launch_bounds__(kLinkThreads) k_topo_link(Cell* __restrict__ cells,
                                                            const DevParams* __restrict__ prm, int64_t cmax,
                                                            BigList big) {
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    for (int64_t k0 = blockIdx.x * (int64_t)kLinkThreads; k0 < C; k0 += (int64_t)gridDim.x * kLinkThreads) {
        const int64_t k = k0 + threadIdx.x;
        int level = -1;
        if (k < C) {
            const Cell c = cells[k];
            if (c.leaf_nch >= 0) {
                link_children(cells, k, c, C, [](int64_t, const Cell&) {});
                if (c.skip - k > big.sub) level = c.level;
            }
        }
        list_upper(level, k, big);
    }
}

// ---- topology, level order and walk groups of mid-size trees in five launches
// (k_topo_count and the four below): the scans and the level sort are folded
// into the kernels that use them.  Every block adds up the earlier tiles'
// totals itself, which beats the scans' launches while there are few tiles
// (fused_tree).  10,000 bodies: ten launches of 51 us in all before, 30 us
// so; 50,000: 66 and 32; 1M: 86 and 53.

constexpr int kTileThreads = 1024;               // bodies or cells per tile, a thread each

// Sum of v over the block's threads before this one, and over all of them.
__device__ __forceinline__ uint32_t tile_exscan(uint32_t v, uint32_t* s_w, uint32_t& total) {
    const int lane = wave_lane(), w = threadIdx.x / kWave;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, kWave);
        if (lane >= o) x += y;
    }
    if (lane == kWave - 1) s_w[w] = x;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < kTileThreads / kWave; ++k) {
        const uint32_t y = s_w[k];
        if (k < w) before += y;
        all += y;
    }
    __syncthreads();
    total = all;
    return before + x - v;
}

// Cells of the bodies, from the counts per body (nper) and per kTopoTile
// bodies (tile_tot).
template <int D>
__global__ void __launch_bounds__(kTileThreads) k_tree_emit(const uint64_t* __restrict__ keys, int64_t n,
                                                            const uint32_t* __restrict__ range,
                                                            const uint32_t* __restrict__ nper,
                                                            const uint32_t* __restrict__ tile_tot,
                                                            uint32_t* __restrict__ cstart, Cell* __restrict__ cells,
                                                            int64_t cmax, DevParams* prm, BigList big) {
    __shared__ uint32_t s_w[kTileThreads / kWave];
    const int t = threadIdx.x;
    if (blockIdx.x == 0 && t < kLevels) big.count[t * BigList::kStride] = 0u;
    const int64_t i = blockIdx.x * (int64_t)kTileThreads + t;
    const uint32_t own = i < n ? nper[i] : 0u;
    const int64_t tiles = blockIdx.x * (int64_t)(kTileThreads / kTopoTile);   // before this block
    uint32_t part = 0, pre, total;
    for (int64_t q = t; q < tiles; q += kTileThreads) part += tile_tot[q];
    tile_exscan(part, s_w, pre);
    const uint32_t at = pre + tile_exscan(own, s_w, total);
    if (i < n) {
        cstart[i] = at;
        emit_cells<D>(i, range[i], at, keys[i], cells, cmax);
        if (i == n - 1) {
            cstart[n] = at + own;
            store_ncells(at + own, cmax, prm);
        }
    }
}

// The cells' ends, and the tile's cells per level (hist[tile][kLevels]).  Also
// clears the tile's group count for k_tree_link.
template <int D>
__global__ void __launch_bounds__(kTileThreads) k_tree_ends(const uint64_t* __restrict__ keys, int64_t n,
                                                            const uint32_t* __restrict__ cstart,
                                                            Cell* __restrict__ cells,
                                                            const DevParams* __restrict__ prm, int64_t cmax,
                                                            uint32_t* __restrict__ hist,
                                                            uint32_t* __restrict__ gtile) {
    __shared__ uint32_t s_n[kLevels];
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    const int t = threadIdx.x;
    const int64_t k = blockIdx.x * (int64_t)kTileThreads + t;
    if (k - t >= C) return;
    if (t < kLevels) s_n[t] = 0u;
    __syncthreads();
    if (k < C) {
        const Cell c = cells[k];
        atomicAdd(&s_n[c.level], 1u);
        topo_end<D>(keys, n, cstart, c, &cells[k]);
    }
    __syncthreads();
    if (t < kLevels) hist[(int64_t)blockIdx.x * kLevels + t] = s_n[t];
    if (t == 0) gtile[blockIdx.x] = 0u;
}

__device__ __forceinline__ bool small_cell(const Cell& c) { return c.count <= kCluster || c.leaf_nch < 0; }
__device__ __forceinline__ uint32_t groups_of(const Cell& c) { return (uint32_t)((c.count + kGroup - 1) / kGroup); }

// Parents and child counts, the upper cells' lists, the level order (a stable
// pass by level: the places of a tile's cells follow from the counts of all
// tiles and their ranks within the tile), and the walk groups each cell is cut
// into (gper, and per tile gtile): those of a cluster cell, which its parent
// tells.
__global__ void __launch_bounds__(kTileThreads) k_tree_link(Cell* __restrict__ cells,
                                                            const DevParams* __restrict__ prm, int64_t cmax,
                                                            BigList big, const uint32_t* __restrict__ hist,
                                                            int last_level, uint32_t* __restrict__ bfs2pre,
                                                            uint32_t* __restrict__ pre2bfs,
                                                            uint32_t* __restrict__ lvl_off,
                                                            uint32_t* __restrict__ gper, uint32_t* __restrict__ gtile) {
    constexpr int kRows = kTileThreads / kLevels, kWaves = kTileThreads / kWave;
    __shared__ uint32_t s_pre[kRows][kLevels], s_tot[kRows][kLevels];
    __shared__ uint32_t s_wc[kWaves][kLevels];
    __shared__ uint32_t s_base[kLevels];
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    const int t = threadIdx.x, lane = wave_lane(), w = t / kWave;
    const int64_t tile = blockIdx.x, k = tile * kTileThreads + t;
    if (k - t >= C) return;
    const Cell c = cells[k < C ? k : C - 1];
    // cells per level in the earlier tiles and in all, 32 tiles side by side
    const int tiles = (int)((C + kTileThreads - 1) / kTileThreads);
    {
        const int l = t % kLevels, row = t / kLevels;
        uint32_t pre = 0, tot = 0;
#pragma unroll 8
        for (int q = row; q < tiles; q += kRows) {
            const uint32_t v = hist[(int64_t)q * kLevels + l];
            tot += v;
            if (q < tile) pre += v;
        }
        s_pre[row][l] = pre;
        s_tot[row][l] = tot;
    }
    if (t < kWaves * kLevels) (&s_wc[0][0])[t] = 0u;
    __syncthreads();
    // rank among the wave's cells of the same level, and the wave's counts
    uint64_t peers = __ballot(k < C);
#pragma unroll
    for (int b = 0; b < 5; ++b) {
        const bool bit = (c.level >> b) & 1;
        const uint64_t bb = __ballot(bit);
        peers &= bit ? bb : ~bb;
    }
    const uint32_t rank = (uint32_t)__popcll(peers & (lane == 0 ? 0ull : ~0ull >> (kWave - lane)));
    if (k < C && rank == 0) s_wc[w][c.level] = (uint32_t)__popcll(peers);
    if (t < kLevels) {
        uint32_t pre = 0, tot = 0;
        for (int r = 0; r < kRows; ++r) {
            pre += s_pre[r][t];
            tot += s_tot[r][t];
        }
        // where the level starts: an exclusive scan over the 32 lanes
        uint32_t x = tot;
#pragma unroll
        for (int o = 1; o < kLevels; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, kWave);
            if (t >= o) x += y;
        }
        s_base[t] = x - tot + pre;
        if (tile == 0) {
            if (t <= last_level + 1) lvl_off[t] = x - tot;
            if (t == kLevels - 1 && last_level == kLevels - 1) lvl_off[kLevels] = x;
        }
    }
    __syncthreads();
    int upper = -1;
    if (k < C) {
        uint32_t p = s_base[c.level] + rank;
        for (int q = 0; q < w; ++q) p += s_wc[q][c.level];
        bfs2pre[p] = (uint32_t)k;
        pre2bfs[k] = p;
        if (k == 0) {
            const uint32_t g = small_cell(c) ? groups_of(c) : 0u;
            gper[0] = g;
            if (g) atomicAdd(&gtile[0], g);
        }
        if (c.leaf_nch >= 0) {
            const bool big_parent = !small_cell(c);
            link_children(cells, k, c, C, [&](int64_t ch, const Cell& cc) {
                const uint32_t g = big_parent && small_cell(cc) ? groups_of(cc) : 0u;
                gper[ch] = g;
                if (g) atomicAdd(&gtile[ch / kTileThreads], g);
            });
            if (c.skip - k > big.sub) upper = c.level;
        }
    }
    list_upper(upper, k, big);
}

// The walk groups, from the counts per cell and per tile.
__global__ void __launch_bounds__(kTileThreads) k_tree_groups(const Cell* __restrict__ cells,
                                                              const uint32_t* __restrict__ gper,
                                                              const uint32_t* __restrict__ gtile, DevParams* prm,
                                                              int64_t cmax, int32_t* __restrict__ gbeg,
                                                              int32_t* __restrict__ gcnt, int64_t gmax) {
    __shared__ uint32_t s_w[kTileThreads / kWave];
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    const int t = threadIdx.x;
    const int64_t tile = blockIdx.x, k = tile * kTileThreads + t;
    if (k - t >= C) return;
    const uint32_t own = k < C ? gper[k] : 0u;
    uint32_t part = 0, pre, total;
    for (int64_t q = t; q < tile; q += kTileThreads) part += gtile[q];
    tile_exscan(part, s_w, pre);
    const uint32_t g0 = pre + tile_exscan(own, s_w, total);
    if (own) {
        const Cell c = cells[k];
        for (uint32_t g = g0; g < g0 + own && (int64_t)g < gmax; ++g) {
            const int32_t o = (int32_t)(g - g0) * kGroup;
            gbeg[g] = c.begin + o;
            gcnt[g] = min(kGroup, c.count - o);
        }
    }
    if (k == C - 1) {
        const uint32_t G = g0 + own;
        prm->ngroups = (int64_t)G > gmax ? (uint32_t)gmax : G;
        if ((int64_t)G > gmax) atomicOr(&prm->status, kFlagOverflow);
    }
}

// ------------------------------------------------------------- moments ----

// A leaf's moments by one lane, bodies in order: bound by the latency of its
// reads, four bodies at a time.  The barrier keeps all four of the quadrupole's
// ahead of its arithmetic; to save registers the compiler waited for them in two
// halves (a leaf of 250,000 coincident bodies 58.7 -> 48.7 ms, 4M bodies whose
// cluster ends in leaves at the deepest level 1.13 -> 0.92 ms for the moments,
// 16.7M clustered bodies 742 -> 721 us, 1M in leaves of 64 63 -> 59).
template <int D>
__device__ void leaf_moments(const Cell& c, const Body* __restrict__ bodies, Moments& mo) {
    double M = 0.0, S0 = 0.0, S1 = 0.0, S2 = 0.0;
#pragma unroll 4
    for (int32_t j = c.begin; j < c.begin + c.count; ++j) {
        const Body b = bodies[j];
        M = M + b.m;
        S0 = S0 + b.m * b.x;
        S1 = S1 + b.m * b.y;
        if (D == 3) S2 = S2 + b.m * b.z;
    }
    mo.M = M;
    mo.S[0] = S0; mo.S[1] = S1; mo.S[2] = S2;
    mo.com[0] = S0 / M; mo.com[1] = S1 / M; mo.com[2] = D == 3 ? S2 / M : 0.0;
    double Q[6] = {0, 0, 0, 0, 0, 0};
    if (D == 3) {
        auto add = [&](const Body& b) {
            const double d0 = b.x - mo.com[0], d1 = b.y - mo.com[1], d2 = b.z - mo.com[2];
            const double r2 = (d0 * d0 + d1 * d1) + d2 * d2;
            Q[0] = Q[0] + b.m * ((3.0 * d0) * d0 - r2);
            Q[1] = Q[1] + b.m * ((3.0 * d1) * d1 - r2);
            Q[2] = Q[2] + b.m * ((3.0 * d2) * d2 - r2);
            Q[3] = Q[3] + b.m * ((3.0 * d0) * d1);
            Q[4] = Q[4] + b.m * ((3.0 * d0) * d2);
            Q[5] = Q[5] + b.m * ((3.0 * d1) * d2);
        };
        const int32_t end = c.begin + c.count;
        int32_t j = c.begin;
        for (; j + 4 <= end; j += 4) {
            Body b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) b[u] = bodies[j + u];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 4; ++u) add(b[u]);
        }
        for (; j < end; ++j) add(bodies[j]);
    }
    for (int q = 0; q < 6; ++q) mo.Q[q] = Q[q];
    mo.pad = 0.0;
}

constexpr int kMomDoubles = 13;                  // M, S, com, Q

// An internal cell's moments from its children's in LDS (kMomDoubles each), by
// eight lanes: lane q sums M (q = 0) or one component of S (q = 1, 2, 3) into
// `sum` and one component of Q (q < 6) into `quad`; all lanes get com.  place(i)
// is where child i's moments are, or -1.  Children are added in digit order; a
// lane reads all of them before it adds (the adds are selected, not branched
// around).  One lane per cell instead waits on some 500 dependent FP64
// operations: 2.2 us a level.
template <int D, typename P>
__device__ __forceinline__ void sum_children(const double (*sm)[kMomDoubles], P&& place, int q, double& sum,
                                             double (&com)[3], double& quad) {
    constexpr int N = 1 << D;
    const int base = (threadIdx.x & (kWave - 1)) - q;
    int at[N];
#pragma unroll
    for (int i = 0; i < N; ++i) at[i] = place(i);
    double x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = sm[max(at[i], 0)][q < 4 ? q : 0];
    double v = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i) v = at[i] >= 0 ? v + x[i] : v;
    sum = v;
    const double c = v / __shfl(v, base, kWave);
    com[0] = __shfl(c, base + 1, kWave);
    com[1] = __shfl(c, base + 2, kWave);
    com[2] = D == 3 ? __shfl(c, base + 3, kWave) : 0.0;
    quad = 0.0;
    if (D == 3) {
        // component q: xx, yy, zz, xy, xz, yz
        const int qa = q < 3 ? q : q == 5 ? 1 : 0, qb = q < 3 ? q : q == 3 ? 1 : 2;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double* k = sm[max(at[i], 0)];
            const double s0 = k[4] - com[0];
            const double s1 = k[5] - com[1];
            const double s2 = k[6] - com[2];
            const double r2 = (s0 * s0 + s1 * s1) + s2 * s2;
            const double sa = qa == 0 ? s0 : qa == 1 ? s1 : s2, sb = qb == 0 ? s0 : qb == 1 ? s1 : s2;
            const double term = k[7 + min(q, 5)] + k[0] * ((3.0 * sa) * sb - (q < 3 ? r2 : 0.0));
            quad = at[i] >= 0 ? quad + term : quad;
        }
    }
}

// The walk record of cell k, in level order.
__device__ __forceinline__ void store_walk(WalkCell* walk, const uint32_t* __restrict__ pre2bfs, int64_t k,
                                           int32_t leaf_nch, int32_t begin, int32_t count, const Moments& mo) {
    WalkCell w;
    w.cx = mo.com[0];
    w.cy = mo.com[1];
    w.cz = mo.com[2];
    w.rcrit2 = INFINITY;
    w.m = (float)mo.M;
    if (leaf_nch < 0) {
        w.a = begin;
        w.b = (count & 0x7fffffff) | (int32_t)0x80000000u;
    } else {
        w.a = (int32_t)pre2bfs[k + 1];           // first child, pre-order k + 1
        w.b = leaf_nch;
    }
    w.pad = 0;
    walk[pre2bfs[k]] = w;
}

// The moments in two launches.  The maximal subtrees of at most SUB cells
// are done in LDS: they are runs of cells in pre-order, so a block takes those
// that start in its SUB cells (at most twice as many cells, a lane
// each), sums the leaves over their bodies and follows the levels from the
// deepest up, with nothing to wait for outside the block.  The few cells above
// them (about C / 75 or C / 150) are done level by level by one block.  A launch per
// level instead, each cell waiting on its children's moments in memory, took
// 5 to 12 us a level, ten launches at 1M bodies.  Children are summed in digit
// order, so the result does not depend on scheduling.

template <int D, int SUB>
__global__ void __launch_bounds__(2 * SUB) __attribute__((amdgpu_waves_per_eu(4, 8))) k_moments_low(const Cell* __restrict__ cells,
                                                             const Body* __restrict__ bodies,
                                                             const uint32_t* __restrict__ pre2bfs,
                                                             const DevParams* __restrict__ prm, int64_t cmax,
                                                             Moments* __restrict__ mom, WalkCell* __restrict__ walk) {
    constexpr int N = 1 << D;
    __shared__ double s_mom[(2 * SUB)][kMomDoubles];
    __shared__ __align__(16) int16_t s_child[(2 * SUB)][N];   // a cell's children by digit, -1 where none
    __shared__ uint16_t s_list[(2 * SUB)];                    // internal cells by level
    __shared__ uint32_t s_lvl[kLevels + 1], s_next[kLevels];
    __shared__ int s_first[2];
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    const int t = threadIdx.x;
    for (int64_t b0 = blockIdx.x * (int64_t)SUB; b0 < C; b0 += (int64_t)gridDim.x * SUB) {
        // the block's run: from the first cell of its SUB that starts a
        // subtree or lies above them, to the next block's
        if (t < 2) s_first[t] = SUB;
        if (t < kLevels) s_next[t] = 0u;
#pragma unroll
        for (int i = 0; i < N; ++i) s_child[t][i] = -1;
        __syncthreads();
        {
            const int64_t k = b0 + t;
            if (k < C) {
                const Cell c = cells[k];
                const bool starts = c.skip - k > SUB || c.parent < 0 ||
                                    cells[c.parent].skip - c.parent > SUB;
                if (starts) atomicMin(&s_first[t / SUB], t % SUB);
            }
        }
        __syncthreads();
        const int64_t k0 = b0 + s_first[0];
        int64_t k1 = b0 + SUB + s_first[1];
        if (k1 > C) k1 = C;
        const int n = s_first[0] < SUB ? (int)(k1 - k0) : 0;
        const int64_t k = k0 + t;
        Cell c;
        Moments mo;
        bool internal = false, leaf = false;
        uint32_t slot = 0;
        if (t < n) {
            c = cells[k];
            leaf = c.leaf_nch < 0;
            internal = !leaf && c.skip - k <= SUB;
            if (c.parent >= k0) s_child[c.parent - k0][c.prefix & (N - 1)] = (int16_t)t;
            if (internal) slot = atomicAdd(&s_next[c.level], 1u);
            if (leaf) {
                leaf_moments<D>(c, bodies, mo);
                double* o = s_mom[t];
                o[0] = mo.M;
                for (int a = 0; a < 3; ++a) {
                    o[1 + a] = mo.S[a];
                    o[4 + a] = mo.com[a];
                }
                for (int a = 0; a < 6; ++a) o[7 + a] = mo.Q[a];
            }
        }
        __syncthreads();
        if (t < kLevels) {
            uint32_t at = 0;
            for (int l = 0; l < t; ++l) at += s_next[l];
            s_lvl[t] = at;
            if (t == kLevels - 1) s_lvl[kLevels] = at + s_next[t];
        }
        __syncthreads();
        if (internal) s_list[s_lvl[c.level] + slot] = (uint16_t)t;
        __syncthreads();
        const int q = t & 7;
        for (int l = kLevels - 1; l >= 0; --l) {
            if (s_lvl[l] == s_lvl[l + 1]) continue;
            for (uint32_t e = s_lvl[l] + t / 8; e < s_lvl[l + 1]; e += (2 * SUB) / 8) {
                const int j = s_list[e];
                double sum, com[3], quad;
                sum_children<D>(s_mom, [&](int i) { return (int)s_child[j][i]; }, q, sum, com, quad);
                if (q < 4) s_mom[j][q] = sum;
                if (q < 3) s_mom[j][4 + q] = q == 0 ? com[0] : q == 1 ? com[1] : com[2];
                if (q < 6) s_mom[j][7 + q] = quad;
            }
            __syncthreads();
        }
        if (leaf || internal) {
            if (internal) {
                const double* o = s_mom[t];
                mo.M = o[0];
                for (int a = 0; a < 3; ++a) {
                    mo.S[a] = o[1 + a];
                    mo.com[a] = o[4 + a];
                }
                for (int a = 0; a < 6; ++a) mo.Q[a] = o[7 + a];
                mo.pad = 0.0;
            }
            mom[k] = mo;
            store_walk(walk, pre2bfs, k, c.leaf_nch, c.begin, c.count, mo);
        }
        __syncthreads();                         // s_first and the rest are rewritten
    }
}

// The cells above, from their lists: levels hi down to lo in one block (a
// barrier separates the levels, and the block's waves share one CU's L1), or
// one level in any number of blocks.  A round takes up to kUpperCells cells of
// a level: their children's moments are
// brought to LDS eight lanes a child (one line per child; a lane per cell
// reading its children itself spends 64 lines per load and took 5 us a level
// of 170 cells), then eight lanes add up a cell.  What leads to the children
// (the cell, its first child's place in level order, the children there) is
// looked up for the first kUpperTable cells before the first round, so a
// level waits on its children's moments only.
constexpr int kUpperThreads = 1024;
constexpr int kUpperCells = kUpperThreads / 8;
constexpr int kUpperTable = 640;
// Cell slots from which the levels get launches of their own (the whole pass in
// us, one block / launches: 1M bodies 87 / 105, 1.8M 142 / 137, 2M 156 / 135, 3M 228
// / 169, 16.7M clustered 1,577 / 723).
constexpr int64_t kUpperSplit = (int64_t)1 << 22;

// Stages of a large tree: of kUpperWide<D> consecutive levels each has a launch
// of many blocks (stages 1 ..); the levels below these (stage 0) and above (the last
// stage) are one block's.  Stage 0 chooses them by the counts: those with the
// most cells beyond a round's, and the deepest of several such choices, as a level
// of one round is cheaper in the last stage.  Against levels 12 to 4 (2D 16 to 6)
// for every tree, us for the moments: 2D, 4M bodies in a compact cluster of a wide
// square 276 / 183, 10M 646 / 323, 3D 10M 3,350 / 2,726, 16.7M clustered 728 / 715;
// where the levels stay, 2D 3M 138 / 141, 3D 3M 205 / 205.  Chosen by each launch
// for itself: 158 and 215.  Stage -1: all levels, in one block.
template <int D>
constexpr int kUpperWide = D == 3 ? 9 : 11;

template <int D>
__global__ void __launch_bounds__(kUpperThreads) k_moments_upper(const Cell* __restrict__ cells,
                                                                 const uint32_t* __restrict__ pre2bfs,
                                                                 const uint32_t* __restrict__ bfs2pre, BigList big,
                                                                 int stage, Moments* mom,
                                                                 WalkCell* __restrict__ walk) {
    constexpr int N = 1 << D, L = D == 3 ? 21 : 31, W = kUpperWide<D>;
    static_assert(L < kLevels && kLevels <= 32, "a level's number has five bits");
    __shared__ double s_mom[kUpperCells * N][kMomDoubles];
    __shared__ uint32_t s_ch[kUpperTable][N];
    __shared__ uint32_t s_k[kUpperTable], s_first[kUpperTable], s_at[kUpperTable];
    __shared__ int32_t s_nch[kUpperTable];
    __shared__ uint32_t s_n[kLevels], s_wide;
    const uint32_t t = threadIdx.x;
    int hi = L, lo = 0;
    if (stage > 0) {
        const int wide = (int)big.count[BigList::kWide];     // the deepest of them
        hi = stage <= W ? wide - stage + 1 : wide - W;
        if (stage <= W) lo = hi;
        if (hi < 0) return;
    }
    if (t < kLevels) s_n[t] = min(big.count[t * BigList::kStride], big.cap);
    if (t == 0) s_wide = 0u;
    __syncthreads();
    if (stage == 0) {
        // the cells beyond a round of the W levels up from t (fewer than 2^27), and t
        if (t <= L) {
            uint32_t n = 0;
            for (int l = max(0, (int)t - W + 1); l <= (int)t; ++l) n += s_n[l] - min(s_n[l], (uint32_t)kUpperCells);
            atomicMax(&s_wide, n << 5 | t);
        }
        __syncthreads();
        lo = (int)(s_wide & 31u) + 1;
        if (t == 0) big.count[BigList::kWide] = (uint32_t)(lo - 1);
        if (hi < lo) return;
    }
    // cell i of level l into the table
    auto look_up = [&](uint32_t slot, int l, uint32_t i) {
        const uint32_t k = big.cell[(size_t)l * big.cap + i];
        const int32_t nch = cells[k].leaf_nch;
        const uint32_t first = pre2bfs[k + 1];
        s_at[slot] = pre2bfs[k];
        s_k[slot] = k;
        s_first[slot] = first;
        s_nch[slot] = nch;
#pragma unroll
        for (int c = 0; c < N; ++c) s_ch[slot][c] = bfs2pre[first + (c < nch ? c : 0)];
    };
    // one block: its first cells, in the order of the rounds
    const uint32_t table = gridDim.x == 1 ? kUpperTable : 0u;
    if (t < table) {
        int l = hi;
        uint32_t i = t;
        while (l >= lo && i >= s_n[l]) i -= s_n[l--];
        if (l >= lo) look_up(t, l, i);
    }
    __syncthreads();
    uint32_t done = 0;                               // cells of the earlier rounds
    for (int l = hi; l >= lo; --l) {
        for (uint32_t i0 = blockIdx.x * kUpperCells; i0 < s_n[l]; i0 += gridDim.x * kUpperCells) {
            const uint32_t m = min((uint32_t)kUpperCells, s_n[l] - i0);
            uint32_t at = done;
            if (at + m > table) {                    // not in the table: over its first, used places
                at = 0;
                if (t < m) look_up(t, l, i0 + t);
                __syncthreads();
            }
            // the children's records, 16 bytes a lane (the last eighth of the
            // eight lanes has none)
            const double2* rec = reinterpret_cast<const double2*>(mom);
#pragma unroll 8
            for (uint32_t e = t / 8; e < m * N; e += kUpperThreads / 8) {
                const uint32_t part = t & 7;
                if (part < 7) {
                    const double2 v = rec[(size_t)s_ch[at + e / N][e % N] * 7 + part];
                    s_mom[e][2 * part] = v.x;
                    if (part < 6) s_mom[e][2 * part + 1] = v.y;
                }
            }
            __syncthreads();
            const uint32_t j = t / 8;
            const int q = (int)(t & 7);
            if (j < m) {
                const int nch = s_nch[at + j];
                double sum, com[3], quad;
                sum_children<D>(s_mom, [&](int i) { return i < nch ? (int)j * N + i : -1; }, q, sum, com, quad);
                double* o = reinterpret_cast<double*>(&mom[s_k[at + j]]);
                if (q < 4) o[q] = sum;
                if (q < 3) o[4 + q] = q == 0 ? com[0] : q == 1 ? com[1] : com[2];
                if (q < 7) o[7 + q] = q < 6 ? quad : 0.0;      // the last is the padding
                if (q == 0) {
                    WalkCell w;
                    w.cx = com[0];
                    w.cy = com[1];
                    w.cz = com[2];
                    w.rcrit2 = INFINITY;
                    w.m = (float)sum;
                    w.a = (int32_t)s_first[at + j];
                    w.b = nch;
                    w.pad = 0;
                    walk[s_at[at + j]] = w;
                }
            }
            done += m;
            __threadfence_block();
            __syncthreads();
        }
    }
}

// ----------------------------------------------------------------- mac ----

template <int D>
__global__ void __launch_bounds__(256) k_mac(const Cell* __restrict__ cells, const Moments* __restrict__ mom,
                                             double theta, const uint32_t* __restrict__ pre2bfs,
                                             WalkCell* __restrict__ walk, double* __restrict__ rc_out,
                                             const DevParams* __restrict__ prm, int64_t cmax) {
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    const double size = prm->size;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < C;
         k += (int64_t)gridDim.x * blockDim.x) {
        if (theta == 0.0) {
            if (rc_out) rc_out[pre2bfs[k]] = INFINITY;
            else walk[pre2bfs[k]].rcrit2 = INFINITY;
            continue;
        }
        const Cell c = cells[k];
        const int l = c.level;
        const double s = ldexp(size, -l);
        uint64_t org[3] = {0, 0, 0};
        for (int j = 1; j <= l; ++j) {
            const unsigned d = (unsigned)((c.prefix >> (D * (l - j))) & ((1u << D) - 1u));
#pragma unroll
            for (int a = 0; a < D; ++a) org[a] = (org[a] << 1) | ((d >> (D - 1 - a)) & 1u);
        }
        double dd[3];
#pragma unroll
        for (int a = 0; a < D; ++a) {
            const double centre = prm->lo[a] + ((double)org[a] + 0.5) * s;
            dd[a] = mom[k].com[a] - centre;
        }
        double d2 = dd[0] * dd[0] + dd[1] * dd[1];
        if (D == 3) d2 = d2 + dd[2] * dd[2];
        const double r = s / theta + sqrt(d2);
        if (rc_out) rc_out[pre2bfs[k]] = r * r;
        else walk[pre2bfs[k]].rcrit2 = r * r;
    }
}

// ---------------------------------------------------------- walk groups ----
// A walk group is a run of at most 64 consecutive bodies in key order that
// never straddles a cluster cell (a maximal cell holding at most kCluster
// bodies, or a leaf deeper than that): the group's bounding box then stays
// inside one compact region even where the Morton curve jumps across empty
// space.  Cluster cells are found in pre-order, so groups come out in body
// order.

__global__ void __launch_bounds__(256) k_group_count(const Cell* __restrict__ cells, const DevParams* __restrict__ prm,
                                                     int64_t cmax, uint32_t* __restrict__ gper) {
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < C; k += (int64_t)gridDim.x * blockDim.x) {
        const Cell c = cells[k];
        const bool cluster = small_cell(c) && (k == 0 || !small_cell(cells[c.parent]));
        gper[k] = cluster ? (uint32_t)((c.count + kGroup - 1) / kGroup) : 0u;
    }
}

__global__ void __launch_bounds__(256) k_group_emit(const Cell* __restrict__ cells, const uint32_t* __restrict__ goff,
                                                    DevParams* prm, int64_t cmax, int32_t* __restrict__ gbeg,
                                                    int32_t* __restrict__ gcnt, int64_t gmax) {
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const uint32_t G = goff[cmax];
        prm->ngroups = (int64_t)G > gmax ? (uint32_t)gmax : G;
        if ((int64_t)G > gmax) atomicOr(&prm->status, kFlagOverflow);
    }
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < C;
         k += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t g0 = goff[k], g1 = goff[k + 1];
        if (g1 == g0) continue;
        const Cell c = cells[k];
        for (uint32_t g = g0; g < g1 && (int64_t)g < gmax; ++g) {
            const int32_t o = (int32_t)(g - g0) * kGroup;
            gbeg[g] = c.begin + o;
            gcnt[g] = min(kGroup, c.count - o);
        }
    }
}

// -------------------------------------------------------------- export ----

__global__ void __launch_bounds__(256) k_export(const Cell* __restrict__ cells, const Moments* __restrict__ mom,
                                                int dim, const DevParams* __restrict__ prm, int64_t cmax,
                                                int32_t* level, uint64_t* prefix, int32_t* begin,
                                                int32_t* count, int32_t* parent, int32_t* skip,
                                                int32_t* nch, int32_t* leaf, double* M, double* com,
                                                double* Q) {
    int64_t C = prm->ncells;
    if (C > cmax) C = cmax;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < C;
         k += (int64_t)gridDim.x * blockDim.x) {
        const Cell c = cells[k];
        if (level) level[k] = c.level;
        if (prefix) prefix[k] = c.prefix;
        if (begin) begin[k] = c.begin;
        if (count) count[k] = c.count;
        if (parent) parent[k] = c.parent;
        if (skip) skip[k] = c.skip;
        if (nch) nch[k] = c.leaf_nch < 0 ? 0 : c.leaf_nch;
        if (leaf) leaf[k] = c.leaf_nch < 0 ? 1 : 0;
        if (M) M[k] = mom[k].M;
        if (com)
            for (int a = 0; a < dim; ++a) com[k * dim + a] = mom[k].com[a];
        if (Q)
            for (int q = 0; q < 6; ++q) Q[k * 6 + q] = mom[k].Q[q];
    }
}

}  // namespace

// ------------------------------------------------------------ launchers ----

int bbox_parts(int64_t n) { return (int)grid_for(n, 1024); }

template <typename T, int D>
static void bbox_part(T* pos, const T* mass, int64_t n, double* part, void* packed, const KickDrift* kick,
                      hipStream_t s) {
    const dim3 nb((unsigned)bbox_parts(n));
    auto* rec = (typename Packed<T>::type*)packed;
    if (kick)
        hipLaunchKernelGGL((k_bbox_part<T, D, true>), nb, dim3(256), 0, s, pos, mass, n, part, rec, (T*)kick->vel,
                           kick->acc, (T)(0.5 * kick->dt), (T)kick->dt);
    else
        hipLaunchKernelGGL((k_bbox_part<T, D, false>), nb, dim3(256), 0, s, pos, mass, n, part, rec, (T*)nullptr,
                           (const float*)nullptr, T(0), T(0));
}

hipError_t launch_bbox(void* pos, const void* mass, int64_t n, int dim, int f64, double* part, void* packed,
                       const KickDrift* kick, DevParams* prm, hipStream_t s) {
    if (f64) {
        if (dim == 3) bbox_part<double, 3>((double*)pos, (const double*)mass, n, part, packed, kick, s);
        else bbox_part<double, 2>((double*)pos, (const double*)mass, n, part, packed, kick, s);
    } else {
        if (dim == 3) bbox_part<float, 3>((float*)pos, (const float*)mass, n, part, packed, kick, s);
        else bbox_part<float, 2>((float*)pos, (const float*)mass, n, part, packed, kick, s);
    }
    if (packed) hipLaunchKernelGGL(k_bbox_final, dim3(1), dim3(256), 0, s, part, bbox_parts(n), dim, prm);
    return hipGetLastError();
}

hipError_t launch_keys(const void* pos, int64_t n, int dim, int f64, const DevParams* prm,
                       uint64_t* keys, uint32_t* idx, hipStream_t s) {
    const unsigned nb = grid_for(n);
    if (f64) {
        if (dim == 3) hipLaunchKernelGGL((k_keys<double, 3>), dim3(nb), dim3(256), 0, s, (const double*)pos, n, prm, keys, idx);
        else hipLaunchKernelGGL((k_keys<double, 2>), dim3(nb), dim3(256), 0, s, (const double*)pos, n, prm, keys, idx);
    } else {
        if (dim == 3) hipLaunchKernelGGL((k_keys<float, 3>), dim3(nb), dim3(256), 0, s, (const float*)pos, n, prm, keys, idx);
        else hipLaunchKernelGGL((k_keys<float, 2>), dim3(nb), dim3(256), 0, s, (const float*)pos, n, prm, keys, idx);
    }
    return hipGetLastError();
}

// One pass of the reduce-then-scan sort (2 or 3 launches).
template <int PER, bool STAGE, class In, class Out>
static void sort_pass(In in, Out out, int64_t n, const uint32_t* n_live, int shift, uint32_t* hist,
                      uint32_t* digit_tot, hipStream_t s) {
    const int64_t tiles = (n + 256 * PER - 1) / (256 * PER);
    hipLaunchKernelGGL((k_sort_hist<PER, In>), dim3((unsigned)tiles), dim3(256), 0, s, in, n, n_live, shift, hist,
                       tiles);
    if (tiles <= kSortScanInScatter) {
        hipLaunchKernelGGL((k_sort_scatter<PER, true, STAGE, In, Out>), dim3((unsigned)tiles), dim3(256), 0, s, in, out, n,
                           n_live, shift, (const uint32_t*)hist, digit_tot, tiles);
        return;
    }
    hipLaunchKernelGGL(k_sort_scan<PER>, dim3(256), dim3(256), 0, s, hist, tiles, n, n_live, digit_tot);
    hipLaunchKernelGGL((k_sort_scatter<PER, false, STAGE, In, Out>), dim3((unsigned)tiles), dim3(256), 0, s, in, out, n,
                       n_live, shift, (const uint32_t*)hist, digit_tot, tiles);
}

template <int PER, bool STAGE>
static void sort_passes(uint64_t* keys_a, uint32_t* idx_a, uint64_t* keys_b, uint32_t* idx_b, int64_t n,
                        const uint32_t* n_live, int passes, uint32_t* hist, uint32_t* digit_tot, hipStream_t s) {
    for (int p = 0; p < passes; ++p) {
        const bool even = (p % 2) == 0;
        const PairsIn in{even ? keys_a : keys_b, even ? idx_a : idx_b};
        const PairsOut out{even ? keys_b : keys_a, even ? idx_b : idx_a};
        sort_pass<PER, STAGE>(in, out, n, n_live, 8 * p, hist, digit_tot, s);
    }
}

hipError_t launch_sort(uint64_t* keys_a, uint32_t* idx_a, uint64_t* keys_b, uint32_t* idx_b,
                       int64_t n, int key_bits, uint32_t* hist, uint32_t* digit_tot, hipStream_t s) {
    const int passes = (key_bits + 7) / 8;    // even for 62/63-bit keys: result lands in _a
    if (n >= kSortStageMin) {
        sort_passes<kSortStagePer, true>(keys_a, idx_a, keys_b, idx_b, n, nullptr, passes, hist, digit_tot, s);
        return hipGetLastError();
    }
    switch (sort_per(n)) {
        case 16: sort_passes<16, false>(keys_a, idx_a, keys_b, idx_b, n, nullptr, passes, hist, digit_tot, s); break;
        case 8: sort_passes<8, false>(keys_a, idx_a, keys_b, idx_b, n, nullptr, passes, hist, digit_tot, s); break;
        default: sort_passes<4, false>(keys_a, idx_a, keys_b, idx_b, n, nullptr, passes, hist, digit_tot, s); break;
    }
    return hipGetLastError();
}

hipError_t launch_gather(const void* packed, const uint32_t* perm, int64_t n, int f64, Body* bodies,
                         float4* bodies32, hipStream_t s) {
    const unsigned nb = grid_for(n);
    if (f64) hipLaunchKernelGGL(k_gather<double>, dim3(nb), dim3(256), 0, s, (const double4*)packed, perm, n, bodies, (float4*)nullptr);
    else hipLaunchKernelGGL(k_gather<float>, dim3(nb), dim3(256), 0, s, (const float4*)packed, perm, n, bodies, bodies32);
    return hipGetLastError();
}

hipError_t launch_scan_u32(const uint32_t* in, int64_t n, uint32_t* out, uint32_t* part, int64_t tiles,
                           hipStream_t s) {
    scan_u32(in, n, nullptr, out, part, tiles, s);
    return hipGetLastError();
}

hipError_t launch_topology(const uint64_t* keys, int64_t n, int dim, int leaf_cap,
                           uint32_t* range, uint32_t* nper, uint32_t* cstart,
                           uint32_t* scan_part, int64_t scan_tiles, Cell* cells,
                           int64_t cmax, DevParams* prm, const BigList& big, hipStream_t s) {
    const unsigned nb = grid_for(n);
    if (dim == 3) hipLaunchKernelGGL(k_topo_count<3>, dim3(nb), dim3(256), 0, s, keys, n, leaf_cap, range, nper, (uint32_t*)nullptr);
    else hipLaunchKernelGGL(k_topo_count<2>, dim3(nb), dim3(256), 0, s, keys, n, leaf_cap, range, nper, (uint32_t*)nullptr);
    scan_u32(nper, n, nullptr, cstart, scan_part, scan_tiles, s);
    if (dim == 3) hipLaunchKernelGGL(k_topo_emit<3>, dim3(nb), dim3(256), 0, s, keys, n, (const uint32_t*)range, (const uint32_t*)cstart, cells, cmax, prm, big);
    else hipLaunchKernelGGL(k_topo_emit<2>, dim3(nb), dim3(256), 0, s, keys, n, (const uint32_t*)range, (const uint32_t*)cstart, cells, cmax, prm, big);
    const unsigned nc = grid_for(cmax);
    if (dim == 3) hipLaunchKernelGGL(k_topo_ends<3>, dim3(nc), dim3(256), 0, s, keys, n, (const uint32_t*)cstart, cells, (const DevParams*)prm, cmax);
    else hipLaunchKernelGGL(k_topo_ends<2>, dim3(nc), dim3(256), 0, s, keys, n, (const uint32_t*)cstart, cells, (const DevParams*)prm, cmax);
    hipLaunchKernelGGL(k_topo_link, dim3(grid_for(cmax / 4)), dim3(kLinkThreads), 0, s, cells, (const DevParams*)prm,
                       cmax, big);
    return hipGetLastError();
}

template <int D>
static void tree_cells(const uint64_t* keys, int64_t n, int leaf_cap, uint32_t* range, uint32_t* nper,
                       uint32_t* cstart, Cell* cells, int64_t cmax, DevParams* prm, const BigList& big,
                       const TreeScratch& a, hipStream_t s) {
    hipLaunchKernelGGL(k_topo_count<D>, dim3(grid_for(n)), dim3(256), 0, s, keys, n, leaf_cap, range, nper, a.tile_tot);
    hipLaunchKernelGGL(k_tree_emit<D>, dim3((unsigned)((n + kTileThreads - 1) / kTileThreads)), dim3(kTileThreads), 0,
                       s, keys, n, (const uint32_t*)range, (const uint32_t*)nper, (const uint32_t*)a.tile_tot, cstart,
                       cells, cmax, prm, big);
    hipLaunchKernelGGL(k_tree_ends<D>, dim3((unsigned)((cmax + kTileThreads - 1) / kTileThreads)), dim3(kTileThreads),
                       0, s, keys, n, (const uint32_t*)cstart, cells, (const DevParams*)prm, cmax, a.hist, a.gtile);
}

hipError_t launch_tree_cells(const uint64_t* keys, int64_t n, int dim, int leaf_cap, uint32_t* range, uint32_t* nper,
                             uint32_t* cstart, Cell* cells, int64_t cmax, DevParams* prm, const BigList& big,
                             const TreeScratch& a, hipStream_t s) {
    if (dim == 3) tree_cells<3>(keys, n, leaf_cap, range, nper, cstart, cells, cmax, prm, big, a, s);
    else tree_cells<2>(keys, n, leaf_cap, range, nper, cstart, cells, cmax, prm, big, a, s);
    return hipGetLastError();
}

hipError_t launch_tree_link(Cell* cells, int64_t cmax, int dim, const DevParams* prm, const BigList& big,
                            uint32_t* bfs2pre, uint32_t* pre2bfs, uint32_t* lvl_off, uint32_t* gper,
                            const TreeScratch& a, hipStream_t s) {
    hipLaunchKernelGGL(k_tree_link, dim3((unsigned)((cmax + kTileThreads - 1) / kTileThreads)), dim3(kTileThreads), 0,
                       s, cells, prm, cmax, big, (const uint32_t*)a.hist, levels_for(dim), bfs2pre, pre2bfs, lvl_off,
                       gper, a.gtile);
    return hipGetLastError();
}

hipError_t launch_tree_groups(const Cell* cells, int64_t cmax, const uint32_t* gper, int32_t* gbeg, int32_t* gcnt,
                              int64_t gmax, DevParams* prm, const TreeScratch& a, hipStream_t s) {
    hipLaunchKernelGGL(k_tree_groups, dim3((unsigned)((cmax + kTileThreads - 1) / kTileThreads)), dim3(kTileThreads), 0,
                       s, cells, gper, (const uint32_t*)a.gtile, prm, cmax, gbeg, gcnt, gmax);
    return hipGetLastError();
}

hipError_t launch_level_order(const Cell* cells, int64_t cmax, int64_t cells_est, int dim, const DevParams* prm,
                              uint32_t* bfs2pre, uint32_t* hist, uint32_t* digit_tot, uint32_t* pre2bfs,
                              uint32_t* lvl_off, hipStream_t s) {
    // one pass by level over the live cells (their count is on the device,
    // so the tile follows the host's estimate of it: the slots are several
    // times more; 1M bodies: 16 against 27 us per pass with tiles sized for
    // the slots)
    const LevelsIn in{cells};
    const LevelsOut out{bfs2pre, pre2bfs, lvl_off, levels_for(dim)};
    switch (sort_per(cells_est)) {
        case 16: sort_pass<16, false>(in, out, cmax, &prm->ncells, 0, hist, digit_tot, s); break;
        case 8: sort_pass<8, false>(in, out, cmax, &prm->ncells, 0, hist, digit_tot, s); break;
        default: sort_pass<4, false>(in, out, cmax, &prm->ncells, 0, hist, digit_tot, s); break;
    }
    return hipGetLastError();
}

hipError_t launch_groups(const Cell* cells, int64_t cmax, uint32_t* gper, uint32_t* goff, uint32_t* scan_part,
                         int64_t scan_tiles, int32_t* gbeg, int32_t* gcnt, int64_t gmax, DevParams* prm,
                         hipStream_t s) {
    const unsigned nb = grid_for(cmax);
    hipLaunchKernelGGL(k_group_count, dim3(nb), dim3(256), 0, s, cells, (const DevParams*)prm, cmax, gper);
    // over the live cells only (their count is on the device)
    const uint32_t* live = &prm->ncells;
    scan_u32(gper, cmax, live, goff, scan_part, scan_tiles, s);
    hipLaunchKernelGGL(k_group_emit, dim3(nb), dim3(256), 0, s, cells, (const uint32_t*)goff, prm, cmax, gbeg,
                       gcnt, gmax);
    return hipGetLastError();
}

template <int D>
static void moments(const Cell* cells, const Body* bodies, int64_t cmax, const uint32_t* bfs2pre,
                    const uint32_t* pre2bfs, const BigList& big, const DevParams* prm, Moments* mom, WalkCell* walk,
                    hipStream_t s) {
    const unsigned nb = (unsigned)std::min<int64_t>((cmax + big.sub - 1) / big.sub, 16384);
    if (big.sub == 128)
        hipLaunchKernelGGL((k_moments_low<D, 128>), dim3(nb), dim3(256), 0, s, cells, bodies, pre2bfs, prm, cmax, mom,
                           walk);
    else
        hipLaunchKernelGGL((k_moments_low<D, 256>), dim3(nb), dim3(512), 0, s, cells, bodies, pre2bfs, prm, cmax, mom,
                           walk);
    auto upper = [&](int stage, unsigned nb) {
        hipLaunchKernelGGL(k_moments_upper<D>, dim3(nb), dim3(kUpperThreads), 0, s, cells, pre2bfs, bfs2pre, big, stage,
                           mom, walk);
    };
    if (cmax < kUpperSplit) {
        upper(-1, 1);
        return;
    }
    constexpr int W = kUpperWide<D>;
    for (int stage = 0; stage <= W + 1; ++stage)
        upper(stage, stage == 0 || stage > W ? 1u : (unsigned)std::min<int64_t>(256, big.cap / kUpperCells + 1));
}

hipError_t launch_moments(const Cell* cells, const Body* bodies, int dim, int64_t cmax, const uint32_t* bfs2pre,
                          const uint32_t* pre2bfs, const BigList& big, const DevParams* prm, Moments* mom,
                          WalkCell* walk, hipStream_t s) {
    if (dim == 3) moments<3>(cells, bodies, cmax, bfs2pre, pre2bfs, big, prm, mom, walk, s);
    else moments<2>(cells, bodies, cmax, bfs2pre, pre2bfs, big, prm, mom, walk, s);
    return hipGetLastError();
}

hipError_t launch_mac(const Cell* cells, const Moments* mom, int dim, double theta, int64_t cmax,
                      const uint32_t* pre2bfs, WalkCell* walk, double* rc_out, const DevParams* prm,
                      hipStream_t s) {
    const unsigned nb = grid_for(cmax);
    if (dim == 3) hipLaunchKernelGGL(k_mac<3>, dim3(nb), dim3(256), 0, s, cells, mom, theta, pre2bfs, walk, rc_out, prm, cmax);
    else hipLaunchKernelGGL(k_mac<2>, dim3(nb), dim3(256), 0, s, cells, mom, theta, pre2bfs, walk, rc_out, prm, cmax);
    return hipGetLastError();
}

hipError_t launch_export(const Cell* cells, const Moments* mom, int dim, int64_t cmax,
                         const DevParams* prm, int32_t* level, uint64_t* prefix, int32_t* begin,
                         int32_t* count, int32_t* parent, int32_t* skip, int32_t* nch,
                         int32_t* leaf, double* M, double* com, double* Q, hipStream_t s) {
    hipLaunchKernelGGL(k_export, dim3(grid_for(cmax)), dim3(256), 0, s, cells, mom, dim, prm, cmax, level,
                       prefix, begin, count, parent, skip, nch, leaf, M, com, Q);
    return hipGetLastError();
}

}  // namespace tc
